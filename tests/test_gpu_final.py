"""The last kernel of a top-k step at the sizes where its split changes: workers beyond one tile of sixteen, one and
two slots of entries per worker and chunk (added up by one wavefront) and more (by all of them), more entries than a
worker's share of the LDS, grids with few and with many chunks, ties that are only partly taken.  Every output equals
the oracle's bit for bit."""
import numpy as np
import pytest
import torch

from paper_2205_05632_amd import binding as B

from parity import Pair

pytestmark = pytest.mark.gpu


def run(n, d, k, steps, draw, label):
    rng = np.random.default_rng(n * 1000 + k)
    p = Pair(n, d, rng.standard_normal(d) * 0.1, B.TOPK, k=k)
    for t in range(steps):
        p.step(draw(rng), 1e-3, label=f"{label} step {t}", with_e=t == steps - 1)
    assert all(p.exact.values()), p.exact
    p.close()


# entries per worker and chunk: k / 3 of the three chunks' 4096 (64: a slot, 128: two, 129: one more)
@pytest.mark.parametrize("n", [1, 16, 17, 33])
@pytest.mark.parametrize("per_chunk", [63, 64, 65, 127, 128, 129, 700])
def test_entries_per_chunk(n, per_chunk):
    d, k = 3 * 4096, 3 * per_chunk
    hot = np.concatenate([c * 4096 + np.arange(per_chunk) * (4096 // per_chunk) for c in range(3)])

    def draw(rng):
        g = rng.standard_normal((n, d)).astype(np.float32) * 1e-3
        g[:, hot] = (rng.standard_normal((n, hot.size)) + 8.0).astype(np.float32)
        return g
    run(n, d, k, 4, draw, f"{n} x {per_chunk}")


@pytest.mark.parametrize("n,d,k", [(3, 20001, 9000), (1, 4097, 4097), (5, 1025, 1024), (18, 8192, 5000)])
def test_more_entries_than_the_lds_share(n, d, k):
    run(n, d, k, 4, lambda rng: rng.standard_normal((n, d)).astype(np.float32), f"{n} x {d} k {k}")


# 512 chunks are the last grid of sixteen wavefronts per chunk, 513 the first of eight
@pytest.mark.parametrize("n,chunks", [(2, 512), (2, 513), (17, 513)])
def test_few_and_many_chunks(n, chunks):
    d = chunks * 4096 - 3
    crowded = np.s_[:, 40_000:60_000]

    def draw(rng):
        g = rng.standard_normal((n, d), dtype=np.float32) * np.float32(1e-2)
        g[crowded] *= np.float32(100.0)
        return g
    run(n, d, 15_000, 4, draw, f"{n} x {chunks} chunks")


@pytest.mark.parametrize("n,d,k", [(4, 30_000, 5_000), (17, 70_000, 333)])
def test_ties_partly_taken(n, d, k):
    def draw(rng):
        return (rng.integers(-3, 4, size=(n, d)) * 0.25).astype(np.float32)
    run(n, d, k, 5, draw, f"ties {n} x {d} k {k}")


# 768 chunks are the last grid of eight wavefronts per chunk, 769 the first of four; eight again from four rows and a
# hundred entries per chunk on
@pytest.mark.parametrize("n,chunks,k", [(4, 768, 15_000), (4, 769, 15_000), (4, 769, 80_000), (3, 769, 80_000)])
def test_eight_and_four_wavefronts(n, chunks, k):
    d = chunks * 4096 - 1
    crowded = np.s_[:, 1_000_001:1_100_001]

    def draw(rng):
        g = rng.standard_normal((n, d), dtype=np.float32) * np.float32(1e-2)
        g[crowded] *= np.float32(100.0)
        return g
    run(n, d, k, 3, draw, f"{n} x {chunks} chunks k {k}")


def step_us(n, chunks, k, crowded):
    d = chunks * 4096
    c = B.Compams(n, d, torch.zeros(d), compressor=B.TOPK, k=k)
    gs = [torch.randn((n, c.ld), device=c.device) for _ in range(3)]
    if crowded:
        for g in gs:
            g[:, d // 10:] *= 1e-3
    times = []
    for _ in range(8):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for t in range(10):
            c.compams_step(gs[t % 3], 1e-3)
        end.record()
        torch.cuda.synchronize()
        times.append(begin.elapsed_time(end) / 10 * 1e3)
    c.close()
    return sorted(times[2:])[3]


def test_a_selection_crowded_into_few_chunks_is_not_much_slower():
    """16 rows of 520 chunks, one entry in ten, spread evenly and all of it in a tenth of the row: 164 and 295 us with four
    wavefronts per chunk, 158 and 202 with eight."""
    n, chunks, k = 16, 520, 520 * 4096 // 10
    assert step_us(n, chunks, k, True) < 1.5 * step_us(n, chunks, k, False)
