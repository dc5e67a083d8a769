"""The dense passes in pages (a die's workgroups take the same 4 KB page of every 32 KB span) at the sizes where the walk
could miss or repeat something: one page more or less than a span, a group of spans or a group of workgroups; and the
first passes of block-sign on magnitudes that leave a quarter's window, in pages (large problems) and in address order.
Everything is compared with the oracle bit for bit, as every operation is fixed."""
import numpy as np
import pytest
import torch

from paper_2205_05632_amd import binding as B

from parity import Pair
from test_gpu_split import run_split

pytestmark = pytest.mark.gpu
PAGE, SPAN, GROUP = 1024, 8192, 32768


def values(rng, n, d, kind):
    g = rng.standard_normal((n, d)).astype(np.float32)
    if kind == "zeros":            # whole quarters of zeros, single ones elsewhere
        g[:, : d // 2] = 0.0
        g[rng.random((n, d)) < 0.1] = 0.0
    elif kind == "wide":           # far below a window of 22 exponents, denormals among them
        g *= (2.0 ** rng.integers(-140, 3, (n, d))).astype(np.float32)
    elif kind == "special":
        g[:, d // 3] = np.inf
        g[:, d // 2] = -np.inf
        g[n // 2, (2 * d) // 3] = np.nan
    elif kind == "ends":           # every quarter's largest magnitude just below a power of two, the others 2^-21 of it
        g = np.where(np.arange(d) % PAGE == 0, np.float32(2.0 - 2.0 ** -23), np.float32(2.0 ** -21)) * np.sign(g + 0.5)
    return g.astype(np.float32)


def run(p, n, d, kind, steps=3, with_e=True):
    rng = np.random.default_rng(d + n)
    for t in range(steps):
        p.step(values(rng, n, d, kind), 1e-3, label=f"{n} x {d} {kind} step {t}", with_e=with_e or t == steps - 1)
    assert all(p.exact.values()), p.exact
    p.close()


def offsets(d, size):
    return np.concatenate([np.arange(0, d, size, dtype=np.int64), [d]])


@pytest.mark.parametrize("kind", ["plain", "zeros", "wide", "special", "ends"])
@pytest.mark.parametrize("n,d,size", [(3, GROUP, 4096), (2, GROUP + PAGE, 1 << 30), (1, 2 * GROUP + 5, 4096),
                                      (3, SPAN - 32, 1000), (5, GROUP + 1, 1 << 30)])
def test_blocksign_values(n, d, size, kind):
    run(Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=offsets(d, size)), n, d, kind)


@pytest.mark.parametrize("n,d,size", [(2, 256, 256), (4, PAGE, 1 << 30), (2, SPAN, 4096), (2, SPAN + PAGE, 300), (2, GROUP - PAGE, 4096),
                                      (1, GROUP + 3, 1 << 30), (3, 9 * 4096, 1000), (2, 17 * 4096 + 256, 65536),
                                      (2, 150 * 4096 - 2048, 4096), (2, 150 * 4096 + 3, 100000), (64, 3000, 1000)])
def test_blocksign_sizes(n, d, size):
    # the residual stays pending between the steps, and is asked for after the last
    run(Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=offsets(d, size)), n, d, "plain", with_e=False)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33])
@pytest.mark.parametrize("d", [1, 255, 1027, SPAN, GROUP - 1, GROUP, GROUP + 1, 3 * GROUP + SPAN + 5])
def test_identity_sizes(n, d):
    run(Pair(n, d, np.ones(d, np.float32), B.NONE), n, d, "plain", with_e=False)


# Sixteen rows at once beyond 7 M coordinates unless there are three to eight.
@pytest.mark.parametrize("n,d", [(1, 7_000_001), (2, 7_000_001), (3, 7_000_001), (8, 7_000_001), (9, 7_000_001), (9, 7_000_000),
                                 (16, 7_000_003), (17, 7_000_003), (33, 7_000_002)])
def test_identity_forms(n, d):
    rng = np.random.default_rng(n)
    p = Pair(n, d, np.ones(d, np.float32), B.NONE)
    base = rng.standard_normal(d).astype(np.float32)
    for t in range(2):
        p.step(np.stack([np.roll(base, 1001 * t + 37 * i) for i in range(n)]), 1e-3, label=f"{n} x {d} step {t}")
    assert all(p.exact.values()), p.exact
    p.close()


# Block-sign goes in pages from 24576 chunks in all rows on.
@pytest.mark.parametrize("n,d,size", [(1600, 16 * 4096 - 3100, 4096), (1100, 23 * 4096 + 1, 100000)])
def test_blocksign_in_pages(n, d, size):
    rng = np.random.default_rng(d)
    p = Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=offsets(d, size))
    base = values(rng, 2, d, "plain")
    odd = [values(rng, 2, d, kind) for kind in ("zeros", "wide", "special", "ends")]
    for t in range(3):
        g = np.stack([np.roll(base[(t + i) % 2], 37 * i + 1001 * t) for i in range(n)])
        for i, o in enumerate(odd):
            g[7 * i + t] = o[t % 2]
        p.step(g, 1e-3, label=f"{n} x {d} step {t}", with_e=(t == 2))
    assert all(p.exact.values()), p.exact
    p.close()


# Top-k goes in pages from 45056 chunks in all rows on: tests of whole rows with as many rows as that takes, of a length at
# which the last span, the last chunk and the last quarter are cut.
@pytest.mark.parametrize("n,d,k", [(700, 65 * 4096 - 3100, 400), (640, 71 * 4096 + 1, 9000)])
def test_topk_in_pages(n, d, k):
    rng = np.random.default_rng(d)
    p = Pair(n, d, np.zeros(d, np.float32), B.TOPK, k=k)
    scale = np.repeat(10.0 ** rng.uniform(-2, 0, d // 5000 + 1), 5000)[:d].astype(np.float32)
    base = rng.standard_normal((2, d)).astype(np.float32)
    for t in range(4):  # (rows are shifted copies: every row its own selection without drawing all of them)
        g = np.stack([np.roll(base[(t + i) % 2], 37 * i + 1001 * t) for i in range(n)]) * scale
        if t == 2:
            g[1] = 1.0                      # equal magnitudes: ties, a list that overflows, the general kernels
            g[2] *= 8.0                     # a threshold far above its window
            g[3, : d // 2] = 0.0
        p.step(g, 1e-3, label=f"{n} x {d} step {t}", with_e=(t == 3))
    assert all(p.exact.values()), p.exact
    p.close()


# Large entries side by side in every row of a matrix whose width is a multiple of the span, so that all of them lie in the same
# pages: the lists hold them all the same, and no row is read again once its window has settled.
@pytest.mark.parametrize("n,d,k,width", [(8, 5700 * 4096 - 100, 230000, SPAN), (8, 5700 * 4096 - 100, 230000, GROUP),
                                         (64, 733 * 4096 - 100, 250000, SPAN)])
def test_large_columns_in_one_page(n, d, k, width):
    ctx = B.Compams(n, d, torch.zeros(d, device="cuda"), compressor=B.TOPK, k=k)
    gen = torch.Generator(device="cuda").manual_seed(5)
    scale = torch.where(torch.arange(d, device="cuda") % width < PAGE, 1.0, 1e-3)
    g = torch.zeros((n, ctx.ld), device="cuda")
    for t in range(12):
        for i in range(n):
            g[i, :d].normal_(generator=gen).mul_(scale)
        ctx.compams_step(g, 1e-3)
        if t >= 6:
            counters = ctx.compams_state("counters").cpu().numpy()
            assert not (counters[:, 5] == 2).any(), (t, counters[:, 5])  # no candidate list overflowed
            assert not counters[:, 0].any(), (t, counters[:, 0])         # no row was read again
    ctx.close()


# The general kernels alone (no window; then no list at all) on rows in pages, with large entries crowded into one quarter of every
# eighth chunk, and with few in any.
@pytest.mark.parametrize("n,d,k,columns", [(700, 65 * 4096 - 3100, 12000, PAGE), (640, 71 * 4096 + 1, 300, 0)])
def test_general_route_in_pages(n, d, k, columns):
    rng = np.random.default_rng(d)
    p = Pair(n, d, np.zeros(d, np.float32), B.TOPK, k=k)
    p.gpu.set_option(B.OPT_BAND, 0)
    base = rng.standard_normal((2, d)).astype(np.float32)
    scale = np.where(np.arange(d) % GROUP < columns, 1.0, 1e-2).astype(np.float32)
    for t in range(4):
        g = np.stack([np.roll(base[(t + i) % 2], 37 * i + 1001 * t) for i in range(n)]) * scale
        g[1] = 1.0  # ties, and a list that overflows
        if t == 3:
            p.gpu.set_option(B.OPT_FORCE_DENSE, 1)
        p.step(g, 1e-3, label=f"{n} x {d} step {t}", with_e=(t == 3))
        counters = p.gpu.compams_state("counters").cpu().numpy()
        assert not counters[:, 4].any()
        if t in (1, 2):
            assert (counters[2:, 0] == 0).all()  # selected from the lists
    assert all(p.exact.values()), p.exact
    p.close()


def test_halves_in_pages():
    run_split(640, 71 * 4096 + 1, B.TOPK, 3, k=9000)
