"""Block-sign layouts in which no block reaches beyond a chunk of 4096 coordinates: the server kernel forms the scales, up to 512 of them
to a chunk.  Both sides of that, irregular blocks, values of every kind, and the workers' half in between, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2205_05632_amd import binding as B

from parity import Pair

pytestmark = pytest.mark.gpu


def offsets(d, layout):
    if layout == "irregular":
        cuts = [c for c in (0, 5, 300, 4096, 4097, 8191, 8192, 8192 + 2048, 12288) if c < d]
    else:
        cuts = list(range(0, d, layout))
    return np.array(cuts + [d], dtype=np.int64)


def values(rng, kind, n, d):
    g = rng.standard_normal((n, d)).astype(np.float32)
    if kind == "wide":
        g = np.ldexp(g, rng.integers(-60, 60, (n, d))).astype(np.float32)
    elif kind == "zeros":
        g[:, rng.random(d) < 0.9] = 0.0
        g[:, : d // 3] = 0.0
    elif kind == "special":
        g[0, d // 2] = np.inf
        g[n - 1, d - 1] = np.nan
    return g


@pytest.mark.parametrize("kind", ["unit", "wide", "zeros", "special"])
@pytest.mark.parametrize("n,d,layout", [
    (1, 1, 4096), (3, 4096, 4096), (5, 3 * 4096 + 100, 4096), (4, 12288 + 77, "irregular"),
    (8, 2 * 4096 + 9, 64), (9, 2 * 4096 + 9, 64),       # 512 and 576 scales to a chunk
    (1, 2 * 4096, 8), (1, 2 * 4096, 4),                 # 512 and 1024
    (128, 4097, 1024), (129, 4097, 1024),               # 512 and 516
    (2, 70 * 4096 - 3, 256), (3, 20000, 4095)])         # many chunks; blocks that do reach beyond a chunk
def test_scales(n, d, layout, kind):
    rng = np.random.default_rng(d + n)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32), B.BLOCKSIGN, block_offsets=offsets(d, layout))
    for t in range(4):
        with np.errstate(all="ignore"):
            p.step(values(rng, kind if t else "unit", n, d), 1e-3, label=f"{n} x {d} / {layout} {kind} step {t}", with_e=t % 2 == 1)
    assert all(p.exact.values()), p.exact
    p.close()


def test_the_workers_half_in_between():
    """The workers' half has no server kernel behind it: the scales come from the first pass or a launch, and the digits it leaves behind
    are those that a whole step begins with."""
    n, d = 3, 5 * 4096
    rng = np.random.default_rng(1)
    theta0 = torch.from_numpy(rng.standard_normal(d).astype(np.float32))
    whole, halves = (B.Compams(n, d, theta0, compressor=B.BLOCKSIGN, block_offsets=offsets(d, 4096)) for _ in range(2))
    for t in range(6):
        g = torch.zeros((n, whole.ld), device="cuda")
        g[:, :d] = torch.from_numpy(rng.standard_normal((n, d)).astype(np.float32)).cuda()
        whole.compams_step(g, 1e-3)
        if t % 3 == 1:
            halves.compams_worker_step(g)
            messages, words = halves.compams_encode()
            sent = [halves.compams_state(x).clone() for x in ("last_scales", "last_signbits")]
            assert not halves.compams_server_step(messages, words, 1e-3).any()
        else:
            halves.compams_step(g, 1e-3)
            sent = [halves.compams_state(x) for x in ("last_scales", "last_signbits")]
        for x, name in zip(sent, ("last_scales", "last_signbits")):
            assert torch.equal(x.view(torch.int32), whole.compams_state(name).view(torch.int32)), (t, name)
    for name in ("theta", "m", "v", "vhat", "e"):
        assert torch.equal(whole.compams_state(name)[..., :d], halves.compams_state(name)[..., :d]), name
    whole.close()
    halves.close()
