"""The state arrays by ordinary accesses and by streaming ones: sizes on both sides of the line ((n + 32) d = 231 M), every
compressor that has it, and the call that stands for itself, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from oracle import compams_oracle as O
from paper_2205_05632_amd import binding as B

from parity import Pair, bits_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("comp,k,size", [(B.TOPK, 7000, 0), (B.BLOCKSIGN, 0, 100000)])
@pytest.mark.parametrize("n,d", [(1, 7_000_000), (1, 7_000_003), (30, 3_725_806), (30, 3_725_807)])
def test_both_sides_of_the_line(n, d, comp, k, size):
    off = np.concatenate([np.arange(0, d, size, dtype=np.int64), [d]]) if size else None
    rng = np.random.default_rng(d)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32), comp, k=k, block_offsets=off)
    base = rng.standard_normal(d).astype(np.float32)
    for t in range(3):
        p.step(np.stack([np.roll(base, 1001 * t + 37 * i) for i in range(n)]), 1e-3, label=f"{n} x {d} step {t}", with_e=t == 2)
    assert all(p.exact.values()), p.exact
    p.close()


@pytest.mark.parametrize("d", [6_999_999, 7_300_001])
def test_static_call_on_both_sides(d):
    k, ld = 3000, B.padded_ld(d)
    rng = np.random.default_rng(d)
    theta0 = rng.standard_normal(d).astype(np.float32)
    theta = torch.from_numpy(theta0).cuda()
    m, v, vhat = (torch.zeros(d, device="cuda") for _ in range(3))
    e = torch.zeros((1, ld), device="cuda")
    idx = torch.zeros((1, k), dtype=torch.int32, device="cuda")
    cpu = O.Oracle(1, d, theta0, compressor=O.TOPK, k=k)
    for t in range(2):
        g = rng.standard_normal((1, d)).astype(np.float32)
        gd = torch.zeros((1, ld), device="cuda")
        gd[:, :d] = torch.from_numpy(g).cuda()
        assert B.compams_step_static(1, d, k, theta, m, v, vhat, e, gd, 1e-3, idx_out=idx) == 0
        cpu.step(g, 1e-3)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy(), cpu.get("idx")), t
        for name, x in (("theta", theta), ("m", m), ("v", v), ("vhat", vhat), ("e", e[:, :d])):
            assert bits_equal(np.ascontiguousarray(x.cpu().numpy()), cpu.get(name)), (t, name)
    cpu.close()
