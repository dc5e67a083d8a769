"""Guess and window for the next step come from the last kernel up to 64 rows, beyond that from the kernel that selects: every row has
them, in whole steps and in the workers' half, and many rows share the work out."""
import numpy as np
import pytest
import torch

from paper_2205_05632_amd import binding as B

from parity import Pair
from test_gpu_topk_blocks import BlockPair

pytestmark = pytest.mark.gpu
CHUNK = 4096


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("n,d,k", [(64, CHUNK, 400), (65, CHUNK, 400), (64, 17 * CHUNK, 2000), (65, 17 * CHUNK, 2000), (1100, 1500, 100), (130, 17 * CHUNK + 3, 3000), (70, 3 * CHUNK, 900)])
def test_every_row_has_its_window(n, d, k, half):
    rng = np.random.default_rng(n)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32), B.TOPK, k=k)
    for t in range(12):
        g = rng.standard_normal((n, d)).astype(np.float32)
        if half:
            gd = torch.zeros((n, p.gpu.ld), device="cuda")
            gd[:, :d] = torch.from_numpy(g).cuda()
            p.gpu.compams_worker_step(gd)
            p.cpu.step(g, 1e-3)
            torch.cuda.synchronize()
            assert np.array_equal(p.gpu.compams_state("last_idx").cpu().numpy(), p.cpu.get("idx")), t
        else:
            p.step(g, 1e-3, label=f"step {t}", with_e=False)
        if t >= 3:  # from here on a row without a window is one that was left out
            missed = p.gpu.compams_state("counters").cpu().numpy()[:, 5]
            assert (missed != 1).all(), (t, np.flatnonzero(missed == 1))
    p.close()


@pytest.mark.parametrize("n", [64, 65, 130])
def test_every_block_of_every_row_has_its_window(n):
    d = 30000
    off = np.array([0, 1200, 5000, 5004, 20000, d], dtype=np.int64)
    kb = np.maximum(1, np.diff(off) // 10)
    rng = np.random.default_rng(1)
    p = BlockPair(n, d, off, kb, np.zeros(d, dtype=np.float32))
    large = np.diff(off) > 1024  # (smaller blocks have no window)
    for t in range(8):
        p.step(rng.standard_normal((n, d)).astype(np.float32))
        p.compare(f"step {t}", with_e=False)
        if t >= 3:
            missed = p.gpu.compams_state("counters").cpu().numpy().reshape(-1, 8)[:, 5].reshape(n, -1)
            assert (missed[:, large] != 1).all(), (t, np.argwhere(missed[:, large] == 1))
    p.close()


def test_four_times_the_rows():
    """A tile of 16 rows to a workgroup in the workers' half: 256 of them take no four times as long as 64 (one wavefront for all rows'
    windows: 90 us of the kernel at 4096 rows)."""
    d, us = CHUNK, {}
    for n in (1024, 4096):
        c = B.Compams(n, d, torch.zeros(d), compressor=B.TOPK, k=40)
        g = [torch.randn((n, c.ld), device="cuda") for _ in range(2)]
        times = []
        for t in range(16):
            c.profile_enable(1)
            c.compams_worker_step(g[t % 2])
            times.append(c.profile_read()["topk_final"][0] * 1e3)
            c.profile_enable(0)
        us[n] = min(times[6:])
        c.close()
    assert us[4096] < 2 * us[1024], us
