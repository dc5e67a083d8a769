"""The two halves of a step run apart (compams_worker_step + compams_encode on one context, compams_server_step
on another), through the C ABI, against the oracle's whole step: bit-identical parameters and moments on the
server side, bit-identical messages and residuals on the worker side."""
import numpy as np
import pytest
import torch

from oracle import compams_oracle as O
from paper_2205_05632_amd import binding as B

from parity import bits_equal

pytestmark = pytest.mark.gpu


def run_split(n, d, compressor, steps, k=0, off=None, same_context=False, seed=0):
    rng = np.random.default_rng(seed + d)
    theta0 = rng.standard_normal(d).astype(np.float32) * 0.1
    t0 = torch.from_numpy(theta0)
    workers = B.Compams(n, d, t0.clone(), compressor=compressor, k=k, block_offsets=off)
    server = workers if same_context else B.Compams(n, d, t0.clone(), compressor=compressor, k=k, block_offsets=off)
    cpu = O.Oracle(n, d, theta0, compressor=compressor, k=k, block_offsets=off)
    for t in range(steps):
        g = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-3, 0, (1, d))).astype(np.float32)
        g[:, ::9] = 0.0
        gp = torch.zeros((n, workers.ld), dtype=torch.float32)
        gp[:, :d] = torch.from_numpy(g)
        workers.compams_worker_step(gp.to(workers.device))
        msgs, words = workers.compams_encode()
        status = server.compams_server_step(msgs, words, 1e-3)
        cpu.step(g, 1e-3)
        torch.cuda.synchronize()
        assert not status.cpu().numpy().any(), f"step {t}: status {status.cpu().numpy()}"
        if compressor == B.TOPK:
            assert np.array_equal(workers.compams_state("last_idx").cpu().numpy(), cpu.get("idx")), f"step {t}: lists"
        else:
            assert np.array_equal(workers.compams_state("last_signbits").cpu().numpy().view(np.uint32), cpu.get("bits"))
        for name in ("theta", "m", "v", "vhat"):
            assert bits_equal(server.compams_state(name).cpu().numpy(), cpu.get(name)), f"step {t}: server {name}"
        if not same_context:   # the workers' context never touches the parameters
            assert bits_equal(workers.compams_state("theta").cpu().numpy(), theta0), f"step {t}: workers' theta moved"
    assert bits_equal(np.ascontiguousarray(workers.compams_state("e").cpu().numpy()), cpu.get("e")), "residuals"
    workers.close()
    if not same_context:
        server.close()
    cpu.close()


@pytest.mark.parametrize("n,d,k", [(4, 65536, 655), (3, 100003, 1000), (2, 8191, 8191), (17, 20000, 7), (1, 5, 2)])
@pytest.mark.parametrize("same_context", [False, True])
def test_topk_halves_equal_the_whole_step(n, d, k, same_context):
    run_split(n, d, B.TOPK, 5, k=k, same_context=same_context)


@pytest.mark.parametrize("n,d,offsets", [(3, 5000, [0, 1, 11, 500, 2548, 5000]), (4, 70000, "fixed4096"),
                                         (2, 50000, "one"), (9, 33000, "ragged")])
@pytest.mark.parametrize("same_context", [False, True])
def test_blocksign_halves_equal_the_whole_step(n, d, offsets, same_context):
    if offsets == "fixed4096":
        off = np.concatenate([np.arange(0, d, 4096), [d]]).astype(np.int64)
    elif offsets == "one":
        off = np.array([0, d], dtype=np.int64)
    elif offsets == "ragged":
        rng = np.random.default_rng(1)
        off = np.concatenate([[0], np.sort(rng.choice(np.arange(1, d), size=300, replace=False)), [d]]).astype(np.int64)
    else:
        off = np.array(offsets, dtype=np.int64)
    run_split(n, d, B.BLOCKSIGN, 5, off=off, same_context=same_context)


def test_server_step_flags_a_malformed_message_and_goes_on():
    n, d, k = 3, 30000, 300
    rng = np.random.default_rng(2)
    w = B.Compams(n, d, torch.zeros(d), compressor=B.TOPK, k=k)
    s = B.Compams(n, d, torch.zeros(d), compressor=B.TOPK, k=k)
    gp = torch.zeros((n, w.ld), dtype=torch.float32)
    gp[:, :d] = torch.from_numpy(rng.standard_normal((n, d)).astype(np.float32))
    w.compams_worker_step(gp.to(w.device))
    msgs, words = w.compams_encode()
    msgs[1, 0] = 9                      # not a message
    msgs[2, 4:12] = -1                  # coordinates run past d
    status = s.compams_server_step(msgs, words, 1e-3)
    torch.cuda.synchronize()
    st = status.cpu().numpy()
    assert st[0] == 0 and st[1] & 1 and st[2] & 4, st
    assert torch.isfinite(s.compams_state("theta")).all()
    w.close(); s.close()


def test_the_identity_compressor_has_no_halves():
    d = 100
    c = B.Compams(2, d, torch.zeros(d), compressor=B.NONE)
    with pytest.raises(B.CompamsError):
        c.compams_worker_step(torch.zeros((2, c.ld), device=c.device))
    c.close()


@pytest.mark.parametrize("n", [1, 16, 17, 33])
def test_workers_half_of_block_topk_over_tiles_of_workers(n):
    """The workers' half has a workgroup per chunk and tile of sixteen workers: lists, values, residuals and the counters
    that the next step starts from, bit for bit."""
    rng = np.random.default_rng(n)
    off = np.array([0, 20, 1044, 5140, 5144, 20000, 36388], dtype=np.int64)
    kb = np.array([1, 1024, 41, 4, 3000, 100], dtype=np.int64)
    d = int(off[-1])
    theta0 = np.zeros(d, dtype=np.float32)
    gpu = B.Compams(n, d, torch.from_numpy(theta0), compressor=B.TOPK_BLOCKS, block_offsets=off, block_k=kb)
    cpu = O.Oracle(n, d, theta0, compressor=O.TOPK_BLOCKS, block_offsets=off, block_k=kb)
    for t in range(4):
        g = rng.standard_normal((n, d), dtype=np.float32) * np.float32(8.0 if t == 3 else 1.0)
        gp = torch.zeros((n, gpu.ld), dtype=torch.float32)
        gp[:, :d] = torch.from_numpy(g)
        gpu.compams_worker_step(gp.to(gpu.device))
        cpu.step(g, 1e-3)
        torch.cuda.synchronize()
        assert np.array_equal(gpu.compams_state("last_idx").cpu().numpy(), cpu.get("idx")), f"step {t}: lists"
        assert bits_equal(gpu.compams_state("last_val").cpu().numpy(), cpu.get("val")), f"step {t}: values"
    assert bits_equal(np.ascontiguousarray(gpu.compams_state("e").cpu().numpy()), cpu.get("e")), "residuals"
    assert bits_equal(gpu.compams_state("theta").cpu().numpy(), theta0)
    gpu.close()
    cpu.close()


def test_workers_half_does_not_go_through_the_tiles_one_after_the_other():
    """300 workers in few chunks: the half alone is far from the whole step, which also adds every list (with all tiles of
    workers in one workgroup 128 of 201 us or worse; with a workgroup per tile 76)."""
    n, d = 300, 50000
    off = np.array([0, 400, 1200, 4000, 8000, 16000, 32000, d], dtype=np.int64)
    kb = np.diff(off) // 100
    ctx = B.Compams(n, d, torch.zeros(d), compressor=B.TOPK_BLOCKS, block_offsets=off, block_k=kb)
    g = [torch.randn((n, ctx.ld), device=ctx.device) for _ in range(3)]

    def us(call):
        for i in range(9):
            call(g[i % 3])
        times = []
        for _ in range(7):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for i in range(20):
                call(g[i % 3])
            end.record()
            torch.cuda.synchronize()
            times.append(begin.elapsed_time(end) / 20 * 1e3)
        return sorted(times)[3]

    whole = us(lambda x: ctx.compams_step(x, 1e-3))
    half = us(ctx.compams_worker_step)
    assert half < 0.55 * whole, (half, whole)
    ctx.close()
