"""GPU parity tests: the HIP library, called through its C ABI, against the CPU oracle.

Bar: selected index sets, selected values, sign patterns and block scales bit-exact; theta, m, v, vhat and
the residuals e within |a - b| <= 1e-5 |b| + 1e-5 max|b| after every step (10 steps in the basic cases).
"""
import json
import os

import numpy as np
import pytest
import torch

from oracle import compams_oracle as O
from paper_2205_05632_amd import binding as B
from composed_blocks import CompamsBlockTopk
from paper_2205_05632_amd import workloads as W

from parity import Pair, bits_equal

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


def run_pair(p, gs, lr=1e-3, label=""):
    for t, g in enumerate(gs):
        p.step(g, lr, label=f"{label} step {t}")


def rand_grads(seed, n, d, steps, scale=1.0):
    rng = np.random.default_rng(seed)
    return [(rng.standard_normal((n, d)) * scale).astype(np.float32) for _ in range(steps)]


# ------------------------------------------------------------------------------------------- top-k
@pytest.mark.parametrize("eps_mode", [B.EPS_IN_SQRT, B.EPS_OUT_SQRT])
def test_topk_tiny_config_10_steps(eps_mode):
    w = W.get("tiny")
    p = Pair(w.n, w.d, W.theta0(w).numpy(), B.TOPK, k=w.k, eps_mode=eps_mode)
    run_pair(p, [W.gradients(w, t).numpy() for t in range(10)], lr=w.lr, label="tiny")
    # every operation is element-wise IEEE fp32 in a fixed order on both sides
    assert all(p.exact.values()), p.exact
    c = p.gpu.compams_state("counters").cpu().numpy()
    assert (c[:, 0] == 0).all(), f"steady-state steps should take candidates from the first pass: {c}"
    p.close()


@pytest.mark.parametrize("n,d,k,ld", [(3, 100003, 1000, None), (2, 4097, 5, 4100), (1, 1, 1, None), (5, 8191, 8191, 8200),
                                      (2, 12288, 1, None), (4, 300001, 150000, None), (17, 20000, 200, None),
                                      (40, 30000, 300, None), (33, 9000, 9000, None), (64, 4097, 40, None),
                                      (300, 5000, 50, None)])
def test_topk_ragged_shapes(n, d, k, ld):
    rng = np.random.default_rng(d + k)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32) * 0.1, B.TOPK, k=k, ld=ld)
    run_pair(p, rand_grads(d, n, d, 4), label=f"ragged d={d} k={k}")
    # columns >= d of e are never touched
    if p.gpu.ld > d:
        assert not p.gpu.e[:, d:].any()
    p.close()


def test_topk_padding_columns_keep_their_contents():
    n, d, ld, k = 2, 1001, 1008, 10
    p = Pair(n, d, np.zeros(d, np.float32), B.TOPK, k=k, ld=ld)
    p.gpu.e[:, d:] = 7.0
    g = np.random.default_rng(0).standard_normal((n, d)).astype(np.float32)
    gp = torch.full((n, ld), 3.0)
    gp[:, :d] = torch.from_numpy(g)
    p.gpu.compams_step(gp.cuda(), 1e-3)
    p.cpu.step(g, 1e-3)
    p.compare("padding")
    assert (p.gpu.e[:, d:] == 7.0).all()
    p.close()


def adversarial_rows(d, rng):
    rows = []
    rows.append(np.full(d, 1.5, np.float32))                               # all equal
    rows.append(np.zeros(d, np.float32))                                   # all zero
    r = np.zeros(d, np.float32); r[::7] = -0.0; r[5::11] = 1e-40; r[3] = 2.0   # +-0, denormals, one large
    rows.append(r)
    rows.append(rng.integers(-3, 4, d).astype(np.float32))                 # few magnitudes: ties at the threshold
    r = rng.standard_normal(d).astype(np.float32); r[10] = np.inf; r[20] = -np.inf
    rows.append(r)
    r = (rng.standard_normal(d) * 1e-42).astype(np.float32)                # all denormal
    rows.append(r)
    r = rng.standard_normal(d).astype(np.float32); r[d // 2:] = r[: d - d // 2]  # every magnitude twice
    rows.append(r)
    return np.stack(rows)


@pytest.mark.parametrize("k", [1, 2, 97, 5000, 20000])
@pytest.mark.parametrize("route", ["default", "dense", "small_cap", "no_predict"])
def test_topk_adversarial_rows_every_route(k, route):
    d = 20000
    rng = np.random.default_rng(k)
    g0 = adversarial_rows(d, rng)
    n = g0.shape[0]
    p = Pair(n, d, np.zeros(d, np.float32), B.TOPK, k=k)
    if route == "dense":
        p.gpu.set_option(B.OPT_FORCE_DENSE, 1)
    elif route == "small_cap":
        p.gpu.set_option(B.OPT_CANDIDATE_CAP, min(d, max(k + 50, 300)))
    elif route == "no_predict":
        p.gpu.set_option(B.OPT_PREDICT, 0)
    # state tensors may hold Inf/NaN here; index sets and values are the point
    for t in range(3):
        g = g0 if t != 1 else g0[::-1].copy()
        p.step(g, 1e-3, label=f"adversarial k={k} {route} step {t}")
    c = p.gpu.compams_state("counters").cpu().numpy()
    if route == "dense":
        assert (c[:, 0] == 4).all()
    if route == "no_predict":
        assert (c[:, 0] >= 1).all()
    p.close()


def test_topk_routes_agree_and_are_counted():
    """Guessed candidates, re-read candidates and no candidates must give identical bytes."""
    n, d, k = 3, 150000, 1500
    gs = rand_grads(5, n, d, 6)
    outs = []
    for route in ("default", "no_predict", "dense", "small_cap"):
        p = Pair(n, d, np.zeros(d, np.float32), B.TOPK, k=k)
        if route == "no_predict":
            p.gpu.set_option(B.OPT_PREDICT, 0)
        if route == "dense":
            p.gpu.set_option(B.OPT_FORCE_DENSE, 1)
        if route == "small_cap":
            p.gpu.set_option(B.OPT_CANDIDATE_CAP, k // 2)   # no list can fit
        reads = []
        for t, g in enumerate(gs):
            p.step(g, 1e-3, label=f"{route} step {t}")
            reads.append(p.gpu.compams_state("counters").cpu().numpy()[:, 0].copy())
        outs.append([p.gpu.compams_state(s).cpu().numpy().copy() for s in ("theta", "e", "last_idx", "last_val")])
        reads = np.array(reads)
        if route == "default":
            assert (reads[0] == 1).all() and (reads[2:] == 0).all(), reads
        elif route == "no_predict":
            assert (reads == 1).all(), reads
        else:
            assert (reads == 4).all(), reads
        p.close()
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("where", ["every eighth chunk", "every chunk"])
def test_topk_candidates_all_in_one_run_of_the_list(where):
    """The candidate list of a row is kept as eight runs, chunk c appending to run c % 8, each with an eighth of the
    capacity.  With every large entry in chunks 0, 8, 16, ... that run outgrows its share although the list as a
    whole would fit: the step has to notice and read the row once more, and the result is the same.  The same
    entries spread over all chunks fit, and the steady-state steps take their candidates from the first pass."""
    n, d, k = 2, 64 * 4096, 6000
    rng = np.random.default_rng(8)
    p = Pair(n, d, np.zeros(d, np.float32), B.TOPK, k=k)
    p.gpu.set_option(B.OPT_CANDIDATE_CAP, 16000)      # an eighth: 2000 entries
    chunks, per_chunk = (range(0, 64, 8), 1496) if where == "every eighth chunk" else (range(64), 187)
    reads = []
    for t in range(5):
        g = (rng.standard_normal((n, d)) * 1e-3).astype(np.float32)
        for c in chunks:
            big = rng.standard_normal((n, per_chunk)) + 3.0 * np.sign(rng.standard_normal((n, per_chunk)))
            g[:, c * 4096:c * 4096 + per_chunk] = big.astype(np.float32)
        p.gpu.e.zero_()                                # keep the large entries where they are from step to step
        p.cpu.set_state(e=np.zeros((n, d), np.float32))
        p.step(g, 1e-3, label=f"{where} step {t}")
        reads.append(p.gpu.compams_state("counters").cpu().numpy()[:, 0].copy())
    reads = np.array(reads)
    if where == "every eighth chunk":
        assert (reads[1:] >= 1).all(), reads           # never from the first pass's list
    else:
        assert (reads[2:] == 0).all(), reads
    p.close()


def test_topk_guess_that_is_too_high_falls_back():
    """Gradients that shrink by 100x make the carried-over bucket too high: the step must notice and re-read."""
    n, d, k = 2, 100000, 1000
    rng = np.random.default_rng(3)
    p = Pair(n, d, np.zeros(d, np.float32), B.TOPK, k=k)
    reads = []
    for t in range(6):
        scale = 1.0 if t < 3 else 1e-4
        g = (rng.standard_normal((n, d)) * scale).astype(np.float32)
        if t == 3:
            p.gpu.e.zero_()                 # drop the residuals so that the threshold really falls
            p.cpu.set_state(e=np.zeros((n, d), np.float32))
        p.step(g, 1e-3, label=f"shrink step {t}")
        reads.append(p.gpu.compams_state("counters").cpu().numpy()[:, 0].copy())
    reads = np.array(reads)
    assert (reads[2] == 0).all() and (reads[3] >= 1).all() and (reads[5] == 0).all(), reads
    p.close()


@pytest.mark.parametrize("n,d,k", [(4, 65536, 655), (3, 100003, 50000), (2, 8191, 8191), (2, 20000, 1)])
def test_topk_deferred_residual_clearing(n, d, k):
    """Between steps the zeroing of the selected residuals is pending; the next first pass must honour it.
    Index sets and parameters are compared after every step, the residuals only at the end."""
    rng = np.random.default_rng(d)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32) * 0.1, B.TOPK, k=k)
    gs = rand_grads(d + 1, n, d, 7)
    for t, g in enumerate(gs):
        p.step(g, 1e-3, label=f"deferred step {t}", with_e=(t == len(gs) - 1))
    assert all(p.exact.values()), p.exact
    # the caller's own view of e is settled by the query above
    assert np.array_equal(p.gpu.e[:, :d].cpu().numpy().view(np.uint32), p.cpu.get("e").view(np.uint32))
    p.close()


def test_topk_is_deterministic():
    n, d, k = 4, 200000, 2000
    gs = rand_grads(9, n, d, 5)
    res = []
    for rep in range(2):
        gpu = B.Compams(n, d, torch.zeros(d), compressor=B.TOPK, k=k)
        for g in gs:
            gp = torch.zeros((n, gpu.ld)); gp[:, :d] = torch.from_numpy(g)
            gpu.compams_step(gp.cuda(), 1e-3)
        torch.cuda.synchronize()
        res.append([gpu.compams_state(s).cpu().numpy().copy() for s in ("theta", "m", "v", "vhat", "e", "last_idx", "last_val")])
        gpu.close()
    for a, b in zip(*res):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


# ------------------------------------------------------------------------------------------- block-sign
@pytest.mark.parametrize("eps_mode", [B.EPS_IN_SQRT, B.EPS_OUT_SQRT])
def test_blocksign_tiny_config_10_steps(eps_mode):
    w = W.get("tiny_blocksign")
    p = Pair(w.n, w.d, W.theta0(w).numpy(), B.BLOCKSIGN, block_offsets=w.block_offsets(), eps_mode=eps_mode)
    run_pair(p, [W.gradients(w, t).numpy() for t in range(10)], lr=w.lr, label="tiny_blocksign")
    assert all(p.exact.values()), p.exact
    p.close()


def ragged_offsets(d, rng, m):
    cuts = np.sort(rng.choice(np.arange(1, d), size=m - 1, replace=False))
    return np.concatenate([[0], cuts, [d]]).astype(np.int64)


@pytest.mark.parametrize("n,d,offsets", [
    (3, 5000, [0, 1, 11, 500, 2548, 5000]),
    (2, 100003, "ragged40"),
    (2, 9000, "unit"),
    (4, 70000, "fixed4096"),
    (2, 50000, "one"),
    (3, 33000, "ragged2000"),
    (21, 20000, "ragged40"),
    (40, 8192, "fixed4096"),
    (300, 6000, "ragged40"),
])
def test_blocksign_block_layouts(n, d, offsets):
    rng = np.random.default_rng(d)
    if offsets == "ragged40":
        off = ragged_offsets(d, rng, 40)
    elif offsets == "ragged2000":
        off = ragged_offsets(d, rng, 2000)
    elif offsets == "unit":
        off = np.arange(d + 1, dtype=np.int64)
    elif offsets == "fixed4096":
        off = np.concatenate([np.arange(0, d, 4096), [d]]).astype(np.int64)
    elif offsets == "one":
        off = np.array([0, d], dtype=np.int64)
    else:
        off = np.array(offsets, dtype=np.int64)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32) * 0.1, B.BLOCKSIGN, block_offsets=off)
    gs = []
    for t in range(5):
        g = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-4, 1, (1, d))).astype(np.float32)
        g[:, ::13] = 0.0
        gs.append(g)
    run_pair(p, gs, label=f"blocksign {offsets}")
    if offsets == "unit":
        assert not p.gpu.compams_state("e").any()     # d_i = 1: the compressor is the identity
    p.close()


@pytest.mark.parametrize("n,d,offsets", [
    (3, 5000, [0, 1, 11, 500, 2548, 5000]),
    (2, 100003, "ragged40"),
    (2, 9000, "unit"),
    (2, 50000, "one"),
    (3, 33000, "ragged2000"),
    (2, 4101, [0, 4094, 4099, 4101]),
])
def test_blocksign_deferred_residual(n, d, offsets):
    """For layouts other than block = chunk the residual e = x - sign(x) mu of a step is applied by the next
    step's first pass (or when e is asked for).  Sign words, scales and parameters are compared after every
    step, the residuals after the 4th step (which settles them: the 5th step then takes the other variant of
    the first pass) and at the end."""
    rng = np.random.default_rng(d + 1)
    if offsets == "ragged40":
        off = ragged_offsets(d, rng, 40)
    elif offsets == "ragged2000":
        off = ragged_offsets(d, rng, 2000)
    elif offsets == "unit":
        off = np.arange(d + 1, dtype=np.int64)
    elif offsets == "one":
        off = np.array([0, d], dtype=np.int64)
    else:
        off = np.array(offsets, dtype=np.int64)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32) * 0.1, B.BLOCKSIGN, block_offsets=off)
    steps = 8
    for t in range(steps):
        g = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-3, 1, (1, d))).astype(np.float32)
        g[:, ::11] = 0.0
        p.step(g, 1e-3, label=f"deferred block-sign {offsets} step {t}", with_e=(t == 3 or t == steps - 1))
    assert all(p.exact.values()), p.exact
    assert np.array_equal(p.gpu.e[:, :d].cpu().numpy().view(np.uint32), p.cpu.get("e").view(np.uint32))
    p.close()


@pytest.mark.parametrize("cached", [0, 3, 4])
@pytest.mark.parametrize("n", [1, 8, 9, 17, 40])
def test_blocksign_server_kernel_shares(n, cached):
    """The server kernel gives a wavefront a share of two of a chunk's rounds and fetches each worker's sign words of
    the share once, sixteen workers per trip; shares that meet a block's or the row's end go round by round, eight
    workers at a time.  Worker counts around the trip sizes, block ends on and off the shares' and the sign words'
    boundaries, a last chunk that is partial, the state accessed in every way (none, some, all arrays kept cached)."""
    d = 5 * 4096 + 777
    rng = np.random.default_rng(n * 10 + cached)
    off = np.array([0, 512, 1024 + 32, 4096, 2 * 4096 + 1, 3 * 4096 + 1024, 4 * 4096 + 2048 - 5, d], dtype=np.int64)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32) * 0.1, B.BLOCKSIGN, block_offsets=off)
    p.gpu.set_option(B.OPT_CACHED_ARRAYS, cached)
    for t in range(4):
        g = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-3, 0, (n, 1))).astype(np.float32)
        p.step(g, 1e-3, label=f"shares n={n} cached={cached} step {t}", with_e=(t == 3))
    assert all(p.exact[s] for s in ("theta", "m", "v", "vhat"))
    p.close()


def test_blocksign_deferred_residual_with_a_block_that_is_not_finite():
    """An infinite entry makes its block's mean infinite; the residual of that block (x - sign(x) * inf) is then
    -inf, +inf or NaN, and the deferred form must produce the same pattern as the oracle's immediate one."""
    n, d = 2, 30000
    rng = np.random.default_rng(4)
    off = np.array([0, 100, 9000, 9001, 20000, d], dtype=np.int64)
    p = Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=off)
    for t in range(4):
        g = rng.standard_normal((n, d)).astype(np.float32)
        if t == 1:
            g[0, 12345] = np.inf
            g[1, 50] = -np.inf
        p.step(g, 1e-3, label=f"non-finite block step {t}", with_e=(t == 3))
    p.close()


def test_blocksign_with_nans_in_the_gradients():
    """A NaN makes its block's mean a NaN (whatever else the block holds, an infinity included) and codes as +1;
    the block's residuals and parameters are NaNs from then on, on both sides, and the other blocks go on bit
    for bit.  NaNs of either sign and with a payload, in one-coordinate, small and large blocks."""
    n, d = 3, 50000
    rng = np.random.default_rng(41)
    off = np.array([0, 1000, 1004, 20000, 20001, 40960, d], dtype=np.int64)
    p = Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=off)
    for t in range(7):
        g = rng.standard_normal((n, d)).astype(np.float32)
        if t in (2, 4):
            g[0, 1001] = np.nan
            g[1, 20000] = -np.nan
            g[0, 45000] = np.uint32(0xFFC12345).view(np.float32)
            g[2, 45001] = np.inf
        with np.errstate(invalid="ignore"):
            p.step(g, 1e-3, label=f"NaN blocks step {t}", with_e=(t in (3, 6)))
    mu = p.cpu.get("mu")
    assert np.isnan(mu[0, [1, 5]]).all() and np.isnan(mu[1, 3]) and np.isfinite(mu[:, [0, 2, 4]]).all()
    p.close()


def test_blocksign_wide_dynamic_range_is_summed_exactly():
    """Magnitudes from denormal to 1e30 in one block: any accumulation that is not exact gets the scale wrong."""
    n, d = 2, 40000
    rng = np.random.default_rng(1)
    off = np.array([0, 10000, 10001, 30000, d], dtype=np.int64)
    p = Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=off)
    for t in range(3):
        g = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-44, 30, (n, d))).astype(np.float32)
        g[0, :10000] = 0.0                    # an all-zero block: scale 0, stays zero
        p.step(g, 1e-3, label=f"wide range step {t}")
    assert not p.gpu.compams_state("e")[0, :10000].any()
    p.close()


@pytest.mark.parametrize("late_exp", [-3, 0, 2, 3, 9, 40])
def test_blocksign_sums_around_the_register_windows(late_exp):
    """The exact block sum runs, inside a lane, over two windows of binary exponents placed by the first entries
    a wavefront meets.  Here the first 256 coordinates of each block are about 1.0 and later ones sit on, just
    inside and far outside the window edges (powers of two from 2^-45 up to 2^late_exp, denormals, zeros, a few
    entries that share mantissa bits across the whole 24-bit width): every route into the sum must agree with the
    oracle to the last bit of the scale."""
    n, d = 2, 3 * 4096 + 123
    rng = np.random.default_rng(100 + late_exp)
    off = np.array([0, 4096 + 17, d], dtype=np.int64)
    p = Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=off)
    for t in range(3):
        g = np.empty((n, d), np.float32)
        exps = rng.integers(-45, late_exp + 1, size=(n, d))
        mant = 1.0 + rng.integers(0, 1 << 23, size=(n, d)) / float(1 << 23)         # full-width mantissas
        g[:] = (np.ldexp(mant, exps) * rng.choice([-1.0, 1.0], size=(n, d))).astype(np.float32)
        for lo in off[:-1]:
            g[:, lo:lo + 256] = (1.0 + rng.random((n, 256))).astype(np.float32)       # what places the windows
        g[:, 700::97] = 0.0
        g[:, 701::193] = np.float32(1e-45)                                            # the smallest denormal
        g[:, 702::389] = np.float32(2.0 ** -126)
        g[0, 5000] = np.float32(2.0 ** (late_exp + 1)) * np.float32(1.9999999)        # above everything else
        p.step(g, 1e-3, label=f"windows late_exp={late_exp} step {t}", with_e=(t == 2))
    assert all(p.exact.values()), p.exact
    p.close()


def test_blocksign_4096_blocks_of_every_kind():
    """Blocks of exactly one chunk: ordinary ones beside a block whose entries span 74 decades (far outside any
    register window), an empty block, a block with one tiny entry and a block of denormals."""
    n, d = 3, 10 * 4096 + 1000
    rng = np.random.default_rng(6)
    off = np.concatenate([np.arange(0, d, 4096), [d]]).astype(np.int64)
    p = Pair(n, d, np.zeros(d, np.float32), B.BLOCKSIGN, block_offsets=off)
    for t in range(4):
        g = rng.standard_normal((n, d)).astype(np.float32)
        g[:, 4096:2 * 4096] *= (10.0 ** rng.uniform(-44, 30, (n, 4096))).astype(np.float32)   # wide block
        g[:, 3 * 4096:4 * 4096] = 0.0                                                            # empty block
        g[:, 5 * 4096 + 7] = 1e-30                                                               # one tiny entry
        g[1, 8 * 4096:9 * 4096] *= 1e-38                                                         # denormal block
        p.step(g, 1e-3, label=f"4096 mixed step {t}")
    assert all(p.exact.values()), p.exact
    p.close()


def test_blocksign_is_deterministic():
    n, d = 3, 120000
    off = np.concatenate([np.arange(0, d, 30011), [d]]).astype(np.int64)
    gs = rand_grads(4, n, d, 4)
    res = []
    for rep in range(2):
        gpu = B.Compams(n, d, torch.zeros(d), compressor=B.BLOCKSIGN, block_offsets=off)
        for g in gs:
            gp = torch.zeros((n, gpu.ld)); gp[:, :d] = torch.from_numpy(g)
            gpu.compams_step(gp.cuda(), 1e-3)
        torch.cuda.synchronize()
        res.append([gpu.compams_state(s).cpu().numpy().copy()
                    for s in ("theta", "m", "v", "vhat", "e", "last_signbits", "last_scales")])
        gpu.close()
    for a, b in zip(*res):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


# ------------------------------------------------------------------------------------------- top-k per block
@pytest.mark.parametrize("n,d,blocks", [(3, 40000, 7), (2, 100000, 30), (5, 8192, 2), (2, 4 * 4096, 4096)])
def test_topk_per_block_composition(n, d, blocks):
    """Top-k inside every block, as one context per block laid over slices of shared buffers, against the oracle's
    per-block compressor: lists, values, parameters, moments and residuals bit for bit."""
    rng = np.random.default_rng(d + blocks)
    cuts = np.sort(rng.choice(np.arange(1, d // 4), size=blocks - 1, replace=False)) * 4
    off = np.concatenate([[0], cuts, [d]]).astype(np.int64)
    kb = np.maximum(1, ((off[1:] - off[:-1]) * 0.03).astype(np.int64))
    theta0 = rng.standard_normal(d).astype(np.float32) * 0.1
    gpu = CompamsBlockTopk(n, d, torch.from_numpy(theta0), off, kb)
    cpu = O.Oracle(n, d, theta0, compressor=O.TOPK_BLOCKS, block_offsets=off, block_k=kb)
    for t in range(5):
        g = (rng.standard_normal((n, d)) * 10.0 ** rng.uniform(-3, 0, (1, d))).astype(np.float32)
        g[:, ::6] = 0.0
        gp = torch.zeros((n, gpu.ld), dtype=torch.float32)
        gp[:, :d] = torch.from_numpy(g)
        gpu.compams_step(gp.to(gpu.device), 1e-3)
        cpu.step(g, 1e-3)
        torch.cuda.synchronize()
        assert np.array_equal(gpu.compams_state("last_idx").cpu().numpy(), cpu.get("idx")), f"step {t}: lists"
        assert np.array_equal(gpu.compams_state("last_val").cpu().numpy().view(np.uint32), cpu.get("val").view(np.uint32))
        for name in ("theta", "m", "v", "vhat") + (("e",) if t == 4 else ()):
            got = np.ascontiguousarray(gpu.compams_state(name).cpu().numpy())
            assert np.array_equal(got.view(np.uint32), cpu.get(name).view(np.uint32)), f"step {t}: {name}"
    gpu.close(); cpu.close()


def test_topk_per_block_needs_aligned_blocks():
    with pytest.raises(B.CompamsError):
        CompamsBlockTopk(2, 100, torch.zeros(100), [0, 50, 100], [1, 1])     # 50 is not a multiple of 4


# ------------------------------------------------------------------------------------------- identity
@pytest.mark.parametrize("n,d", [(4, 65536), (3, 10001), (16, 5), (37, 20001)])
def test_identity_compressor(n, d):
    rng = np.random.default_rng(d)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32) * 0.1, B.NONE)
    run_pair(p, rand_grads(d, n, d, 10, scale=0.3), label="none")
    assert all(p.exact[s] for s in ("theta", "m", "v", "vhat"))
    p.close()


@pytest.mark.parametrize("compressor", ["topk", "blocksign", "none"])
@pytest.mark.parametrize("beta1,beta2,eps,eps_mode", [
    (0.0, 0.0, 1e-3, B.EPS_IN_SQRT),          # no memory at all: m is the average, v its square
    (0.5, 0.9, 0.0, B.EPS_OUT_SQRT),          # no epsilon: the quotient alone
    (0.99, 0.9999, 1e-12, B.EPS_IN_SQRT),
    (0.9, 0.999, 0.5, B.EPS_OUT_SQRT),        # an epsilon that dominates the root
])
def test_hyper_parameters_away_from_the_defaults_and_a_learning_rate_that_changes(compressor, beta1, beta2, eps, eps_mode):
    """The moment and parameter lines of Algorithm 2 with other constants than the experiments' (Section 5.1),
    and a learning rate that differs from step to step (zero, negative and large ones among them): it is an
    argument of each step, not part of the context."""
    n, d = 3, 3 * 4096 + 99
    rng = np.random.default_rng(int(beta1 * 100) + 7)
    kw = {"topk": dict(k=300), "blocksign": dict(block_offsets=np.array([0, 5, 4096, 9000, d], np.int64)), "none": {}}[compressor]
    comp = {"topk": B.TOPK, "blocksign": B.BLOCKSIGN, "none": B.NONE}[compressor]
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32) * 0.1, comp, beta1=beta1, beta2=beta2, eps=eps,
             eps_mode=eps_mode, **kw)
    for t, lr in enumerate([1e-3, 0.0, 0.25, -1e-2, 3e-5, 10.0, 1e-3]):
        g = (rng.standard_normal((n, d)) * 0.3 + 0.01).astype(np.float32)
        p.step(g, lr, label=f"{compressor} b1={beta1} b2={beta2} eps={eps} lr={lr} step {t}")
    assert all(p.exact[s] for s in ("theta", "m", "v", "vhat"))
    p.close()


def test_identity_compressor_with_infinite_gradients():
    """Algorithm 1 has no residual: an infinite entry of one worker's gradient makes that coordinate's average,
    m and v infinite and its parameter a NaN, and they stay so (beta * Inf + finite); the library keeps e at
    zero.  The oracle's literal error line of Algorithm 2 (x - x in fp32) leaves a NaN there instead, which the
    next step carries into m and v, so those coordinates are checked against the closed form and all the others
    against the oracle, bit for bit."""
    n, d = 3, 30000
    rng = np.random.default_rng(15)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32) * 0.1, B.NONE)
    pos, neg, nan = [7, 4096, d - 1], [8, 20000], [100, 9000]
    special = np.array(pos + neg + nan)
    rest = np.setdiff1d(np.arange(d), special)
    for t in range(6):
        g = (rng.standard_normal((n, d)) * 0.3).astype(np.float32)
        if t == 2:
            g[1, pos] = np.inf
            g[2, neg] = -np.inf
            g[0, nan] = np.nan
        with np.errstate(invalid="ignore", over="ignore"):
            p.step(g, 1e-3, check=False)
        torch.cuda.synchronize()
        got = {s: p.gpu.compams_state(s).cpu().numpy() for s in ("theta", "m", "v", "vhat")}
        for s, a in got.items():
            assert bits_equal(a[rest], p.cpu.get(s)[rest]), f"step {t}: {s} away from the special entries"
        if t >= 2:
            assert (got["m"][pos] == np.inf).all() and (got["m"][neg] == -np.inf).all(), got["m"][special]
            assert (got["v"][pos + neg] == np.inf).all() and (got["vhat"][pos + neg] == np.inf).all()
            assert np.isnan(got["theta"][special]).all()
            assert np.isnan(got["m"][nan]).all() and np.isnan(got["v"][nan]).all()
    assert p.gpu.e is None            # no residual array exists for this compressor
    p.close()


def test_degenerate_compressors_are_the_identity():
    """Top-k with k = d and block-sign with one coordinate per block keep everything (the compressors with q = 0
    of Remark 1): the step then is distributed AMSGrad without compression, bit for bit, and e stays zero."""
    n, d, steps = 3, 20003, 5
    rng = np.random.default_rng(77)
    theta0 = torch.from_numpy(rng.standard_normal(d).astype(np.float32) * 0.1)
    gs = rand_grads(78, n, d, steps, scale=0.5)
    for g in gs:
        g[:, ::7] = 0.0
    ctxs = {
        "none": B.Compams(n, d, theta0.clone(), compressor=B.NONE),
        "topk": B.Compams(n, d, theta0.clone(), compressor=B.TOPK, k=d),
        "blocksign": B.Compams(n, d, theta0.clone(), compressor=B.BLOCKSIGN,
                               block_offsets=np.arange(d + 1, dtype=np.int64)),
    }
    for g in gs:
        for c in ctxs.values():
            gp = torch.zeros((n, c.ld), dtype=torch.float32)
            gp[:, :d] = torch.from_numpy(g)
            c.compams_step(gp.to(c.device), 1e-3)
    ref = {s: ctxs["none"].compams_state(s).cpu().numpy() for s in ("theta", "m", "v", "vhat")}
    for name in ("topk", "blocksign"):
        for s, want in ref.items():
            got = ctxs[name].compams_state(s).cpu().numpy()
            assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), (name, s)
        assert not ctxs[name].compams_state("e")[:, :d].any(), name
    for c in ctxs.values():
        c.close()


# ------------------------------------------------------------------------------------------- hand-derived case
@pytest.mark.parametrize("eps_mode,key", [(B.EPS_IN_SQRT, "theta_eps_in"), (B.EPS_OUT_SQRT, "theta_eps_out")])
def test_worked_example_on_gpu(eps_mode, key):
    with open(os.path.join(HERE, "golden", "worked_example_d8.json")) as f:
        G = json.load(f)
    for comp, part in ((B.TOPK, G["topk"]), (B.BLOCKSIGN, G["blocksign"])):
        kw = dict(k=part["k"]) if comp == B.TOPK else dict(block_offsets=part["block_offsets"])
        gpu = B.Compams(G["n"], G["d"], torch.tensor(G["theta1"], dtype=torch.float32), compressor=comp,
                        eps_mode=eps_mode, **kw)
        for t in range(2):
            gpu.compams_step(torch.tensor(G["g"][t], dtype=torch.float32).cuda(), G["lr"])
            torch.cuda.synchronize()
            assert np.array_equal(gpu.compams_state("e").cpu().numpy(), np.array(part["e"][t], np.float32))
            np.testing.assert_allclose(gpu.compams_state("theta").cpu().numpy(), part[key][t], rtol=2e-6, atol=0)
            if comp == B.TOPK:
                assert gpu.compams_state("last_idx").cpu().tolist() == part["idx"][t]
            else:
                assert np.array_equal(gpu.compams_state("last_scales").cpu().numpy(), np.array(part["mu"][t], np.float32))
                bits = gpu.compams_state("last_signbits").cpu().numpy()[:, 0]
                assert [[(int(bits[i]) >> j) & 1 for j in range(8)] for i in range(2)] == part["neg"][t]
        gpu.close()


# ------------------------------------------------------------------------------------------- resume
def test_keep_state_resumes_bit_exactly():
    n, d, k = 2, 30000, 300
    gs = rand_grads(21, n, d, 6)
    a = B.Compams(n, d, torch.zeros(d), compressor=B.TOPK, k=k)
    for g in gs[:3]:
        gp = torch.zeros((n, a.ld)); gp[:, :d] = torch.from_numpy(g); a.compams_step(gp.cuda(), 1e-3)
    st = {s: a.compams_state(s).clone() for s in ("m", "v", "vhat", "e")}
    b = B.Compams(n, d, a.compams_state("theta").clone(), compressor=B.TOPK, k=k, state=st)
    for g in gs[3:]:
        gp = torch.zeros((n, a.ld)); gp[:, :d] = torch.from_numpy(g)
        a.compams_step(gp.cuda(), 1e-3); b.compams_step(gp.cuda(), 1e-3)
    torch.cuda.synchronize()
    for s in ("theta", "m", "v", "vhat", "e", "last_idx"):
        assert torch.equal(a.compams_state(s), b.compams_state(s)), s
    a.close(); b.close()


# ------------------------------------------------------------------------------------------- long runs
@pytest.mark.parametrize("compressor", ["topk", "blocksign", "topk_blocks"])
def test_hundred_steps_with_a_drifting_gradient_scale(compressor):
    """A long run whose gradient scale decays, now and then jumps by a decade either way, and whose rows differ in
    scale: the carried-over threshold guesses go stale again and again, the pending residual updates are applied a
    hundred times, and everything still has to agree with the oracle after every tenth step (the lists and sign
    words at every step they are looked at, the state bit for bit at the end)."""
    n, d = 4, 3 * 4096 * 5 + 8
    rng = np.random.default_rng(77)
    theta0 = (rng.standard_normal(d) * 0.1).astype(np.float32)
    off = np.array([0, 4096 * 4, 4096 * 4 + 1000, 4096 * 11, d], dtype=np.int64)
    if compressor == "topk_blocks":
        from test_gpu_topk_blocks import BlockPair
        p = BlockPair(n, d, off, np.array([160, 10, 290, 200], dtype=np.int64), theta0)
    elif compressor == "topk":
        p = Pair(n, d, theta0, B.TOPK, k=600)
    else:
        p = Pair(n, d, theta0, B.BLOCKSIGN, block_offsets=off)
    scale = 1.0
    rows = (10.0 ** rng.uniform(-1, 1, (n, 1)))
    rereads = 0
    for t in range(100):
        scale *= 0.97
        if t % 13 == 12:
            scale *= 10.0 ** rng.choice([-1.0, 1.0])
        g = (rng.standard_normal((n, d)) * scale * rows).astype(np.float32)
        look = t % 10 == 9
        if compressor == "topk_blocks":
            p.step(g)
            if look:
                p.compare(f"step {t}", with_e=(t == 99))
        else:
            p.step(g, 1e-3, check=look, label=f"{compressor} step {t}", with_e=(t == 99))
        if compressor != "blocksign":
            torch.cuda.synchronize()
            rereads += int((p.gpu.compams_state("counters").cpu().numpy().reshape(-1, B.COUNTERS_PER_ROW)[:, 0] > 0).sum())
    if compressor == "topk":
        assert all(p.exact.values()), p.exact
    if compressor != "blocksign":
        assert rereads > 0, "the jumps in scale should have made some guesses fail"
    p.close()


def test_inplace_probe_adds_one_to_every_element_and_nothing_else():
    """The measurement aid for the server's lines: values are exact, the ragged last workgroup stops at count."""
    for count, arrays in ((4096 * 3 + 20, 4), (8, 1), (4096, 3), (70000, 2)):
        for cached in range(5):
            bufs = [torch.arange(count + 8, dtype=torch.float32, device="cuda") * (a + 1) for a in range(arrays)]
            B.compams_inplace_probe([b[:count] for b in bufs], cached)
            torch.cuda.synchronize()
            for a, b in enumerate(bufs):
                want = torch.arange(count + 8, dtype=torch.float32) * (a + 1)
                want[:count] += 1.0
                assert torch.equal(b.cpu(), want), (count, arrays, cached, a)


@pytest.mark.parametrize("cached", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("case", ["topk", "topk_blocks", "blocksign", "none", "split"])
def test_every_count_of_cached_state_arrays_gives_the_same_bytes(case, cached):
    """The server kernels exist in five forms (0..4 of theta, m, v, vhat kept in the memory-side cache, the others
    streamed); the library picks one by size, so small problems would only ever run one of them.  Forced here:
    each form against the oracle, for every compressor and for the server half of a split step."""
    n, d = 5, 3 * 4096 + 1234
    rng = np.random.default_rng(100 + cached)
    theta0 = (rng.standard_normal(d) * 0.1).astype(np.float32)
    off = np.array([0, 400, 4096 + 8, 2 * 4096 + 100, d], dtype=np.int64)
    gs = rand_grads(7, n, d, 5, scale=0.3)
    if case == "split":
        k = d // 50
        wk = B.Compams(n, d, torch.from_numpy(theta0), compressor=B.TOPK, k=k)
        sv = B.Compams(n, d, torch.from_numpy(theta0), compressor=B.TOPK, k=k)
        sv.set_option(B.OPT_CACHED_ARRAYS, cached)
        cpu = O.Oracle(n, d, theta0, compressor=O.TOPK, k=k)
        for t, g in enumerate(gs):
            gp = torch.zeros((n, wk.ld), dtype=torch.float32)
            gp[:, :d] = torch.from_numpy(g)
            wk.compams_worker_step(gp.to(wk.device))
            msgs, words = wk.compams_encode()
            sv.compams_server_step(msgs, words, 1e-3)
            cpu.step(g, 1e-3)
            torch.cuda.synchronize()
            for name in ("theta", "m", "v", "vhat"):
                assert bits_equal(sv.compams_state(name).cpu().numpy(), cpu.get(name)), f"{name} after step {t}"
        wk.close(); sv.close(); cpu.close()
        return
    if case == "topk_blocks":
        from test_gpu_topk_blocks import BlockPair
        kb = np.maximum(1, (off[1:] - off[:-1]) // 40)
        p = BlockPair(n, d, off, kb, theta0)
        p.gpu.set_option(B.OPT_CACHED_ARRAYS, cached)
        for t, g in enumerate(gs):
            p.step(g)
            p.compare(f"blocks, {cached} cached, step {t}", with_e=(t == len(gs) - 1))
        p.gpu.close(); p.cpu.close()
        return
    kw = {"topk": dict(k=d // 50), "blocksign": dict(block_offsets=off), "none": {}}[case]
    comp = {"topk": B.TOPK, "blocksign": B.BLOCKSIGN, "none": B.NONE}[case]
    p = Pair(n, d, theta0, comp, **kw)
    for bad in (-2, 5):
        with pytest.raises(B.CompamsError):
            p.gpu.set_option(B.OPT_CACHED_ARRAYS, bad)
    p.gpu.set_option(B.OPT_CACHED_ARRAYS, -1)   # the library's own choice: allowed for every compressor
    p.gpu.set_option(B.OPT_CACHED_ARRAYS, cached)
    run_pair(p, gs, label=f"{case}, {cached} cached")
    assert all(p.exact[s] for s in ("theta", "m", "v", "vhat"))
    p.close()


@pytest.mark.parametrize("n,d,blocks", [(3, 64 * 4096, 64), (2, 64 * 4096 + 4, 64), (2, 64 * 4096, 65), (5, 9001, 1), (1, 37, 37),
                                        (33, 4096, 3), (2, 250_001, 2),
                                        # one set of digits: up to 8 chunks, else 128 workgroups; several: 16, else 512
                                        (2, 64 * 4096, 64), (17, 8 * 4096, 8), (15, 8 * 4096 + 5, 9), (14, 9 * 4096, 9),
                                        (33, 16 * 4096, 2), (8, 64 * 4096, 2), (9, 64 * 4096 - 7, 2), (31, 17 * 4096, 1)])
def test_blocksign_scales_of_short_rows(n, d, blocks):
    """Of short rows in small grids the row's last workgroup forms the scales, else a launch of its own (never the
    former beyond 64 chunks or blocks): the same sums, cleared for the next step, with entries that miss the register
    windows and a block that is not finite."""
    rng = np.random.default_rng(d + blocks)
    cuts = np.sort(rng.choice(np.arange(1, d), size=blocks - 1, replace=False))
    off = np.concatenate([[0], cuts, [d]]).astype(np.int64)
    p = Pair(n, d, rng.standard_normal(d), B.BLOCKSIGN, block_offsets=off)
    for t in range(4):
        g = (rng.standard_normal((n, d)) * 2.0 ** rng.integers(-40, 3, size=(n, d))).astype(np.float32)
        if t == 2 and blocks > 2:
            g[0, off[1]] = np.inf
        with np.errstate(all="ignore"):
            p.step(g, 1e-3, label=f"short row {d} x {blocks} step {t}", with_e=t == 3)
    assert all(p.exact.values()), p.exact
    p.close()


def blocksign_step_us(n, chunks, blocks):
    d = chunks * 4096
    c = B.Compams(n, d, torch.zeros(d), compressor=B.BLOCKSIGN,
                  block_offsets=np.linspace(0, d, blocks + 1).astype(np.int64))
    g = torch.randn((n, c.ld), device=c.device)
    times = []
    for _ in range(9):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(40):
            c.compams_step(g, 1e-3)
        end.record()
        torch.cuda.synchronize()
        times.append(begin.elapsed_time(end) / 40 * 1e3)
    c.close()
    return sorted(times)[4]


def test_forming_the_scales_in_the_first_pass_is_not_the_slower_way():
    """64 rows of 64 and of 65 chunks, a block per chunk: the longer ones always have a launch of its own for the scales.  With the
    row's last workgroup forming them the shorter ones took 68 us against 53."""
    assert blocksign_step_us(64, 64, 64) < 1.12 * blocksign_step_us(64, 65, 65)
