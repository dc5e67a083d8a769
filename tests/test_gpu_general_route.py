"""The general route in one launch and in four, on both sides of the line (4096 chunks in all rows): steps in which all, some or none
of the rows miss their window, with lists and without, whole rows and blocks, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from paper_2205_05632_amd import binding as B

from parity import Pair
from test_gpu_topk_blocks import BlockPair, make_blocks

pytestmark = pytest.mark.gpu
CHUNK = 4096
GENERAL = ("topk_general", "topk_level0", "topk_level1", "topk_level2", "topk_count")


def went(c):
    """Per problem: whether it took the general route in the last step, and whether from the list that the first pass had made."""
    counters = c.compams_state("counters").cpu().numpy().reshape(-1, 8)
    missed = counters[:, 5] != 0
    return missed, missed & (counters[:, 0] == 0)


def provoked(kind, steps, alone=False):
    """Whether the steps (from the third on, where there are windows) took the ways that the kind of gradient is there for."""
    if kind == "steady":
        return not any(missed.any() for missed, _ in steps)
    if kind == "some":  # in one step rows inside their windows and rows outside whose lists held (one row: one after the other)
        return any(listed.any() and (alone or not missed.all()) for missed, listed in steps)
    if kind == "jump":  # all of them, and lists that did not hold
        return any((missed & ~listed).all() for missed, listed in steps)
    return any(missed.any() for missed, _ in steps)


def gradients(kind, base, t, n, d):
    g = np.stack([np.roll(base, 1013 * t + 41 * i) for i in range(n)])
    if kind == "jump":        # up and down tenfold: lists that overflow, lists with too few entries
        g *= np.float32(10.0 ** (t % 2))
    elif kind == "some":      # every third row, by a little: listed, but outside its window, and more than three buckets up
        g[t % 3::3] *= np.float32(1.0 + 0.3 * (t % 4))
    elif kind == "levels":    # few magnitudes: the threshold's bucket holds most of the row
        g = np.round(g * 2) / 2
    elif kind == "equal":     # one magnitude: no list fits
        g = np.where(g < 0, np.float32(-1), np.float32(1))
    return np.ascontiguousarray(g, dtype=np.float32)


@pytest.mark.parametrize("kind", ["steady", "jump", "some", "levels", "equal"])
@pytest.mark.parametrize("n,d,k", [(3, 17 * CHUNK + 1, 700), (2, 64 * CHUNK, 2000), (64, 64 * CHUNK, 2600), (17, 241 * CHUNK, 9000),
                                   (1, 1000 * CHUNK - 5, 40000)])
def test_whole_rows(n, d, k, kind):
    rng = np.random.default_rng(d + n)
    base = rng.standard_normal(d).astype(np.float32)
    p = Pair(n, d, rng.standard_normal(d).astype(np.float32), B.TOPK, k=k)
    steps, missed, counters = 7, 0, None
    for t in range(steps):
        p.step(gradients(kind, base, t, n, d), 1e-3, label=f"{kind} {n} x {d} step {t}", with_e=t == steps - 1, check=t % 2 == 0 or n < 10)
        counters = p.gpu.compams_state("counters").cpu().numpy()
        missed += int((counters[:, 5] != 0).sum()) if t > 2 else 0
    p.compare(f"{kind} {n} x {d}")
    assert missed > 0 or kind in ("steady", "some"), "no row took the general route"
    assert all(p.exact.values()), p.exact
    p.close()


@pytest.mark.parametrize("kind", ["steady", "jump", "some", "levels"])
@pytest.mark.parametrize("n,d,blocks", [(3, 70000, 9), (8, 400000, 30), (40, 103 * CHUNK, 6)])
def test_blocks(n, d, blocks, kind):
    rng = np.random.default_rng(d)
    off, kb = make_blocks(d, blocks, rng)
    base = rng.standard_normal(d).astype(np.float32)
    p = BlockPair(n, d, off, kb, np.zeros(d, dtype=np.float32))
    for t in range(6):
        p.step(gradients(kind, base, t, n, d))
        if t % 2:
            p.compare(f"{kind} {n} x {d} step {t}", with_e=t == 5)


@pytest.mark.parametrize("blocks", [0, 3])
@pytest.mark.parametrize("n,d", [(4, 80 * CHUNK), (1, 257 * CHUNK - 3), (16, 20 * CHUNK + 1)])
def test_lists_made_again(n, d, blocks):
    """The corrected gradients themselves shrink and grow tenfold.  Where they have shrunk no list holds: level 1 makes them all again
    from the rows, about one entry to a chunk, so that many workgroups write parts of one line of the list that the next parts read."""
    rng = np.random.default_rng(d)
    off = np.array([d * b // blocks // 4 * 4 for b in range(blocks)] + [d], dtype=np.int64) if blocks else None
    kept = d // CHUNK
    if blocks:
        p = BlockPair(n, d, off, np.full(blocks, max(1, kept // blocks), dtype=np.int64), np.zeros(d, dtype=np.float32))
    else:
        p = Pair(n, d, np.zeros(d), B.TOPK, k=kept)
    for t in range(6):
        x = rng.standard_normal((n, d)).astype(np.float32) * np.float32(10.0 ** -(t % 2))
        p.step(x - p.cpu.get("e") if t else x, 1e-3)
        counters = p.gpu.compams_state("counters").cpu().numpy().reshape(-1, 8)
        p.compare(f"{n} x {d} step {t}", with_e=t == 5)
        if t > 1 and t % 2:
            assert (counters[:, 0] == 1).all() and (counters[:, 5] != 0).all(), (t, counters)
    p.close()


def test_threshold_that_rises():
    """The corrected gradients grow by 30 %: the list holds, but the threshold's bucket lies above the ones that level 0 keeps histograms
    of.  All workgroups sweep the list for it, in one launch (51 us) as in four (52); by one workgroup alone it took 277."""
    n, d, k = 1, 1000 * CHUNK - 5, 200_000
    rng = np.random.default_rng(3)
    pairs = {band: Pair(n, d, np.zeros(d), B.TOPK, k=k) for band in (1, 0)}
    pairs[0].gpu.set_option(B.OPT_BAND, 0)  # four launches
    us = {1: [], 0: []}
    scale, buckets = np.float32(1), 0
    for t in range(16):
        rises = t % 4 == 3
        if rises:
            scale *= np.float32(1.3)
        x = rng.standard_normal((n, d)).astype(np.float32) * scale
        for band, p in pairs.items():
            p.gpu.profile_enable(1)
            p.step(x - p.cpu.get("e") if t else x, 1e-3, label=f"step {t}", with_e=False)
            times = p.gpu.profile_read()
            p.gpu.profile_enable(0)
            if rises:
                c = p.gpu.compams_state("counters").cpu().numpy().reshape(-1, 8)
                assert c[0, 0] == 0 and c[0, 5] == (4 if band else 1), c
                us[band].append(sum(ms for name, (ms, _) in times.items() if name in GENERAL) * 1e3)
        tau = int(pairs[1].gpu.compams_state("last_threshold").cpu().numpy().view(np.uint32)[0]) >> 19
        assert not rises or tau >= buckets + 3, (tau, buckets)  # (the guess lies a bucket below the last threshold's, or at it)
        buckets = tau
    assert min(us[1]) < 1.5 * min(us[0]), us
    for p in pairs.values():
        p.close()


@pytest.mark.parametrize("n,d,k,one,cap", [
    (2, 80 * CHUNK, 32 * CHUNK, True, 0), (2, 80 * CHUNK, 32 * CHUNK + 1, False, 0),    # two fifths of a row
    (16, 80 * CHUNK, 16 * CHUNK, True, 0), (16, 80 * CHUNK, 16 * CHUNK + 1, False, 0),  # 2^20 entries of all rows
    (64, 64 * CHUNK, 2600, True, 0), (64, 64 * CHUNK + 1, 2600, False, 0),              # 4096 chunks
    (4, 80 * CHUNK, 2000, True, 5000), (4, 80 * CHUNK, 2000, False, 4999)])             # two fifths of a list
def test_which_form(n, d, k, one, cap):
    """Steps that keep much take the route every time, and its four launches: 16 x 1 M, k = d / 2, 201 us, in one launch 248."""
    rng = np.random.default_rng(k)
    p = Pair(n, d, np.zeros(d), B.TOPK, k=k)
    if cap:
        p.gpu.set_option(B.OPT_CANDIDATE_CAP, cap)
    base = rng.standard_normal(d).astype(np.float32)
    for t in range(4):
        p.gpu.profile_enable(1)
        p.step(gradients("some", base, t, n, d), 1e-3, label=f"step {t}", with_e=False)
        used = {name for name, (_, launches) in p.gpu.profile_read().items() if launches}
        p.gpu.profile_enable(0)
        assert ("topk_general" in used) == (one and t > 0) and ("topk_level0" in used) == (not one or t == 0), (t, used)
    p.close()


def test_two_streams_at_a_time():
    """Two contexts whose rows all miss, on two streams at once: neither's tasks wait for the other's."""
    n, d, k = 4, 80 * CHUNK, 3000
    rng = np.random.default_rng(5)
    base = rng.standard_normal(d).astype(np.float32)
    theta = rng.standard_normal(d).astype(np.float32)
    pairs = [Pair(n, d, theta, B.TOPK, k=k) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in pairs]
    grads = [[torch.zeros((n, p.gpu.ld), device="cuda") for _ in range(2)] for p in pairs]
    for c, pair_grads in enumerate(grads):
        for t, g in enumerate(pair_grads):
            g[:, :d] = torch.from_numpy(gradients("jump", base, t + c, n, d)).cuda()
    torch.cuda.synchronize()
    for t in range(8):
        for p, s, g in zip(pairs, streams, grads):
            with torch.cuda.stream(s):
                p.gpu.compams_step(g[t % 2], 1e-3)
    torch.cuda.synchronize()
    for c, p in enumerate(pairs):
        for t in range(8):
            p.cpu.step(gradients("jump", base, t % 2 + c, n, d), 1e-3)
        p.compare(f"context {c}")
        p.close()


@pytest.mark.parametrize("kind", ["steady", "jump", "some", "levels"])
@pytest.mark.parametrize("n,d,k,blocks", [(3, 17 * CHUNK + 1, 700, 0), (17, 241 * CHUNK, 9000, 0), (1, 1000 * CHUNK - 5, 40000, 0),
                                          (3, 70000, 0, 9), (8, 400000, 0, 30)])
def test_ways_that_are_provoked(n, d, k, blocks, kind):
    """The kinds of gradient take, by the counters, the ways that they are there for."""
    rng = np.random.default_rng(d if blocks else d + n)
    if blocks:
        off, kb = make_blocks(d, blocks, rng)
        base = rng.standard_normal(d).astype(np.float32)
        c = B.Compams(n, d, torch.zeros(d), compressor=B.TOPK_BLOCKS, block_offsets=off, block_k=kb)
    else:
        base = rng.standard_normal(d).astype(np.float32)
        c = B.Compams(n, d, torch.from_numpy(rng.standard_normal(d).astype(np.float32)), compressor=B.TOPK, k=k)
    seen, grads = [], torch.zeros((n, c.ld), device="cuda")
    for t in range(7):
        grads[:, :d] = torch.from_numpy(gradients(kind, base, t, n, d)).cuda()
        c.compams_step(grads, 1e-3)
        seen.append(went(c))
    assert provoked(kind, seen[2:], alone=n == 1), seen
    c.close()


def test_two_streams_that_miss():
    """Two contexts on two streams, of which by the counters all rows take the general route in three steps at least."""
    n, d, k = 4, 80 * CHUNK, 3000
    rng = np.random.default_rng(5)
    base = rng.standard_normal(d).astype(np.float32)
    pairs = [Pair(n, d, np.zeros(d, dtype=np.float32), B.TOPK, k=k) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    grads = [[torch.zeros((n, p.gpu.ld), device="cuda") for _ in range(2)] for p in pairs]
    for c, pair_grads in enumerate(grads):
        for t, g in enumerate(pair_grads):
            g[:, :d] = torch.from_numpy(gradients("jump", base, t + c, n, d)).cuda()
    torch.cuda.synchronize()
    counters = [[], []]
    for t in range(8):
        for p, s, g, seen in zip(pairs, streams, grads, counters):
            with torch.cuda.stream(s):
                p.gpu.compams_step(g[t % 2], 1e-3)
                seen.append(p.gpu.compams_state("counters").clone())
    torch.cuda.synchronize()
    for c, p in enumerate(pairs):
        missed = [(m[:, 5] != 0).all().item() for m in counters[c][2:]]
        assert sum(missed) >= 3, missed
        for t in range(8):
            p.cpu.step(gradients("jump", base, t % 2 + c, n, d), 1e-3)
        p.compare(f"context {c}")
        p.close()
