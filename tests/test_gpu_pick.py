"""Rows short enough for the selection by one workgroup (16 chunks of 4096 coordinates; 17 take the other kernels): the
candidate list and the row itself as source, one and several histogram levels, up to and beyond 1024 entries left to
rank, ties cut off at a coordinate, infinities, NaNs and zeros.  Every output equals the oracle's bit for bit."""
import numpy as np
import pytest
import torch

from paper_2205_05632_amd import binding as B

from parity import Pair

pytestmark = pytest.mark.gpu


def values(kind, rng, n, d):
    g = rng.standard_normal((n, d)).astype(np.float32)
    if kind == "levels":            # few distinct magnitudes: many ties, some of them cut off
        g = (rng.integers(-2, 3, size=(n, d)) * 0.5).astype(np.float32)
    elif kind == "equal":           # one magnitude: everything is a tie
        g = np.where(g < 0, np.float32(-1.5), np.float32(1.5))
    elif kind == "narrow":          # all magnitudes within one histogram bucket of the first level
        g = (np.sign(g) * (1.0 + 1e-4 * np.abs(g))).astype(np.float32)
    elif kind == "wide":            # sixty binary orders of magnitude
        g = (g * 2.0 ** rng.integers(-30, 30, size=(n, d))).astype(np.float32)
    elif kind == "zeros":           # more zeros than there are entries to leave out
        g[:, rng.random(d) < 0.97] = 0.0
    elif kind == "special":
        g[:, ::97] = np.inf
        g[:, 5::101] = -np.inf
        g[:, 7::103] = np.nan
        g[:, 9::107] = np.float32(3.3e38)
    return g


@pytest.mark.parametrize("kind", ["normal", "levels", "equal", "narrow", "wide", "zeros", "special"])
@pytest.mark.parametrize("n,d,k", [(3, 16 * 4096, 655), (2, 16 * 4096 + 1, 655), (4, 9000, 4000), (1, 4095, 4095), (5, 1025, 1)])
def test_short_rows(kind, n, d, k):
    rng = np.random.default_rng(d + k)
    p = Pair(n, d, np.zeros(d), B.TOPK, k=k)
    for t in range(6):
        with np.errstate(all="ignore"):
            p.step(values(kind, rng, n, d), 1e-3, label=f"{kind} {d} step {t}", with_e=t in (2, 5))
        if t == 3:
            p.gpu.set_option(B.OPT_CANDIDATE_CAP, max(1, k // 2))   # from here on no list fits: the row itself
    assert all(p.exact.values()), p.exact
    p.close()


@pytest.mark.parametrize("d", [16 * 4096, 17 * 4096])
def test_the_two_selections_meet_at_sixteen_chunks(d):
    """Window and guess are the same bookkeeping on both sides of the line: steady steps are counted alike."""
    n, k = 3, 500
    rng = np.random.default_rng(d)
    p = Pair(n, d, np.zeros(d), B.TOPK, k=k)
    for t in range(12):
        p.step(rng.standard_normal((n, d)).astype(np.float32), 1e-3, label=f"{d} step {t}", with_e=False)
    torch.cuda.synchronize()
    c = p.gpu.compams_state("counters").cpu().numpy()
    assert (c[:, 0] == 0).all() and (c[:, 4] > 0).all() and (c[:, 5] == 0).all(), c
    p.close()


@pytest.mark.parametrize("option,value", [(B.OPT_PREDICT, 0), (B.OPT_FORCE_DENSE, 1), (B.OPT_BAND, 0)])
@pytest.mark.parametrize("kind", ["normal", "equal"])
def test_short_rows_with_options(kind, option, value):
    """Without a guess the general kernels take the row, in between steps that one workgroup per row has taken."""
    n, d, k = 3, 5 * 4096 + 8, 300
    rng = np.random.default_rng(option + value)
    p = Pair(n, d, np.zeros(d), B.TOPK, k=k)
    for t in range(9):
        if t in (3, 6):
            p.gpu.set_option(option, value if t == 3 else 1 - value)
        p.step(values(kind, rng, n, d), 1e-3, label=f"{kind} option {option} step {t}", with_e=t in (4, 8))
    assert all(p.exact.values()), p.exact
    p.close()


@pytest.mark.parametrize("listed", [True, False])
@pytest.mark.parametrize("ties", [255, 256, 257, 4000])
def test_ties_around_what_is_ranked(ties, listed):
    """The entries left in the threshold's bucket are ranked up to 256 of them; more are equal keys, cut at a coordinate.
    From the list, and from a row whose list does not fit."""
    n, d = 2, 16 * 4096
    k = 100 + ties // 2
    rng = np.random.default_rng(ties)
    p = Pair(n, d, np.zeros(d), B.TOPK, k=k)
    if not listed:
        p.gpu.set_option(B.OPT_CANDIDATE_CAP, 1)
    for t in range(4):
        g = (rng.standard_normal((n, d)) * 1e-3).astype(np.float32)
        for row in g:
            at = rng.choice(d, size=100 + ties, replace=False)
            row[at[:100]] = 64.0 + 4.0 * t
            row[at[100:]] = 16.0
        p.step(g, 1e-3, label=f"{ties} ties step {t}", with_e=t == 3)
    assert all(p.exact.values()), p.exact
    p.close()


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("left", [1, 2, 63, 64, 65, 255, 256, 257])
def test_entries_left_to_rank(left, ties):
    """Up to 64 are ranked by every wavefront for itself, up to 256 by the workgroup, beyond that there is one more histogram."""
    n, d, above = 2, 5000, 100
    rng = np.random.default_rng(left)
    p = Pair(n, d, np.zeros(d), B.TOPK, k=above + (left + 1) // 2)
    for t in range(5):
        g = (rng.standard_normal((n, d)) * 1e-6).astype(np.float32)
        for i in range(n):
            where = rng.permutation(d)[: above + left]
            g[i, where[:above]] = 10.0 + rng.random(above)
            step = np.zeros(left) if ties else np.arange(left)
            g[i, where[above:]] = np.float32(1.0) + step.astype(np.float32) * np.float32(2.0 ** -23)
        # what is kept leaves the residual, what is left out comes back: the sign turns it over and the next gradient replaces it
        e = p.cpu.get("e") if t else np.zeros((n, d), dtype=np.float32)
        p.step(g - e, 1e-3, label=f"{left} left, step {t}", with_e=t == 4)
    assert all(p.exact.values()), p.exact
    p.close()
