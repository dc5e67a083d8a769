"""The call without a workspace where its sample also gives a window (k / d from 8 in 4096 on): on both sides of that line, rows kept
as one run and as eight, few and many buckets, and values whose sample misleads, bit for bit against the oracle, calls in a row."""
import numpy as np
import pytest
import torch

from oracle import compams_oracle as O
from paper_2205_05632_amd import binding as B

from parity import bits_equal

pytestmark = pytest.mark.gpu


def values(rng, kind, n, d):
    x = rng.standard_normal((n, d)).astype(np.float32)
    if kind == "layers":        # most of the selection in a few chunks
        x *= np.repeat(10.0 ** rng.uniform(-4, 0, (d + 8191) // 8192), 8192)[:d].astype(np.float32)
    elif kind == "few":         # the threshold's bucket holds most of the row
        x = (rng.integers(-3, 4, (n, d)) * 0.25).astype(np.float32)
    elif kind == "unsampled":   # what is kept lies between the sampled quads
        x[:, 4::16] *= 1000.0
    elif kind == "zeros":
        x[:, : d - d // 64] = 0.0
    elif kind == "huge":        # up to the largest finite magnitudes, and beyond
        x = np.ldexp(x, 126).astype(np.float32)
        x[:, 5] = np.inf
    return x


@pytest.mark.parametrize("kind", ["unit", "layers", "few", "unsampled", "zeros", "huge"])
@pytest.mark.parametrize("n,d,k", [(2, 65537, 127), (2, 65537, 129), (3, 64 * 4096, 2700), (1, 300007, 6000), (2, 63 * 4096 + 1, 20000),
                                   (1, 1_000_003, 30000)])
def test_sampled_window(n, d, k, kind):
    rng = np.random.default_rng(d + k)
    ld = B.padded_ld(d)
    theta0 = rng.standard_normal(d).astype(np.float32)
    theta = torch.from_numpy(theta0).cuda()
    m, v, vhat = (torch.zeros(d, device="cuda") for _ in range(3))
    e = torch.zeros((n, ld), device="cuda")
    idx = torch.zeros((n, k), dtype=torch.int32, device="cuda")
    val = torch.zeros((n, k), device="cuda")
    cpu = O.Oracle(n, d, theta0, compressor=O.TOPK, k=k)
    for t in range(2):
        g = values(rng, kind, n, d)
        gd = torch.zeros((n, ld), device="cuda")
        gd[:, :d] = torch.from_numpy(g).cuda()
        assert B.compams_step_static(n, d, k, theta, m, v, vhat, e, gd, 1e-3, idx_out=idx, val_out=val) == 0
        cpu.step(g, 1e-3)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy(), cpu.get("idx")), t
        assert bits_equal(val.cpu().numpy(), cpu.get("val")), t
        for name, x in (("theta", theta), ("m", m), ("v", v), ("vhat", vhat), ("e", e[:, :d])):
            a, b = np.ascontiguousarray(x.cpu().numpy()), cpu.get(name)
            assert np.array_equal(np.isnan(a), np.isnan(b)) and bits_equal(a[~np.isnan(a)], b[~np.isnan(b)]), (t, name)
    cpu.close()


@pytest.mark.parametrize("kind", ["unit", "layers", "few", "unsampled", "zeros", "huge"])
@pytest.mark.parametrize("n,d,k", [(1, 640 * 4096, 5300), (1, 640 * 4096 + 1, 5300),    # from here on 32 entries
                                   (16, 256 * 4096, 2100), (16, 256 * 4096 + 1, 2100),  # and here, by all rows
                                   (2, 70000, 43750), (2, 70000, 43751)])               # nearly all kept
def test_where_a_window_is_looked_for(n, d, k, kind):
    test_sampled_window(n, d, k, kind)


@pytest.mark.parametrize("most,d,k", [(680, 1, 1), (54, 65536, 655), (54, 65537, 655), (39, 300007, 3000)])
def test_what_the_call_admits(most, d, k):
    """The most rows it has ever taken of these shapes, and one more: the band list is made of the room that is left."""
    rng = np.random.default_rng(d)
    for n, want in ((most, 0), (most + 1, 3)):
        ld = B.padded_ld(d)
        theta, m, v, vhat = (torch.zeros(d, device="cuda") for _ in range(4))
        e, g = torch.zeros((n, ld), device="cuda"), torch.zeros((n, ld), device="cuda")
        g[:, :d] = torch.from_numpy(rng.standard_normal(d).astype(np.float32)).cuda()
        idx = torch.zeros((n, k), dtype=torch.int32, device="cuda")
        status = B.compams_step_static(n, d, k, theta, m, v, vhat, e, g, 1e-3, idx_out=idx)
        torch.cuda.synchronize()
        assert B.compams_strerror(status) == ("ok" if want == 0 else "workspace too small"), (n, status)
        if want == 0:
            x = g[0, :d].abs()
            keep = torch.sort(torch.topk(x, k).indices).values.to(torch.int32)
            assert torch.equal(idx, keep.expand(n, k))


def test_windows_fit():
    """A call of which a row's window does not fit takes the band kernel and the general route as well.  With a band list of 4 k + 8192
    entries that were two calls out of three here, 108 us where the others took 78; now nine out of ten take up to 88."""
    n, d, k = 8, 1565811, 4587
    ld = B.padded_ld(d)
    theta, m, v, vhat = (torch.zeros(d, device="cuda") for _ in range(4))
    e = torch.zeros((n, ld), device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(1)
    grads = [torch.empty((n, ld), device="cuda").normal_(generator=gen) for _ in range(3)]
    events = []
    for t in range(40):
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        grads[0].add_(0.0)  # (work in front of the call: its launches are not waited for)
        begin.record()
        assert B.compams_step_static(n, d, k, theta, m, v, vhat, e, grads[t % 3], 1e-3) == 0
        end.record()
        events.append((begin, end))
    torch.cuda.synchronize()
    us = sorted(a.elapsed_time(b) * 1e3 for a, b in events[5:])
    assert us[len(us) * 9 // 10] < 1.28 * us[len(us) // 5], us
