"""Rows of 65536 and 131072 samples in chunks of 16384 points, and dk of rows of 32768: heads split into two shares of rows, runs
of rows that cross from head to head, each output left out, magnitudes far from one."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2302_06646_amd as lc
import workloads as wl
from gpu_harness import DD_TOL, TOL, GpuRun, _compare, check_full, sample_heads

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_options():
    for name, value in lc.OPTION_DEFAULTS.items():
        lc.longconv_set_option(name, value)
    yield
    for name, value in lc.OPTION_DEFAULTS.items():
        lc.longconv_set_option(name, value)


def _w(**kw):
    return dataclasses.replace(wl.WORKLOADS["4a"], **kw)


# one row; two shares of a row and of two and one; N = 131072 reads eight parts of a row
@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("B,H,N", [(1, 1, 65536), (2, 2, 65536), (3, 1, 65536), (1, 2, 131072), (3, 1, 131072), (3, 2, 32768)])
def test_every_row(B, H, N, io):
    check_full(wl.generate(_w(N=N, dtype=io), B=B, H=H))


# more rows than runs: 64 runs of rows at N = 65536 (of two and one rows), 32 at 131072, 128 at 32768; whole heads for dk
@pytest.mark.parametrize("B,H,N,io", [(3, 35, 65536, wl.BF16), (2, 18, 131072, wl.F16), (1, 130, 32768, wl.F16)])
def test_runs_of_rows_across_heads(B, H, N, io):
    inp = wl.generate(_w(N=N, dtype=io), B=B, H=H)
    g = GpuRun(inp)
    hs = sample_heads(H, B, seed=N, min_rows=4)
    k64, D64 = inp.k.astype(np.float64)[hs], inp.D.astype(np.float64)[hs]
    y = g.fwd()
    du, dk, dD = g.bwd()
    for x in (y, du, dk, dD):
        assert np.all(np.isfinite(x))
    rdu, rdk, rdD = oracle.longconv_bwd(inp.dy[:, hs], inp.u[:, hs], k64, D64)
    _compare({"y": y[:, hs], "du": du[:, hs], "dk": dk[hs], "dD": dD[hs]},
             {"y": oracle.longconv_fwd(inp.u[:, hs], k64, D64), "du": rdu, "dk": rdk, "dD": rdD}, TOL[io], f"runs N{N}", DD_TOL)


@pytest.mark.parametrize("N,io,fuse", [(65536, wl.F16, 1), (65536, wl.BF16, 0), (131072, wl.BF16, 1), (32768, wl.BF16, 1)])
def test_outputs_left_out(N, io, fuse):
    lc.longconv_set_option("fuse_bwd", fuse)
    inp = wl.generate(_w(N=N, dtype=io), B=3, H=1)
    want = dict(zip(("du", "dk", "dD"), oracle.longconv_bwd(inp.dy, inp.u, inp.k.astype(np.float64), inp.D.astype(np.float64))))
    for name in want:
        g = GpuRun(inp)
        got = dict(zip(("du", "dk", "dD"), g.bwd(**{n: n == name for n in want})))
        _compare({name: got[name]}, {name: want[name]}, TOL[io], f"{name} alone", DD_TOL)
        for other in want:
            if other != name:
                assert np.all(np.isnan(got[other])), f"{other} was written"


@pytest.mark.parametrize("N,amp", [(32768, 38000.0), (65536, 43000.0), (131072, 23000.0)])
def test_large_samples_a_chunk_apart(N, amp):
    # R fp16 samples N / R apart: a component of a chunk's sum over them is at most sum_n max(cos, sin)(2 pi n / 4R) <= 1.71, 3.02
    # and 5.6 of them, and half of that (R > 2) has to fit fp16.  y of N = 32768 goes another way
    H = 3
    inp = wl.generate(_w(N=N, dtype=wl.F16), B=1, H=H)
    g = GpuRun(inp)
    for t, at in ((g.u, 100), (g.dy, 7)):
        t.zero_()
        t[..., at::16384] = amp
    g.dy *= 2.0 ** -15                                       # dk stays below 2^18, du below 1
    g.k.zero_()
    g.k[:, 3], g.D[:] = 0.25, 0.125
    u, dy = (t.cpu().numpy().astype(np.float64) for t in (g.u, g.dy))
    k64, D64 = g.k.cpu().numpy().astype(np.float64), g.D.cpu().numpy().astype(np.float64)
    got, want = {}, {}
    if N > 32768:
        got["y"], want["y"] = g.fwd(), oracle.longconv_fwd(u, k64, D64)
    du, got["dk"], got["dD"] = g.bwd()
    want["du"], want["dk"], want["dD"] = oracle.longconv_bwd(dy, u, k64, D64)
    got["du"] = du
    _compare(got, want, TOL[wl.F16], f"large samples N{N}", DD_TOL)


@pytest.mark.parametrize("N", [65536, 131072])
def test_small_fp16_rows(N):
    # rows of a few times fp16's smallest normal number (6.1e-5), which fp16 rows may have: the usual bound
    inp = wl.generate(_w(N=N, dtype=wl.F16), B=2, H=2)
    g = GpuRun(inp)
    g.u *= 1.5e-4
    g.dy *= 1.5e-4
    u, dy = (t.cpu().numpy().astype(np.float64) for t in (g.u, g.dy))
    k64, D64 = inp.k.astype(np.float64), inp.D.astype(np.float64)
    y = g.fwd()
    du, dk, dD = g.bwd()
    rdu, rdk, rdD = oracle.longconv_bwd(dy, u, k64, D64)
    _compare({"y": y, "du": du, "dk": dk, "dD": dD}, {"y": oracle.longconv_fwd(u, k64, D64), "du": rdu, "dk": rdk, "dD": rdD},
             TOL[wl.F16], f"small rows N{N}", DD_TOL)


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("N", [32768, 65536, 131072])
def test_dk_of_one_tap(N, io):
    # rows of one sample each: the spectrum's product is flat and dk a single tap, the largest number that a chunk's inverse
    # transform can make of a spectrum of that size.  Magnitudes on both sides of a power of two, and
    # lags that are odd and even multiples of a chunk's shares; the other taps hold nothing but rounding
    lags = [0, 1, N // 32, N // 16, N // 8, N // 4, 3 * N // 8, N // 2, N - 1]
    for size in (1.0, 1.1, 1.5, 1.999):
        inp = wl.generate(_w(N=N, dtype=io), B=1, H=len(lags))
        g = GpuRun(inp)
        g.u.zero_()
        g.dy.zero_()
        g.u[0, :, 0] = 1.0
        for h, lag in enumerate(lags):
            g.dy[0, h, lag] = size
        want = np.zeros(g.dk.shape)
        want[range(len(lags)), lags] = float(g.dy[0, 0, 0])
        _, dk, _ = g.bwd(du=False)
        _compare({"dk": dk}, {"dk": want}, TOL[io], f"one tap N{N} {size}")


@pytest.mark.parametrize("N", [32768, 65536])
def test_dk_of_rows_with_a_mean(N):
    # the sums over rows grow as N^2 in the first bins, beyond fp16: each chunk's inverse transform has its own power of two.
    # fp16 rounding is relative to that peak (dk = N x means in every tap), so the bound is the usual one
    inp = wl.generate(_w(N=N, dtype=wl.F16), B=3, H=1)
    g = GpuRun(inp)
    g.u.copy_(g.u * 0.25 + 1.0)
    g.dy.copy_(g.dy * 0.25 + 1.0)
    u, dy = (t.cpu().numpy().astype(np.float64) for t in (g.u, g.dy))
    _, rdk, rdD = oracle.longconv_bwd(dy, u, inp.k.astype(np.float64), inp.D.astype(np.float64))
    _, dk, dD = g.bwd(du=False)
    _compare({"dk": dk, "dD": dD}, {"dk": rdk, "dD": rdD}, TOL[wl.F16], f"mean N{N}", DD_TOL)


# more than two shares of a head's rows, whose results wait in du: three of uneven rows, as many as half the batch, du by a kernel of its
# own (N = 32768, and without fuse_bwd); without du there are two
@pytest.mark.parametrize("B,H,N,io,fuse", [(7, 1, 65536, wl.F16, 1), (16, 2, 65536, wl.BF16, 1), (9, 3, 131072, wl.BF16, 1), (11, 2, 32768, wl.F16, 1),
                                           (23, 1, 32768, wl.BF16, 1), (9, 1, 65536, wl.F16, 0)])
def test_shares_that_wait_in_du(B, H, N, io, fuse):
    lc.longconv_set_option("fuse_bwd", fuse)
    inp = wl.generate(_w(N=N, dtype=io), B=B, H=H)
    check_full(inp)
    g = GpuRun(inp)
    first, again = g.bwd(), g.bwd()
    assert all(np.array_equal(a, b) for a, b in zip(first, again))
    du, dk, dD = g.bwd(du=False)
    rdu, rdk, rdD = oracle.longconv_bwd(inp.dy, inp.u, inp.k.astype(np.float64), inp.D.astype(np.float64))
    _compare({"dk": dk, "dD": dD}, {"dk": rdk, "dD": rdD}, TOL[io], f"two shares N{N}", DD_TOL)
