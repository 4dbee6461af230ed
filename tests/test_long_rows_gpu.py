"""Rows of 8192 and 16384 samples, which one workgroup at a time takes through LDS: grids whose workgroups own one row, uneven
runs of rows that cross from head to head, heads split into shares of rows, and each output of the backward pass left out."""
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


def _w(key, **kw):
    return dataclasses.replace(wl.WORKLOADS[key], **kw)


# one row; a share of one row and one of two; three heads of odd batches; more rows than the device holds workgroups, in runs of
# two (N = 8192 at 300 heads: the last run of the grid is shorter)
@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("B,H,N", [(1, 1, 8192), (1, 2, 16384), (3, 1, 16384), (5, 3, 8192), (2, 5, 16384)])
def test_every_row(B, H, N, io):
    check_full(wl.generate(_w("3", N=N, dtype=io), B=B, H=H))


@pytest.mark.parametrize("B,H,N,io", [(3, 300, 8192, wl.BF16), (2, 300, 16384, wl.F16)])
def test_runs_of_rows_across_heads(B, H, N, io):
    inp = wl.generate(_w("3", N=N, dtype=io), B=B, H=H)
    g = GpuRun(inp)
    hs = sample_heads(H, B, seed=N)
    k64, D64 = inp.k.astype(np.float64)[hs], inp.D.astype(np.float64)[hs]
    y = g.fwd()
    du, dk, dD = g.bwd()
    for x in (y, du, dk, dD):
        assert np.all(np.isfinite(x))
    rdu, rdk, rdD = oracle.longconv_bwd(inp.dy[:, hs], inp.u[:, hs], k64, D64)
    _compare({"y": y[:, hs], "du": du[:, hs], "dk": dk[hs], "dD": dD[hs]},
             {"y": oracle.longconv_fwd(inp.u[:, hs], k64, D64), "du": rdu, "dk": rdk, "dD": rdD}, TOL[io], f"runs N{N}", DD_TOL)


# A workgroup asks for the next row while it works on one: runs of two and three rows and of one and two, where nothing follows the last.
@pytest.mark.parametrize("B,H,N,io", [(3, 171, 32768, wl.F16), (1, 257, 32768, wl.BF16), (1, 257, 16384, wl.BF16)])
def test_ends_of_runs_of_one_to_three_rows(B, H, N, io):
    inp = wl.generate(_w("3", N=N, dtype=io), B=B, H=H)
    g = GpuRun(inp)
    hs = sample_heads(H, B, seed=N)
    k64, D64 = inp.k.astype(np.float64)[hs], inp.D.astype(np.float64)[hs]
    y = g.fwd()
    du, dk, dD = g.bwd()
    for x in (y, du, dk, dD):
        assert np.all(np.isfinite(x))
    rdu, rdk, rdD = oracle.longconv_bwd(inp.dy[:, hs], inp.u[:, hs], k64, D64)
    _compare({"y": y[:, hs], "du": du[:, hs], "dk": dk[hs], "dD": dD[hs]},
             {"y": oracle.longconv_fwd(inp.u[:, hs], k64, D64), "du": rdu, "dk": rdk, "dD": rdD}, TOL[io], f"runs N{N}", DD_TOL)


@pytest.mark.parametrize("N,io", [(8192, wl.F16), (16384, wl.BF16)])
@pytest.mark.parametrize("fuse", [1, 0])
def test_outputs_left_out(N, io, fuse):
    lc.longconv_set_option("fuse_bwd", fuse)
    inp = wl.generate(_w("3", N=N, dtype=io), B=3, H=2)
    want = dict(zip(("du", "dk", "dD"), oracle.longconv_bwd(inp.dy, inp.u, inp.k.astype(np.float64), inp.D.astype(np.float64))))
    for name in want:
        g = GpuRun(inp)
        got = dict(zip(("du", "dk", "dD"), g.bwd(**{n: n == name for n in want})))
        _compare({name: got[name]}, {name: want[name]}, TOL[io], f"{name} alone", DD_TOL)
        for other in want:
            if other != name:
                assert np.all(np.isnan(got[other])), f"{other} was written"


@pytest.mark.parametrize("N", [8192, 16384])
def test_not_a_number_stays_in_its_row(N):
    # rows of a workgroup's run share exchange buffer, prefetch and exponents
    inp = wl.generate(_w("3", N=N, dtype=wl.BF16), B=5, H=1)
    g = GpuRun(inp)
    y0 = g.fwd()
    du0 = g.bwd()[0]
    g.u[2, 0, 7] = float("nan")
    g.dy[2, 0, 7] = float("inf")
    y1 = g.fwd()
    du1, dk1, _ = g.bwd()
    keep = [0, 1, 3, 4]
    assert np.array_equal(y0[keep], y1[keep]) and np.array_equal(du0[keep], du1[keep])
    assert not np.all(np.isfinite(y1[2])) and not np.all(np.isfinite(du1[2])) and not np.all(np.isfinite(dk1))


# N = 32768: a row for every compute unit, and one more (workgroups of two rows)
@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("H", [256, 257])
def test_one_row_a_workgroup(H, io):
    inp = wl.generate(_w("3", N=32768, dtype=io), B=1, H=H)
    g = GpuRun(inp)
    hs = sample_heads(H, 1, seed=H)
    y, du = g.fwd()[:, hs], g.bwd(dk=False, dD=False)[0][:, hs]
    k64, D64 = inp.k.astype(np.float64)[hs], inp.D.astype(np.float64)[hs]
    _compare({"y": y, "du": du}, {"y": oracle.longconv_fwd(inp.u[:, hs], k64, D64),
                                  "du": oracle.longconv_bwd(inp.dy[:, hs], inp.u[:, hs], k64, D64)[0]}, TOL[io], f"one row a workgroup, H={H}")
