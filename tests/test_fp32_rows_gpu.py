"""fp32 rows of 2048 .. 16384 samples, each by itself through a transform of N twisted points: edges of the item grid, shares of a
head's rows and the accumulator that waits in the workspace, optional outputs, rows that do not touch each other."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2302_06646_amd as lc
import workloads as wl
from gpu_harness import GpuRun, check_full, check_sampled, sample_heads

pytestmark = pytest.mark.gpu


def _inputs(N, B, H):
    return wl.generate(dataclasses.replace(wl.WORKLOADS["1"], N=N, dtype=wl.F32), B=B, H=H)


# one item, fewer than the eight XCDs, not a multiple of eight; odd and even batches
@pytest.mark.parametrize("N", [2048, 4096, 8192, 16384])
@pytest.mark.parametrize("B,H", [(1, 1), (2, 3), (5, 2)])
def test_rows_and_gradients(N, B, H):
    assert f"L=2^{N.bit_length() - 1} of rows outer_radix=1" in lc.longconv_plan_string(N, lc.F32)
    check_full(_inputs(N, B, H))


# several rows in a share (the accumulator waits in the workspace from row to row, at N = 2048 in registers): even and uneven
# shares, and heads enough for one share each
@pytest.mark.parametrize("N,B,H", [(2048, 9, 300), (2048, 3, 1030), (4096, 7, 260), (4096, 2, 1030), (8192, 5, 200), (8192, 3, 513),
                                   (16384, 3, 100), (16384, 2, 257)])
def test_shares_of_several_rows(N, B, H):
    check_sampled(_inputs(N, B, H), sample_heads(H, B, seed=N + B))


@pytest.mark.parametrize("N", [2048, 8192])
def test_optional_outputs_and_repeats(N):
    g = GpuRun(_inputs(N, 3, 5))
    du, dk, dD = g.bwd()
    ks = g.kspec()
    for want in ((True, False, False), (False, True, False), (False, False, True), (True, True, True)):
        for t in (g.du, g.dk, g.dD):
            t.fill_(float("nan"))
        got = g.bwd(kspec=ks, du=want[0], dk=want[1], dD=want[2])
        for a, b, asked in zip(got, (du, dk, dD), want):
            if not asked:
                assert np.all(np.isnan(a))
            elif want == (True, False, False):
                # du alone comes from the convolution kernel, whose products are contracted by themselves: two results that lie
                # within 2e-7 of the exact one each (as measured against 64 bits) lie within 4e-7 of each other
                assert wl.rel_l2(a, b) <= 4e-7
            else:
                assert np.array_equal(a, b)                  # (the sums run in the same order every time)


@pytest.mark.parametrize("N", [2048, 16384])
def test_rows_do_not_touch_each_other(N):
    g = GpuRun(_inputs(N, 3, 2))
    y = g.fwd()
    du, _, _ = g.bwd()
    g.u[1, 0, 7] = float("nan")
    g.dy[1, 0, 9] = float("inf")
    y2 = g.fwd()
    du2, dk2, dD2 = g.bwd()
    keep = [(0, 0), (2, 0), (0, 1), (1, 1), (2, 1)]
    assert all(np.array_equal(y[i], y2[i]) and np.array_equal(du[i], du2[i]) for i in keep)
    assert not np.all(np.isfinite(y2[1, 0])) and not np.all(np.isfinite(du2[1, 0]))
    assert not np.all(np.isfinite(dk2[0])) and np.all(np.isfinite(dk2[1])) and np.isfinite(dD2[1])


# A row by itself is as near to the exact result as a row without a partner was in a pair of rows, transformed
# in 2N points (bounds: measured there, y 1.65 and 1.62e-7, dk 2.38 and 2.36e-7; means over heads vary by 0.01e-7)
@pytest.mark.parametrize("N,tol_y,tol_dk", [(2048, 1.65e-7, 2.38e-7), (4096, 1.62e-7, 2.36e-7)])
def test_error_of_a_row_without_a_partner(N, tol_y, tol_dk):
    H = 64
    gen = torch.Generator(device="cuda").manual_seed(N)
    rand = lambda *n: torch.randn(*n, generator=gen, device="cuda")
    u, dy, D = rand(1, H, N), rand(1, H, N), rand(H)
    k = rand(H, N) / N ** 0.5 * torch.exp(-4.0 * torch.arange(N, device="cuda") / N)
    y, du, dk, dD = torch.empty_like(u), torch.empty_like(u), torch.empty_like(k), torch.empty_like(D)
    ws = lc.new_workspace(1, H, N, wl.F32, True)
    lc.longconv_fwd(u, k, D, y, ws)
    lc.longconv_bwd(dy, u, k, D, du, dk, dD, ws)
    n = lambda t: t.cpu().numpy().astype(np.float64)
    ry = oracle.longconv_fwd(n(u), n(k), n(D))
    rdu, rdk, _ = oracle.longconv_bwd(n(dy), n(u), n(k), n(D))
    errs = {"y": wl.rel_l2(n(y), ry), "du": wl.rel_l2(n(du), rdu), "dk": wl.rel_l2(n(dk), rdk)}
    print(f"[fp32 rows] N{N} " + " ".join(f"{a}={b:.3e}" for a, b in errs.items()), flush=True)
    assert errs["y"] <= tol_y and errs["du"] <= tol_y and errs["dk"] <= tol_dk


# results of 2 to 64 shares added up: eight, four, two and one at a time, one number a thread and (heads enough) four
@pytest.mark.parametrize("N,B,H", [(4096, 2, 1), (4096, 6, 3), (2048, 15, 2), (4096, 16, 1), (4096, 64, 2), (4096, 8, 100), (16384, 16, 16)])
def test_sums_of_many_shares(N, B, H):
    check_full(_inputs(N, B, H))


# N = 2048: two rows of many heads in one share, of fewer in two; in between, fewer shares than there is room for
@pytest.mark.parametrize("B,H", [(2, 255), (2, 400), (4, 400), (8, 129)])
def test_shares_of_short_rows(B, H):
    assert lc.longconv_workspace_bytes(B, H, 2048, lc.F32, 1) >= lc.longconv_workspace_bytes(B - 1, H, 2048, lc.F32, 1)
    check_sampled(_inputs(2048, B, H), sample_heads(H, B, seed=B + H))


# N = 8192: the last number of rows whose convolution pads its exchanges in one way, and the first of the other
@pytest.mark.parametrize("B,H", [(2, 1024), (3, 683)])
def test_many_rows_of_8192(B, H):
    check_sampled(_inputs(8192, B, H), sample_heads(H, B, seed=H))
