"""Backward pass of rows of 2048 and 4096 samples whose heads alone fill half the device: two or three shares of a head's rows,
uneven ones among them, and one share next to the rule's edges (128 and 512 heads)."""
import dataclasses

import numpy as np
import pytest

import oracle
import workloads as wl
import test_gated_gpu as tg
from gpu_harness import DD_TOL, TOL, GpuRun, _compare, sample_heads
from oracle import gated

pytestmark = pytest.mark.gpu


def _shares_taken(g):
    """How many shares of a head's rows the backward call takes: with the spectrum at hand it writes nothing to its workspace but
    the shares' dk and dD, [shares][H][N + 1] fp32 numbers (one share: nothing)."""
    ks = g.kspec()
    g.ws.fill_(0xFF)
    g.bwd(kspec=ks)
    blocks = int((g.ws.view(-1, 256) != 0xFF).any(dim=1).sum())
    return max(1, round(blocks * 256 / (g.H * (g.N + 1) * 4)))


# three shares of 5 and 6 rows, three of 11 and 10; three shares of more than one turn; two shares; one (few rows; the edges of
# the rule, and on its other side four)
@pytest.mark.parametrize("B,H,N,io,shares", [(16, 130, 2048, wl.BF16, 3), (32, 130, 4096, wl.F16, 3), (32, 340, 2048, wl.F16, 3),
                                             (25, 260, 4096, wl.BF16, 2), (1, 129, 2048, wl.BF16, 1), (2, 512, 2048, wl.F16, 1),
                                             (2, 513, 4096, wl.F16, 1), (17, 128, 2048, wl.F16, 4)])
def test_shares_of_many_heads(B, H, N, io, shares):
    inp = wl.generate(dataclasses.replace(wl.WORKLOADS["2"], N=N, dtype=io), B=B, H=H)
    g = GpuRun(inp)
    assert _shares_taken(g) == shares
    hs = sample_heads(H, B, seed=N + H)
    k64, D64 = inp.k.astype(np.float64)[hs], inp.D.astype(np.float64)[hs]
    du, dk, dD = g.bwd()
    for x in (du, dk, dD):
        assert np.all(np.isfinite(x))
    rdu, rdk, rdD = oracle.longconv_bwd(inp.dy[:, hs], inp.u[:, hs], k64, D64)
    _compare({"du": du[:, hs], "dk": dk[hs], "dD": dD[hs]}, {"du": rdu, "dk": rdk, "dD": rdD}, TOL[io], f"shares N{N}", DD_TOL)


# three shares of a head's rows: all at once, and in more than one turn
@pytest.mark.parametrize("B,H", [(16, 130), (32, 340)])
def test_shares_of_gated_rows(B, H):
    N, io = 2048, wl.BF16
    inp, g_s, g_v = tg._inputs(N, io, B, H, 5)
    _, du, dk, dD, dg = tg._run(inp, g_s)
    hs = sample_heads(H, B, seed=5)
    k64, D64 = inp.k.astype(np.float64)[hs], inp.D.astype(np.float64)[hs]
    rdu, rdk, rdD, rdg = gated.gated_bwd(inp.dy[:, hs], g_v[:, hs], inp.u[:, hs], k64, D64)
    for name, a, b in (("du", du[:, hs], rdu), ("dk", dk[hs], rdk), ("dg", dg[:, hs], rdg), ("dD", dD[hs], rdD)):
        e = wl.rel_l2(a, b)
        assert np.isfinite(e) and e <= (1e-5 if name == "dD" else 3e-3), (name, e)


# twice the groups of waves in workgroups that have a compute unit to themselves (N = 2048 and gated 1024): uneven and even shares
# of a group, the fewest rows that take them and one less, one and more heads than half the device
@pytest.mark.parametrize("N,B,H,io", [(2048, 2, 200, wl.BF16), (2048, 3, 200, wl.F16), (2048, 5, 256, wl.BF16), (2048, 24, 256, wl.F16),
                                      (2048, 3, 1, wl.BF16), (2048, 5, 257, wl.BF16), (1024, 4, 200, wl.BF16), (1024, 5, 200, wl.F16),
                                      (1024, 11, 256, wl.BF16), (1024, 11, 3, wl.F16)])
def test_groups_of_waves(N, B, H, io):
    inp, g_s, g_v = tg._inputs(N, io, B, H, 7)
    _, du, dk, dD, dg = tg._run(inp, g_s)
    hs = sample_heads(H, B, seed=7)
    k64, D64 = inp.k.astype(np.float64)[hs], inp.D.astype(np.float64)[hs]
    rdu, rdk, rdD, rdg = gated.gated_bwd(inp.dy[:, hs], g_v[:, hs], inp.u[:, hs], k64, D64)
    for name, a, b in (("du", du[:, hs], rdu), ("dk", dk[hs], rdk), ("dg", dg[:, hs], rdg), ("dD", dD[hs], rdD)):
        e = wl.rel_l2(a, b)
        assert np.isfinite(e) and e <= (1e-5 if name == "dD" else 3e-3), (name, e)
    du, dk, dD = GpuRun(inp).bwd()
    rdu, rdk, rdD = oracle.longconv_bwd(inp.dy[:, hs], inp.u[:, hs], k64, D64)
    _compare({"du": du[:, hs], "dk": dk[hs], "dD": dD[hs]}, {"du": rdu, "dk": rdk, "dD": rdD}, TOL[io], f"groups N{N}", DD_TOL)
