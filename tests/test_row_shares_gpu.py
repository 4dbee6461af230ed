"""Backward pass of rows of 2048 and 4096 samples whose heads alone fill half the device: two or three shares of a head's rows,
uneven ones among them, and one share next to the rule's edges (128 and 512 heads)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2302_06646_amd as lc
import workloads as wl
import test_gated_gpu as tg
from gpu_harness import _TD, DD_TOL, TOL, GpuRun, _compare, sample_heads
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


# N = 2048, two shares as the groups of waves of one workgroup: dk is the sum of two rows, each from an inverse transform of its own
# (in fp16), as with two workgroups.  Calls for the even and for the odd rows make the same two rows, up to the order of their fp32
# sums in front of the same rounding (2e-5); one inverse of the whole sum would be 6e-4 off.
@pytest.mark.parametrize("layer,B,H,io", [("plain", 24, 256, wl.BF16), ("plain", 19, 200, wl.F16), ("gated", 24, 200, wl.F16),
                                          ("gated", 25, 256, wl.BF16), ("image", 24, 256, wl.BF16)])
def test_two_shares_in_one_workgroup(layer, B, H, io):
    gen = torch.Generator(device="cuda").manual_seed(B + H)
    shape = (32, 32) if layer == "image" else (2048,)
    u, dy, g = (torch.randn(B, H, *shape, generator=gen, device="cuda").to(_TD[io]) for _ in range(3))
    k, D = torch.randn(H, *shape, generator=gen, device="cuda") / 32, torch.randn(H, generator=gen, device="cuda")

    def grads(rows):
        u_, dy_, g_ = (t[rows].contiguous() for t in (u, dy, g))
        du, dk, dD, dg = torch.empty_like(u_), torch.empty_like(k), torch.empty_like(D), torch.empty_like(u_)
        n = u_.shape[0]
        if layer == "image":
            lc.longconv2d_bwd(dy_, u_, k, D, du, dk, dD, lc.new_workspace2d(n, H, *shape, io, True))
        elif layer == "gated":
            lc.longconv_bwd_gated(dy_, g_, u_, k, D, du, dk, dD, dg, lc.new_workspace(n, H, 2048, io, 2))
        else:
            lc.longconv_bwd(dy_, u_, k, D, du, dk, dD, lc.new_workspace(n, H, 2048, io, True))
        return dk.double().cpu().numpy(), dD.double().cpu().numpy()

    (dk, dD), (dk0, dD0), (dk1, dD1) = grads(slice(None)), grads(slice(0, None, 2)), grads(slice(1, None, 2))
    assert wl.rel_l2(dk, dk0 + dk1) <= 1e-4
    assert wl.rel_l2(dD, dD0 + dD1) <= 1e-5
