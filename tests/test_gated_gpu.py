"""Gated long convolution (output times a second sequence) and its backward through the C ABI against the float64
oracle: every plan family, all three I/O dtypes, optional outputs."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2302_06646_amd as lc
import workloads as wl
from gpu_harness import TOL, DD_TOL, _compare, to_dev, to_f64
from oracle import gated

pytestmark = pytest.mark.gpu


def _inputs(N, io, B, H, seed=0):
    kind = {wl.F32: "decay256", wl.F16: "decay_alpha_squash", wl.BF16: "squash_pool"}[io]
    w = wl.Workload(6, B, H, N, io, kind)
    inp = wl.generate(w, seed_extra=seed)
    g32 = np.random.default_rng(991 + N + seed).standard_normal((B, H, N), dtype=np.float32)
    g_s, g_v = wl.quantize(g32, io)
    return inp, g_s, g_v


def _run(inp, g_s, want_du=True, want_dk=True, want_dD=True, want_dg=True):
    io = inp.w.dtype
    B, H, N = inp.u_store.shape
    u, dy, g = to_dev(inp.u_store, io), to_dev(inp.dy_store, io), to_dev(g_s, io)
    k, D = torch.from_numpy(inp.k).cuda(), torch.from_numpy(inp.D).cuda()
    y = torch.full_like(u, float("nan"))
    du, dg = torch.full_like(u, float("nan")), torch.full_like(u, float("nan"))
    dk, dD = torch.full_like(k, float("nan")), torch.full_like(D, float("nan"))
    ws = lc.new_workspace(B, H, N, io, 2)
    lc.longconv_fwd_gated(u, k, D, g, y, ws)
    lc.longconv_bwd_gated(dy, g, u, k, D, du if want_du else None, dk if want_dk else None,
                          dD if want_dD else None, dg if want_dg else None, ws)
    torch.cuda.synchronize()
    return (to_f64(y, io), to_f64(du, io), dk.cpu().numpy().astype(np.float64), dD.cpu().numpy().astype(np.float64),
            to_f64(dg, io))


CASES = [(1024, wl.F32), (256, wl.BF16), (1024, wl.BF16), (2048, wl.F16), (4096, wl.BF16), (16384, wl.F16),
         (65536, wl.F16)]


@pytest.mark.parametrize("N,io", CASES)
def test_gated_layer_against_the_oracle(N, io):
    B, H = (3, 2) if N <= 16384 else (1, 2)
    inp, g_s, g_v = _inputs(N, io, B, H)
    y, du, dk, dD, dg = _run(inp, g_s)
    k64, D64 = inp.k.astype(np.float64), inp.D.astype(np.float64)
    ry = gated.gated_fwd(inp.u, k64, D64, g_v)
    rdu, rdk, rdD, rdg = gated.gated_bwd(inp.dy, g_v, inp.u, k64, D64)
    tol = TOL[io]
    errs = _compare({"y": y, "du": du, "dk": dk, "dg": dg}, {"y": ry, "du": rdu, "dk": rdk, "dg": rdg}, tol,
                    f"gated N={N} io={wl.DTYPE_NAMES[io]}")
    e_dD = wl.rel_l2(dD, rdD)
    assert e_dD <= DD_TOL, e_dD        # the fp32 sum of dy g u from the three tensors, on every dtype
    assert errs


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
def test_gated_rows_of_32768_samples(io):
    # the gate in the store of the single-row kernel (forward, and dg as the forward pass gated by dy)
    test_gated_layer_against_the_oracle(32768, io)


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("N", [256, 512, 1024, 2048, 4096, 8192, 16384, 32768, 65536])
def test_gate_meets_heads_of_other_magnitudes(N, io):
    # A head with a small concentrated kernel is stored with a power of two taken out (2^-22 for 1e-4 at one tap), so its
    # outputs are large numbers until they get it back; the gate (y) or dy (dg), of order 64 here, must not meet them
    # before that: fp16 ends at 65504, and y and dg themselves are of order 1e-2 there.  Next to it an ordinary head and a
    # large one.  dz = dy g stays of order one.
    B, H = 2 if N <= 16384 else 1, 3
    inp, _, g_v = _inputs(N, io, B, H, seed=5)
    k, D = inp.k.copy(), inp.D.copy()
    k[0] = 0.0; k[0, 0] = 1e-4; D[0] = 0.0
    k[2] *= 2.0 ** 9; D[2] *= 2.0 ** 9
    k64, D64 = k.astype(np.float64), D.astype(np.float64)
    for big in ("y", "dg"):
        s = np.array([64.0, 64.0, 1.0 / 64.0])[None, :, None] ** (1 if big == "y" else -1)
        g_s, g = wl.quantize((s * g_v).astype(np.float32), io)
        dy_s, dy = wl.quantize((inp.dy / s).astype(np.float32), io)
        y, du, dk, dD, dg = _run(dataclasses.replace(inp, k=k, D=D, dy_store=dy_s, dy=dy), g_s)
        rdu, rdk, rdD, rdg = gated.gated_bwd(dy, g, inp.u, k64, D64)
        got = {"du": du, "dk": dk, big: y if big == "y" else dg}
        want = {"du": rdu, "dk": rdk, big: gated.gated_fwd(inp.u, k64, D64, g) if big == "y" else rdg}
        heads = slice(None) if big == "y" else slice(0, 2)      # (the large head's dg lies below fp16's normal range)
        got[big], want[big] = got[big][:, heads], want[big][:, heads]
        _compare(got, want, TOL[io], f"gate and heads of other magnitudes, {big}, N={N} io={wl.DTYPE_NAMES[io]}")


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("N,B,H", [(256, 18, 520), (512, 9, 520), (1024, 9, 1100), (2048, 7, 780), (4096, 7, 400)])
def test_gated_long_runs_of_rows(N, B, H, io):
    # workgroups with many rows, which run the middle of the kernels' row pipelines: gradients as small as a mean loss
    # makes them (bf16), rows of other magnitudes and zero rows among them, heads with a power of two taken out
    inp, g_s, g_v = _inputs(N, io, B, H, seed=7)
    rng = np.random.default_rng(57 + N)
    ks = np.where(rng.random(H) < 0.3, 2.0 ** rng.integers(-9, 9, size=H), 1.0)
    k, D = (inp.k * ks[:, None]).astype(np.float32), (inp.D * ks).astype(np.float32)
    us = ds = np.ones((B, H, 1))
    if io == wl.BF16:
        us = np.where(rng.random((B, H, 1)) < 0.3, 10.0 ** rng.uniform(-6, 6, size=(B, H, 1)), 1.0)
        ds = np.where(rng.random((B, H, 1)) < 0.3, 10.0 ** rng.uniform(-9, 3, size=(B, H, 1)), 1e-4)
        us[rng.random((B, H, 1)) < 0.05] = 0.0
        ds[rng.random((B, H, 1)) < 0.05] = 0.0
    u_s, u = wl.quantize((inp.u * us).astype(np.float32), io)
    dy_s, dy = wl.quantize((inp.dy * ds).astype(np.float32), io)
    out = _run(dataclasses.replace(inp, k=k, D=D, u_store=u_s, u=u, dy_store=dy_s, dy=dy), g_s)
    assert all(np.all(np.isfinite(v)) for v in out)
    hs = sorted({0, 1, H // 3, H // 3 + 1, H // 2, H - 1, int(np.argmin(ks)), int(np.argmax(ks))})
    y, du, dk, dD, dg = (v[:, hs] if v.ndim == 3 else v[hs] for v in out)
    k64, D64 = k[hs].astype(np.float64), D[hs].astype(np.float64)
    rdu, rdk, rdD, rdg = gated.gated_bwd(dy[:, hs], g_v[:, hs], u[:, hs], k64, D64)
    label = f"gated long runs, N={N} B={B} H={H} io={wl.DTYPE_NAMES[io]}"
    # (dD: rows of wildly different size meet in one fp32 dot product, a few 1e-5)
    _compare({"y": y, "dk": dk, "dg": dg, "dD": dD}, {"y": gated.gated_fwd(u[:, hs], k64, D64, g_v[:, hs]), "dk": rdk, "dg": rdg, "dD": rdD},
             TOL[io], label, dd_tol=1e-4)
    # du is rounded twice in bf16, dz on the way in and du on the way out, by 2^-9 at most each; the transforms add 1e-3
    _compare({"du": du}, {"du": rdu}, 2 * 2.0 ** -9 + 1e-3 if io == wl.BF16 else TOL[io], label)


def test_optional_outputs_and_error_codes():
    inp, g_s, g_v = _inputs(1024, wl.BF16, 2, 2)
    y, du, dk, dD, dg = _run(inp, g_s, want_du=False, want_dk=False, want_dD=False)
    assert np.all(np.isnan(du)) and np.all(np.isnan(dk)) and np.all(np.isnan(dD))
    k64, D64 = inp.k.astype(np.float64), inp.D.astype(np.float64)
    rdg = gated.gated_bwd(inp.dy, g_v, inp.u, k64, D64)[3]
    assert wl.rel_l2(dg, rdg) <= TOL[wl.BF16]
    y2, du2, dk2, dD2, dg2 = _run(inp, g_s, want_dg=False)
    assert np.all(np.isnan(dg2)) and np.all(np.isfinite(du2))
    # a backward workspace without room for dz is refused before anything is launched
    io = wl.BF16
    B, H, N = inp.u_store.shape
    u, dy, g = to_dev(inp.u_store, io), to_dev(inp.dy_store, io), to_dev(g_s, io)
    k, D = torch.from_numpy(inp.k).cuda(), torch.from_numpy(inp.D).cuda()
    small = lc.new_workspace(B, H, N, io, 1)
    with pytest.raises(lc.LongconvError, match="workspace"):
        lc.longconv_bwd_gated(dy, g, u, k, D, torch.empty_like(u), None, None, None, small)
    assert lc.longconv_workspace_bytes(B, H, N, io, 2) >= lc.longconv_workspace_bytes(B, H, N, io, 1) + B * H * N * 2


# dD by shares of a head's samples, beside dz where the backward pass needs that: one share, several even and uneven ones, as many as
# there may be; u at any address where dD alone is asked for
@pytest.mark.parametrize("N,io,B,H", [(8192, wl.F16, 1, 1), (8192, wl.BF16, 3, 1), (16384, wl.F32, 5, 2), (32768, wl.F16, 7, 3),
                                      (131072, wl.BF16, 2, 3), (65536, wl.F16, 40, 1)])
def test_shares_of_dD(N, io, B, H):
    gen = torch.Generator(device="cuda").manual_seed(N + B)
    td = {wl.F32: torch.float32, wl.F16: torch.float16, wl.BF16: torch.bfloat16}[io]
    rand = lambda *n: torch.randn(*n, generator=gen, device="cuda").to(td)
    dy, g, u = rand(B, H, N), rand(B, H, N), rand(B, H, N)
    k, D = torch.randn(H, N, generator=gen, device="cuda") / N, torch.randn(H, generator=gen, device="cuda")
    want = torch.zeros(H, dtype=torch.float64, device="cuda")
    size = torch.zeros(H, dtype=torch.float64, device="cuda")
    for b in range(B):
        p = dy[b].double() * g[b].double() * u[b].double()
        want += p.sum(-1)
        size += p.abs().sum(-1)
    ws = lc.new_workspace(B, H, N, io, 2)
    outs = []
    for all_of_it in (True, False):
        du, dk, dD = torch.empty_like(u), torch.empty_like(k), torch.full_like(D, float("nan"))
        lc.longconv_bwd_gated(dy, g, u, k, D, du if all_of_it else None, dk if all_of_it else None, dD, None, ws)
        if all_of_it:
            # the same dz as the ungated pass gets from torch: products of two numbers of the I/O type, rounded once
            du2, dk2 = torch.empty_like(u), torch.empty_like(k)
            lc.longconv_bwd((dy.float() * g.float()).to(td), u, k, D, du2, dk2, None, lc.new_workspace(B, H, N, io, 1))
            assert torch.equal(du, du2) and torch.equal(dk, dk2)
        outs.append(dD)
    odd = torch.empty(B * H * N + 1, dtype=td, device="cuda")[1:].view(B, H, N).copy_(u)
    dD = torch.full_like(D, float("nan"))
    lc.longconv_bwd_gated(dy, g, odd, k, D, None, None, dD, None, ws)
    outs.append(dD)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    # a lane's chain of at most per / 256 pieces of 8 terms in fp32, then two short trees; errors of a sum of terms of either sign
    # stay below eps / 2 times the chain's length times the sum of magnitudes, and are far below it
    chain = 8 * (B * N // 8 // 256 // max(1, min(256, B * N // 8192)) + 2) + 16
    assert torch.all((outs[0].double() - want).abs() <= 6e-8 * chain * size)


# N = 256: as many pairs of rows as the forward launch takes waves at once (bf16, a device of 256 compute units: 5 workgroups of 4 waves
# on each), and one more, with a last row that has no partner
@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("B,H", [(8, 1280), (3, 2561)])
def test_gated_rows_of_256(B, H, io):
    inp, g_s, g_v = _inputs(256, io, B, H, seed=11)
    y = _run(inp, g_s)[0]
    assert np.all(np.isfinite(y))
    hs = sorted({0, 1, H // 2, H - 2, H - 1, *np.random.default_rng(H).choice(H, size=24, replace=False).tolist()})
    want = gated.gated_fwd(inp.u[:, hs], inp.k[hs].astype(np.float64), inp.D[hs].astype(np.float64), g_v[:, hs])
    _compare({"y": y[:, hs]}, {"y": want}, TOL[io], f"gated rows of 256, B={B} H={H} io={wl.DTYPE_NAMES[io]}")
