"""The kernel regularisers of Algorithm 1 lines 1-3 on the device (longconv_kreg_fwd / longconv_kreg_bwd through the
C ABI) against the float64 oracle, alone and chained with the convolution."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _draw(H, N, std, q, seed):
    rng = np.random.default_rng(seed)
    k = (std * rng.standard_normal((H, N))).astype(np.float32)
    mask = None if q == 0 else ((rng.random((H, N)) >= q) / (1.0 - q)).astype(np.float32)
    g = rng.standard_normal((H, N)).astype(np.float32)
    return k, mask, g


@pytest.mark.parametrize("H,N,p,lam,q", [(37, 1024, 1, 0.003, 0.2), (5, 16384, 3, 1e-4, 0.0), (3, 256, 0, 0.0, 0.0),
                                         (2, 512, 32, 0.002, 0.5), (4, 131072, 2, 0.0, 0.1), (70, 4096, 1, 0.05, 0.0)])
def test_regularisers_forward_and_chain_against_oracle(H, N, p, lam, q):
    import paper_2302_06646_amd as lc
    from oracle import kreg
    k, mask, g = _draw(H, N, 0.02, q, seed=N + p)
    dk_ = torch.from_numpy(k).cuda()
    dm = None if mask is None else torch.from_numpy(mask).cuda()
    dg = torch.from_numpy(g).cuda()
    kbar = torch.full_like(dk_, float("nan"))
    dk = torch.full_like(dk_, float("nan"))
    lc.longconv_kreg_fwd(dk_, dm, kbar, p, lam)
    lc.longconv_kreg_bwd(dk_, dm, dg, dk, p, lam)
    torch.cuda.synchronize()
    k64 = k.astype(np.float64)
    m64 = None if mask is None else mask.astype(np.float64)
    lam64 = float(np.float32(lam))
    want = kreg.kernel_reg_fwd(k64, m64, p, lam64)
    got = kbar.cpu().numpy().astype(np.float64)
    scale = np.abs(k64).max() * (1.0 if mask is None else np.abs(m64).max())
    err = np.abs(got - want).max() / scale
    print(f"[kreg] H{H} N{N} p{p} lam{lam} q{q}: fwd max err / scale = {err:.2e}", flush=True)
    assert err <= 2e-6                                   # Squash is continuous: fp32 rounding only
    assert np.all((got == 0) | (np.abs(want) > 0) | (np.abs(got) <= 2e-6 * scale))
    # backward: the gate |K2| > lambda is a decision; entries whose K2 sits within fp32 rounding of lambda may take
    # either side, everything else must agree to rounding
    k2 = kreg.smooth(kreg.dropout(k64, m64), p)
    margin = np.abs(np.abs(k2) - lam64)
    sure = margin > 4e-7 * max(scale, lam64)
    gate_sure = (np.abs(k2) > lam64) | ~sure             # unsure entries: evaluate both sides
    g64 = g.astype(np.float64)

    def chain(gate):
        d2 = g64 * gate
        N_ = d2.shape[-1]
        d1 = kreg.smooth(d2, p)                          # Smooth with this boundary rule is its own transpose
        return d1 if m64 is None else d1 * m64
    hi = chain(gate_sure)
    lo = chain((np.abs(k2) > lam64) & sure)
    got_dk = dk.cpu().numpy().astype(np.float64)
    ref = kreg.kernel_reg_bwd(k64, m64, p, lam64, g64)
    if np.all(sure):
        assert np.abs(got_dk - ref).max() <= 2e-6 * np.abs(ref).max()
    else:                                                # between the two admissible gates, entry by entry
        a, b = np.minimum(lo, hi), np.maximum(lo, hi)
        tol = 2e-6 * max(np.abs(ref).max(), 1e-30)
        assert np.all(got_dk >= a - tol) and np.all(got_dk <= b + tol)
    print(f"[kreg] unsure gate entries: {int((~sure).sum())} of {sure.size}", flush=True)


@pytest.mark.parametrize("key,B,H,p,lam,q", [("2", 6, 5, 1, 0.003, 0.25), ("3", 2, 2, 2, 1e-4, 0.0)])
def test_regularised_convolution_end_to_end(key, B, H, p, lam, q):
    """Algorithm 1 as a whole: raw K -> regularisers -> convolution, and the gradient of the raw K through
    longconv_bwd and the chain, against the oracle composite."""
    import oracle
    import paper_2302_06646_amd as lc
    from gpu_harness import GpuRun, TOL
    from oracle import kreg
    inp = wl.generate(wl.WORKLOADS[key], B=B, H=H)
    N = inp.w.N
    rng = np.random.default_rng(5)
    kraw = (rng.standard_normal((H, N)) * (0.02 if key == "2" else 1.0 / np.sqrt(N))).astype(np.float32)
    mask = None if q == 0 else ((rng.random((H, N)) >= q) / (1.0 - q)).astype(np.float32)
    d_kraw = torch.from_numpy(kraw).cuda()
    d_mask = None if mask is None else torch.from_numpy(mask).cuda()
    g = GpuRun(inp)
    lc.longconv_kreg_fwd(d_kraw, d_mask, g.k, p, lam)            # g.k now holds kbar
    y = g.fwd()
    du, dkbar, dD = g.bwd()
    dk_raw = torch.empty_like(g.k)
    lc.longconv_kreg_bwd(d_kraw, d_mask, g.dk, dk_raw, p, lam)
    torch.cuda.synchronize()
    m64 = None if mask is None else mask.astype(np.float64)
    lam64 = float(np.float32(lam))
    kbar = kreg.kernel_reg_fwd(kraw.astype(np.float64), m64, p, lam64)
    D64 = inp.D.astype(np.float64)
    ry = oracle.longconv_fwd(inp.u, kbar, D64)
    rdu, rdkbar, rdD = oracle.longconv_bwd(inp.dy, inp.u, kbar, D64)
    rdk = kreg.kernel_reg_bwd(kraw.astype(np.float64), m64, p, lam64, rdkbar)
    tol = TOL[inp.w.dtype]
    errs = {"y": wl.rel_l2(y, ry), "du": wl.rel_l2(du, rdu), "dk_raw": wl.rel_l2(dk_raw.cpu().numpy(), rdk)}
    print("[kreg end to end] " + " ".join(f"{a}={b:.2e}" for a, b in errs.items()), flush=True)
    for name, e in errs.items():
        assert e <= tol, f"{name}: {e:.3e}"


# a wave takes 256 entries and their halo: the narrowest and widest windows with one and with several of them in a row
@pytest.mark.parametrize("N", [256, 1024])
@pytest.mark.parametrize("p", [1, 15, 16, 31, 32])
def test_windows_across_waves(N, p):
    test_regularisers_forward_and_chain_against_oracle(3, N, p, 0.002, 0.2)


def test_closed_gate_drops_any_gradient():
    import paper_2302_06646_amd as lc
    k = torch.zeros(2, 512, device="cuda")
    k[:, 300] = 1.0
    g = torch.full_like(k, float("nan"))
    g[:, 296:305] = 1.0
    dk = torch.full_like(k, float("nan"))
    lc.longconv_kreg_bwd(k, None, g, dk, 2, 0.1)
    assert torch.isfinite(dk).all()
    want = torch.zeros(2, 512)
    for n in range(298, 303):                            # K2 = 1/5 > lambda there, zero elsewhere
        want[:, n - 2:n + 3] += 0.2
    assert torch.allclose(dk.cpu(), want, atol=1e-6)
