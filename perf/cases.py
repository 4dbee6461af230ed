"""The work that programs using this library have it do, as cases to be timed and compared.

A case names one of five paths through the public entry points:

  step     one layer of one training step: (regularised kernel ->) spectrum -> forward -> backward with all gradients
           (-> gradient of the raw kernel); the kernel changes every step, so the spectrum belongs to the pass
  fwd      inference with a spectrum computed once and kept
  gated    the training step of the gated layer
  image    the training step of the 2-D layer
  learned  the training step of the layer with learned Butterfly blocks

All tensors, workspaces and (fwd) the cached spectrum are what such a program keeps from call to call, so `prepare`
makes them and `run` only calls the library.  Lengths are powers of two (the library's own limit); batch and head
counts are anything.
"""
import math

import numpy as np
import torch

import paper_2302_06646_amd as lc

_IO = {"fp32": (lc.F32, torch.float32, 4), "fp16": (lc.F16, torch.float16, 2), "bf16": (lc.BF16, torch.bfloat16, 2)}


def listed():
    return [
        # the smallest training step there is a configuration for: nothing but launches and host work
        dict(name="tiny_step_fp32", path="step", B=2, H=4, N=1024, io="fp32", kernel="decay256", reg=False, grad=1.0),
        # one sequence through one layer of language-model width, kernel fixed: latency of a serving call
        dict(name="serve_one_bf16", path="fwd", B=1, H=768, N=1024, io="bf16", kernel="squash_pool"),
        # many short sequences: the low end of the wide sweep
        dict(name="short_step_bf16", path="step", B=64, H=1024, N=256, io="bf16", kernel="squash_pool", reg=False,
             grad=1.0),
        # language-model block, Algorithm 1 whole: dropout, smooth and squash of the kernel around the convolution
        dict(name="lm_step_bf16", path="step", B=16, H=768, N=1024, io="bf16", kernel="raw", reg=True, grad=1.0),
        # gated layer, odd batch and head counts, gradients as small as a mean loss makes them
        dict(name="gated_odd_bf16", path="gated", B=7, H=193, N=2048, io="bf16", kernel="squash_pool", grad=1e-4),
        # the largest: the high end of the wide sweep
        dict(name="wide_step_bf16", path="step", B=64, H=1024, N=4096, io="bf16", kernel="squash_pool", reg=False,
             grad=1.0),
        # long-range task, the headline benchmark
        dict(name="long16k_step_fp16", path="step", B=8, H=256, N=16384, io="fp16", kernel="decay_alpha_squash",
             reg=False, grad=1.0),
        # inference past the on-chip length, the length sweep's shape
        dict(name="long32k_fwd_fp16", path="fwd", B=32, H=128, N=32768, io="fp16", kernel="decay4"),
        # one very long sequence (the longest task)
        dict(name="one64k_step_fp16", path="step", B=1, H=128, N=65536, io="fp16", kernel="decay4", reg=False,
             grad=1.0),
        # full precision past the on-chip length of the fp32 engine
        dict(name="long8k_step_fp32", path="step", B=4, H=96, N=8192, io="fp32", kernel="decay256", reg=False,
             grad=1.0),
        # image layer on 32 x 32 images
        dict(name="image32_step_bf16", path="image", B=64, H=256, N1=32, N2=32, io="bf16", grad=1.0),
        # learned transforms at the language-model block's shape
        dict(name="learned_step_bf16", path="learned", B=16, H=768, N=1024, io="bf16", grad=1.0),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the same paths: any supported length, 1 ... 64 sequences, 4 ... 1024 heads, all three I/O types, as
    much work as the largest listed case at most (paths whose work per sample is higher get fewer samples)."""
    path = rng.choice(["step", "step", "step", "fwd", "fwd", "gated", "image", "learned"])
    c = dict(path=path)
    if path == "image":
        c["N1"] = 1 << rng.randint(4, 8)
        c["N2"] = min(256, max(8, c["N1"] * rng.choice([1, 1, 2]) // rng.choice([1, 1, 2])))
        while c["N1"] * c["N2"] < 128:
            c["N2"] *= 2
        n, per_sample = c["N1"] * c["N2"], 12
        c["io"] = rng.choice(["bf16", "bf16", "fp16"])
    elif path == "learned":
        n, per_sample = 1 << rng.randint(8, 11), 8
        c["N"] = n
        c["io"] = rng.choice(["bf16", "fp16"])
    else:
        c["io"] = rng.choice(["bf16", "bf16", "fp16", "fp16", "fp32"]) if path != "gated" else rng.choice(["bf16", "fp16"])
        n = 1 << (rng.randint(8, 15) if c["io"] == "fp32" else rng.randint(8, 17))
        c["N"] = n
        per_sample = 24 if c["io"] == "fp32" else (8 if n > 16384 else 1) * (2 if path == "gated" else 1)
        c["kernel"] = "squash_pool" if n <= 4096 else rng.choice(["decay_alpha_squash", "decay4"])
    most = (1 << 28) // per_sample // n
    c["B"] = _log_int(rng, 1, min(64, most))
    c["H"] = _log_int(rng, 4, max(4, min(1024, most // c["B"])))
    if path == "step":
        c["reg"] = rng.random() < 0.3
        if c["reg"]:
            c["kernel"] = "raw"
    if path != "fwd":
        c["grad"] = rng.choice([1.0, 1e-4]) if c["io"] == "bf16" and path != "learned" else 1.0
    return c


_P, _LAMBDA, _KEEP = 1, 0.003, 0.8      # smoothing half width, squash threshold, dropout's share of kept taps


def _kernel(kind, H, N, randn, rand):
    """The synthetic kernels of the workloads module, drawn on the device."""
    t = torch.arange(N, device="cuda", dtype=torch.float32)[None, :]
    squash = lambda k, lam: torch.sign(k) * torch.clamp(k.abs() - lam, min=0.0)
    if kind == "decay256":
        return randn(H, N) * torch.exp(-t / 256.0)
    if kind == "raw":
        return 0.02 * randn(H, N)
    if kind == "squash_pool":
        p = torch.nn.functional.pad(squash(0.02 * randn(H, N), 0.003), (1, 1))
        return ((p[:, :-2] + p[:, 1:-1] + p[:, 2:]) / 3.0).contiguous()
    if kind == "decay_alpha_squash":
        a = 0.5 + 7.5 * rand(H, 1)
        return squash(randn(H, N) / N ** 0.5 * torch.exp(-a * t / N), 1e-4)
    if kind == "decay4":
        return randn(H, N) / N ** 0.5 * torch.exp(-4.0 * t / N)
    raise ValueError(kind)


def _blocks(H, N, sign, randn):
    """Learned blocks some way into training: the DFT's (or its conjugate's) moved by a tenth."""
    A = np.zeros((3, 16, 16, 2), dtype=np.float32)
    mask = np.zeros((3, 16, 16, 1), dtype=np.float32)
    for s, r in enumerate((16, 16, 2 * N // 256)):
        F = np.exp(sign * 2j * np.pi * np.outer(np.arange(r), np.arange(r)) / r)
        A[s, :r, :r, 0], A[s, :r, :r, 1] = F.real, F.imag
        mask[s, :r, :r] = 1.0
    return torch.from_numpy(A).cuda() + 0.1 * torch.from_numpy(mask).cuda() * randn(H, 3, 16, 16, 2)


def prepare(case, seed):
    c, path = case, case["path"]
    io, td, _ = _IO[c["io"]]
    B, H = c["B"], c["H"]
    shape = (B, H, c["N1"], c["N2"]) if path == "image" else (B, H, c["N"])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    randn = lambda *n: torch.randn(*n, generator=gen, device="cuda")
    rand = lambda *n: torch.rand(*n, generator=gen, device="cuda")
    half = lambda x: x if td == torch.float32 else x.to(td)
    s = dict(path=path, io=io)
    s["u"] = half(randn(*shape))
    s["y"] = torch.empty_like(s["u"])
    s["D"] = randn(H)
    if path == "image":
        s["k"] = randn(H, c["N1"], c["N2"]) / (c["N1"] * c["N2"]) ** 0.5
        s["ws"] = lc.new_workspace2d(B, H, c["N1"], c["N2"], io, True)
    elif path == "learned":
        N = c["N"]
        s["k"] = _kernel("decay4", H, N, randn, rand)
        s["Af"], s["Ai"] = _blocks(H, N, -1, randn), _blocks(H, N, +1, randn)
        s["shat"] = torch.empty(H, 2 * N, 2, device="cuda")
        s["dAf"], s["dAi"], s["dshat"] = (torch.empty_like(s[n]) for n in ("Af", "Ai", "shat"))
        s["ws"] = torch.empty(lc.longconv_lbfly_workspace_bytes(B, H, N, io), dtype=torch.uint8, device="cuda")
    else:
        N = c["N"]
        s["k"] = _kernel(c["kernel"], H, N, randn, rand)
        s["ks"] = lc.new_kspec(H, N, io)
        s["ws"] = lc.new_workspace(B, H, N, io, {"fwd": 0, "step": 1, "gated": 2}[path])
    if path == "fwd":
        lc.longconv_kspec_compute(s["k"], s["D"], s["ks"], io, s["ws"])
        return s
    s["dy"] = half(c["grad"] * randn(*shape))
    s["du"], s["dk"], s["dD"] = (torch.empty_like(s[n]) for n in ("u", "k", "D"))
    if path == "gated":
        s["g"] = half(randn(*shape))
        s["dg"] = torch.empty_like(s["u"])
    s["reg"] = bool(c.get("reg"))
    if s["reg"]:
        s["mask"] = (rand(H, c["N"]) < _KEEP).float() / _KEEP
        s["kbar"], s["dkbar"] = torch.empty_like(s["k"]), torch.empty_like(s["k"])
    return s


def run(s):
    u, k, D, y, ws, path = s["u"], s["k"], s["D"], s["y"], s["ws"], s["path"]
    if path == "fwd":
        lc.longconv_fwd(u, k, D, y, ws, kspec=s["ks"])
        return {"y": y}
    dy, du, dk, dD = s["dy"], s["du"], s["dk"], s["dD"]
    out = {"y": y, "du": du, "dk": dk, "dD": dD}
    if path == "step":
        ks = s["ks"]
        if s["reg"]:
            lc.longconv_kreg_fwd(k, s["mask"], s["kbar"], _P, _LAMBDA)
            lc.longconv_kspec_compute(s["kbar"], D, ks, s["io"], ws)
            lc.longconv_fwd(u, s["kbar"], D, y, ws, kspec=ks)
            lc.longconv_bwd(dy, u, s["kbar"], D, du, s["dkbar"], dD, ws, kspec=ks)
            lc.longconv_kreg_bwd(k, s["mask"], s["dkbar"], dk, _P, _LAMBDA)
        else:
            lc.longconv_kspec_compute(k, D, ks, s["io"], ws)
            lc.longconv_fwd(u, k, D, y, ws, kspec=ks)
            lc.longconv_bwd(dy, u, k, D, du, dk, dD, ws, kspec=ks)
    elif path == "gated":
        ks = s["ks"]
        lc.longconv_kspec_compute(k, D, ks, s["io"], ws)
        lc.longconv_fwd_gated(u, k, D, s["g"], y, ws, kspec=ks)
        lc.longconv_bwd_gated(dy, s["g"], u, k, D, du, dk, dD, s["dg"], ws, kspec=ks)
        out["dg"] = s["dg"]
    elif path == "image":
        lc.longconv2d_fwd(u, k, D, y, ws)
        lc.longconv2d_bwd(dy, u, k, D, du, dk, dD, ws)
    else:
        lc.longconv_lbfly_spectrum(k, D, s["shat"])
        lc.longconv_lbfly_fwd(u, s["shat"], s["Af"], s["Ai"], y)
        lc.longconv_lbfly_bwd(dy, u, s["shat"], s["Af"], s["Ai"], du, s["dshat"], s["dAf"], s["dAi"], ws)
        lc.longconv_lbfly_spectrum_bwd(s["dshat"], dk, dD)
        out.update(dshat=s["dshat"], dAf=s["dAf"], dAi=s["dAi"])
    return out


def _fft_flops(B, H, N):
    """Forward and backward operation counts: 2.5 L log2 L for a real transform of L = 2N points."""
    lg, rows = math.log2(2 * N), B * H
    return rows * (10 * N * lg + 8 * N), rows * (15 * N * lg + 18 * N) + H * 5 * N * lg


def work(case):
    """Tensors of the caller read or written once (u, y, dy, du, gate; k, dk, D, dD, masks, blocks in fp32; not the
    spectrum, which is k again), and the transforms' operation counts; for the learned layer the block products
    themselves (three times the forward's: forward, rows' and blocks' gradients)."""
    c, path = case, case["path"]
    B, H, sz = c["B"], c["H"], _IO[c["io"]][2]
    N = c["N1"] * c["N2"] if path == "image" else c["N"]
    rows, par = B * H * N * sz, H * N * 4 + H * 4
    if path == "fwd":
        return {"bytes": 2 * rows + par, "flops": _fft_flops(B, H, N)[0]}
    nbytes, flops = 4 * rows + 2 * par, sum(_fft_flops(B, H, N))
    # (u is read once for the forward and the backward pass together: 4 tensors, not 5)
    if path == "gated":
        nbytes += 2 * rows
        flops += _fft_flops(B, H, N)[0] / 2 + 3 * B * H * N
    elif path == "image":
        flops *= 2                                          # twice the points: padded in both directions
    elif path == "learned":
        L = 2 * N
        nbytes += 4 * H * 3 * 16 * 16 * 2 * 4
        flops = 3.0 * B * H * 2 * 8 * L * (16 + 16 + L // 256)
    elif c["reg"]:
        nbytes += H * N * 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """fp32 I/O is fp32 throughout.  fp16 / bf16 I/O computes with fp16 operands and fp32 sums (about 1e-3 in either
    implementation) and rounds its results to the I/O type (1.6e-3 for bf16); the learned layer chains more
    roundings of its blocks and rows."""
    if case["io"] == "fp32":
        return {"rel": 1e-5}
    return {"rel": 5e-3 if case["path"] == "learned" else 4e-3}
