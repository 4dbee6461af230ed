"""bf16 rows far outside fp16's exponent range (the transforms carry fp16 between their stages): tiny gradients,
large activations, rows of one head that differ by many orders of magnitude.  Every row (y, du) and every head
(dk, dD) must meet the same bound as data of order one."""
import dataclasses

import numpy as np
import pytest

import workloads as wl
from gpu_harness import check_full

pytestmark = pytest.mark.gpu


def scaled_inputs(N, B, H, u_scale, dy_scale, k_scale=None, D_scale=None, seed=0, dtype=wl.BF16):
    """Workload-2 style inputs (bf16 unless said otherwise); row (b,h) of u is multiplied by u_scale[b,h]
    (broadcast), likewise dy; head h of k by k_scale[h] and D[h] by D_scale[h]; u and dy are rounded to the I/O
    dtype again afterwards."""
    w = wl.Workload(2, B, H, N, dtype, "squash_pool")
    inp = wl.generate(w, seed_extra=seed)
    us = np.broadcast_to(np.asarray(u_scale, dtype=np.float64), (B, H))[:, :, None]
    ds = np.broadcast_to(np.asarray(dy_scale, dtype=np.float64), (B, H))[:, :, None]
    u_s, u_v = wl.quantize((inp.u * us).astype(np.float32), dtype)
    dy_s, dy_v = wl.quantize((inp.dy * ds).astype(np.float32), dtype)
    k, D = inp.k, inp.D
    if k_scale is not None:
        k = (k.astype(np.float64) * np.asarray(k_scale, dtype=np.float64)[:, None]).astype(np.float32)
    if D_scale is not None:
        D = (D.astype(np.float64) * np.asarray(D_scale, dtype=np.float64)).astype(np.float32)
    return dataclasses.replace(inp, u_store=u_s, dy_store=dy_s, u=u_v, dy=dy_v, k=k, D=D)


LENGTHS = [256, 512, 1024, 2048, 4096, 8192, 16384]      # every single-pass plan


@pytest.mark.parametrize("N", LENGTHS)
def test_tiny_gradients_and_large_activations(N):
    # dy ~ N(0, 1e-10) (standard deviation 1e-5), u ~ N(0, 1e6)
    check_full(scaled_inputs(N, 5, 3, 1e3, 1e-5), label=f"u 1e3, dy 1e-5, N={N}")


@pytest.mark.parametrize("N", LENGTHS)
def test_rows_of_one_head_at_very_different_magnitudes(N):
    B, H = 6, 2
    rng = np.random.default_rng(7 + N)
    us = 10.0 ** (rng.choice([-1, 1], size=(B, H)) * rng.uniform(2, 8, size=(B, H)))
    ds = 10.0 ** np.where(rng.random((B, H)) < 0.7, rng.uniform(-12, -3, size=(B, H)), rng.uniform(2, 4, size=(B, H)))
    us[0, 0], ds[0, 0] = 1.0, 1.0            # rows inside the band next to the others
    us[3, 1], ds[2, 0] = 1.0, 1.0
    check_full(scaled_inputs(N, B, H, us, ds, seed=1), label=f"mixed magnitudes, N={N}")


@pytest.mark.parametrize("N", [32768, 65536])
def test_multi_pass_lengths_scale_per_head(N):
    # the multi-pass plans rescale per head (all rows of a head by one power of two): uniform tiny gradients and
    # large activations, and heads at very different magnitudes
    check_full(scaled_inputs(N, 3, 2, 1e3, 1e-5), label=f"u 1e3, dy 1e-5, N={N}")
    us = np.array([[1e-6, 3e4]])
    ds = np.array([[2e-9, 1.0]])
    check_full(scaled_inputs(N, 2, 2, us, ds, seed=2), label=f"heads at different magnitudes, N={N}")


# The stored spectrum is fp16: a head whose spectrum lies outside fp16's comfortable range is stored with a power of
# two taken out, which the convolution kernels give back where they pack their output.  One wave length, the
# cooperative lengths and two multi-pass lengths; every row of every head to the bound of data of order one.
@pytest.mark.parametrize("N", [256, 1024, 4096, 16384, 65536, 131072])
def test_kernels_of_any_magnitude_bf16(N):
    B = 3 if N <= 16384 else 2
    ks = np.array([2.0 ** -20, 2.0 ** 20, 1.0, 2.0 ** -30, 2.0 ** 12, 1e-3, 3e4])
    Ds = np.array([2.0 ** -20, 2.0 ** 20, 1.0, 1.0, 2.0 ** -5, 1e3, 3e-4])      # skip term with, above and below the kernel
    H = len(ks) if N <= 16384 else 4
    check_full(scaled_inputs(N, B, H, 1.0, 1.0, k_scale=ks[:H], D_scale=Ds[:H], seed=3), label=f"kernel magnitudes, N={N}")


@pytest.mark.parametrize("N", [512, 8192, 32768])
def test_kernels_of_other_magnitudes_fp16(N):
    # fp16 rows and outputs have to stay inside fp16's own range: heads at 2^-9 and 2^9 with rows of order one
    ks = np.array([2.0 ** -9, 2.0 ** 9, 1.0, 2.0 ** -6])
    check_full(scaled_inputs(N, 3, 4, 1.0, 1.0, k_scale=ks, D_scale=ks, seed=4, dtype=wl.F16), label=f"kernel magnitudes fp16, N={N}")


def test_kernel_magnitude_with_rows_out_of_band():
    # both rescalings at once on a single-pass plan: tiny gradients, large activations and kernels far from one
    ks = np.array([2.0 ** -18, 2.0 ** 15, 1.0])
    check_full(scaled_inputs(2048, 4, 3, 1e3, 1e-5, k_scale=ks, D_scale=ks, seed=5), label="rows and kernels out of range, N=2048")
    check_full(scaled_inputs(16384, 3, 3, 1e3, 1e-5, k_scale=ks, D_scale=ks, seed=6), label="rows and kernels out of range, N=16384")


@pytest.mark.parametrize("N", [256, 1024, 2048, 8192, 16384])
def test_rows_of_a_pair_a_few_times_apart(N):
    # the two rows of a pair share one complex transform, so the rounding of the larger is an error of the smaller:
    # rows that differ by a factor of four and more have to be scaled one by one even when both are of "ordinary"
    # size, and a row of ordinary size next to one that needs scaling anyway is scaled with it
    B, H = 8, 3
    us = np.ones((B, H)); ds = np.ones((B, H))
    us[0:2, 0] = [0.1, 1.0]; us[2:4, 0] = [3.5, 0.09]; us[4:6, 0] = [0.3, 1e4]; us[6:8, 0] = [0.26, 3.9]
    ds[0:2, 0] = [1.0, 0.08]; ds[2:4, 0] = [0.3, 3e-6]; ds[4:6, 0] = [2.0, 0.5]; ds[6:8, 0] = [0.07, 0.9]
    rng = np.random.default_rng(11 + N)
    us[:, 1] = 10.0 ** rng.uniform(-1.2, 1.2, size=B); ds[:, 1] = 10.0 ** rng.uniform(-1.2, 1.2, size=B)
    us[:, 2] = 10.0 ** rng.uniform(-6, 6, size=B); ds[:, 2] = 10.0 ** rng.uniform(-9, 3, size=B)
    check_full(scaled_inputs(N, B, H, us, ds, seed=7), label=f"rows a few times apart, N={N}")


def _random_magnitude_cases(n, seed):
    rng = np.random.default_rng(seed)
    lengths = [256, 512, 1024, 2048, 4096, 8192, 16384, 32768, 65536]
    p = np.array([4, 4, 4, 4, 3, 3, 2, 1, 1], dtype=float)
    cases = []
    for _ in range(n):
        N = int(rng.choice(lengths, p=p / p.sum()))
        B = int(rng.integers(1, 12)) if N <= 4096 else int(rng.integers(1, 5))
        H = int(rng.integers(1, 7)) if N <= 16384 else int(rng.integers(1, 3))
        cases.append((N, B, H, int(rng.integers(0, 10000)), bool(rng.integers(0, 2))))
    return cases


@pytest.mark.parametrize("N,B,H,seed,kernels", _random_magnitude_cases(48, 20230213))
def test_random_magnitudes(N, B, H, seed, kernels):
    # rows at 10^-6 ... 10^6 (u) and 10^-9 ... 10^3 (dy), drawn row by row up to N = 16384 and head by head beyond (the
    # multi-pass plans scale per head), kernels and skip terms at 2^-24 ... 2^20 in half of the cases: y, du and dk to
    # the bound of data of order one, every row and head.  dD is a plain fp32 dot product over all rows of a head:
    # where rows of wildly different size meet in one sum its relative error reaches a few 1e-5 (1e-7 otherwise).
    rng = np.random.default_rng(seed)
    shape = (B, H) if N <= 16384 else (1, H)
    us = np.broadcast_to(10.0 ** rng.uniform(-6, 6, size=shape), (B, H)).copy()
    ds = np.broadcast_to(10.0 ** rng.uniform(-9, 3, size=shape), (B, H)).copy()
    ks = 2.0 ** rng.integers(-24, 20, size=H) if kernels else None
    Ds = 2.0 ** rng.integers(-24, 20, size=H) if kernels else None
    check_full(scaled_inputs(N, B, H, us, ds, k_scale=ks, D_scale=Ds, seed=seed), label=f"random magnitudes, N={N}", dd_tol=1e-4)


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("N", [256, 512, 1024, 2048, 4096])
def test_dk_of_rows_with_a_mean(N, io):
    # Rows with a mean add up in the first bins of dk's accumulator: rows of constant 4 reach 4 * 4 * 24 * 207 = 79000
    # at N = 256 and 512, and more beyond (fp16 ends at 65504), while dk itself is an ordinary fp32 number.  Heads enough
    # that one workgroup has all rows of a head; every other head's rows carry noise around the mean, one head's dy
    # is small.
    from gpu_harness import GpuRun, TOL, _compare
    import oracle
    B, H = 24, 129 if N == 4096 else 257
    inp = wl.generate(wl.Workload(2, B, H, N, io, "squash_pool"))
    u, dy = inp.u + 4.0, inp.dy + 4.0
    u[:, ::2] = dy[:, ::2] = 4.0
    dy[:, 3] = 2.0 ** -10
    (u_s, u_v), (dy_s, dy_v) = wl.quantize(u.astype(np.float32), io), wl.quantize(dy.astype(np.float32), io)
    g = GpuRun(dataclasses.replace(inp, u_store=u_s, dy_store=dy_s, u=u_v, dy=dy_v))
    heads = [0, 1, 2, 3, H - 1]
    want = oracle.longconv_bwd(dy_v[:, heads], u_v[:, heads], inp.k[heads].astype(np.float64), inp.D[heads].astype(np.float64))[1]
    for du in (True, False):                 # du, dk and dD from one kernel, and dk by itself
        dk = g.bwd(du=du)[1]
        assert np.all(np.isfinite(dk))
        _compare({"dk": dk[heads]}, {"dk": want}, TOL[io], f"rows with a mean, N={N} io={wl.DTYPE_NAMES[io]} du={du}")


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("N", [256, 512, 1024, 2048, 4096, 32768, 65536])
def test_outputs_of_rows_with_a_mean(N, io):
    # A row of mean A meets sum k in the first bin: as 2N zero-padded points A sum k 2^(s-1), s the log2 of the transform's
    # scale, which may come up to 0.9 of fp16's 65504; the N twisted points of single rows must leave as much room.
    s = {256: 4, 512: 5, 1024: 5, 2048: 6, 4096: 6}.get(N, 7)
    A, B, H = 8.0, 3, 2
    K = 0.9 * 65504 / 2 ** (s - 1) / A
    inp = wl.generate(wl.Workload(2, B, H, N, io, "squash_pool"))
    (u_s, u_v), (dy_s, dy_v) = (wl.quantize((A + x).astype(np.float32), io) for x in (0.1 * inp.u, 0.1 * inp.dy))
    k, D = inp.k.copy(), inp.D.copy()
    k -= k.mean(axis=1, keepdims=True)           # (sum k is K: the taps' noise has no mean of its own)
    k[:, 0] += K / 2
    D[:] = K / 2
    from gpu_harness import GpuRun, TOL, _compare
    import oracle
    g = GpuRun(dataclasses.replace(inp, u_store=u_s, dy_store=dy_s, u=u_v, dy=dy_v, k=k, D=D))
    k64, D64 = k.astype(np.float64), D.astype(np.float64)
    _compare({"y": g.fwd(), "du": g.bwd(dk=False, dD=False)[0]},
             {"y": oracle.longconv_fwd(u_v, k64, D64), "du": oracle.longconv_bwd(dy_v, u_v, k64, D64)[0]}, TOL[io],
             f"outputs of rows with a mean, N={N} io={wl.DTYPE_NAMES[io]}")


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("N,B,H", [(256, 18, 1200), (512, 9, 1200), (1024, 9, 1100), (2048, 7, 800), (4096, 7, 400)])
def test_long_runs_of_rows_and_heads_of_other_magnitudes(N, B, H, io):
    # Workgroups with many rows: the kernels have code of their own for the middle of a run, with and without powers of
    # two, which shapes of a few rows do not reach.  More rows than four times what the device holds at once, heads whose
    # spectrum has a power of two taken out next to ordinary ones, and (bf16) rows out of band or zero anywhere.
    from gpu_harness import GpuRun, TOL, _compare
    import oracle
    rng = np.random.default_rng(31 + N)
    ks = np.where(rng.random(H) < 0.3, 2.0 ** rng.integers(-9, 9, size=H), 1.0)
    us = ds = np.ones((B, H))
    if io == wl.BF16:
        us = np.where(rng.random((B, H)) < 0.3, 10.0 ** rng.uniform(-6, 6, size=(B, H)), 1.0)
        ds = np.where(rng.random((B, H)) < 0.3, 10.0 ** rng.uniform(-9, 3, size=(B, H)), 1.0)
        us[rng.random((B, H)) < 0.05] = 0.0
        ds[rng.random((B, H)) < 0.05] = 0.0
    inp = scaled_inputs(N, B, H, us, ds, k_scale=ks, D_scale=ks, seed=8, dtype=io)
    heads = sorted({0, 1, H // 3, H // 3 + 1, H // 2, H - 1, int(np.argmin(ks)), int(np.argmax(ks))})
    g = GpuRun(inp)
    got = dict(zip(("y", "du", "dk", "dD"), (g.fwd(), *g.bwd())))
    assert all(np.all(np.isfinite(v)) for v in got.values())
    k64, D64 = inp.k[heads].astype(np.float64), inp.D[heads].astype(np.float64)
    want = dict(zip(("y", "du", "dk", "dD"), (oracle.longconv_fwd(inp.u[:, heads], k64, D64),
                                              *oracle.longconv_bwd(inp.dy[:, heads], inp.u[:, heads], k64, D64))))
    got = {n: v[:, heads] if v.ndim == 3 else v[heads] for n, v in got.items()}
    # (dD: rows of wildly different size meet in one fp32 dot product, see test_random_magnitudes)
    _compare(got, want, TOL[io], f"long runs, N={N} B={B} H={H} io={wl.DTYPE_NAMES[io]}", dd_tol=1e-4)


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
def test_rows_of_one_head_apart_at_32768(io):
    # y and du are scaled row by row there, dk head by head: rows far apart in size, the largest u with the largest dy (a
    # head's dk is then that row's, and the others' share of it lies far below the bound)
    us, ds = np.array([[1.0], [1e3], [1e-4]]), np.array([[1.0], [1e2], [1e-5]])
    if io == wl.F16:
        us, ds = np.array([[1.0], [8.0], [0.25]]), np.array([[0.5], [4.0], [1.0]])
    check_full(scaled_inputs(32768, 3, 2, us, ds, seed=9, dtype=io), label="rows of one head apart", dd_tol=1e-4)


# One sample outside the band in a row that otherwise lies inside it: the waves that hold the row decide by themselves whether it
# has to be scaled, each from its own words, and a single word has to be enough.  Of either sign (bf16 patterns above 2^121 are NaN
# when read as fp16, where the maximum of |x| is taken), in the first or the last wave's words, in u alone or in dy alone: head
# 4 place + 2 sign + tensor, rows inside the band around it.
# Outputs are cut from a linear convolution of 2N samples, and the rounding of a transform is relative to all of it: of a sample six
# before a row's end six samples are kept.  Rows (dk: heads) are held to the usual bound, relative to what they were cut from.
@pytest.mark.parametrize("power", [4, 100, 122])
@pytest.mark.parametrize("N,gate", [(2048, False), (4096, False), (1024, True), (2048, True)])
def test_one_sample_out_of_band(N, gate, power):
    from gpu_harness import GpuRun, TOL
    import oracle
    from oracle import gated
    from test_gated_gpu import _run
    B, H, io = 3, 8, wl.BF16
    inp = wl.generate(wl.Workload(2, B, H, N, io, "squash_pool"))
    u, dy = inp.u.copy(), inp.dy.copy()
    for h in range(H):
        x, at = (u, dy)[h & 1], (5, N - 6)[h >> 2]
        x[h % B, h, at] = (1.0, -1.0)[(h >> 1) & 1] * 2.0 ** power
    (u_s, u_v), (dy_s, dy_v) = wl.quantize(u.astype(np.float32), io), wl.quantize(dy.astype(np.float32), io)
    inp = dataclasses.replace(inp, u_store=u_s, dy_store=dy_s, u=u_v, dy=dy_v)
    k64, D64 = inp.k.astype(np.float64), inp.D.astype(np.float64)
    norm = lambda x: np.linalg.norm(x, axis=-1)
    f = lambda x: np.fft.fft(x, 2 * N)
    kd = k64.copy()
    kd[:, 0] += D64
    g_v = np.ones((B, H, N))
    if gate:
        g_s, g_v = wl.quantize(np.broadcast_to(np.where(np.arange(N) % 3 == 1, -1.0, 1.0), (B, H, N)).astype(np.float32), io)
        got = dict(zip(("y", "du", "dk", "dD", "dg"), _run(inp, g_s)))
    else:
        g = GpuRun(inp)
        got = dict(zip(("y", "du", "dk", "dD"), (g.fwd(), *g.bwd())))
    want = dict(zip(("du", "dk", "dD", "dg"), gated.gated_bwd(dy_v, g_v, u_v, k64, D64)), y=gated.gated_fwd(u_v, k64, D64, g_v))
    whole = {"y": norm(np.fft.ifft(f(u_v) * f(kd))), "du": norm(np.fft.ifft(f(dy_v * g_v) * f(kd).conj())),
             "dk": norm(np.fft.ifft((f(dy_v * g_v) * f(u_v).conj()).sum(axis=0)))}
    whole["dg"] = np.maximum(norm(want["dg"]), norm(dy_v) * whole["y"] / (2 * N) ** 0.5)
    errs = {n: float(np.max(norm(got[n] - want[n]) / whole[n])) for n in got if n != "dD"}
    errs["dD"] = float(np.max(np.abs(got["dD"] - want["dD"]) / (norm(norm(u_v).T) * norm(norm(dy_v).T))))
    print(f"[parity] one sample of 2^{power}, N={N} gate={gate}: " + " ".join(f"{n}={e:.2e}" for n, e in errs.items()), flush=True)
    for n, e in errs.items():
        assert np.isfinite(e) and e <= (1e-6 if n == "dD" else TOL[io]), f"{n}: {e:.3e}"
