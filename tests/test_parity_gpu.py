"""GPU parity: the HIP path, called through the C ABI, against the float64 CPU oracle on the
same seeded inputs.  Bounds: relative L2 <= 1e-5 (fp32 I/O), <= 3e-3 (fp16/bf16 I/O)."""
import dataclasses
import os

import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu_and_default_options():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2302_06646_amd as lc
    for name, value in lc.OPTION_DEFAULTS.items():      # whatever the environment or an earlier test left
        lc.longconv_set_option(name, value)
    yield
    for name, value in lc.OPTION_DEFAULTS.items():
        lc.longconv_set_option(name, value)


def _opt(name, value):
    import paper_2302_06646_amd as lc
    lc.longconv_set_option(name, value)


def _w(key, **kw):
    return dataclasses.replace(wl.WORKLOADS[key], **kw)


def test_cfg1_fp32_full():
    from gpu_harness import check_full
    check_full(wl.generate(wl.WORKLOADS["1"]))


@pytest.mark.parametrize("key,B,H", [("2", 4, 6), ("2", 3, 2), ("5_256", 6, 5), ("5_512", 4, 4),
                                     ("5_2048", 4, 3), ("5_4096", 2, 3), ("3", 4, 2), ("3", 1, 2)])
def test_reduced_configs_half_io(key, B, H):
    from gpu_harness import check_full
    check_full(wl.generate(wl.WORKLOADS[key], B=B, H=H))


@pytest.mark.parametrize("N", [256, 512, 2048, 4096, 8192])
def test_fp32_lengths(N):
    from gpu_harness import check_full
    check_full(wl.generate(_w("1", N=N), B=3, H=2))


@pytest.mark.parametrize("key", ["4a", "4b"])
def test_cfg4_long_sequences_multipass(key):
    from gpu_harness import check_full
    check_full(wl.generate(wl.WORKLOADS[key], H=2))


@pytest.mark.parametrize("N,io", [(16384, wl.F32), (65536, wl.F32), (32768, wl.BF16)])
def test_other_long_sequences(N, io):
    from gpu_harness import check_full
    check_full(wl.generate(_w("4a", N=N, dtype=io), B=2, H=2))


@pytest.mark.parametrize("engine", ["valu", "mfma"])
@pytest.mark.parametrize("inner", [9, 10])
def test_forced_multipass_small(engine, inner):
    # the multi-pass split exercised at a size the oracle checks in full
    from gpu_harness import check_full
    _opt("engine", {"valu": 1, "mfma": 2}[engine])
    _opt("inner_log2", inner)
    io = wl.F32 if engine == "valu" else wl.F16
    check_full(wl.generate(_w("1", N=2048, dtype=io), B=3, H=3), label=f"{engine} inner=2^{inner}")


@pytest.mark.parametrize("key,B,H", [("2", 5, 3), ("3", 2, 2), ("5_4096", 3, 2)])
def test_staged_matrix_core_kernel(key, B, H):
    # the in-place staged kernel (normally only used for 256-point transforms) forced at other lengths
    from gpu_harness import check_full
    _opt("staged_kernel", 1)
    check_full(wl.generate(wl.WORKLOADS[key], B=B, H=H), label="staged")


def test_valu_engine_with_half_io():
    from gpu_harness import check_full
    _opt("engine", 1)
    check_full(wl.generate(wl.WORKLOADS["2"], B=3, H=3))
    check_full(wl.generate(wl.WORKLOADS["3"], B=2, H=2))


@pytest.mark.parametrize("key", ["1", "2"])
def test_cached_spectrum_equals_on_the_fly_and_runs_are_bitwise_repeatable(key):
    from gpu_harness import GpuRun
    g = GpuRun(wl.generate(wl.WORKLOADS[key], B=4, H=4))
    y0 = g.fwd().copy()
    du0, dk0, dD0 = [a.copy() for a in g.bwd()]
    ks = g.kspec()
    assert np.array_equal(g.fwd(kspec=ks), y0)
    du1, dk1, dD1 = g.bwd(kspec=ks)
    assert np.array_equal(du1, du0) and np.array_equal(dk1, dk0) and np.array_equal(dD1, dD0)
    for _ in range(3):
        du2, dk2, dD2 = g.bwd()
        assert np.array_equal(dk2, dk0) and np.array_equal(dD2, dD0) and np.array_equal(du2, du0)


def test_optional_gradients():
    from gpu_harness import GpuRun
    g = GpuRun(wl.generate(wl.WORKLOADS["2"], B=2, H=2))
    du, dk, dD = [a.copy() for a in g.bwd()]
    g.du.fill_(7.0); g.dk.fill_(7.0); g.dD.fill_(7.0)
    # (a call for all three runs one fused kernel on this workload, partial calls the separate kernels: the
    # results agree to rounding, not bitwise)
    tol = 2 * 3e-3
    du1, dk1, dD1 = g.bwd(du=False)
    assert np.all(du1 == 7.0) and wl.rel_l2(dk1, dk) <= tol and wl.rel_l2(dD1, dD) <= tol
    g.du.fill_(7.0); g.dk.fill_(7.0); g.dD.fill_(7.0)
    du2, dk2, dD2 = g.bwd(dk=False, dD=False)
    assert wl.rel_l2(du2, du) <= tol and np.all(dk2 == 7.0) and np.all(dD2 == 7.0)
    g.du.fill_(7.0); g.dk.fill_(7.0); g.dD.fill_(7.0)
    du3, dk3, dD3 = g.bwd(dk=False)                      # du and dD only: dk stays untouched
    assert wl.rel_l2(du3, du) <= tol and np.all(dk3 == 7.0) and wl.rel_l2(dD3, dD) <= tol
    g.du.fill_(7.0); g.dk.fill_(7.0); g.dD.fill_(7.0)
    du4, dk4, dD4 = g.bwd(dD=False)                      # du and dk only
    assert np.array_equal(du4, du) and np.array_equal(dk4, dk) and np.all(dD4 == 7.0)


def test_delta_and_shifted_delta_on_gpu():
    # closed forms straight on the device path: k = e_s shifts u by s with zeros in front
    from gpu_harness import GpuRun
    inp = wl.generate(wl.WORKLOADS["1"], B=2, H=3)
    inp.k[:] = 0.0
    inp.k[0, 0] = 1.0; inp.k[1, 5] = 1.0; inp.k[2, 1023] = 1.0
    inp.D[:] = 0.0
    y = GpuRun(inp).fwd()
    u = inp.u
    np.testing.assert_allclose(y[:, 0], u[:, 0], atol=2e-5)
    np.testing.assert_allclose(y[:, 1, 5:], u[:, 1, :-5], atol=2e-5)
    np.testing.assert_allclose(y[:, 1, :5], 0.0, atol=2e-5)
    np.testing.assert_allclose(y[:, 2, 1023], u[:, 2, 0], atol=2e-5)
    np.testing.assert_allclose(y[:, 2, :1023], 0.0, atol=2e-5)


@pytest.mark.parametrize("N,io", [(1024, wl.F16), (2048, wl.BF16), (16384, wl.F16), (8192, wl.BF16),
                                  (65536, wl.F16), (131072, wl.F16)])
def test_closed_forms_on_the_matrix_core_kernels(N, io):
    """Delta, shifted delta, all-ones kernel and skip term on the device for one wave-autonomous, one cooperative
    and one multi-pass length per half dtype, without the oracle: k = e_s gives y[t] = u[t-s] with zeros in
    front (a circular implementation wraps), k = 1 gives the prefix sum, D adds D u; the backward of a shifted
    delta shifts dy the other way and dk[s'] of it is the lag-s' correlation.  Error per row relative to the
    row's norm, bound 3e-3."""
    from gpu_harness import GpuRun, TOL
    B, H = 3, 5
    inp = wl.generate(_w("3", N=N, dtype=io), B=B, H=H)
    s1, s2 = 7, N - 3
    inp.k[:] = 0.0
    inp.k[0, 0] = 1.0           # delta
    inp.k[1, s1] = 1.0          # short shift
    inp.k[2, s2] = 1.0          # shift by almost the whole length
    c1 = 0.5 / np.sqrt(N)
    inp.k[3, :] = c1            # scaled all-ones kernel: prefix sums of order one
    inp.k[4, 0] = 0.5           # half a delta plus a skip term
    inp.D[:] = 0.0
    inp.D[4] = -1.25
    g = GpuRun(inp)
    y = g.fwd()
    du, dk, dD = g.bwd()
    u, dy = inp.u, inp.dy
    tol = TOL[io]
    want_y = np.zeros_like(u)
    want_y[:, 0] = u[:, 0]
    want_y[:, 1, s1:] = u[:, 1, :N - s1]
    want_y[:, 2, s2:] = u[:, 2, :N - s2]
    want_y[:, 3] = np.cumsum(u[:, 3], axis=-1) * np.float64(np.float32(c1))
    want_y[:, 4] = (0.5 - 1.25) * u[:, 4]
    # head 2 keeps three samples of the shifted row: its error is measured against the norm of the whole shifted
    # row (what the transform carries), every other row against its own norm
    def errs(x, want, src):
        num = np.linalg.norm(x - want, axis=-1)
        den = np.linalg.norm(want, axis=-1)
        den[:, 2] = np.linalg.norm(src[:, 2], axis=-1)
        return num / den
    e = errs(y, want_y, u)
    print(f"[closed forms] N={N} io={wl.DTYPE_NAMES[io]} y per head: " + " ".join(f"{v:.2e}" for v in e.max(axis=0)),
          flush=True)
    assert e.max() <= tol
    assert np.abs(y[:, 1, :s1]).max() <= tol * np.abs(u[:, 1]).max()          # nothing wraps around
    assert np.abs(y[:, 2, :s2]).max() <= tol * np.abs(u[:, 2]).max() * 4
    want_du = np.zeros_like(dy)
    want_du[:, 0] = dy[:, 0]
    want_du[:, 1, :N - s1] = dy[:, 1, s1:]
    want_du[:, 2, :N - s2] = dy[:, 2, s2:]
    want_du[:, 3] = np.cumsum(dy[:, 3, ::-1], axis=-1)[:, ::-1] * np.float64(np.float32(c1))
    want_du[:, 4] = (0.5 - 1.25) * dy[:, 4]
    e = errs(du, want_du, dy)
    print(f"[closed forms] du per head: " + " ".join(f"{v:.2e}" for v in e.max(axis=0)), flush=True)
    assert e.max() <= tol
    # dD and the first taps of dk straight from their definitions (float64 on the host)
    want_dD = np.einsum("bhn,bhn->h", dy, u)
    assert wl.rel_l2(dD, want_dD) <= 1e-5
    for lag in (0, 1, s1):
        want = np.einsum("bhn,bhn->h", dy[:, :, lag:], u[:, :, :N - lag])
        scale = np.sqrt(np.mean(want ** 2))
        assert np.max(np.abs(dk[:, lag] - want)) <= 4 * tol * scale, f"dk lag {lag}"


@pytest.mark.parametrize("key", ["2", "3", "4a", "4b", "5_256", "5_512", "5_2048", "5_4096"])
def test_full_size_sampled(key):
    # BASELINE sizes in the launch configuration the benchmark times, checked on whole heads: the first, the
    # last and seeded ones in between, at least 32 (b,h) rows (32 heads where the batch is a single row)
    from gpu_harness import check_sampled, sample_heads
    w = wl.WORKLOADS[key]
    check_sampled(wl.generate(w), sample_heads(w.H, w.B, seed=w.N + w.wid))


@pytest.mark.parametrize("N,B,H", [(256, 3, 2), (512, 1, 3), (1024, 6, 1), (2048, 3, 2), (4096, 3, 2), (8192, 3, 2),
                                   (16384, 3, 1), (32768, 1, 2)])
def test_fp32_engine_every_length(N, B, H):
    # every radix schedule of the fp32 engine, the last pair half empty or the pairs dealt to several workgroups, and
    # the gradients asked for alone (the fused backward kernel without du, the convolution kernel for du)
    from gpu_harness import GpuRun, check_full
    inp = wl.generate(_w("1", N=N), B=B, H=H)
    check_full(inp, label=f"fp32 N={N}")
    g = GpuRun(inp)
    du, dk, dD = [a.copy() for a in g.bwd()]
    g.dk.fill_(float("nan")), g.dD.fill_(float("nan")), g.du.fill_(float("nan"))
    dk1, dD1 = g.bwd(du=False)[1:]
    assert np.array_equal(dk1, dk) and np.array_equal(dD1, dD)
    assert wl.rel_l2(g.bwd(dk=False, dD=False)[0], du) < 1e-6


@pytest.mark.parametrize("io,B,H", [(wl.F16, 1, 1), (wl.BF16, 3, 2), (wl.BF16, 5, 61)])
def test_single_rows_of_32768_samples(io, B, H):
    # one twisted transform per row: the only row of the call; an odd count with rows outside the bf16 band (each row is
    # scaled by itself, so each meets the tolerance by itself); more rows than compute units, where a workgroup takes
    # several, of two heads, and the last workgroup is short
    import oracle
    from gpu_harness import TOL, GpuRun, _compare, check_full, check_sampled
    inp = wl.generate(wl.Workload(6, B, H, 32768, io, "decay_alpha_squash"))
    if B == 3:
        s = 2.0 ** np.array([-40, 0, 12])[:, None, None]        # powers of two: exact in bf16
        for name in ("u", "dy"):
            x = getattr(inp, name) * s
            st, x = wl.quantize(x.astype(np.float32), io)
            setattr(inp, name, x), setattr(inp, name + "_store", st)
    if B == 3:
        check_full(inp, backward=False, label="single rows")
        du = GpuRun(inp).bwd(dk=False, dD=False)[0]
        want = oracle.longconv_bwd(inp.dy, inp.u, inp.k.astype(np.float64), inp.D.astype(np.float64))[0]
        _compare({"du": du}, {"du": want}, TOL[io], "single rows, du alone")
    elif H <= 2:
        check_full(inp, label="single rows")
    else:
        check_sampled(inp, [0, 31, H - 1], label="single rows")


@pytest.mark.parametrize("io,B,H", [(wl.F16, 3, 2), (wl.BF16, 2, 65)])
def test_rows_of_65536_samples_in_two_chunks(io, B, H):
    # an odd batch; as many chunks as compute units and a few more (a workgroup takes two of different rows)
    from gpu_harness import check_full, check_sampled
    inp = wl.generate(wl.Workload(6, B, H, 65536, io, "decay4"))
    if H <= 2:
        check_full(inp, label="rows in two chunks")
    else:
        check_sampled(inp, [0, 33, H - 1], label="rows in two chunks")


@pytest.mark.parametrize("io", [wl.F16, wl.BF16])
@pytest.mark.parametrize("B,H", [(1, 3), (2, 5), (3, 2), (5, 64), (9, 3), (17, 2), (16, 129), (33, 257)])
def test_rows_of_1024_samples_one_wave_each(B, H, io):
    # one, two and four waves in the backward kernel; one share of the rows and several, even and ragged, more rows than
    # waves on the device; dk and dD by themselves equal those of the call with du
    from gpu_harness import GpuRun, check_full, check_sampled
    inp = wl.generate(wl.Workload(6, B, H, 1024, io, "squash_pool"))
    if B * H <= 64:
        check_full(inp, label="one wave a row")
    else:
        check_sampled(inp, [0, H // 2, H - 1], label="one wave a row")
    g = GpuRun(inp)
    dk, dD = g.bwd()[1:]
    g.dk.fill_(float("nan")), g.dD.fill_(float("nan"))
    dk1, dD1 = g.bwd(du=False)[1:]
    assert np.array_equal(dk, dk1) and np.array_equal(dD, dD1)
