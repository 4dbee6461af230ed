// Kernel regularisers in front of the long convolution (Algorithm 1 lines 1-3; Section 3.1 "Regularizing the
// Kernel"): Kbar = Squash(Smooth(dropout(K))) and the chain rule back through the three steps.
//
//   K1 = M * K                                   dropout, the mask M (0 or 1/(1-q)) is the caller's
//   K2[n] = (2p+1)^-1 sum_{|d| <= p} K1[n+d]     Smooth: centred window, zeros outside 0..N-1, always / (2p+1)
//   Kbar = sign(K2) max(|K2| - lambda, 0)        Squash
//   dK = M * Smooth^T( dKbar * [|K2| > lambda] ) (Smooth with this boundary rule is its own transpose)
//
// Plain streaming kernels, bound by one round trip to memory and the launch: a workgroup is one wave (no barriers) with 256
// consecutive entries of one head, and asks for everything it needs before it uses any of it, four entries of each tensor per lane
// and their halo; the masked kernel goes through LDS (2p entries per side for the backward chain, which needs K2 on a halo of p).
// H = 768, N = 1024, p = 1, against a workgroup of 256 threads with an entry each: forward 5.3 -> 4.4 us, backward, which asked for
// the gradient behind the gate and for the mask a second time, 6.9 -> 5.1; with two entries per lane the two take 1.5 us more.
#include "engines.hpp"

namespace lc {
namespace {

constexpr int KT = 64, KV = 4, KE = KT * KV;      // lanes, entries of a lane (64 apart), entries of a workgroup
constexpr int KREG_P_MAX = 32;                    // widest half window

template <bool BWD>
__global__ void __launch_bounds__(KT)
kreg_kernel(const float* __restrict__ k, const float* __restrict__ mask, const float* __restrict__ dkbar,
            float* __restrict__ out, int64_t N, int p, float lam)
{
    constexpr int KH = (BWD ? 4 : 2) * KREG_P_MAX / KT;      // entries of a lane in the halos, at the widest window
    __shared__ float s1[KE + 4 * KREG_P_MAX];      // K1 on [n0 - halo, n0 + KE + halo)
    __shared__ float s2[KE + 2 * KREG_P_MAX];      // backward: gated gradient on [n0 - p, n0 + KE + p)
    const int64_t h = blockIdx.y, n0 = (int64_t)blockIdx.x * KE;
    const int t = threadIdx.x, halo = BWD ? 2 * p : p;
    const float* kr = k + h * N;
    const float* mr = mask ? mask + h * N : nullptr;
    const float inv = 1.0f / (float)(2 * p + 1);
    // entry e of a window's two halos of `w` entries -> its place relative to the window of KE entries behind the left one
    const auto halo_at = [&](int e, int w) { return e < w ? e - w : KE + e - w; };
    const auto get = [&](const float* row, int64_t n) { return n >= 0 && n < N ? row[n] : 0.f; };
    float kv[KV], mv[KV], kh[KH], mh[KH], gv[KV], gh = 0.f;
#pragma unroll
    for (int j = 0; j < KV; ++j) {
        kv[j] = get(kr, n0 + t + KT * j);
        mv[j] = mr ? get(mr, n0 + t + KT * j) : 1.f;
        if (BWD) gv[j] = get(dkbar + h * N, n0 + t + KT * j);
    }
#pragma unroll
    for (int j = 0; j < KH; ++j) {
        const int e = t + KT * j;
        const int64_t n = e < 2 * halo ? n0 + halo_at(e, halo) : -1;
        kh[j] = get(kr, n);
        mh[j] = mr ? get(mr, n) : 1.f;
    }
    if (BWD && t < 2 * p) gh = get(dkbar + h * N, n0 + halo_at(t, p));
#pragma unroll
    for (int j = 0; j < KV; ++j) s1[halo + t + KT * j] = kv[j] * mv[j];
#pragma unroll
    for (int j = 0; j < KH; ++j)
        if (t + KT * j < 2 * halo) s1[halo + halo_at(t + KT * j, halo)] = kh[j] * mh[j];
    __syncthreads();
    // sums of s[i .. i + 2p] at the lane's entries, i = at + t + 64 j, side by side (one after the other they wait for LDS alone)
    const auto windows = [&](const float* s, int at, float (&a)[KV]) {
#pragma unroll
        for (int j = 0; j < KV; ++j) a[j] = 0.f;
        for (int d = 0; d <= 2 * p; ++d)
#pragma unroll
            for (int j = 0; j < KV; ++j) a[j] += s[at + t + KT * j + d];
    };
    float a[KV];
    if (!BWD) {
        windows(s1, 0, a);
#pragma unroll
        for (int j = 0; j < KV; ++j) {
            const int64_t n = n0 + t + KT * j;
            const float k2 = a[j] * inv, m = fabsf(k2) - lam;
            if (n < N) out[h * N + n] = m > 0.f ? copysignf(m, k2) : 0.f;
        }
        return;
    }
    // (a gate that is closed drops the gradient, whatever it is; beyond the row there is none)
    windows(s1, p, a);
    if (t < 2 * p) {
        const int i = halo_at(t, p);
        const int64_t q = n0 + i;
        float b = 0.f;
        for (int d = 0; d <= 2 * p; ++d) b += s1[p + i + d];
        s2[p + i] = q >= 0 && q < N && fabsf(b * inv) > lam ? gh : 0.f;
    }
#pragma unroll
    for (int j = 0; j < KV; ++j) s2[p + t + KT * j] = n0 + t + KT * j < N && fabsf(a[j] * inv) > lam ? gv[j] : 0.f;
    __syncthreads();
    windows(s2, 0, a);
#pragma unroll
    for (int j = 0; j < KV; ++j) {
        const int64_t n = n0 + t + KT * j;
        if (n < N) out[h * N + n] = mr ? a[j] * inv * mv[j] : a[j] * inv;
    }
}

}  // namespace

hipError_t kreg_fwd(const float* k, const float* mask, float* kbar, int64_t H, int64_t N, int p, float lam,
                    hipStream_t st)
{
    if (p < 0 || p > KREG_P_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((N + KE - 1) / KE), (unsigned)H);
    hipLaunchKernelGGL(kreg_kernel<false>, grid, dim3(KT), 0, st, k, mask, (const float*)nullptr, kbar, N, p, lam);
    return hipGetLastError();
}

hipError_t kreg_bwd(const float* k, const float* mask, const float* dkbar, float* dk, int64_t H, int64_t N, int p,
                    float lam, hipStream_t st)
{
    if (p < 0 || p > KREG_P_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((N + KE - 1) / KE), (unsigned)H);
    hipLaunchKernelGGL(kreg_kernel<true>, grid, dim3(KT), 0, st, k, mask, dkbar, dk, N, p, lam);
    return hipGetLastError();
}

}  // namespace lc
