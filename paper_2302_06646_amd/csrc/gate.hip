// Output gate of the long convolution (the H3-style layer of Section 4.1 multiplies the outputs of two sequence
// operators element by element): y = g * z, z the ungated output of Eq. 1, and the two products of its backward
// pass, dz = dy * g and dg = dy * z.  Plain streaming kernel, bound by memory: eight elements per lane, fp32
// product of the two I/O-dtype values, rounded once.  Where the convolution's own kernel applies the gate before
// its store (see wconv_kernel) this kernel is not launched.
#include <type_traits>

#include "engines.hpp"
#include "mfma_util.hpp"

namespace lc {
namespace {

template <class IO>
__device__ __forceinline__ void mul8(const uint4& a, const uint4& b, uint4& o)
{
    const uint32_t wa[4] = {a.x, a.y, a.z, a.w}, wb[4] = {b.x, b.y, b.z, b.w};
    uint32_t wo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (mu::IsBf<IO>::v) {
            const float a0 = __uint_as_float(wa[i] << 16), a1 = __uint_as_float(wa[i] & 0xffff0000u);
            const float b0 = __uint_as_float(wb[i] << 16), b1 = __uint_as_float(wb[i] & 0xffff0000u);
            wo[i] = mu::pack_bf2(a0 * b0, a1 * b1);
        } else {
            union { uint32_t u; mu::h2 h; } x, y;
            x.u = wa[i]; y.u = wb[i];
            wo[i] = mu::pack_h2((float)x.h[0] * (float)y.h[0], (float)x.h[1] * (float)y.h[1]);
        }
    }
    o = make_uint4(wo[0], wo[1], wo[2], wo[3]);
}

template <class IO>
__global__ void __launch_bounds__(256)
ew_mul_kernel(const typename IO::T* __restrict__ a, const typename IO::T* __restrict__ b, typename IO::T* out, size_t n8)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (size_t)gridDim.x * 256) {
        uint4 o;
        mul8<IO>(reinterpret_cast<const uint4*>(a)[i], reinterpret_cast<const uint4*>(b)[i], o);
        reinterpret_cast<uint4*>(out)[i] = o;
    }
}

__global__ void __launch_bounds__(256)
ew_mul_f32_kernel(const float* __restrict__ a, const float* __restrict__ b, float* out, size_t n4)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
        const float4 x = reinterpret_cast<const float4*>(a)[i], y = reinterpret_cast<const float4*>(b)[i];
        reinterpret_cast<float4*>(out)[i] = make_float4(x.x * y.x, x.y * y.y, x.z * y.z, x.w * y.w);
    }
}

// 16 bytes of dy, g and u: s + sum dy g u in fp32 (dy g unrounded), and, if wanted, dz = dy g in the I/O dtype
template <class IO>
__device__ __forceinline__ float gate_piece(const uint4& y, const uint4& g, const uint4& u, uint4& z, float s)
{
    const uint32_t wy[4] = {y.x, y.y, y.z, y.w}, wg[4] = {g.x, g.y, g.z, g.w}, wu[4] = {u.x, u.y, u.z, u.w};
    uint32_t wz[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (std::is_same<IO, IoF32>::value) {
            const float p = __uint_as_float(wy[i]) * __uint_as_float(wg[i]);
            wz[i] = __float_as_uint(p);
            s = __builtin_fmaf(p, __uint_as_float(wu[i]), s);
        } else {
            float p[2], v[2];
            if (mu::IsBf<IO>::v) {
                p[0] = __uint_as_float(wy[i] << 16) * __uint_as_float(wg[i] << 16);
                p[1] = __uint_as_float(wy[i] & 0xffff0000u) * __uint_as_float(wg[i] & 0xffff0000u);
                v[0] = __uint_as_float(wu[i] << 16);
                v[1] = __uint_as_float(wu[i] & 0xffff0000u);
                wz[i] = mu::pack_bf2(p[0], p[1]);
            } else {
                union { uint32_t u; mu::h2 h; } a, b, c;
                a.u = wy[i]; b.u = wg[i]; c.u = wu[i];
                p[0] = (float)a.h[0] * (float)b.h[0];
                p[1] = (float)a.h[1] * (float)b.h[1];
                v[0] = (float)c.h[0];
                v[1] = (float)c.h[1];
                wz[i] = mu::pack_h2(p[0], p[1]);
            }
            s = __builtin_fmaf(p[0], v[0], s);
            s = __builtin_fmaf(p[1], v[1], s);
        }
    }
    z = make_uint4(wz[0], wz[1], wz[2], wz[3]);
    return s;
}

// dz (may be null) and the sums of dy g u over a share of a head: workgroup (share, h) takes `per` consecutive 16-byte pieces of
// the head's B rows.  Bound by memory: four streams, where dz and a dot product by one workgroup per head read dy and g twice,
// sample by sample.  Gated steps, before and now: B=16, H=7, N=131072 bf16 2921 -> 470 us, B=64, H=32, N=16384 2035 -> 280, B=8,
// H=256, N=16384 fp16 466 -> 275, B=4, H=50, N=8192 83 -> 47, B=1, H=1024, N=8192 136 -> 122.  Error of dD against 64 bits
// 1.2e-7 to 1.8e-7 there (was 1.2e-7 to 1.3e-6).  u_words: u is 16-byte aligned (it need not be where only dD is asked for).
template <class IO>
__global__ void __launch_bounds__(256)
gate_bwd_kernel(const uint4* __restrict__ dy, const uint4* __restrict__ g, const typename IO::T* __restrict__ u, uint4* __restrict__ dz,
                float* __restrict__ part, int64_t H, int lg_row, int64_t pieces, int64_t per, int u_words)
{
    constexpr int E = 16 / sizeof(typename IO::T);
    __shared__ float red[4];
    const int64_t h = blockIdx.y, i0 = (int64_t)blockIdx.x * per, i1 = i0 + per < pieces ? i0 + per : pieces;
    float s = 0.f;
#pragma unroll 2
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
        const size_t at = ((size_t)((i >> lg_row) * H + h) << lg_row) + (size_t)(i & ((int64_t(1) << lg_row) - 1));
        uint4 v, z;
        if (u_words) {
            v = reinterpret_cast<const uint4*>(u)[at];
        } else {
            union { uint4 q; typename IO::T e[E]; } x;
#pragma unroll
            for (int e = 0; e < E; ++e) x.e[e] = u[at * E + e];
            v = x.q;
        }
        s = gate_piece<IO>(dy[at], g[at], v, z, s);
        if (dz) dz[at] = z;
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[(size_t)h * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// dD[h] = sum of the head's shares, in a fixed order: one wave per head
__global__ void __launch_bounds__(64)
gate_sum_kernel(const float* __restrict__ part, float* __restrict__ dD, int shares)
{
    const float* p = part + (size_t)blockIdx.x * shares;
    float s = 0.f;
    for (int i = threadIdx.x; i < shares; i += 64) s += p[i];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if (threadIdx.x == 0) dD[blockIdx.x] = s;
}

template <class IO>
hipError_t gate_bwd_go(const void* dy, const void* g, const void* u, void* dz, float* dD, float* part, const Problem& pr, hipStream_t st)
{
    constexpr int E = 16 / sizeof(typename IO::T);
    int lg_row = 0;
    while ((int64_t(E) << lg_row) < pr.N) ++lg_row;
    const int64_t pieces = pr.B << lg_row;
    // shares of a head: eight workgroups per compute unit (what it holds), of at least four pieces a thread
    int64_t n = (8 * (int64_t)compute_units() + pr.H - 1) / pr.H;
    if (n > pieces / 1024) n = pieces / 1024;
    if (n > GATE_SHARES) n = GATE_SHARES;
    if (n < 1) n = 1;
    const int64_t per = (pieces + n - 1) / n;
    n = (pieces + per - 1) / per;
    hipLaunchKernelGGL((gate_bwd_kernel<IO>), dim3((unsigned)n, (unsigned)pr.H), dim3(256), 0, st, (const uint4*)dy, (const uint4*)g,
                       (const typename IO::T*)u, (uint4*)dz, n > 1 ? part : dD, pr.H, lg_row, pieces, per,
                       (reinterpret_cast<uintptr_t>(u) & 15u) == 0 ? 1 : 0);
    if (n > 1) hipLaunchKernelGGL(gate_sum_kernel, dim3((unsigned)pr.H), dim3(64), 0, st, part, dD, (int)n);
    return hipGetLastError();
}

}  // namespace

hipError_t gate_bwd(const void* dy, const void* g, const void* u, void* dz, float* dD, float* part, const Problem& pr, hipStream_t st)
{
    if (pr.io == LONGCONV_F32) return gate_bwd_go<IoF32>(dy, g, u, dz, dD, part, pr, st);
    if (pr.io == LONGCONV_F16) return gate_bwd_go<IoF16>(dy, g, u, dz, dD, part, pr, st);
    return gate_bwd_go<IoBF16>(dy, g, u, dz, dD, part, pr, st);
}

// out = a * b, element by element, n elements of the I/O dtype (n a multiple of 8; out may be a or b)
hipError_t ew_mul(const void* a, const void* b, void* out, size_t n, int io, hipStream_t st)
{
    const size_t per = io == LONGCONV_F32 ? 4 : 8, nv = n / per;
    const size_t want = (nv + 255) / 256, cap = (size_t)compute_units() * 16;
    const unsigned grid = (unsigned)(want < cap ? (want ? want : 1) : cap);
    if (io == LONGCONV_F32)
        hipLaunchKernelGGL(ew_mul_f32_kernel, dim3(grid), dim3(256), 0, st, (const float*)a, (const float*)b, (float*)out, nv);
    else if (io == LONGCONV_F16)
        hipLaunchKernelGGL((ew_mul_kernel<IoF16>), dim3(grid), dim3(256), 0, st, (const __half*)a, (const __half*)b,
                           (__half*)out, nv);
    else if (io == LONGCONV_BF16)
        hipLaunchKernelGGL((ew_mul_kernel<IoBF16>), dim3(grid), dim3(256), 0, st, (const uint16_t*)a, (const uint16_t*)b,
                           (uint16_t*)out, nv);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace lc
