// 16 x 16 tiles of complex fp16 numbers in planar form, for kernels that chain two 16-point blocks in registers.
//
// A matrix instruction leaves its result as (X = lane % 16, Y = 4 (lane / 16) + register) and takes an operand in the same
// form with Y the contracted index; which of its two operands the data is decides whether X stays (data second) or the new index
// takes the lanes and X the registers (data first).  A lane's operand is four real parts, then four imaginary parts (the
// matrices' K index runs in that order), so LDS holds planes of 16-bit numbers, written as runs of four and read either the same
// way or transposed.  LDS serves an 8-byte access 16 lanes at a time over 32 banks; where these lanes sit in 16 different rows
// of 16 numbers they all want the same quarter of their rows, so the users of this file store a row's quarters XORed with a hash
// of the row.
#pragma once
#include "common.hpp"

namespace lc {
namespace planar {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

struct Cx {
    h8 re, im;      // complex in: operands giving the real and imaginary part of the result
};
struct Rl {
    h4 re, im;      // real in
};
union H8P {
    h8 v;
    h4 p[2];        // planes
    uint2 u[2];
    uint4 w;
};

__device__ __forceinline__ f4 mm(const h8& a, const h8& b)
{
    const f4 z = {0.f, 0.f, 0.f, 0.f};
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, z, 0, 0, 0);
}
__device__ __forceinline__ f4 mm(const h4& a, const h4& b)
{
    const f4 z = {0.f, 0.f, 0.f, 0.f};
    return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, z, 0, 0, 0);
}
// four 16-bit numbers a lane: lane i of 16 gives the address of numbers 4 (i % 4) .. + 3 of row i / 4 and receives column i of
// the four rows (all lanes active)
__device__ __forceinline__ h4 tr_read(const _Float16* s)
{
    typedef __fp16 t4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) t4 lds_t4;
    union { t4 t; h4 h; } cv;
    cv.t = __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_t4*)(s));
    return cv.h;
}
__device__ __forceinline__ h4 rd4(const _Float16* s) { return *reinterpret_cast<const h4*>(s); }
__device__ __forceinline__ void wr4(_Float16* s, const h4& v) { *reinterpret_cast<h4*>(s) = v; }
__device__ __forceinline__ h4 cvt4(const f4& v) { return __builtin_convertvector(v, h4); }
__device__ __forceinline__ H8P planes(const f4& re, const f4& im)
{
    H8P x;
    x.p[0] = cvt4(re);
    x.p[1] = cvt4(im);
    return x;
}
// (re + i im) * w, or * conj(w), four numbers, fp32
template <bool CONJ>
__device__ __forceinline__ void cmul4(f4& re, f4& im, const f4& wr, const f4& wi)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float2 v = make_float2(re[r], im[r]), w = make_float2(wr[r], wi[r]);
        const float2 p = CONJ ? cmulc(v, w) : cmul(v, w);
        re[r] = p.x;
        im[r] = p.y;
    }
}
// matrix operands: lane = (o = lane % 16 the result's index, g), entries in order of the input's index i = 4g .. 4g+3
template <class F>
__device__ __forceinline__ Cx make_cx(F&& entry, int lane)
{
    Cx M;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float2 w = entry(lane & 15, 4 * (lane >> 4) + e);
        M.re[e] = (_Float16)w.x;
        M.re[4 + e] = (_Float16)(-w.y);
        M.im[e] = (_Float16)w.y;
        M.im[4 + e] = (_Float16)w.x;
    }
    return M;
}
template <class F>
__device__ __forceinline__ Rl make_rl(F&& entry, int lane)
{
    Rl M;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float2 w = entry(lane & 15, 4 * (lane >> 4) + e);
        M.re[e] = (_Float16)w.x;
        M.im[e] = (_Float16)w.y;
    }
    return M;
}
__device__ __forceinline__ float2 scaled(float2 w, float s) { return make_float2(w.x * s, w.y * s); }
__device__ __forceinline__ float2 conj2(float2 w) { return make_float2(w.x, -w.y); }

}  // namespace planar
}  // namespace lc
