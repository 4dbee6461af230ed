// What the kernels of engine_long.hip (rows of 8192 and 16384 samples) and engine_chunk.hip (chunks of 16384 points of longer
// rows) share: geometry, a wave's constants, the three phases on tiles, and the places of numbers in LDS.
#pragma once
#include "engines.hpp"
#include "mfma_util.hpp"
#include "planar.hpp"

namespace lc {
namespace longrows {
using namespace planar;
using mu::IsBf;

template <int LG, int TPW_ = 8, int NAL_ = 0>
struct LR {
    static constexpr int lg = LG, TPW = TPW_;            // TPW: tiles of a wave
    static constexpr int NAL = NAL_;                     // of them, last ones whose matrices over d_a wait in LDS
    static constexpr int N = 1 << LG, TC = N / 256, TE = TC / 16, te = LG - 12;
    static constexpr int NW = TC / TPW, NT = 64 * NW, KB = 16 / NW;       // waves, threads, k_b's of a wave in phase 2
    static constexpr int SHIFT = 7;                       // forward chain: 2^-7, inverse: 2^-6 (see RC::SHIFT in engine_rows.hip)
    static constexpr int PC = N / 8 / NT, STEP = 8 * NT;  // 16-byte pieces of a row per thread, numbers between them
    static constexpr int EX = TC * 512, RAW = N;          // numbers of the exchange buffer and of a row on its way
    // quarter q of row k_b of tile t: rows permuted among four by d_c % 4, so that four d_c of one k_b meet four bank groups,
    // quarters by k_b / 4 and d_c / 4
    static __device__ __forceinline__ int at(int t, int kb, int q)
    {
        const int dc = t >> te;
        return t * 512 + (kb ^ (dc & 3)) * 16 + 4 * ((q ^ (kb >> 2) ^ (dc >> 2)) & 3);
    }
    // piece p (the eight samples of wave p's tiles) of block m = 16 d_a + d_b of a row: eight lanes' pieces fill the banks
    static __device__ __forceinline__ int piece(int m, int p) { return m * TC + 8 * (p ^ (TC == 64 ? m & 7 : (m >> 1) & 3)); }

    // constants, in units of 16 bytes per lane: per tile the matrices over d_a (forward; inverse, real part), w_256^(lane (4g+r)),
    // per k_b those over d_c (forward, inverse: two units each); then what goes to LDS: over d_b for each d_e and over d_e for
    // each unit of four results (forward and inverse); last, for the backward pass, the inverse matrix over k_a without the
    // tile's factor, and these factors, planar
    static constexpr int U_A = 0, U_AI = TC, U_TW = 2 * TC, U_C = U_TW + 1, U_CI = U_C + 32, U_LDS = U_CI + 32;
    static constexpr int U_B = 0, U_BI = 2 * TE, U_E = 4 * TE, U_EI = 6 * TE, N_LDS = 8 * TE;       // from U_LDS
    static constexpr int U_AP = U_LDS + N_LDS, U_S = U_AP + 1, UNITS = U_S + TC / 16;
    // factors: the tiles' factors are there, too
    static constexpr size_t lds(bool factors) { return sizeof(_Float16) * (EX + RAW) + 1024 * (N_LDS + NAL * NW) + (factors ? 64 * TC : 0); }
};

// the constants of both lengths, one behind the other
constexpr int LONG_TAB = LR<13>::UNITS + LR<14>::UNITS;
template <int LG>
__host__ __device__ constexpr int tab_offset() { return LG == 13 ? 0 : LR<13>::UNITS; }

// a wave's own constants.  TILE_AI: the inverse matrices over k_a carry the tiles' factors (the backward pass has no registers
// for these); INV: there is an inverse
template <class L_, bool INV, bool TILE_AI, int NAL = 0>
struct LK {
    using L = L_;
    Rl A[L::TPW - NAL];
    uint4* al;             // this lane's place of the others
    h8 AI[TILE_AI ? L::TPW : 1];
    Cx C[L::KB], CI[INV ? L::KB : 1];
    h4 cr, ci;             // w_256^(lane (4g + r)): k_a d_b either way round
    __device__ __forceinline__ Rl a(int kt) const
    {
        if (kt < L::TPW - NAL) return A[kt < L::TPW - NAL ? kt : 0];
        H8P x;
        x.w = al[(kt - (L::TPW - NAL)) * 64];
        return Rl{x.p[0], x.p[1]};
    }
    __device__ __forceinline__ void load(const uint4* __restrict__ tab, int wave, int lane, uint4* lds = nullptr)
    {
        al = lds + wave * NAL * 64 + lane;
        const uint4* p = tab + (size_t)tab_offset<L::lg>() * 64 + lane;
        H8P x;
        const auto unit = [&](int u) { x.w = p[(size_t)u * 64]; return x; };
#pragma unroll
        for (int k = 0; k < L::TPW; ++k) {
            unit(L::U_A + L::TPW * wave + k);
            if (k < L::TPW - NAL) A[k < L::TPW - NAL ? k : 0] = Rl{x.p[0], x.p[1]};
            else al[(k - (L::TPW - NAL)) * 64] = x.w;
            if (INV && TILE_AI) AI[TILE_AI ? k : 0] = unit(L::U_AI + L::TPW * wave + k).v;
        }
        if (INV && !TILE_AI) AI[0] = unit(L::U_AP).v;
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            const int kb = wave * L::KB + j;
            C[j].re = unit(L::U_C + 2 * kb).v;
            C[j].im = unit(L::U_C + 2 * kb + 1).v;
            if (INV) {
                CI[INV ? j : 0].re = unit(L::U_CI + 2 * kb).v;
                CI[INV ? j : 0].im = unit(L::U_CI + 2 * kb + 1).v;
            }
        }
        unit(L::U_TW);
        cr = x.p[0];
        ci = x.p[1];
    }
};
// the shared matrices (and the tiles' factors) to LDS
template <class L>
__device__ __forceinline__ void load_shared(uint4* sm, const uint4* __restrict__ tab, int tid, bool s)
{
    const uint4* p = tab + (size_t)(tab_offset<L::lg>() + L::U_LDS) * 64;
    for (int i = tid; i < L::N_LDS * 64; i += L::NT) sm[i] = p[i];
    if (s)
        for (int i = tid; i < L::TC * 4; i += L::NT) sm[L::N_LDS * 64 + i] = p[(L::U_S - L::U_LDS) * 64 + i];
}
__device__ __forceinline__ Cx shared_mat(const uint4* m, int u)       // m: this lane's column
{
    Cx M;
    H8P x;
    x.w = m[u * 64];
    M.re = x.v;
    x.w = m[(u + 1) * 64];
    M.im = x.v;
    return M;
}
// (yr + i yi) * (wr + i wi), or * conj, four numbers in packed fp16
template <bool CONJ>
__device__ __forceinline__ H8P cmul_planes(const f4& yr, const f4& yi, const h4& wr, const h4& wi)
{
    const h4 a = cvt4(yr), b = cvt4(yi);
    H8P x;
    x.p[0] = CONJ ? __builtin_elementwise_fma(b, wi, a * wr) : __builtin_elementwise_fma(-b, wi, a * wr);
    x.p[1] = CONJ ? __builtin_elementwise_fma(-a, wi, b * wr) : __builtin_elementwise_fma(a, wi, b * wr);
    return x;
}

// the same with wr + i wi in either precision, in fp32 and rounded once: four instructions more.  It stands where it takes the
// errors of single rows below those of the 2N-point transform of a pair that they are measured against (white rows, B = 1, fp16:
// y 6.9e-4 and dk 9.5e-4 at N = 8192, 7.2e-4 and 9.6e-4 at 16384): in the spectrum, in dk's inverse transform, and at N = 8192 in
// the product of the convolution and in dy's phase 1.  Everywhere it would cost the convolution 12% and the backward pass 15%.
template <bool CONJ, class W>
__device__ __forceinline__ H8P cmul_once(const f4& yr, const f4& yi, const W& wr, const W& wi)
{
    H8P x;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float c = (float)wr[r], d = CONJ ? -(float)wi[r] : (float)wi[r];
        x.p[0][r] = (_Float16)__builtin_fmaf(-yi[r], d, yr[r] * c);
        x.p[1][r] = (_Float16)__builtin_fmaf(yr[r], d, yi[r] * c);
    }
    return x;
}

typedef uint32_t u4w __attribute__((ext_vector_type(4)));
// operands (lane d_b, d_a = 4g ..) of a pair of tiles from its raw words; e: the row's exponent (bf16)
template <class IO>
__device__ __forceinline__ void pair_ops(const uint32_t (&w)[4], int e, h4 (&op)[2])
{
    union { uint32_t u[2]; h4 v; } a, b;
    if constexpr (IsBf<IO>::v) {
        float lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            lo[r] = ldexpf(__uint_as_float(w[r] << 16), -e);
            hi[r] = ldexpf(__uint_as_float(w[r] & 0xffff0000u), -e);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a.u[i] = mu::pack_h2(lo[2 * i], lo[2 * i + 1]);
            b.u[i] = mu::pack_h2(hi[2 * i], hi[2 * i + 1]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a.u[i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x05040100u);
            b.u[i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x07060302u);
        }
    }
    op[0] = a.v;
    op[1] = b.v;
}
template <class IO>
__device__ __forceinline__ uint32_t pack_io(float a, float b) { return IsBf<IO>::v ? mu::pack_bf2(a, b) : mu::pack_h2(a, b); }
template <class IO>
__device__ __forceinline__ float io_half(uint32_t w, int i)
{
    if (IsBf<IO>::v) return __uint_as_float(i ? w & 0xffff0000u : w << 16);
    union { uint32_t u; h4 v; } c;
    c.u = w;
    return (float)c.v[i];
}

// what rounding (re, im) to x left
__device__ __forceinline__ H8P left_over(const f4& re, const f4& im, const H8P& x)
{
    return planes(re - __builtin_convertvector(x.p[0], f4), im - __builtin_convertvector(x.p[1], f4));
}

// phase 1 of the wave's tile kt: dst = this lane's place (row k_b = c, quarter g)
template <class L, bool ONCE, class KT>
__device__ __forceinline__ void phase1_tile(const h4& op, const KT& K, int kt, const uint4* mats, _Float16* dst)
{
    const Rl A = K.a(kt);
    const f4 yr = mm(op, A.re), yi = mm(op, A.im);
    const H8P x = ONCE ? cmul_once<false>(yr, yi, K.cr, K.ci) : cmul_planes<false>(yr, yi, K.cr, K.ci);      // lane k_a, d_b = 4g ..
    const Cx M = shared_mat(mats, L::U_B + 2 * (kt % L::TE));
    const H8P z = planes(mm(x.v, M.re), mm(x.v, M.im));                                        // lane k_b, k_a = 4g ..
    wr4(dst, z.p[0]);
    wr4(dst + 256, z.p[1]);
}
// phase 3: src transposed (lane k_a, k_b = 4g ..); samples (lane d_b, d_a = 4g ..).  s: the tile's factors for k_a = 4g .., unless
// they are in the matrix
template <class L, bool TILE_AI, bool ONCE, class KT>
__device__ __forceinline__ f4 phase3_tile(const _Float16* src, const KT& K, int kt, const uint4* mats, const uint4* s)
{
    H8P x;
    x.p[0] = tr_read(src);
    x.p[1] = tr_read(src + 256);
    const Cx M = shared_mat(mats, L::U_BI + 2 * (kt % L::TE));
    const f4 yr = mm(x.v, M.re), yi = mm(x.v, M.im);                                           // lane d_b, k_a = 4g ..
    H8P m;
    if constexpr (ONCE) {
        f4 wr, wi;
        H8P f;
        if (!TILE_AI) f.w = *s;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float2 c = make_float2((float)K.cr[r], (float)K.ci[r]);
            const float2 w = TILE_AI ? c : cmul(c, make_float2((float)f.p[0][r], (float)f.p[1][r]));
            wr[r] = w.x;
            wi[r] = w.y;
        }
        m = cmul_once<true>(yr, yi, wr, wi);
    } else {
        h4 wr = K.cr, wi = K.ci;
        if (!TILE_AI) {
            H8P f;
            f.w = *s;
            wr = __builtin_elementwise_fma(-f.p[1], K.ci, f.p[0] * K.cr);
            wi = __builtin_elementwise_fma(f.p[0], K.ci, f.p[1] * K.cr);
        }
        m = cmul_planes<true>(yr, yi, wr, wi);
    }
    return mm(K.AI[TILE_AI ? kt : 0], m.v);
}
// forward half of phase 2 for the wave's k_b number j: units m of four results, register q = (r, k_e): lane k_a, k_c = 4g + r,
// r = m 4/TE + q / TE; use(m, re, im) takes them one after the other.  src: transposed, tile (d_c = 4g + c / 4, d_e = 0)
template <class L, class KT, class F>
__device__ __forceinline__ void phase2_fwd(const _Float16* src, const KT& K, int j, const uint4* mats, F&& use)
{
    constexpr int TE = L::TE;
    f4 zr[TE], zi[TE];
#pragma unroll
    for (int de = 0; de < TE; ++de) {
        H8P x;
        x.p[0] = tr_read(src + de * 512);
        x.p[1] = tr_read(src + de * 512 + 256);
        zr[de] = mm(K.C[j].re, x.v);
        zi[de] = mm(K.C[j].im, x.v);
    }
    H8P x[TE];
#pragma unroll
    for (int m = 0; m < TE; ++m) {
        f4 a, b;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = zr[q % TE][m * (4 / TE) + q / TE];
            b[q] = zi[q % TE][m * (4 / TE) + q / TE];
        }
        x[m] = planes(a, b);
    }
#pragma unroll
    for (int m = 0; m < TE; ++m) {
        const Cx M = shared_mat(mats, L::U_E + 2 * m);
        use(m, mm(M.re, x[m].v), mm(M.im, x[m].v));
    }
}
// inverse half; v: the units' operands; dst: row (d_c = c, d_e = 0), quarter g.  SPLIT: operands are v + rest, and so are those of
// the second step, the rests of the roundings to fp16 (dk, once per workgroup: its accumulator is fp32)
template <class L, bool SPLIT, class KT>
__device__ __forceinline__ void phase2_inv(_Float16* dst, const KT& K, int j, const uint4* mats, const H8P (&v)[L::TE],
                                           const H8P (&rest)[L::TE])
{
    constexpr int TE = L::TE;
    f4 zr[TE], zi[TE];
#pragma unroll
    for (int m = 0; m < TE; ++m) {
        const Cx M = shared_mat(mats, L::U_EI + 2 * m);
        f4 a = mm(M.re, v[m].v), b = mm(M.im, v[m].v);
        if constexpr (SPLIT) {
            a += mm(M.re, rest[m].v);
            b += mm(M.im, rest[m].v);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            zr[q % TE][m * (4 / TE) + q / TE] = a[q];
            zi[q % TE][m * (4 / TE) + q / TE] = b[q];
        }
    }
#pragma unroll
    for (int de = 0; de < TE; ++de) {
        const H8P m = planes(zr[de], zi[de]);
        f4 a = mm(m.v, K.CI[j].re), b = mm(m.v, K.CI[j].im);
        if constexpr (SPLIT) {
            const H8P l = left_over(zr[de], zi[de], m);
            a += mm(l.v, K.CI[j].re);
            b += mm(l.v, K.CI[j].im);
        }
        const H8P x = planes(a, b);                                          // lane d_c, k_a = 4g ..
        wr4(dst + de * 512, x.p[0]);
        wr4(dst + de * 512 + 256, x.p[1]);
    }
}

// places of a lane in the exchange buffer and in a row
template <class L>
struct Places {
    static constexpr int ND = L::TPW / L::TE;        // values of d_c among the wave's tiles
    int own[ND], own_tr[ND];                    // tile t0 + TE i: row k_b = c, quarter g; transposed (lane k_a, k_b = 4g ..)
    int mid[L::KB], mid_tr[L::KB];              // k_b number j, d_e = 0: row d_c = c, quarter g; transposed (lane k_a, d_c = 4g ..)
    int raw;                                    // piece of (d_a = 4g, d_b = c); d_a + 1: 16 TC further
    __device__ __forceinline__ void make(int wave, int lane)
    {
        const int c = lane & 15, g = lane >> 4;
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            own[i] = L::at(L::TPW * wave + L::TE * i, c, g);
            own_tr[i] = L::at(L::TPW * wave + L::TE * i, 4 * g + (c >> 2), c & 3);
        }
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            mid[j] = L::at(c << L::te, wave * L::KB + j, g);
            mid_tr[j] = L::at((4 * g + (c >> 2)) << L::te, wave * L::KB + j, c & 3);
        }
        raw = L::piece(64 * g + c, wave * L::TPW / 8) + wave * L::TPW % 8;
    }
    static __device__ __forceinline__ int in_group(int k) { return (k % L::TE) * 512; }      // tile k from its group's first
};
template <class L>
__device__ __forceinline__ void read_pieces(u4w (&w)[4], const _Float16* raw)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = *reinterpret_cast<const u4w*>(raw + r * 16 * L::TC);
}
// one word of them: the samples of tiles 2p, 2p + 1 (a quarter of the registers, four times the accesses)
template <class L>
__device__ __forceinline__ void read_pair(uint32_t (&w)[4], const _Float16* raw, int p)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = reinterpret_cast<const uint32_t*>(raw + r * 16 * L::TC)[p];
}
template <class L>
__device__ __forceinline__ void write_pieces(const u4w (&w)[4], _Float16* raw)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) *reinterpret_cast<u4w*>(raw + r * 16 * L::TC) = w[r];
}
// this thread's pieces of a row in memory order, numbers tid + i NT: place of the first; the others STEP apart
template <class L>
__device__ __forceinline__ int piece_of(int tid)
{
    return L::piece(tid / (L::TC / 8), tid % (L::TC / 8));
}
// p + i, both uniform, kept as a scalar address: not to be turned into one per lane, in registers ahead of a loop
template <class T>
__device__ __forceinline__ T* uniform(T* p, size_t i)
{
    asm volatile("" : "+s"(i));
    return p + i;
}
// Memory behind a descriptor: 16 bytes at a lane's offset and a uniform one, without 64-bit addresses per lane; outside of `bytes`
// loads give zero and stores do nothing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}
__device__ __forceinline__ u4w row_load(__amdgpu_buffer_rsrc_t d, int lane_off, int off)
{
    return __builtin_bit_cast(u4w, __builtin_amdgcn_raw_buffer_load_b128(d, lane_off, off, 0));
}
__device__ __forceinline__ void row_store(__amdgpu_buffer_rsrc_t d, int lane_off, int off, const u4w& v)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, d, lane_off, off, BUF_ONCE);
}
// pattern of the largest sample of a wave's pieces (bf16): see band_or_exact
template <int PC>
__device__ __forceinline__ uint32_t pieces_max(const u4w (&v)[PC])
{
    uint32_t m[1] = {0u};
#pragma unroll
    for (int i = 0; i < PC; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) m[0] = mu::absmax_acc(m[0], v[i][q]);
    mu::band_or_exact<1>(m);
    return m[0];
}

template <class F>
hipError_t set_lds(F* f, size_t bytes)
{
    return hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

}  // namespace longrows
}  // namespace lc
