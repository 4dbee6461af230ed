// Matrix-core engine for single rows of N = 256 .. 4096 samples: spectrum, convolution (forward and du) and the
// whole backward pass.
//
// A real row needs only N complex points, without zero padding and without a second row to pair it with.  The
// causal convolution of two rows of N samples has 2N - 1 samples, so it equals its own remainder modulo
// x^2N + 1 = (x^N - i)(x^N + i) over the reals, and that ring is the complex numbers' C[z]/(z^N - i): with
// w = exp(i pi / 2N), w^N = i, the twisted row x[n] w^-n has an ordinary N-point transform
//     X[f] = sum_n x[n] exp(-2 pi i n (4 f + 1) / 4N),
// products of such transforms are convolutions modulo z^N - i, c[n] + i c[n+N], and the real part is the causal
// convolution truncated to N samples.  The conjugate spectrum gives the correlation the same way.  (Right-angle
// convolution: R. E. Blahut, Fast Algorithms for Digital Signal Processing, and Nussbaumer's negacyclic rings.)
// Against two rows as real and imaginary part of a 2N-point transform this takes one factor of two less in every
// transform (4096 samples are 16*16*16, two digits in registers and one exchange through LDS, instead of four
// digits), half the spectrum bins, no lost half at an odd batch, and rows that are scaled one by one.
//
// N = 16*16*TC, n = (d_a 16 + d_b) TC + d_c, f = k_a + 16 k_b + 256 k_c.  An MFMA tile has two index positions,
// X = lane % 16 and Y = (lane / 16, register); a contraction runs over Y, data as B operand keeps (X, Y), data as
// A operand comes out transposed.
//   phase 1 (tile d_c):   samples, X = d_b, Y = d_a  -[F16 over d_a, real input]-> X = k_a, Y = d_b  * w_256^(k_a d_b)
//                         -[F16 over d_b]-> X = k_a, Y = k_b -> LDS
//   phase 2 (tile = 16 columns (k_a, k_b) times the TC values of d_c): [F_TC over d_c] * spectrum [F_TC^-1]
//   phase 3 (tile d_c):   X = k_a, Y = k_b -[F16^-1 over k_b]-> X = d_b, Y = k_a * conj(w_256^(k_a d_b))
//                         -[F16^-1 over k_a, real part only]-> X = d_b, Y = d_a: samples
// The twist w^-n and all factors that depend on d_c are folded into the matrices of the tile's two 16-point blocks,
// so one twiddle table (four words per lane) serves every tile and both directions.  Constants stay in registers.
// From N = 2048 on a wave owns tiles 2w, 2w+1 of all three phases and TC/2 waves share a row; up to N = 1024 a wave owns
// whole rows, at N = 1024 with four tiles (the gated backward pass, which has no registers for them, shares it between two).
#include "engines.hpp"
#include "mfma_util.hpp"

namespace lc {
namespace {
using namespace mu;

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
// keeps the phases of an iteration apart in the instruction stream: mixed by the scheduler they need more than the 128
// registers that four waves per SIMD leave
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#define MFMA16(a, b, acc) __builtin_amdgcn_mfma_f32_16x16x16f16((a), (b), (acc), 0, 0, 0)

template <int LG>
struct RC {
    static constexpr int N = 1 << LG, cb = LG - 8, TC = 1 << cb;
    static constexpr int NWR = TC >= 4 ? TC / 2 : 1;      // waves that share a row
    static constexpr int RPI = TC == 1 ? 2 : 1;           // rows a group of waves takes at a time
    static constexpr int NS = TC == 1 ? 1 : 2;            // of a pair of tiles: those with constants and bins of their own
    // kernels whose waves own whole rows: pairs of tiles of a wave (one row's up to N = 1024), and tiles with their own constants
    static constexpr int NP = TC == 4 ? 2 : 1, NT = NP * NS;
    // words between the planes of two d_c in the exchange buffer: phase 2 reads four planes at once, and these
    // strides put its 64 lanes on 64 banks
    static constexpr int P = TC == 16 ? 260 : (TC == 8 ? 264 : 256);
    static constexpr int XW = TC == 1 ? 0 : TC * P;       // words of one exchange buffer
    static constexpr int SW = N / 2 + (TC == 4 ? 128 : 0);   // words of a staged row (see stage_word)
    static constexpr int COLS = 256 / TC;                 // columns of a phase-2 tile
    // A forward chain scales by 2^-SHIFT, an inverse one by twice that, in its last block, whose result stays fp32.  N bins
    // of N points are all the energy there is where a pair's transform had 2N, so at equal scales the products with the
    // spectrum, in fp16, were 1.8 times as large as a pair's and rows of a mean A overflowed from A sum k = 1137 at N = 4096.
    static constexpr int SHIFT = 4 + (cb >= 3 ? 2 : (cb >= 1 ? 1 : 0));
};

// ---- constant tables: lane-ordered 16-byte units, per length 6 units per tile and 4 common ones ---------------------
constexpr int ROWS_MIN = 8, ROWS_MAX = 12;
__host__ __device__ constexpr int tab_units(int lg) { return 6 * (1 << (lg - 8)) + 4; }
__host__ __device__ constexpr int tab_offset(int lg)
{
    int o = 0;
    for (int l = ROWS_MIN; l < lg; ++l) o += tab_units(l);
    return o;
}
constexpr int TAB_TOTAL = tab_offset(ROWS_MAX + 1);
static __device__ uint4 g_rows_tab[TAB_TOTAL * 64];

// d_b at index position i: natural, except at N = 256 (even ones first, see load_words256)
__device__ __forceinline__ int db_of(int lg, int i) { return lg == 8 ? 2 * (i & 7) + (i >> 3) : i; }
// phase 2's Y position -> (column group, d_c or k_c)
__device__ __forceinline__ void yc_of(int cb, int i, int& s, int& d)
{
    const int y = i >> 2, r = i & 3;
    if (cb == 4) { s = 0; d = i; }
    else if (cb == 3) { s = y >> 1; d = 4 * (y & 1) + r; }
    else if (cb == 2) { s = y; d = r; }
    else { s = y + 4 * (r >> 1); d = r & 1; }
}

__global__ void fill_rows_tab_kernel(uint4* tab, int lg)
{
    const int cb = lg - 8, TC = 1 << cb;
    const double N = (double)(1 << lg);
    const int unit = blockIdx.x, lane = threadIdx.x, x = lane & 15, y = lane >> 4;
    union { _Float16 h[8]; uint4 u; } o;
    // exp(-2 pi i t), scaled
    auto w = [](double t, double sc, double& re, double& im) {
        double s, c;
        sincospi(-2.0 * t, &s, &c);
        re = c * sc; im = s * sc;
    };
    double re, im;
    if (unit < 6 * TC) {
        const int dc = unit / 6, what = unit % 6;
        for (int q = 0; q < 4; ++q) {
            const int yr = 4 * y + q;
            // block over d_a, and the one over d_b with the inner twiddle; each scaled by 1/4
            auto fa = [&](int ka, int da) { w(da * ka / 16.0 + da / 64.0 + dc * (4.0 * ka + 1.0) / (4.0 * N), 0.25, re, im); };
            auto fb = [&](int kb, int db) { w(db * kb / 16.0 + db / 1024.0 + (double)dc * kb / (16.0 * TC), 0.25, re, im); };
            switch (what) {
                case 0: fa(x, yr); o.h[q] = (_Float16)re; o.h[4 + q] = (_Float16)im; break;
                case 1: fb(x, db_of(lg, yr)); o.h[2 * q] = (_Float16)re; o.h[2 * q + 1] = (_Float16)(-im); break;
                case 2: fb(x, db_of(lg, yr)); o.h[2 * q] = (_Float16)im; o.h[2 * q + 1] = (_Float16)re; break;
                // conjugates, other index on the lanes
                case 3: fb(yr, db_of(lg, x)); o.h[2 * q] = (_Float16)re; o.h[2 * q + 1] = (_Float16)im; break;
                case 4: fb(yr, db_of(lg, x)); o.h[2 * q] = (_Float16)(-im); o.h[2 * q + 1] = (_Float16)re; break;
                // twice as large: see SHIFT
                default: fa(yr, x); o.h[2 * q] = (_Float16)(2.0 * re); o.h[2 * q + 1] = (_Float16)(2.0 * im); break;
            }
        }
    } else {
        const int what = unit - 6 * TC;
        for (int q = 0; q < 4; ++q) {
            const int yr = 4 * y + q;
            if (what == 0) {
                w(x * db_of(lg, yr) / 256.0, 1.0, re, im);
                o.h[2 * q] = (_Float16)re; o.h[2 * q + 1] = (_Float16)im;
            } else if (what == 1) {
                w(db_of(lg, x) * yr / 256.0, 1.0, re, im);
                o.h[2 * q] = (_Float16)re; o.h[2 * q + 1] = (_Float16)im;
            } else {
                re = im = 0.0;
                if (TC > 1) {
                    int si, ki, sk, dk;
                    yc_of(cb, x, si, ki);
                    yc_of(cb, yr, sk, dk);
                    if (si == sk) w((double)(ki * dk % TC) / TC, cb >= 3 ? 0.25 : 0.5, re, im);
                }
                o.h[2 * q] = (_Float16)(what == 2 ? re : im);
                o.h[2 * q + 1] = (_Float16)(what == 2 ? -im : re);
            }
        }
    }
    tab[(size_t)unit * 64 + lane] = o.u;
}

template <int LG, int NT = RC<LG>::NS>
struct RK {
    h4 fa_re[NT], fa_im[NT];      // [F16 over d_a]: B operand of a 16x16x16 product
    h8 b_re[NT], b_im[NT];        // [F16 over d_b]: A operand
    h8 bi_re[NT], bi_im[NT];      // its adjoint: B operand
    h8 ai[NT];                            // adjoint of [F16 over d_a], real rows of the product only
    H8U t1, t1i;                                  // w_256^(k_a d_b), k_a (t1) or d_b (t1i) on the lanes
    h8 c_re, c_im;                                // I (x) F_TC
};
template <int LG, int NT>
__device__ __forceinline__ void load_consts(RK<LG, NT>& K, const uint4* __restrict__ tab, int t0, int lane)
{
    using C = RC<LG>;
    const uint4* p = tab + (size_t)tab_offset(LG) * 64 + lane;
    union { uint4 u; struct { h4 a, b; } h; } v;
    H8U x;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const uint4* q = p + (size_t)(t0 + k) * 6 * 64;
        v.u = q[0]; K.fa_re[k] = v.h.a; K.fa_im[k] = v.h.b;
        x.u = q[64]; K.b_re[k] = x.v;
        x.u = q[128]; K.b_im[k] = x.v;
        x.u = q[192]; K.bi_re[k] = x.v;
        x.u = q[256]; K.bi_im[k] = x.v;
        x.u = q[320]; K.ai[k] = x.v;
    }
    p += (size_t)C::TC * 6 * 64;
    K.t1.u = p[0];
    K.t1i = K.t1;
    if (C::TC == 1) K.t1i.u = p[64];
    else { x.u = p[128]; K.c_re = x.v; x.u = p[192]; K.c_im = x.v; }
}

// Constants that a loop is about to use have to have arrived: a wait in front of the loop (an empty statement that reads
// them).  Otherwise the loop's own waits have to allow for them in every iteration, and with them for whatever was asked
// for since.
__device__ __forceinline__ void arrived(h8& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void arrived(h4& v) { asm volatile("" : "+v"(v)); }
template <int LG, int NT>
__device__ __forceinline__ void arrived(RK<LG, NT>& K)
{
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        arrived(K.fa_re[k]); arrived(K.fa_im[k]); arrived(K.ai[k]);
        arrived(K.b_re[k]); arrived(K.b_im[k]); arrived(K.bi_re[k]); arrived(K.bi_im[k]);
    }
    arrived(K.t1.v); arrived(K.t1i.v);
    if (RC<LG>::TC > 1) { arrived(K.c_re); arrived(K.c_im); }
}

// The factors of the complex products are read anew in every iteration, as far as the compiler can see.  Otherwise it computes their
// exchanged and negated halves in front of the loop, which the packed instructions have modifiers for, and keeps them: a register
// for every word of twiddles and spectrum, 16 of rconv_kernel's 128.  With the gate that kernel spilled four and reloaded them in
// every row: gated forward, bf16, B=16, H=300, N=4096 36.5 -> 32.5 us, B=7, H=193, N=2048 10.7 -> 9.8.
template <int LG, int NT, int NK>
__device__ __forceinline__ void keep_words(RK<LG, NT>& K, H8U (&kk)[NK])
{
    arrived(K.t1.v);
    if (RC<LG>::TC == 1) arrived(K.t1i.v);
    else K.t1i = K.t1;
#pragma unroll
    for (int k = 0; k < NK; ++k) arrived(kk[k].v);
}

// ---- global memory: a row (two rows at N = 256) behind a buffer descriptor; lanes that must not touch memory carry
// an offset beyond it (loads give zero, stores do nothing) ------------------------------------------------------------
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr uint32_t NOWHERE = 0x80000000u;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}
__device__ __forceinline__ uint32_t buf_load(rsrc_t r, uint32_t off)
{
    return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
}
__device__ __forceinline__ void buf_store(rsrc_t r, uint32_t off, uint32_t v)
{
    __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)off, 0, BUF_ONCE);
}

// Sample n of the row -> element of memory.  pad = 0: itself.  pad = N2 (2-D layer): rows of N2 elements stand for
// rows of 2 N2 samples whose second half is zero: nothing is kept for n with bit N2 set.
__device__ __forceinline__ uint32_t elem_of(uint32_t n, uint32_t pad)
{
    if (pad == 0) return n;
    return (n & pad) ? NOWHERE : (((n & ~(2 * pad - 1)) >> 1) | (n & (pad - 1)));
}
// byte offsets of the four words (register r = d_a % 4) of this lane's samples: tiles t0, t0+1 side by side; at
// N = 256 the samples of d_b = 2j, 2j+1, j = lane % 8, of row (lane / 8) % 2
template <int LG>
__device__ __forceinline__ void word_offsets(uint32_t (&off)[4], int t0, int lane, uint32_t pad, uint32_t row_step)
{
    using C = RC<LG>;
    const int x = lane & 15, y = lane >> 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int da = 4 * y + r;
        const uint32_t n = C::TC == 1 ? da * 16 + 2 * (x & 7) : (da * 16 + x) * C::TC + t0;
        const uint32_t e = elem_of(n, pad);
        off[r] = e == NOWHERE ? NOWHERE : 2u * e + (C::TC == 1 && x >= 8 ? row_step : 0u);
    }
}

// ---- bf16 rows: exponent of the power of two a row is divided by -----------------------------------------------------
// Largest-magnitude pattern over the words of one wave: the stand-in BAND_LOW if the cheap test shows that they lie in
// 2 .. 8, otherwise measured.  At N = 256 lanes 0-7 and 8-15 of every 16 hold different rows: m[0], m[1].
template <int RPI, int NP>
__device__ __forceinline__ void words_max(const uint32_t (&w)[NP][4], uint32_t (&m)[RPI])
{
    uint32_t a = 0u;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r) a = absmax_acc(a, w[p][r]);
    if constexpr (RPI == 1) {
        m[0] = a;
        band_or_exact<1>(m);
    } else {
        const uint32_t v = max(a & 0x7fffu, (a >> 16) & 0x7fffu);
        const bool big = __builtin_amdgcn_ballot_w64(v >= BAND_HIGH) != 0;
        const uint64_t lg = __builtin_amdgcn_ballot_w64(v >= BAND_LOW);
        if (__builtin_expect(big || !(lg & 0x00ff00ff00ff00ffull) || !(lg & 0xff00ff00ff00ff00ull), 0)) {
            uint32_t q = v;
            q = max(q, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)q, 0xB1, 0xf, 0xf, true));
            q = max(q, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)q, 0x4E, 0xf, 0xf, true));
            q = max(q, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)q, 0x141, 0xf, 0xf, true));
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                uint32_t s = 0u;
#pragma unroll
                for (int j = 0; j < 4; ++j) s = max(s, (uint32_t)__builtin_amdgcn_readlane((int)q, 16 * j + 8 * i));
                m[i] = s;
            }
        } else {
            m[0] = m[1] = BAND_LOW;
        }
    }
}

// ---- phases -----------------------------------------------------------------------------------------------------------
__device__ __forceinline__ h4 h4_of(uint32_t a, uint32_t b)
{
    union { uint32_t w[2]; h4 v; } u;
    u.w[0] = a; u.w[1] = b;
    return u.v;
}
// y * w and y * conj(w) of packed words
__device__ __forceinline__ uint32_t cmul_h2(uint32_t yw, h2 w)
{
    union { uint32_t u; h2 h; } y, o;
    y.u = yw;
    const h2 yx = {y.h[0], y.h[0]}, yy = {y.h[1], y.h[1]};
    const h2 ws = {-w[1], w[0]};
    o.h = __builtin_elementwise_fma(yy, ws, yx * w);
    return o.u;
}
// (yr + i yi) * w with real and imaginary part exchanged in the result word; CONJ: * conj(w)
template <bool CONJ>
__device__ __forceinline__ uint32_t cmul_swap(float yr, float yi, h2 w)
{
    const f2 v = {yr, yi};
    const h2 y = __builtin_convertvector(v, h2);
    const h2 yx = {y[0], y[0]}, yy = {y[1], y[1]};
    union { h2 h; uint32_t u; } cv;
    if (CONJ) {
        const h2 a = {-w[1], w[0]};                       // im, re of yr conj(w) ...
        cv.h = __builtin_elementwise_fma(yx, a, yy * w);  // ... and of i yi conj(w) = yi (w1 + i w0)
    } else {
        const h2 a = {w[1], w[0]}, b = {w[0], -w[1]};
        cv.h = __builtin_elementwise_fma(yx, a, yy * b);
    }
    return cv.u;
}

// Phase 1 of a pair of the wave's tiles (pair p: 2p, 2p + 1 of them).  w: raw words of the row(s); e: exponents (bf16 rows only).  The result goes to the
// exchange buffer at xw (this lane's place in plane t0), at N = 256 it stays in registers: z[row][k_b % 4] complex.
template <int LG, class IO, bool SCALED>
__device__ __forceinline__ void phase1_ops(const uint32_t (&w)[4], int e0, int e1, int lane, h4 (&op)[2])
{
    using C = RC<LG>;
    if constexpr (IsBf<IO>::v) {
        float lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) { lo[r] = __uint_as_float(w[r] << 16); hi[r] = __uint_as_float(w[r] & 0xffff0000u); }
        if constexpr (SCALED) {
            const int e = C::TC == 1 && (lane & 8) ? e1 : e0;
#pragma unroll
            for (int r = 0; r < 4; ++r) { lo[r] = ldexpf(lo[r], -e); hi[r] = ldexpf(hi[r], -e); }
        }
        op[0] = h4_of(pack_h2(lo[0], lo[1]), pack_h2(lo[2], lo[3]));
        op[1] = h4_of(pack_h2(hi[0], hi[1]), pack_h2(hi[2], hi[3]));
    } else {
        op[0] = h4_of(__builtin_amdgcn_perm(w[1], w[0], 0x05040100u), __builtin_amdgcn_perm(w[3], w[2], 0x05040100u));
        op[1] = h4_of(__builtin_amdgcn_perm(w[1], w[0], 0x07060302u), __builtin_amdgcn_perm(w[3], w[2], 0x07060302u));
    }
}
template <int LG, int NT>
__device__ __forceinline__ void phase1(const h4 (&op)[2], const RK<LG, NT>& K, uint32_t* xw, f4 (&zr)[2], f4 (&zi)[2], int p = 0)
{
    using C = RC<LG>;
    xw += 2 * p * C::P;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 r[2], s[2];
    H8U m[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        r[k] = MFMA16(op[k], K.fa_re[2 * p + k % C::NS], zero);
        s[k] = MFMA16(op[k], K.fa_im[2 * p + k % C::NS], zero);
    }
    if constexpr (C::TC == 1) {
        // tile k holds d_b = 2j + k of row 0 in its first 32 lanes and of row 1 in the others: exchanged to tile = row
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const auto q = __builtin_amdgcn_permlane32_swap(pack_h2(r[0][j], s[0][j]), pack_h2(r[1][j], s[1][j]), false, false);
            m[0].w[j] = cmul_h2(q[0], K.t1.c[j]);
            m[1].w[j] = cmul_h2(q[1], K.t1.c[j]);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) m[k].w[j] = cmul_pack(r[k][j], s[k][j], K.t1.c[j]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        zr[k] = MFMA(K.b_re[2 * p + k % C::NS], m[k].v, zero);
        zi[k] = MFMA(K.b_im[2 * p + k % C::NS], m[k].v, zero);
    }
    if constexpr (C::TC > 1) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
            *reinterpret_cast<uint4*>(xw + k * C::P) = make_uint4(pack_h2(zr[k][0], zi[k][0]), pack_h2(zr[k][1], zi[k][1]),
                                                                  pack_h2(zr[k][2], zi[k][2]), pack_h2(zr[k][3], zi[k][3]));
    }
}

// word offset of register r from the lane's place in a phase-2 tile
template <int LG>
__device__ __forceinline__ constexpr int p2_off(int r)
{
    return RC<LG>::cb == 1 ? (r & 1) * RC<LG>::P + (r >> 1) * 64 : r * RC<LG>::P;
}
// the lane's place in phase-2 tile t
template <int LG>
__device__ __forceinline__ int p2_base(int t, int lane)
{
    using C = RC<LG>;
    const int x = lane & 15, y = lane >> 4;
    int a = t * C::COLS + x;
    if (C::cb == 4) a += 4 * y * C::P;
    else if (C::cb == 3) a += 4 * (y & 1) * C::P + (y >> 1) * 16;
    else a += y * 16;
    return a;
}
// forward half: [F_TC over d_c] of the wave's two tiles.  The second tile's place is hidden from the compiler: it would
// pair the tiles' words in one instruction and then need a register move per word to line up the MFMA operands.
template <int LG>
__device__ __forceinline__ void phase2_read(const uint32_t* xp, H8U (&m)[2])
{
    int d = RC<LG>::COLS;
    asm("" : "+v"(d));
    const uint32_t* xq = xp + d;
#pragma unroll
    for (int r = 0; r < 4; ++r) m[0].w[r] = xp[p2_off<LG>(r)];
#pragma unroll
    for (int r = 0; r < 4; ++r) m[1].w[r] = xq[p2_off<LG>(r)];
}
template <int LG, int NT>
__device__ __forceinline__ void phase2_fwd(const H8U (&m)[2], const RK<LG, NT>& K, f4 (&yr)[2], f4 (&yi)[2])
{
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 2; ++k) { yr[k] = MFMA(K.c_re, m[k].v, zero); yi[k] = MFMA(K.c_im, m[k].v, zero); }
}
// inverse half, in place; m: words with real and imaginary part exchanged (the forward blocks then give the
// adjoint's result, exchanged again)
template <int LG, int NT>
__device__ __forceinline__ void phase2_inv(uint32_t* xp, const RK<LG, NT>& K, const H8U (&m)[2])
{
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 zr[2], zi[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) { zr[k] = MFMA(K.c_re, m[k].v, zero); zi[k] = MFMA(K.c_im, m[k].v, zero); }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) xp[k * RC<LG>::COLS + p2_off<LG>(r)] = pack_h2(zi[k][r], zr[k][r]);
}

// Phase 3 of the wave's two tiles: v[k] = samples, register r = d_a % 4, X = d_b (N = 256: tile k = samples
// d_b = 2j + k, as loaded).  m: words read from the exchange buffer, at N = 256 the words of the two rows.
template <int LG>
__device__ __forceinline__ void phase3_read(const uint32_t* xw, H8U (&m)[2])
{
#pragma unroll
    for (int k = 0; k < 2; ++k) m[k].u = *reinterpret_cast<const uint4*>(xw + k * RC<LG>::P);
}
template <int LG, int NT>
__device__ __forceinline__ void phase3(H8U (&m)[2], const RK<LG, NT>& K, f4 (&v)[2], int p = 0)
{
    using C = RC<LG>;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 r[2], s[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        r[k] = MFMA(m[k].v, K.bi_re[2 * p + k % C::NS], zero);
        s[k] = MFMA(m[k].v, K.bi_im[2 * p + k % C::NS], zero);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) m[k].w[j] = cmul_pack_conj(r[k][j], s[k][j], K.t1i.c[j]);
    if constexpr (C::TC == 1) {
        // tile = row -> tile k = the d_b = 2j + k of both rows (row 0 in lanes 0-7 of every 16)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int a = (int)m[0].w[j], b = (int)m[1].w[j];
            m[0].w[j] = (uint32_t)__builtin_amdgcn_update_dpp(a, b, 0x128, 0xf, 0xC, false);      // row_ror:8
            m[1].w[j] = (uint32_t)__builtin_amdgcn_update_dpp(b, a, 0x128, 0xf, 0x3, false);
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) v[k] = MFMA(K.ai[2 * p + k % C::NS], m[k].v, zero);
}
template <class IO>
__device__ __forceinline__ uint32_t pack_io(float a, float b) { return IsBf<IO>::v ? pack_bf2(a, b) : pack_h2(a, b); }
template <class IO>
__device__ __forceinline__ float lo_of(uint32_t w)
{
    if (IsBf<IO>::v) return __uint_as_float(w << 16);
    union { uint32_t u; h2 h; } c; c.u = w; return (float)c.h[0];
}
template <class IO>
__device__ __forceinline__ float hi_of(uint32_t w)
{
    if (IsBf<IO>::v) return __uint_as_float(w & 0xffff0000u);
    union { uint32_t u; h2 h; } c; c.u = w; return (float)c.h[1];
}
template <class IO>
__device__ __forceinline__ float dot_words(uint32_t a, uint32_t b, float s)
{
    union { uint32_t u; h2 h; bf2 b; } x, y;
    x.u = a; y.u = b;
    return IsBf<IO>::v ? __builtin_amdgcn_fdot2_f32_bf16(x.b, y.b, s, false) : __builtin_amdgcn_fdot2(x.h, y.h, s, false);
}
// Rows that several waves share travel between memory and LDS in 16-byte pieces, one per thread, side by side; the waves
// read and write their own words (4 bytes, a fraction of every 16 per wave: straight from memory every line would be
// fetched by each of the waves, and written several times) in these LDS copies, one barrier later or earlier.  Word index such that a wave's words spread over the banks; 16-byte pieces stay
// whole, and a lane's four words stay N / 32 words apart.
template <int LG>
__device__ __forceinline__ int stage_word(int w)
{
    return RC<LG>::TC == 16 ? w ^ ((w >> 4) & 4) : (RC<LG>::TC == 4 ? w + ((w >> 7) << 5) : w);
}

// which workgroup of a persistent grid: consecutive ones on one XCD (they share a head's spectrum in its L2)
__device__ __forceinline__ int xcd_swizzle(int b, int n) { return (n & 7) ? b : (b & 7) * (n >> 3) + (b >> 3); }

// a row of a [B, H, ...] tensor, walked head by head: `step` bytes to the next row of the head, `wrap` more from the row
// behind a head's last to the next head's first
struct RowPtr {
    const char* p;
    int b;
    __device__ __forceinline__ void next(int B, int64_t step, int64_t wrap)
    {
        p += step;
        if (++b == B) { b = 0; p += wrap; }
    }
};
// Which code an iteration runs.  Whole: every phase has a row (no conditions).  Scaled: some power of two is not one.
template <bool W, bool S> struct Mode { static constexpr bool whole = W, scaled = S; };
// samples times 2^ex -> word of the I/O dtype.  The power of two comes before the rounding: samples of a head whose stored
// spectrum left one out may lie outside fp16's range until they have it back, gated ones in particular.
template <class IO, bool SCALED>
__device__ __forceinline__ uint32_t out_word(float a, float b, int ex)
{
    return SCALED ? pack_io<IO>(ldexpf(a, ex), ldexpf(b, ex)) : pack_io<IO>(a, b);
}

// Waves of workgroups that share a compute unit issue in the order of their age where they compete, so that the older workgroup
// runs at the speed it has alone and the younger one with what is left: of two at N = 4096 a row in 1.75 and 3.5 us, and when the
// first is through with its rows the second runs the rest by itself.  So the issue priority rises with the number of the
// workgroup, in steps of the 256 compute units of a whole device (LEVELS of them; with another number of units the results are the
// same and the priorities fall elsewhere).  Set behind the constants' way in; at the kernel's start it changed nothing.  bf16, back to
// back on the same tensors and (behind the comma) on tensors in turn that exceed the last-level cache: forward B=8, H=64, N=4096 9.7 ->
// 8.9 us, 10.4 -> 9.7, B=16, H=64, N=2048 9.7 -> 8.9, 10.2 -> 9.3, B=32, H=256, N=512 7.6 -> 7.1, 8.3 -> 8.3; steps B=64, H=1024, N=256
// 47.5 -> 46.0, 64.8 -> 63.3, gated B=7, H=193, N=2048 37.1 -> 36.2, 38.3 -> 37.7.  (The backward kernels of 1024 samples and more lose
// 1 % or nothing, those of one workgroup per compute unit have nobody to share with.)
template <int LEVELS>
__device__ __forceinline__ void younger_first()
{
    constexpr unsigned CU = 256;
    if (LEVELS > 1 && blockIdx.x >= 3 * CU) __builtin_amdgcn_s_setprio(3);
    else if (LEVELS > 1 && blockIdx.x >= 2 * CU) __builtin_amdgcn_s_setprio(2);
    else if (blockIdx.x >= CU) __builtin_amdgcn_s_setprio(1);
}

typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u4v buf_load4(rsrc_t r, uint32_t off)
{
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
}
// -------------------------------------------------------------------------------------
// Convolution of all rows, rows shared by NWR waves (N >= 2048).  Persistent workgroups, each with a run of consecutive
// rows (head by head).  Software pipeline over rows, one barrier per row: iteration t stores row t - 3, runs phase 3 of
// row t - 2, phase 2 of row t - 1 and phase 1 of row t, puts row t + 1 into LDS and asks for row t + 2.  Phase 3 reads
// the planes that the same wave's phase 1 then writes, so two exchange buffers serve all three phases.
// Loads and stores are issued in every iteration, with an empty descriptor where there is no row: conditional ones
// would make the compiler wait for younger requests than it has to.
// Bound by matrix and vector issue, which add up.
// Whole steps, row pairs in 2N points against rows: B=64, H=1024, N=4096 1564 -> 837 us; N=256 85 -> 67 us.
// -------------------------------------------------------------------------------------
template <int LG, class IO, bool CONJ, bool GATE>
__global__ void __launch_bounds__(RC<LG>::NWR * 64) __attribute__((amdgpu_waves_per_eu(4)))
rconv_kernel(const typename IO::T* __restrict__ in, const float2* __restrict__ kspec, typename IO::T* __restrict__ out,
             const typename IO::T* __restrict__ gate, int B, int H, int items, uint32_t pad, const uint4* __restrict__ tab)
{
    using C = RC<LG>;
    constexpr bool BF = IsBf<IO>::v;
    __shared__ __align__(16) uint32_t xbuf[2 * C::XW];
    __shared__ __align__(16) uint32_t raw[2 * C::SW];
    __shared__ __align__(16) uint32_t stg[2 * C::SW];
    __shared__ __align__(16) uint32_t mxs[2 * 8];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t0 = 2 * wave;
    const int x = lane & 15, y = lane >> 4;
    const int g = xcd_swizzle(blockIdx.x, gridDim.x);
    const int each = items / (int)gridDim.x, more = items - each * (int)gridDim.x;
    const int i0 = g * each + min(g, more), n = each + (g < more);          // this workgroup's rows
    if (n <= 0) return;
    const uint32_t row_bytes = (pad ? C::N / 2 : C::N) * 2u;
    const int64_t step = (int64_t)H * row_bytes, wrap = (int64_t)row_bytes - B * step;
    int h = i0 / B, b = i0 - h * B;                 // row of phase 1
    const int64_t o0 = (int64_t)b * step + (int64_t)h * row_bytes;
    RowPtr pi = {reinterpret_cast<const char*>(in) + o0, b}, po = {reinterpret_cast<const char*>(out) + o0, b};
    RowPtr pg = {reinterpret_cast<const char*>(gate) + o0, b};
    const uint32_t fe = elem_of(8u * threadIdx.x, pad), foff = fe == NOWHERE ? NOWHERE : 2u * fe;
    u4v rr = buf_load4(make_rsrc(pi.p, row_bytes), foff);                   // this thread's piece of a row
    pi.next(B, step, wrap);
    uint32_t off[4], ga[4] = {0u, 0u, 0u, 0u};
    if (GATE) word_offsets<LG>(off, t0, lane, pad, 0u);
    RK<LG> K;
    load_consts<LG>(K, tab, t0, lane);
    H8U kk[2];
    int es1 = 0, es2 = 0;                  // spectrum exponents of the rows in phases 2 and 3
    auto load_spec = [&]() {
        const uint4* ks = reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(kspec) + (size_t)h * 2 * C::N);
        kk[0].u = ks[t0 * 64 + lane];
        kk[1].u = ks[(t0 + 1) * 64 + lane];
        es1 = spec_exp_of(kspec, H, 2 * C::N)[h];
    };
    uint32_t* xw = xbuf + (size_t)t0 * C::P + 4 * lane;           // phases 1 and 3
    uint32_t* xp = xbuf + p2_base<LG>(t0, lane);                  // phase 2
    const int sw = stage_word<LG>(((4 * y * 16 + x) * C::TC + t0) / 2), sf = stage_word<LG>(4 * threadIdx.x);
    int e0 = 0, e1 = 0, e2 = 0;            // row exponents (bf16) of the rows in phases 1, 2 and 3
    // row t has arrived: into LDS, with the pattern of its largest sample; row t + 1 is asked for
    auto arrive = [&](int t) {
        if constexpr (BF) {
            uint32_t m[1];
            const uint32_t w[1][4] = {{rr[0], rr[1], rr[2], rr[3]}};
            words_max(w, m);
            if (lane == 0) mxs[(t & 1) * 8 + wave] = m[0];
        }
        *reinterpret_cast<u4v*>(raw + (t & 1) * C::SW + sf) = rr;
        rr = buf_load4(make_rsrc(pi.p, t + 1 < n ? row_bytes : 0u), foff);
        pi.next(B, step, wrap);
    };
    load_spec();
    arrived(K);
    arrived(kk[0].v); arrived(kk[1].v);
    arrive(0);
    __syncthreads();
    auto iter = [&](auto mode, int t) {
        using M = decltype(mode);
        const bool do1 = M::whole || t < n, do2 = M::whole || (t >= 1 && t - 1 < n), do3 = M::whole || (t >= 2 && t - 2 < n);
        const int bt = (t & 1) * C::XW, bs = C::XW - bt;
        H8U m3[2], m2[2];
        uint32_t w[4];
        keep_words(K, kk);
        if (do1) {
            const uint32_t* rw = raw + (t & 1) * C::SW + sw;
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = rw[r * (C::N / 32)];
        }
        if (do3) phase3_read<LG>(xw + bt, m3);
        const u4v q = *reinterpret_cast<const u4v*>(stg + ((t - 1) & 1) * C::SW + sf);
        if (do1) {
            h4 op[2];
            f4 zr[2], zi[2];
            phase1_ops<LG, IO, M::scaled>(w, e0, 0, lane, op);
            phase1<LG>(op, K, xw + bt, zr, zi);
        }
        __builtin_amdgcn_raw_buffer_store_b128(q, make_rsrc(po.p, M::whole || t >= 3 ? row_bytes : 0u), (int)foff, 0, BUF_ONCE);
        if (M::whole || t >= 3) po.next(B, step, wrap);
        SCHED_FENCE();
        if (do2) phase2_read<LG>(xp + bs, m2);
        if (do3) {
            f4 v[2];
            phase3<LG>(m3, K, v);
            uint32_t* st = stg + (t & 1) * C::SW + sw;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                st[r * (C::N / 32)] = GATE ? out_word<IO, M::scaled>(v[0][r] * lo_of<IO>(ga[r]), v[1][r] * hi_of<IO>(ga[r]), es2 + e2)
                                           : out_word<IO, M::scaled>(v[0][r], v[1][r], es2 + e2);
        }
        SCHED_FENCE();
        if (GATE) {                                     // the gate of row t - 1, for the next iteration's phase 3
            const rsrc_t d = make_rsrc(pg.p, do2 ? row_bytes : 0u);
#pragma unroll
            for (int r = 0; r < 4; ++r) ga[r] = buf_load(d, off[r]);
            if (do2) pg.next(B, step, wrap);
        }
        if (do2) {
            f4 yr[2], yi[2];
            phase2_fwd<LG>(m2, K, yr, yi);
            H8U mm[2];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) mm[k].w[r] = cmul_swap<CONJ>(yr[k][r], yi[k][r], kk[k].c[r]);
            phase2_inv<LG>(xp + bs, K, mm);
        }
        es2 = es1; e2 = e1; e1 = e0;
        SCHED_FENCE();
        // The spectrum before the row: requests are counted in their order, and phase 2 would have to wait for a row asked for
        // in front of its spectrum, half an iteration early, in every iteration.  (No faster where the rows come from the
        // last-level cache.)
        if (do1) {
            if (b == 0 && t > 0) load_spec();           // the next phase 2 is another head's
            if (++b == B) { b = 0; ++h; }
        }
        SCHED_FENCE();
        arrive(t + 1);
        __syncthreads();
    };
    // exponent of row t; what kind of iteration t is: 0 at the ends, 1 whole, 2 whole and nothing scaled
    auto prep = [&](int t) {
        if constexpr (BF) {
            int e = e0;
            if (t < n) {
                const uint32_t* mw = mxs + (t & 1) * 8;
                e = 0;                                   // every wave found its words in the band
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(mw[lane & (C::NWR - 1)] != BAND_LOW) != 0, 0)) {
                    uint32_t mm = 0u;
#pragma unroll
                    for (int w = 0; w < C::NWR; ++w) mm = max(mm, mw[w]);
                    e = row_exponent(__builtin_amdgcn_readfirstlane((int)mm));
                }
            }
            e0 = e;
        }
        return t >= 3 && t < n ? ((e0 | e2 | es2) == 0 ? 2 : 1) : 0;
    };
    // (a loop of its own for each kind: iterations of one kind following each other keep everything in place)
    younger_first<C::NWR == 4 ? 3 : 1>();
    for (int t = 0;;) {
        int kind = prep(t);
        while (kind == 2) { iter(Mode<true, false>{}, t); kind = prep(++t); }
        while (kind == 1) { iter(Mode<true, true>{}, t); kind = prep(++t); }
        if (t >= n + 3) break;
        if (kind == 0) { iter(Mode<false, true>{}, t); ++t; }
    }
}

// Words of pass rows at the lane's offsets: one load of 8 bytes where the wave owns two pairs of tiles.
template <int NP>
__device__ __forceinline__ void load_words(rsrc_t d, const uint32_t (&off)[4], uint32_t (&w)[NP][4])
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if constexpr (NP == 2) {
            const u2v v = __builtin_amdgcn_raw_buffer_load_b64(d, (int)off[r], 0, 0);
            w[0][r] = v[0]; w[1][r] = v[1];
        } else {
            w[0][r] = buf_load(d, off[r]);
        }
    }
}
template <int NP>
__device__ __forceinline__ void store_words(rsrc_t d, const uint32_t (&off)[4], const uint32_t (&w)[NP][4])
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if constexpr (NP == 2) {
            const u2v v = {w[0][r], w[1][r]};
            __builtin_amdgcn_raw_buffer_store_b64(v, d, (int)off[r], 0, BUF_ONCE);
        } else {
            buf_store(d, off[r], w[0][r]);
        }
    }
}

// The same for rows that one wave owns (N = 256: two rows at a time; N = 512; N = 1024: four tiles): no barrier, no
// staging (a wave's words already cover 32 to 128 contiguous bytes), and nothing to fill and drain for a wave's few rows.
// N = 1024 as a row pipeline of two waves (rconv_kernel's), kernel time in us, there -> here, bf16: B=1, H=768
// 6.7 -> 4.8; B=16, H=256 12.2 -> 8.6; B=16, H=768 21.3 -> 17.1; B=64, H=1024 75.7 -> 68.9 (3.9 TB/s).
// Three waves per SIMD at N = 1024 (168 registers, without the gate; two before keep_words): B=16, H=768 16.9 -> 15.2, B=64,
// H=1024 72 -> 67.
template <int LG, class IO, bool CONJ, bool GATE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(RC<LG>::NP == 2 ? (GATE ? 2 : 3) : 4)))
rconv1_kernel(const typename IO::T* __restrict__ in, const float2* __restrict__ kspec, typename IO::T* __restrict__ out,
              const typename IO::T* __restrict__ gate, int B, int H, int bpi, int items, uint32_t pad,
              const uint4* __restrict__ tab)
{
    using C = RC<LG>;
    constexpr bool BF = IsBf<IO>::v;
    constexpr int NP = C::NP, NT = C::NT;
    __shared__ __align__(16) uint32_t xbuf[C::TC == 1 ? 4 : 4 * C::XW];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ng = gridDim.x * 4, g = xcd_swizzle(blockIdx.x, gridDim.x) * 4 + wave;
    const int each = items / ng, more = items - each * ng;
    const int i0 = g * each + min(g, more), i1 = i0 + each + (g < more);    // this wave's passes
    if (i1 <= i0) return;
    const uint32_t row_bytes = pad ? C::N : 2 * C::N;
    const uint32_t row_step = (uint32_t)H * row_bytes;            // from a row to the next of its head
    const int64_t step = (int64_t)C::RPI * row_step, wrap = (int64_t)row_bytes - bpi * step;
    int h = i0 / bpi;
    const int b0 = i0 - h * bpi;                                  // RowPtr::b counts passes of RPI rows
    const int64_t o0 = (int64_t)b0 * step + (int64_t)h * row_bytes;
    RowPtr pi = {reinterpret_cast<const char*>(in) + o0, b0}, po = {reinterpret_cast<const char*>(out) + o0, b0};
    RowPtr pg = {reinterpret_cast<const char*>(gate) + o0, b0};
    const int odd = C::RPI == 2 ? B >> 1 : bpi;                   // the pass without a second row
    auto rsrc = [&](const RowPtr& q) { return make_rsrc(q.p, C::RPI == 2 && q.b != odd ? row_bytes + row_step : row_bytes); };
    uint32_t off[4];
    word_offsets<LG>(off, 0, lane, pad, row_step);
    uint32_t w[NP][4], gn[NP][4];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r) gn[p][r] = 0u;
    auto load = [&](RowPtr& q, uint32_t (&v)[NP][4], bool any) {  // (an empty descriptor where there is no row)
        load_words<NP>(any ? rsrc(q) : make_rsrc(q.p, 0u), off, v);
        q.next(bpi, step, wrap);
    };
    load(pi, w, true);
    if (GATE) load(pg, gn, true);
    RK<LG, NT> K;
    load_consts<LG>(K, tab, 0, lane);
    younger_first<LG < 10 ? 3 : 1>();
    uint32_t* xb = xbuf + (C::TC == 1 ? 0 : wave * C::XW);
    uint32_t* xw = xb + 4 * lane;
    uint32_t* xp = xb + p2_base<LG>(0, lane);
    H8U kk[NT];
    int es = 0;
    auto load_spec = [&]() {
        const uint4* ks = reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(kspec) + (size_t)h * 2 * C::N);
#pragma unroll
        for (int k = 0; k < NT; ++k) kk[k].u = ks[k * 64 + lane];
        es = spec_exp_of(kspec, H, 2 * C::N)[h];
    };
    load_spec();                                                  // (on its way together with the row and the constants)
    arrived(K);
#pragma unroll
    for (int k = 0; k < NT; ++k) arrived(kk[k].v);
    int ea = 0, eb = 0;                                           // exponents (bf16) of the pass's row(s)
    auto iter = [&](auto mode, int i) {
        using M = decltype(mode);
        h4 op[NP][2];
        f4 zr[2], zi[2], v[2];
        keep_words(K, kk);
        H8U m[2];
        uint32_t ga[NP][4], o[NP][4];
#pragma unroll
        for (int p = 0; p < NP; ++p) phase1_ops<LG, IO, M::scaled>(w[p], ea, eb, lane, op[p]);
        if (GATE) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int r = 0; r < 4; ++r) ga[p][r] = gn[p][r];
        }
        load(pi, w, i + 1 < i1);
        if (GATE) load(pg, gn, i + 1 < i1);
        SCHED_FENCE();                                  // (the loads go out here)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            phase1<LG>(op[p], K, xw, zr, zi, p);
            if (NP > 1) SCHED_FENCE();
        }
        if constexpr (C::TC == 1) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    m[k].w[r] = CONJ ? cmul_pack_conj(zr[k][r], zi[k][r], kk[0].c[r]) : cmul_pack(zr[k][r], zi[k][r], kk[0].c[r]);
        } else {
            wave_lds_fence();
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                f4 yr[2], yi[2];
                phase2_read<LG>(xp + 2 * p * C::COLS, m);
                phase2_fwd<LG>(m, K, yr, yi);
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) m[k].w[r] = cmul_swap<CONJ>(yr[k][r], yi[k][r], kk[2 * p + k % C::NS].c[r]);
                phase2_inv<LG>(xp + 2 * p * C::COLS, K, m);
                if (NP > 1) SCHED_FENCE();
            }
            wave_lds_fence();
        }
        const int ex = es + (C::TC == 1 && (lane & 8) ? eb : ea);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if constexpr (C::TC > 1) phase3_read<LG>(xw + 2 * p * C::P, m);
            phase3<LG>(m, K, v, p);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                o[p][r] = GATE ? out_word<IO, M::scaled>(v[0][r] * lo_of<IO>(ga[p][r]), v[1][r] * hi_of<IO>(ga[p][r]), ex)
                               : out_word<IO, M::scaled>(v[0][r], v[1][r], ex);
            if (NP > 1) SCHED_FENCE();
        }
        store_words<NP>(rsrc(po), off, o);
        po.next(bpi, step, wrap);
        h += po.b == 0;
    };
    // the pass has arrived: spectrum of a new head, exponents; is anything scaled?
    auto prep = [&](int i) {
        if (po.b == 0 && i != i0) {
            load_spec();
#pragma unroll
            for (int k = 0; k < NT; ++k) arrived(kk[k].v);
        }
        if constexpr (BF) {
            uint32_t m[C::RPI];
            words_max(w, m);
            ea = row_exponent(m[0]);
            if (C::RPI == 2) eb = row_exponent(m[C::RPI - 1]);
        }
        return (es | ea | eb) != 0;
    };
    for (int i = i0;;) {
        bool scaled = prep(i);
        while (!scaled) {
            iter(Mode<true, false>{}, i);
            if (++i == i1) return;
            scaled = prep(i);
        }
        iter(Mode<true, true>{}, i);
        if (++i == i1) return;
    }
}

// -------------------------------------------------------------------------------------
// Spectrum of the kernel (Algorithm 2 lines 1-2), one group of NWR waves per head: phase 1 and the forward half of
// phase 2 of the row scaled by a power of two to magnitude one.  Stored: (kscale FFT + kscale D) 2^-e_h as fp16
// complex in phase 2's lane order (word (tile 64 + lane) 4 + register), e_h in the trailer (spec_exponent).
// Bound by one round trip per head.  H=768, N=1024: 4.8 us (2N points: 6 us).
// -------------------------------------------------------------------------------------
template <int LG>
__global__ void __launch_bounds__(RC<LG>::NWR * 64)
rkspec_kernel(const float* __restrict__ k, const float* __restrict__ D, float2* __restrict__ kspec, int H, float kscale,
              uint32_t pad, const uint4* __restrict__ tab)
{
    using C = RC<LG>;
    __shared__ __align__(16) uint32_t xbuf[C::TC == 1 ? 4 : C::XW];
    __shared__ float wmax[3][8];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t0 = 2 * wave;
    const int h = blockIdx.x;
    const uint32_t row_bytes = (pad ? C::N / 2 : C::N) * 4u;
    const rsrc_t d = make_rsrc(reinterpret_cast<const char*>(k) + (size_t)h * row_bytes, row_bytes);
    uint32_t off[4];
    word_offsets<LG>(off, t0, lane, pad, NOWHERE);      // N = 256: the other row's lanes read zeros
    float v[4][2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t o = (off[r] & NOWHERE) ? NOWHERE : 2u * off[r];
        v[r][0] = __uint_as_float(buf_load(d, o));
        v[r][1] = __uint_as_float(buf_load(d, o == NOWHERE ? NOWHERE : o + 4u));
    }
    const float Dh = D[h];
    RK<LG> K;
    load_consts<LG>(K, tab, t0, lane);
    float m = 0.f, a = 0.f, mp = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            m = fmaxf(m, fabsf(v[r][i]));
            const float z = fabsf(v[r][i] + ((r == 0 && i == 0 && threadIdx.x == 0) ? Dh : 0.f));     // thread 0 holds k_0
            a += z;
            mp = fmaxf(mp, z);
        }
    for (int o = 32; o > 0; o >>= 1) {
        m = fmaxf(m, __shfl_xor(m, o, 64));
        mp = fmaxf(mp, __shfl_xor(mp, o, 64));
        a += __shfl_xor(a, o, 64);
    }
    if (C::NWR > 1) {
        if (lane == 0) { wmax[0][wave] = m; wmax[1][wave] = a; wmax[2][wave] = mp; }
        __syncthreads();
        m = wmax[0][0]; a = wmax[1][0]; mp = wmax[2][0];
#pragma unroll
        for (int w = 1; w < C::NWR; ++w) { m = fmaxf(m, wmax[0][w]); a += wmax[1][w]; mp = fmaxf(mp, wmax[2][w]); }
    }
    const float s = head_scale_of(m);
    const int es = spec_exponent(kscale * a, kscale * mp);
    if (threadIdx.x == 0) spec_exp_of(kspec, H, 2 * C::N)[h] = es;
    uint32_t w[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = pack_h2(v[r][0] * s, v[r][1] * s);
    h4 op[2];
    phase1_ops<LG, IoF16, false>(w, 0, 0, lane, op);
    f4 yr[2], yi[2];
    phase1<LG>(op, K, xbuf + (C::TC == 1 ? 0 : t0 * C::P + 4 * lane), yr, yi);
    if constexpr (C::TC > 1) {
        if (C::NWR > 1) __syncthreads(); else wave_lds_fence();
        H8U m2[2];
        phase2_read<LG>(xbuf + p2_base<LG>(t0, lane), m2);
        phase2_fwd<LG>(m2, K, yr, yi);
    }
    const float alpha = ldexpf(kscale * (float)(1 << C::SHIFT) / s, -es), beta = ldexpf(Dh * kscale, -es);
    uint4* o = reinterpret_cast<uint4*>(reinterpret_cast<uint32_t*>(kspec) + (size_t)h * 2 * C::N);
#pragma unroll
    for (int q = 0; q < C::NS; ++q)
        o[(t0 + q) * 64 + lane] = make_uint4(pack_h2(yr[q][0] * alpha + beta, yi[q][0] * alpha),
                                             pack_h2(yr[q][1] * alpha + beta, yi[q][1] * alpha),
                                             pack_h2(yr[q][2] * alpha + beta, yi[q][2] * alpha),
                                             pack_h2(yr[q][3] * alpha + beta, yi[q][3] * alpha));
}

// acc += conj(U) W 2^down
template <bool SCALED>
__device__ __forceinline__ void acc_tile(float2 (&acc)[4], const f4& ur, const f4& ui, const f4& wr, const f4& wi, int down)
{
    if constexpr (SCALED) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float a = ldexpf(wr[j], down), b = ldexpf(wi[j], down);
            acc[j].x = __builtin_fmaf(ui[j], b, __builtin_fmaf(ur[j], a, acc[j].x));
            acc[j].y = __builtin_fmaf(-ui[j], a, __builtin_fmaf(ur[j], b, acc[j].y));
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[j].x = __builtin_fmaf(ui[j], wi[j], __builtin_fmaf(ur[j], wr[j], acc[j].x));
            acc[j].y = __builtin_fmaf(-ui[j], wr[j], __builtin_fmaf(ur[j], wi[j], acc[j].y));
        }
    }
    // not to be moved past the end of the iteration: the sums read MFMA results, and no branch may come in between
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(acc[j].x), "+v"(acc[j].y));
}

// The waves' partial accumulators through LDS (red: NWV * NA * 4 * 64 float2) and added in group order by the first
// group's waves; returns the exponent of the sum's unit.  The caller puts a barrier in front if red is in use.
template <int NA, int NWR, int NGRP, bool BF>
__device__ __forceinline__ int acc_reduce(float2 (&acc)[NA][4], int eref, float2* red, int* erefs, int wave, int lane)
{
    if constexpr (NGRP == 1) return BF ? eref : 0;
#pragma unroll
    for (int k = 0; k < NA; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) red[((wave * NA + k) * 4 + j) * 64 + lane] = acc[k][j];
    if (BF && lane == 0 && wave % NWR == 0) erefs[wave / NWR] = eref;
    __syncthreads();
    int etop = 0;
    if constexpr (BF) {
        etop = erefs[0];
#pragma unroll
        for (int gi = 1; gi < NGRP; ++gi) etop = max(etop, erefs[gi]);
        etop = __builtin_amdgcn_readfirstlane(etop);
    }
    if (wave < NWR) {
#pragma unroll
        for (int k = 0; k < NA; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float2 s = acc[k][j];
                if constexpr (BF) { s.x = ldexpf(s.x, eref - etop); s.y = ldexpf(s.y, eref - etop); }
#pragma unroll
                for (int gi = 1; gi < NGRP; ++gi) {
                    float2 v = red[(((gi * NWR + wave) * NA + k) * 4 + j) * 64 + lane];
                    if constexpr (BF) { v.x = ldexpf(v.x, erefs[gi] - etop); v.y = ldexpf(v.y, erefs[gi] - etop); }
                    s.x += v.x; s.y += v.y;
                }
                acc[k][j] = s;
            }
    }
    return etop;
}

// -------------------------------------------------------------------------------------
// Whole backward pass of a head (or of a share of its rows) per workgroup, rows shared by NWR waves (N >= 2048, gated
// N >= 1024): du, dk
// and dD from one read of dy and u.  Per row: W = transform of dy, U = transform of u, du = inverse of W conj(K),
// A += conj(U) W in fp32 registers; dk is one inverse transform of A at the end.  Software pipeline as in rconv_kernel:
// phase 1 of both rows t, phase 2 of rows t - 1, phase 3 of du's row t - 2, row t - 3 stored, one barrier per row.
// NGRP groups of waves take every NGRP-th row; at the end they add their A in group order or, as two shares in one workgroup (see
// rows_bwd_nsplit), each turn their A into a row of dk, and these are added as those of two workgroups are.
// GATE (gated layer): dy is replaced by dz = dy g (rounded to the I/O dtype) as the rows arrive, dD sums dy g u in fp32,
// and U's own inverse of U K gives z for dg = dy z.
// -------------------------------------------------------------------------------------
template <int LG, bool GATE, bool WIDE> struct BwdCfg {
    // WIDE: twice the groups, for launches that give a compute unit one workgroup; N = 4096 has no LDS for them
    static constexpr bool can_widen = LG < 12;
    static constexpr bool can_pair = LG == 11 && WIDE;      // two shares in one workgroup
    static constexpr int NGRP = (LG == 10 ? 2 : 1) * (WIDE ? 2 : 1), NWV = NGRP * RC<LG>::NWR;
    // LDS words of a group: two exchange buffers, two rows on the way in and two on the way out for each tensor
    static constexpr int GW = 4 * RC<LG>::XW + (GATE ? 8 : 6) * RC<LG>::SW;
    static constexpr size_t lds = ((size_t)NGRP * GW + 2 * 8 * 2 + 8 + 8) * 4;
};
template <class T>
struct BwdArgs {
    const T* dy;
    const T* u;
    const T* g;
    const float2* kspec;
    T* du;
    T* dg;
    float* dk;
    float* dD;
    int B, H, nsplit, paired;
    float dkscale;
    uint32_t pad;
    const uint4* tab;
};
// dz = dy g in place of dy, and the fp32 sum of dy g u
template <class IO>
__device__ __forceinline__ float gate_words(uint32_t (&d)[4], const uint32_t (&g)[4], const uint32_t (&u)[4], float s)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float a = lo_of<IO>(d[r]) * lo_of<IO>(g[r]), b = hi_of<IO>(d[r]) * hi_of<IO>(g[r]);
        s = __builtin_fmaf(b, hi_of<IO>(u[r]), __builtin_fmaf(a, lo_of<IO>(u[r]), s));
        d[r] = pack_io<IO>(a, b);
    }
    return s;
}

// Three transforms per row against the convolution's two, at half its waves per SIMD (accumulators).
// Gated step B=7, H=193, N=2048: five kernels 93 us, this one 41 us.
template <int LG, class IO, bool DU, bool GATE, bool WIDE>
__global__ void __launch_bounds__((BwdCfg<LG, GATE, WIDE>::NWV * 64)) __attribute__((amdgpu_waves_per_eu(2)))
rbwd_kernel(const BwdArgs<typename IO::T> q)
{
    using C = RC<LG>;
    using Q = BwdCfg<LG, GATE, WIDE>;
    static_assert(DU || !GATE, "the gated form comes with du");
    constexpr bool BF = IsBf<IO>::v;
    constexpr int NGRP = Q::NGRP, NWR = C::NWR;
    extern __shared__ uint4 lds4[];
    uint32_t* lds = reinterpret_cast<uint32_t*>(lds4);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave / NWR, t0 = 2 * (wave % NWR), gt = threadIdx.x % (NWR * 64);
    const int x = lane & 15, y = lane >> 4;
    const int B = q.B, H = q.H, nsplit = q.nsplit;
    const uint32_t pad = q.pad;
    uint32_t* xd = lds + grp * Q::GW;                   // dy: two exchange buffers
    uint32_t* xu = xd + 2 * C::XW;                      // u: two
    uint32_t* raw = xu + 2 * C::XW;                     // dy (two rows), u (two rows) on the way in
    uint32_t* stg = raw + 4 * C::SW;                    // du (and dg) on the way out: two rows each
    uint32_t* mxs = lds + NGRP * Q::GW;                 // [2][8][2] patterns of the waves' words
    float* dred = reinterpret_cast<float*>(mxs + 32);   // [8]
    int* erefs = reinterpret_cast<int*>(dred + 8);      // [8]
    // workgroups of a head's shares are H apart: every head's first share first
    const int h = blockIdx.x % (unsigned)H, split = blockIdx.x / (unsigned)H;
    const int b0 = split * NGRP, bstep = nsplit * NGRP;               // group g takes rows b0 + g, b0 + g + bstep, ...
    const int niter = (B - b0 + bstep - 1) / bstep;                   // of the first group (>= 1); barriers stay uniform
    const int nmine = (B - b0 - grp + bstep - 1) / bstep;             // of this group
    const int nmin = (B - b0 - (NGRP - 1) + bstep - 1) / bstep;       // of the last
    const uint32_t row_bytes = (pad ? C::N / 2 : C::N) * 2u;
    const int64_t o0 = ((int64_t)(b0 + grp) * H + h) * row_bytes, step = (int64_t)bstep * H * row_bytes;
    const char* pdy = reinterpret_cast<const char*>(q.dy) + o0;      // rows to load
    const char* pu = reinterpret_cast<const char*>(q.u) + o0;
    const char* pg = reinterpret_cast<const char*>(q.g) + o0;
    const char* pdy3 = pdy;                                          // dy again, for dg
    char* pdu = reinterpret_cast<char*>(q.du) + o0;                  // rows to store
    char* pdg = reinterpret_cast<char*>(q.dg) + o0;
    const uint32_t fe = elem_of(8u * gt, pad), foff = fe == NOWHERE ? NOWHERE : 2u * fe;
    u4v rd, ru, rg = {0u, 0u, 0u, 0u};                               // this thread's pieces of the rows
    auto ask = [&](int t) {
        const uint32_t bytes = t < nmine ? row_bytes : 0u;           // (an empty descriptor where there is no row)
        rd = buf_load4(make_rsrc(pdy, bytes), foff); pdy += step;
        ru = buf_load4(make_rsrc(pu, bytes), foff); pu += step;
        if (GATE) { rg = buf_load4(make_rsrc(pg, bytes), foff); pg += step; }
    };
    ask(0);
    uint32_t off[4], dz[4] = {0u, 0u, 0u, 0u};
    if (GATE) word_offsets<LG>(off, t0, lane, pad, 0u);
    RK<LG> K;
    load_consts<LG>(K, q.tab, t0, lane);
    H8U kk[2];
    kk[0].u = kk[1].u = make_uint4(0u, 0u, 0u, 0u);
    int es = 0;
    if (DU) {
        const uint4* ks = reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(q.kspec) + (size_t)h * 2 * C::N);
        kk[0].u = ks[t0 * 64 + lane];
        kk[1].u = ks[(t0 + 1) * 64 + lane];
        es = spec_exp_of(q.kspec, H, 2 * C::N)[h];
    }
    const int xwo = t0 * C::P + 4 * lane, xpo = p2_base<LG>(t0, lane);
    const int sw = stage_word<LG>(((4 * y * 16 + x) * C::TC + t0) / 2), sf = stage_word<LG>(4 * gt);
    float2 acc[2][4];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[k][j] = make_float2(0.f, 0.f);
    float dsum = 0.f;
    int eref = EXP_NONE, ep0 = 0, ep1 = 0;                           // units of A and of the products
    int ed0 = 0, ed1 = 0, ed2 = 0, eu0 = 0, eu1 = 0, eu2 = 0;        // row exponents (bf16) in phases 1, 2, 3
    // rows t have arrived: gate, dot product, patterns, into LDS; rows t + 1 are asked for
    auto arrive = [&](int t) {
        uint32_t d[4] = {rd[0], rd[1], rd[2], rd[3]};
        const uint32_t v[4] = {ru[0], ru[1], ru[2], ru[3]}, g[4] = {rg[0], rg[1], rg[2], rg[3]};
        if (GATE) {
            dsum = gate_words<IO>(d, g, v, dsum);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) dsum = dot_words<IO>(d[r], v[r], dsum);
        }
        if constexpr (BF) {
            uint32_t md = 0u, mu_ = 0u;
#pragma unroll
            for (int r = 0; r < 4; ++r) { md = absmax_acc(md, d[r]); mu_ = absmax_acc(mu_, v[r]); }
            band_or_exact2(md, mu_);
            if (lane == 0) *reinterpret_cast<uint2*>(mxs + ((t & 1) * 8 + wave) * 2) = make_uint2(md, mu_);
        }
        *reinterpret_cast<uint4*>(raw + (t & 1) * C::SW + sf) = make_uint4(d[0], d[1], d[2], d[3]);
        *reinterpret_cast<uint4*>(raw + (2 + (t & 1)) * C::SW + sf) = make_uint4(v[0], v[1], v[2], v[3]);
        // All uses of rows t stand in front of the request for rows t + 1, which then takes their registers.  Otherwise the sum
        // of products is moved behind it, the rows come into registers of their own, are copied at the end of the same iteration
        // and so waited for there: bf16, B=64, H=1024, N=4096 521 -> 488 us, B=32, H=512, N=2048 71 -> 66.  (Rows in fp16 have no
        // branch to be moved across; holding the scheduler back costs them 1 %.)
        if constexpr (BF) {
            asm volatile("" : "+v"(dsum));
            SCHED_FENCE();
        }
        ask(t + 1);
    };
    arrived(K);
    arrived(kk[0].v); arrived(kk[1].v);
    arrive(0);
    __syncthreads();
    auto iter = [&](auto mode, int t) {
        using M = decltype(mode);
        const bool do1 = M::whole || t < nmine, do2 = M::whole || (t >= 1 && t - 1 < nmine);
        const bool do3 = DU && (M::whole || (t >= 2 && t - 2 < nmine));
        const int bt = (t & 1) * C::XW, bs = C::XW - bt;             // buffers of phases 1 and 3, and of phase 2
        H8U m3[2], n3[2], m2[2], n2[2];
        uint32_t wd[4], wu[4];
        if (do1) {
            const uint32_t* rw = raw + (t & 1) * C::SW + sw;
#pragma unroll
            for (int r = 0; r < 4; ++r) { wd[r] = rw[r * (C::N / 32)]; wu[r] = rw[2 * C::SW + r * (C::N / 32)]; }
        }
        if (do3) {
            phase3_read<LG>(xd + xwo + bt, m3);
            if (GATE) phase3_read<LG>(xu + xwo + bt, n3);
        }
        if (do1) {
            h4 op[2];
            f4 zr[2], zi[2];
            phase1_ops<LG, IO, M::scaled>(wd, ed0, 0, lane, op);
            phase1<LG>(op, K, xd + xwo + bt, zr, zi);
            phase1_ops<LG, IO, M::scaled>(wu, eu0, 0, lane, op);
            phase1<LG>(op, K, xu + xwo + bt, zr, zi);
        }
        if (DU) {
            const uint32_t bytes = M::whole || (t >= 3 && t - 3 < nmine) ? row_bytes : 0u;
            u4v o = *reinterpret_cast<const u4v*>(stg + ((t - 1) & 1) * C::SW + sf);
            __builtin_amdgcn_raw_buffer_store_b128(o, make_rsrc(pdu, bytes), (int)foff, 0, BUF_ONCE);
            if (M::whole || t >= 3) pdu += step;
            if (GATE) {
                o = *reinterpret_cast<const u4v*>(stg + (2 + ((t - 1) & 1)) * C::SW + sf);
                __builtin_amdgcn_raw_buffer_store_b128(o, make_rsrc(pdg, bytes), (int)foff, 0, BUF_ONCE);
                if (M::whole || t >= 3) pdg += step;
            }
        }
        if (do2) {
            phase2_read<LG>(xd + xpo + bs, m2);
            phase2_read<LG>(xu + xpo + bs, n2);
        }
        if (do3) {
            f4 v[2];
            phase3<LG>(m3, K, v);
            uint32_t* st = stg + (t & 1) * C::SW + sw;
#pragma unroll
            for (int r = 0; r < 4; ++r) st[r * (C::N / 32)] = out_word<IO, M::scaled>(v[0][r], v[1][r], es + ed2);
            if (GATE) {
                phase3<LG>(n3, K, v);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    st[2 * C::SW + r * (C::N / 32)] =
                        out_word<IO, M::scaled>(v[0][r] * lo_of<IO>(dz[r]), v[1][r] * hi_of<IO>(dz[r]), es + eu2);
            }
        }
        if (GATE) {                                     // dy of row t - 1, for the next iteration's dg
            const rsrc_t r3 = make_rsrc(pdy3, do2 ? row_bytes : 0u);
#pragma unroll
            for (int r = 0; r < 4; ++r) dz[r] = buf_load(r3, off[r]);
            if (do2) pdy3 += step;
        }
        if (do2) {
            f4 wr[2], wi[2], yr[2], yi[2];
            int down = 0;
            if constexpr (BF && M::scaled) down = acc_align<2>(acc, eref, ep1);    // (its branch: not behind an MFMA)
            phase2_fwd<LG>(m2, K, wr, wi);
            phase2_fwd<LG>(n2, K, yr, yi);
            if (DU) {
                H8U mm[2];
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mm[k].w[r] = cmul_swap<true>(wr[k][r], wi[k][r], kk[k].c[r]);
                phase2_inv<LG>(xd + xpo + bs, K, mm);
            }
            if (GATE) {
                H8U mm[2];
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mm[k].w[r] = cmul_swap<false>(yr[k][r], yi[k][r], kk[k].c[r]);
                phase2_inv<LG>(xu + xpo + bs, K, mm);
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) acc_tile<BF && M::scaled>(acc[k], yr[k], yi[k], wr[k], wi[k], down);
        }
        ed2 = ed1; ed1 = ed0;
        eu2 = eu1; eu1 = eu0;
        ep1 = ep0;
        SCHED_FENCE();                                  // (not into the middle: the rows were asked for one iteration ago)
        arrive(t + 1);
        __syncthreads();
    };
    // exponents of rows t; what kind of iteration t is: 0 at the ends, 1 whole, 2 whole and nothing scaled
    auto prep = [&](int t) {
        if constexpr (BF) {
            int d = ed0, v = eu0, p = ep0;               // (assigned once: stores on either side of a branch were merged in memory)
            if (t < nmine) {
                const uint32_t* mw = mxs + ((t & 1) * 8 + grp * NWR) * 2;
                d = v = p = 0;                           // every wave found its words in the band
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(mw[lane & (2 * NWR - 1)] != BAND_LOW) != 0, 0)) {
                    uint32_t md = 0u, mu_ = 0u;
#pragma unroll
                    for (int w = 0; w < NWR; ++w) { md = max(md, mw[2 * w]); mu_ = max(mu_, mw[2 * w + 1]); }
                    md = __builtin_amdgcn_readfirstlane((int)md);
                    mu_ = __builtin_amdgcn_readfirstlane((int)mu_);
                    d = row_exponent(md);
                    v = row_exponent(mu_);
                    p = md && mu_ ? d + v : EXP_NONE;
                }
            }
            ed0 = d; eu0 = v; ep0 = p;
        }
        if (t < 3 || t >= nmin) return 0;
        return (ed0 | eu0 | ed2 | es | (GATE ? eu2 : 0)) == 0 && (!BF || ep1 == eref) ? 2 : 1;
    };
    const int last = niter + (DU ? 3 : 1);
    for (int t = 0;;) {
        int kind = prep(t);
        while (kind == 2) { iter(Mode<true, false>{}, t); kind = prep(++t); }
        while (kind == 1) { iter(Mode<true, true>{}, t); kind = prep(++t); }
        if (t >= last) break;
        if (kind == 0) { iter(Mode<false, true>{}, t); ++t; }
    }

    for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
    if (lane == 0) dred[wave] = dsum;
    const bool paired = Q::can_pair && q.paired;
    const int nsum = paired ? NGRP : 1;                  // sums A that are turned into a row of dk, each by its group
    int etop = BF ? eref : 0;
    if (!paired) etop = acc_reduce<2, NWR, NGRP, BF>(acc, eref, reinterpret_cast<float2*>(lds), erefs, wave, lane);
    const size_t ho = (size_t)split * H + h;
    uint32_t* peaks = mxs;                               // [nsum * NWR] (the rows' patterns are done with)
    const uint32_t peak = acc_peak<2>(acc);
    if (lane == 0 && grp < nsum) peaks[wave] = peak;
    __syncthreads();                                     // (the reduction's words lie in the buffers that follow, too)
    if (q.dk) {
        if (grp < nsum) {
            uint32_t m = peaks[grp * NWR];
#pragma unroll
            for (int w = 1; w < NWR; ++w) m = max(m, peaks[grp * NWR + w]);
            const int ea = __builtin_amdgcn_readfirstlane(acc_exponent(m));
            etop += ea;
            H8U mm[2];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) mm[k].w[r] = pack_h2(ldexpf(acc[k][r].y, -ea), ldexpf(acc[k][r].x, -ea));
            phase2_inv<LG>(xd + xpo, K, mm);
        }
        __syncthreads();
        float* fs = reinterpret_cast<float*>(xu);        // the row of dk in the group's u buffers
        if (grp < nsum) {
            H8U m3[2];
            f4 v[2];
            phase3_read<LG>(xd + xwo, m3);
            phase3<LG>(m3, K, v);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<float2*>(fs + ((4 * y + r) * 16 + x) * C::TC + t0) =
                    make_float2(ldexpf(v[0][r] * q.dkscale, etop), ldexpf(v[1][r] * q.dkscale, etop));
        }
        __syncthreads();
        const uint32_t kb = (pad ? C::N / 2 : C::N) * 4u;
        const rsrc_t d = make_rsrc(reinterpret_cast<const char*>(q.dk) + ho * kb, kb);
        fs = reinterpret_cast<float*>(lds + 2 * C::XW);
        for (int i = threadIdx.x; i < C::N / 4; i += Q::NWV * 64) {
            const uint32_t e = elem_of(4u * i, pad);
            f4 v = *reinterpret_cast<const f4*>(fs + 4 * i);
            if (paired) v += *reinterpret_cast<const f4*>(fs + Q::GW + 4 * i);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, v), d, (int)(e == NOWHERE ? NOWHERE : 4u * e), 0, 0);
        }
    }
    if (threadIdx.x == 0 && q.dD) {
        float s = 0.f;
        for (int g = 0; g < nsum; ++g) {
            float t = 0.f;
            for (int w = 0; w < Q::NWV / nsum; ++w) t += dred[g * NWR + w];
            s += t;
        }
        q.dD[ho] = s;
    }
}

// The same for rows that one wave owns (N = 256: two rows at a time; N = 512; N = 1024: four tiles), NWV independent waves
// per workgroup.  N = 1024 as a row pipeline (rbwd_kernel, two groups of two waves), kernel time in us, there -> here,
// bf16: B=1, H=768 16.5 -> 8.1; B=5, H=64 12.0 -> 9.7; B=16, H=256 20.3 -> 14.4; B=16, H=768 37.4 -> 30.2; B=64, H=1024
// 137 -> 110.  (Gated N = 1024 spills 50 registers and more and is 1.5 times as slow as the pipeline.)  With the factors' words kept
// once (keep_words) N = 1024 spills none, where it had 6 to 14, B=1, H=768 7.9 -> 6.8, B=16, H=768 31.1 -> 29.6, and N = 512 has
// three waves per SIMD in place of two: B=64, H=1024 60.2 -> 54.7.  With the gate N = 256 and 512 have registers enough either way; fp16
// at N = 256 keeps the exchanged halves, too (words alone and with them: B=32, H=1024 23.2 and 21.0 us, B=64, H=512 19.4 and 18.5; bf16 21.3 and 22.9,
// out of band 22.4 and 22.0; N = 512, B=16, H=256 8.9 and 9.2, B=32, H=300 19.4 and 19.1).
template <int LG, class IO, bool DU, bool GATE, int NWV>
__global__ void __launch_bounds__(NWV * 64) __attribute__((amdgpu_waves_per_eu(2)))
rbwd1_kernel(const BwdArgs<typename IO::T> q)
{
    using C = RC<LG>;
    static_assert(DU || !GATE, "the gated form comes with du");
    constexpr bool BF = IsBf<IO>::v;
    constexpr int NP = C::NP, NS = C::NS, NT = C::NT;
    // the reduction's words: at N = 1024 in the exchange buffers, which are as large (two workgroups per compute unit)
    __shared__ __align__(16) uint32_t xbuf[C::TC == 1 ? 4 : NWV * 2 * C::XW];
    __shared__ float2 own[NP > 1 ? 1 : NWV * NT * 4 * 64];
    static_assert(NP == 1 || 2 * C::XW == NT * 4 * 64 * 2, "the accumulators of a wave fill its exchange buffers");
    float2* red = NP > 1 ? reinterpret_cast<float2*>(xbuf) : own;
    __shared__ float dred[NWV];
    __shared__ int erefs[NWV];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int B = q.B, H = q.H, nsplit = q.nsplit;
    const uint32_t pad = q.pad;
    const int h = blockIdx.x % (unsigned)H, split = blockIdx.x / (unsigned)H;
    const int npass = (B + C::RPI - 1) / C::RPI, pstep = nsplit * NWV, odd = C::RPI == 2 ? B >> 1 : npass;
    const uint32_t row_bytes = pad ? C::N : 2 * C::N, row_step = (uint32_t)H * row_bytes;
    const int p0 = split * NWV + wave;
    const int64_t o0 = (int64_t)p0 * C::RPI * row_step + (int64_t)h * row_bytes, step = (int64_t)pstep * C::RPI * row_step;
    const char* pdy = reinterpret_cast<const char*>(q.dy) + o0;
    const char* pu = reinterpret_cast<const char*>(q.u) + o0;
    const char* pg = reinterpret_cast<const char*>(q.g) + o0;
    char* pdu = reinterpret_cast<char*>(q.du) + o0;
    char* pdg = reinterpret_cast<char*>(q.dg) + o0;
    uint32_t off[4];
    word_offsets<LG>(off, 0, lane, pad, row_step);
    uint32_t wd[NP][4], wu[NP][4], gn[NP][4];
    auto bytes_of = [&](int p) { return C::RPI == 2 && p != odd ? row_bytes + row_step : row_bytes; };
    auto load = [&](const char*& ptr, int p, uint32_t (&w)[NP][4]) {
        load_words<NP>(make_rsrc(ptr, p < npass ? bytes_of(p) : 0u), off, w);      // (an empty descriptor where there is no row)
        ptr += step;
    };
    auto load_all = [&](int p) {
        load(pdy, p, wd);
        load(pu, p, wu);
        if (GATE) load(pg, p, gn);
    };
    load_all(p0);
    RK<LG, NT> K;
    load_consts<LG>(K, q.tab, 0, lane);
    H8U kk[NT];
    int es = 0;
    if (DU) {
        const uint4* ks = reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(q.kspec) + (size_t)h * 2 * C::N);
#pragma unroll
        for (int k = 0; k < NT; ++k) kk[k].u = ks[k * 64 + lane];
        es = spec_exp_of(q.kspec, H, 2 * C::N)[h];
    }
    uint32_t* xd = xbuf + (C::TC == 1 ? 0 : wave * 2 * C::XW);
    uint32_t* xu = xd + C::XW;
    const int xwo = C::TC == 1 ? 0 : 4 * lane, xpo = C::TC == 1 ? 0 : p2_base<LG>(0, lane);
    float2 acc[NT][4];
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[k][j] = make_float2(0.f, 0.f);
    arrived(K);
    if (DU) {
#pragma unroll
        for (int k = 0; k < NT; ++k) arrived(kk[k].v);
    }
    float dsum = 0.f;
    int eref = EXP_NONE;
    int eda = 0, edb = 0, eua = 0, eub = 0, epa = 0, epb = 0;      // exponents (bf16) of the pass's row(s), and of their products
    uint32_t gy[NP][4];                                  // dy's own words (gated layer)
    auto iter = [&](auto mode, int p) {
        using M = decltype(mode);
        h4 od[NP][2], ou[NP][2];
        if constexpr (!(GATE && LG == 8 && !BF)) keep_words(K, kk);
        f4 wr[2], wi[2], yr[2], yi[2], v[2];
        H8U m[2], n[2];
        uint32_t wy[NP][4], o[NP][4], og[NP][4];
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            phase1_ops<LG, IO, M::scaled>(wd[c], eda, edb, lane, od[c]);
            phase1_ops<LG, IO, M::scaled>(wu[c], eua, eub, lane, ou[c]);
            if (GATE) {
#pragma unroll
                for (int r = 0; r < 4; ++r) wy[c][r] = gy[c][r];
            }
        }
        load_all(p + pstep);
        SCHED_FENCE();                                  // (the loads go out here)
        if constexpr (BF && M::scaled) acc_align<NT>(acc, eref, C::TC == 1 ? max(epa, epb) : epa);
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            phase1<LG>(od[c], K, xd + xwo, wr, wi, c);
            phase1<LG>(ou[c], K, xu + xwo, yr, yi, c);
        }
        if constexpr (C::TC > 1) wave_lds_fence();
        auto accumulate = [&](int c) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                // N = 256: tile k is row k and both add to the same bins
                const int epk = C::TC == 1 && k == 1 ? epb : epa;
                acc_tile<BF && M::scaled>(acc[2 * c + k % NS], yr[k], yi[k], wr[k], wi[k], min(epk - eref, 0));
            }
        };
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            if constexpr (C::TC > 1) {
                phase2_read<LG>(xd + xpo + 2 * c * C::COLS, m);
                phase2_read<LG>(xu + xpo + 2 * c * C::COLS, n);
                phase2_fwd<LG>(m, K, wr, wi);
                phase2_fwd<LG>(n, K, yr, yi);
            }
            if (DU) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const h2 kw = kk[2 * c + k % NS].c[r];
                        m[k].w[r] = C::TC == 1 ? cmul_pack_conj(wr[k][r], wi[k][r], kw) : cmul_swap<true>(wr[k][r], wi[k][r], kw);
                        if (GATE) n[k].w[r] = C::TC == 1 ? cmul_pack(yr[k][r], yi[k][r], kw) : cmul_swap<false>(yr[k][r], yi[k][r], kw);
                    }
                if constexpr (C::TC > 1) {
                    phase2_inv<LG>(xd + xpo + 2 * c * C::COLS, K, m);
                    if (GATE) phase2_inv<LG>(xu + xpo + 2 * c * C::COLS, K, n);
                }
            }
            if constexpr (NP > 1) accumulate(c);
        }
        if (DU) {
            if constexpr (C::TC > 1) wave_lds_fence();
#pragma unroll
            for (int c = 0; c < NP; ++c) {
                if constexpr (C::TC > 1) {
                    phase3_read<LG>(xd + xwo + 2 * c * C::P, m);
                    if (GATE) phase3_read<LG>(xu + xwo + 2 * c * C::P, n);
                }
                phase3<LG>(m, K, v, c);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    o[c][r] = out_word<IO, M::scaled>(v[0][r], v[1][r], es + (C::TC == 1 && (lane & 8) ? edb : eda));
                if (GATE) {
                    phase3<LG>(n, K, v, c);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        og[c][r] = out_word<IO, M::scaled>(v[0][r] * lo_of<IO>(wy[c][r]), v[1][r] * hi_of<IO>(wy[c][r]),
                                                           es + (C::TC == 1 && (lane & 8) ? eub : eua));
                }
            }
            store_words<NP>(make_rsrc(pdu, bytes_of(p)), off, o);
            pdu += step;
            if (GATE) {
                store_words<NP>(make_rsrc(pdg, bytes_of(p)), off, og);
                pdg += step;
            }
        }
        if constexpr (NP == 1) accumulate(0);           // (behind the stores: the products' registers are there)
    };
    // the pass has arrived: gate, dot product, exponents; is anything scaled?
    auto prep = [&]() {
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            if (GATE) {
#pragma unroll
                for (int r = 0; r < 4; ++r) gy[c][r] = wd[c][r];
                dsum = gate_words<IO>(wd[c], gn[c], wu[c], dsum);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) dsum = dot_words<IO>(wd[c][r], wu[c][r], dsum);
            }
        }
        if constexpr (BF) {
            uint32_t md[C::RPI], mu_[C::RPI];
            words_max(wd, md);
            words_max(wu, mu_);
            eda = row_exponent(md[0]);
            eua = row_exponent(mu_[0]);
            epa = md[0] && mu_[0] ? eda + eua : EXP_NONE;
            if constexpr (C::RPI == 2) {
                edb = row_exponent(md[1]);
                eub = row_exponent(mu_[1]);
                epb = md[1] && mu_[1] ? edb + eub : EXP_NONE;
            }
        }
        return (es | eda | edb | eua | eub) != 0 || (BF && (epa != eref || (C::RPI == 2 && epb != eref)));
    };
    if (LG < 10) younger_first<1>();
    for (int p = p0; p < npass;) {
        bool scaled = prep();
        while (!scaled) {
            iter(Mode<true, false>{}, p);
            p += pstep;
            if (p >= npass) break;
            scaled = prep();
        }
        if (p >= npass) break;
        iter(Mode<true, true>{}, p);
        p += pstep;
    }

    for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
    if (lane == 0) dred[wave] = dsum;
    if (NP > 1 && NWV > 1) __syncthreads();              // (the exchange buffers become the reduction's)
    int etop = acc_reduce<NT, 1, NWV, BF>(acc, eref, red, erefs, wave, lane);
    const size_t ho = (size_t)split * H + h;
    if (wave != 0) return;
    if (lane == 0 && q.dD) {
        float t = dred[0];
        for (int w = 1; w < NWV; ++w) t += dred[w];
        q.dD[ho] = t;
    }
    if (!q.dk) return;
    const int ea = acc_exponent(acc_peak<NT>(acc));
    etop += ea;
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) { acc[k][r].x = ldexpf(acc[k][r].x, -ea); acc[k][r].y = ldexpf(acc[k][r].y, -ea); }
    H8U m[2];
    f4 v[NP][2];
#pragma unroll
    for (int c = 0; c < NP; ++c) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (C::TC == 1) m[k].w[r] = k == 0 ? pack_h2(acc[0][r].x, acc[0][r].y) : 0u;
                else m[k].w[r] = pack_h2(acc[2 * c + k % NS][r].y, acc[2 * c + k % NS][r].x);
            }
        if constexpr (C::TC > 1) phase2_inv<LG>(xd + xpo + 2 * c * C::COLS, K, m);
    }
    if constexpr (C::TC > 1) wave_lds_fence();
#pragma unroll
    for (int c = 0; c < NP; ++c) {
        if constexpr (C::TC > 1) phase3_read<LG>(xd + xwo + 2 * c * C::P, m);
        phase3<LG>(m, K, v[c], c);
    }
    const uint32_t kb = (pad ? C::N / 2 : C::N) * 4u;
    const rsrc_t d = make_rsrc(reinterpret_cast<const char*>(q.dk) + ho * kb, kb);
    word_offsets<LG>(off, 0, lane, pad, NOWHERE);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int at = (int)((off[r] & NOWHERE) ? NOWHERE : 2u * off[r]);
        auto bits = [&](int c, int k) { return __float_as_uint(ldexpf(v[c][k][r] * q.dkscale, etop)); };
        if constexpr (NP == 2) {
            const u4v o = {bits(0, 0), bits(0, 1), bits(1, 0), bits(1, 1)};
            __builtin_amdgcn_raw_buffer_store_b128(o, d, at, 0, 0);
        } else {
            const u2v o = {bits(0, 0), bits(0, 1)};
            __builtin_amdgcn_raw_buffer_store_b64(o, d, at, 0, 0);
        }
    }
}

// ---- launches ----------------------------------------------------------------------------------------------------------
// Workgroups of kernel `f` the device holds at once.
template <class F>
hipError_t resident(F f, int threads, size_t lds, int& cache)
{
    if (cache) return hipSuccess;
    int nb = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, threads, lds);
    if (e != hipSuccess) return e;
    cache = (nb < 1 ? 1 : nb) * compute_units();
    return hipSuccess;
}

// Workgroups of a persistent grid: with as many as the device holds, a few more rows than those leave most of them idle for the
// last turn; as many turns with even shares keep fewer waves, and their constants and memory requests, in each other's way
// (kernel time, fp16: 8192 passes on 7168 waves, B=64, H=256, N=256 8.9 -> 6.8 us; B=2, H=768, N=2048 10.6 -> 9.2; B=3,
// H=2048, N=512 8.2 -> 7.0).
int even_grid(int want, int cap)
{
    const int turns = (want + cap - 1) / cap;
    return (want + turns - 1) / turns;
}

template <int LG, class IO, bool CONJ, bool GATE>
hipError_t rconv_run(const void* in, const float2* kspec, void* out, const Problem& pr, const uint4* tab, hipStream_t st)
{
    using T = typename IO::T;
    using C = RC<LG>;
    static int cap = 0;
    hipError_t e;
    if constexpr (LG > 10) {
        const int items = (int)(pr.B * pr.H);
        e = resident(rconv_kernel<LG, IO, CONJ, GATE>, C::NWR * 64, 0, cap);
        if (e != hipSuccess) return e;
        const int nb = even_grid(items, cap);
        hipLaunchKernelGGL((rconv_kernel<LG, IO, CONJ, GATE>), dim3(nb), dim3(C::NWR * 64), 0, st, (const T*)in, kspec, (T*)out,
                           (const T*)pr.gate, (int)pr.B, (int)pr.H, items, pr.pad, tab);
    } else {
        const int bpi = (int)((pr.B + C::RPI - 1) / C::RPI), items = bpi * (int)pr.H;
        e = resident(rconv1_kernel<LG, IO, CONJ, GATE>, 256, 0, cap);
        if (e != hipSuccess) return e;
        // With the gate rows of 256 samples in bf16 would be held by seven workgroups of a compute unit; five, in longer runs, are
        // faster (us, seven and five: B=40, H=1024 14.1 and 12.6, B=64, H=512 11.1 and 10.4, B=24, H=512 5.9 and 5.45, B=16, H=768
        // 5.8 and 5.5; B=48, H=700 11.1 and 11.8, B=64, H=768 15.85 and 16.2).
        if (LG == 8 && GATE && IsBf<IO>::v) cap = cap < 5 * compute_units() ? cap : 5 * compute_units();
        const int nb = even_grid((items + 3) / 4, cap);
        hipLaunchKernelGGL((rconv1_kernel<LG, IO, CONJ, GATE>), dim3(nb), dim3(256), 0, st, (const T*)in, kspec, (T*)out,
                           (const T*)pr.gate, (int)pr.B, (int)pr.H, bpi, items, pr.pad, tab);
    }
    return hipGetLastError();
}
template <int LG, class IO>
hipError_t rconv_go(const void* in, const float2* kspec, void* out, bool conj, const Problem& pr, const uint4* tab, hipStream_t st)
{
    if (pr.gate) return conj ? hipErrorInvalidValue : rconv_run<LG, IO, false, true>(in, kspec, out, pr, tab, st);
    return conj ? rconv_run<LG, IO, true, false>(in, kspec, out, pr, tab, st)
                : rconv_run<LG, IO, false, false>(in, kspec, out, pr, tab, st);
}
template <int LG>
hipError_t rkspec_go(const float* k, const float* D, float2* kspec, int64_t H, float kscale, uint32_t pad, const uint4* tab, hipStream_t st)
{
    hipLaunchKernelGGL((rkspec_kernel<LG>), dim3((unsigned)H), dim3(RC<LG>::NWR * 64), 0, st, k, D, kspec, (int)H, kscale, pad, tab);
    return hipGetLastError();
}
template <int LG, class IO, bool DU, bool GATE, int NWV>
hipError_t rbwd1_run(const BwdArgs<typename IO::T>& a, hipStream_t st)
{
    hipLaunchKernelGGL((rbwd1_kernel<LG, IO, DU, GATE, NWV>), dim3((unsigned)(a.H * a.nsplit)), dim3(64 * NWV), 0, st, a);
    return hipGetLastError();
}
template <int LG, class IO, bool DU, bool GATE, bool WIDE>
hipError_t rbwd_launch(const BwdArgs<typename IO::T>& a, hipStream_t st)
{
    using Q = BwdCfg<LG, GATE, WIDE>;
    const auto kern = rbwd_kernel<LG, IO, DU, GATE, WIDE>;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)Q::lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.H * a.nsplit)), dim3(Q::NWV * 64), Q::lds, st, a);
    return hipGetLastError();
}
// Whether the workgroups of a backward call (N = 2048, gated N = 1024) take twice the groups of waves: where each has a compute
// unit to itself, with one wave per SIMD, which issues an instruction every 8 cycles (two: every 5.6).  Whole steps, bf16: N=2048
// B=8, H=200 29.3 -> 28.0 us, B=7, H=193 gated 38.7 -> 37.2; N=1024 gated B=16, H=256 36.7 -> 34.2.  One row a group gives it
// nothing to do but the longer ends (N=2048 B=2, H=200 21.7 -> 22.1).
bool wide_bwd(int64_t workgroups, int64_t rows, int groups) { return workgroups <= compute_units() && rows > 2 * groups; }
template <int LG, class IO, bool DU, bool GATE>
hipError_t rbwd_run(const BwdArgs<typename IO::T>& a, hipStream_t st)
{
    if constexpr (LG < 10) {
        return rbwd1_run<LG, IO, DU, GATE, 4>(a, st);
    } else if constexpr (LG == 10 && !GATE) {
        // no more waves than the share has rows (B=1, H=768: four of them, three idle, 11.6 us, one 8.1)
        const int each = (a.B + a.nsplit - 1) / a.nsplit;
        if (each == 1) return rbwd1_run<LG, IO, DU, GATE, 1>(a, st);
        if (each == 2) return rbwd1_run<LG, IO, DU, GATE, 2>(a, st);
        return rbwd1_run<LG, IO, DU, GATE, 4>(a, st);
    } else {
        using Q = BwdCfg<LG, GATE, false>;
        if constexpr (Q::can_widen)
            if (wide_bwd(a.H * a.nsplit, (a.B + a.nsplit - 1) / a.nsplit, Q::NGRP)) return rbwd_launch<LG, IO, DU, GATE, true>(a, st);
        return rbwd_launch<LG, IO, DU, GATE, false>(a, st);
    }
}
template <int LG, class IO>
hipError_t rbwd_go(const BwdArgs<typename IO::T>& a, hipStream_t st)
{
    if (a.g) return a.du && a.dg ? rbwd_run<LG, IO, true, true>(a, st) : hipErrorInvalidValue;
    return a.du ? rbwd_run<LG, IO, true, false>(a, st) : rbwd_run<LG, IO, false, false>(a, st);
}

#define ROWS_SWITCH(lg, FN, ...)                                  \
    switch (lg) {                                                 \
        case 8: return FN(8) __VA_ARGS__;                         \
        case 9: return FN(9) __VA_ARGS__;                         \
        case 10: return FN(10) __VA_ARGS__;                       \
        case 11: return FN(11) __VA_ARGS__;                       \
        case 12: return FN(12) __VA_ARGS__;                       \
        default: return hipErrorInvalidValue;                     \
    }

}  // namespace

hipError_t rows_fill_tables(const void** tab_out, hipStream_t st)
{
    uint4* p = nullptr;
    hipError_t e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(g_rows_tab));
    if (e != hipSuccess) return e;
    for (int lg = ROWS_MIN; lg <= ROWS_MAX; ++lg)
        hipLaunchKernelGGL(fill_rows_tab_kernel, dim3(tab_units(lg)), dim3(64), 0, st, p + (size_t)tab_offset(lg) * 64, lg);
    *tab_out = p;
    return hipGetLastError();
}

// Shares of a head's rows in the backward kernel: about as many workgroups as the device holds at once when heads are few
// (half of it at N = 1024 ungated, a row a wave), and at least two rows (passes of two rows at N = 256) for every group of
// waves.  More than one share costs a second launch, about 3.5 us, so where the heads alone fill a quarter of the device a
// share has at least eight rows a group (fp16, kernel time of one share against two: B=16, H=256, N=512 8.4 and 10.5 us;
// B=3, H=256, N=2048 10.1 and 13.2); gated rows of 4096 samples are worth it (B=4, H=128 bf16 21.5 and 19.8).  N = 1024
// ungated, few heads: the root of the rows, where the rows a wave is spared and the partial results that come with them
// balance (fp16: B=16, H=16 2 shares 10.4 us, 4 9.3; B=64, H=32 4 shares 14.3, 8 12.9, 16 17.3).
// N >= 2048 with more than half as many heads as the device has compute units, up to twice as many: what a compute unit has to
// do depends on how H * s workgroups fall on the 256 of them, so the estimate below picks s.  A share's rows and the ends of
// its pipeline count once per workgroup on the fullest unit; two resident workgroups (N = 2048) take 1.32 times one's time; the
// shares' sum is a launch and its bytes.  bf16, a call before and now: N=2048 H=130 B=16 26.7 -> 23.1 us, gated 33.6 -> 27.8 (3
// shares, not 2); H=340 B=32 65 -> 58, gated 90 -> 75 (3, not 1); N=4096 H=340 B=32 135 -> 123, gated 179 -> 159 (2, not 1).
// Its sum does not depend on the gate and grows with s, so a gated call never has fewer shares than an ungated one.
static bool many_heads(int64_t H, int lg) { return lg >= 11 && H > 128 && H <= 512; }
static float many_load(int64_t H, int lg, int s)      // of the fullest unit, in workgroups that run alone
{
    const int on_cu = (int)((H * s + 255) / 256);
    return lg == 11 ? 1.32f * (on_cu / 2) + (on_cu & 1) : (float)on_cu;
}
static int rows_bwd_nsplit_many(int64_t B, int64_t H, int lg, bool gated)
{
    const float row_us = lg == 11 ? (gated ? 1.7f : 1.33f) : (gated ? 2.3f : 1.65f);
    const float ends = lg == 11 ? 4.f : 5.f;
    int best = 1;
    float least = 0.f;
    for (int s = 1; s <= 3 && s <= B; ++s) {
        const float sum = s > 1 ? 3.5f + (float)s * (float)H * (float)(8 << lg) * 2e-7f : 0.f;
        const float us = row_us * many_load(H, lg, s) * ((float)((B + s - 1) / s) + ends) + sum;
        if (s == 1 || us < least) { best = s; least = us; }
    }
    return best;
}
// N = 2048: two shares that would meet on one compute unit are the two groups of waves of one workgroup instead (wide_bwd), without
// a launch to add them up.  Each group takes its sum through an inverse transform (fp16 operands) of its own and the two rows of dk
// are added in fp32, as two shares' are: the same dk and dD to the bit (one inverse of both sums moved dk by 6e-4, the size of that
// rounding, neither nearer to nor farther from the exact one: 8.4e-4) in the same time, since the second group has nothing else to do.
// Steps, two workgroups and one: B=24, H=256 bf16 62.8 -> 56.8 us, gated 74.4 -> 67.4; 32 x 32 images, B=64, H=200 fp16 94.9 -> 90.3.
static bool rows_bwd_paired(int64_t B, int64_t H, int lg, bool gated)
{
    return lg == 11 && many_heads(H, lg) && H <= compute_units() && rows_bwd_nsplit_many(B, H, lg, gated) == 2;
}
int rows_bwd_nsplit(int64_t B, int64_t H, int lg, bool gated)
{
    if (many_heads(H, lg)) return rows_bwd_paired(B, H, lg, gated) ? 1 : rows_bwd_nsplit_many(B, H, lg, gated);
    const bool wave_rows = lg == 10 && !gated;
    const int ngrp = lg >= 11 ? 1 : lg == 10 && gated ? 2 : 4;
    const int64_t units = lg == 8 ? (B + 1) / 2 : B;
    int64_t s = (lg == 12 || wave_rows ? 256 : 512) / H;
    const int64_t least = ngrp * (s < 4 && !(gated && lg == 12) ? 8 : 2);
    int64_t most = (units + least - 1) / least;
    if (wave_rows && s >= 4)
        for (most = units / 4; most > 1 && most * most > units;) --most;
    if (s > most) s = most;
    if (s > 64) s = 64;
    return s < 1 ? 1 : (int)s;
}
// The other rule grows with B; of the estimate's choices s = 1 is faster at any B than an s that loads the fullest unit s times.
int rows_bwd_room(int64_t B, int64_t H, int lg)
{
    if (!many_heads(H, lg)) return rows_bwd_nsplit(B, H, lg, true);
    int room = 1;
    for (int s = 2; s <= 3 && s <= B; ++s)
        if (many_load(H, lg, s) < s * many_load(H, lg, 1)) room = s;
    return room;
}
float rows_chain_scale(int lg)
{
    switch (lg) {
        case 8: return 1.0f / (1 << RC<8>::SHIFT);
        case 9: return 1.0f / (1 << RC<9>::SHIFT);
        case 10: return 1.0f / (1 << RC<10>::SHIFT);
        case 11: return 1.0f / (1 << RC<11>::SHIFT);
        default: return 1.0f / (1 << RC<12>::SHIFT);
    }
}

hipError_t rows_kspec(const float* k, const float* D, float2* kspec, int64_t H, const Plan& pl, uint32_t pad, const Tables& tb,
                      hipStream_t st)
{
    const uint4* tab = (const uint4*)tb.rtab;
#define RF(L) rkspec_go<L>
    ROWS_SWITCH(pl.order.wave_lg, RF, (k, D, kspec, H, pl.kscale, pad, tab, st))
#undef RF
}
template <class IO>
static hipError_t conv_io(const void* in, const float2* kspec, void* out, bool conj, const Problem& pr, int lg, const uint4* tab,
                          hipStream_t st)
{
#define RF(L) rconv_go<L, IO>
    ROWS_SWITCH(lg, RF, (in, kspec, out, conj, pr, tab, st))
#undef RF
}
hipError_t rows_conv(const void* in, const float2* kspec, void* out, bool conj, const Problem& pr, const Plan& pl,
                     const Tables& tb, hipStream_t st)
{
    const uint4* tab = (const uint4*)tb.rtab;
    if (pr.io == LONGCONV_F16) return conv_io<IoF16>(in, kspec, out, conj, pr, pl.order.wave_lg, tab, st);
    if (pr.io == LONGCONV_BF16) return conv_io<IoBF16>(in, kspec, out, conj, pr, pl.order.wave_lg, tab, st);
    return hipErrorInvalidValue;
}
template <class IO>
static hipError_t bwd_io(const void* dy, const void* u, const float2* kspec, void* du, float* dk, float* dD, void* dg, int nsplit,
                         const Problem& pr, const Plan& pl, const uint4* tab, hipStream_t st)
{
    using T = typename IO::T;
    const BwdArgs<T> a = {(const T*)dy, (const T*)u, (const T*)pr.gate, kspec, (T*)du, (T*)dg, dk, dD, (int)pr.B, (int)pr.H, nsplit,
                          rows_bwd_paired(pr.B, pr.H, pl.order.wave_lg, pr.gate != nullptr) ? 1 : 0, pl.dkscale, pr.pad, tab};
#define RF(L) rbwd_go<L, IO>
    ROWS_SWITCH(pl.order.wave_lg, RF, (a, st))
#undef RF
}
hipError_t rows_bwd(const void* dy, const void* u, const float2* kspec, void* du, float* dk, float* dD, void* dg, int nsplit,
                    const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
    const uint4* tab = (const uint4*)tb.rtab;
    if (pr.io == LONGCONV_F16) return bwd_io<IoF16>(dy, u, kspec, du, dk, dD, dg, nsplit, pr, pl, tab, st);
    if (pr.io == LONGCONV_BF16) return bwd_io<IoBF16>(dy, u, kspec, du, dk, dD, dg, nsplit, pr, pl, tab, st);
    return hipErrorInvalidValue;
}

}  // namespace lc
