// Matrix-core engine for rows of N = 65536 and 131072 samples, and for dk of rows of 32768: each row's N-point twisted transform
// (engine_rows.hip) as R = N / L chunks of L = 16384 points.  With f = k_1 + R f', n = n_2 + L n_1, W = exp(-2 pi i / 4N):
//     X[f] = sum_(n_2) w_L^(n_2 f') W^(n_2 (4 k_1 + 1)) s[n_2],     s[n_2] = sum_(n_1) x[n_2 + L n_1] exp(-2 pi i n_1 (4 k_1 + 1) / 4R).
// A workgroup owns chunk k_1 of a head and walks (a share of) its rows.  It forms s in fp32 while it stages the row and takes it
// through the phases of long_rows.hpp, whose matrices carry the chunk's twist W^(n_2 (4 k_1 + 1)) as they carry the row's at
// N = 16384.  The inverse leaves z[n_2], complex, untwisted, as planes in the caller's workspace, and a last kernel forms
//     y[n_2 + L n_1] = Re sum_(k_1) exp(2 pi i n_1 (4 k_1 + 1) / 4R) z_(k_1)[n_2].
// The R workgroups that read one row follow each other on one XCD, so memory sees the row once.
#include <type_traits>

#include "long_rows.hpp"

namespace lc {
namespace {
using namespace longrows;

using L = LR<14>;
constexpr int TE = L::TE, PC = L::PC, NA = L::KB * TE;

// Constants of chunk k_1, units of 16 bytes per lane: per tile the matrix over d_a (planar, one operand: see phase1_chunk), over
// d_b for each d_e (forward, inverse), the inverse over k_a without the tile's factor (real, imaginary part), and these factors.
// All else is what rows of 16384 samples use.
constexpr int C_A = 0, C_B = L::TC, C_AI = C_B + 4 * TE, C_S = C_AI + 2, C_UNITS = C_S + L::TC / 16;
static __device__ uint4 g_chunk_tab[14 * C_UNITS * 64];             // R = 2, 4, 8
template <int R>
__host__ __device__ constexpr int chunk_tab() { return (R - 2) * C_UNITS * 64; }

// s is rounded to fp16 divided by this, and the matrices over d_a give it back.  R equal samples N / R apart, all that there is of a
// row, then stay finite up to 38370, 43470 and 23490 (R = 2, 4, 8); undivided R = 4 and 8 ended at 21730 and 11740.  More would
// cost rows close to fp16's smallest normal number: with rows of 1e-4 (and kernels of 300) the error of y at N = 131072 is
// 7.6e-4 either way, and 8.9e-4 divided by R.
__host__ __device__ constexpr float staged_down(int R) { return R > 2 ? 2.f : 1.f; }
// N points where the spectrum's scale has 1/2N: the factor of two that is missing stands in the inverse transform's last block,
// over k_a.  At R = 8 it stands in the first, over d_e: the products with the spectrum are a sixteenth of the rows there, and
// every rounding behind them meets fp16's smallest normal number the sooner (rows of 1e-4, error of y: 3.1e-3 with the factor in
// the last block, 2.1e-3 in the first).  At R = 4 there is nothing to gain, and a row of 16 equal outputs 1024 apart would leave
// fp16 in front of the last block from 16400 on, not 32800.
__host__ __device__ constexpr float inverse_up(int R) { return R == 8 ? 1.f : 2.f; }

template <int R>
__global__ void fill_chunk_tab_kernel(uint4* tab)
{
    const int unit = blockIdx.x, k1 = blockIdx.y, lane = threadIdx.x, o = lane & 15, g = lane >> 4;
    const double phi = (4.0 * k1 + 1.0) / (4.0 * R * L::N);          // the twist of n_2, in turns
    union { _Float16 h[8]; uint4 u; } v;
    double re, im;
    const auto w = [&](double t, double sc) {
        double s, c;
        sincospi(-2.0 * (t - floor(t)), &s, &c);
        re = c * sc;
        im = s * sc;
    };
    const auto a = [&](int ka, int da, int t) { w(da * ka / 16.0 + da * 16 * L::TC * phi + t * ((double)ka / L::N + phi), 0.25); };
    const auto b = [&](int kb, int db, int de) { w(db * kb / 16.0 + db * L::TC * phi + (double)(de * kb) / (256 * TE), 0.25); };
    const auto put = [&](int x, int part, bool conj) {
        const double i2 = conj ? -im : im;
        v.h[x] = (_Float16)(part ? i2 : re);
        v.h[4 + x] = (_Float16)(part ? re : -i2);
    };
    for (int x = 0; x < 4; ++x) {
        const int i = 4 * g + x;
        if (unit < C_B) {
            a(o, i, unit);
            v.h[x] = (_Float16)(re * staged_down(R));
            v.h[4 + x] = (_Float16)(im * staged_down(R));
        } else if (unit < C_AI) {
            const int m = unit - C_B, de = (m % (2 * TE)) >> 1;
            const bool inv = m >= 2 * TE;
            if (inv) b(i, o, de);
            else b(o, i, de);
            put(x, m & 1, inv);
        } else if (unit < C_S) {
            a(i, o, 0);
            re *= inverse_up(R);
            im *= inverse_up(R);
            put(x, unit - C_AI, true);
        } else {
            const int e = (unit - C_S) * 64 + lane, t = e >> 2;
            w(t * ((double)(4 * (e & 3) + x) / L::N + phi), 1.0);
            v.h[x] = (_Float16)re;
            v.h[4 + x] = (_Float16)im;
        }
    }
    tab[chunk_tab<R>() + ((size_t)k1 * C_UNITS + unit) * 64 + lane] = v.u;
}

// a wave's constants; the matrices of its last NAL tiles wait in LDS
template <bool INV, int NAL>
struct CK {
    h8 A[8 - NAL], AI[2];
    uint4* al;
    Cx C[L::KB], CI[INV ? L::KB : 1];
    h4 cr, ci;
    __device__ __forceinline__ h8 a(int kt) const
    {
        if (kt < 8 - NAL) return A[kt < 8 - NAL ? kt : 0];
        H8P x;
        x.w = al[(kt - (8 - NAL)) * 64];
        return x.v;
    }
    __device__ __forceinline__ void load(const uint4* __restrict__ ltab, const uint4* __restrict__ ctab, int wave, int lane, uint4* lds)
    {
        const uint4 *p = ltab + (size_t)tab_offset<14>() * 64 + lane, *q = ctab + lane;
        H8P x;
        al = lds + wave * NAL * 64 + lane;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            x.w = q[(C_A + 8 * wave + k) * 64];
            if (k < 8 - NAL) A[k < 8 - NAL ? k : 0] = x.v;
            else al[(k - (8 - NAL)) * 64] = x.w;
        }
        const auto unit = [&](int u) { x.w = p[(size_t)u * 64]; return x.v; };
        if (INV) {
            x.w = q[C_AI * 64];
            AI[0] = x.v;
            x.w = q[(C_AI + 1) * 64];
            AI[1] = x.v;
        }
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            const int kb = wave * L::KB + j;
            C[j].re = unit(L::U_C + 2 * kb);
            C[j].im = unit(L::U_C + 2 * kb + 1);
            if (INV) {
                CI[INV ? j : 0].re = unit(L::U_CI + 2 * kb);
                CI[INV ? j : 0].im = unit(L::U_CI + 2 * kb + 1);
            }
        }
        unit(L::U_TW);
        cr = x.p[0];
        ci = x.p[1];
    }
};
constexpr int SHARED = L::N_LDS * 64 + L::TC * 4;       // matrices over d_b and d_e, the tiles' factors
template <int R>
__device__ __forceinline__ void load_chunk_shared(uint4* sm, const uint4* __restrict__ ltab, const uint4* __restrict__ ctab, int tid)
{
    const uint4* p = ltab + (size_t)(tab_offset<14>() + L::U_LDS) * 64;
    for (int i = tid; i < L::N_LDS * 64; i += L::NT) {
        H8P x;
        x.w = i < 4 * TE * 64 ? ctab[C_B * 64 + i] : p[i];
        if (inverse_up(R) != 2.f && i >= L::U_EI * 64) x.v *= (_Float16)(2.f / inverse_up(R));
        sm[i] = x.w;
    }
    for (int i = tid; i < L::TC * 4; i += L::NT) sm[L::N_LDS * 64 + i] = ctab[C_S * 64 + i];
}
constexpr size_t chunk_lds(int nal) { return sizeof(_Float16) * L::EX + 16 * SHARED + 1024 * nal * L::NW; }

// workgroup -> chunk k_1 and a run of consecutive items of a list, the same runs for all chunks; the R workgroups of a run follow
// each other on one XCD.  A workgroup keeps its chunk, and with it its constants, from head to head (B=1, H=128, N=65536 forward:
// 41.6 us with a workgroup per head and chunk, 34.6 in runs of two heads.)
template <int R>
struct Run {
    int k1, i0, i1;
    __device__ __forceinline__ explicit Run(int items)
    {
        const unsigned G = gridDim.x;
        const unsigned v = (G & 7u) ? blockIdx.x : (blockIdx.x & 7u) * (G >> 3) + (blockIdx.x >> 3);
        const int s = (int)(v / R), n = (int)(G / R), each = items / n, more = items - each * n;
        k1 = (int)(v % R);
        i0 = s * each + min(s, more);
        i1 = i0 + each + (s < more);
    }
};
// exp(-2 pi i n (4 k1 + 1) / 4R) s / staged_down
template <int R>
__device__ __forceinline__ void outer_factors(float2 (&f)[R], const float2* __restrict__ tw, int k1, float s)
{
    constexpr int lg = R == 2 ? 3 : R == 4 ? 4 : 5;  // 4R
#pragma unroll
    for (int n = 0; n < R; ++n) {
        const float2 w = tw_full(tw, (uint32_t)((n * (4 * k1 + 1)) & (4 * R - 1)) << (TW_LOG2 - lg));
        f[n] = make_float2(w.x * s * (1.f / staged_down(R)), w.y * s * (1.f / staged_down(R)));
    }
}
// s of eight samples (words of two fp16 or bf16 numbers), as planes
template <class IO, int R>
__device__ __forceinline__ void combine(const u4w (&v)[R], const float2 (&f)[R], u4w& re, u4w& im)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float a[2], b[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            a[e] = io_half<IO>(v[0][q], e) * f[0].x;
            b[e] = 0.f;
#pragma unroll
            for (int n = 1; n < R; ++n) {
                const float x = io_half<IO>(v[n][q], e);
                a[e] = __builtin_fmaf(x, f[n].x, a[e]);
                b[e] = n == 1 ? x * f[n].y : __builtin_fmaf(x, f[n].y, b[e]);
            }
        }
        re[q] = mu::pack_h2(a[0], a[1]);
        im[q] = mu::pack_h2(b[0], b[1]);
    }
}
// A row on its way, in groups of G of a thread's pieces of all its parts; registers for EARLY groups, asked for ahead
template <class IO, int R, int G, int EARLY>
struct RowIn {
    static constexpr int NG = PC / G;
    u4w v[EARLY][G][R];
    __device__ __forceinline__ void ask(int slot, int group, const typename IO::T* row, int tid)
    {
        const u4w* p = reinterpret_cast<const u4w*>(row);
#pragma unroll
        for (int i = 0; i < G; ++i)
#pragma unroll
            for (int n = 0; n < R; ++n) v[slot][i][n] = uniform(p, (size_t)n * (L::N / 8) + (group * G + i) * L::NT)[(unsigned)tid];
    }
    __device__ __forceinline__ void put(int slot, int group, _Float16* mine, const float2 (&f)[R])
    {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            u4w re, im;
            combine<IO, R>(v[slot][i], f, re, im);
            *reinterpret_cast<u4w*>(mine + (group * G + i) * L::STEP) = re;
            *reinterpret_cast<u4w*>(mine + L::N + (group * G + i) * L::STEP) = im;
        }
    }
    __device__ __forceinline__ void ask_first(const typename IO::T* row, int tid)
    {
#pragma unroll
        for (int g = 0; g < EARLY; ++g) ask(g, g, row, tid);
    }
    // the row's s into the exchange buffer, planes one behind the other; its first groups are on their way
    __device__ __forceinline__ void stage(_Float16* mine, const typename IO::T* row, const float2 (&f)[R], int tid)
    {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            put(g % EARLY, g, mine, f);
            if (g + EARLY < NG) ask(g % EARLY, g + EARLY, row, tid);
        }
    }
};
// Phase 1 of all the wave's tiles from the staged planes, which lie where its results go: everything is read first.  The matrix is
// one operand (real parts, imaginary parts); s goes in twice, as (re, -im) and (im, re).
template <bool ONCE, class KT>
__device__ __forceinline__ void phase1_chunk(const KT& K, const uint4* mats, const Places<L>& P, _Float16* ex)
{
    u4w wr[4], wi[4];
    read_pieces<L>(wr, ex + P.raw);
    read_pieces<L>(wi, ex + L::N + P.raw);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        h4 re[2], im[2];
        pair_ops<IoF16>({wr[0][p], wr[1][p], wr[2][p], wr[3][p]}, 0, re);
        pair_ops<IoF16>({wi[0][p], wi[1][p], wi[2][p], wi[3][p]}, 0, im);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int kt = 2 * p + k;
            const h8 A = K.a(kt);
            H8P d1, d2;
            d1.p[0] = re[k];
            d1.p[1] = -im[k];
            d2.p[0] = im[k];
            d2.p[1] = re[k];
            const f4 yr = mm(d1.v, A), yi = mm(d2.v, A);
            const H8P x = ONCE ? cmul_once<false>(yr, yi, K.cr, K.ci) : cmul_planes<false>(yr, yi, K.cr, K.ci);
            const Cx M = shared_mat(mats, L::U_B + 2 * (kt % TE));
            const H8P z = planes(mm(x.v, M.re), mm(x.v, M.im));
            _Float16* dst = ex + P.own[kt / TE] + P.in_group(kt);
            wr4(dst, z.p[0]);
            wr4(dst + 256, z.p[1]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}
// Phase 3 of all the wave's tiles and the planes of z back where the row was staged (words of fp16 numbers, times 2^-e)
template <bool ONCE, class KT>
__device__ __forceinline__ void phase3_chunk(const KT& K, const uint4* mats, const uint4* factors, const Places<L>& P, _Float16* ex)
{
    u4w zr[4], zi[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        f4 vr[2], vi[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int kt = 2 * p + k;
            const _Float16* src = ex + P.own_tr[kt / TE] + P.in_group(kt);
            H8P x, f;
            x.p[0] = tr_read(src);
            x.p[1] = tr_read(src + 256);
            f.w = factors[4 * kt];
            const Cx M = shared_mat(mats, L::U_BI + 2 * (kt % TE));
            const f4 yr = mm(x.v, M.re), yi = mm(x.v, M.im);
            H8P m;
            if constexpr (ONCE) {
                f4 wr, wi;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float2 w = cmul(make_float2((float)K.cr[r], (float)K.ci[r]), make_float2((float)f.p[0][r], (float)f.p[1][r]));
                    wr[r] = w.x;
                    wi[r] = w.y;
                }
                m = cmul_once<true>(yr, yi, wr, wi);
            } else {
                const h4 wr = __builtin_elementwise_fma(-f.p[1], K.ci, f.p[0] * K.cr);
                const h4 wi = __builtin_elementwise_fma(f.p[0], K.ci, f.p[1] * K.cr);
                m = cmul_planes<true>(yr, yi, wr, wi);
            }
            vr[k] = mm(K.AI[0], m.v);
            vi[k] = mm(K.AI[1], m.v);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            zr[r][p] = mu::pack_h2(vr[0][r], vr[1][r]);
            zi[r][p] = mu::pack_h2(vi[0][r], vi[1][r]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    write_pieces<L>(zr, ex + P.raw);
    write_pieces<L>(zi, ex + L::N + P.raw);
    __syncthreads();
}
__device__ __forceinline__ void store_planes(_Float16* dst, const _Float16* mine, int tid)
{
    u4w* p = reinterpret_cast<u4w*>(dst);
#pragma unroll
    for (int i = 0; i < PC; ++i) {
        uniform(p, i * L::NT)[(unsigned)tid] = *reinterpret_cast<const u4w*>(mine + i * L::STEP);
        uniform(p, L::N / 8 + i * L::NT)[(unsigned)tid] = *reinterpret_cast<const u4w*>(mine + L::N + i * L::STEP);
    }
}

// -------------------------------------------------------------------------------------------------------------------
// Convolution (forward; CONJ: du) of a chunk of a run of rows: z planes of row b to ws[((h B + b) R + k_1) 2 L].  Bound by issue
// and by the row's way in: about 9 us a row and chunk against 6.7 for a row of 16384 samples.  B=8, H=128, N=65536 fp16, whole call:
// 257 us as two chunks of 32768 points with the first digit summed in fp16, 250 here, 215 with the next row asked for ahead.
// (Eight registers are spilled at R = 8.)
// -------------------------------------------------------------------------------------------------------------------
template <class IO, int R, bool CONJ>
__global__ void __launch_bounds__(L::NT) __attribute__((amdgpu_waves_per_eu(2)))
chunk_conv_kernel(const typename IO::T* __restrict__ in, const float2* __restrict__ kspec, _Float16* __restrict__ ws, int B, int H,
                  const float2* __restrict__ tw, const uint4* __restrict__ ltab, const uint4* __restrict__ chtab,
                  const uint32_t* __restrict__ rows_max)
{
    extern __shared__ uint4 lds4[];
    _Float16* ex = reinterpret_cast<_Float16*>(lds4);
    uint4* shared = reinterpret_cast<uint4*>(ex + L::EX);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4;
    const Run<R> me(B * H);
    int h = me.i0 / B, b = me.i0 - h * B;            // of the row in work
    const typename IO::T* row = in + row_off(b, h, H, (int64_t)R * L::N);
    RowIn<IO, R, 8 / R, 2> x;
    x.ask_first(row, tid);
    const uint4* ctab = chtab + chunk_tab<R>() + (size_t)me.k1 * C_UNITS * 64;
    float2 f[R];
    _Float16* mine = ex + piece_of<L>(tid);
    CK<true, 0> K;
    K.load(ltab, ctab, wave, lane, nullptr);
    load_chunk_shared<R>(shared, ltab, ctab, tid);
    const uint4 *mats = shared + lane, *factors = shared + L::N_LDS * 64 + 8 * wave * 4 + g;
    Places<L> P;
    P.make(wave, lane);
    H8P ks[NA];
    const auto load_head = [&]() __attribute__((always_inline)) {
        outer_factors<R>(f, tw, me.k1, ldexpf(1.f, rows_max ? -mu::row_exponent(rows_max[h]) : 0));
        const uint4* kp = reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(kspec) + ((size_t)h * 2 * R + me.k1) * L::N) +
                          (size_t)wave * NA * 64;
#pragma unroll
        for (int i = 0; i < NA; ++i) ks[i].w = kp[i * 64 + lane];
    };
    load_head();
    for (int t = me.i0; t < me.i1; ++t) {
        x.stage(mine, row, f, tid);
        __syncthreads();
        phase1_chunk<false>(K, mats, P, ex);
        const int hw = h, bw = b;
        const bool more = t + 1 < me.i1;
        if (++b == B) { b = 0; ++h; }
        if (more) row = in + row_off(b, h, H, (int64_t)R * L::N);
        if (more) x.ask(0, 0, row, tid);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            H8P v[TE];
            phase2_fwd<L>(ex + P.mid_tr[j], K, j, mats, [&](int m, const f4& yr, const f4& yi) __attribute__((always_inline)) {
                v[m] = cmul_planes<CONJ>(yr, yi, ks[j * TE + m].p[0], ks[j * TE + m].p[1]);
            });
            phase2_inv<L, false>(ex + P.mid[j], K, j, mats, v, v);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (more) x.ask(1, 1, row, tid);
        __syncthreads();
        if (more && b == 0) load_head();
        phase3_chunk<false>(K, mats, factors, P, ex);
        store_planes(ws + (((size_t)hw * B + bw) * R + me.k1) * 2 * L::N, mine, tid);
    }
}

// -------------------------------------------------------------------------------------------------------------------
// Backward pass of a chunk: U = transform of u, W = transform of dy, A += conj(U) W in fp32; du's z planes per row as above
// (ws_du may be null), at the end those of the inverse transform of A 2^-e to ws_A[(share H + h) R + k_1] with e behind them
// (exps), and the chunk's part of dD (piece n_1 = k_1 of the rows) to dD_part at the same index.  There are no
// registers to ask for the next row ahead: with 32 of them, spills made B=8, H=128, N=65536 430 us instead of 386 (as eight chunks
// per pair of rows for dk, and du by itself: 690).  As it is, 2 are spilled at R = 4 and 14 to 21 at R = 8.
// -------------------------------------------------------------------------------------------------------------------
template <class T>
struct CBwdArgs {
    const T* dy;
    const T* u;
    const float2* kspec;
    _Float16* ws_du;
    _Float16* ws_A;
    int* exps;
    float* dD_part;
    int B, H, nshare;
    const float2* tw;
    const uint4* ltab;
    const uint4* chtab;
    const uint32_t* max_u;
    const uint32_t* max_dy;
};
constexpr int CNAL = 7;
template <class IO, int R, bool DU>
__global__ void __launch_bounds__(L::NT) __attribute__((amdgpu_waves_per_eu(2)))
chunk_bwd_kernel(const CBwdArgs<typename IO::T> q)
{
    constexpr bool BF = IsBf<IO>::v;
    extern __shared__ uint4 lds4[];
    __shared__ float dred[L::NW];
    __shared__ uint32_t peaks[L::NW];
    _Float16* ex = reinterpret_cast<_Float16*>(lds4);
    uint4* shared = reinterpret_cast<uint4*>(ex + L::EX);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4;
    const int B = q.B, H = q.H;
    const Run<R> me(H * q.nshare);
    const size_t step = (size_t)q.nshare * H * R * L::N;
    const uint4* ctab = q.chtab + chunk_tab<R>() + (size_t)me.k1 * C_UNITS * 64;
    _Float16* mine = ex + piece_of<L>(tid);
    CK<true, CNAL> K;
    K.load(q.ltab, ctab, wave, lane, shared + SHARED);
    load_chunk_shared<R>(shared, q.ltab, ctab, tid);
    const uint4 *mats = shared + lane, *factors = shared + L::N_LDS * 64 + 8 * wave * 4 + g;
    Places<L> P;
    P.make(wave, lane);
    RowIn<IO, R, 8 / R, 1> x;
    for (int item = me.i0; item < me.i1; ++item) {
        const int h = item / q.nshare, share = item - h * q.nshare;
        float2 fu[R], fd[R];
        outer_factors<R>(fu, q.tw, me.k1, ldexpf(1.f, q.max_u ? -mu::row_exponent(q.max_u[h]) : 0));
        outer_factors<R>(fd, q.tw, me.k1, ldexpf(1.f, q.max_dy ? -mu::row_exponent(q.max_dy[h]) : 0));
        const typename IO::T *pu = q.u + row_off(share, h, H, (int64_t)R * L::N), *pd = q.dy + row_off(share, h, H, (int64_t)R * L::N);
        const uint32_t* kh = reinterpret_cast<const uint32_t*>(q.kspec) + ((size_t)h * 2 * R + me.k1) * L::N;
        const uint4* kp = DU ? reinterpret_cast<const uint4*>(kh) + (size_t)wave * NA * 64 : nullptr;
        float2 acc[NA][4];
#pragma unroll
        for (int k = 0; k < NA; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[k][j] = make_float2(0.f, 0.f);
        float dsum = 0.f;
        for (int b = share; b < B; b += q.nshare) {
            {
                RowIn<IO, R, 8 / R, 2> xu;                  // (the registers of U are free: N = 131072, H=64 90.5 -> 88.8 us)
                xu.ask_first(pu, tid);
                xu.stage(mine, pu, fu, tid);
            }
            __syncthreads();
            phase1_chunk<false>(K, mats, P, ex);
            __syncthreads();
            H8P U[NA];
#pragma unroll
            for (int j = 0; j < L::KB; ++j) {
                phase2_fwd<L>(ex + P.mid_tr[j], K, j, mats, [&](int m, const f4& yr, const f4& yi) __attribute__((always_inline)) {
                    U[j * TE + m] = planes(yr, yi);
                });
                __builtin_amdgcn_sched_barrier(0);
            }
            if (q.dD_part) {
                const u4w *a = reinterpret_cast<const u4w*>(pu + me.k1 * L::N), *d = reinterpret_cast<const u4w*>(pd + me.k1 * L::N);
#pragma unroll
                for (int i = 0; i < PC; ++i) {
                    const u4w va = uniform(a, i * L::NT)[(unsigned)tid], vd = uniform(d, i * L::NT)[(unsigned)tid];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        union { uint32_t u; mu::h2 h; mu::bf2 b; } x, y;
                        x.u = va[r];
                        y.u = vd[r];
                        dsum = BF ? __builtin_amdgcn_fdot2_f32_bf16(x.b, y.b, dsum, false) : __builtin_amdgcn_fdot2(x.h, y.h, dsum, false);
                    }
                }
            }
            __syncthreads();
            x.ask_first(pd, tid);
            x.stage(mine, pd, fd, tid);
            __syncthreads();
            phase1_chunk<false>(K, mats, P, ex);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < L::KB; ++j) {
                H8P v[TE];
                if (DU) {
#pragma unroll
                    for (int m = 0; m < TE; ++m) v[m].w = uniform(kp, (j * TE + m) * 64)[(unsigned)lane];
                }
                phase2_fwd<L>(ex + P.mid_tr[j], K, j, mats, [&](int m, const f4& yr, const f4& yi) __attribute__((always_inline)) {
                    const H8P& x = U[j * TE + m];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float ur = (float)x.p[0][r], ui = (float)x.p[1][r];
                        float2& s = acc[j * TE + m][r];
                        s.x = __builtin_fmaf(ui, yi[r], __builtin_fmaf(ur, yr[r], s.x));
                        s.y = __builtin_fmaf(-ui, yr[r], __builtin_fmaf(ur, yi[r], s.y));
                    }
                    if (DU) v[m] = cmul_planes<true>(yr, yi, v[m].p[0], v[m].p[1]);
                });
                if (DU) phase2_inv<L, false>(ex + P.mid[j], K, j, mats, v, v);
                // the sums read MFMA results: not to be moved behind a branch
#pragma unroll
                for (int k = j * TE; k < (j + 1) * TE; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) asm volatile("" : "+v"(acc[k][r].x), "+v"(acc[k][r].y));
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();
            pu += step;
            pd += step;
            if (DU) {
                phase3_chunk<false>(K, mats, factors, P, ex);
                store_planes(q.ws_du + (((size_t)h * B + b) * R + me.k1) * 2 * L::N, mine, tid);
            }
        }
        const size_t at = ((size_t)share * H + h) * R + me.k1;
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
        const uint32_t peak = mu::acc_peak<NA>(acc);
        if (lane == 0) { dred[wave] = dsum; peaks[wave] = peak; }
        __syncthreads();
        if (tid == 0 && q.dD_part) {
            float s = 0.f;
            for (int w = 0; w < L::NW; ++w) s += dred[w];
            q.dD_part[at] = s;
        }
        if (!q.ws_A) continue;
        uint32_t m = peaks[0];
#pragma unroll
        for (int w = 1; w < L::NW; ++w) m = max(m, peaks[w]);
        // (the inverse gains 2^8 on the way to z, which is fp16: A's largest component goes to 2^6 .. 2^7, so that z stays below 46342)
        const int ea = __builtin_amdgcn_readfirstlane(mu::acc_exponent(m)) + 1;
        if (tid == 0) q.exps[at] = ea;
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            H8P v[TE], rest[TE];
#pragma unroll
            for (int m = 0; m < TE; ++m) {
                f4 a, b;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    a[r] = ldexpf(acc[j * TE + m][r].x, -ea);
                    b[r] = ldexpf(acc[j * TE + m][r].y, -ea);
                }
                v[m] = planes(a, b);
                rest[m] = left_over(a, b, v[m]);
            }
            phase2_inv<L, true>(ex + P.mid[j], K, j, mats, v, rest);
        }
        __syncthreads();
        phase3_chunk<true>(K, mats, factors, P, ex);
        store_planes(q.ws_A + at * 2 * L::N, mine, tid);
    }
}

// -------------------------------------------------------------------------------------------------------------------
// Kernel spectrum of a chunk: kscale (FFT + D) as fp16 words in the lane order of phase 2, with the head's exponent.  R = 4: the
// row waits in registers while its maximum is searched; R = 8: maxima and sums come from the caller (rs).
// -------------------------------------------------------------------------------------------------------------------
template <int R>
__global__ void __launch_bounds__(L::NT) __attribute__((amdgpu_waves_per_eu(2)))
chunk_kspec_kernel(const float* __restrict__ k, const float* __restrict__ D, const float* __restrict__ rs, float2* __restrict__ kspec,
                   int H, float kscale_over_c, float kscale, const float2* __restrict__ tw, const uint4* __restrict__ ltab,
                   const uint4* __restrict__ chtab)
{
    extern __shared__ uint4 lds4[];
    __shared__ float mred[3][L::NW];
    _Float16* ex = reinterpret_cast<_Float16*>(lds4);
    uint4* shared = reinterpret_cast<uint4*>(ex + L::EX);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Run<R> me(H);
    constexpr bool HOLD = R == 4;
    static_assert(4 * L::N == 128 * L::NT, "a thread touches 128 bytes");
    f4 v[HOLD ? PC : 1][R][2];
    const auto piece = [&](int to, int n, int i, int h) __attribute__((always_inline)) {
        const f4* p = reinterpret_cast<const f4*>(k + (size_t)h * R * L::N) + (size_t)n * (L::N / 4) + 2 * (tid + i * L::NT);
        v[to][n][0] = p[0];
        v[to][n][1] = p[1];
    };
    const auto ask = [&](int h) __attribute__((always_inline)) {
        if (HOLD) {
#pragma unroll
            for (int i = 0; i < PC; ++i)
#pragma unroll
                for (int n = 0; n < R; ++n) piece(HOLD ? i : 0, n, i, h);
        }
    };
    const uint4* ctab = chtab + chunk_tab<R>() + (size_t)me.k1 * C_UNITS * 64;
    CK<false, 0> K;
    K.load(ltab, ctab, wave, lane, nullptr);
    load_chunk_shared<R>(shared, ltab, ctab, tid);
    const uint4* mats = shared + lane;
    Places<L> P;
    P.make(wave, lane);
    _Float16* mine = ex + piece_of<L>(tid);
    for (int h = me.i0; h < me.i1; ++h) {
        ask(h);
        const float Dh = D[h];
        // the head's largest magnitude; sum and maximum with the skip term counted in the lag-0 tap
        float m = 0.f, a = 0.f, mp = 0.f;
        if constexpr (HOLD) {
#pragma unroll
            for (int i = 0; i < PC; ++i)
#pragma unroll
                for (int n = 0; n < R; ++n)
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const float x = v[i][n][q >> 2][q & 3];
                        const float x0 = i == 0 && n == 0 && q == 0 && tid == 0 ? fabsf(x + Dh) : fabsf(x);
                        m = fmaxf(m, fabsf(x));
                        a += x0;
                        mp = fmaxf(mp, x0);
                    }
            for (int o = 32; o > 0; o >>= 1) {
                m = fmaxf(m, __shfl_xor(m, o, 64));
                mp = fmaxf(mp, __shfl_xor(mp, o, 64));
                a += __shfl_xor(a, o, 64);
            }
            if (lane == 0) { mred[0][wave] = m; mred[1][wave] = a; mred[2][wave] = mp; }
            __syncthreads();
            m = mred[0][0]; a = mred[1][0]; mp = mred[2][0];
#pragma unroll
            for (int w = 1; w < L::NW; ++w) { m = fmaxf(m, mred[0][w]); a += mred[1][w]; mp = fmaxf(mp, mred[2][w]); }
        } else {
            m = rs[h];
            a = rs[H + h];
            mp = rs[2 * H + h];
        }
        const float r = head_scale_of(m);
        float2 f[R];
        outer_factors<R>(f, tw, me.k1, r);
#pragma unroll
        for (int i = 0; i < PC; ++i) {
            if (!HOLD) {
#pragma unroll
                for (int n = 0; n < R; ++n) piece(0, n, i, h);
            }
            u4w re, im;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float s[2], t[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    s[e] = t[e] = 0.f;
#pragma unroll
                    for (int n = 0; n < R; ++n) {
                        const float x = v[HOLD ? i : 0][n][q >> 1][2 * (q & 1) + e];
                        s[e] = __builtin_fmaf(x, f[n].x, s[e]);
                        if (n) t[e] = __builtin_fmaf(x, f[n].y, t[e]);
                    }
                }
                re[q] = mu::pack_h2(s[0], s[1]);
                im[q] = mu::pack_h2(t[0], t[1]);
            }
            *reinterpret_cast<u4w*>(mine + i * L::STEP) = re;
            *reinterpret_cast<u4w*>(mine + L::N + i * L::STEP) = im;
        }
        // One word of every 128 bytes of the next head, of a part each for the R workgroups that read it: no registers are free to ask
        // for the head itself (32 spills, 31 us at B=1, H=128, N=65536), but this much has it in the XCD's L2 when they ask (25.9 -> 23.8;
        // R = 8, which asks piece by piece, 35.7 -> 37.1 at H=64)
        uint32_t near = 0;
        if (HOLD) near = uniform(reinterpret_cast<const uint32_t*>(k), ((size_t)min(h + 1, H - 1) * R + me.k1) * L::N)[(unsigned)tid * 32];
        __syncthreads();
        phase1_chunk<true>(K, mats, P, ex);
        __syncthreads();
        const int es = spec_exponent(kscale * a, kscale * mp);
        if (tid == 0 && me.k1 == 0) spec_exp_of(kspec, H, 2 * (int64_t)R * L::N)[h] = es;
        const float alpha = ldexpf(kscale_over_c / r, -es), beta = ldexpf(Dh * kscale, -es);
        uint4* out = reinterpret_cast<uint4*>(reinterpret_cast<uint32_t*>(kspec) + ((size_t)h * 2 * R + me.k1) * L::N);
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            phase2_fwd<L>(ex + P.mid_tr[j], K, j, mats, [&](int m, const f4& yr, const f4& yi) __attribute__((always_inline)) {
                out[((wave * L::KB + j) * TE + m) * 64 + lane] = planes(yr * alpha + beta, yi * alpha).w;
            });
        }
        if (HOLD) asm volatile("" ::"v"(near));
        __syncthreads();                             // (the buffer, and mred)
    }
}

// -------------------------------------------------------------------------------------------------------------------
// Last step: rows from their chunks' planes, eight points n_2 a thread.  Bound by memory: B=1, H=128, N=65536 10 us, 50 MB
// -------------------------------------------------------------------------------------------------------------------
constexpr int CB = 256;
__device__ __forceinline__ void planes_of(float (&re)[8], float (&im)[8], const _Float16* z)
{
    const h8 a = *reinterpret_cast<const h8*>(z), b = *reinterpret_cast<const h8*>(z + L::N);
#pragma unroll
    for (int e = 0; e < 8; ++e) { re[e] = (float)a[e]; im[e] = (float)b[e]; }
}
// cos, sin of 2 pi n (4 k + 1) / 4R, n and k compile-time constants after unrolling
template <int R>
__device__ __forceinline__ float2 outer_unit(int n, int k)
{
    constexpr float C[9] = {1.f, 0.98078528040323043f, 0.92387953251128674f, 0.83146961230254524f, 0.70710678118654752f,
                            0.55557023301960218f, 0.38268343236508977f, 0.19509032201612825f, 0.f};
    const int m = (n * (4 * k + 1) * (8 / R)) & 31, q = m >> 3, r = m & 7;           // in 32nds of a turn
    const float c = C[r], s = C[8 - r];
    return q == 0 ? make_float2(c, s) : q == 1 ? make_float2(-s, c) : q == 2 ? make_float2(-c, -s) : make_float2(s, -c);
}
template <class IO, int R>
__global__ void __launch_bounds__(CB)
chunk_rows_kernel(const _Float16* __restrict__ ws, typename IO::T* __restrict__ out, int B, int H,
                  const typename IO::T* __restrict__ gate, const uint32_t* __restrict__ max_a, const int* __restrict__ spec_exp)
{
    constexpr int nbx = L::N / (8 * CB);
    const int item = blockIdx.x / nbx, h = item / B, n2 = ((blockIdx.x % nbx) * CB + threadIdx.x) * 8;
    const int e2 = spec_exp[h] + (max_a ? mu::row_exponent(max_a[h]) : 0);
    const size_t o = row_off(item - h * B, h, H, (int64_t)R * L::N) + n2;
    float y[R][8];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        float re[8], im[8];
        planes_of(re, im, ws + ((size_t)item * R + k) * 2 * L::N + n2);
#pragma unroll
        for (int n = 0; n < R; ++n) {
            const float2 w = outer_unit<R>(n, k);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = k ? __builtin_fmaf(re[e], w.x, y[n][e]) : re[e] * w.x;
                y[n][e] = __builtin_fmaf(-im[e], w.y, x);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < R; ++n) {
        u4w w, gw;
        if (gate) gw = *reinterpret_cast<const u4w*>(gate + o + (size_t)n * L::N);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float a = y[n][2 * q], b = y[n][2 * q + 1];
            if (gate) { a *= io_half<IO>(gw[q], 0); b *= io_half<IO>(gw[q], 1); }
            w[q] = pack_io<IO>(ldexpf(a, e2), ldexpf(b, e2));
        }
        put_once(reinterpret_cast<u4w*>(out + o + (size_t)n * L::N), w);
    }
}
// the same for dk, fp32, over the shares of a head; the first thread of a head adds up dD
template <int R>
__global__ void __launch_bounds__(CB)
chunk_dk_kernel(const _Float16* __restrict__ ws, const int* __restrict__ exps, const float* __restrict__ dD_part, float* __restrict__ dk,
                float* __restrict__ dD, int H, int nshare, float scale, const uint32_t* __restrict__ max_a,
                const uint32_t* __restrict__ max_b)
{
    constexpr int nbx = L::N / (8 * CB);
    const int h = blockIdx.x / nbx, n2 = ((blockIdx.x % nbx) * CB + threadIdx.x) * 8;
    if (dD && n2 == 0) {
        float t = 0.f;
        for (int s = 0; s < nshare; ++s)
            for (int k = 0; k < R; ++k) t += dD_part[((size_t)s * H + h) * R + k];
        dD[h] = t;
    }
    if (!dk) return;
    const int er = (max_a ? mu::row_exponent(max_a[h]) : 0) + (max_b ? mu::row_exponent(max_b[h]) : 0);
    float y[R][8];
#pragma unroll
    for (int n = 0; n < R; ++n)
#pragma unroll
        for (int e = 0; e < 8; ++e) y[n][e] = 0.f;
    for (int s = 0; s < nshare; ++s) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const size_t at = ((size_t)s * H + h) * R + k;
            const int ea = exps[at] + er;
            float re[8], im[8];
            planes_of(re, im, ws + at * 2 * L::N + n2);
#pragma unroll
            for (int e = 0; e < 8; ++e) { re[e] = ldexpf(re[e] * scale, ea); im[e] = ldexpf(im[e] * scale, ea); }
#pragma unroll
            for (int n = 0; n < R; ++n) {
                const float2 w = outer_unit<R>(n, k);
#pragma unroll
                for (int e = 0; e < 8; ++e) y[n][e] = __builtin_fmaf(-im[e], w.y, __builtin_fmaf(re[e], w.x, y[n][e]));
            }
        }
    }
#pragma unroll
    for (int n = 0; n < R; ++n)
#pragma unroll
        for (int q = 0; q < 2; ++q)
            *reinterpret_cast<f4*>(dk + (size_t)h * R * L::N + (size_t)n * L::N + n2 + 4 * q) =
                f4{y[n][4 * q], y[n][4 * q + 1], y[n][4 * q + 2], y[n][4 * q + 3]};
}

// workgroups for a list of items: a compute unit holds one, and each takes as many items as the fullest has to
int runs(int64_t items, int R)
{
    const int64_t slots = compute_units() / R > 0 ? compute_units() / R : 1, per = (items + slots - 1) / slots;
    return (int)((items + per - 1) / per) * R;
}

template <class IO, int R>
hipError_t conv_io(const void* in, const float2* kspec, void* out, void* ws, bool conj, const Problem& pr, const Tables& tb, hipStream_t st)
{
    using T = typename IO::T;
    const int nwg = runs(pr.B * pr.H, R);
    const auto go = [&](auto kern) {
        const hipError_t e = set_lds(kern, chunk_lds(0));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)nwg), dim3(L::NT), chunk_lds(0), st, (const T*)in, kspec, (_Float16*)ws, (int)pr.B,
                           (int)pr.H, tb.tw, (const uint4*)tb.ltab, (const uint4*)tb.chtab, pr.max_a);
        return hipGetLastError();
    };
    const hipError_t e = conj ? go(chunk_conv_kernel<IO, R, true>) : go(chunk_conv_kernel<IO, R, false>);
    if (e != hipSuccess) return e;
    return chunk_rows(ws, out, pr, R, st);
}
template <class IO, int R>
hipError_t bwd_io(const void* dy, const void* u, const float2* kspec, void* ws_du, void* ws_A, int* exps, float* dD_part, int ns,
                  const Problem& pr, const Tables& tb, hipStream_t st)
{
    using T = typename IO::T;
    const CBwdArgs<T> a{(const T*)dy, (const T*)u, kspec, (_Float16*)ws_du, (_Float16*)ws_A, exps, dD_part, (int)pr.B, (int)pr.H, ns,
                        tb.tw, (const uint4*)tb.ltab, (const uint4*)tb.chtab, pr.max_a, pr.max_b};
    const auto go = [&](auto kern) {
        const hipError_t e = set_lds(kern, chunk_lds(CNAL));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)runs(pr.H * ns, R)), dim3(L::NT), chunk_lds(CNAL), st, a);
        return hipGetLastError();
    };
    if constexpr (R > 2)
        if (ws_du) return go(chunk_bwd_kernel<IO, R, true>);
    return go(chunk_bwd_kernel<IO, R, false>);
}

}  // namespace

hipError_t chunk_fill_tables(const void** tab_out, hipStream_t st)
{
    uint4* p = nullptr;
    const hipError_t e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(g_chunk_tab));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fill_chunk_tab_kernel<2>, dim3(C_UNITS, 2), dim3(64), 0, st, p);
    hipLaunchKernelGGL(fill_chunk_tab_kernel<4>, dim3(C_UNITS, 4), dim3(64), 0, st, p);
    hipLaunchKernelGGL(fill_chunk_tab_kernel<8>, dim3(C_UNITS, 8), dim3(64), 0, st, p);
    *tab_out = p;
    return hipGetLastError();
}

hipError_t chunk_kspec(const float* k, const float* D, const float* rs, float2* kspec, int64_t H, const Plan& pl, const Tables& tb,
                       hipStream_t st)
{
    const auto go = [&](auto kern, int R) {
        const hipError_t e = set_lds(kern, chunk_lds(0));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)runs(H, R)), dim3(L::NT), chunk_lds(0), st, k, D, rs, kspec, (int)H,
                           pl.kscale * (float)(1 << L::SHIFT), pl.kscale, tb.tw, (const uint4*)tb.ltab, (const uint4*)tb.chtab);
        return hipGetLastError();
    };
    return pl.log2R == 2 ? go(chunk_kspec_kernel<4>, 4) : go(chunk_kspec_kernel<8>, 8);
}

hipError_t chunk_rows(const void* ws, void* out, const Problem& pr, int R, hipStream_t st)
{
    const dim3 grid((unsigned)(L::N / (8 * CB) * pr.B * pr.H));
#define GO(IO, RR) hipLaunchKernelGGL((chunk_rows_kernel<IO, RR>), grid, dim3(CB), 0, st, (const _Float16*)ws, (IO::T*)out, (int)pr.B, \
                                      (int)pr.H, (const IO::T*)pr.gate, pr.max_a, pr.spec_exp)
    if (pr.io == LONGCONV_F16) { if (R == 4) GO(IoF16, 4); else GO(IoF16, 8); }
    else if (pr.io == LONGCONV_BF16) { if (R == 4) GO(IoBF16, 4); else GO(IoBF16, 8); }
    else return hipErrorInvalidValue;
#undef GO
    return hipGetLastError();
}

hipError_t chunk_conv(const void* in, const float2* kspec, void* out, void* ws, bool conj, const Problem& pr, const Plan& pl,
                      const Tables& tb, hipStream_t st)
{
#define GO(IO)                                                                              \
    return pl.log2R == 2 ? conv_io<IO, 4>(in, kspec, out, ws, conj, pr, tb, st)             \
                         : conv_io<IO, 8>(in, kspec, out, ws, conj, pr, tb, st)
    if (pr.io == LONGCONV_F16) GO(IoF16);
    if (pr.io == LONGCONV_BF16) GO(IoBF16);
#undef GO
    return hipErrorInvalidValue;
}

// Shares of a head's rows where one leaves at least half of a whole device's 256 compute units idle (one holds one workgroup): two, or (more: where
// their results find room) the number that ends first, a row 12 us and another share 2 in chunk_dk_kernel, which reads all of them.
// Steps, two shares at most and now: B=64, H=4, N=65536 bf16 614 -> 267 us, B=31, H=12 fp16 355 -> 228; B=64, H=4, N=32768 354 -> 134,
// B=10, H=21 137 -> 120; B=16, H=7, N=131072 bf16 359 -> 298; B=7, H=4, N=65536 101.6 -> 90.3.
int chunk_bwd_shares(int64_t B, int64_t H, int log2R, bool more)
{
    int64_t most = 256 / (H << log2R);
    if (most < 2 || B < 2) return 1;
    if (!more || most > (B - 1) / 2) most = more && (B - 1) / 2 > 2 ? (B - 1) / 2 : 2;
    int64_t best = 2, best_t = 6 * ((B + 1) / 2) + 2;
    for (int64_t s = 3; s <= most; ++s) {
        const int64_t t = 6 * ((B + s - 1) / s) + s;
        if (t < best_t) { best = s; best_t = t; }
    }
    return (int)best;
}

hipError_t chunk_bwd(const void* dy, const void* u, const float2* kspec, void* du, void* ws_du, float* dk, float* dD, void* ws_A,
                     int* exps, float* dD_part, int ns, const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
    const int R = 1 << pl.log2R;
    if (du && R == 2) return hipErrorInvalidValue;   // (rows of 32768 samples have their spectrum in another order)
    hipError_t e = hipErrorInvalidValue;
    void *wd = du ? ws_du : nullptr, *wa = dk ? ws_A : nullptr;
    float* dp = dD ? dD_part : nullptr;
#define GO(IO)                                                                                   \
    e = R == 2   ? bwd_io<IO, 2>(dy, u, kspec, nullptr, wa, exps, dp, ns, pr, tb, st)            \
        : R == 4 ? bwd_io<IO, 4>(dy, u, kspec, wd, wa, exps, dp, ns, pr, tb, st)                 \
                 : bwd_io<IO, 8>(dy, u, kspec, wd, wa, exps, dp, ns, pr, tb, st)
    if (pr.io == LONGCONV_F16) GO(IoF16);
    if (pr.io == LONGCONV_BF16) GO(IoBF16);
#undef GO
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)(L::N / (8 * CB) * pr.H));
    // two forward chains and one inverse chain of twice the scale, 1 / N
    const float dkscale = 1.0f / (2.0f * (float)pr.N) * (float)(1 << 3 * L::SHIFT);
#define GO(RR) hipLaunchKernelGGL(chunk_dk_kernel<RR>, grid, dim3(CB), 0, st, (const _Float16*)ws_A, exps, dD_part, dk, dD, (int)pr.H, ns, \
                                  dkscale, pr.max_a, pr.max_b)
    if (R == 2) GO(2);
    else if (R == 4) GO(4);
    else GO(8);
#undef GO
    if ((e = hipGetLastError()) != hipSuccess || !du) return e;
    Problem pc = pr;                                 // du: the powers of two of dy's rows and of the spectrum
    pc.max_a = pr.max_b;
    return chunk_rows(ws_du, du, pc, R, st);
}

}  // namespace lc
