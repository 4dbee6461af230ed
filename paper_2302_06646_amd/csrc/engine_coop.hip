// Workgroup-cooperative chained kernels for 8192 <= L2 <= 32768 (one row of 32768 samples, or one chunk of
// the multi-pass split, per workgroup at a time; it lives in LDS only between phases).
//
// L2 = 16 * 16 * 16 * TE, TE = 2^te in {2,4,8}; TC = 16*TE.  Time index
// n = d_a*16*TC + d_b*TC + d_c*TE + d_e, frequency f = k_a + 16 k_b + 256 k_c + 4096 k_e
// (Section 3.2 "Butterfly Decomposition", applied three times; twiddles of Appendix C.1).
// As in the wave-autonomous kernels an "A-role" MFMA (data as A operand) contracts the slot index
// and transposes the tile, a "B-role" MFMA contracts it in place, so two digits are contracted
// per trip through registers and the row crosses LDS only twice per transform pair:
//   phase 1 (tile t = d_c*TE+d_e): [A: F16 over d_a] * w_L^(k_a(d_b TC + t))
//                                  -> [B: F16 over d_b] * w_{16TC}^(k_b t) -> LDS
//   phase 2 (tile = (k_a, high bits of k_b)): LDS -> [A: F16 over d_c] * w_TC^(k_c d_e)
//            -> [B: F_TE over d_e] * spectrum -> [A: F_TE^-1] * conj -> [B: F16^-1 over k_c] -> LDS
//   phase 3 (tile t): LDS * conj(w_{16TC}) -> [A: F16^-1 over k_b] * conj(w_L) -> [B: F16^-1 over k_a]
// Each wave owns groups of 8 consecutive tiles in every phase; workgroup barriers separate
// the phases.  The w_{16TC} twiddles come from a small table in LDS, the w_TC ones are per-lane constants.
//
// Two forms of phases 1 and 3.  Direct (dk and spectrum from pass A's workspace): operands straight from global
// memory in the tile's lane order, w_L twiddles from a lane-ordered global table (16 bytes per lane and tile).
// Staged (whatever takes rows): the whole workgroup moves them between global memory and LDS in unit-stride
// runs, phases 1 and 3 run in place on LDS, and the w_L twiddle is a per-lane constant times an LDS table.
#include <type_traits>

#include "engines.hpp"
#include "mfma_util.hpp"

namespace lc {

constexpr int NTB = 4;   // tiles advanced together per wave (instruction-level parallelism)

template <int LG>
struct CC {
    static constexpr int cb = LG - 8, TC = 1 << cb, te = cb - 4, TE = 1 << te, L = 1 << LG;
    static constexpr int PITCH = 4 * TC + 1;           // 16-byte chunks per k_a row
    static constexpr int XWORDS = 16 * PITCH * 4;      // exchange buffer, 32-bit words
    static constexpr int NW = TC / 8 > 8 ? 8 : TC / 8; // waves per workgroup
    static constexpr int NG = TC / (8 * NW);           // groups of 8 tiles per wave and phase
    // constant table in uint4 units (global): lane-ordered w_L twiddles, then the w_{16TC} table
    static constexpr int T0F = 0;                      // [TC][64]
    static constexpr int T0I = TC * 64;                // [TC][64]
    static constexpr int T1F = 2 * TC * 64;            // [TC][4]   (t, lane/16): four fp16 complex
    static constexpr int T1I = T1F + TC * 4;           // [TC][4]
    static constexpr int TAB_U4 = T1I + TC * 4;
};

__host__ __device__ constexpr size_t coop_tab_offset(int LG)
{
    size_t o = 0;
    for (int l = 13; l < LG; ++l) o += ((size_t)(1 << (l - 8)) * 136) * 16;
    return o;
}
constexpr size_t COOP_TAB_TOTAL = coop_tab_offset(16);

__device__ unsigned char g_coop_tab[COOP_TAB_TOTAL] __attribute__((aligned(256)));

// T0F : w_L^(k_a (d_b TC + t)),       k_a = lane%16, d_b = 4 (lane/16) + j
// T0I : conj w_L^(k_a (n_b TC + t)),  n_b = lane%16, k_a = 4 (lane/16) + j
// T1F : w_{16TC}^(k_b t), T1I its conjugate, k_b = 4 g + j
__global__ void fill_coop_tab_kernel(unsigned char* tab, int LG)
{
    const int cb = LG - 8, TC = 1 << cb, L = 1 << LG;
    _Float16* base = reinterpret_cast<_Float16*>(tab + coop_tab_offset(LG));
    _Float16* T0f = base;
    _Float16* T0i = base + (size_t)TC * 64 * 8;
    _Float16* T1f = base + (size_t)2 * TC * 64 * 8;
    _Float16* T1i = T1f + (size_t)TC * 4 * 8;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= L) return;
    const int j = i & 3, lane = (i >> 2) & 63, t = i >> 8;
    const int x = lane & 15, y = 4 * (lane >> 4) + j;
    double s, c;
    sincospi(-2.0 * (double)((x * (y * TC + t)) & (L - 1)) / (double)L, &s, &c);
    T0f[((size_t)t * 64 + lane) * 8 + 2 * j] = (_Float16)c;
    T0f[((size_t)t * 64 + lane) * 8 + 2 * j + 1] = (_Float16)s;
    sincospi(+2.0 * (double)((y * (x * TC + t)) & (L - 1)) / (double)L, &s, &c);
    T0i[((size_t)t * 64 + lane) * 8 + 2 * j] = (_Float16)c;
    T0i[((size_t)t * 64 + lane) * 8 + 2 * j + 1] = (_Float16)s;
    if (x == 0) {
        const int g = lane >> 4;
        sincospi(-2.0 * (double)((y * t) & (16 * TC - 1)) / (double)(16 * TC), &s, &c);
        T1f[((size_t)t * 4 + g) * 8 + 2 * j] = (_Float16)c;
        T1f[((size_t)t * 4 + g) * 8 + 2 * j + 1] = (_Float16)s;
        T1i[((size_t)t * 4 + g) * 8 + 2 * j] = (_Float16)c;
        T1i[((size_t)t * 4 + g) * 8 + 2 * j + 1] = (_Float16)(-s);
    }
}

hipError_t coop_fill_tables(const void** tab_out, hipStream_t st)
{
    unsigned char* p = nullptr;
    hipError_t e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(g_coop_tab));
    if (e != hipSuccess) return e;
    for (int LG = 13; LG <= 15; ++LG)
        hipLaunchKernelGGL(fill_coop_tab_kernel, dim3((1 << LG) / 256), dim3(256), 0, st, p, LG);
    *tab_out = p;
    return hipGetLastError();
}

namespace {

using namespace mu;

// fp16 complex times fp16 complex, packed (v_pk_mul_f16 + v_pk_fma_f16)
__device__ __forceinline__ uint32_t cmul_h2(uint32_t yu, h2 w)
{
    union { uint32_t u; h2 h; } a, r;
    a.u = yu;
    const h2 yx = {a.h[0], a.h[0]}, yy = {a.h[1], a.h[1]};
    const h2 ws = {-w[1], w[0]};
    r.h = __builtin_elementwise_fma(yy, ws, yx * w);
    return r.u;
}

template <int LG>
struct Consts {
    Mats F16, I16, FL, IL;
    h2 t2f[4], t2i[4];
};

template <int LG>
__device__ __forceinline__ void make_consts(Consts<LG>& K, const float2* __restrict__ tw, int lane)
{
    using C = CC<LG>;
    K.F16 = plain_mats(4, false, tw, lane);
    K.I16 = plain_mats(4, true, tw, lane);
    K.FL = plain_mats(C::te, false, tw, lane);
    K.IL = plain_mats(C::te, true, tw, lane);
    const int x = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        // forward: lane k_c = x, row (e, d_e) = 4g+j ; inverse: lane (e, d_e) = x, row k_c = 4g+j
        const int de_f = (4 * g + j) & (C::TE - 1), de_i = x & (C::TE - 1);
        const float2 wf = tw_full(tw, (uint32_t)((x * de_f) & (C::TC - 1)) << (TW_LOG2 - C::cb));
        const float2 wi = tw_full(tw, (uint32_t)(((4 * g + j) * de_i) & (C::TC - 1)) << (TW_LOG2 - C::cb));
        K.t2f[j] = h2{(_Float16)wf.x, (_Float16)wf.y};
        K.t2i[j] = h2{(_Float16)wi.x, (_Float16)(-wi.y)};
    }
}

// phase 1 arithmetic on the operand words of 8 tiles, w[j][tile] fp16 complex
template <int LG, int NB = NTB>
__device__ __forceinline__ void phase1_core(const uint32_t (&w)[4][8], uint32_t* xb, const uint4* gtab,
                                            const uint4* t1f, const Mats& F1, const Mats& F2, int t0, int lane)
{
    using C = CC<LG>;
    const int c = lane & 15, g = lane >> 4;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    const int w1 = (c * C::PITCH + g * C::TC) * 4;
#pragma unroll
    for (int tb = 0; tb < 8; tb += NB) {
        H8U tw0[NB], tw1[NB];
        f4 yr[NB], yi[NB], zr[NB], zi[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int t = t0 + tb + k;
            tw0[k].u = gtab[C::T0F + t * 64 + lane];
            tw1[k].u = t1f[t * 4 + g];
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int tt = tb + k;
            H8U x;
#pragma unroll
            for (int j = 0; j < 4; ++j) x.w[j] = w[j][tt];
            yr[k] = MFMA(x.v, F1.re, zero);
            yi[k] = MFMA(x.v, F1.im, zero);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            H8U u;
#pragma unroll
            for (int j = 0; j < 4; ++j) u.w[j] = cmul_pack(yr[k][j], yi[k][j], tw0[k].c[j]);
            zr[k] = MFMA(F2.re, u.v, zero);
            zi[k] = MFMA(F2.im, u.v, zero);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            uint4 o;
            o.x = cmul_pack(zr[k][0], zi[k][0], tw1[k].c[0]);
            o.y = cmul_pack(zr[k][1], zi[k][1], tw1[k].c[1]);
            o.z = cmul_pack(zr[k][2], zi[k][2], tw1[k].c[2]);
            o.w = cmul_pack(zr[k][3], zi[k][3], tw1[k].c[3]);
            *reinterpret_cast<uint4*>(&xb[w1 + 4 * (t0 + tb + k)]) = o;
        }
        __builtin_amdgcn_sched_barrier(0);   // one batch at a time: bounds register pressure
    }
}

// ---- phase 1 for the 8 tiles t0..t0+7 of one wave, operands from a chunk of L fp16 complex values
// (pass-A output of the multi-pass split) ------------------------------------------------------
template <int LG, int NB = NTB>
__device__ __forceinline__ void phase1(const __half2* chunk, uint32_t* xb, const uint4* gtab, const uint4* t1f,
                                       const Consts<LG>& K, int t0, int lane)
{
    using C = CC<LG>;
    const int c = lane & 15, g = lane >> 4;
    uint32_t w[4][8];       // [j][tile] complex words
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n0 = (4 * g + j) * 16 * C::TC + c * C::TC + t0;
        load_words<4>(chunk + n0, &w[j][0]);
        load_words<4>(chunk + n0 + 4, &w[j][4]);
    }
    phase1_core<LG, NB>(w, xb, gtab, t1f, K.F16, K.F16, t0, lane);
}

// word address of (tile t2, reg 0) for this lane in phase 2; reg j adds j*TE*4 words
template <int LG>
__device__ __forceinline__ int phase2_base(int t2, int lane)
{
    using C = CC<LG>;
    const int x = lane & 15, g = lane >> 4;
    const int de = x & (C::TE - 1), e = x >> C::te;
    const int ka = t2 >> C::te, kb = ((t2 & (C::TE - 1)) << (4 - C::te)) | e;
    const int t = (4 * g) * C::TE + de;
    return (ka * C::PITCH + (kb >> 2) * C::TC + t) * 4 + (kb & 3);
}

// tile t2 = t0 + k, t0 a multiple of TE = 8 tiles: words from t0's place
template <int LG>
__device__ __forceinline__ constexpr int phase2_step(int k)
{
    using C = CC<LG>;
    const int kb = (k & (C::TE - 1)) << (4 - C::te);
    return ((k >> C::te) * C::PITCH + (kb >> 2) * C::TC) * 4 + (kb & 3);
}

// forward half of phase 2 on one tile: LDS -> [A: F16 over d_c] * w_TC -> [B: F_TE over d_e]
template <int LG>
__device__ __forceinline__ void phase2_fwd(const H8U& x, const Consts<LG>& K, f4& zr, f4& zi)
{
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    const f4 yr = MFMA(x.v, K.F16.re, zero), yi = MFMA(x.v, K.F16.im, zero);
    H8U u;
#pragma unroll
    for (int j = 0; j < 4; ++j) u.w[j] = cmul_pack(yr[j], yi[j], K.t2f[j]);
    zr = MFMA(K.FL.re, u.v, zero);
    zi = MFMA(K.FL.im, u.v, zero);
}
template <int LG>
__device__ __forceinline__ void phase2_fwd(const uint32_t* xb, int base, const Consts<LG>& K, f4& zr, f4& zi)
{
    H8U x;
#pragma unroll
    for (int j = 0; j < 4; ++j) x.w[j] = xb[base + j * CC<LG>::TE * 4];
    phase2_fwd<LG>(x, K, zr, zi);
}

// inverse half of phase 2 on one tile: (already multiplied) spectrum values m -> LDS
template <int LG>
__device__ __forceinline__ void phase2_inv_regs(const Consts<LG>& K, const H8U& m, H8U& out)
{
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    const f4 yr = MFMA(m.v, K.IL.re, zero), yi = MFMA(m.v, K.IL.im, zero);
    H8U u;
#pragma unroll
    for (int j = 0; j < 4; ++j) u.w[j] = cmul_pack(yr[j], yi[j], K.t2i[j]);
    const f4 vr = MFMA(K.I16.re, u.v, zero), vi = MFMA(K.I16.im, u.v, zero);
#pragma unroll
    for (int j = 0; j < 4; ++j) out.w[j] = pack_h2(vr[j], vi[j]);
}
template <int LG>
__device__ __forceinline__ void phase2_inv(uint32_t* xb, int base, const Consts<LG>& K, const H8U& m)
{
    H8U o;
    phase2_inv_regs<LG>(K, m, o);
#pragma unroll
    for (int j = 0; j < 4; ++j) xb[base + j * CC<LG>::TE * 4] = o.w[j];
}

// phase 3 on two tiles t, t+1: returns real parts r[k] and imaginary parts s[k] of the time samples
template <int LG>
__device__ __forceinline__ void phase3_two(const uint32_t* xb, const uint4* gtab, const uint4* t1i,
                                           const Consts<LG>& K, int t, int lane, f4 (&r)[2], f4 (&s)[2])
{
    using C = CC<LG>;
    const int c = lane & 15, g = lane >> 4;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    const int w1 = (c * C::PITCH + g * C::TC) * 4;
    H8U tw0[2], tw1[2], x[2];
    f4 yr[2], yi[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        tw0[k].u = gtab[C::T0I + (t + k) * 64 + lane];
        tw1[k].u = t1i[(t + k) * 4 + g];
        x[k].u = *reinterpret_cast<const uint4*>(&xb[w1 + 4 * (t + k)]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[k].w[j] = cmul_h2(x[k].w[j], tw1[k].c[j]);
        yr[k] = MFMA(x[k].v, K.I16.re, zero);
        yi[k] = MFMA(x[k].v, K.I16.im, zero);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        H8U u;
#pragma unroll
        for (int j = 0; j < 4; ++j) u.w[j] = cmul_pack(yr[k][j], yi[k][j], tw0[k].c[j]);
        r[k] = MFMA(K.I16.re, u.v, zero);
        s[k] = MFMA(K.I16.im, u.v, zero);
    }
}

// -------------------------------------------------------------------------------------
// The staged layout.  The phase-1 tile of a wave takes samples a tile count apart, so loading its operands straight
// from global memory touches 16 bytes of every 256; here the whole workgroup moves the points between global memory
// and LDS in unit-stride 16-byte runs instead, into the very slots that phase 1 reads and phase 3 writes: point
// n = d_a 16 TC + d_b TC + t, an fp16 complex word, lives in word (d_b PITCH + (d_a / 4) TC + t) 4 + d_a % 4 -- the
// slot phase 1 fills with output (k_a, k_b) = (d_b, d_a) of tile t, and phase 3 the other way round, each lane reading
// and writing only its own 16 bytes.  The next runs are fetched into registers before phase 1 and stored to LDS by the
// lane that has just drained the same slots, so global latency is covered by the three phases and no phase but the
// second (spectrum) issues global loads: the w_L twiddle of phases 1 and 3 is the product of a per-lane constant
// w_256^(k_a d_b) and an LDS table w_L^(k_a t).
// -------------------------------------------------------------------------------------
__device__ __forceinline__ h2 cmul_hh(h2 a, h2 w)
{
    const h2 ax = {a[0], a[0]}, ay = {a[1], a[1]};
    const h2 ws = {-w[1], w[0]};
    return __builtin_elementwise_fma(ay, ws, ax * w);
}

// SW: the slots of eight consecutive t change places, in pairs, by XOR with the low bits of t / 8.  Four lanes of a row on its way
// write (read) samples eight apart at a time, whose slots lie in the same banks otherwise (B=32, H=128, N=32768 fp16: 312
// us, LDS busy 44% of the time and half of that in conflicts; 279 and 32%).
template <int LG, bool SW>
__device__ __forceinline__ void tile_places(int (&at)[4], int w1, int t0)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) at[j] = w1 + 4 * t0 + 8 * (SW ? j ^ ((t0 >> 3) & 3) : j);
}
// Phase 1 in place on the staged layout, 8 tiles t0..t0+7 of one wave: each lane reads its own 16 bytes
// of a tile (samples d_a = 4g..4g+3 of column d_b = c) and writes outputs (k_a, k_b) = (c, 4g..4g+3) there.
// F1 is the first-stage matrix (rows of the zero padding cleared when those slots hold stale data).
struct NothingElse { __device__ __forceinline__ void operator()(int) const {} };
template <int LG, int NB, bool SW = false, class Also = NothingElse>
__device__ __forceinline__ void phase1_inplace(uint32_t* xb, const uint4* t1f, const uint32_t* vt, const Mats& F1,
                                               const Mats& F2, const h2 (&cF)[4], int t0, int lane, Also&& also = Also())
{
    using C = CC<LG>;
    const int c = lane & 15, g = lane >> 4;
    const int w1 = (c * C::PITCH + g * C::TC) * 4;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    int at[4];                                           // places of tiles t0, t0 + 2, ..; the next tile is 4 words on
    tile_places<LG, SW>(at, w1, t0);
#pragma unroll
    for (int tb = 0; tb < 8; tb += NB) {
        H8U x[NB], tw1[NB];
        h2 v[NB];
        f4 yr[NB], yi[NB], zr[NB], zi[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int t = t0 + tb + k;
            x[k].u = *reinterpret_cast<const uint4*>(&xb[at[(tb + k) >> 1] + ((tb + k) & 1) * 4]);
            tw1[k].u = t1f[t * 4 + g];
            union { uint32_t u; h2 h; } cv;
            cv.u = vt[t * 16 + c];
            v[k] = cv.h;
        }
        also(tb / NB);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            yr[k] = MFMA(x[k].v, F1.re, zero);
            yi[k] = MFMA(x[k].v, F1.im, zero);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            H8U u;
#pragma unroll
            for (int j = 0; j < 4; ++j) u.w[j] = cmul_pack(yr[k][j], yi[k][j], cmul_hh(cF[j], v[k]));
            zr[k] = MFMA(F2.re, u.v, zero);
            zi[k] = MFMA(F2.im, u.v, zero);
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            uint4 o;
            o.x = cmul_pack(zr[k][0], zi[k][0], tw1[k].c[0]);
            o.y = cmul_pack(zr[k][1], zi[k][1], tw1[k].c[1]);
            o.z = cmul_pack(zr[k][2], zi[k][2], tw1[k].c[2]);
            o.w = cmul_pack(zr[k][3], zi[k][3], tw1[k].c[3]);
            *reinterpret_cast<uint4*>(&xb[at[(tb + k) >> 1] + ((tb + k) & 1) * 4]) = o;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Phase 3 on tiles t, t+1 of the staged layout with the factored w_L twiddle: real parts r[k], imaginary
// parts s[k] of time samples (d_a, d_b) = (4g+j, c) of each tile.
template <int LG>
__device__ __forceinline__ void phase3_two_lds(const uint32_t* xb, const uint4* t1i, const uint32_t* vt,
                                               const Consts<LG>& K, const h2 (&cF)[4], int t, int lane,
                                               f4 (&r)[2], f4 (&s)[2])
{
    using C = CC<LG>;
    const int c = lane & 15, g = lane >> 4;
    const int w1 = (c * C::PITCH + g * C::TC) * 4;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    H8U tw1[2], x[2], vv[2];
    f4 yr[2], yi[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        tw1[k].u = t1i[(t + k) * 4 + g];
        x[k].u = *reinterpret_cast<const uint4*>(&xb[w1 + 4 * (t + k)]);
        vv[k].u = *reinterpret_cast<const uint4*>(&vt[(t + k) * 16 + 4 * g]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[k].w[j] = cmul_h2(x[k].w[j], tw1[k].c[j]);
        yr[k] = MFMA(x[k].v, K.I16.re, zero);
        yi[k] = MFMA(x[k].v, K.I16.im, zero);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        H8U u;
#pragma unroll
        for (int j = 0; j < 4; ++j) u.w[j] = cmul_pack_conj(yr[k][j], yi[k][j], cmul_hh(cF[j], vv[k].c[j]));
        r[k] = MFMA(K.I16.re, u.v, zero);
        s[k] = MFMA(K.I16.im, u.v, zero);
    }
}

// tables of the staged layout: w_{16TC} (both directions) and w_L^(k_a t); exchange buffer cleared
template <int LG, int NT>
__device__ __forceinline__ void staged_tables(uint4* lds4, const uint4* gtab, const float2* __restrict__ tw, int tid,
                                              int gap)
{
    using C = CC<LG>;
    uint4* t1f = lds4 + C::XWORDS / 4 + gap;             // `gap` 16-byte units between the slots and the tables
    uint32_t* vt = reinterpret_cast<uint32_t*>(t1f + C::TC * 8);
    for (int i = tid; i < C::TC * 8; i += NT) t1f[i] = gtab[C::T1F + i];
    for (int i = tid; i < C::TC * 16; i += NT) {
        const float2 w = tw_full(tw, (uint32_t)(((i & 15) * (i >> 4)) & (C::L - 1)) << (TW_LOG2 - LG));
        vt[i] = pack_h2(w.x, w.y);
    }
    for (int i = tid; i < C::XWORDS / 4; i += NT) lds4[i] = make_uint4(0u, 0u, 0u, 0u);
}

// run r of a row pair -> first sample n: four lanes cover 64 contiguous bytes of a row, the next lane
// bits pick d_a % 4 and d_b % 4, so that a wave's 4-byte LDS accesses (word stride 4 along t) spread
// over 32 banks while global accesses keep 64-byte segments
template <int LG>
__device__ __forceinline__ constexpr int staged_run_n(int r)
{
    using C = CC<LG>;
    constexpr int QB = C::cb - 3;
    const int q = (r & 3) | (((r >> 6) & ((1 << (QB - 2)) - 1)) << 2);
    const int da = ((r >> 2) & 3) | ((r >> (QB + 6)) << 2);
    const int db = ((r >> 4) & 3) | (((r >> (QB + 4)) & 3) << 2);
    return (da << (C::cb + 4)) + (db << C::cb) + 8 * q;
}
// what run i NT + r adds to run r, NT a multiple of the runs that share d_a / 4 and the high bit of d_b
template <int LG>
__device__ __forceinline__ constexpr int run_step(int r) { return staged_run_n<LG>(r); }
// word of sample n of the pair in the exchange buffer (consecutive samples are 4 words apart)
template <int LG>
__device__ __forceinline__ constexpr int staged_slot(int n)
{
    using C = CC<LG>;
    const int t = n & (C::TC - 1), db = (n >> C::cb) & 15, da = n >> (C::cb + 4);
    return (db * C::PITCH + (da >> 2) * C::TC + t) * 4 + (da & 3);
}

template <int LG>
__host__ __device__ constexpr size_t coop_staged_lds_bytes() { return (size_t)CC<LG>::XWORDS * 4 + (size_t)CC<LG>::TC * 8 * 16 + (size_t)CC<LG>::TC * 16 * 4; }

// -------------------------------------------------------------------------------------
// Inner convolution of the multi-pass split on the staged layout: chunk k1 (L fp16 complex values of pass
// A's output) of every row pair, in place in the workspace.  Work items (head, chunk, pair), consecutive
// ones (same spectrum slice) per workgroup; a chunk moves between the workspace and the slots in
// unit-stride 16-byte runs of four values.  Lane bits of a run: two for the position in a 64-byte
// segment, then d_a % 4 and d_b % 4 (the 4-byte LDS accesses of a wave then hit 64 different banks).
// -------------------------------------------------------------------------------------
// (1/4) F16[m][sig] w_{2^lt}^(k1 sig 2^wl) as MFMA operand: the contraction index sig carries the phase
__device__ __forceinline__ Mats phase_mats(int k1, int wl, int lt, const float2* __restrict__ tw, int lane)
{
    const int m = lane & 15, g = lane >> 4;
    Mats A;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int sig = 4 * g + q;
        const uint32_t idx = ((uint32_t)((m * sig) & 15) << (TW_LOG2 - 4)) + ((uint32_t)(k1 * sig) << (wl + TW_LOG2 - lt));
        const float2 w = tw_full(tw, idx & (TW_L - 1));
        A.re[2 * q] = (_Float16)(w.x * 0.25f);
        A.re[2 * q + 1] = (_Float16)(-w.y * 0.25f);
        A.im[2 * q] = (_Float16)(w.y * 0.25f);
        A.im[2 * q + 1] = (_Float16)(w.x * 0.25f);
    }
    return A;
}

// forward w_{16TC} table times the tile part w_{2^LR L}^(k1 t) of pass A's twist
template <int LG, int LR, int NT>
__device__ __forceinline__ void twisted_t1f(uint4* t1f, const uint4* gtab, int k1, const float2* __restrict__ tw, int tid)
{
    using C = CC<LG>;
    for (int i = tid; i < C::TC * 4; i += NT) {
        const float2 w = tw_full(tw, (uint32_t)(k1 * (i >> 2)) << (TW_LOG2 - LG - LR));
        const h2 tau = {(_Float16)w.x, (_Float16)w.y};
        H8U e;
        e.u = gtab[C::T1F + i];
#pragma unroll
        for (int j = 0; j < 4; ++j) e.w[j] = cmul_h2(e.w[j], tau);
        t1f[i] = e.u;
    }
}

// run r of a chunk of complex values (16-byte runs of four) -> first value n; lane bits as for the rows:
// position in a 64-byte segment, d_a % 4, d_b % 4
template <int LG>
__device__ __forceinline__ int chunk_run_n(int r)
{
    using C = CC<LG>;
    constexpr int QB = C::cb - 2;                // runs per (d_a, d_b) row = TC / 4
    const int q = (r & 3) | (((r >> 6) & ((1 << (QB - 2)) - 1)) << 2);
    const int da = ((r >> 2) & 3) | ((r >> (QB + 6)) << 2);
    const int db = ((r >> 4) & 3) | (((r >> (QB + 4)) & 3) << 2);
    return (da << (C::cb + 4)) + (db << C::cb) + 4 * q;
}

// -------------------------------------------------------------------------------------
// Single rows of N = L = 32768 samples, forward and du: one N-point transform of the twisted row
//     X[f] = sum_n x[n] exp(-2 pi i n (4 f + 1) / 4N),
// whose products are convolutions modulo z^N - i; the real part, untwisted, is the causal convolution truncated to N
// samples (see engine_rows.hip).  The row's transform fits one compute unit, so rows go from memory to memory in one
// kernel.  (As row pairs in two chunks of a 65536-point transform the same matrix work needs a complex fp16 workspace
// of twice the rows' bytes written, and read back by a pass C kernel, and has two chunks where an odd last row needs one.)
// B=32, H=128, N=32768 fp16: 670 us as pairs in two chunks, 279 us here (1.9 TB/s); what is left is matrix and vector issue.
// The twist W^n, W = exp(-2 pi i / 4N), n = d_a 16 TC + d_b TC + t, takes no instructions: its d_a factor sits in the
// matrices over d_a of both directions, its d_b factor in the lanes' w_256 constants and its t factor in the w_L table,
// which phases 1 and 3 (conjugated) share.  The next row is prefetched in registers; a bf16 row outside the band is scaled by
// a power of two (band_or_exact).
// -------------------------------------------------------------------------------------
template <int LG, class IO, int NWV, int NB, bool CONJ, bool GATE, bool RUNS>
__global__ void __launch_bounds__(NWV * 64) __attribute__((amdgpu_waves_per_eu(2)))
coop_conv_row_kernel(const typename IO::T* __restrict__ in, const float2* __restrict__ kspec,
                     typename IO::T* __restrict__ out, const typename IO::T* __restrict__ gate, int64_t B, int64_t H,
                     int per, const float2* __restrict__ tw, const unsigned char* __restrict__ ctab)
{
    using C = CC<LG>;
    constexpr int NT = NWV * 64;
    constexpr int RPL = (C::L / 8) / NT;             // 16-byte runs (8 samples) of the row per lane
    static_assert(RPL * NT * 8 == C::L, "runs must tile the row");
    extern __shared__ uint4 lds4[];
    uint32_t* xb = reinterpret_cast<uint32_t*>(lds4);
    uint4* t1f = lds4 + C::XWORDS / 4;
    uint4* t1i = t1f + C::TC * 4;
    uint32_t* vt = reinterpret_cast<uint32_t*>(t1i + C::TC * 4);      // [TC][16]: w_L^(k_a t) W^t
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    const unsigned G = gridDim.x;
    const unsigned vid = (G & 7u) ? blockIdx.x : (blockIdx.x & 7u) * (G >> 3) + (blockIdx.x >> 3);
    // work items (head, row), `per` consecutive ones per workgroup (a head's rows share its spectrum)
    const int nrow = (int)B, total = (int)H * nrow;
    const int it0 = (int)vid * per, it1 = it0 + per < total ? it0 + per : total;
    const uint4* gtab = reinterpret_cast<const uint4*>(ctab + coop_tab_offset(LG));

    auto run_n = [&](int i) { return staged_run_n<LG>(i * NT + tid); };
    uint4 pa[RPL];
    // quarter Q of a row's runs; without a row (an empty descriptor) the requests go out all the same and ask for nothing, so that
    // they are in one stream with the rest
    auto fetch = [&](int it, bool any, auto q) __attribute__((always_inline)) {
        constexpr int Q = decltype(q)::value;
        const typename IO::T* p = in + row_off(it % nrow, it / nrow, H, C::L);
        const __amdgpu_buffer_rsrc_t d = __builtin_amdgcn_make_buffer_rsrc(const_cast<typename IO::T*>(p), 0, any ? C::L * 2 : 0, 0x00027000);
#pragma unroll
        for (int i = Q * RPL / 4; i < (Q + 1) * RPL / 4; ++i)
            pa[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(d, 2 * run_n(i), 0, 0));
        asm volatile("; %0" :: "n"(Q));         // (the quarters' code is not to be merged: their registers would be in memory)
    };
    const std::integral_constant<int, 0> q0;
    const std::integral_constant<int, 1> q1;
    const std::integral_constant<int, 2> q2;
    const std::integral_constant<int, 3> q3;
    if (it0 < it1) {                 // the first row is on its way while the constants are built
        fetch(it0, true, q0); fetch(it0, true, q1); fetch(it0, true, q2); fetch(it0, true, q3);
    }

    Consts<LG> K;
    make_consts<LG>(K, tw, lane);
    const Mats F1 = phase_mats(1, C::cb + 4, LG + 2, tw, lane);
    h8 I3;                           // conjugate of the same entries, real part of the product only; d_a on the lanes
    h2 c1[4], c3[4];                 // w_256^(k_a d_b) W^(d_b TC): d_b = 4g+j in phase 1, d_b = c in phase 3
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t y = (uint32_t)(4 * g + j);
        const float2 a = tw_full(tw, ((((c * y) & 15u) << (TW_LOG2 - 4)) + ((uint32_t)c << (TW_LOG2 - 6))) & (TW_L - 1));
        I3[2 * j] = (_Float16)(a.x * 0.5f);          // 2/4: N points where the spectrum's scale has 1/2N
        I3[2 * j + 1] = (_Float16)(a.y * 0.5f);
        const uint32_t b = ((c * y) & 255u) << (TW_LOG2 - 8);
        const float2 w1 = tw_full(tw, (b + (y << (TW_LOG2 - 10))) & (TW_L - 1));
        const float2 w3 = tw_full(tw, (b + ((uint32_t)c << (TW_LOG2 - 10))) & (TW_L - 1));
        c1[j] = h2{(_Float16)w1.x, (_Float16)w1.y};
        c3[j] = h2{(_Float16)w3.x, (_Float16)w3.y};
    }
    int ng = C::TC / (8 * NWV);
    asm volatile("" : "+s"(ng));
    const int w1 = (c * C::PITCH + g * C::TC) * 4;

    // bf16 rows outside the band are scaled by a power of two
    __shared__ uint32_t dr_mx[NWV];
    // word of sample e of run i: pairs of samples change places by the low bits of the run's t / 8
    int sl[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) sl[e] = staged_slot<LG>(run_n(0)) + 8 * (e ^ ((run_n(0) >> 3) & 3));
    auto slot = [&](int i, int e) { return sl[e >> 1] + (e & 1) * 4 + staged_slot<LG>(run_step<LG>(i * NT)); };
    auto measure = [&]() {
        uint32_t m[1] = {0u};
#pragma unroll
        for (int i = 0; i < RPL; ++i)
            m[0] = absmax_acc(absmax_acc(absmax_acc(absmax_acc(m[0], pa[i].x), pa[i].y), pa[i].z), pa[i].w);
        band_or_exact<1>(m);
        if (lane == 0) dr_mx[wave] = m[0];
    };
    auto stage = [&](int ea) {
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            uint32_t wa[4] = {pa[i].x, pa[i].y, pa[i].z, pa[i].w};
            if (IsBf<IO>::v) {
#pragma unroll
                for (int m = 0; m < 4; ++m) wa[m] = __builtin_expect(ea != 0, 0) ? bf2_to_h2_scaled(wa[m], ea) : bf2_to_h2(wa[m]);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                xb[slot(i, 2 * m)] = wa[m] & 0xffffu;
                xb[slot(i, 2 * m + 1)] = wa[m] >> 16;
            }
        }
    };
    auto drain = [&](int it, int ea) {
        const size_t o = row_off(it % nrow, it / nrow, H, C::L);
        uint4 ga[GATE ? RPL : 1];
        if constexpr (GATE) {
#pragma unroll
            for (int i = 0; i < RPL; ++i) ga[i] = *reinterpret_cast<const uint4*>(gate + o + run_n(i));
        }
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            const int n = run_n(i);
            uint32_t wa[4];
            if constexpr (GATE) {                        // fp32 samples: gate and power of two, then one rounding
                float x[8];
                const uint32_t gw[4] = {ga[i].x, ga[i].y, ga[i].z, ga[i].w};
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    union { uint32_t u; h2 h; } q;
                    q.u = gw[m];
                    x[2 * m] = __uint_as_float(xb[slot(i, 2 * m)]) * (IsBf<IO>::v ? __uint_as_float(gw[m] << 16) : (float)q.h[0]);
                    x[2 * m + 1] = __uint_as_float(xb[slot(i, 2 * m + 1)]) *
                                   (IsBf<IO>::v ? __uint_as_float(gw[m] & 0xffff0000u) : (float)q.h[1]);
                }
                if (__builtin_expect(ea != 0, 0)) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = ldexpf(x[e], ea);
                }
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    wa[m] = IsBf<IO>::v ? pack_bf2(x[2 * m], x[2 * m + 1]) : pack_h2(x[2 * m], x[2 * m + 1]);
            } else {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    union { uint32_t u; h2 h; } a;
                    a.u = __builtin_amdgcn_perm(xb[slot(i, 2 * m + 1)], xb[slot(i, 2 * m)], 0x05040100u);
                    wa[m] = IsBf<IO>::v ? pack_bf2((float)a.h[0], (float)a.h[1]) : a.u;
                }
                if (__builtin_expect(ea != 0, 0)) {
#pragma unroll
                    for (int m = 0; m < 4; ++m) wa[m] = out_rescaled<IsBf<IO>::v>(wa[m], ea);
                }
            }
            put_once(reinterpret_cast<uint4*>(out + o + n), make_uint4(wa[0], wa[1], wa[2], wa[3]));
        }
    };

    staged_tables<LG, NT>(lds4, gtab, tw, tid, 0);
    for (int i = tid; i < C::TC * 16; i += NT) {         // (a lane rewrites the entries it wrote itself)
        const uint32_t t = (uint32_t)i >> 4;
        const float2 w = tw_full(tw, (((((uint32_t)i & 15u) * t) << (TW_LOG2 - LG)) + (t << (TW_LOG2 - LG - 2))) & (TW_L - 1));
        vt[i] = pack_h2(w.x, w.y);
    }
    __syncthreads();
    if (it0 < it1) {
        if constexpr (IsBf<IO>::v) measure();
        stage(0);
    }
    for (int it = it0; it < it1; ++it) {
        const int h = __builtin_amdgcn_readfirstlane(it / nrow);
        const uint4* ks = reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(kspec) + (size_t)h * C::L);
        asm volatile("" : "+s"(ks));
        const int es = spec_exp_of(kspec, H, 2 * (int64_t)C::L)[h];
        __syncthreads();             // staged row visible
        int ea = 0;
        if constexpr (IsBf<IO>::v) {
            uint32_t ma = 0u;
#pragma unroll
            for (int w = 0; w < NWV; ++w) ma = max(ma, dr_mx[w]);
            ma = (uint32_t)__builtin_amdgcn_readfirstlane((int)ma);
            if (__builtin_expect(!rows_in_band(ma, ma), 0)) {
                int eb = 0;
                pair_exponents(ma, 0u, ea, eb);
                if (ea != 0) {
                    stage(ea);
                    __syncthreads();
                }
            }
        }
        const bool more = RUNS && it + 1 < it1;

        // ---- phase 1, in place.  The next row is asked for piece by piece: asked for at once, the requests of eight waves held the
        // later four of them back by some 2500 cycles of 33000 per row, and the others at the barrier (forward, B=32, H=128 fp16
        // 246 -> 241 us, B=7, H=193 bf16 110.0 -> 105.1, fp16 107.0 -> 102.8).  RUNS: there are workgroups with a second row; with one
        // each, the requests that ask for nothing cost 0.1 to 0.3 us (fp16, B=1, H=128 26.3 and, without, 26.0; bf16, B=2, H=64 26.4 and
        // 26.3; with the gate they cost nothing, 33.9 and 34.2 at B=2, H=128, and that kernel has no such form).
        static_assert(C::TC == 16 * NWV && NB == 4 && RPL % 4 == 0, "two groups of two batches of tiles per wave");
        const int next = more ? it + 1 : it;
        phase1_inplace<LG, NB, true>(xb, t1f, vt, F1, K.F16, c1, wave * 8, lane, [&](int b) __attribute__((always_inline)) {
            if (RUNS && b == 0) fetch(next, more, q0);
            else if (RUNS) fetch(next, more, q1);
        });
        phase1_inplace<LG, NB, true>(xb, t1f, vt, F1, K.F16, c1, (NWV + wave) * 8, lane, [&](int b) __attribute__((always_inline)) {
            if (RUNS && b == 0) fetch(next, more, q2);
            else if (RUNS) fetch(next, more, q3);
        });
        __syncthreads();
        asm volatile("" : "+s"(ks));

        // ---- phase 2
#pragma unroll 1
        for (int gi = 0; gi < ng; ++gi) {
            const int t0 = (gi * NWV + wave) * 8;
            // this lane's words d_c = 4g + j of tile t0; tile t0 + k: phase2_step(k) on
            int at[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) at[j] = phase2_base<LG>(t0, lane) + j * C::TE * 4 + 4 * (((c & 7) ^ (2 * j)) - (c & 7));
#pragma unroll
            for (int tb = 0; tb < 8; tb += NB) {
                f4 zr[NB], zi[NB];
                H8U kk[NB];
#pragma unroll
                for (int k = 0; k < NB; ++k) kk[k].u = ks[(t0 + tb + k) * 64 + lane];
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    H8U x;
#pragma unroll
                    for (int j = 0; j < 4; ++j) x.w[j] = xb[at[j] + phase2_step<LG>(tb + k)];
                    phase2_fwd<LG>(x, K, zr[k], zi[k]);
                }
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    H8U m, o;
#pragma unroll
                    for (int j = 0; j < 4; ++j)      // correlation (du): the conjugate spectrum
                        m.w[j] = CONJ ? cmul_pack_conj(zr[k][j], zi[k][j], kk[k].c[j])
                                      : cmul_pack(zr[k][j], zi[k][j], kk[k].c[j]);
                    phase2_inv_regs<LG>(K, m, o);
#pragma unroll
                    for (int j = 0; j < 4; ++j) xb[at[j] + phase2_step<LG>(tb + k)] = o.w[j];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();

        // ---- phase 3, in place, real part only: samples (d_a, d_b) = (4g+j, c) of each tile.  Samples that
        // meet a gate fill their slots in fp32: gate and power of two come before the one rounding, to the I/O dtype.
#pragma unroll 1
        for (int gi = 0; gi < ng; ++gi) {
            const int t0 = (gi * NWV + wave) * 8;
            const f4 zero = {0.f, 0.f, 0.f, 0.f};
            int at[4];
            tile_places<LG, true>(at, w1, t0);
#pragma unroll
            for (int tb = 0; tb < 8; tb += 2) {
                H8U tw1[2], x[2], vv[2];
                f4 yr[2], yi[2], r[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int t = t0 + tb + k;
                    tw1[k].u = t1i[t * 4 + g];
                    x[k].u = *reinterpret_cast<const uint4*>(&xb[at[(tb + k) >> 1] + ((tb + k) & 1) * 4]);
                    vv[k].u = *reinterpret_cast<const uint4*>(&vt[t * 16 + 4 * g]);
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[k].w[j] = cmul_h2(x[k].w[j], tw1[k].c[j]);
                    yr[k] = MFMA(x[k].v, K.I16.re, zero);
                    yi[k] = MFMA(x[k].v, K.I16.im, zero);
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    H8U u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) u.w[j] = cmul_pack_conj(yr[k][j], yi[k][j], cmul_hh(c3[j], vv[k].c[j]));
                    r[k] = MFMA(I3, u.v, zero);
                }
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if constexpr (GATE)
                        *reinterpret_cast<f4*>(&xb[at[(tb + k) >> 1] + ((tb + k) & 1) * 4]) = r[k];
                    else
                        *reinterpret_cast<uint4*>(&xb[at[(tb + k) >> 1] + ((tb + k) & 1) * 4]) = make_uint4(
                            pack_h2(r[k][0], 0.f), pack_h2(r[k][1], 0.f), pack_h2(r[k][2], 0.f), pack_h2(r[k][3], 0.f));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        drain(it, ea + es);          // (the lane that drains a slot stages the next row's sample there)
        if (more) {
            if constexpr (IsBf<IO>::v) measure();
            stage(0);
        }
        if (!RUNS) break;
    }
}

template <int LG, int NWV, int NB, bool CONJ>
__global__ void __launch_bounds__(NWV * 64) __attribute__((amdgpu_waves_per_eu(2)))
coop_conv_kernel(const float2* __restrict__ kspec, __half2* __restrict__ ws, int npairs, int log2R, int total, int per,
                 const float2* __restrict__ tw, const unsigned char* __restrict__ ctab)
{
    using C = CC<LG>;
    constexpr int NT = NWV * 64;
    constexpr int RPL = (C::L / 4) / NT;             // 16-byte runs per lane
    extern __shared__ uint4 lds4[];
    uint32_t* xb = reinterpret_cast<uint32_t*>(lds4);
    uint4* t1f = lds4 + C::XWORDS / 4;
    uint4* t1i = t1f + C::TC * 4;
    uint32_t* vt = reinterpret_cast<uint32_t*>(t1i + C::TC * 4);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    const unsigned G = gridDim.x;
    const unsigned vid = (G & 7u) ? blockIdx.x : (blockIdx.x & 7u) * (G >> 3) + (blockIdx.x >> 3);
    const int it0 = (int)vid * per, it1 = it0 + per < total ? it0 + per : total;
    const int64_t Ltot = (int64_t)C::L << log2R;
    const uint4* gtab = reinterpret_cast<const uint4*>(ctab + coop_tab_offset(LG));
    Consts<LG> K;
    make_consts<LG>(K, tw, lane);
    h2 cF[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 w = tw_full(tw, (uint32_t)((c * (4 * g + j)) & 255) << (TW_LOG2 - 8));
        cF[j] = h2{(_Float16)w.x, (_Float16)w.y};
    }
    int ng = C::TC / (8 * NWV);
    asm volatile("" : "+s"(ng));
    const int w1 = (c * C::PITCH + g * C::TC) * 4;

    auto run_n = [&](int i) { return chunk_run_n<LG>(i * NT + tid); };
    // items (head, chunk k1, pair)
    const int nch = 1 << log2R;
    auto chunk_of = [&](int it) {
        const int hk = it / npairs, p = it - hk * npairs;
        const int h = hk / nch, k1 = hk - h * nch;
        return ws + ((size_t)h * npairs + p) * Ltot + (size_t)k1 * C::L;
    };
    auto stage = [&](int it) {
        const uint4* src = reinterpret_cast<const uint4*>(chunk_of(it));
#pragma unroll
        for (int i0 = 0; i0 < RPL; i0 += 4) {
            uint4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = src[run_n(i0 + i) / 4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int a0 = staged_slot<LG>(run_n(i0 + i));
                xb[a0] = v[i].x; xb[a0 + 4] = v[i].y; xb[a0 + 8] = v[i].z; xb[a0 + 12] = v[i].w;
            }
        }
    };
    auto drain = [&](int it) {
        uint4* dst = reinterpret_cast<uint4*>(chunk_of(it));
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            const int n = run_n(i), a0 = staged_slot<LG>(n);
            dst[n / 4] = make_uint4(xb[a0], xb[a0 + 4], xb[a0 + 8], xb[a0 + 12]);
        }
    };

    staged_tables<LG, NT>(lds4, gtab, tw, tid, 0);
    __syncthreads();
    if (it0 < it1) stage(it0);
    for (int it = it0; it < it1; ++it) {
        const int hk = it / npairs, hh = hk / nch;
        const uint4* ks = reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(kspec) +
                                                         (size_t)hh * Ltot + (size_t)(hk - hh * nch) * C::L);
        __syncthreads();             // staged chunk visible

        // ---- phase 1, in place
#pragma unroll 1
        for (int gi = 0; gi < ng; ++gi)
            phase1_inplace<LG, NB>(xb, t1f, vt, K.F16, K.F16, cF, (gi * NWV + wave) * 8, lane);
        __syncthreads();

        // ---- phase 2
#pragma unroll 1
        for (int gi = 0; gi < ng; ++gi)
#pragma unroll
        for (int tb = 0; tb < 8; tb += NB) {
            const int t0 = (gi * NWV + wave) * 8;
            int base[NB];
            f4 zr[NB], zi[NB];
            H8U kk[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int t2 = t0 + tb + k;
                base[k] = phase2_base<LG>(t2, lane);
                kk[k].u = ks[t2 * 64 + lane];
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) phase2_fwd<LG>(xb, base[k], K, zr[k], zi[k]);
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                H8U m;
#pragma unroll
                for (int j = 0; j < 4; ++j)      // correlation (du): the conjugate spectrum
                    m.w[j] = CONJ ? cmul_pack_conj(zr[k][j], zi[k][j], kk[k].c[j])
                                  : cmul_pack(zr[k][j], zi[k][j], kk[k].c[j]);
                phase2_inv<LG>(xb, base[k], K, m);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();

        // ---- phase 3, in place
#pragma unroll 1
        for (int gi = 0; gi < ng; ++gi) {
            const int t0 = (gi * NWV + wave) * 8;
#pragma unroll
            for (int tb = 0; tb < 8; tb += 2) {
                f4 r[2], s2[2];
                phase3_two_lds<LG>(xb, t1i, vt, K, cF, t0 + tb, lane, r, s2);
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    *reinterpret_cast<uint4*>(&xb[w1 + 4 * (t0 + tb + k)]) =
                        make_uint4(pack_h2(r[k][0], s2[k][0]), pack_h2(r[k][1], s2[k][1]),
                                   pack_h2(r[k][2], s2[k][2]), pack_h2(r[k][3], s2[k][3]));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        drain(it);
        if (it + 1 < it1) stage(it + 1);
    }
}

// -------------------------------------------------------------------------------------
// dk and dD of the multi-pass split: one workgroup per (head, chunk k1) loops over all row pairs of the
// head in order, reading chunk k1 of pass A's outputs.  Per pair: Z = transform of the u chunk (kept as
// fp16 in registers), W = transform of the dy chunk, A += conj(Z) W in fp32 registers, in the lane order
// of phase 2; then the inverse half of phase 2 and phase 3 give the chunk that pass C turns into dk.  A wave holds Z and A for 8 phase-2 tiles at a time.
// With NG > 1 tile groups per wave (L = 32768) the batch is walked once per group (the second
// walk finds its rows in cache), and the inverse half-spectrum of every group but the last is
// parked in the caller's workspace (`zbuf`, written and read once per head) until phase 3:
// registers for all groups at once do not exist, and parking Z per pair instead costs an order
// of magnitude more memory traffic than the second walk.
// -------------------------------------------------------------------------------------
template <int LG>
__global__ void __launch_bounds__(CC<LG>::NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
coop_dk_kernel(const __half2* __restrict__ ws_u, const __half2* __restrict__ ws_dy, __half2* __restrict__ ws_A,
               float* __restrict__ dD_part, uint4* __restrict__ zbuf, int npairs, int log2R, float dDscale,
               const float2* __restrict__ tw, const unsigned char* __restrict__ ctab)
{
    using C = CC<LG>;
    constexpr int NB = 2;      // phase-1 tiles in flight (the accumulators leave no room for more)
    extern __shared__ uint4 lds4[];
    __shared__ float red[C::NW];
    uint32_t* xb = reinterpret_cast<uint32_t*>(lds4);
    uint4* t1f = lds4 + C::XWORDS / 4;
    uint4* t1i = t1f + C::TC * 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    const int h = blockIdx.x, k1 = blockIdx.y;
    const int64_t Ltot = (int64_t)C::L << log2R;
    const uint4* gtab = reinterpret_cast<const uint4*>(ctab + coop_tab_offset(LG));
    for (int i = tid; i < C::TC * 8; i += C::NW * 64) t1f[i] = gtab[C::T1F + i];
    Consts<LG> K;
    make_consts<LG>(K, tw, lane);
    __syncthreads();
    uint4* zb = zbuf + ((size_t)h * gridDim.y + k1) * (C::TC * 64) + lane;
    int ng = C::NG;
    asm volatile("" : "+s"(ng));       // opaque trip count: one copy of the loop bodies (register pressure)
    float dsum = 0.f;

    for (int gi = 0; gi < ng; ++gi) {
        const int t2_0 = (gi * C::NW + wave) * 8;      // this wave's 8 phase-2 tiles of the group
        float2 acc[8][4];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = make_float2(0.f, 0.f);

        for (int p = 0; p < npairs; ++p) {
            asm volatile("" : "+s"(gtab));
            const size_t coff = ((size_t)h * npairs + p) * Ltot + (size_t)k1 * C::L;
            uint32_t z[8][4];
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {     // 0: u pair -> Z, 1: dy pair -> W
                asm volatile("" : "+s"(gtab));
                const __half2* csrc = pass == 0 ? ws_u : ws_dy;
#pragma unroll 1
                for (int g2 = 0; g2 < ng; ++g2) {
                    phase1<LG, NB>(csrc + coff, xb, gtab, t1f, K, (g2 * C::NW + wave) * 8, lane);
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    f4 zr, zi;
                    phase2_fwd<LG>(xb, phase2_base<LG>(t2_0 + i, lane), K, zr, zi);
                    if (pass == 0) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) z[i][j] = pack_h2(zr[j], zi[j]);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            union { uint32_t u; h2 hh; } cv;
                            cv.u = z[i][j];
                            const float a = (float)cv.hh[0], b = (float)cv.hh[1];
                            // conj(Z) * W, one fused multiply-add per term
                            acc[i][j].x = __builtin_fmaf(b, zi[j], __builtin_fmaf(a, zr[j], acc[i][j].x));
                            acc[i][j].y = __builtin_fmaf(-b, zr[j], __builtin_fmaf(a, zi[j], acc[i][j].y));
                        }
                    }
                    if (i & 1) __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
            }
        }

#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) dsum += acc[i][j].x;
        if (ws_A) {
            // inverse half of phase 2: the last group goes to the exchange buffer, earlier ones are parked
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                H8U m;
#pragma unroll
                for (int j = 0; j < 4; ++j) m.w[j] = pack_h2(acc[i][j].x, acc[i][j].y);
                if (gi + 1 < ng) {
                    H8U v;
                    phase2_inv_regs<LG>(K, m, v);
                    zb[(size_t)(t2_0 + i) * 64] = v.u;
                } else {
                    phase2_inv<LG>(xb, phase2_base<LG>(t2_0 + i, lane), K, m);
                }
            }
        }
    }

    if (dD_part) {
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
        if (lane == 0) red[wave] = dsum;
        __syncthreads();
        if (tid == 0) {
            float t = 0.f;
            for (int w = 0; w < C::NW; ++w) t += red[w];
            dD_part[(size_t)h * gridDim.y + k1] = t * dDscale;
        }
    }
    if (!ws_A) return;

    // parked groups back into the exchange buffer (each lane reads what it wrote itself)
    for (int gi = 0; gi + 1 < ng; ++gi)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t2 = (gi * C::NW + wave) * 8 + i;
            H8U v;
            v.u = zb[(size_t)t2 * 64];
            const int base = phase2_base<LG>(t2, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) xb[base + j * C::TE * 4] = v.w[j];
        }
    __syncthreads();
    __half2* achunk = ws_A + (size_t)h * Ltot + (size_t)k1 * C::L;
#pragma unroll 1
    for (int gi = 0; gi < ng; ++gi) {
        const int t0 = (gi * C::NW + wave) * 8;
        // 8 tiles = 8 consecutive samples per (lane, j): stored as 32-byte runs
        uint32_t oc[4][8];     // fp16 complex words
#pragma unroll
        for (int tb = 0; tb < 8; tb += 2) {
            f4 r[2], s[2];
            phase3_two<LG>(xb, gtab, t1i, K, t0 + tb, lane, r, s);
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    oc[j][tb + k] = pack_h2(r[k][j], s[k][j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n0 = (4 * g + j) * 16 * C::TC + c * C::TC + t0;
            uint4* dst = reinterpret_cast<uint4*>(achunk + n0);
            dst[0] = make_uint4(oc[j][0], oc[j][1], oc[j][2], oc[j][3]);
            dst[1] = make_uint4(oc[j][4], oc[j][5], oc[j][6], oc[j][7]);
        }
    }
}

// -------------------------------------------------------------------------------------
// Kernel spectrum of a multi-pass split from a pass-A workspace, for the chained kernels' lane order.
// grid = (H, R): chunk k1 of the pass-A output of the kernel pre-scaled by a power of two from rs[h] (the
// head's maximum; pass A used the same scale).  Phase 1 and the forward half of phase 2 as in the
// convolution; value stored = kscale * (FFT([k,0]) + D[h]) as fp16 complex (one 32-bit word per bin).
// (coop_kspec_rows_kernel below reads k itself, where the plan takes pass A inside.)
// -------------------------------------------------------------------------------------
template <int LG>
__global__ void __launch_bounds__(CC<LG>::NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
coop_kspec_kernel(const __half2* __restrict__ ws, const float* __restrict__ D, const float* __restrict__ rs,
                  float2* __restrict__ kspec, int log2R, float kscale_over_c, float kscale,
                  const float2* __restrict__ tw, const unsigned char* __restrict__ ctab)
{
    using C = CC<LG>;
    extern __shared__ uint4 lds4[];
    uint32_t* xb = reinterpret_cast<uint32_t*>(lds4);
    uint4* t1f = lds4 + C::XWORDS / 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int h = blockIdx.x, k1 = blockIdx.y;
    const int64_t Ltot = (int64_t)C::L << log2R;
    const uint4* gtab = reinterpret_cast<const uint4*>(ctab + coop_tab_offset(LG));
    for (int i = tid; i < C::TC * 8; i += C::NW * 64) t1f[i] = gtab[C::T1F + i];
    Consts<LG> K;
    make_consts<LG>(K, tw, lane);
    const float r = head_scale_of(rs[h]);
    const __half2* chunk = ws + (size_t)h * Ltot + (size_t)k1 * C::L;
    __syncthreads();
#pragma unroll
    for (int gi = 0; gi < C::NG; ++gi) {
        phase1<LG>(chunk, xb, gtab, t1f, K, (gi * C::NW + wave) * 8, lane);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // rs: [0, H) the heads' maxima, [H, 2H) and [2H, 3H) the bounds on their largest spectrum bin
    const int es = spec_exponent(kscale * rs[gridDim.x + h], kscale * rs[2 * gridDim.x + h]);
    if (k1 == 0 && tid == 0) spec_exp_of(kspec, gridDim.x, Ltot)[h] = es;
    const float alpha = ldexpf(kscale_over_c / r, -es), beta = ldexpf(D[h] * kscale, -es);
    uint4* out = reinterpret_cast<uint4*>(reinterpret_cast<uint32_t*>(kspec) + (size_t)h * Ltot + (size_t)k1 * C::L);
#pragma unroll
    for (int gi = 0; gi < C::NG; ++gi)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t2 = (gi * C::NW + wave) * 8 + i;
            f4 zr, zi;
            phase2_fwd<LG>(xb, phase2_base<LG>(t2, lane), K, zr, zi);
            out[t2 * 64 + lane] = make_uint4(pack_h2(zr[0] * alpha + beta, zi[0] * alpha), pack_h2(zr[1] * alpha + beta, zi[1] * alpha),
                                             pack_h2(zr[2] * alpha + beta, zi[2] * alpha), pack_h2(zr[3] * alpha + beta, zi[3] * alpha));
        }
}

// Kernel spectrum of rows of N = 2^LG samples (coop_conv_row_kernel), staged form, one workgroup per head: the row stays in
// registers between the search of the head's maximum (power-of-two pre-scale) and the conversion, one round trip to memory;
// phase 1 runs in place with the twist in its operands, the forward half of phase 2 writes kscale (FFT + D[h]).
template <int LG>
__global__ void __launch_bounds__(CC<LG>::NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
coop_kspec_rows_kernel(const float* __restrict__ k, const float* __restrict__ D, float2* __restrict__ kspec, float kscale_over_c,
                       float kscale,
                       const float2* __restrict__ tw, const unsigned char* __restrict__ ctab)
{
    using C = CC<LG>;
    constexpr int NT = C::NW * 64;
    constexpr int RPA = (C::L / 8) / NT;                 // runs of eight samples per lane
    extern __shared__ uint4 lds4[];
    __shared__ float mred[3][C::NW];
    uint32_t* xb = reinterpret_cast<uint32_t*>(lds4);
    uint4* t1f = lds4 + C::XWORDS / 4;
    uint4* t1i = t1f + C::TC * 4;
    uint32_t* vt = reinterpret_cast<uint32_t*>(t1i + C::TC * 4);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4;
    const unsigned G = gridDim.x;
    const int h = (int)((G & 7u) ? blockIdx.x : (blockIdx.x & 7u) * (G >> 3) + (blockIdx.x >> 3));
    const uint4* gtab = reinterpret_cast<const uint4*>(ctab + coop_tab_offset(LG));
    const float* kr = k + (size_t)h * C::L;

    // the row starts travelling first; tables and operands are built behind it (their loads return after
    // the row's, so one round trip to memory covers everything)
    float4 v[RPA][2];
#pragma unroll
    for (int i = 0; i < RPA; ++i) {
        const float4* src = reinterpret_cast<const float4*>(kr + staged_run_n<LG>(i * NT + tid));
        v[i][0] = src[0];
        v[i][1] = src[1];
    }
    const float Dh = D[h];
    staged_tables<LG, NT>(lds4, gtab, tw, tid, 0);
    twisted_t1f<LG, 2, NT>(t1f, gtab, 1, tw, tid);       // (a lane rewrites the entries it wrote itself)
    // constants of the transform (table look-ups in global memory)
    Consts<LG> K;
    make_consts<LG>(K, tw, lane);
    h2 cF[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 w = tw_full(tw, (uint32_t)((c * (4 * g + j)) & 255) << (TW_LOG2 - 8));
        cF[j] = h2{(_Float16)w.x, (_Float16)w.y};
    }
    const Mats F1 = phase_mats(1, C::cb + 4, LG + 2, tw, lane), F2 = phase_mats(1, C::cb, LG + 2, tw, lane);
    // the head's largest magnitude; a, mp: sum and maximum of the magnitudes with the skip term counted in the lag-0 tap
    // (run 0 of lane 0 starts at k_0), the two bounds on the head's largest spectrum bin (spec_exponent)
    float m = 0.f, a = 0.f, mp = 0.f;
#pragma unroll
    for (int i = 0; i < RPA; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float4 x = v[i][q];
            m = fmaxf(m, fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w))));
            const float x0 = fabsf(x.x + (i == 0 && q == 0 && tid == 0 ? Dh : 0.f));
            a += (x0 + fabsf(x.y)) + (fabsf(x.z) + fabsf(x.w));
            mp = fmaxf(mp, fmaxf(fmaxf(x0, fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w))));
        }
    for (int o = 32; o > 0; o >>= 1) {
        m = fmaxf(m, __shfl_xor(m, o, 64));
        mp = fmaxf(mp, __shfl_xor(mp, o, 64));
        a += __shfl_xor(a, o, 64);
    }
    if (lane == 0) { mred[0][wave] = m; mred[1][wave] = a; mred[2][wave] = mp; }
    __syncthreads();                                     // (also covers the cleared slots)
    m = mred[0][0]; a = mred[1][0]; mp = mred[2][0];
    for (int w = 1; w < C::NW; ++w) { m = fmaxf(m, mred[0][w]); a += mred[1][w]; mp = fmaxf(mp, mred[2][w]); }
    const float r = head_scale_of(m);
#pragma unroll
    for (int i = 0; i < RPA; ++i) {
        const int a0 = staged_slot<LG>(staged_run_n<LG>(i * NT + tid));
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float4 q = v[i][e >> 2];
            const float x = ((e & 3) == 0 ? q.x : (e & 3) == 1 ? q.y : (e & 3) == 2 ? q.z : q.w) * r;
            xb[a0 + 4 * e] = pack_h2(x, 0.f);
        }
    }

    __syncthreads();
#pragma unroll 1
    for (int gi = 0; gi < C::NG; ++gi) phase1_inplace<LG, 2>(xb, t1f, vt, F1, F2, cF, (gi * C::NW + wave) * 8, lane);
    __syncthreads();
    const int es = spec_exponent(kscale * a, kscale * mp);
    if (tid == 0) spec_exp_of(kspec, G, (int64_t)C::L * 2)[h] = es;
    const float alpha = ldexpf(kscale_over_c / r, -es), beta = ldexpf(Dh * kscale, -es);
    uint4* out = reinterpret_cast<uint4*>(reinterpret_cast<uint32_t*>(kspec) + (size_t)h * C::L);
#pragma unroll 1
    for (int gi = 0; gi < C::NG; ++gi)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t2 = (gi * C::NW + wave) * 8 + i;
            f4 zr, zi;
            phase2_fwd<LG>(xb, phase2_base<LG>(t2, lane), K, zr, zi);
            out[t2 * 64 + lane] = make_uint4(pack_h2(zr[0] * alpha + beta, zi[0] * alpha), pack_h2(zr[1] * alpha + beta, zi[1] * alpha),
                                             pack_h2(zr[2] * alpha + beta, zi[2] * alpha), pack_h2(zr[3] * alpha + beta, zi[3] * alpha));
        }
}

template <int LG>
size_t coop_lds_bytes() { return (size_t)CC<LG>::XWORDS * 4 + (size_t)CC<LG>::TC * 8 * 16; }

template <int LG, class IO, bool CONJ, bool GATE, bool RUNS>
hipError_t coop_conv_row_launch(const void* in, const float2* kspec, void* out, int per, const Problem& pr, const Tables& tb,
                                hipStream_t st)
{
    using T = typename IO::T;
    constexpr int NWV = CC<LG>::NW;
    const auto kern = coop_conv_row_kernel<LG, IO, NWV, NTB, CONJ, GATE, RUNS>;
    const size_t lds = coop_staged_lds_bytes<LG>();
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const long total = pr.H * pr.B;                      // (head, row) items; the row fills a compute unit's LDS
    hipLaunchKernelGGL(kern, dim3((unsigned)((total + per - 1) / per)), dim3(NWV * 64), lds, st, (const T*)in, kspec, (T*)out,
                       (const T*)pr.gate, pr.B, pr.H, per, tb.tw, (const unsigned char*)tb.ctab);
    return hipGetLastError();
}
template <int LG, class IO, bool CONJ, bool GATE>
hipError_t coop_conv_row_go(const void* in, const float2* kspec, void* out, const Problem& pr, const Tables& tb,
                            hipStream_t st)
{
    const long cus = compute_units(), per = (pr.H * pr.B + cus - 1) / cus;
    return per > 1 || GATE ? coop_conv_row_launch<LG, IO, CONJ, GATE, true>(in, kspec, out, (int)per, pr, tb, st)
                           : coop_conv_row_launch<LG, IO, CONJ, GATE, GATE>(in, kspec, out, 1, pr, tb, st);
}

// rows, or the inner convolution of the multi-pass split in the workspace
template <int LG, class IO>
hipError_t coop_conv_go(const void* in, const float2* kspec, void* out, __half2* ws, bool conj, const Problem& pr, const Plan& pl,
                        const Tables& tb, hipStream_t st)
{
    constexpr int NWV = CC<LG>::NW, NB = NTB;
    if constexpr (LG == COOP_MAX_LOG2) {
        if (pl.row1) {
            if (pr.gate)
                return conj ? hipErrorInvalidValue : coop_conv_row_go<LG, IO, false, true>(in, kspec, out, pr, tb, st);
            return conj ? coop_conv_row_go<LG, IO, true, false>(in, kspec, out, pr, tb, st)
                        : coop_conv_row_go<LG, IO, false, false>(in, kspec, out, pr, tb, st);
        }
    }
    const size_t lds = coop_staged_lds_bytes<LG>();
    const long total = pr.H * ((long)pr.npairs << pl.log2R);          // (head, chunk, pair) items
    auto launch = [&](auto kern, int& resident) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        if (resident == 0) {
            int nb = 0;
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, NWV * 64, lds);
            if (e != hipSuccess) return e;
            resident = (nb > 0 ? nb : 1) * compute_units();
        }
        const int per = (int)((total + resident - 1) / resident);
        hipLaunchKernelGGL(kern, dim3((unsigned)((total + per - 1) / per)), dim3(NWV * 64), lds, st, kspec, ws, pr.npairs, pl.log2R,
                           (int)total, per, tb.tw, (const unsigned char*)tb.ctab);
        return hipGetLastError();
    };
    static int res[2] = {0, 0};
    return conj ? launch(coop_conv_kernel<LG, NWV, NB, true>, res[1]) : launch(coop_conv_kernel<LG, NWV, NB, false>, res[0]);
}

// multi-pass dk: chunks of pass A's outputs in, chunks for pass C and partial dD sums out
template <int LG>
hipError_t coop_dk_go(const __half2* ws_u, const __half2* ws_dy, __half2* ws_A, float* dD_part, void* zbuf,
                      const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
    using C = CC<LG>;
    const size_t lds = coop_lds_bytes<LG>();
    dim3 grid((unsigned)pr.H, 1u << pl.log2R);
    const int shift = 6 + (C::te >= 2 ? 1 : 0);      // three radix-16 stages (1/4 each) and F_TE
    const float dDscale = pl.dkscale / (float)(1 << shift);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(coop_dk_kernel<LG>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((coop_dk_kernel<LG>), grid, dim3(C::NW * 64), lds, st, ws_u, ws_dy, ws_A, dD_part, (uint4*)zbuf,
                       pr.npairs, pl.log2R, dDscale, tb.tw, (const unsigned char*)tb.ctab);
    return hipGetLastError();
}

template <int LG>
hipError_t coop_kspec_go(const float* k, const __half2* ws, const float* D, const float* rs, float2* kspec,
                         int64_t H, int64_t N, const Plan& pl, const Tables& tb, hipStream_t st)
{
    using C = CC<LG>;
    const size_t lds = coop_lds_bytes<LG>();
    dim3 grid((unsigned)H, 1u << pl.log2R);
    const int shift = 6 + (C::te >= 2 ? 1 : 0);
    const float koc = pl.kscale * (float)(1 << shift);
    if constexpr (LG == COOP_MAX_LOG2) {
        if (pl.row1) {                               // (ws and rs unused)
            const size_t lds_rows = coop_staged_lds_bytes<LG>();
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(coop_kspec_rows_kernel<LG>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_rows);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(coop_kspec_rows_kernel<LG>, dim3((unsigned)H), dim3(C::NW * 64), lds_rows, st, k, D, kspec, koc,
                               pl.kscale, tb.tw, (const unsigned char*)tb.ctab);
            return hipGetLastError();
        }
    }
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(coop_kspec_kernel<LG>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(coop_kspec_kernel<LG>, grid, dim3(C::NW * 64), lds, st, ws, D, rs, kspec, pl.log2R, koc,
                       pl.kscale, tb.tw, (const unsigned char*)tb.ctab);
    return hipGetLastError();
}

}  // namespace

hipError_t coop_conv(const void* in, const float2* kspec, void* out, __half2* ws, bool conj,
                     const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
#define GO(LG, IO) return coop_conv_go<LG, IO>(in, kspec, out, ws, conj, pr, pl, tb, st)
    if (pr.io == LONGCONV_F16) {
        if (pl.log2L2 == 13) GO(13, IoF16);
        if (pl.log2L2 == 14) GO(14, IoF16);
        if (pl.log2L2 == 15) GO(15, IoF16);
    } else if (pr.io == LONGCONV_BF16) {
        if (pl.log2L2 == 13) GO(13, IoBF16);
        if (pl.log2L2 == 14) GO(14, IoBF16);
        if (pl.log2L2 == 15) GO(15, IoBF16);
    }
#undef GO
    return hipErrorInvalidValue;
}

hipError_t coop_kspec(const float* k, const __half2* ws, const float* D, const float* rs, float2* kspec, int64_t H,
                      int64_t N, const Plan& pl, const Tables& tb, hipStream_t st)
{
    if (pl.log2L2 == 13) return coop_kspec_go<13>(k, ws, D, rs, kspec, H, N, pl, tb, st);
    if (pl.log2L2 == 14) return coop_kspec_go<14>(k, ws, D, rs, kspec, H, N, pl, tb, st);
    if (pl.log2L2 == 15) return coop_kspec_go<15>(k, ws, D, rs, kspec, H, N, pl, tb, st);
    return hipErrorInvalidValue;
}

hipError_t coop_dk(const void* dy, const void* u, float* dk, float* dD, int nsplit, const __half2* ws_u,
                   const __half2* ws_dy, __half2* ws_A, float* dD_part, void* zbuf, const Problem& pr, const Plan& pl,
                   const Tables& tb, hipStream_t st)
{
    // multi-pass: ws_A is null when only dD is wanted
    if (pl.log2L2 == 13) return coop_dk_go<13>(ws_u, ws_dy, dk ? ws_A : nullptr, dD_part, zbuf, pr, pl, tb, st);
    if (pl.log2L2 == 14) return coop_dk_go<14>(ws_u, ws_dy, dk ? ws_A : nullptr, dD_part, zbuf, pr, pl, tb, st);
    if (pl.log2L2 == 15) return coop_dk_go<15>(ws_u, ws_dy, dk ? ws_A : nullptr, dD_part, zbuf, pr, pl, tb, st);
    return hipErrorInvalidValue;
}

}  // namespace lc
