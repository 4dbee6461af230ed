// Matrix-core engine for single rows of N = 8192 and 16384 samples: spectrum, convolution (forward and du) and the whole backward
// pass, on the transform of engine_rows.hip (N points per row, twisted: products are convolutions modulo z^N - i).
//
// N = 16*16*16*TE, TC = 16 TE; n = d_a 16 TC + d_b TC + t, t = d_c TE + d_e; f = k_a + 16 k_b + 256 k_c + 4096 k_e.  A
// workgroup of TC / 8 waves owns one row at a time, whose points cross LDS twice per pair of transforms (see planar.hpp):
//   phase 1 (tile t, wave t / 8):       samples -[F16 over d_a, real input]-> * w_256^(k_a d_b) -[F16 over d_b]-> LDS
//   phase 2 (k_b, wave k_b NW / 16):    its TE tiles d_e: [F16 over d_c], [F_TE over d_e], * spectrum, and the mirror image -> LDS
//   phase 3 (tile t):                   [F16^-1 over k_b] * conj(w_256^(k_a d_b)) -[F16^-1 over k_a, real part]-> samples
// With two waves per SIMD these kernels run at about six cycles per instruction, whatever it is (the units could take one every 4.4, and
// matrix instructions of one wave beside the other's; two waves do not fill the waits), so what counts is how many there are.  All twiddles but one sit in the matrices: w_N^(k_a t) w_4N^t in the tile's own matrix over d_a (registers, eight
// tiles per wave), w_256^(k_b d_c) in the wave's matrices over d_c (registers), w_256TE^(d_e k_b) in the matrices over d_b and
// w_16TE^(d_e k_c) in those over d_e (few, shared by all waves: LDS).  The step over d_e contracts between tiles: for one k_c of
// every lane the TE tiles' numbers are a matrix operand as they lie, with K = (lane group, d_e) and a matrix that is block
// diagonal over the lane groups.
//
// Phases 1 and 3 meet a tile in the same wave, so phase 3 of one row and phase 1 of the next run as one part between two
// barriers on one exchange buffer; rows travel in 16-byte pieces through LDS, whose places for a row on its way in become those
// of a row on its way out: phase 3 writes the pieces that phase 1 of the same lane has read.
#include <type_traits>

#include "long_rows.hpp"

namespace lc {
namespace {
using namespace longrows;

static __device__ uint4 g_long_tab[LONG_TAB * 64];
template <int LG>
__global__ void fill_long_tab_kernel(uint4* tab)
{
    using L = LR<LG>;
    constexpr int TE = L::TE;
    const int unit = blockIdx.x, lane = threadIdx.x, o = lane & 15, g = lane >> 4;
    const double N = (double)L::N;
    union { _Float16 h[8]; uint4 u; } v;
    double re = 0.0, im = 0.0;
    const auto w = [&](double t, double sc) {        // exp(-2 pi i t), scaled
        double s, c;
        sincospi(-2.0 * t, &s, &c);
        re = c * sc;
        im = s * sc;
    };
    const auto a = [&](int ka, int da, int t) { w(da * ka / 16.0 + da / 64.0 + t * (4.0 * ka + 1.0) / (4.0 * N), 0.25); };
    const auto b = [&](int kb, int db, int de) { w(db * kb / 16.0 + db / 1024.0 + (double)(de * kb) / (256 * TE), 0.25); };
    const auto c = [&](int kc, int dc, int kb) { w(dc * kc / 16.0 + dc * kb / 256.0, 0.25); };
    // result q of unit m and lane group: (r, k_e), r = register; the same for slots (r, d_e)
    const auto e = [&](int m, int gq, int q, int gi, int i) {
        const int r = m * (4 / TE) + i / TE, de = i % TE, ke = q % TE;
        if (gq != gi || q / TE != i / TE) { re = im = 0.0; return; }
        w((double)(de * ke) / TE + (double)(de * (4 * gi + r)) / (16 * TE), 0.5);
    };
    // planar operand entry x of four: part 0 (re, -im) or 1 (im, re); conj: of the conjugate
    const auto put = [&](int x, int part, bool conj) {
        const double i2 = conj ? -im : im;
        v.h[x] = (_Float16)(part ? i2 : re);
        v.h[4 + x] = (_Float16)(part ? re : -i2);
    };
    if (unit >= L::U_S) {                            // [t][g]: four real parts, four imaginary parts
        const int i = (unit - L::U_S) * 64 + lane, t = i >> 2;
        for (int x = 0; x < 4; ++x) {
            w(t * (4.0 * (4 * (i & 3) + x) + 1.0) / (4.0 * N), 1.0);
            v.h[x] = (_Float16)re;
            v.h[4 + x] = (_Float16)im;
        }
        tab[(size_t)unit * 64 + lane] = v.u;
        return;
    }
    for (int x = 0; x < 4; ++x) {
        const int i = 4 * g + x;
        if (unit < L::U_AI) {
            a(o, i, unit);
            v.h[x] = (_Float16)re;
            v.h[4 + x] = (_Float16)im;
        } else if (unit < L::U_TW || unit == L::U_AP) {
            a(i, o, unit == L::U_AP ? 0 : unit - L::U_AI);
            re *= 2.0;
            im *= 2.0;
            put(x, 0, true);
        } else if (unit == L::U_TW) {
            w(o * i / 256.0, 1.0);
            v.h[x] = (_Float16)re;
            v.h[4 + x] = (_Float16)im;
        } else if (unit < L::U_CI) {
            c(o, i, (unit - L::U_C) >> 1);
            put(x, (unit - L::U_C) & 1, false);
        } else if (unit < L::U_LDS) {
            c(i, o, (unit - L::U_CI) >> 1);
            put(x, (unit - L::U_CI) & 1, true);
        } else {
            const int m = unit - L::U_LDS, k = (m % (2 * TE)) >> 1;
            if (m < L::U_BI) b(o, i, k);
            else if (m < L::U_E) b(i, o, k);
            else if (m < L::U_EI) e(k, o >> 2, o & 3, g, x);
            else e(k, g, x, o >> 2, o & 3);
            put(x, m & 1, m >= L::U_EI || (m >= L::U_BI && m < L::U_E));
        }
    }
    tab[(size_t)unit * 64 + lane] = v.u;
}

// -------------------------------------------------------------------------------------------------------------------
// Convolution (forward; CONJ: du) of all rows.  Persistent workgroups with even runs of consecutive (head, row) items, two
// barriers per row.  Bound by issue and waits of two waves per SIMD: per 256 points of a row 15 matrix and 64 vector instructions, at most
// 400 of the 790 cycles that a SIMD takes for them.
// B=8, H=256, N=16384 fp16: 83 us as pairs of rows in 32768-point transforms, 54 here; B=64, H=128, N=8192: 129, 91.  Four waves per
// SIMD with four tiles each (128 registers) were tried: 2 to 4 % faster at 16384, slower at 8192 and for few rows, and only with eight
// spilled registers or the tiles' factors rounded by themselves.
// -------------------------------------------------------------------------------------------------------------------
template <int LG, class IO, bool CONJ, bool GATE>
__global__ void __launch_bounds__(LR<LG>::NT) __attribute__((amdgpu_waves_per_eu(2)))
lconv_kernel(const typename IO::T* __restrict__ in, const float2* __restrict__ kspec, typename IO::T* __restrict__ out,
             const typename IO::T* __restrict__ gate, int B, int H, int items, const uint4* __restrict__ tab)
{
    using L = LR<LG>;
    constexpr bool BF = IsBf<IO>::v;
    constexpr int TE = L::TE, PC = L::PC;
    extern __shared__ uint4 lds4[];
    _Float16 *ex = reinterpret_cast<_Float16*>(lds4), *raw = ex + L::EX;
    uint4* shared = reinterpret_cast<uint4*>(raw + L::RAW);
    __shared__ uint32_t mxs[2][8];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, g = lane >> 4;
    const unsigned G = gridDim.x;
    const int wg = (G & 7u) ? (int)blockIdx.x : (int)((blockIdx.x & 7u) * (G >> 3) + (blockIdx.x >> 3));   // neighbours on one XCD
    const int each = items / (int)G, more = items - each * (int)G;
    const int i0 = wg * each + min(wg, more), n = each + (wg < more);
    if (n <= 0) return;
    int h = i0 / B, b = i0 - h * B;                  // row of phase 1
    int ho = h, bo = b;                              // row that is stored
    int hl = h, bl = b;                              // row that is asked for
    // With the gate memory is reached through descriptors: a lane's 64-bit addresses cost 14 to 26 spilled registers at N = 8192 (with
    // descriptors 1 and 4; B=16, H=256 bf16 61.8 and 58.8 us).  Without it plain addresses are as fast, and 3 % faster where a workgroup
    // has one row.  At N = 16384 nothing is spilled either way (fp16 plain and descriptors: B=7, H=193 43.3 and 42.8, B=16, H=256 109.7 and
    // 110.9; bf16 45.5 and 46.0, 118.5 and 119.7, B=2, H=128 11.7 and 12.0).
    constexpr bool DESC = GATE && !(LG == 14 && BF);
    u4w pf[PC];
    const auto ask = [&]() {
        const typename IO::T* p = in + row_off(bl, hl, H, L::N);
#pragma unroll
        for (int i = 0; i < PC; ++i)
            pf[i] = DESC ? row_load(row_rsrc(p, L::N * 2), 16 * tid, i * 16 * L::NT) : reinterpret_cast<const u4w*>(p)[tid + i * L::NT];
        if (++bl == B) { bl = 0; ++hl; }
    };
    ask();
    LK<L, true, true> K;
    K.load(tab, wave, lane);
    load_shared<L>(shared, tab, tid, false);
    const uint4* mats = shared + lane;
    Places<L> P;
    P.make(wave, lane);
    _Float16* mine = raw + piece_of<L>(tid);
    H8P ks[L::KB][TE];                               // the wave's bins, as phase 2 meets them
    int es0 = 0, es1 = 0, e0 = 0, e1 = 0;            // exponents of spectrum and row: in phases 1 and 2, and in phase 3
    const auto load_spec = [&]() {
        const uint4* s = reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(kspec) + (size_t)h * 2 * L::N);
#pragma unroll
        for (int j = 0; j < L::KB; ++j)
#pragma unroll
            for (int ke = 0; ke < TE; ++ke) {
                const int u = ((wave * L::KB + j) * TE + ke) * 64;
                ks[j][ke].w = DESC ? __builtin_bit_cast(uint4, row_load(row_rsrc(s, L::N * 4), 16 * lane, 16 * u)) : s[u + lane];
            }
        es0 = spec_exp_of(kspec, H, 2 * (int64_t)L::N)[h];
    };
    load_spec();
    const auto arrive = [&](int t) {                 // row t has arrived
        if constexpr (BF) {
            const uint32_t m = pieces_max<PC>(pf);
            if (lane == 0) mxs[t & 1][wave] = m;
        }
#pragma unroll
        for (int i = 0; i < PC; ++i) *reinterpret_cast<u4w*>(mine + i * L::STEP) = pf[i];
    };
    arrive(0);
    if (n > 1) ask();
    __syncthreads();
    const _Float16* rp = raw + P.raw;
    u4w ga[GATE ? 4 : 1];                            // the gate at this lane's pieces of the row in phase 3
    const auto ask_gate = [&](int bb, int hh) {
        if constexpr (GATE) {
            const typename IO::T* p = gate + row_off(bb, hh, H, L::N) + (64 * g + c) * L::TC + 8 * wave;
#pragma unroll
            for (int r = 0; r < 4; ++r) ga[r] = *reinterpret_cast<const u4w*>(p + r * 16 * L::TC);
        }
    };
    // phase 3 of one row and phase 1 of the next
    const auto part_a = [&](auto do3_, auto do1_, int ex3, int ein) __attribute__((always_inline)) {
        constexpr bool do3 = decltype(do3_)::value, do1 = decltype(do1_)::value;
        u4w w[4], o[4];
        if (do1) read_pieces<L>(w, rp);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            h4 op[2];
            if (do1) pair_ops<IO>({w[0][p], w[1][p], w[2][p], w[3][p]}, ein, op);
            f4 v[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int kt = 2 * p + k;
                if (do3) v[k] = phase3_tile<L, true, false>(ex + P.own_tr[kt / TE] + P.in_group(kt), K, kt, mats, nullptr);
                if (do1) phase1_tile<L, false>(op[k], K, kt, mats, ex + P.own[kt / TE] + P.in_group(kt));
            }
            if (do3) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float x = v[0][r], y = v[1][r];
                    if constexpr (GATE) { x *= io_half<IO>(ga[r][p], 0); y *= io_half<IO>(ga[r][p], 1); }
                    o[r][p] = pack_io<IO>(ldexpf(x, ex3), ldexpf(y, ex3));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (do3) write_pieces<L>(o, raw + P.raw);
    };
    // row t is in phase 2; row t - 1 is stored, row t + 1 put into LDS
    const auto part_b = [&](int t) __attribute__((always_inline)) {
        if (t + 1 < n) {
            arrive(t + 1);
            if (t + 2 < n) ask();
        }
        ask_gate(b, h);
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            H8P v[TE];
            phase2_fwd<L>(ex + P.mid_tr[j], K, j, mats, [&](int m, const f4& yr, const f4& yi) __attribute__((always_inline)) {
                const H8P& k = ks[j][m];
                v[m] = LG == 13 ? cmul_once<CONJ>(yr, yi, k.p[0], k.p[1]) : cmul_planes<CONJ>(yr, yi, k.p[0], k.p[1]);
            });
            phase2_inv<L, false>(ex + P.mid[j], K, j, mats, v, v);
            __builtin_amdgcn_sched_barrier(0);
        }
        e1 = e0;
        es1 = es0;
        if (++b == B) { b = 0; ++h; }
    };
    const auto store = [&]() {
        typename IO::T* p = out + row_off(bo, ho, H, L::N);
#pragma unroll
        for (int i = 0; i < PC; ++i) {
            const u4w v = *reinterpret_cast<const u4w*>(mine + i * L::STEP);
            if (DESC) row_store(row_rsrc(p, L::N * 2), 16 * tid, i * 16 * L::NT, v);
            else put_once(reinterpret_cast<u4w*>(p) + tid + i * L::NT, v);
        }
        if (++bo == B) { bo = 0; ++ho; }
    };
    const auto exponent = [&](int t) {
        if constexpr (BF) {
            uint32_t m = 0u;
#pragma unroll
            for (int w = 0; w < L::NW; ++w) m = max(m, mxs[t & 1][w]);
            e0 = mu::row_exponent(__builtin_amdgcn_readfirstlane((int)m));
        }
    };
    const std::true_type yes;
    const std::false_type no;
    exponent(0);
    part_a(no, yes, 0, e0);
    __syncthreads();
    part_b(0);
    __syncthreads();
    for (int t = 1; t < n; ++t) {
        exponent(t);
        part_a(yes, yes, es1 + e1, e0);
        if (b == 0) load_spec();                     // (another head's row goes through phase 2 next)
        __syncthreads();
        store();
        part_b(t);
        __syncthreads();
    }
    part_a(yes, no, es1 + e1, 0);
    __syncthreads();
    store();
}

// -------------------------------------------------------------------------------------------------------------------
// Whole backward pass of a head (or of a share of its rows) per workgroup: du, dk and dD from one read of dy and u.  Per row
// U = transform of u, W = transform of dy, A += conj(U) W in fp32 registers, du = inverse of W conj(K); dk is one inverse
// transform of A at the end.  Four parts per row between barriers, on one exchange buffer (U stays in registers, fp16, between
// the second and the fourth) and one place for a row of samples, where u, du of the row before, and dy take turns:
//     [phase 3 of row t-1's du, phase 1 of u_t]  [phase 2 of u_t; du stored, dy_t in]  [phase 1 of dy_t]
//     [phase 2 of dy_t, A, inverse half for du; u_(t+1) in]
// dD needs both rows at once: u is read a second time, from cache, when dy arrives.  DU = false: dk and dD alone.
// Bound by memory as much as by issue: B=8, H=256, N=16384 fp16 moves up to 510 MB in 111 us (4.6 TB/s; a large copy 5.1) for
// 235 MB of rows and gradients, with vector instructions in half of the cycles and matrix instructions in a quarter.  What is read
// beyond the rows is the spectrum for every row again (117 MB), u's second reading (67) and spilled registers: the sums alone take
// a quarter of them, and 20 to 22 have no place.  With more of them in the loop the reloads wait behind the row in flight: 167 us,
// 112 with the matrices of three tiles per wave and their factors in LDS, 107 with the rows' addresses kept scalar, 104
// with requests and stores spread over the tiles (as pairs, dk in two walks and du by itself: 197).  N = 8192 takes four tiles per wave (LB) and spills nothing: with eight, B=64, H=128 289 us,
// with four 167 (as pairs 325).
// -------------------------------------------------------------------------------------------------------------------
template <class T>
struct LBwdArgs {
    const T* dy;
    const T* u;
    const float2* kspec;
    T* du;
    float* dk;
    float* dD;
    int B, H, nsplit;
    float dkscale;
    const uint4* tab;
};
template <int LG>
using LB = LR<LG, LG == 13 ? 4 : 8, LG == 14 ? 3 : 0>;
template <int LG, class IO, bool DU>
__global__ void __launch_bounds__(LB<LG>::NT) __attribute__((amdgpu_waves_per_eu(2)))
lbwd_kernel(const LBwdArgs<typename IO::T> q)
{
    using L = LB<LG>;
    constexpr bool BF = IsBf<IO>::v;
    constexpr int TE = L::TE, PC = L::PC, NA = L::KB * TE;
    constexpr bool TAI = LG == 13;                   // (registers for it: four tiles per wave)
    extern __shared__ uint4 lds4[];
    _Float16 *ex = reinterpret_cast<_Float16*>(lds4), *raw = ex + L::EX;
    uint4* shared = reinterpret_cast<uint4*>(raw + L::RAW);
    __shared__ uint32_t mxs[2][2][8];                // patterns of the waves' pieces: u and dy, by row parity
    __shared__ float dred[8];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, g = lane >> 4;
    const int B = q.B, H = q.H, nsplit = q.nsplit;
    const int h = blockIdx.x % (unsigned)H, split = blockIdx.x / (unsigned)H;
    const int n = (B - split + nsplit - 1) / nsplit;                  // rows of this workgroup, nsplit apart (>= 1)
    const size_t step = (size_t)nsplit * H * (L::N / 8);
    const u4w* pu = reinterpret_cast<const u4w*>(q.u + row_off(split, h, H, L::N));
    const u4w* pd = reinterpret_cast<const u4w*>(q.dy + row_off(split, h, H, L::N));
    u4w* po = DU ? reinterpret_cast<u4w*>(q.du + row_off(split, h, H, L::N)) : nullptr;
    u4w pa[PC], pb[PC];
    // Rows are asked for half by half, between the tiles, and stored between the k_b's: all at once, the requests of eight waves held
    // the later four back by some 1800 cycles of 21000 per row, and the others at the barrier.  Where there is no row an empty
    // descriptor asks for nothing: in a condition the pieces would come into registers of their own, be copied and so waited for.
    // Backward, fp16, N=16384: B=8, H=256 98.5 -> 95.7 us, B=32, H=128 183 -> 176, B=1, H=256 27.2 -> 25.2; bf16 within 2 %.
    const auto ask = [&](u4w (&v)[PC], const u4w* p, bool any, auto from, auto to) __attribute__((always_inline)) {
        const auto d = row_rsrc(p, any ? L::N * 2 : 0);
#pragma unroll
        for (int i = decltype(from)::value; i < decltype(to)::value; ++i) v[i] = row_load(d, 16 * tid, i * 16 * L::NT);
    };
    const std::integral_constant<int, 0> none;
    const std::integral_constant<int, PC / 2> half;
    const std::integral_constant<int, PC> all;
    ask(pa, pu, true, none, all);
    LK<L, true, TAI, L::NAL> K;
    K.load(q.tab, wave, lane, shared + L::N_LDS * 64 + L::TC * 4);
    load_shared<L>(shared, q.tab, tid, true);
    const uint4 *mats = shared + lane, *factors = shared + L::N_LDS * 64 + L::TPW * wave * 4 + g;
    Places<L> P;
    P.make(wave, lane);
    _Float16* mine = raw + piece_of<L>(tid);
    const uint4* ks = DU ? reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(q.kspec) + (size_t)h * 2 * L::N) +
                               (size_t)wave * NA * 64
                         : nullptr;
    const int es = DU ? spec_exp_of(q.kspec, H, 2 * (int64_t)L::N)[h] : 0;
    float2 acc[NA][4];
#pragma unroll
    for (int k = 0; k < NA; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[k][j] = make_float2(0.f, 0.f);
    float dsum = 0.f;
    const auto arrive = [&](const u4w (&v)[PC], int source, int t) {  // row t of u (0) or dy (1)
        if constexpr (BF) {
            const uint32_t m = pieces_max<PC>(v);
            if (lane == 0) mxs[source][t & 1][wave] = m;
        }
#pragma unroll
        for (int i = 0; i < PC; ++i) *reinterpret_cast<u4w*>(mine + i * L::STEP) = v[i];
    };
    arrive(pa, 0, 0);
    __syncthreads();
    const auto pattern = [&](int source, int t) {
        uint32_t m = 0u;
#pragma unroll
        for (int w = 0; w < L::NW; ++w) m = max(m, mxs[source][t & 1][w]);
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
    };
    H8P U[NA];
    int eref = mu::EXP_NONE, ed = 0, eu = 0;         // unit of A; exponents (bf16) of the rows of dy and u
    uint32_t mu_ = 0u, md = 0u;
    const auto part_a = [&](auto do3_, auto do1_, bool any) __attribute__((always_inline)) {      // (any: rows pd and pu are asked for)
        constexpr bool do3 = DU && decltype(do3_)::value, do1 = decltype(do1_)::value;
        const int ex3 = es + ed;
#pragma unroll
        for (int p = 0; p < L::TPW / 2; ++p) {
            h4 op[2];
            uint32_t w[4];
            if (do1) {
                read_pair<L>(w, raw + P.raw, p);
                pair_ops<IO>(w, eu, op);
            }
            f4 v[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int kt = 2 * p + k;
                if (do3) v[k] = phase3_tile<L, TAI, false>(ex + P.own_tr[kt / TE] + P.in_group(kt), K, kt, mats, factors + 4 * kt);
                if (do1) phase1_tile<L, false>(op[k], K, kt, mats, ex + P.own[kt / TE] + P.in_group(kt));
            }
            if (do1) {
                constexpr int LASTP = L::TPW / 2 - 1;
                if (p == 0) ask(pa, pd, any, none, half);
                if (p == (LASTP > 1)) ask(pa, pd, any, half, all);
                if (p == LASTP - (LASTP > 1)) ask(pb, pu, any, none, half);
                if (p == LASTP) ask(pb, pu, any, half, all);
            }
            if (do3) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    reinterpret_cast<uint32_t*>(raw + P.raw + r * 16 * L::TC)[p] = pack_io<IO>(ldexpf(v[0][r], ex3), ldexpf(v[1][r], ex3));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // pieces i0 .. i1 - 1 of a row of du
    const auto store = [&](const u4w (&o)[PC], bool any, int i0, int i1) __attribute__((always_inline)) {
        const auto d = row_rsrc(po, any ? L::N * 2 : 0);
#pragma unroll
        for (int i = 0; i < PC; ++i)
            if (i >= i0 && i < i1) row_store(d, 16 * tid, i * 16 * L::NT, o[i]);
    };
    const auto done = [&](u4w (&o)[PC]) __attribute__((always_inline)) {      // the row that phase 3 left
#pragma unroll
        for (int i = 0; i < PC; ++i) o[i] = *reinterpret_cast<const u4w*>(mine + i * L::STEP);
    };
    // the other three parts of row t
    const auto rest = [&](int t) __attribute__((always_inline)) {
        u4w o[PC];
        if (DU) done(o);
#pragma unroll
        for (int i = 0; i < PC; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                union { uint32_t u; mu::h2 h; mu::bf2 b; } x, y;
                x.u = pa[i][r];
                y.u = pb[i][r];
                dsum = BF ? __builtin_amdgcn_fdot2_f32_bf16(x.b, y.b, dsum, false) : __builtin_amdgcn_fdot2(x.h, y.h, dsum, false);
            }
        arrive(pa, 1, t);
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            phase2_fwd<L>(ex + P.mid_tr[j], K, j, mats, [&](int m, const f4& yr, const f4& yi) __attribute__((always_inline)) {
                U[j * TE + m] = planes(yr, yi);
            });
            if (DU) store(o, t > 0, j * PC / L::KB, (j + 1) * PC / L::KB);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (DU && t > 0) po += step;
        __syncthreads();
        if (t + 1 < n) pu += step;
        if constexpr (BF) {
            md = pattern(1, t);
            ed = mu::row_exponent(md);
            const int ep = md && mu_ ? ed + eu : mu::EXP_NONE;
            if (ep != eref) {
                // a term smaller than A's unit: U takes the power of two, and loses what is 2^-24 of the largest term
                const int down = mu::acc_align<NA>(acc, eref, ep);
                if (down != 0) {
                    const _Float16 f = (_Float16)ldexpf(1.f, down);
#pragma unroll
                    for (int k = 0; k < NA; ++k) {
                        U[k].p[0] *= f;
                        U[k].p[1] *= f;
                    }
                }
            }
        }
        {
#pragma unroll
            for (int p = 0; p < L::TPW / 2; ++p) {
                h4 op[2];
                uint32_t w[4];
                read_pair<L>(w, raw + P.raw, p);
                pair_ops<IO>(w, ed, op);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int kt = 2 * p + k;
                    phase1_tile<L, LG == 13>(op[k], K, kt, mats, ex + P.own[kt / TE] + P.in_group(kt));
                }
                if (p == 0) ask(pb, pu, t + 1 < n, none, half);
                if (p == 1) ask(pb, pu, t + 1 < n, half, all);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        if (t + 1 < n) arrive(pb, 0, t + 1);
#pragma unroll
        for (int j = 0; j < L::KB; ++j) {
            H8P kk[TE], v[TE];
            if (DU) {
#pragma unroll
                for (int m = 0; m < TE; ++m) kk[m].w = uniform(ks, (j * TE + m) * 64)[(unsigned)lane];
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
                if (DU) v[m] = cmul_planes<true>(yr, yi, kk[m].p[0], kk[m].p[1]);
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
    };
    const std::true_type yes;
    const std::false_type no;
    const auto exponent = [&](int t) {
        if constexpr (BF) {
            mu_ = pattern(0, t);
            eu = mu::row_exponent(mu_);
        }
    };
    exponent(0);
    part_a(no, yes, true);
    __syncthreads();
    rest(0);
    for (int t = 1; t < n; ++t) {
        exponent(t);
        pd += step;
        part_a(yes, yes, true);
        __syncthreads();
        rest(t);
    }
    if (DU) {
        part_a(yes, no, false);
        __syncthreads();
        u4w o[PC];
        done(o);
        store(o, true, 0, PC);
    }

    for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
    if (lane == 0) dred[wave] = dsum;
    uint32_t* peaks = &mxs[0][0][0];
    const uint32_t peak = mu::acc_peak<NA>(acc);
    __syncthreads();
    if (lane == 0) peaks[wave] = peak;
    __syncthreads();
    const size_t ho = (size_t)split * H + h;
    if (q.dk) {
        uint32_t m = peaks[0];
#pragma unroll
        for (int w = 1; w < L::NW; ++w) m = max(m, peaks[w]);
        const int ea = __builtin_amdgcn_readfirstlane(mu::acc_exponent(m)), etop = (BF ? eref : 0) + ea;
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
        f4 v[L::TPW];
#pragma unroll
        for (int kt = 0; kt < L::TPW; ++kt)
            v[kt] = phase3_tile<L, TAI, true>(ex + P.own_tr[kt / TE] + P.in_group(kt), K, kt, mats, factors + 4 * kt);
        __syncthreads();
        // the row of dk, fp32, where the points were
        float* row = reinterpret_cast<float*>(ex);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < L::TPW; k += 4) {
                f4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = ldexpf(v[k + e][r] * q.dkscale, etop);
                *reinterpret_cast<f4*>(row + L::piece(64 * g + 16 * r + c, wave * L::TPW / 8) + wave * L::TPW % 8 + k) = o;
            }
        __syncthreads();
        f4* out = reinterpret_cast<f4*>(q.dk + ho * L::N);
        for (int i = tid; i < L::N / 4; i += L::NT) {
            const int e = i >> 1;
            out[i] = *reinterpret_cast<const f4*>(row + L::piece(e / (L::TC / 8), e % (L::TC / 8)) + 4 * (i & 1));
        }
    }
    if (tid == 0 && q.dD) {
        float s = 0.f;
        for (int w = 0; w < L::NW; ++w) s += dred[w];
        q.dD[ho] = s;
    }
}

// -------------------------------------------------------------------------------------------------------------------
// Kernel spectrum, one workgroup per head: kscale (FFT + D) as fp16 words in the lane order of phase 2, with the head's
// exponent (spec_exponent).
// -------------------------------------------------------------------------------------------------------------------
template <int LG>
__global__ void __launch_bounds__(LR<LG>::NT) __attribute__((amdgpu_waves_per_eu(2)))
lkspec_kernel(const float* __restrict__ k, const float* __restrict__ D, float2* __restrict__ kspec, float kscale_over_c,
              float kscale, const uint4* __restrict__ tab)
{
    using L = LR<LG>;
    constexpr int TE = L::TE, PC = L::PC;
    extern __shared__ uint4 lds4[];
    _Float16 *ex = reinterpret_cast<_Float16*>(lds4), *raw = ex + L::EX;
    uint4* shared = reinterpret_cast<uint4*>(raw + L::RAW);
    __shared__ float mred[3][8];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.x;
    const f4* kr = reinterpret_cast<const f4*>(k + (size_t)h * L::N);
    f4 v[PC][2];
#pragma unroll
    for (int i = 0; i < PC; ++i) {
        v[i][0] = kr[2 * (tid + i * L::NT)];
        v[i][1] = kr[2 * (tid + i * L::NT) + 1];
    }
    const float Dh = D[h];
    LK<L, false, false> K;
    K.load(tab, wave, lane);
    load_shared<L>(shared, tab, tid, false);
    const uint4* mats = shared + lane;
    Places<L> P;
    P.make(wave, lane);
    // the head's largest magnitude; sum and maximum with the skip term counted in the lag-0 tap
    float m = 0.f, a = 0.f, mp = 0.f;
#pragma unroll
    for (int i = 0; i < PC; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float x = v[i][q >> 2][q & 3], x0 = i == 0 && q == 0 && tid == 0 ? fabsf(x + Dh) : fabsf(x);
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
    const float r = head_scale_of(m);
#pragma unroll
    for (int i = 0; i < PC; ++i) {
        u4w w;
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = mu::pack_h2(v[i][q >> 1][2 * (q & 1)] * r, v[i][q >> 1][2 * (q & 1) + 1] * r);
        *reinterpret_cast<u4w*>(raw + piece_of<L>(tid) + i * L::STEP) = w;
    }
    __syncthreads();
    u4w w[4];
    read_pieces<L>(w, raw + P.raw);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        h4 op[2];
        pair_ops<IoF16>({w[0][p], w[1][p], w[2][p], w[3][p]}, 0, op);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int kt = 2 * p + q;
            phase1_tile<L, true>(op[q], K, kt, mats, ex + P.own[kt / TE] + P.in_group(kt));
        }
    }
    __syncthreads();
    const int es = spec_exponent(kscale * a, kscale * mp);
    if (tid == 0) spec_exp_of(kspec, gridDim.x, 2 * (int64_t)L::N)[h] = es;
    const float alpha = ldexpf(kscale_over_c / r, -es), beta = ldexpf(Dh * kscale, -es);
    uint4* out = reinterpret_cast<uint4*>(reinterpret_cast<uint32_t*>(kspec) + (size_t)h * 2 * L::N);
#pragma unroll
    for (int j = 0; j < L::KB; ++j) {
        phase2_fwd<L>(ex + P.mid_tr[j], K, j, mats, [&](int m, const f4& yr, const f4& yi) __attribute__((always_inline)) {
            out[((wave * L::KB + j) * TE + m) * 64 + lane] = planes(yr * alpha + beta, yi * alpha).w;
        });
    }
}

template <int LG, class IO, bool CONJ, bool GATE>
hipError_t conv_go(const void* in, const float2* kspec, void* out, const Problem& pr, const Tables& tb, hipStream_t st)
{
    using L = LR<LG>;
    using T = typename IO::T;
    const auto kern = lconv_kernel<LG, IO, CONJ, GATE>;
    hipError_t e = set_lds(kern, L::lds(false));
    if (e != hipSuccess) return e;
    static int resident = 0;
    if (resident == 0) {
        int nb = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, L::NT, L::lds(false));
        if (e != hipSuccess) return e;
        resident = (nb > 0 ? nb : 1) * compute_units();
    }
    // as many workgroups as fill their turns evenly
    const int64_t items = pr.H * pr.B, per = (items + resident - 1) / resident;
    hipLaunchKernelGGL(kern, dim3((unsigned)((items + per - 1) / per)), dim3(L::NT), L::lds(false), st, (const T*)in, kspec, (T*)out,
                       (const T*)pr.gate, (int)pr.B, (int)pr.H, (int)items, (const uint4*)tb.ltab);
    return hipGetLastError();
}

template <int LG, class IO>
hipError_t conv_io(const void* in, const float2* kspec, void* out, bool conj, const Problem& pr, const Tables& tb, hipStream_t st)
{
    if (pr.gate) return conj ? hipErrorInvalidValue : conv_go<LG, IO, false, true>(in, kspec, out, pr, tb, st);
    return conj ? conv_go<LG, IO, true, false>(in, kspec, out, pr, tb, st) : conv_go<LG, IO, false, false>(in, kspec, out, pr, tb, st);
}

template <int LG, class IO, bool DU>
hipError_t bwd_go(const void* dy, const void* u, const float2* kspec, void* du, float* dk, float* dD, int nsplit,
                  const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
    using L = LB<LG>;
    using T = typename IO::T;
    const hipError_t e = set_lds(lbwd_kernel<LG, IO, DU>, L::lds(true));
    if (e != hipSuccess) return e;
    const LBwdArgs<T> a{(const T*)dy, (const T*)u, kspec, (T*)du, dk, dD, (int)pr.B, (int)pr.H, nsplit, pl.dkscale, (const uint4*)tb.ltab};
    hipLaunchKernelGGL((lbwd_kernel<LG, IO, DU>), dim3((unsigned)(pr.H * nsplit)), dim3(L::NT), L::lds(true), st, a);
    return hipGetLastError();
}
template <int LG, class IO>
hipError_t bwd_io(const void* dy, const void* u, const float2* kspec, void* du, float* dk, float* dD, int nsplit,
                  const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
    return du ? bwd_go<LG, IO, true>(dy, u, kspec, du, dk, dD, nsplit, pr, pl, tb, st)
              : bwd_go<LG, IO, false>(dy, u, kspec, du, dk, dD, nsplit, pr, pl, tb, st);
}

template <int LG>
hipError_t kspec_go(const float* k, const float* D, float2* kspec, int64_t H, const Plan& pl, const Tables& tb, hipStream_t st)
{
    using L = LR<LG>;
    const hipError_t e = set_lds(lkspec_kernel<LG>, L::lds(false));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(lkspec_kernel<LG>, dim3((unsigned)H), dim3(L::NT), L::lds(false), st, k, D, kspec,
                       pl.kscale * (float)(1 << L::SHIFT), pl.kscale, (const uint4*)tb.ltab);
    return hipGetLastError();
}

}  // namespace

hipError_t long_fill_tables(const void** tab_out, hipStream_t st)
{
    uint4* p = nullptr;
    const hipError_t e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(g_long_tab));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fill_long_tab_kernel<13>, dim3(LR<13>::UNITS), dim3(64), 0, st, p);
    hipLaunchKernelGGL(fill_long_tab_kernel<14>, dim3(LR<14>::UNITS), dim3(64), 0, st, p + tab_offset<14>() * 64);
    *tab_out = p;
    return hipGetLastError();
}

float long_chain_scale() { return 1.0f / (float)(1 << LR<LONG_MAX_LOG2>::SHIFT); }

hipError_t long_kspec(const float* k, const float* D, float2* kspec, int64_t H, const Plan& pl, const Tables& tb, hipStream_t st)
{
    if (pl.order.long_lg == 13) return kspec_go<13>(k, D, kspec, H, pl, tb, st);
    if (pl.order.long_lg == 14) return kspec_go<14>(k, D, kspec, H, pl, tb, st);
    return hipErrorInvalidValue;
}

hipError_t long_conv(const void* in, const float2* kspec, void* out, bool conj, const Problem& pr, const Plan& pl, const Tables& tb,
                     hipStream_t st)
{
    if (pr.io == LONGCONV_F16) {
        if (pl.order.long_lg == 13) return conv_io<13, IoF16>(in, kspec, out, conj, pr, tb, st);
        if (pl.order.long_lg == 14) return conv_io<14, IoF16>(in, kspec, out, conj, pr, tb, st);
    } else if (pr.io == LONGCONV_BF16) {
        if (pl.order.long_lg == 13) return conv_io<13, IoBF16>(in, kspec, out, conj, pr, tb, st);
        if (pl.order.long_lg == 14) return conv_io<14, IoBF16>(in, kspec, out, conj, pr, tb, st);
    }
    return hipErrorInvalidValue;
}

hipError_t long_bwd(const void* dy, const void* u, const float2* kspec, void* du, float* dk, float* dD, int nsplit,
                    const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
#define GO(LG, IO) return bwd_io<LG, IO>(dy, u, kspec, du, dk, dD, nsplit, pr, pl, tb, st)
    if (pr.io == LONGCONV_F16) {
        if (pl.order.long_lg == 13) GO(13, IoF16);
        if (pl.order.long_lg == 14) GO(14, IoF16);
    } else if (pr.io == LONGCONV_BF16) {
        if (pl.order.long_lg == 13) GO(13, IoBF16);
        if (pl.order.long_lg == 14) GO(14, IoBF16);
    }
#undef GO
    return hipErrorInvalidValue;
}

// Shares of a head's rows: the number that ends first where each compute unit holds one workgroup (eight waves of more than 200
// registers at either length), and a workgroup's constants and its inverse transform cost as much as about a row and a half, a
// second launch as half a row.  How many are tried at most bounds the workspace.
static int64_t most_shares(int64_t B, int64_t H)
{
    int64_t most = 384 / H;
    if (most > (B + 1) / 2) most = (B + 1) / 2;
    if (most > 64) most = 64;
    most = most > 1 ? most + 2 : 2;
    return most < B ? most : B;
}
static int64_t turns(int64_t workgroups) { return (workgroups + 255) / 256; }
int long_bwd_nsplit(int64_t B, int64_t H)
{
    const int64_t most = most_shares(B, H);
    int64_t best = 1, best_t = -1;
    for (int64_t s = 1; s <= most; ++s) {
        const int64_t t = turns(s * H) * (2 * ((B + s - 1) / s) + 3) + (s > 1 ? 1 : 0);
        if (best_t < 0 || t < best_t) { best = s; best_t = t; }
    }
    return (int)best;
}
// (one share ends before s shares of s times its turns, whatever B)
int long_bwd_room(int64_t B, int64_t H)
{
    int64_t room = 1;
    for (int64_t s = 2; s <= most_shares(B, H); ++s)
        if (turns(s * H) < s * turns(H)) room = s;
    return (int)room;
}

}  // namespace lc
