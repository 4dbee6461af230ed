// fp32 engine: the whole FFT convolution of one row pair, or (N = 2048 .. 16384) of one row, on the vector ALUs.  It serves fp32
// I/O (where fp16 matrix-core operands cannot meet the accuracy bound) and, for every dtype, the spectrum of plans whose consumer is
// the staged matrix-core kernel.
//
// Transform convention (paper Eq. 2 with the sequence zero padded to L = 2N): mixed radix, in place.  A stage of
// radix r and span Ls (stride M = Ls / r) takes position blk*Ls + d*M + q to blk*Ls + k*M + q,
//     forward (decimation in frequency): DFT over d, then w_Ls^(k q);     inverse: w_Ls^(-k q), then DFT^-1 over k,
// so the digit-reversed order in which the forward stages leave the frequencies is what the inverse stages start
// from and the pointwise product needs no permutation (Section 3.2, "eliminates permutations over the input").
//
// Layout: a workgroup of T = L2 / P threads owns one sequence of L2 = 2^LG points, P per thread in registers.  Every
// stage is a butterfly of up to P points in registers; between two stages the points cross LDS once, each thread
// writing the positions it holds and reading those of its next butterfly (one barrier: the positions a thread reads
// are the ones it writes next).  Stage 0 takes its P points straight from the rows (thread q: samples q + d T, so every
// load is a unit-stride run) and the last inverse stage stores them the same way.  What bounds it: about 60
// vector instructions per point and transform at 3 or 4 exchanges, against LDS at 16 bytes per point and exchange; the
// radix-2 form it replaces crossed LDS once per bit (14 times at L = 16384) with a table look-up per butterfly, and
// ran N = 8192, B=4, H=96 at 108 us per convolution and 152 us for dk.
#include <type_traits>

#include "engines.hpp"

namespace lc {
namespace {

// ---- radix schedule ---------------------------------------------------------------------------------------------
// Points per thread by length: more points mean fewer exchanges, fewer points more waves for the same work.
constexpr int points_log2(int LG) { return LG <= 8 ? 2 : LG <= 11 ? 3 : 4; }
constexpr int stages(int LG) { return (LG + points_log2(LG) - 1) / points_log2(LG); }
// bits of stage s: the first one as wide as a thread holds points (it reads the rows), the others as even as they go
constexpr int stage_bits(int LG, int s)
{
    const int lp = points_log2(LG), n = stages(LG) - 1;
    if (s == 0) return lp;
    const int rem = LG - lp;
    return rem / n + (s - 1 < rem % n ? 1 : 0);
}
// log2 of the span of stage s
constexpr int span_log2(int LG, int s)
{
    int l = LG;
    for (int i = 0; i < s; ++i) l -= stage_bits(LG, i);
    return l;
}

// LDS position of point p, with a slot of padding behind every 2^K.  16 lanes are served at a time, so sixteen leaves their runs of
// neighbours whole, and eight spreads the lanes of a last stage of radix 8 or 4.  Cycles per access of the exchanges of a transform, summed
// over them, for eight and sixteen: 2^8 points 12 and 12 (of 6), 2^9 5 and 6, 2^10 12 and 12, 2^11 10 and 8, 2^12 8 and 4, 2^13 and 2^14 9
// and 8, 2^15 11 and 6.  Measured, fp32 us: backward N = 512 (2^10) B=16 H=256 18.8 and 20.3, N = 1024 (2^11) B=64 H=256 90.1 and 87.1,
// N = 16384 (single rows of 2^14) B=4 H=64 49.0 and 46.7, N = 65536 (2^14) B=2 H=32 129.3 and 125.8; step N = 4096 (rows of 2^12) B=32
// H=1024 1333 and 1308.
template <int K>
__host__ __device__ constexpr int phys(int p) { return p + (p >> K); }
constexpr int fft_pad(int LG) { return LG >= 11 ? 4 : 3; }
// whether the backward kernel parks the transform of u in memory (see fbwd_kernel)
constexpr bool valu_parks(int LG) { return LG >= 14; }
constexpr bool row_parks(int LG) { return points_log2(LG) == 4; }        // (frow_bwd_kernel)
// which single rows take the butterflies' constants (N = 2048: and the twist's, on the way in) in two parts; see frow_conv_kernel
constexpr bool row_fine(int LG) { return LG <= 12; }

// ---- butterflies in registers -------------------------------------------------------------------------------------
// v * exp(-+ 2 pi i m / 32): m a compile-time constant after unrolling.  FINE (even m only, the butterflies' own): constants in two
// fp32 parts, so that their rounding, the same for every point of every stage, is out of the result: at 4096 points, radix 16,
// it is a third of a transform's squared error, for 8 and 8 instructions more per butterfly.
template <bool INV, bool FINE = false>
__device__ __forceinline__ float2 rot32(float2 v, int m)
{
    constexpr float C[5] = {1.f, 0.98078528040323043f, 0.92387953251128674f, 0.83146961230254524f, 0.70710678118654752f};
    constexpr float S[5] = {0.f, 0.19509032201612825f, 0.38268343236508977f, 0.55557023301960218f, 0.70710678118654752f};
    m &= 31;
    const int q = m >> 3, r = m & 7;
    float2 t = v;
    if (FINE && r) {
        // cos of an eighth and a sixteenth of a turn (high, low part); tan of a sixteenth
        constexpr float H = 0.70710678118654752f, HL = (float)(0.70710678118654752440 - (double)H);
        constexpr float Q = 0.92387953251128676f, QL = (float)(0.92387953251128675613 - (double)Q), TQ = 0.41421356237309505f;
        const float sy = INV ? v.y : -v.y, sx = INV ? v.x : -v.x;      // (v.x, v.y) turned by a quarter: (-sy, sx)
        const float2 w = r == 4 ? make_float2(v.x - sy, v.y + sx)
                       : r == 2 ? make_float2(__builtin_fmaf(-sy, TQ, v.x), __builtin_fmaf(sx, TQ, v.y))
                                : make_float2(__builtin_fmaf(v.x, TQ, -sy), __builtin_fmaf(v.y, TQ, sx));
        t = r == 4 ? make_float2(__builtin_fmaf(w.x, H, w.x * HL), __builtin_fmaf(w.y, H, w.y * HL))
                   : make_float2(__builtin_fmaf(w.x, Q, w.x * QL), __builtin_fmaf(w.y, Q, w.y * QL));
    } else if (r == 4) {
        t = INV ? make_float2((v.x - v.y) * C[4], (v.x + v.y) * C[4]) : make_float2((v.x + v.y) * C[4], (v.y - v.x) * C[4]);
    } else if (r) {
        const float c = r < 4 ? C[r] : S[8 - r], s = (r < 4 ? S[r] : C[8 - r]) * (INV ? 1.f : -1.f);
        t = make_float2(v.x * c - v.y * s, v.x * s + v.y * c);
    }
    if (q == 0) return t;
    if (q == 2) return make_float2(-t.x, -t.y);
    return ((q == 1) != INV) ? make_float2(t.y, -t.x) : make_float2(-t.y, t.x);
}

// natural order in and out, stride ST between the elements
template <int R, bool INV, bool FINE = false, int ST = 1>
__device__ __forceinline__ void dft(float2* x)
{
    if constexpr (R == 2) {
        const float2 a = x[0], b = x[ST];
        x[0] = cadd(a, b);
        x[ST] = csub(a, b);
    } else if constexpr (R == 4) {
        const float2 a = cadd(x[0], x[2 * ST]), b = csub(x[0], x[2 * ST]);
        const float2 c = cadd(x[ST], x[3 * ST]), d = csub(x[ST], x[3 * ST]);
        const float2 e = INV ? make_float2(-d.y, d.x) : make_float2(d.y, -d.x);
        x[0] = cadd(a, c);
        x[ST] = cadd(b, e);
        x[2 * ST] = csub(a, c);
        x[3 * ST] = csub(b, e);
    } else {
        // n = A n1 + n2 (n1 < B), k = k1 + B k2
        constexpr int B = 4, A = R / 4;
        float2 t[R];
#pragma unroll
        for (int n2 = 0; n2 < A; ++n2) {
            float2 y[B];
#pragma unroll
            for (int n1 = 0; n1 < B; ++n1) y[n1] = x[(A * n1 + n2) * ST];
            dft<B, INV, FINE>(y);
#pragma unroll
            for (int k1 = 0; k1 < B; ++k1) t[k1 * A + n2] = rot32<INV, FINE>(y[k1], n2 * k1 * (32 / R));
        }
#pragma unroll
        for (int k1 = 0; k1 < B; ++k1) {
            dft<A, INV, FINE>(t + k1 * A);
#pragma unroll
            for (int k2 = 0; k2 < A; ++k2) x[(k1 + B * k2) * ST] = t[k1 * A + k2];
        }
    }
}

// forward DFT of R points whose upper half is zero (zero padding): x[0 .. R/2) in, x[0 .. R) out
template <int R>
__device__ __forceinline__ void dft_half_in(float2* x)
{
    float2 e[R / 2], o[R / 2];
#pragma unroll
    for (int n = 0; n < R / 2; ++n) { e[n] = x[n]; o[n] = rot32<false>(x[n], n * (32 / R)); }
    dft<R / 2, false>(e);
    dft<R / 2, false>(o);
#pragma unroll
    for (int k = 0; k < R / 2; ++k) { x[2 * k] = e[k]; x[2 * k + 1] = o[k]; }
}
// inverse DFT of R points of which only outputs 0 .. R/2 are wanted (truncation)
template <int R>
__device__ __forceinline__ void dft_half_out(float2* x)
{
    float2 e[R / 2], o[R / 2];
#pragma unroll
    for (int k = 0; k < R / 2; ++k) { e[k] = x[2 * k]; o[k] = x[2 * k + 1]; }
    dft<R / 2, true>(e);
    dft<R / 2, true>(o);
#pragma unroll
    for (int n = 0; n < R / 2; ++n) x[n] = cadd(e[n], rot32<true>(o[n], n * (32 / R)));
}

// exp(-2 pi i d / 4R), d < R: the twist's share of a butterfly of R points (single rows); LOW: what fp32 leaves of it
template <int R, bool LOW = false>
__device__ __forceinline__ float2 twist_unit(int d)
{
    static_assert(R == 8 || R == 16, "the points of a thread");
    constexpr double C[17] = {1., 0.99518472667219689, 0.98078528040323045, 0.95694033573220887, 0.92387953251128676, 0.88192126434835503,
                              0.83146961230254524, 0.77301045336273696, 0.70710678118654752, 0.63439328416364550, 0.55557023301960222,
                              0.47139673682599764, 0.38268343236508977, 0.29028467725446237, 0.19509032201612827, 0.098017140329560602, 0.};
    const int m = d * (16 / R);
    const double c = C[m], s = -C[16 - m];
    return LOW ? make_float2((float)(c - (double)(float)c), (float)(s - (double)(float)s)) : make_float2((float)c, (float)s);
}

// The compiler keeps what it can prove unchanged: without this it would hold every twiddle and spectrum value of a
// transform in registers from one transform (and one turn of the pair loop) to the next, and spill.
// (The pointer itself stays visible: hidden, its loads become flat ones, which every wait for LDS waits for as well.)
template <class T>
__device__ __forceinline__ T* fresh(T* p)
{
    size_t zero = 0;
    asm volatile("" : "+s"(zero));
    return p + zero;
}
// p[i + lane], i the same for all lanes
template <class T>
__device__ __forceinline__ T* at(T* p, size_t i, int lane) { return p + i + (unsigned)lane; }
__device__ __forceinline__ int fresh(int v)      // the same for addresses derived from the thread's number
{
    asm volatile("" : "+v"(v));
    return v;
}

// ---- stage twiddles -----------------------------------------------------------------------------------------------
// The table holds w_{2^l}^q, q < 2^(l-1), at entry 2^(l-1) + q.  w_Ls^(k q) for a radix-r stage needs q < Ls / r: the
// powers 1, 2, 4, 8 are unit-stride runs of the tables of l = lgs, lgs-1, lgs-2, lgs-3, the others products of them.
template <int BITS>
struct StageTw {
    float2 w[BITS];
    __device__ __forceinline__ void load(const float2* __restrict__ ft, int lgs, int q)
    {
#pragma unroll
        for (int i = 0; i < BITS; ++i) w[i] = *at(ft, 1 << (lgs - 1 - i), q);
    }
    // x[k] *= w^k (INV: conj), as w^(k & ~3) and then w^(k & 3): as many multiplications as forming all the powers, and
    // only six of them live
    template <bool INV>
    __device__ __forceinline__ void apply(float2* x) const
    {
        constexpr int R = 1 << BITS;
        const auto mul = [](float2 v, float2 t) { return INV ? cmulc(v, t) : cmul(v, t); };
#pragma unroll
        for (int g = 1; g < R / 4; ++g) {
            const float2 t = g == 1 ? w[2] : g == 2 ? w[BITS - 1] : cmul(w[2], w[BITS - 1]);
#pragma unroll
            for (int k = 0; k < 4; ++k) x[4 * g + k] = mul(x[4 * g + k], t);
        }
        if constexpr (BITS == 1) {
            x[1] = mul(x[1], w[0]);
        } else {
            const float2 t3 = cmul(w[0], w[1]);
#pragma unroll
            for (int g = 0; g < R / 4; ++g) {
                x[4 * g + 1] = mul(x[4 * g + 1], w[0]);
                x[4 * g + 2] = mul(x[4 * g + 2], w[1]);
                x[4 * g + 3] = mul(x[4 * g + 3], t3);
            }
        }
    }
};

// The same with every power from a table (Tables::stw) and one multiplication per point: the least rounding, for the
// transforms that have the registers.  A radix-r stage of stride M reads w_{r M}^(k q) as w_{16 M}^((16 k / r) q).
template <int BITS>
struct StageTwAll {
    float2 w[(1 << BITS) - 1];
    __device__ __forceinline__ void load(const float2* __restrict__ stw, int lgs, int q)
    {
        const int lgM = lgs - BITS;
#pragma unroll
        for (int k = 1; k < (1 << BITS); ++k) w[k - 1] = *at(stw, stw_offset(lgM + 4) + ((k << (4 - BITS)) << lgM), q);
    }
    template <bool INV>
    __device__ __forceinline__ void apply(float2* x) const
    {
#pragma unroll
        for (int k = 1; k < (1 << BITS); ++k) x[k] = INV ? cmulc(x[k], w[k - 1]) : cmul(x[k], w[k - 1]);
    }
};

// Single rows, with tables in two factors, x[k] *= w^(k & ~3) w^(k & 3), each from a table: half the loads and registers of one
// factor for every power, 12 multiplications more at radix 16.  TWIST: stage 0 of N = 2^lgs samples, with the twist of its
// points' q, w_4N^((4k + 1) q), which rides on the factors of the groups of four.
template <int BITS, bool TWIST>
struct StageTwPairs {
    static constexpr int R = 1 << BITS, G0 = TWIST ? 0 : 1, NG = R / 4 > G0 ? R / 4 - G0 : 1;
    float2 f[NG], w[3];
    __device__ __forceinline__ void load(const float2* __restrict__ stw, int lgs, int q)
    {
        const int lgM = lgs - BITS;
#pragma unroll
        for (int g = G0; g < R / 4; ++g)
            f[g - G0] = *at(stw, TWIST ? twist_offset(lgs) + ((4 * g) << lgM) : stw_offset(lgM + 4) + (((4 * g) << (4 - BITS)) << lgM), q);
#pragma unroll
        for (int k = 1; k < 4 && k < R; ++k) w[k - 1] = *at(stw, stw_offset(lgM + 4) + ((k << (4 - BITS)) << lgM), q);
    }
    template <bool INV>
    __device__ __forceinline__ void apply(float2* x) const
    {
        const auto mul = [](float2 v, float2 t) { return INV ? cmulc(v, t) : cmul(v, t); };
#pragma unroll
        for (int k = 0; k < R; ++k) {
            if (k / 4 >= G0) x[k] = mul(x[k], f[k / 4 >= G0 ? k / 4 - G0 : 0]);
            if (k & 3) x[k] = mul(x[k], w[(k & 3) - 1]);
        }
    }
};
// the twist's stage with every power from its table
template <int BITS>
struct StageTwTwist {
    float2 w[1 << BITS];
    __device__ __forceinline__ void load(const float2* __restrict__ stw, int lg, int q)
    {
#pragma unroll
        for (int k = 0; k < (1 << BITS); ++k) w[k] = *at(stw, twist_offset(lg) + (k << (lg - BITS)), q);
    }
    template <bool INV>
    __device__ __forceinline__ void apply(float2* x) const
    {
#pragma unroll
        for (int k = 0; k < (1 << BITS); ++k) x[k] = INV ? cmulc(x[k], w[k]) : cmul(x[k], w[k]);
    }
};
// Which of them a stage of a single row takes, by time and error: at N = 2048 (eight points per thread) two factors in the
// inner stages (B=16, H=256 step 90.7 us, one factor everywhere 98), beyond in stage 0 (B=4, H=96, N=8192 step 59.3 us, one
// everywhere 64.4, two everywhere 58.8 with 9 % more error).
template <int LG, int BITS, bool FIRST>
using RowTw = typename std::conditional<FIRST, typename std::conditional<LG == 11, StageTwTwist<BITS>, StageTwPairs<BITS, true>>::type,
                                        typename std::conditional<LG == 11, StageTwPairs<BITS, false>, StageTwAll<BITS>>::type>::type;

// ALL: the tables handed to the transforms are Tables::stw and every power comes from there
// TWIST: N points of a single real row (see frow_conv_kernel), in and out as the real parts of x; x[n] w^-n with
// w = exp(i pi / 2N), where n = q + d T of a thread's points: the part of d is a constant of the butterfly, that of q rides on
// the twiddles of stage 0
template <int LG, bool ALL = false, bool TWIST = false, int PAD = fft_pad(LG)>
struct Fft {
    static constexpr int N = 1 << LG, P = 1 << points_log2(LG), T = N / P, S = stages(LG);
    static constexpr size_t LDS = sizeof(float2) * phys<PAD>(N);
    static constexpr bool FINE = TWIST && row_fine(LG);

    template <int s>
    struct St {
        static constexpr int bits = stage_bits(LG, s), r = 1 << bits, G = P / r;
        static constexpr int lgs = span_log2(LG, s), lgM = lgs - bits;
        static constexpr bool twist = TWIST && s == 0;
        typename std::conditional<TWIST, RowTw<LG, bits, twist>, typename std::conditional<ALL, StageTwAll<bits>, StageTw<bits>>::type>::type tw[G];
        // butterfly g of thread tid: number tid + g T, q = its low lgM bits
        __device__ __forceinline__ static int q_of(int tid, int g) { return (tid + g * T) & ((1 << lgM) - 1); }
        __device__ __forceinline__ static int base(int tid, int g)
        {
            const int b = tid + g * T;
            return ((b >> lgM) << lgs) | (b & ((1 << lgM) - 1));
        }
        __device__ __forceinline__ void load_tw(const float2* __restrict__ ft, int tid)
        {
            if constexpr (lgM > 0) {
#pragma unroll
                for (int g = 0; g < G; ++g) tw[g].load(ft, lgs, q_of(tid, g));
            }
        }
        template <bool INV>
        __device__ __forceinline__ void twiddle(float2 (&x)[P]) const
        {
            if constexpr (lgM > 0) {
#pragma unroll
                for (int g = 0; g < G; ++g) tw[g].template apply<INV>(x + g * r);
            }
        }
        __device__ __forceinline__ static void write(const float2 (&x)[P], float2* sm, int tid)
        {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float2* b = sm + phys<PAD>(base(tid, g));
#pragma unroll
                for (int d = 0; d < r; ++d) b[phys<PAD>(d << lgM)] = x[g * r + d];
            }
        }
        __device__ __forceinline__ static void read(float2 (&x)[P], const float2* sm, int tid)
        {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float2* b = sm + phys<PAD>(base(tid, g));
#pragma unroll
                for (int d = 0; d < r; ++d) x[g * r + d] = b[phys<PAD>(d << lgM)];
            }
        }
    };

    // x holds the points of stage s; HALF: those of stage 0 have a zero upper half
    template <bool HALF, int s = 0>
    static __device__ __forceinline__ void fwd_from(float2 (&x)[P], const St<s>& st, float2* sm,
                                                    const float2* __restrict__ ft, int tid)
    {
        using C = St<s>;
        if constexpr (C::twist) {
#pragma unroll
            for (int d = 0; d < P; ++d) {
                const float2 c = twist_unit<P>(d);
                if (FINE && LG == 11 && d) {
                    const float2 l = twist_unit<P, true>(d);
                    x[d] = make_float2(__builtin_fmaf(x[d].x, c.x, x[d].x * l.x), __builtin_fmaf(x[d].x, c.y, x[d].x * l.y));
                } else {
                    x[d] = make_float2(x[d].x * c.x, x[d].x * c.y);
                }
            }
        }
#pragma unroll
        for (int g = 0; g < C::G; ++g) {
            if constexpr (HALF && s == 0) dft_half_in<C::r>(x + g * C::r);
            else dft<C::r, false, FINE>(x + g * C::r);
        }
        st.template twiddle<false>(x);
        if constexpr (s + 1 < S) {
            St<s + 1> nx;
            __builtin_amdgcn_sched_barrier(0);
            nx.load_tw(ft, tid);               // in front of the barrier: the loads fly while the waves meet
            C::write(x, sm, tid);
            __syncthreads();
            St<s + 1>::read(x, sm, tid);
            __builtin_amdgcn_sched_barrier(0);
            fwd_from<HALF, s + 1>(x, nx, sm, ft, tid);
        }
    }
    template <bool HALF>
    static __device__ __forceinline__ void fwd(float2 (&x)[P], float2* sm, const float2* __restrict__ ft, int tid)
    {
        ft = fresh(ft);
        tid = fresh(tid);
        St<0> st;
        st.load_tw(ft, tid);
        fwd_from<HALF, 0>(x, st, sm, ft, tid);
    }
    // inverse of the above; HALF: only the lower half of stage 0's points is wanted
    template <bool HALF, int s = S - 1>
    static __device__ __forceinline__ void inv_from(float2 (&x)[P], const St<s>& st, float2* sm,
                                                    const float2* __restrict__ ft, int tid)
    {
        using C = St<s>;
        st.template twiddle<true>(x);
#pragma unroll
        for (int g = 0; g < C::G; ++g) {
            if constexpr (HALF && s == 0) dft_half_out<C::r>(x + g * C::r);
            else dft<C::r, true, FINE>(x + g * C::r);
        }
        if constexpr (C::twist) {
#pragma unroll
            for (int d = 0; d < P; ++d) {
                const float2 c = twist_unit<P>(d);
                x[d].x = __builtin_fmaf(x[d].y, c.y, x[d].x * c.x);
            }
        }
        if constexpr (s > 0) {
            St<s - 1> nx;
            __builtin_amdgcn_sched_barrier(0);
            nx.load_tw(ft, tid);
            C::write(x, sm, tid);
            __syncthreads();
            St<s - 1>::read(x, sm, tid);
            __builtin_amdgcn_sched_barrier(0);
            inv_from<HALF, s - 1>(x, nx, sm, ft, tid);
        }
    }
    template <bool HALF>
    static __device__ __forceinline__ void inv(float2 (&x)[P], float2* sm, const float2* __restrict__ ft, int tid)
    {
        ft = fresh(ft);
        tid = fresh(tid);
        St<S - 1> st;
        st.load_tw(ft, tid);
        inv_from<HALF, S - 1>(x, st, sm, ft, tid);
    }

    // inner frequency of register j of thread tid after the forward stages (digits k_0 + r_0 (k_1 + r_1 (...)))
    static __device__ __forceinline__ uint32_t freq_of(int tid, int j)
    {
        using C = St<S - 1>;
        const uint32_t pos = (uint32_t)C::base(tid, j / C::r) + (j % C::r);
        uint32_t f = 0;
        int have = 0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int b = stage_bits(LG, s);
            f |= ((pos >> (span_log2(LG, s) - b)) & ((1u << b) - 1u)) << have;
            have += b;
        }
        return f;
    }
    // the stored spectrum of a chunk: registers 2i and 2i+1 of a thread side by side, neighbouring threads next to
    // each other, so that every load is a unit-stride run of 16 bytes per lane
    static __device__ __forceinline__ size_t spec_at(int tid, int i) { return (size_t)i * (2 * T) + 2 * tid; }
};

// ---- pass A while loading (multi-pass split) ------------------------------------------------------------------------
// Chunk k1's input sample n2 is w_L^(n2 k1) sum_{n1 < R/2} w_R^(n1 k1) z[n1 L2 + n2] (Section 3.2, "Three-Pass
// Algorithm"): formed from the rows by every chunk's workgroup, so that no complex workspace is written and read in
// front of the inner transforms.  The twist of sample q + d T is that of q times a factor that only depends on d.
template <int LG>
struct Chunk {
    int log2R, k1;
    float2 wq;                  // w_L^(k1 q)
    const float2* tw;
    __device__ __forceinline__ void init(const float2* __restrict__ tw_, int log2R_, int k1_, int tid)
    {
        tw = tw_; log2R = log2R_; k1 = k1_;
        wq = tw_full(tw, ((uint32_t)(k1 * tid) << (TW_LOG2 - LG - log2R)) & (TW_L - 1));
    }
    __device__ __forceinline__ float2 root(int n1) const      // w_R^(n1 k1)
    {
        return tw_full(tw, (uint32_t)((n1 * k1) & ((1 << log2R) - 1)) << (TW_LOG2 - log2R));
    }
    __device__ __forceinline__ float2 twist(int d) const      // w_L^(k1 (q + d T))
    {
        using F = Fft<LG>;
        return cmul(wq, tw_full(tw, ((uint32_t)(k1 * d * F::T) << (TW_LOG2 - LG - log2R)) & (TW_L - 1)));
    }
};

// ---- kernel spectrum (Algorithm 2 lines 1-2) -------------------------------------------------------------------------
// grid = (R, H).  The skip term D[h]*u is the convolution with a delta of height D[h], whose spectrum is the constant
// D[h]; it is added here so the fused kernels never touch D.  OWN: stored in the lane order of this file's kernels;
// otherwise scattered to the consumer's order.
template <int LG, bool OWN>
__global__ void __launch_bounds__(Fft<LG>::T)
fkspec_kernel(const float* __restrict__ k, const float* __restrict__ D, float2* __restrict__ kspec, int64_t N, int log2R,
              SpecOrder consumer, float scale, const float2* __restrict__ tw, const float2* __restrict__ ft)
{
    using F = Fft<LG>;
    constexpr int P = F::P, T = F::T;
    extern __shared__ float2 sm[];
    const int k1 = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const float* kr = k + (size_t)h * N;
    float2 x[P];
    if (log2R == 0) {
#pragma unroll
        for (int d = 0; d < P / 2; ++d) x[d] = make_float2(kr[tid + d * T], 0.f);
        F::template fwd<true>(x, sm, ft, tid);
    } else {
        Chunk<LG> c;
        c.init(tw, log2R, k1, tid);
#pragma unroll
        for (int d = 0; d < P; ++d) x[d] = make_float2(0.f, 0.f);
        for (int n1 = 0; n1 < (1 << log2R) / 2; ++n1) {
            const float2 w = c.root(n1);
#pragma unroll
            for (int d = 0; d < P; ++d) {
                const float v = kr[((size_t)n1 << LG) + tid + d * T];
                x[d].x += w.x * v;
                x[d].y += w.y * v;
            }
        }
#pragma unroll
        for (int d = 0; d < P; ++d) x[d] = cmul(x[d], c.twist(d));
        F::template fwd<false>(x, sm, ft, tid);
    }
    const float dh = D ? D[h] : 0.f;
    float2* out = kspec + ((size_t)h << (LG + log2R));
    if (OWN) out += (size_t)k1 << LG;
#pragma unroll
    for (int i = 0; i < P / 2; ++i) {
        const float2 a = make_float2((x[2 * i].x + dh) * scale, x[2 * i].y * scale);
        const float2 b = make_float2((x[2 * i + 1].x + dh) * scale, x[2 * i + 1].y * scale);
        if (OWN) {
            *reinterpret_cast<float4*>(out + F::spec_at(tid, i)) = make_float4(a.x, a.y, b.x, b.y);
        } else {
            out[spec_pos((uint32_t)k1 + (F::freq_of(tid, 2 * i) << log2R), consumer)] = a;
            out[spec_pos((uint32_t)k1 + (F::freq_of(tid, 2 * i + 1) << log2R), consumer)] = b;
        }
    }
}

// Spectrum of each head's filter in natural frequency order, Shat[h,f] = sum_{s<N} k[h,s] exp(-2 pi i f s / L) + D[h], and
// its adjoint dk[h,s] = Re sum_f exp(+2 pi i f s / L) dShat[h,f], dD[h] = Re sum_f dShat[h,f] (learned Butterfly layer,
// block-size study).  One workgroup per head; the frequencies go through LDS once more, so that memory sees whole
// lines.  Bound by memory latency and launch (12 MB at H = 768, N = 1024): a radix-2 transform with its L points in LDS
// throughout took 22.6 and 20.8 us there, this one 8.0 and 7.4, at 2-10 % less rounding error.
// The LDS place of frequency f XORs its low four bits with those from 4 and from 7 on: 16 neighbouring threads meet 16 banks
// both with neighbouring pairs of frequencies and with those of their last stage (2^9 points: two cycles there; as padded as
// the transform's own exchanges: two and two to eight).  H = 1030, N = 1024 9.2 -> 8.2 us and 6.9 -> 6.0, H = 768 7.0 -> 6.6 and
// 5.3 -> 4.85; N = 2048, H = 768 10.3 -> 9.5 and 7.45 -> 7.35.  Up to 2^10 points the XORs cost more than the conflicts, and the places
// are padded: padded and XORed, H = 300, N = 256 2.50 and 2.60 us, 2.56 and 2.63, N = 512 3.23 and 3.39, 3.05 and 3.13.
template <int LG>
__device__ __forceinline__ int natural_place(uint32_t f)
{
    return LG <= 10 ? phys<fft_pad(LG)>((int)f) : (int)(f ^ (((f >> 4) ^ (f >> 7)) & 15u));
}
template <int LG>
__global__ void __launch_bounds__(Fft<LG>::T)
spectrum_natural_kernel(const float* __restrict__ k, const float* __restrict__ D, float2* __restrict__ shat,
                        const float2* __restrict__ stw)
{
    using F = Fft<LG, true>;
    constexpr int P = F::P, T = F::T;
    extern __shared__ float2 sm[];
    const int h = blockIdx.x, tid = threadIdx.x;
    const float* kr = k + ((size_t)h << (LG - 1));
    const float dh = D[h];
    float2 x[P];
#pragma unroll
    for (int d = 0; d < P / 2; ++d) x[d] = make_float2(kr[tid + d * T], 0.f);
    F::template fwd<true>(x, sm, stw, tid);
    __syncthreads();                    // the last stage's points have been read
#pragma unroll
    for (int j = 0; j < P; ++j) sm[natural_place<LG>(F::freq_of(tid, j))] = x[j];
    __syncthreads();
    float4* out = reinterpret_cast<float4*>(shat + ((size_t)h << LG));
#pragma unroll
    for (int i = 0; i < P / 2; ++i) {
        const int f = 2 * (tid + i * T);
        const float2 a = sm[natural_place<LG>(f)], b = sm[natural_place<LG>(f + 1)];
        out[tid + i * T] = make_float4(a.x + dh, a.y, b.x + dh, b.y);
    }
}

template <int LG>
__global__ void __launch_bounds__(Fft<LG>::T)
spectrum_natural_bwd_kernel(const float2* __restrict__ dshat, float* __restrict__ dk, float* __restrict__ dD,
                            const float2* __restrict__ stw)
{
    using F = Fft<LG, true>;
    constexpr int P = F::P, T = F::T;
    extern __shared__ float2 sm[];
    const int h = blockIdx.x, tid = threadIdx.x;
    const float4* in = reinterpret_cast<const float4*>(dshat + ((size_t)h << LG));
#pragma unroll
    for (int i = 0; i < P / 2; ++i) {
        const int f = 2 * (tid + i * T);
        const float4 v = in[tid + i * T];
        sm[natural_place<LG>(f)] = make_float2(v.x, v.y);
        sm[natural_place<LG>(f + 1)] = make_float2(v.z, v.w);
    }
    __syncthreads();
    float2 x[P];
#pragma unroll
    for (int j = 0; j < P; ++j) x[j] = sm[natural_place<LG>(F::freq_of(tid, j))];
    __syncthreads();
    F::template inv<true>(x, sm, stw, tid);
    if (dk) {
        float* out = dk + ((size_t)h << (LG - 1));
#pragma unroll
        for (int d = 0; d < P / 2; ++d) out[tid + d * T] = x[d].x;
    }
    if (dD && tid == 0) dD[h] = x[0].x;
}

// the points of stage 0 of one source's row pair
template <int LG, class IO, bool CHUNK>
__device__ __forceinline__ void load_pair(float2 (&x)[Fft<LG>::P], const typename IO::T* __restrict__ ra,
                                          const typename IO::T* __restrict__ rb, bool has_b, const Chunk<LG>& c, int tid)
{
    tid = fresh(tid);
    constexpr int P = Fft<LG>::P, T = Fft<LG>::T;
    if constexpr (!CHUNK) {
#pragma unroll
        for (int d = 0; d < P / 2; ++d) {          // (a missing second row: rb = ra, read and dropped, no branches)
            const float a = IO::ld(ra, tid + d * T), b = IO::ld(rb, tid + d * T);
            x[d] = make_float2(a, has_b ? b : 0.f);
        }
    } else {
#pragma unroll
        for (int d = 0; d < P; ++d) x[d] = make_float2(0.f, 0.f);
        for (int n1 = 0; n1 < (1 << c.log2R) / 2; ++n1) {
            const float2 w = c.root(n1);
            const typename IO::T* pa = ra + ((size_t)n1 << LG);
            const typename IO::T* pb = rb + ((size_t)n1 << LG);
            if (has_b) {
#pragma unroll
                for (int d = 0; d < P; ++d) {
                    const float2 z = make_float2(IO::ld(pa, tid + d * T), IO::ld(pb, tid + d * T));
                    x[d].x += z.x * w.x - z.y * w.y;
                    x[d].y += z.x * w.y + z.y * w.x;
                }
            } else {
#pragma unroll
                for (int d = 0; d < P; ++d) {
                    const float v = IO::ld(pa, tid + d * T);
                    x[d].x += v * w.x;
                    x[d].y += v * w.y;
                }
            }
        }
#pragma unroll
        for (int d = 0; d < P; ++d) x[d] = cmul(x[d], c.twist(d));
    }
}
// rows (or chunk k1 of the pair's complex workspace) <- the points of stage 0
template <int LG, class IO, bool CHUNK>
__device__ __forceinline__ void store_pair(const float2 (&x)[Fft<LG>::P], typename IO::T* __restrict__ ra,
                                           typename IO::T* __restrict__ rb, bool has_b, float2* __restrict__ chunk, int tid)
{
    tid = fresh(tid);
    constexpr int P = Fft<LG>::P, T = Fft<LG>::T;
    if constexpr (!CHUNK) {
#pragma unroll
        for (int d = 0; d < P / 2; ++d) IO::once(ra, tid + d * T, x[d].x);
        if (has_b) {
#pragma unroll
            for (int d = 0; d < P / 2; ++d) IO::once(rb, tid + d * T, x[d].y);
        }
    } else {
#pragma unroll
        for (int d = 0; d < P; ++d) chunk[tid + d * T] = x[d];
    }
}

template <class F, bool CONJ>
__device__ __forceinline__ void times_spectrum(float2 (&x)[F::P], const float2* __restrict__ ks, int tid)
{
    tid = fresh(tid);
#pragma unroll
    for (int i = 0; i < F::P / 2; ++i) {
        const float4 k = *at(reinterpret_cast<const float4*>(ks), F::spec_at(0, i) / 2, tid);
        const float2 ka = make_float2(k.x, k.y), kb = make_float2(k.z, k.w);
        x[2 * i] = CONJ ? cmulc(x[2 * i], ka) : cmul(x[2 * i], ka);
        x[2 * i + 1] = CONJ ? cmulc(x[2 * i + 1], kb) : cmul(x[2 * i + 1], kb);
    }
}

// ---- fused convolution of one row pair (Eq. 2 fused as in Section 3.2 "Kernel Fusion") --------------------------------
//   single pass: z[n] = in[2p,h,n] + i*in[2p+1,h,n], zero padded to L; forward, multiply by the stored spectrum (or its
//     conjugate: correlation, used for du), inverse, keep the first N samples: re -> out row 2p, im -> out row 2p+1.
//     Convolution with a real kernel is real-linear, so the two rows never mix.
//   CHUNK: the same on chunk k1 of the multi-pass split, pass A taken while loading, result to the pair's complex
//     workspace (Eq. 3: m independent convolutions of length l).
// grid = (npairs, H, R)
template <int LG, class IO, bool CHUNK>
__global__ void __launch_bounds__(Fft<LG>::T)
fconv_kernel(const typename IO::T* __restrict__ in, const float2* __restrict__ kspec, typename IO::T* __restrict__ out,
             float2* __restrict__ ws, int conj, int64_t B, int64_t H, int64_t N, int log2R, const float2* __restrict__ tw,
             const float2* __restrict__ ft)
{
    using F = Fft<LG>;
    extern __shared__ float2 sm[];
    const int p = blockIdx.x, h = blockIdx.y, k1 = blockIdx.z, tid = threadIdx.x;
    const bool has_b = (2 * p + 1) < B;
    const size_t oa = row_off(2 * p, h, H, N), ob = row_off(has_b ? 2 * p + 1 : 2 * p, h, H, N);
    float2 x[F::P];
    Chunk<LG> c;
    if constexpr (CHUNK) c.init(tw, log2R, k1, tid);
    load_pair<LG, IO, CHUNK>(x, in + oa, in + ob, has_b, c, tid);
    F::template fwd<!CHUNK>(x, sm, ft, tid);
    const float2* ks = kspec + ((size_t)h << (LG + log2R)) + ((size_t)k1 << LG);
    if (conj) times_spectrum<F, true>(x, ks, tid);
    else times_spectrum<F, false>(x, ks, tid);
    F::template inv<!CHUNK>(x, sm, ft, tid);
    float2* chunk = CHUNK ? ws + (((size_t)h * gridDim.x + p) << (LG + log2R)) + ((size_t)k1 << LG) : nullptr;
    store_pair<LG, IO, CHUNK>(x, out + oa, out + ob, has_b, chunk, tid);
}

// ---- backward: du, dk and dD in one walk over the head's row pairs ------------------------------------------------------
// One workgroup per (share, head, chunk); share s of nsplit takes pairs s, s + nsplit, ... in order (deterministic).
// Per pair: u -> Z, dy -> W, A += conj(Z) W in registers, then (du asked for) W conj(K) back through the inverse.  The
// real part of the inverse transform of A is the sum over both rows of the correlation dy (x) u, i.e. the pair's share of
// dk (the cross terms between the two rows are purely imaginary).  dD is the plain dot product, taken while both
// sources' rows are in registers.  dy is read and transformed once for both gradients.
//   dk: [nsplit][H][N] real samples times `scale`, or (CHUNK) A: [nsplit][H][R][L2] complex for pass C
//   dD: [nsplit][H]
// At L2 = 16384 a thread may hold 128 registers (sixteen waves); accumulators, Z and the points in work do not fit into
// them (spilled: 120 registers a thread), so Z waits in zbuf, [R][H][nsplit] sequences that stay in L2, written and
// read by the same thread (B=4, H=96, N=8192, then in pairs: 62 -> 47 us).  48 are spilled all the same.
template <int LG, class IO, bool CHUNK>
__global__ void __launch_bounds__(Fft<LG>::T)
fbwd_kernel(const typename IO::T* __restrict__ dy, const typename IO::T* __restrict__ u, const float2* __restrict__ kspec,
            typename IO::T* __restrict__ du, float2* __restrict__ ws_du, float* __restrict__ dk, float2* __restrict__ ws_A,
            float* __restrict__ dD, float4* __restrict__ zbuf, int64_t B, int64_t H, int64_t N, int npairs, int log2R,
            float scale, const float2* __restrict__ tw, const float2* __restrict__ ft)
{
    constexpr bool PARK = valu_parks(LG);
    constexpr bool PREFETCH = LG <= 13;       // dy's rows fetched with u's: where the registers for them are there
    if constexpr (PARK) zbuf += ((size_t)(blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) << (LG - 1);
    using F = Fft<LG>;
    constexpr int P = F::P, T = F::T;
    extern __shared__ float2 sm[];
    __shared__ float red[T >= 64 ? T / 64 : 1];
    const int share = blockIdx.x, nsplit = gridDim.x, h = blockIdx.y, k1 = blockIdx.z, tid = threadIdx.x;
    const bool want_du = CHUNK ? ws_du != nullptr : du != nullptr;
    const float2* ks = kspec + ((size_t)h << (LG + log2R)) + ((size_t)k1 << LG);
    Chunk<LG> c;
    if constexpr (CHUNK) c.init(tw, log2R, k1, tid);
    float2 acc[P];
#pragma unroll
    for (int i = 0; i < P; ++i) acc[i] = make_float2(0.f, 0.f);
    float dsum = 0.f;
    for (int p = share; p < npairs; p += nsplit) {
        const bool has_b = (2 * p + 1) < B;
        const size_t oa = row_off(2 * p, h, H, N), ob = row_off(has_b ? 2 * p + 1 : 2 * p, h, H, N);
        float2 z[P], w[P];
        load_pair<LG, IO, CHUNK>(z, u + oa, u + ob, has_b, c, tid);
        if constexpr (!CHUNK && PREFETCH) {
            load_pair<LG, IO, CHUNK>(w, dy + oa, dy + ob, has_b, c, tid);
#pragma unroll
            for (int d = 0; d < P / 2; ++d) dsum += z[d].x * w[d].x + z[d].y * w[d].y;
        } else if (CHUNK && k1 == 0 && dD) {
            // (several samples in flight: one at a time, N = 65536 took 64 round trips to memory in a row)
            for (int row = 0; row < (has_b ? 2 : 1); ++row) {
                const typename IO::T* pu = u + (row ? ob : oa);
                const typename IO::T* pd = dy + (row ? ob : oa);
#pragma unroll 16
                for (int n = 0; n < (int)N; n += T) dsum += IO::ld(pu, n + tid) * IO::ld(pd, n + tid);
            }
        }
        F::template fwd<!CHUNK>(z, sm, ft, tid);
        if constexpr (PARK) {
            const int t = fresh(tid);
#pragma unroll
            for (int i = 0; i < P / 2; ++i) zbuf[i * T + t] = make_float4(z[2 * i].x, z[2 * i].y, z[2 * i + 1].x, z[2 * i + 1].y);
        }
        if constexpr (CHUNK || !PREFETCH) load_pair<LG, IO, CHUNK>(w, dy + oa, dy + ob, has_b, c, tid);
        if constexpr (!CHUNK && !PREFETCH) {  // (u once more, from L2, instead of dy's rows held through z's transform)
            if (dD) {
                float2 v[P];
                load_pair<LG, IO, CHUNK>(v, u + oa, u + ob, has_b, c, fresh(tid));
#pragma unroll
                for (int d = 0; d < P / 2; ++d) dsum += v[d].x * w[d].x + v[d].y * w[d].y;
            }
        }
        __syncthreads();                      // the last stage of z has been read everywhere
        F::template fwd<!CHUNK>(w, sm, ft, tid);
        if constexpr (PARK) {
            const float4* zb = fresh(zbuf);
            const int t = fresh(tid);
#pragma unroll
            for (int i = 0; i < P / 2; ++i) {
                const float4 v = zb[i * T + t];
                z[2 * i] = make_float2(v.x, v.y);
                z[2 * i + 1] = make_float2(v.z, v.w);
            }
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {         // acc += conj(z) * w
            acc[i].x += z[i].x * w[i].x + z[i].y * w[i].y;
            acc[i].y += z[i].x * w[i].y - z[i].y * w[i].x;
        }
        if (want_du) {
            times_spectrum<F, true>(w, fresh(ks), tid);
            F::template inv<!CHUNK>(w, sm, ft, tid);
            float2* chunk = CHUNK ? ws_du + (((size_t)h * npairs + p) << (LG + log2R)) + ((size_t)k1 << LG) : nullptr;
            store_pair<LG, IO, CHUNK>(w, du + oa, du + ob, has_b, chunk, tid);
        } else {
            __syncthreads();
        }
    }
    if (CHUNK ? ws_A != nullptr : dk != nullptr) {
        __syncthreads();
        F::template inv<!CHUNK>(acc, sm, ft, tid);
        const size_t row = (size_t)share * H + h;
        if constexpr (!CHUNK) {
            float* o = dk + row * N;
#pragma unroll
            for (int d = 0; d < P / 2; ++d) o[tid + d * T] = acc[d].x * scale;
        } else {
            float2* o = ws_A + (row << (LG + log2R)) + ((size_t)k1 << LG);
#pragma unroll
            for (int d = 0; d < P; ++d) o[tid + d * T] = acc[d];
        }
    }
    if (dD && k1 == 0) {                      // fixed-order sum over the workgroup
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
        if ((tid & 63) == 0) red[tid >> 6] = dsum;
        __syncthreads();
        if (tid == 0) {
            float t = 0.f;
            for (int i = 0; i < (T + 63) / 64; ++i) t += red[i];
            dD[(size_t)share * H + h] = t;
        }
    }
}

// ---- single fp32 rows of N = 2048 .. 16384 samples ----------------------------------------------------------------------
// The transform of engine_rows.hip in fp32: N twisted points of one real row, whose products are convolutions modulo z^N - i
// with the causal convolution as real part.  Against pairs of rows in 2N points it takes the same arithmetic a row, half the
// LDS, half the spectrum, and twice the workgroups: two rows of 8192 samples share a compute unit and hide each other's
// barriers and memory, and the backward kernel spills little (12 and 16 registers at N = 4096 and 16384, where a pair spilled 43);
// N = 16384 takes no chunks.  Bound by vector issue: 105 instructions per point for a convolution, at 2.6 cycles and four waves
// per SIMD.  Whole steps back to back, pairs and rows: B=4, H=96, N=8192 77.0 -> 58.4 us, B=2, H=300 138 -> 92; B=4, H=96, N=16384
// 197 -> 126; N=4096 44.4 -> 36.1, B=32, H=1024 1336 -> 1326; N=2048 29.0 -> 23.8.  Slower than pairs were: N = 2048 with 16000 rows and
// more (B=16, H=1024 287 -> 296, B=32, H=1024 541 -> 592): there the exchanges bind, three of them where 4096 points of a pair have
// two; with sixteen points a thread (two exchanges) the forward pass of the last is faster, 213 -> 182, but the backward kernel, whose
// accumulator then waits in memory, slower by more (step 575 -> 640); workgroups that keep on, with the next row asked for ahead,
// take 237 for 214.
// Error against 64 bits, y and dk, B = 4 and (a row without a partner had an easier time in a pair) B = 1, pairs -> rows, 1e-7: N = 2048
// 1.91 -> 1.48, 2.83 -> 2.28 and 1.65 -> 1.47, 2.38 -> 2.25; 4096 1.93 -> 1.42, 2.86 -> 2.23 and 1.62 -> 1.41, 2.36 -> 2.19; 8192 2.13 ->
// 1.69, 3.13 -> 2.61 and 1.82 -> 1.69, 2.63 -> 2.58; 16384 2.22 -> 1.82, 3.29 -> 2.79 and 1.89 -> 1.81, 2.77 -> 2.76.  Up to 4096 this
// takes the constants in two parts (row_fine): with one, B = 1 was at 1.72, 2.61 and 1.70, 2.57; time the same to 3 % more (B=1, H=1,
// N=2048 15.6 -> 16.0 us; B=8, H=200 45.2 -> 45.1; N=4096 B=8, H=129 69.5 -> 68.5).
// Neighbouring items on one XCD: the rows of a head share its spectrum there.
__device__ __forceinline__ int item_of(int items)
{
    const int per = (items + 7) >> 3;
    return (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);       // (may lie beyond the last)
}
template <int LG>
using RowFft = Fft<LG, true, true>;
template <int LG>
__device__ __forceinline__ void load_row(float2 (&x)[RowFft<LG>::P], const float* __restrict__ row, int tid)
{
    tid = fresh(tid);
#pragma unroll
    for (int d = 0; d < RowFft<LG>::P; ++d) x[d].x = *at(row, d * RowFft<LG>::T, tid);
}
template <int LG>
__device__ __forceinline__ void store_row(const float2 (&x)[RowFft<LG>::P], float* __restrict__ row, int tid)
{
    tid = fresh(tid);
#pragma unroll
    for (int d = 0; d < RowFft<LG>::P; ++d) put_once(at(row, d * RowFft<LG>::T, tid), x[d].x);
}

template <int LG>
__global__ void __launch_bounds__(RowFft<LG>::T)
frow_kspec_kernel(const float* __restrict__ k, const float* __restrict__ D, float2* __restrict__ kspec, float scale,
                  const float2* __restrict__ stw)
{
    using F = RowFft<LG>;
    extern __shared__ float2 sm[];
    const int h = blockIdx.x, tid = threadIdx.x;
    float2 x[F::P];
    load_row<LG>(x, k + ((size_t)h << LG), tid);
    const float dh = D[h];
    F::template fwd<false>(x, sm, stw, tid);
    float2* out = kspec + ((size_t)h << LG);
#pragma unroll
    for (int i = 0; i < F::P / 2; ++i)
        *at(reinterpret_cast<float4*>(out), F::spec_at(0, i) / 2, tid) =
            make_float4((x[2 * i].x + dh) * scale, x[2 * i].y * scale, (x[2 * i + 1].x + dh) * scale, x[2 * i + 1].y * scale);
}

// Paddings of the convolution at N = 8192, two workgroups on a compute unit: behind every eight slots up to eight rows a unit, behind
// every sixteen beyond (us, eight and sixteen: 512 rows 17.2 and 18.7, 600 23.4 and 25.1, 1024 30.6 and 31.8, 2048 57.2 and 57.2, 3200 88.8
// and 87.3, 4096 111.6 and 109.6; the backward kernel, and one workgroup on a unit: sixteen or no difference).
constexpr int conv_pad(int LG, int64_t rows) { return LG == 13 && rows <= 2048 ? 3 : fft_pad(LG); }
template <int LG, int PAD>
__global__ void __launch_bounds__(RowFft<LG>::T) __attribute__((amdgpu_waves_per_eu(4)))
frow_conv_kernel(const float* __restrict__ in, const float2* __restrict__ kspec, float* __restrict__ out, int conj, int B, int H,
                 const float2* __restrict__ stw)
{
    using F = Fft<LG, true, true, PAD>;
    extern __shared__ float2 sm[];
    const int item = item_of(B * H), tid = threadIdx.x;
    if (item >= B * H) return;
    const int h = item / B;
    const size_t o = row_off(item - h * B, h, H, F::N);
    float2 x[F::P];
    load_row<LG>(x, in + o, tid);
    F::template fwd<false>(x, sm, stw, tid);
    const float2* ks = kspec + ((size_t)h << LG);
    if (conj) times_spectrum<F, true>(x, ks, tid);
    else times_spectrum<F, false>(x, ks, tid);
    F::template inv<false>(x, sm, stw, tid);
    store_row<LG>(x, out + o, tid);
}

// du, dk and dD in one walk over a share of the head's rows, as fbwd_kernel.  A, the sum of conj(U) W, waits in `acc` ([H][nsplit]
// sequences, written and read by the same thread) while the next row is transformed: with it, and U, and the points in work, 128
// registers are not enough.  A share of one row never touches it.
template <int LG>
__global__ void __launch_bounds__(RowFft<LG>::T) __attribute__((amdgpu_waves_per_eu(4)))
frow_bwd_kernel(const float* __restrict__ dy, const float* __restrict__ u, const float2* __restrict__ kspec, float* __restrict__ du,
                float* __restrict__ dk, float* __restrict__ dD, float4* __restrict__ acc, int B, int H, int nsplit, float scale,
                const float2* __restrict__ stw)
{
    using F = RowFft<LG>;
    constexpr int P = F::P, T = F::T;
    extern __shared__ float2 sm[];
    __shared__ float red[T / 64];
    const int item = item_of(H * nsplit), tid = threadIdx.x;
    if (item >= H * nsplit) return;
    const int h = item / nsplit, share = item - h * nsplit;
    acc += (size_t)item << (LG - 1);
    const float2* ks = kspec + ((size_t)h << LG);
    constexpr bool PARK = row_parks(LG);
    float dsum = 0.f;
    float2 z[P], sum[PARK ? 1 : P];
    if constexpr (!PARK) {
#pragma unroll
        for (int i = 0; i < P; ++i) sum[i] = make_float2(0.f, 0.f);
    }
    for (int b = share; b < B; b += nsplit) {
        const size_t o = row_off(b, h, H, F::N);
        float2 w[P];
        load_row<LG>(z, u + o, tid);
        load_row<LG>(w, dy + o, tid);
#pragma unroll
        for (int d = 0; d < P; ++d) dsum = __builtin_fmaf(z[d].x, w[d].x, dsum);
        F::template fwd<false>(z, sm, stw, tid);
        __syncthreads();                      // the last stage of z has been read everywhere
        F::template fwd<false>(w, sm, stw, tid);
#pragma unroll
        for (int i = 0; i < P; ++i) z[i] = cmulc(w[i], z[i]);
        if constexpr (PARK) {
            float4* a = fresh(acc);
            const int t = fresh(tid);
            if (b != share) {
#pragma unroll
                for (int i = 0; i < P / 2; ++i) {
                    const float4 v = *at(a, i * T, t);
                    z[2 * i].x += v.x; z[2 * i].y += v.y;
                    z[2 * i + 1].x += v.z; z[2 * i + 1].y += v.w;
                }
            }
            if (b + nsplit < B) {
#pragma unroll
                for (int i = 0; i < P / 2; ++i) *at(a, i * T, t) = make_float4(z[2 * i].x, z[2 * i].y, z[2 * i + 1].x, z[2 * i + 1].y);
            }
        } else {
#pragma unroll
            for (int i = 0; i < P; ++i) sum[i] = cadd(sum[i], z[i]);
        }
        if (du) {
            times_spectrum<F, true>(w, fresh(ks), tid);
            F::template inv<false>(w, sm, stw, tid);
            store_row<LG>(w, du + o, tid);
        } else {
            __syncthreads();
        }
    }
    if (dk) {
        __syncthreads();
        if constexpr (!PARK) {
#pragma unroll
            for (int i = 0; i < P; ++i) z[i] = sum[i];
        }
        F::template inv<false>(z, sm, stw, tid);
        float* o = dk + (((size_t)share * H + h) << LG);
#pragma unroll
        for (int d = 0; d < P; ++d) *at(o, d * T, tid) = z[d].x * scale;
    }
    if (dD) {                                 // fixed-order sum over the workgroup
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
        if ((tid & 63) == 0) red[tid >> 6] = dsum;
        __syncthreads();
        if (tid == 0) {
            float t = 0.f;
            for (int i = 0; i < T / 64; ++i) t += red[i];
            dD[(size_t)share * H + h] = t;
        }
    }
}

template <class F>
hipError_t set_lds(F* f, size_t bytes)
{
    return hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// twiddles of the stages: entry 2^(l-1) + q = w_{2^l}^q
__device__ float2 g_ftw[1 << VALU_INNER_MAX_LOG2];
__global__ void fill_ftw_kernel(float2* ft)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 1 || i >= (1 << VALU_INNER_MAX_LOG2)) return;
    const int l = 32 - __clz(i), q = i - (1 << (l - 1));
    double s, c;
    sincospi(-2.0 * (double)q / (double)(1 << l), &s, &c);
    ft[i] = make_float2((float)c, (float)s);
}

template <int LG>
__global__ void fill_twist_kernel(float2* stw)
{
    constexpr int T = Fft<LG>::T;
    const int i = blockIdx.x * blockDim.x + threadIdx.x, k = i / T, q = i % T;
    double s, c;
    sincospi(-2.0 * (double)((4 * k + 1) * q) / (double)(4 << LG), &s, &c);
    stw[twist_offset(LG) + i] = make_float2((float)c, (float)s);
}

#define LC_LG_SWITCH(lg, CALL)                \
    switch (lg) {                             \
        case 8: return CALL(8);               \
        case 9: return CALL(9);               \
        case 10: return CALL(10);             \
        case 11: return CALL(11);             \
        case 12: return CALL(12);             \
        case 13: return CALL(13);             \
        case 14: return CALL(14);             \
        default: return hipErrorInvalidValue; \
    }

template <int LG>
hipError_t kspec_go(const float* k, const float* D, float2* kspec, int64_t H, int64_t N, int log2R, const SpecOrder* consumer,
                    float scale, const Tables& tb, hipStream_t st)
{
    const dim3 grid(1u << log2R, (unsigned)H);
    hipError_t e;
    if (!consumer) {
        if ((e = set_lds(fkspec_kernel<LG, true>, Fft<LG>::LDS)) != hipSuccess) return e;
        hipLaunchKernelGGL((fkspec_kernel<LG, true>), grid, dim3(Fft<LG>::T), Fft<LG>::LDS, st, k, D, kspec, N, log2R,
                           SpecOrder{}, scale, tb.tw, tb.ftw);
    } else {
        if ((e = set_lds(fkspec_kernel<LG, false>, Fft<LG>::LDS)) != hipSuccess) return e;
        hipLaunchKernelGGL((fkspec_kernel<LG, false>), grid, dim3(Fft<LG>::T), Fft<LG>::LDS, st, k, D, kspec, N, log2R,
                           *consumer, scale, tb.tw, tb.ftw);
    }
    return hipGetLastError();
}

#define LC_ROWS_SWITCH(lg, CALL)              \
    switch (lg) {                             \
        case 11: return CALL(11);             \
        case 12: return CALL(12);             \
        case 13: return CALL(13);             \
        case 14: return CALL(14);             \
        default: return hipErrorInvalidValue; \
    }

template <int LG>
hipError_t rows_kspec_go(const float* k, const float* D, float2* kspec, int64_t H, float scale, const Tables& tb, hipStream_t st)
{
    const hipError_t e = set_lds(frow_kspec_kernel<LG>, RowFft<LG>::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(frow_kspec_kernel<LG>, dim3((unsigned)H), dim3(RowFft<LG>::T), RowFft<LG>::LDS, st, k, D, kspec, scale, tb.stw);
    return hipGetLastError();
}
// workgroups for a list of items (see item_of)
dim3 item_grid(int64_t items) { return dim3((unsigned)((items + 7) / 8 * 8)); }
template <int LG, int PAD>
hipError_t rows_conv_launch(const float* in, const float2* kspec, float* out, bool conj, const Problem& pr, const Tables& tb, hipStream_t st)
{
    constexpr size_t lds = Fft<LG, true, true, PAD>::LDS;
    const hipError_t e = set_lds(frow_conv_kernel<LG, PAD>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((frow_conv_kernel<LG, PAD>), item_grid(pr.B * pr.H), dim3(RowFft<LG>::T), lds, st, in, kspec, out,
                       conj ? 1 : 0, (int)pr.B, (int)pr.H, tb.stw);
    return hipGetLastError();
}
template <int LG>
hipError_t rows_conv_go(const float* in, const float2* kspec, float* out, bool conj, const Problem& pr, const Tables& tb, hipStream_t st)
{
    return conv_pad(LG, pr.B * pr.H) == 3 ? rows_conv_launch<LG, conv_pad(LG, 0)>(in, kspec, out, conj, pr, tb, st)
                                          : rows_conv_launch<LG, fft_pad(LG)>(in, kspec, out, conj, pr, tb, st);
}
template <int LG>
hipError_t rows_bwd_go(const float* dy, const float* u, const float2* kspec, float* du, float* dk, float* dD, void* acc, int nsplit,
                       const Problem& pr, float scale, const Tables& tb, hipStream_t st)
{
    const hipError_t e = set_lds(frow_bwd_kernel<LG>, RowFft<LG>::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(frow_bwd_kernel<LG>, item_grid(pr.H * nsplit), dim3(RowFft<LG>::T), RowFft<LG>::LDS, st, dy, u, kspec, du, dk, dD,
                       (float4*)acc, (int)pr.B, (int)pr.H, nsplit, scale, tb.stw);
    return hipGetLastError();
}

template <int LG>
hipError_t natural_go(const float* k, const float* D, float2* shat, int64_t H, const Tables& tb, hipStream_t st)
{
    const hipError_t e = set_lds(spectrum_natural_kernel<LG>, Fft<LG>::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(spectrum_natural_kernel<LG>, dim3((unsigned)H), dim3(Fft<LG>::T), Fft<LG>::LDS, st, k, D, shat, tb.stw);
    return hipGetLastError();
}
template <int LG>
hipError_t natural_bwd_go(const float2* dshat, float* dk, float* dD, int64_t H, const Tables& tb, hipStream_t st)
{
    const hipError_t e = set_lds(spectrum_natural_bwd_kernel<LG>, Fft<LG>::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(spectrum_natural_bwd_kernel<LG>, dim3((unsigned)H), dim3(Fft<LG>::T), Fft<LG>::LDS, st, dshat, dk, dD,
                       tb.stw);
    return hipGetLastError();
}

template <int LG, class IO, bool CHUNK>
hipError_t conv_go(const void* in, const float2* kspec, void* out, float2* ws, bool conj, const Problem& pr, int log2R,
                   const Tables& tb, hipStream_t st)
{
    using T = typename IO::T;
    const hipError_t e = set_lds(fconv_kernel<LG, IO, CHUNK>, Fft<LG>::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fconv_kernel<LG, IO, CHUNK>), dim3(pr.npairs, (unsigned)pr.H, 1u << log2R), dim3(Fft<LG>::T),
                       Fft<LG>::LDS, st, (const T*)in, kspec, (T*)out, ws, conj ? 1 : 0, pr.B, pr.H, pr.N, log2R, tb.tw,
                       tb.ftw);
    return hipGetLastError();
}

// pairs of whole rows: of fp32 rows there are those up to N = 1024 (longer ones run by themselves, see make_plan)
template <class IO>
constexpr int alone(int LG) { return std::is_same<IO, IoF32>::value && LG > VALU_ROWS_MIN_LOG2 ? VALU_ROWS_MIN_LOG2 : LG; }
template <class IO>
hipError_t conv_io(const void* in, const float2* kspec, void* out, float2* ws, bool conj, const Problem& pr,
                   const Plan& pl, const Tables& tb, hipStream_t st)
{
#define CALL(LG)                                                                            \
    (pl.log2R ? conv_go<LG, IO, true>(in, kspec, out, ws, conj, pr, pl.log2R, tb, st)        \
              : conv_go<alone<IO>(LG), IO, false>(in, kspec, out, ws, conj, pr, 0, tb, st))
    LC_LG_SWITCH(pl.log2L2, CALL)
#undef CALL
}

template <int LG, class IO, bool CHUNK>
hipError_t bwd_go(const void* dy, const void* u, const float2* kspec, void* du, float2* ws_du, float* dk, float2* ws_A,
                  float* dD, void* zbuf, int nsplit, const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
    using T = typename IO::T;
    const hipError_t e = set_lds(fbwd_kernel<LG, IO, CHUNK>, Fft<LG>::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fbwd_kernel<LG, IO, CHUNK>), dim3(nsplit, (unsigned)pr.H, 1u << pl.log2R), dim3(Fft<LG>::T),
                       Fft<LG>::LDS, st, (const T*)dy, (const T*)u, kspec, (T*)du, ws_du, dk, ws_A, dD, (float4*)zbuf, pr.B, pr.H, pr.N,
                       pr.npairs, pl.log2R, pl.dkscale, tb.tw, tb.ftw);
    return hipGetLastError();
}

template <class IO>
hipError_t bwd_io(const void* dy, const void* u, const float2* kspec, void* du, float2* ws_du, float* dk, float2* ws_A,
                  float* dD, void* zbuf, int nsplit, const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
#define CALL(LG)                                                                                            \
    (pl.log2R ? bwd_go<LG, IO, true>(dy, u, kspec, nullptr, ws_du, nullptr, ws_A, dD, zbuf, nsplit, pr, pl, tb, st) \
              : bwd_go<alone<IO>(LG), IO, false>(dy, u, kspec, du, nullptr, dk, nullptr, dD, zbuf, nsplit, pr, pl, tb, st))
    LC_LG_SWITCH(pl.log2L2, CALL)
#undef CALL
}

}  // namespace

hipError_t valu_fill_tables(const float2** ftw, hipStream_t st)
{
    float2* p = nullptr;
    const hipError_t e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(g_ftw));
    if (e != hipSuccess) return e;
    constexpr int n = 1 << VALU_INNER_MAX_LOG2;
    hipLaunchKernelGGL(fill_ftw_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p);
    *ftw = p;
    return hipGetLastError();
}

hipError_t valu_fill_twist(float2* stw, hipStream_t st)
{
    hipLaunchKernelGGL(fill_twist_kernel<11>, dim3((1 << 11) / 256), dim3(256), 0, st, stw);
    hipLaunchKernelGGL(fill_twist_kernel<12>, dim3((1 << 12) / 256), dim3(256), 0, st, stw);
    hipLaunchKernelGGL(fill_twist_kernel<13>, dim3((1 << 13) / 256), dim3(256), 0, st, stw);
    hipLaunchKernelGGL(fill_twist_kernel<14>, dim3((1 << 14) / 256), dim3(256), 0, st, stw);
    return hipGetLastError();
}

void valu_fill_plan(Plan& pl)
{
    pl.order = SpecOrder{};
    if (pl.log2R) pl.order.bits[pl.order.ndig++] = (unsigned char)pl.log2R;
    const int lg = pl.vrow ? pl.vrow : pl.log2L2;
    for (int s = 0; s < stages(lg); ++s) pl.order.bits[pl.order.ndig++] = (unsigned char)stage_bits(lg, s);
    pl.kscale = pl.dkscale = 1.0f / (float)(int64_t(1) << (pl.vrow ? pl.vrow : pl.log2L));
}

hipError_t valu_kspec(const float* k, const float* D, float2* kspec, int64_t H, int64_t N, const SpecOrder* consumer,
                      float scale, const Tables& tb, int log2R, int log2L2, hipStream_t st)
{
#define CALL(LG) kspec_go<LG>(k, D, kspec, H, N, log2R, consumer, scale, tb, st)
    LC_LG_SWITCH(log2L2, CALL)
#undef CALL
}

hipError_t valu_rows_kspec(const float* k, const float* D, float2* kspec, int64_t H, const Plan& pl, const Tables& tb, hipStream_t st)
{
#define CALL(LG) rows_kspec_go<LG>(k, D, kspec, H, pl.kscale, tb, st)
    LC_ROWS_SWITCH(pl.vrow, CALL)
#undef CALL
}

hipError_t spectrum_natural(const float* k, const float* D, float* shat, int64_t H, int64_t N, const Tables& tb,
                            hipStream_t st)
{
#define CALL(LG) natural_go<LG>(k, D, (float2*)shat, H, tb, st)
    switch (N) {
        case 256: return CALL(9);
        case 512: return CALL(10);
        case 1024: return CALL(11);
        case 2048: return CALL(12);
        case 4096: return CALL(13);
        default: return hipErrorInvalidValue;
    }
#undef CALL
}

hipError_t spectrum_natural_bwd(const float* dshat, float* dk, float* dD, int64_t H, int64_t N, const Tables& tb,
                                hipStream_t st)
{
#define CALL(LG) natural_bwd_go<LG>((const float2*)dshat, dk, dD, H, tb, st)
    switch (N) {
        case 256: return CALL(9);
        case 512: return CALL(10);
        case 1024: return CALL(11);
        case 2048: return CALL(12);
        case 4096: return CALL(13);
        default: return hipErrorInvalidValue;
    }
#undef CALL
}

hipError_t valu_conv(const void* in, const float2* kspec, void* out, float2* ws, bool conj, const Problem& pr,
                     const Plan& pl, const Tables& tb, hipStream_t st)
{
    if (pl.vrow) {
#define CALL(LG) rows_conv_go<LG>((const float*)in, kspec, (float*)out, conj, pr, tb, st)
        LC_ROWS_SWITCH(pl.vrow, CALL)
#undef CALL
    }
    switch (pr.io) {
        case LONGCONV_F32: return conv_io<IoF32>(in, kspec, out, ws, conj, pr, pl, tb, st);
        case LONGCONV_F16: return conv_io<IoF16>(in, kspec, out, ws, conj, pr, pl, tb, st);
        default: return conv_io<IoBF16>(in, kspec, out, ws, conj, pr, pl, tb, st);
    }
}

// Workgroups that fill the device: one, two or about four of them per compute unit by their LDS
int valu_bwd_room(int64_t B, int64_t H, const Plan& pl)
{
    const int lg = pl.vrow ? pl.vrow : pl.log2L2, target = lg >= 14 ? 256 : lg == 13 ? 512 : 1024;
    const int64_t units = pl.vrow ? B : (B + 1) / 2;
    int64_t s = target / (H << pl.log2R);
    if (s > units) s = units;
    if (s > 64) s = 64;
    return s < 1 ? 1 : (int)s;
}
// Single rows of 2048 samples: fewer, where the rows that a share is spared do not make up for its company on a compute unit and for
// the sum of partial results.  A row takes 4.9, 5.8, 7.6 and 9.1 us with one to four workgroups on the fullest unit; the sum 2 us and
// its bytes.  Backward calls, as many as there is room for and by this: B=2, H=400 21.7 -> 17.8 us, B=2, H=300 18.4 -> 17.6, B=4,
// H=400 30.7 -> 29.5, B=8, H=129 25.7 -> 24.3.  At N = 4096 and above more shares were faster wherever there is room for them.
int valu_bwd_nsplit(int64_t B, int64_t H, const Plan& pl)
{
    const int room = valu_bwd_room(B, H, pl);
    if (pl.vrow != 11) return room;
    const float row_us[5] = {0.f, 4.9f, 5.8f, 7.6f, 9.1f};
    int best = 1;
    float least = 0.f;
    for (int s = 1; s <= room; ++s) {
        const int on_cu = (int)((H * s + compute_units() - 1) / compute_units());
        const float us = ((float)(on_cu / 4) * row_us[4] + row_us[on_cu % 4]) * (float)((B + s - 1) / s) +
                         (s > 1 ? 2.f + (float)s * (float)H * 2048.f * 2e-6f : 0.f);
        if (s == 1 || us < least) { best = s; least = us; }
    }
    return best;
}

size_t valu_zbuf_bytes(int64_t B, int64_t H, int nsplit, const Plan& pl)
{
    if (pl.vrow) return row_parks(pl.vrow) && B > nsplit ? ((size_t)H * nsplit << pl.vrow) * sizeof(float2) : 0;
    return valu_parks(pl.log2L2) ? ((size_t)H * nsplit << pl.log2L) * sizeof(float2) : 0;
}

hipError_t valu_bwd(const void* dy, const void* u, const float2* kspec, void* du, float2* ws_du, float* dk, float2* ws_A,
                    float* dD, void* zbuf, int nsplit, const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st)
{
    if (pl.vrow) {
#define CALL(LG) rows_bwd_go<LG>((const float*)dy, (const float*)u, kspec, (float*)du, dk, dD, zbuf, nsplit, pr, pl.dkscale, tb, st)
        LC_ROWS_SWITCH(pl.vrow, CALL)
#undef CALL
    }
    switch (pr.io) {
        case LONGCONV_F32: return bwd_io<IoF32>(dy, u, kspec, du, ws_du, dk, ws_A, dD, zbuf, nsplit, pr, pl, tb, st);
        case LONGCONV_F16: return bwd_io<IoF16>(dy, u, kspec, du, ws_du, dk, ws_A, dD, zbuf, nsplit, pr, pl, tb, st);
        default: return bwd_io<IoBF16>(dy, u, kspec, du, ws_du, dk, ws_A, dD, zbuf, nsplit, pr, pl, tb, st);
    }
}

}  // namespace lc
