// Learned Butterfly extension (Section 3.3): the FFT convolution of Eq. 2 in its Butterfly form (Section 3.2: small
// dense blocks interleaved with fixed twiddle diagonals, Appendix C.1), with the values of the blocks given per head
// instead of fixed to the DFT.  The stored spectrum (Algorithm 2 lines 1-2, the skip term as a constant added to it)
// stays what it is in the fixed path; only the transforms around it are learned:
//
//     y[b,h,t] = Re( T_B[h]( Shat[h] . T_A[h]( [u[b,h], 0_N] ) ) )[t],      0 <= t < N
//
//   L = 2N = 2^LG points, three stages.  Position p = (d_0, d_1, d_2), d_0 most significant; d_0 and d_1 have four bits
//   (block size 16 = the matrix unit's tile), d_2 the remaining LG - 8 bits (block size 2 .. 16, run as the block
//   diagonal 16 x 16 matrix I (x) A_2, which costs the matrix unit the same).
//   T_A: for s = 0, 1, 2 apply block A_s[h] along digit s, then (s < 2) the twiddle
//        w_s(p) = exp(-2 pi i k_s (p mod M_s) / (16 M_s)), M_s the stride of digit s.  With A_s = DFT this is the
//        decimation-in-frequency FFT and frequency k_0 + 16 k_1 + 256 k_2 sits at position (k_0, k_1, k_2).
//   T_B: the mirror image, s = 2, 1, 0: (s < 2) conj(w_s), then block B_s[h] along digit s; 1/L at the end.
//
// Every block product is one pair of v_mfma_f32_16x16x32_f16 per 16 columns (real form of the complex product, K =
// 16 slots x (re, im)), data as fp16 complex between stages, fp32 accumulation; every stage carries a fixed
// power of two (1/4 per 16-point block) so that DFT-like blocks keep the data at unit magnitude, undone in fp32 at
// the end.  Backward: the forward chain is run again next to the gradient's, and the gradient of a block is the 16 x 16
// complex matrix sum over columns of (gradient at the block's output) x conj(the block's input), two more MFMAs per 16
// columns with the columns as the K dimension, accumulated in fp32 registers over the rows a workgroup owns.
#include <type_traits>

#include "engines.hpp"
#include "planar.hpp"

namespace lc {
namespace {
using namespace planar;

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

constexpr int NBLK = 256;                       // entries of one 16 x 16 block
__host__ __device__ constexpr int stage_shift(int b) { return b == 4 ? 2 : (b >= 2 ? 1 : 0); }
__host__ __device__ constexpr int total_shift(int lg) { return 4 + stage_shift(lg - 8); }

__device__ __forceinline__ h2 pack(float re, float im)
{
    const f2 v = {re, im};
    return __builtin_convertvector(v, h2);
}

// ---- the register-chained form ------------------------------------------------------------------------------------------
// With T = L / 256 = the last radix, tile t = (all d_0, d_1 at d_2 = t) is one 16 x 16 matrix of points (planar.hpp) that
// two blocks contract one after the other: both 16-point blocks of a direction run in registers, and only d_2 crosses LDS.
//   * Twiddles: w_0 = w_256^(k_0 d_1) w_L^(k_0 t), w_1 = w_16T^(k_1 t).  Everything that depends on t is a row or column
//     scale of the tile's own matrices; what is left, w_256^(lane (4g + r)), is four numbers per lane, the same for all
//     tiles and both directions, multiplied in fp32.
//   * Exchange buffer: [d_2][plane][k_0][k_1], 8 words of padding per d_2; the hash of a row's quarters, of (d_2, k_0),
//     makes 16 rows of one d_2, and 16 slots of a middle tile, fill all banks.
template <int LG>
struct Geo {
    static constexpr int L = 1 << LG, N = L / 2, LB = LG - 8, T = 1 << LB;
    static constexpr int XS = 512 + 16;                       // numbers of a tile in the exchange buffer
    static constexpr int IS = 264, OS = 136;                  // and of a tile of rows coming in (16 x 16, 8 zero) and going out
    static constexpr float yscale() { return (float)(1 << 2 * total_shift(LG)) / (float)L; }
    // quarter q of row (d_2, k_0) of the exchange buffer
    static __device__ __forceinline__ int at(int d2, int k0, int q)
    {
        const int f = T == 16 ? d2 >> 2 : T == 8 ? (d2 >> 2) | ((d2 & 1) << 1) : T == 4 ? d2 : 2 * d2;
        return d2 * XS + k0 * 16 + 4 * ((q ^ (k0 >> 2) ^ f) & 3);
    }
    // the row that is slot s of middle tile m: d_2 = s mod T, k_0 = ...
    static __device__ __forceinline__ int slot_at(int m, int s, int q) { return at(s & (T - 1), m * (16 / T) + (s >> LB), q); }
};

constexpr int ROW = 17;        // stride of 16 complex numbers in LDS: lanes that read down a column meet 16 different banks
// entries of the matrices of a tile, from the head's blocks in LDS (forward, then inverse); w: w_0 of k_0 or w_1 of k_1 (LaneTw)
template <int LG>
struct Entries {
    using G = Geo<LG>;
    const float2 *A, *B;
    __device__ __forceinline__ float2 a0(int k0, int d0, float2 w) const { return scaled(cmul(A[k0 * ROW + d0], w), 0.25f); }
    __device__ __forceinline__ float2 a1(int k1, int d1, float2 w) const { return scaled(cmul(A[(16 + k1) * ROW + d1], w), 0.25f); }
    __device__ __forceinline__ float2 b1(int d1, int k1, float2 w) const { return scaled(cmulc(B[(16 + d1) * ROW + k1], w), 0.25f); }
    __device__ __forceinline__ float2 b0(int d0, int k0, float2 w) const { return scaled(cmulc(B[d0 * ROW + k0], w), 0.25f); }
    // the last block, block diagonal over the k_0's that share a middle tile
    __device__ __forceinline__ float2 last(const float2* M, int o, int i) const
    {
        const float2 v = M[(32 + (o & (G::T - 1))) * ROW + (i & (G::T - 1))];
        return (o >> G::LB) == (i >> G::LB) ? scaled(v, 1.0f / (float)(1 << stage_shift(G::LB))) : make_float2(0.f, 0.f);
    }
};
// The twiddles of one lane's operands, o = lane % 16 and i = 4g .. 4g+3 as result's and input's index, either way round: w_0 =
// w_L^(k_0 t) and w_1 = w_16T^(k_1 t) at o (w0c, w1c) and at i (w0q, w1q).  Asked for in front of the head's data, not one by one
// where they are used.
template <int LG>
struct LaneTw {
    using G = Geo<LG>;
    float2 w0c, w1c, w0q[4], w1q[4];
    __device__ __forceinline__ void load(const float2* __restrict__ stw, int t, int lane)
    {
        const int c = lane & 15, q = 4 * (lane >> 4);
        const float2 *p0 = stw + stw_offset(LG) + t, *p1 = stw + stw_offset(4 + G::LB) + t;
        w0c = p0[c << (LG - 4)];
        w1c = p1[c << G::LB];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            w0q[r] = p0[(q + r) << (LG - 4)];
            w1q[r] = p1[(q + r) << G::LB];
        }
    }
};
// w_256^(c d), d = 4g .. 4g+3
__device__ __forceinline__ void inner_twiddles(f4& wr, f4& wi, const float2* __restrict__ stw, int lane)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float2 v = stw[stw_offset(8) + 16 * (4 * (lane >> 4) + r) + (lane & 15)];
        wr[r] = v.x;
        wi[r] = v.y;
    }
}
// What a workgroup of T waves needs of its head travels in whole lines, through LDS: the six blocks (1536 numbers) and the
// spectrum in natural order (L numbers).  Gathered straight from memory, lane by lane, the
// constants of a workgroup cost more than eight rows of work.
template <int LG>
struct HeadData {
    using G = Geo<LG>;
    static constexpr int NT = 64 * G::T, HALF = 3 * NBLK / 2, NB = (2 * HALF + NT - 1) / NT;     // 16-byte pieces of the blocks
    static constexpr int BLK = 96 * ROW;                                // the spectrum's place behind the blocks
    static constexpr size_t bytes = sizeof(float2) * (BLK + G::L / 16 * ROW);
    f4 blk[NB], sp[2];
    __device__ __forceinline__ void load(const float2* Af, const float2* Ai, const float2* shat, int h, int tid)
    {
        const f4* a = reinterpret_cast<const f4*>(Af + (size_t)h * 3 * NBLK);
        const f4* b = reinterpret_cast<const f4*>(Ai + (size_t)h * 3 * NBLK) - HALF;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int e = min(tid + i * NT, 2 * HALF - 1);
            blk[i] = (e < HALF ? a : b)[e];
        }
        const f4* s = reinterpret_cast<const f4*>(shat + (size_t)h * G::L);
        sp[0] = s[tid];
        sp[1] = s[tid + NT];
    }
    static __device__ __forceinline__ void put2(float2* sm, int e, const f4& v)      // numbers 2e, 2e + 1
    {
        float2* p = sm + (e >> 3) * ROW + 2 * (e & 7);
        p[0] = make_float2(v[0], v[1]);
        p[1] = make_float2(v[2], v[3]);
    }
    __device__ __forceinline__ void put(float2* sm, int tid) const
    {
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (NB * NT == 2 * HALF || tid + i * NT < 2 * HALF) put2(sm, tid + i * NT, blk[i]);
        put2(sm + BLK, tid, sp[0]);
        put2(sm + BLK, tid + NT, sp[1]);
    }
};

// frequency in slot s of middle tile m at k_1 (row: stride of 16 numbers)
template <int LG>
__device__ __forceinline__ int freq_at(int m, int s, int k1, int row = 16)
{
    using G = Geo<LG>;
    return m * (16 / G::T) + (s >> G::LB) + row * (k1 + 16 * (s & (G::T - 1)));
}

template <class IO>
__device__ __forceinline__ uint32_t to_h2(uint32_t w)
{
    if constexpr (std::is_same<IO, IoBF16>::value) {
        const h2 h = pack(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
        return __builtin_bit_cast(uint32_t, h);
    }
    return w;
}
// Samples 2 tid, 2 tid + 1 of a row into the tiles [t][d_0][d_1] of the workgroup's T waves, and back
template <int LG>
__device__ __forceinline__ void row_in(_Float16* s, uint32_t w, int tid)
{
    using G = Geo<LG>;
    const h2 v = __builtin_bit_cast(h2, w);
    const int e = (2 * tid) >> G::LB;          // d_0, d_1; a row's quarters are XORed with d_0 / 4
    _Float16* p = s + ((2 * tid) & (G::T - 1)) * G::IS + (e ^ ((e >> 6) << 2));
    p[0] = v[0];
    p[G::IS] = v[1];
}
template <int LG>
__device__ __forceinline__ uint32_t row_out(const _Float16* s, int tid)
{
    using G = Geo<LG>;
    const int e = (2 * tid) >> G::LB;
    const uint16_t* p = reinterpret_cast<const uint16_t*>(s) + ((2 * tid) & (G::T - 1)) * G::OS + (e ^ ((e >> 6) << 2));
    return (uint32_t)p[0] | ((uint32_t)p[G::OS] << 16);
}
// four results of a row's tile (lane d_0 < 8, d_1 = 4g ..) as I/O numbers
template <class IO>
__device__ __forceinline__ void put_out(_Float16* tile, const f4& v, int lane)
{
    if ((lane & 15) >= 8) return;
    _Float16* p = tile + (lane & 15) * 16 + 4 * ((lane >> 4) ^ ((lane & 15) >> 2));
    if constexpr (std::is_same<IO, IoBF16>::value) {
        typedef __bf16 b4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<b4*>(p) = __builtin_convertvector(v, b4);
    } else {
        wr4(p, cvt4(v));
    }
}

// -------------------------------------------------------------------------------------------------------------------
// Forward.  One wave per tile: wave t owns tile t of the 16-point blocks and middle tile t.  The grid is what the device holds
// at once; a workgroup takes `per` consecutive rows of the (head, batch row) list, head by head, as a pipeline with two
// barriers per row:
//     [inverse blocks of row b-1, forward blocks of row b]  barrier  [last blocks and spectrum of row b, rows in and out]
// (a wave's tile of the exchange buffer is its own in the first part, so the two rows need one buffer).  Bound by issue: 11
// matrix and 83 vector instructions per 256 points and row, 112 with what a workgroup spends on its matrices (B=16, H=768,
// N=1024); two rows per barrier were no faster.  The form it replaced took every block through LDS with its own addresses,
// twiddle loads and barrier: that shape in bf16 77 us, this one 36 (53 before the quarters were hashed, 41 with a workgroup per 8
// rows of one head).  N = 256 spills 3 registers, N = 2048 5.
// -------------------------------------------------------------------------------------------------------------------
template <int LG, class IO>
__global__ void __launch_bounds__(64 << (LG - 8)) __attribute__((amdgpu_waves_per_eu(4)))
lb_fwd_kernel(const typename IO::T* __restrict__ u, const float2* __restrict__ shat, const float2* __restrict__ Af,
              const float2* __restrict__ Ai, typename IO::T* __restrict__ y, int B, int H, int64_t per,
              const float2* __restrict__ stw)
{
    using G = Geo<LG>;
    constexpr int T = G::T, N = G::N;
    constexpr size_t work = sizeof(_Float16) * T * (G::XS + G::IS + G::OS);
    __shared__ f4 smem[(work > HeadData<LG>::bytes ? work : HeadData<LG>::bytes) / 16];
    _Float16 *ex = reinterpret_cast<_Float16*>(smem), *in = ex + T * G::XS, *outb = in + T * G::IS;
    float2* sm2 = reinterpret_cast<float2*>(smem);
    const int tid = threadIdx.x, lane = tid & 63, t = tid >> 6, c = lane & 15, g = lane >> 4;
    _Float16* mine = ex + G::at(t, c, g);                                            // (k_0 = c, k_1 = 4g ..) of tile t
    const _Float16* tin = in + t * G::IS + 16 * (c >> 2) + 64 * g + 4 * ((c & 3) ^ g);   // transposed: lane d_1, d_0 = 4g ..
    const _Float16* mid_in = ex + G::slot_at(t, 4 * g + (c >> 2), c & 3);            // transposed: lane k_1, slots 4g ..
    _Float16* mid_out = ex + G::slot_at(t, c, g);                                    // lane slot, k_1 = 4g ..
    f4 cr, ci;
    inner_twiddles(cr, ci, stw, lane);

    int64_t item = (int64_t)blockIdx.x * per;
    const int64_t end = item + per < (int64_t)B * H ? item + per : (int64_t)B * H;
    while (item < end) {
        const int h = (int)(item / B), b0 = (int)(item - (int64_t)h * B);
        const int n = (int)(end - item < B - b0 ? end - item : B - b0);              // rows b0 .. b0 + n of this head
        item += n;
        HeadData<LG> hd;
        hd.load(Af, Ai, shat, h, tid);
        const uint32_t* up = reinterpret_cast<const uint32_t*>(u + row_off(b0, h, H, N)) + tid;
        uint32_t* yp = reinterpret_cast<uint32_t*>(y + row_off(b0, h, H, N)) + tid;
        const size_t step = (size_t)H * (N / 2);
        uint32_t w = *up, wn = n > 1 ? up[step] : 0u;
        up += 2 * step;
        LaneTw<LG> W;
        W.load(stw, t, lane);
        hd.put(sm2, tid);
        __syncthreads();
        const Entries<LG> E{sm2, sm2 + 48 * ROW};
        const Rl A0 = make_rl([&](int o, int i) { return E.a0(o, i, W.w0c); }, lane);
        const Cx A1 = make_cx([&](int o, int i) { return E.a1(o, i, W.w1c); }, lane);
        const Cx A2 = make_cx([&](int o, int i) { return E.last(E.A, o, i); }, lane);
        const Cx B2 = make_cx([&](int o, int i) { return E.last(E.B, o, i); }, lane);
        const Cx B1 = make_cx([&](int o, int i) { return E.b1(o, i, W.w1q[i & 3]); }, lane);
        const h8 B0 = make_cx([&](int o, int i) { return scaled(E.b0(o, i, W.w0q[i & 3]), G::yscale()); }, lane).re;
        f4 sr, si;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float2 s = sm2[HeadData<LG>::BLK + freq_at<LG>(t, 4 * g + r, c, ROW)];
            sr[r] = s.x;
            si[r] = s.y;
        }
        __syncthreads();
        for (int i = tid; i < T * G::IS / 2; i += 64 * T) reinterpret_cast<uint32_t*>(in)[i] = 0;
        __syncthreads();
        row_in<LG>(in, to_h2<IO>(w), tid);
        __syncthreads();

        const auto forward = [&]() {
            const h4 x = tr_read(tin);
            f4 yr = mm(x, A0.re), yi = mm(x, A0.im);                    // lane k_0, d_1 = 4g ..
            cmul4<false>(yr, yi, cr, ci);
            const H8P x1 = planes(yr, yi);
            const H8P x2 = planes(mm(A1.re, x1.v), mm(A1.im, x1.v));    // lane k_0, k_1 = 4g ..
            wr4(mine, x2.p[0]);
            wr4(mine + 256, x2.p[1]);
        };
        const auto middle = [&]() {
            H8P x;
            x.p[0] = tr_read(mid_in);
            x.p[1] = tr_read(mid_in + 256);
            f4 zr = mm(A2.re, x.v), zi = mm(A2.im, x.v);                // lane k_1, slots 4g ..
            cmul4<false>(zr, zi, sr, si);
            const H8P m = planes(zr, zi);
            const H8P v = planes(mm(m.v, B2.re), mm(m.v, B2.im));       // lane slot, k_1 = 4g ..
            wr4(mid_out, v.p[0]);
            wr4(mid_out + 256, v.p[1]);
        };
        const auto inverse = [&]() {
            H8P x;
            x.p[0] = rd4(mine);
            x.p[1] = rd4(mine + 256);
            f4 yr = mm(x.v, B1.re), yi = mm(x.v, B1.im);                // lane d_1, k_0 = 4g ..
            cmul4<true>(yr, yi, cr, ci);
            put_out<IO>(outb + t * G::OS, mm(planes(yr, yi).v, B0), lane);
        };
        const auto next_row_in = [&](int b) {                           // row b + 1; row b + 2 asked for
            row_in<LG>(in, to_h2<IO>(wn), tid);
            if (b + 2 < n) {
                wn = *up;
                up += step;
            }
        };
        forward();
        __syncthreads();
        middle();
        next_row_in(0);
        __syncthreads();
        for (int b = 1; b < n; ++b) {
            inverse();
            forward();
            __syncthreads();
            put_once(yp, row_out<LG>(outb, tid));
            yp += step;
            middle();
            next_row_in(b);
            __syncthreads();
        }
        inverse();
        __syncthreads();
        put_once(yp, row_out<LG>(outb, tid));
        __syncthreads();                                                // (the next head's constants go where the rows were)
    }
}

// -------------------------------------------------------------------------------------------------------------------
// Backward, register-chained.  grid = (nsplit, H): workgroup (sp, h) owns rows b = sp, sp + nsplit, ... of head h.  dy goes through
// the adjoint of the inverse blocks exactly as u goes through the forward blocks, so there are two chains of waves side by side, u's
// and dy's, with a wave per tile each and the forward kernel's two barriers per row:
//     [row b-1: the input of B_0 from that of B_1 | gradients through A_1, A_0; du.  row b: u through A_0, A_1 | dy through
//      B_0^H, B_1^H]  barrier  [row b: last blocks, spectrum, and their adjoints]
// The gradient of a block is the 16 x 16 sum over columns of (gradient at its output) x conj(its input): two more matrix
// products per tile with the columns as K, on operands whose lanes are the slots.  u's waves keep the sums of the B's and of the
// spectrum, dy's those of the A's; the operand that the other chain makes is read from LDS.  Both index orders of a tile are needed:
// what passes the exchange buffers is read from there either way, the rest takes a wave's own 1 KB of LDS.  u's waves take
// the gradient at the product with the spectrum a second time, rather than wait for dy's.
// The twiddle factors that were folded into a tile's matrices scale rows or columns of its 16 x 16 sums: applied once, at
// the end, where the waves' sums meet in wave order.
// Per 256 points and row 35 matrix and 195 vector instructions, and 9 KB written to LDS and 27 read.  One wave for both chains had 33 and
// 187, but needed 240 registers, and its two waves per SIMD left the chip waiting for LDS and for results; now four fit, without spills
// in the row loop, since the last stage's matrices (the same for all tiles) are read from LDS.  Vector instructions are issued in 66 %
// of the cycles (57 before), LDS is active in 44 (31).  N = 1024: a row takes 3280 cycles of a compute unit, a head's constants and
// matrices 8900, its sums 4300.  bf16, B=16, H=768: N = 256 33.0 -> 29.4 us, 512 55.6 -> 47.7, 1024 99.2 -> 91.6.  Workgroups that stay
// for the next head, with its constants asked for in front of the sums, spilled 66 registers: 96.
// -------------------------------------------------------------------------------------------------------------------
struct LbGrads {            // where the sums go: of share sp and head h at index sp * H + h
    float2 *shat, *qf, *qi;
    int q_stride;
};

// numbers in LDS: what the first parts leave for the middle one, what the middle one leaves for the last, a row of both tensors on
// its way in, du on its way out; then a first part's x_1 or g_1 for the other chain's last part, by the row's parity, a wave's own
// 1 KB and the last stage's matrices, or in the end the sums
template <int LG>
constexpr int lbb_kept() { return Geo<LG>::T * (4 * Geo<LG>::XS + 2 * Geo<LG>::IS + Geo<LG>::OS); }
template <int LG>
constexpr size_t lbb_lds()
{
    const size_t work = sizeof(_Float16) * (Geo<LG>::T * 6 * 512 + 4 * 1024), red = sizeof(float2) * 6 * NBLK * Geo<LG>::T;
    const size_t a = sizeof(_Float16) * lbb_kept<LG>() + (work > red ? work : red);
    return a > HeadData<LG>::bytes ? a : HeadData<LG>::bytes;
}

__device__ __forceinline__ void outer(const H8P& G, const H8P& X, f4& qr, f4& qi)
{
    H8P s;
    s.u[0] = make_uint2(X.u[1].x ^ 0x80008000u, X.u[1].y ^ 0x80008000u);
    s.u[1] = X.u[0];
    qr = __builtin_amdgcn_mfma_f32_16x16x32_f16(G.v, X.v, qr, 0, 0, 0);      // Gr Xr + Gi Xi
    qi = __builtin_amdgcn_mfma_f32_16x16x32_f16(G.v, s.v, qi, 0, 0, 0);      // Gi Xr - Gr Xi
}

template <int LG, class IO, int chain>
__device__ __forceinline__ void
lb_bwd_chain(f4* lds4, const int t, const typename IO::T* __restrict__ dy, const typename IO::T* __restrict__ u,
              const float2* __restrict__ shat, const float2* __restrict__ Af, const float2* __restrict__ Ai,
              typename IO::T* __restrict__ du, LbGrads out, int B, int H, const float2* __restrict__ stw)
{
    using G = Geo<LG>;
    constexpr int T = G::T, N = G::N, LB = G::LB;
    const int sp = blockIdx.x, nsplit = gridDim.x, h = blockIdx.y;
    const int wave = chain * T + t, lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4, tid = 64 * t + lane;
    _Float16 *exs = reinterpret_cast<_Float16*>(lds4), *exo = exs + 2 * T * G::XS, *ins = exo + 2 * T * G::XS;
    _Float16 *outb = ins + 2 * T * G::IS, *kept = exs + lbb_kept<LG>(), *priv = kept + 4 * T * 512;
    h8* mats = reinterpret_cast<h8*>(priv + 2 * T * 512) + lane;          // [A_2, B_2, B_2^H, A_2^H][re, im][lane]
    float2* sm2 = reinterpret_cast<float2*>(lds4);
    const size_t step = (size_t)nsplit * H * (N / 2);
    const uint32_t* xp = reinterpret_cast<const uint32_t*>((chain ? dy : u) + row_off(sp, h, H, N)) + tid;
    uint32_t* dp = reinterpret_cast<uint32_t*>(du ? du + row_off(sp, h, H, N) : nullptr) + tid;
    const int n = (B - sp + nsplit - 1) / nsplit;                       // rows of this workgroup
    HeadData<LG> hd;
    if (chain == 0) hd.load(Af, Ai, shat, h, tid);
    uint32_t wx = *xp, nx = n > 1 ? xp[step] : 0u;
    xp += 2 * step;
    f4 cr, ci;
    inner_twiddles(cr, ci, stw, lane);
    LaneTw<LG> W;
    W.load(stw, t, lane);
    if (chain == 0) hd.put(sm2, tid);
    __syncthreads();
    // The chain's matrices of the first part and the last: u's A_0, A_1, B_1; dy's the adjoints of B_0, B_1, A_1, A_0
    const Entries<LG> E{sm2, sm2 + 48 * ROW};
    Rl M0;
    Cx M1, M4;
    h8 M5;
    if (chain == 0) {
        M0 = make_rl([&](int o, int i) { return E.a0(o, i, W.w0c); }, lane);
        M1 = make_cx([&](int o, int i) { return E.a1(o, i, W.w1c); }, lane);
        M4 = make_cx([&](int o, int i) { return E.b1(o, i, W.w1q[i & 3]); }, lane);
        M5 = M1.re;                                                     // (not used)
    } else {
        M0 = make_rl([&](int o, int i) { return conj2(E.b0(i, o, W.w0c)); }, lane);
        M1 = make_cx([&](int o, int i) { return conj2(E.b1(i, o, W.w1c)); }, lane);
        M4 = make_cx([&](int o, int i) { return conj2(E.a1(i, o, W.w1q[i & 3])); }, lane);
        M5 = make_cx([&](int o, int i) { return scaled(conj2(E.a0(i, o, W.w0q[i & 3])), G::yscale()); }, lane).re;
    }
    // the last stage's do not depend on t: in LDS, A_2, B_2, and their adjoints in the other order
    Cx L0, L1;
    if (t == 0) {
        if (chain == 0) {
            L0 = make_cx([&](int o, int i) { return E.last(E.A, o, i); }, lane);
            L1 = make_cx([&](int o, int i) { return E.last(E.B, o, i); }, lane);
        } else {
            L0 = make_cx([&](int o, int i) { return conj2(E.last(E.B, i, o)); }, lane);
            L1 = make_cx([&](int o, int i) { return conj2(E.last(E.A, i, o)); }, lane);
        }
    }
    f4 sr, si;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float2 s = sm2[HeadData<LG>::BLK + freq_at<LG>(t, 4 * g + r, c, ROW)];
        sr[r] = s.x;
        si[r] = chain ? -s.y : s.y;                                     // (dy's chain multiplies by the conjugate)
    }
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 q0r = zero, q0i = zero, q1r = zero, q1i = zero, q2r = zero, q2i = zero;      // sums: u's waves B_0, B_1, B_2; dy's A_0, A_1, A_2
    f4 dsr = zero, dsi = zero;                                                      // the spectrum's (u's waves)

    const int own = G::at(t, c, g), own_tr = G::at(t, 4 * g + (c >> 2), c & 3);      // tile t: row c, or transposed
    const int mid = G::slot_at(t, c, g), mid_tr = G::slot_at(t, 4 * g + (c >> 2), c & 3);
    const int trow = 16 * (4 * g + (c >> 2)) + 4 * ((c & 3) ^ g), row = 16 * c + 4 * (g ^ (c >> 2));   // a plain 16 x 16 tile
    _Float16 *ex = exs + chain * T * G::XS, *eo = exo + chain * T * G::XS;
    const _Float16* ey = exs + (1 - chain) * T * G::XS + mid;                        // the other chain's, as slots
    const _Float16 *tin = ins + (chain * T + t) * G::IS + trow, *tother = ins + ((1 - chain) * T + t) * G::IS + row;
    _Float16* pv = priv + wave * 512;
    _Float16* kmine = kept + wave * 512 + row;                                       // + parity * 2 T * 512
    const _Float16* kother = kept + ((1 - chain) * T + t) * 512 + trow;
    const auto transposed = [&](const H8P& x) {
        H8P y;
        wr4(pv + row, x.p[0]);
        wr4(pv + row + 256, x.p[1]);
        y.p[0] = tr_read(pv + trow);
        y.p[1] = tr_read(pv + trow + 256);
        return y;
    };
    __syncthreads();
    // both rows' tiles: the padding, d_0 >= 8, stays zero; a row's samples are the other half
    if (t == 0) {
        mats[chain * 256] = L0.re;
        mats[chain * 256 + 64] = L0.im;
        mats[chain * 256 + 128] = L1.re;
        mats[chain * 256 + 192] = L1.im;
    }
    for (int i = threadIdx.x; i < T * 128; i += 128 * T) reinterpret_cast<uint32_t*>(ins + (i >> 6) * G::IS + 128)[i & 63] = 0;
    row_in<LG>(ins + chain * T * G::IS, to_h2<IO>(wx), tid);
    __syncthreads();

    h4 other;               // the other tensor's samples, kept from a row's first part to its last
    const auto first = [&](int b) __attribute__((always_inline)) {
        const h4 x = tr_read(tin);
        other = rd4(tother);                                            // lane d_0, d_1 = 4g ..
        f4 yr = mm(x, M0.re), yi = mm(x, M0.im);                        // lane k_0, d_1 = 4g ..
        cmul4<false>(yr, yi, cr, ci);
        const H8P x1 = planes(yr, yi);
        _Float16* k = kmine + (b & 1) * 2 * T * 512;                    // (read transposed by the other chain's wave t)
        wr4(k, x1.p[0]);
        wr4(k + 256, x1.p[1]);
        const H8P x2 = planes(mm(M1.re, x1.v), mm(M1.im, x1.v));        // lane k_0, k_1 = 4g ..
        wr4(ex + own, x2.p[0]);
        wr4(ex + own + 256, x2.p[1]);
    };
    const auto middle = [&]() __attribute__((always_inline)) {
        H8P x, yt;
        x.p[0] = tr_read(ex + mid_tr);                                  // lane k_1, slots 4g ..
        x.p[1] = tr_read(ex + mid_tr + 256);
        yt.p[0] = rd4(ey);                                              // the other chain's: lane slot, k_1 = 4g ..
        yt.p[1] = rd4(ey + 256);
        const h8* m = mats + chain * 256;
        f4 zr = mm(m[0], x.v), zi = mm(m[64], x.v);                    // lane k_1, slots 4g ..
        if (chain == 0) {
            H8P y;
            const _Float16* e = exs + T * G::XS + mid_tr;
            y.p[0] = tr_read(e);
            y.p[1] = tr_read(e + 256);
            const f4 hr = mm(mats[256], y.v), hi = mm(mats[320], y.v);          // gradient at the product with the spectrum
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                dsr[r] += hr[r] * zr[r] + hi[r] * zi[r];
                dsi[r] += hi[r] * zr[r] - hr[r] * zi[r];
            }
        }
        cmul4<false>(zr, zi, sr, si);
        const H8P w = planes(zr, zi);
        const H8P wt = transposed(w);
        const H8P v = planes(mm(w.v, m[128]), mm(w.v, m[192]));           // lane slot, k_1 = 4g ..
        wr4(eo + mid, v.p[0]);
        wr4(eo + mid + 256, v.p[1]);
        if (chain == 0) outer(yt, wt, q2r, q2i);
        else outer(wt, yt, q2r, q2i);
    };
    const auto last = [&](int b) __attribute__((always_inline)) {
        H8P v, vt, kt;
        v.p[0] = rd4(eo + own);                                         // lane k_0, k_1 = 4g ..
        v.p[1] = rd4(eo + own + 256);
        vt.p[0] = tr_read(eo + own_tr);                                 // lane k_1, k_0 = 4g ..
        vt.p[1] = tr_read(eo + own_tr + 256);
        const _Float16* k = kother + (b & 1) * 2 * T * 512;
        kt.p[0] = tr_read(k);                                           // lane d_1, k_0 = 4g ..
        kt.p[1] = tr_read(k + 256);
        if (chain == 0) {
            f4 yr = mm(M4.re, v.v), yi = mm(M4.im, v.v);                // lane k_0, d_1 = 4g ..
            cmul4<true>(yr, yi, cr, ci);
            const H8P w0 = planes(yr, yi);
            outer(kt, vt, q1r, q1i);
            q0r = __builtin_amdgcn_mfma_f32_16x16x16f16(other, w0.p[0], q0r, 0, 0, 0);
            q0i = __builtin_amdgcn_mfma_f32_16x16x16f16(other, w0.p[1], q0i, 0, 0, 0);     // (minus the imaginary part)
        } else {
            f4 yr = mm(v.v, M4.re), yi = mm(v.v, M4.im);                // lane d_1, k_0 = 4g ..
            cmul4<true>(yr, yi, cr, ci);
            const H8P g6 = planes(yr, yi);
            outer(vt, kt, q1r, q1i);
            const H8P g6t = transposed(g6);                             // lane k_0, d_1 = 4g ..
            q0r = __builtin_amdgcn_mfma_f32_16x16x16f16(g6t.p[0], other, q0r, 0, 0, 0);
            q0i = __builtin_amdgcn_mfma_f32_16x16x16f16(g6t.p[1], other, q0i, 0, 0, 0);
            put_out<IO>(outb + t * G::OS, mm(g6.v, M5), lane);
        }
    };
    const auto rows_in = [&](int b) {                                   // row b + 1; row b + 2 asked for
        row_in<LG>(ins + chain * T * G::IS, to_h2<IO>(nx), tid);
        if (b + 2 < n) {
            nx = *xp;
            xp += step;
        }
    };
    first(0);
    __syncthreads();
    middle();
    rows_in(0);
    __syncthreads();
    for (int b = 1; b < n; ++b) {
        last(b - 1);
        first(b);
        __syncthreads();
        if (du && chain == 0) {
            put_once(dp, row_out<LG>(outb, tid));
            dp += step;
        }
        middle();
        rows_in(b);
        __syncthreads();
    }
    W.load(stw, t, lane);                    // (for the sums below; no registers for them in the loop)
    last(n - 1);
    __syncthreads();
    if (du && chain == 0) put_once(dp, row_out<LG>(outb, tid));

    const size_t at = (size_t)sp * H + h;
    if (out.shat && chain == 0) {
        float2* ps = out.shat + at * G::L;
#pragma unroll
        for (int r = 0; r < 4; ++r) ps[freq_at<LG>(t, 4 * g + r, c)] = make_float2(dsr[r] * G::yscale(), dsi[r] * G::yscale());
    }
    // the waves' sums, [block][chain][wave][entry], behind du's last row; then entry by entry in wave order
    float2* sums = reinterpret_cast<float2*>(kept);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float2* p = sums + ((1 - chain) * T + t) * NBLK + (4 * g + r) * 16 + c;
        p[0] = chain ? cmulc(make_float2(q0r[r], q0i[r]), W.w0q[r]) : cmul(make_float2(q0r[r], -q0i[r]), W.w0c);
        p[2 * T * NBLK] = chain ? cmulc(make_float2(q1r[r], q1i[r]), W.w1q[r]) : cmul(make_float2(q1r[r], q1i[r]), W.w1c);
        p[4 * T * NBLK] = make_float2(q2r[r], q2i[r]);
    }
    __syncthreads();
    for (int e3 = threadIdx.x; e3 < 6 * NBLK; e3 += 128 * T) {
        const int which = (e3 / NBLK) & 1, s = e3 / (2 * NBLK), e = e3 % NBLK, i = e / 16, j = e % 16;
        float2* q = which ? out.qi : out.qf;
        if (!q) continue;
        float2 a = make_float2(0.f, 0.f);
        const float2* p = sums + (e3 / NBLK) * T * NBLK;
        if (s < 2) {
            for (int w = 0; w < T; ++w) a = cadd(a, p[w * NBLK + e]);
        } else if (i < T && j < T) {             // the diagonal blocks of I (x) A_2 all carry the same parameters
            for (int w = 0; w < T; ++w)
                for (int d = 0; d < 16; d += T) a = cadd(a, p[w * NBLK + (d + i) * 16 + d + j]);
        }
        const float sc = G::yscale() / (float)(1 << stage_shift(s == 2 ? LB : 4));
        q[at * out.q_stride + s * NBLK + e] = make_float2(a.x * sc, a.y * sc);
    }
}

// Waves 0 .. T - 1 do u's chain, the others dy's.  Both meet the same barriers from code of their own: in lb_bwd_chain none stands in a
// condition on the chain, and none may.
template <int LG, class IO>
__global__ void __launch_bounds__(128 << (LG - 8)) __attribute__((amdgpu_waves_per_eu(4)))
lb_bwd_kernel(const typename IO::T* __restrict__ dy, const typename IO::T* __restrict__ u,
              const float2* __restrict__ shat, const float2* __restrict__ Af, const float2* __restrict__ Ai,
              typename IO::T* __restrict__ du, LbGrads out, int B, int H, const float2* __restrict__ stw)
{
    extern __shared__ f4 lds4[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave < Geo<LG>::T) lb_bwd_chain<LG, IO, 0>(lds4, wave, dy, u, shat, Af, Ai, du, out, B, H, stw);
    else lb_bwd_chain<LG, IO, 1>(lds4, wave - Geo<LG>::T, dy, u, shat, Af, Ai, du, out, B, H, stw);
}

// Sums the partial results over the shares (fixed order): grid (pieces of a head's results, H)
__global__ void __launch_bounds__(256)
lb_reduce_kernel(const float2* __restrict__ part_shat, const float2* __restrict__ part_q, float2* __restrict__ dshat,
                 float2* __restrict__ dAf, float2* __restrict__ dAi, int64_t H, int L, int nsplit)
{
    const int e = blockIdx.x * 256 + threadIdx.x, h = blockIdx.y;
    const float2* p;
    size_t stride;
    float2* out;
    if (e < L) {
        p = part_shat + (size_t)h * L + e;
        stride = (size_t)H * L;
        out = dshat ? dshat + (size_t)h * L + e : nullptr;
    } else {
        const int q = e - L;
        if (q >= 6 * NBLK) return;
        p = part_q + (size_t)h * 6 * NBLK + q;
        stride = (size_t)H * 6 * NBLK;
        float2* d = q < 3 * NBLK ? dAf : dAi;
        out = d ? d + (size_t)h * 3 * NBLK + q % (3 * NBLK) : nullptr;
    }
    if (!out) return;
    float2 a = make_float2(0.f, 0.f);
    for (int sp = 0; sp < nsplit; ++sp) a = cadd(a, p[sp * stride]);
    *out = a;
}

// -------------------------------------------------------------------------------------------------------------------
// Backward of N = 2048: the same pipeline with sixteen tiles, two per wave (t = 2 wave and 2 wave + 1: one set of addresses).  Two tiles' matrices and sums
// would be 220 registers, so
//   * the twiddle that tile t adds to w_256^(k_0 d_1) is multiplied with it in fp32, w_L^(k_0 (16 d_1 + t)): the outer blocks and
//     their sums are then the same for all tiles (the gradient of A_1's input comes out with k_0 on the lanes, like all the others);
//   * the blocks in the middle, A_1 and B_1 of every tile and A_2 and B_2, wait in LDS as planes (34 KB), read as they are or
//     transposed for their adjoints.
// grid = (nsplit, H), as above.  Bound by issue at two waves per SIMD; 29 registers spilled, two reloaded in the row loop.  A row takes
// 3.2 us, a workgroup's matrices and sums 15.  B=64, H=256 bf16: 842 -> 218 us against the form it replaced (every block a trip
// through LDS with its own barrier, seven buffers); steps B=16, H=100 fp16 155.5 -> 71.4, B=2, H=300 116 -> 63, B=64, H=1024 3777 ->
// 1256.  Errors of du, dshat and both blocks' gradients against 64 bits are 0 to 2 % lower.
// -------------------------------------------------------------------------------------------------------------------
struct Lb2 {
    using G = Geo<12>;
    static constexpr int NW = 8, NT = 64 * NW, T = G::T;
    static constexpr int WORK = T * (2 * G::XS + 2 * G::IS + G::OS) + NW * 512;       // 16-bit numbers
    static constexpr int MATS = 512 * (2 * T + 2);
    static constexpr size_t lds = sizeof(_Float16) * (WORK + MATS);
    static_assert(HeadData<12>::bytes <= sizeof(_Float16) * WORK, "the head's data passes through where the rows are");
    static_assert(sizeof(float2) * 4 * NBLK * NW <= lds, "and the sums leave");
};

template <class IO>
__global__ void __launch_bounds__(Lb2::NT) __attribute__((amdgpu_waves_per_eu(2)))
lb_bwd2_kernel(const typename IO::T* __restrict__ dy, const typename IO::T* __restrict__ u, const float2* __restrict__ shat,
               const float2* __restrict__ Af, const float2* __restrict__ Ai, typename IO::T* __restrict__ du, LbGrads out, int B, int H,
               const float2* __restrict__ stw)
{
    constexpr int LG = 12, NW = Lb2::NW, NT = Lb2::NT;
    using G = Geo<LG>;
    constexpr int T = G::T, N = G::N;
    extern __shared__ f4 lb2_mem[];
    _Float16 *exu = reinterpret_cast<_Float16*>(lb2_mem), *exg = exu + T * G::XS, *inu = exg + T * G::XS;
    _Float16 *ing = inu + T * G::IS, *outb = ing + T * G::IS, *priv = outb + T * G::OS, *mats = priv + NW * 512;
    float2* sm2 = reinterpret_cast<float2*>(lb2_mem);
    const int sp = blockIdx.x, nsplit = gridDim.x, h = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4;
    const size_t step = (size_t)nsplit * H * (N / 2);
    const uint32_t* up = reinterpret_cast<const uint32_t*>(u + row_off(sp, h, H, N)) + tid;
    const uint32_t* gp = reinterpret_cast<const uint32_t*>(dy + row_off(sp, h, H, N)) + tid;
    uint32_t* dp = reinterpret_cast<uint32_t*>(du ? du + row_off(sp, h, H, N) : nullptr) + tid;
    const int n = (B - sp + nsplit - 1) / nsplit;                       // rows of this workgroup
    uint32_t nu[2], ng[2];                                              // words tid and tid + NT of the next row
    const auto ask = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            nu[j] = up[j * NT];
            ng[j] = gp[j * NT];
        }
        up += step;
        gp += step;
    };
    const auto rows_put = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            row_in<LG>(inu, to_h2<IO>(nu[j]), tid + j * NT);
            row_in<LG>(ing, to_h2<IO>(ng[j]), tid + j * NT);
        }
    };
    {
        HeadData<LG> hd[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) hd[j].load(Af, Ai, shat, h, tid + j * NT);
        ask();
#pragma unroll
        for (int j = 0; j < 2; ++j) hd[j].put(sm2, tid + j * NT);
    }
    const int trow = 16 * (4 * g + (c >> 2)) + 4 * ((c & 3) ^ g), row = 16 * c + 4 * (g ^ (c >> 2));   // a plain 16 x 16 tile
    // complex matrices as planes of such tiles: A_1, B_1 of tile t at 2t, 2t + 1; A_2, B_2 behind them
    const auto mat_put = [&](int m, const Cx& x) {
        H8P v;
        v.v = x.re;
        wr4(mats + m * 512 + row, v.p[0]);
        v.v = x.im;
        wr4(mats + m * 512 + 256 + row, v.p[0]);
    };
    const auto mat = [&](int m) {                                       // (planes P, Q: P - Q and Q + P as K runs)
        H8P re, im;
        re.p[0] = im.p[1] = rd4(mats + m * 512 + row);
        im.p[0] = rd4(mats + m * 512 + 256 + row);
        re.u[1] = make_uint2(im.u[0].x ^ 0x80008000u, im.u[0].y ^ 0x80008000u);
        return Cx{re.v, im.v};
    };
    const auto mat_adj = [&](int m) {
        H8P re, im;
        re.p[0] = im.p[1] = tr_read(mats + m * 512 + trow);
        re.p[1] = tr_read(mats + m * 512 + 256 + trow);
        im.u[0] = make_uint2(re.u[1].x ^ 0x80008000u, re.u[1].y ^ 0x80008000u);
        return Cx{re.v, im.v};
    };
    f4 cr[2], ci[2];                                                    // w_L^(k_0 (16 d_1 + t)), lane k_0, d_1 = 4g ..
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float2 v = stw[stw_offset(LG) + (c << (LG - 4)) + T * (4 * g + r) + 2 * wave + j];
            cr[j][r] = v.x;
            ci[j][r] = v.y;
        }
    __syncthreads();
    const Entries<LG> E{sm2, sm2 + 48 * ROW};
    const float2 one = make_float2(1.f, 0.f);
    const Rl A0 = make_rl([&](int o, int i) { return E.a0(o, i, one); }, lane);
    const Rl B0H = make_rl([&](int o, int i) { return conj2(E.b0(i, o, one)); }, lane);
    const h8 A0H = make_cx([&](int o, int i) { return scaled(conj2(E.a0(i, o, one)), G::yscale()); }, lane).re;
    f4 sr[2], si[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int t = 2 * wave + j;
        LaneTw<LG> W;
        W.load(stw, t, lane);
        mat_put(2 * t, make_cx([&](int o, int i) { return E.a1(o, i, W.w1c); }, lane));
        mat_put(2 * t + 1, make_cx([&](int o, int i) { return E.b1(o, i, W.w1q[i & 3]); }, lane));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float2 s = sm2[HeadData<LG>::BLK + freq_at<LG>(t, 4 * g + r, c, ROW)];
            sr[j][r] = s.x;
            si[j][r] = s.y;
        }
    }
    if (wave < 2) mat_put(2 * T + wave, make_cx([&](int o, int i) { return E.last(wave ? E.B : E.A, o, i); }, lane));
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 a0r = zero, a0i = zero, a2r = zero, a2i = zero, b0r = zero, b0i = zero, b2r = zero, b2i = zero;      // sums of the blocks'
    f4 a1r[2] = {zero, zero}, a1i[2] = {zero, zero}, b1r[2] = {zero, zero}, b1i[2] = {zero, zero};           // gradients
    f4 dsr[2] = {zero, zero}, dsi[2] = {zero, zero};
    _Float16* pv = priv + wave * 512;
    const auto transposed = [&](const H8P& x) {
        H8P y;
        wr4(pv + row, x.p[0]);
        wr4(pv + row + 256, x.p[1]);
        y.p[0] = tr_read(pv + trow);
        y.p[1] = tr_read(pv + trow + 256);
        return y;
    };
    __syncthreads();
    // both rows' tiles: the padding, d_0 >= 8, stays zero; a row's samples are the other half
    for (int i = tid; i < T * 128; i += NT) reinterpret_cast<uint32_t*>(inu + (i >> 6) * G::IS + 128)[i & 63] = 0;
    rows_put();
    if (n > 1) ask();
    __syncthreads();

    H8P x1t[2], g1t[2];     // kept from a row's first part to its last
    h4 uo[2], go[2];
    const auto first = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = 2 * wave + j, own = G::at(t, c, g);          // tile t: row c
            {
                const h4 x = tr_read(inu + t * G::IS + trow);
                uo[j] = rd4(inu + t * G::IS + row);                     // lane d_0, d_1 = 4g ..
                f4 yr = mm(x, A0.re), yi = mm(x, A0.im);                // lane k_0, d_1 = 4g ..
                cmul4<false>(yr, yi, cr[j], ci[j]);
                const H8P x1 = planes(yr, yi);
                x1t[j] = transposed(x1);                                // lane d_1, k_0 = 4g ..
                const Cx A1 = mat(2 * t);
                const H8P x2 = planes(mm(A1.re, x1.v), mm(A1.im, x1.v));            // lane k_0, k_1 = 4g ..
                wr4(exu + own, x2.p[0]);
                wr4(exu + own + 256, x2.p[1]);
            }
            {
                const h4 x = tr_read(ing + t * G::IS + trow);
                go[j] = rd4(ing + t * G::IS + row);
                f4 yr = mm(x, B0H.re), yi = mm(x, B0H.im);
                cmul4<false>(yr, yi, cr[j], ci[j]);
                const H8P g1 = planes(yr, yi);
                g1t[j] = transposed(g1);
                const Cx B1H = mat_adj(2 * t + 1);
                const H8P g2 = planes(mm(B1H.re, g1.v), mm(B1H.im, g1.v));
                wr4(exg + own, g2.p[0]);
                wr4(exg + own + 256, g2.p[1]);
            }
        }
    };
    const auto middle = [&]() {
        const Cx A2 = mat(2 * T), B2 = mat(2 * T + 1), A2H = mat_adj(2 * T), B2H = mat_adj(2 * T + 1);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = 2 * wave + j, mid = G::slot_at(t, c, g), mid_tr = G::slot_at(t, 4 * g + (c >> 2), c & 3);
            H8P x, xt, y, yt;
            x.p[0] = tr_read(exu + mid_tr);                             // lane k_1, slots 4g ..
            x.p[1] = tr_read(exu + mid_tr + 256);
            xt.p[0] = rd4(exu + mid);                                   // lane slot, k_1 = 4g ..
            xt.p[1] = rd4(exu + mid + 256);
            y.p[0] = tr_read(exg + mid_tr);
            y.p[1] = tr_read(exg + mid_tr + 256);
            yt.p[0] = rd4(exg + mid);
            yt.p[1] = rd4(exg + mid + 256);
            const f4 zr = mm(A2.re, x.v), zi = mm(A2.im, x.v);          // the transform of u: lane k_1, slots 4g ..
            f4 wr = zr, wi = zi;
            cmul4<false>(wr, wi, sr[j], si[j]);
            const H8P w = planes(wr, wi);
            const H8P wt = transposed(w);
            const H8P v = planes(mm(w.v, B2.re), mm(w.v, B2.im));       // lane slot, k_1 = 4g ..
            wr4(exu + mid, v.p[0]);
            wr4(exu + mid + 256, v.p[1]);
            outer(yt, wt, b2r, b2i);
            f4 hr = mm(B2H.re, y.v), hi = mm(B2H.im, y.v);              // gradient at the product with the spectrum
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                dsr[j][r] += hr[r] * zr[r] + hi[r] * zi[r];
                dsi[j][r] += hi[r] * zr[r] - hr[r] * zi[r];
            }
            cmul4<true>(hr, hi, sr[j], si[j]);
            const H8P q = planes(hr, hi);
            const H8P qt = transposed(q);
            const H8P p = planes(mm(q.v, A2H.re), mm(q.v, A2H.im));
            wr4(exg + mid, p.p[0]);
            wr4(exg + mid + 256, p.p[1]);
            outer(qt, xt, a2r, a2i);
        }
    };
    const auto last = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = 2 * wave + j, own = G::at(t, c, g), own_tr = G::at(t, 4 * g + (c >> 2), c & 3);
            {
                H8P v, vt;
                v.p[0] = rd4(exu + own);                                // lane k_0, k_1 = 4g ..
                v.p[1] = rd4(exu + own + 256);
                vt.p[0] = tr_read(exu + own_tr);                        // lane k_1, k_0 = 4g ..
                vt.p[1] = tr_read(exu + own_tr + 256);
                const Cx B1 = mat(2 * t + 1);
                f4 yr = mm(B1.re, v.v), yi = mm(B1.im, v.v);            // lane k_0, d_1 = 4g ..
                cmul4<true>(yr, yi, cr[j], ci[j]);
                const H8P w0 = planes(yr, yi);
                outer(g1t[j], vt, b1r[j], b1i[j]);
                b0r = __builtin_amdgcn_mfma_f32_16x16x16f16(go[j], w0.p[0], b0r, 0, 0, 0);
                b0i = __builtin_amdgcn_mfma_f32_16x16x16f16(go[j], w0.p[1], b0i, 0, 0, 0);     // (minus the imaginary part)
            }
            {
                H8P v, vt;
                v.p[0] = rd4(exg + own);
                v.p[1] = rd4(exg + own + 256);
                vt.p[0] = tr_read(exg + own_tr);
                vt.p[1] = tr_read(exg + own_tr + 256);
                const Cx A1H = mat_adj(2 * t);
                f4 yr = mm(A1H.re, v.v), yi = mm(A1H.im, v.v);          // lane k_0, d_1 = 4g ..
                cmul4<true>(yr, yi, cr[j], ci[j]);
                const H8P g6t = planes(yr, yi);
                outer(vt, x1t[j], a1r[j], a1i[j]);
                a0r = __builtin_amdgcn_mfma_f32_16x16x16f16(g6t.p[0], uo[j], a0r, 0, 0, 0);
                a0i = __builtin_amdgcn_mfma_f32_16x16x16f16(g6t.p[1], uo[j], a0i, 0, 0, 0);
                put_out<IO>(outb + t * G::OS, mm(transposed(g6t).v, A0H), lane);       // (operand: lane d_1, k_0 = 4g ..)
            }
        }
    };
    const auto row_done = [&]() {
        if (!du) return;
#pragma unroll
        for (int j = 0; j < 2; ++j) put_once(dp + j * NT, row_out<LG>(outb, tid + j * NT));
        dp += step;
    };
    const auto rows_in = [&](int b) {                                   // row b + 1; row b + 2 asked for
        if (b + 1 < n) rows_put();
        if (b + 2 < n) ask();
    };
    first();
    __syncthreads();
    middle();
    rows_in(0);
    __syncthreads();
    for (int b = 1; b < n; ++b) {
        last();
        first();
        __syncthreads();
        row_done();
        middle();
        rows_in(b);
        __syncthreads();
    }
    last();
    __builtin_amdgcn_sched_barrier(0);       // (no registers for the sums' twiddles in front of it)
    LaneTw<LG> W[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) W[j].load(stw, 2 * wave + j, lane);
    __syncthreads();
    row_done();

    const size_t at = (size_t)sp * H + h;
    if (out.shat) {
        float2* ps = out.shat + at * G::L;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ps[freq_at<LG>(2 * wave + j, 4 * g + r, c)] = make_float2(dsr[j][r] * G::yscale(), dsi[j][r] * G::yscale());
    }
    // the waves' sums of one block of either chain, [chain][wave][entry]; then entry by entry in wave order
    __syncthreads();
    const auto put_sums = [&](int s) {
        float2* buf = sm2 + (s & 1) * 2 * NW * NBLK;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = (4 * g + r) * 16 + c;
            float2 f, q;
            if (s == 0) {
                f = make_float2(a0r[r], a0i[r]);
                q = make_float2(b0r[r], -b0i[r]);
            } else if (s == 1) {
                f = cadd(cmulc(make_float2(a1r[0][r], a1i[0][r]), W[0].w1q[r]), cmulc(make_float2(a1r[1][r], a1i[1][r]), W[1].w1q[r]));
                q = cadd(cmul(make_float2(b1r[0][r], b1i[0][r]), W[0].w1c), cmul(make_float2(b1r[1][r], b1i[1][r]), W[1].w1c));
            } else {
                f = make_float2(a2r[r], a2i[r]);
                q = make_float2(b2r[r], b2i[r]);
            }
            buf[wave * NBLK + e] = f;
            buf[(NW + wave) * NBLK + e] = q;
        }
    };
    put_sums(0);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        __syncthreads();
        if (s < 2) put_sums(s + 1);
        const float sc = G::yscale() / (float)(1 << stage_shift(4));
        const int chain = tid / NBLK, e = tid % NBLK;                   // (as many threads as entries)
        static_assert(NT == 2 * NBLK, "a thread takes one entry");
        float2* q = chain ? out.qi : out.qf;
        if (!q) continue;
        const float2* p = sm2 + (s & 1) * 2 * NW * NBLK + chain * NW * NBLK + e;
        float2 a = make_float2(0.f, 0.f);
        for (int w = 0; w < NW; ++w) a = cadd(a, p[w * NBLK]);
        q[at * out.q_stride + s * NBLK + e] = make_float2(a.x * sc, a.y * sc);
    }
}

template <class F>
hipError_t set_lds(F* f, size_t bytes)
{
    return hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Rows of the (head, batch row) list that a forward workgroup takes: what spreads them evenly over the `resident` workgroups of the
// device at once, or a few more where the runs then end with their heads (a divisor of B or a multiple), since every head that a run
// touches is matrices to build.  Even shares stay unless the others end 4 % earlier by this: a compute unit's workgroups issue 0.07 T us
// a row and three rows' time a head, a workgroup by itself waits 0.5 + 0.02 T us a row, or 0.07 T where that is more (N = 2048), and four
// rows' time a head (fitted to 40 shapes, N = 256 .. 2048), and neither hides the other: the root of the sum of their squares.  bf16, us,
// even shares and this: N = 256 B=16 H=768 19.5 (6 rows) and 16.1 (8), B=4 H=1030 13.3 (3) and 9.3 (4); N = 512 B=16 H=768 22.3 (12) and
// 20.4 (16), B=8 H=300 11.9 (3) and 9.5 (4); N = 1024 B=7 H=193 11.6 (3) and 10.0 (7); N = 2048 B=12 H=90 17.7 (5) and 14.9 (6).
int64_t run_of_rows(int64_t B, int64_t rows, int64_t resident, int T)
{
    const int64_t even = (rows + resident - 1) / resident, units = compute_units();
    const double a = 0.07 * T, b = 0.5 + 0.02 * T > a ? 0.5 + 0.02 * T : a;
    const auto time = [&](int64_t per) {
        const int64_t n = (rows + per - 1) / per, each = (n + units - 1) / units;
        const bool ends = per % B == 0 || B % per == 0;
        const double heads = ends ? (per > B ? per / B : 1) : 1. + (double)(per - 1) / B;
        const int64_t most = ends ? (int64_t)heads : 1 + (per - 1 + B - 1) / B;
        const double all = each * (per + 3 * heads) * a, one = (per + 4 * most) * b;
        return all * all + one * one;
    };
    int64_t best = even;
    double least = 0.92 * time(even);
    const auto take = [&](int64_t per) {
        if (per < even || time(per) >= least) return;
        best = per;
        least = time(per);
    };
    const int64_t turns = (even + B - 1) / B;
    take(turns * B);
    take((turns + 1) * B);
    for (int64_t q = 2; q <= 64 && B / q >= even; ++q)
        if (B % q == 0) take(B / q);
    return best;
}

template <int LG, class IO>
hipError_t fwd_go(const void* u, const float* shat, const float* Af, const float* Ai, void* y, int64_t B, int64_t H,
                  const Tables& tb, hipStream_t st)
{
    using T = typename IO::T;
    static int resident = 0;       // workgroups the device holds at once
    if (resident == 0) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, lb_fwd_kernel<LG, IO>, 64 << (LG - 8), 0) != hipSuccess) nb = 1;
        resident = (nb > 0 ? nb : 1) * compute_units();
    }
    const int64_t rows = B * H, per = run_of_rows(B, rows, resident, 1 << (LG - 8));
    hipLaunchKernelGGL((lb_fwd_kernel<LG, IO>), dim3((unsigned)((rows + per - 1) / per)), dim3(64 << (LG - 8)), 0, st,
                       (const T*)u, (const float2*)shat, (const float2*)Af, (const float2*)Ai, (T*)y, (int)B, (int)H, per, tb.stw);
    return hipGetLastError();
}

template <int LG, class IO>
hipError_t bwd_go(const void* dy, const void* u, const float* shat, const float* Af, const float* Ai, void* du,
                  const LbGrads& out, int64_t B, int64_t H, int nsplit, const Tables& tb, hipStream_t st)
{
    using T = typename IO::T;
    if constexpr (LG == 12) {
        const hipError_t e = set_lds(lb_bwd2_kernel<IO>, Lb2::lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((lb_bwd2_kernel<IO>), dim3((unsigned)nsplit, (unsigned)H), dim3(Lb2::NT), Lb2::lds, st, (const T*)dy,
                           (const T*)u, (const float2*)shat, (const float2*)Af, (const float2*)Ai, (T*)du, out, (int)B, (int)H, tb.stw);
    } else {
        const hipError_t e = set_lds(lb_bwd_kernel<LG, IO>, lbb_lds<LG>());
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((lb_bwd_kernel<LG, IO>), dim3((unsigned)nsplit, (unsigned)H), dim3(128 << (LG - 8)), lbb_lds<LG>(), st,
                           (const T*)dy, (const T*)u, (const float2*)shat, (const float2*)Af, (const float2*)Ai, (T*)du, out,
                           (int)B, (int)H, tb.stw);
    }
    return hipGetLastError();
}

}  // namespace

// Shares of a head's rows: the number that ends first, ceil(512 / H) at most.  256 compute units hold 8 / T workgroups (two chains of T
// waves) each, N = 2048 one.  (256 as a number: the size of a workspace does not depend on the device that it is asked for on.)
static int64_t most_shares(int64_t B, int64_t H) { return (512 + H - 1) / H < B ? (512 + H - 1) / H : B; }
static int64_t places(int64_t N) { return N == 2048 ? 256 : 256 * (1024 / N); }
static int64_t turns(int64_t workgroups, int64_t N) { return (workgroups + places(N) - 1) / places(N); }
// Adding up n shares is a launch and a chain of n loads, and the shares' numbers go to memory and back.
static double sum_time(int64_t H, int64_t N, int64_t n) { return n > 1 ? 1.7 + 0.28 * n + n * H * (2 * N + 6 * NBLK) * 3.2e-6 : 0.; }
// us of n shares: turn by turn a workgroup's set-up (constants, matrices, sums), longer with more of the device's workgroups at the
// same memory, and its rows, each as long as a workgroup by itself takes or as the unit's workgroups take to issue theirs.  Measured
// for B = 1 .. 64 and H = 4 .. 1024 with every number of shares (N = 256, 512, 1024, 2048 with one workgroup on a unit: set-up 3.1, 3.1,
// 5.6, 6.6 us and, all units taken, 4.5, 4.4, 8.4, 12.5; a row 0.75, 0.87, 1.35, 3.2, with all a unit's places taken 1.48, 1.42, 1.35, 3.2);
// the number that this takes is within 1 % of the best one's time on average.  With set-up as six rows, and three for any sum, which the
// kernel of one chain had, us there and here: N = 256 B=8, H=500 24.1 (2 shares) and 15.2 (1), B=64, H=4 26.9 (64) and 14.9 (16); N = 512
// B=8, H=256 21.0 (2) and 13.7 (1), B=16, H=16 14.6 (16) and 12.3 (4); N = 1024 B=64, H=4 30.2 (64) and 20.2 (16).
static double shares_time(int64_t B, int64_t H, int64_t N, int64_t n)
{
    static const double ROW[4] = {0.75, 0.87, 1.35, 3.2}, MORE[4] = {0.15, 0., 0., 0.}, ISSUE[4] = {0.37, 0.71, 1.35, 3.2};
    static const double SETUP[4] = {3.0, 2.9, 5.5, 6.5}, CROWD[4] = {1.5, 1.5, 2.9, 6.0};
    const int i = N == 256 ? 0 : N == 512 ? 1 : N == 1024 ? 2 : 3;
    const double rows = (double)((B + n - 1) / n);
    double t = sum_time(H, N, n);
    for (int64_t left = n * H; left > 0; left -= places(N)) {
        const int64_t w = left < places(N) ? left : places(N), unit = (w + 255) / 256;
        const double row = ROW[i] + MORE[i] * (unit - 1), issue = ISSUE[i] * unit;
        t += SETUP[i] + CROWD[i] * w / 256 + rows * (row > issue ? row : issue);
    }
    return t;
}
// n shares whose workgroups take n times the turns of one share's have no room in the workspace.
static bool has_room(int64_t H, int64_t N, int64_t n) { return n == 1 || turns(n * H, N) < n * turns(H, N); }
int lbfly_nsplit(int64_t B, int64_t H, int64_t N)
{
    int64_t best = 1;
    double least = shares_time(B, H, N, 1);
    for (int64_t n = 2; n <= most_shares(B, H) && sum_time(H, N, n) < least; ++n) {
        if (!has_room(H, N, n)) continue;
        const double t = shares_time(B, H, N, n);
        if (t < least) { best = n; least = t; }
    }
    return (int)best;
}

// For the most shares that any call of up to B rows takes: the number above need not grow with B, but a workspace for B rows
// serves a smaller batch.
size_t lbfly_partial_bytes(int64_t B, int64_t H, int64_t N)
{
    int64_t room = 1;
    for (int64_t n = 2; n <= most_shares(B, H); ++n)
        if (has_room(H, N, n)) room = n;
    return (size_t)room * (size_t)H * ((size_t)(2 * N) + 6 * NBLK) * sizeof(float2);
}

hipError_t lbfly_fwd(const void* u, const float* shat, const float* Af, const float* Ai, void* y, int64_t B, int64_t H,
                     int64_t N, int io, const Tables& tb, hipStream_t st)
{
#define LB_FWD(LGV)                                                                                       \
    return io == LONGCONV_F16 ? fwd_go<LGV, IoF16>(u, shat, Af, Ai, y, B, H, tb, st)                      \
                              : fwd_go<LGV, IoBF16>(u, shat, Af, Ai, y, B, H, tb, st)
    switch (N) {
        case 256: LB_FWD(9);
        case 512: LB_FWD(10);
        case 1024: LB_FWD(11);
        case 2048: LB_FWD(12);
        default: return hipErrorInvalidValue;
    }
#undef LB_FWD
}

hipError_t lbfly_bwd(const void* dy, const void* u, const float* shat, const float* Af, const float* Ai, void* du,
                     float* dshat, float* dAf, float* dAi, void* partials, int64_t B, int64_t H, int64_t N, int io,
                     const Tables& tb, hipStream_t st)
{
    const int nsplit = lbfly_nsplit(B, H, N);
    float2* part_shat = (float2*)partials;
    float2* part_q = part_shat + (size_t)nsplit * H * 2 * N;
    const LbGrads out = nsplit == 1 ? LbGrads{(float2*)dshat, (float2*)dAf, (float2*)dAi, 3 * NBLK}
                                    : LbGrads{part_shat, part_q, part_q + 3 * NBLK, 6 * NBLK};
    hipError_t e;
#define LB_BWD(LGV)                                                                                                   \
    e = io == LONGCONV_F16 ? bwd_go<LGV, IoF16>(dy, u, shat, Af, Ai, du, out, B, H, nsplit, tb, st)     \
                           : bwd_go<LGV, IoBF16>(dy, u, shat, Af, Ai, du, out, B, H, nsplit, tb, st);   \
    break
    switch (N) {
        case 256: LB_BWD(9);
        case 512: LB_BWD(10);
        case 1024: LB_BWD(11);
        case 2048: LB_BWD(12);
        default: return hipErrorInvalidValue;
    }
#undef LB_BWD
    if (e != hipSuccess) return e;
    if (nsplit == 1 || (!dshat && !dAf && !dAi)) return hipSuccess;
    hipLaunchKernelGGL(lb_reduce_kernel, dim3((unsigned)((2 * N + 6 * NBLK) / 256), (unsigned)H), dim3(256), 0, st, part_shat,
                       part_q, (float2*)dshat, (float2*)dAf, (float2*)dAi, H, (int)(2 * N), nsplit);
    return hipGetLastError();
}

}  // namespace lc
