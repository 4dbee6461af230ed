// Internal launch interfaces between the C-ABI layer and the kernel files.
#pragma once
#include "common.hpp"

namespace lc {

// compute units of the current device (asked once per translation unit; 256 if the query fails)
inline int compute_units()
{
    static int n = 0;
    if (n == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            n = v;
        else
            n = 256;
    }
    return n;
}


struct Problem {
    int64_t B, H, N;
    int io;          // longconv_dtype_t of u, y, dy, du
    int npairs;      // ceil(B/2): two batch rows of one head are transformed as re + i*im
    const void* gate = nullptr;   // convolutions only: [B,H,N] I/O dtype, multiplied into the output before the store
    // bf16 rows that go through chunks (engine_chunk.hip): per head, the bf16 pattern of the largest magnitude of the input
    // rows (max_a: the convolution's input, or u for dk; max_b: dy for dk).  Heads outside the band are scaled by a power of
    // two where the rows are converted, and back in the last step.
    const uint32_t* max_a = nullptr;
    const uint32_t* max_b = nullptr;
    // convolutions of the multi-pass plans with an fp16 spectrum: the per-head exponents of the stored spectrum
    // (spec_exponent), which pass C gives back; NULL = none
    const int* spec_exp = nullptr;
    // single-row kernels: N2 of the 2-D layer, whose image rows of N2 elements stand for 2 N2 samples, the second half
    // zero (not stored, and dropped on output); 0 = rows as they are
    uint32_t pad = 0;
};
// mx[h] = bf16 pattern of max |in[b,h,:]| over b (zeroed first); rows of 16-bit floats only
hipError_t rows_absmax(const void* in, uint32_t* mx, const Problem& pr, hipStream_t st);
// which plans apply Problem::gate inside their own store (the others leave it to a pass of its own)
bool conv_applies_gate(const Plan& pl);

// ---- outer passes of the multi-pass split (multipass.hip) ------------------------
// Pass A (matrix-core engine, fp16 workspace): ws[(h*npairs+p)*L + k1*L2 + n2] = scale * w_L^(n2*k1) * sum_{n1<R/2} w_R^(n1*k1) z[n1*L2+n2],
// z = row(2p) + i*row(2p+1) of `in` (I/O dtype `io`; rows beyond B read as zero).
// If in2/ws2 are given the same is done for a second tensor in the same launch and, if
// dD_part != NULL, per-block partial sums of in*in2 are written for the dD reduction.
hipError_t outer_fwd(const void* in, const void* in2, void* ws, void* ws2, float* dD_part,
                     const Problem& pr, int log2R, int log2L2, float scale, const float2* tw, hipStream_t st,
                     const float* head_max = nullptr);
// stats[h] = max_n |k[h,n]| (consumers derive the head's power-of-two pre-scale with head_scale_of()),
// stats[H + h] and stats[2H + h] = the upper and lower bound statistics of spec_exponent(); the buffer holds
// head_stats_floats(H, N) floats (the three statistics and the partial results they are summed from).
size_t head_stats_floats(int64_t H, int64_t N);
hipError_t head_stats(const float* k, const float* D, float* stats, int64_t H, int64_t N, hipStream_t st);
int outer_fwd_blocks_per_head(const Problem& pr, int log2L2);
// Pass C: rows of `out` <- scale * sum_{k1} conj(w_R^(n1*k1) w_L^(n2*k1)) ws[...], n1 < R/2 only
// (truncation to the first N samples); re -> row 2p, im -> row 2p+1.
hipError_t outer_inv(const void* ws, void* out, const Problem& pr, int log2R, int log2L2, float scale,
                     bool ws_f16, const float2* tw, hipStream_t st);
// dD[h] = sum_b sum_t dy[b,h,t] u[b,h,t], plain fp32 dot product (one workgroup per head).
hipError_t head_dot(const void* dy, const void* u, float* dD, const Problem& pr, hipStream_t st);
// dD[h] = sum of the per-block partials written by outer_fwd.
hipError_t reduce_dD(const float* part, float* dD, int64_t H, int nblk, hipStream_t st);

// dz = dy g (not written if null) and dD[h] = sum_b sum_t dy g u in fp32, fixed order (gated layer); part: H * GATE_SHARES floats (gate.hip)
constexpr int64_t GATE_SHARES = 256;
hipError_t gate_bwd(const void* dy, const void* g, const void* u, void* dz, float* dD, float* part, const Problem& pr, hipStream_t st);

// out = a * b, element by element, n elements of the I/O dtype (n a multiple of 8; out may alias a or b) (gate.hip)
hipError_t ew_mul(const void* a, const void* b, void* out, size_t n, int io, hipStream_t st);

// 2-D convolution through the 1-D path (conv2d.hip): rows padded to twice their width with zeros, and back
hipError_t pad_rows(const void* src, void* dst, size_t rows, size_t row_bytes, hipStream_t st);
hipError_t unpad_rows(const void* src, void* dst, size_t rows, size_t row_bytes, hipStream_t st);

// ---- learned Butterfly extension (lbfly.hip): N = 256 .. 2048, fp16 / bf16 rows -----------------------------------
// rows are split over this many workgroups per head in the backward pass; the partial sums of up to B rows need
// lbfly_partial_bytes
int lbfly_nsplit(int64_t B, int64_t H, int64_t N);
size_t lbfly_partial_bytes(int64_t B, int64_t H, int64_t N);
hipError_t lbfly_fwd(const void* u, const float* shat, const float* Af, const float* Ai, void* y, int64_t B, int64_t H,
                     int64_t N, int io, const Tables& tb, hipStream_t st);
hipError_t lbfly_bwd(const void* dy, const void* u, const float* shat, const float* Af, const float* Ai, void* du,
                     float* dshat, float* dAf, float* dAi, void* partials, int64_t B, int64_t H, int64_t N, int io,
                     const Tables& tb, hipStream_t st);

// ---- block-size study (bsize.hip): forward convolution of fp16 rows with DFT blocks of 2^log2r points, N = 1024, 4096
hipError_t blocksize_fwd(const void* u, const float* shat, void* y, int64_t B, int64_t H, int64_t N, int log2r,
                         const Tables& tb, hipStream_t st);

// ---- kernel regularisers (kreg.hip): Kbar = Squash(Smooth(dropout(K))) and the chain back to K -----------------
constexpr int KREG_MAX_P = 32;
hipError_t kreg_fwd(const float* k, const float* mask, float* kbar, int64_t H, int64_t N, int p, float lam,
                    hipStream_t st);
hipError_t kreg_bwd(const float* k, const float* mask, const float* dkbar, float* dk, int64_t H, int64_t N, int p,
                    float lam, hipStream_t st);

// ---- fp32 VALU engine (engine_valu.hip) --------------------------------------------
constexpr int VALU_INNER_MAX_LOG2 = 14;
constexpr int VALU_ROWS_MIN_LOG2 = TWIST_MIN, VALU_ROWS_MAX_LOG2 = TWIST_MAX;      // fp32 rows that run by themselves (Plan::vrow)
hipError_t valu_fill_tables(const float2** ftw, hipStream_t st);
void valu_fill_plan(Plan& pl);
hipError_t valu_fill_twist(float2* stw, hipStream_t st);       // the part of Tables::stw behind STW_TOTAL
// Spectrum of all heads in fp32, as R = 2^log2R chunks of 2^log2L2 points (pass A taken inside the kernel), stored in
// the order of the engine's own kernels, or scattered to `consumer`'s order if that is given.
hipError_t valu_kspec(const float* k, const float* D, float2* kspec, int64_t H, int64_t N, const SpecOrder* consumer,
                      float scale, const Tables& tb, int log2R, int log2L2, hipStream_t st);
// Spectrum of [k, 0] plus D in natural frequency order, fp32, and its adjoint (dk and dD may be null); N = 256 .. 4096.
hipError_t spectrum_natural(const float* k, const float* D, float* shat, int64_t H, int64_t N, const Tables& tb,
                            hipStream_t st);
hipError_t spectrum_natural_bwd(const float* dshat, float* dk, float* dD, int64_t H, int64_t N, const Tables& tb,
                                hipStream_t st);
hipError_t valu_rows_kspec(const float* k, const float* D, float2* kspec, int64_t H, const Plan& pl, const Tables& tb, hipStream_t st);
// Multi-pass plans: pass A is taken inside the kernels, ws receives pass C's input.
hipError_t valu_conv(const void* in, const float2* kspec, void* out, float2* ws, bool conj, const Problem& pr,
                     const Plan& pl, const Tables& tb, hipStream_t st);
// du, dk and dD in one kernel; any of du / ws_du (multi-pass), dk / ws_A (multi-pass) and dD may be null.  nsplit > 1: dk
// (or ws_A) and dD point to partial buffers [nsplit][...] that sum_partials() adds up in share order.
// zbuf: valu_zbuf_bytes() of scratch.
int valu_bwd_nsplit(int64_t B, int64_t H, const Plan& pl);
int valu_bwd_room(int64_t B, int64_t H, const Plan& pl);       // the most it takes for up to B rows; never falls as B grows
size_t valu_zbuf_bytes(int64_t B, int64_t H, int nsplit, const Plan& pl);
hipError_t valu_bwd(const void* dy, const void* u, const float2* kspec, void* du, float2* ws_du, float* dk, float2* ws_A,
                    float* dD, void* zbuf, int nsplit, const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st);

// ---- fp16 MFMA engine (engine_mfma.hip) ---------------------------------------------
constexpr int MFMA_INNER_MAX_LOG2 = 15;
void mfma_fill_plan(Plan& pl);
hipError_t mfma_conv(const void* in, const float2* kspec, void* out, __half2* ws, bool conj,
                     const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st);
// Multi-pass: dD_part[h*R + k1] receives chunk k1's share of dD[h] (sum them with reduce_dD).
hipError_t mfma_dk(const void* dy, const void* u, float* dk, float* dD, int nsplit, const __half2* ws_u,
                   const __half2* ws_dy, __half2* ws_A, float* dD_part, void* zbuf, const Problem& pr,
                   const Plan& pl, const Tables& tb, hipStream_t st);
// out[i] = sum_s part[s * n + i], s in share order (bitwise repeatable); dk (n_dk values) and dD (n_dD) in one launch
hipError_t sum_partials(const float* dk_part, float* dk, size_t n_dk, const float* dD_part, float* dD, size_t n_dD,
                        int nsplit, hipStream_t st);

// ---- single rows of N = 256 .. 4096 samples on the matrix cores (engine_rows.hip) -----------
constexpr int ROWS_MIN_LOG2 = 8, ROWS_MAX_LOG2 = 12;
hipError_t rows_fill_tables(const void** tab_out, hipStream_t st);
float rows_chain_scale(int lg);      // scale of a forward transform of N = 2^lg samples; an inverse one has twice that
// Spectrum (finds each head's pre-scale itself).  pad: see Problem::pad.
hipError_t rows_kspec(const float* k, const float* D, float2* kspec, int64_t H, const Plan& pl, uint32_t pad, const Tables& tb,
                      hipStream_t st);
hipError_t rows_conv(const void* in, const float2* kspec, void* out, bool conj, const Problem& pr, const Plan& pl,
                     const Tables& tb, hipStream_t st);
// du, dk and dD in one kernel, from one read of dy and u; du (and with it kspec), dk and dD may be null.  nsplit > 1: the
// rows of a head are dealt to nsplit workgroups, dk and dD then point to partial buffers [nsplit][H][N] and [nsplit][H]
// that sum_partials() adds up in share order.
int rows_bwd_nsplit(int64_t B, int64_t H, int lg, bool gated);
// the most shares that any call of up to B rows takes, gated or not: a workspace for B rows serves a smaller batch
int rows_bwd_room(int64_t B, int64_t H, int lg);
// With Problem::gate: the gated layer's backward pass (du and dg both given), dg = dy (ungated output).
hipError_t rows_bwd(const void* dy, const void* u, const float2* kspec, void* du, float* dk, float* dD, void* dg, int nsplit,
                    const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st);

// ---- single rows of N = 8192 and 16384 samples on the matrix cores (engine_long.hip) -----------
constexpr int LONG_MIN_LOG2 = 13, LONG_MAX_LOG2 = 14;
hipError_t long_fill_tables(const void** tab_out, hipStream_t st);
float long_chain_scale();            // scale of a forward transform; an inverse one has twice that
hipError_t long_kspec(const float* k, const float* D, float2* kspec, int64_t H, const Plan& pl, const Tables& tb, hipStream_t st);
hipError_t long_conv(const void* in, const float2* kspec, void* out, bool conj, const Problem& pr, const Plan& pl, const Tables& tb,
                     hipStream_t st);

// du, dk and dD in one kernel; du (and with it kspec), dk and dD may be null.  nsplit > 1: as rows_bwd
int long_bwd_nsplit(int64_t B, int64_t H);
int long_bwd_room(int64_t B, int64_t H);         // as rows_bwd_room
hipError_t long_bwd(const void* dy, const void* u, const float2* kspec, void* du, float* dk, float* dD, int nsplit,
                    const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st);

// ---- rows of N = 65536 and 131072 samples, N / 16384 chunks of their N-point transforms (engine_chunk.hip) ----
// (and dk and dD of rows of 32768 samples, whose convolutions fit a compute unit: row1)
inline bool chunk_plan(const Plan& pl) { return pl.fuse_a && pl.log2R >= 2; }
inline bool chunk_dk_plan(const Plan& pl) { return pl.fuse_a; }
hipError_t chunk_fill_tables(const void** tab_out, hipStream_t st);
// rs: head_stats of k (N = 131072 only)
hipError_t chunk_kspec(const float* k, const float* D, const float* rs, float2* kspec, int64_t H, const Plan& pl, const Tables& tb,
                       hipStream_t st);
// ws: 4 B H N bytes; pr.spec_exp, pr.gate and pr.max_a (powers of two the rows go in with) go into the output
hipError_t chunk_conv(const void* in, const float2* kspec, void* out, void* ws, bool conj, const Problem& pr, const Plan& pl,
                      const Tables& tb, hipStream_t st);
hipError_t chunk_rows(const void* ws, void* out, const Problem& pr, int R, hipStream_t st);
// du (with ws_du as ws above and pr.spec_exp; may be null), dk and dD (may be null).  Each share of a head's rows leaves
// 4 H N bytes in ws_A and H N / 16384 numbers in exps and dD_part.  pr.max_a, pr.max_b: of u and dy
// more: for more than (B - 1) / 2 of them there is no room, otherwise for two
int chunk_bwd_shares(int64_t B, int64_t H, int log2R, bool more);
hipError_t chunk_bwd(const void* dy, const void* u, const float2* kspec, void* du, void* ws_du, float* dk, float* dD, void* ws_A,
                     int* exps, float* dD_part, int ns, const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st);

// ---- cooperative chained matrix-core kernels for 2^13 <= L2 <= 2^15 (engine_coop.hip) --------
constexpr int COOP_MIN_LOG2 = 13, COOP_MAX_LOG2 = 15;
hipError_t coop_fill_tables(const void** tab_out, hipStream_t st);
hipError_t coop_conv(const void* in, const float2* kspec, void* out, __half2* ws, bool conj,
                     const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st);
// ws: pass-A output of the pre-scaled kernel (multi-pass plans only).
hipError_t coop_kspec(const float* k, const __half2* ws, const float* D, const float* rs, float2* kspec, int64_t H,
                      int64_t N, const Plan& pl, const Tables& tb, hipStream_t st);
// zbuf: H * 2N * 4 bytes of scratch (transform of the current u pair, parked between the two transforms)
hipError_t coop_dk(const void* dy, const void* u, float* dk, float* dD, int nsplit, const __half2* ws_u,
                   const __half2* ws_dy, __half2* ws_A, float* dD_part, void* zbuf, const Problem& pr, const Plan& pl,
                   const Tables& tb, hipStream_t st);

}  // namespace lc
