// C-ABI layer of liblongconv: argument validation, planning, workspace carving, dispatch.
// Every step of the path runs in the kernels of engine_rows.hip (rows of 256..4096 samples), engine_long.hip (8192 and 16384),
// engine_coop.hip (32768, and the inner transforms of the forced multi-pass split), engine_chunk.hip (65536 and 131072),
// multipass.hip (outer passes), engine_valu.hip (fp32 I/O), engine_mfma.hip (first-generation in-place kernel, kept as a
// cross-check behind a switch and for 256-point inner transforms), kreg.hip (kernel regularisers), gate.hip (the gate's streaming
// pass) and conv2d.hip (row padding of the 2-D convolution), lbfly.hip (learned Butterfly extension), bsize.hip (block-size
// study); nothing here computes on the host.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>

#include "engines.hpp"

namespace lc {

// One immutable table per device: exp(-2 pi i j / 2^18), j < 2^17 (Appendix C.1 twiddles).
static __device__ float2 g_tw[TW_L / 2];

__global__ void fill_tw_kernel(float2* tw)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= TW_L / 2) return;
    double s, c;
    sincospi(-2.0 * (double)j / (double)TW_L, &s, &c);
    tw[j] = make_float2((float)c, (float)s);
}

static __device__ float2 g_stw[STW_ALL];

__global__ void fill_stw_kernel(float2* stw)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= STW_TOTAL) return;
    const int lgLs = 31 - __clz(i + 32);           // table holding entry i
    const int q = i + 32 - (1 << lgLs);
    const int lgM = lgLs - 4;
    const int d = q >> lgM, suf = q & ((1 << lgM) - 1);
    double s, c;
    sincospi(-2.0 * (double)(d * suf) / (double)(1 << lgLs), &s, &c);
    stw[i] = make_float2((float)c, (float)s);
}

static thread_local char t_hip_err[256] = "";
static hipError_t note(hipError_t e, const char* what)
{
    if (e != hipSuccess) snprintf(t_hip_err, sizeof(t_hip_err), "%s: %s", what, hipGetErrorString(e));
    return e;
}

constexpr int MAX_DEV = 64;
static std::mutex g_init_mu;
static Tables g_tab[MAX_DEV] = {};

// Workspace of longconv_fwd_noalloc: one copy per device in that device's memory, held until the process ends.
// Host code never uses the array's name as an address: the device address is looked up once per device
// (hipGetSymbolAddress, in get_tables) and kept in g_scratch_ptr.
static __device__ __align__(256) unsigned char scratch[LONGCONV_STATIC_SCRATCH_BYTES];
static void* g_scratch_ptr[MAX_DEV] = {};

// Returns the device's table pointer, filling the table on first use (then syncs `st` once).
static hipError_t get_tables(Tables* out, hipStream_t st, bool sync_device, void** scratch_out = nullptr)
{
    int dev = 0;
    hipError_t e = note(hipGetDevice(&dev), "hipGetDevice");
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEV) return note(hipErrorInvalidDevice, "device index");
    std::lock_guard<std::mutex> g(g_init_mu);
    if (!g_tab[dev].tw) {
        float2 *p = nullptr, *q = nullptr;
        e = note(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(g_tw)), "hipGetSymbolAddress");
        if (e != hipSuccess) return e;
        e = note(hipGetSymbolAddress((void**)&q, HIP_SYMBOL(g_stw)), "hipGetSymbolAddress");
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(fill_tw_kernel, dim3(TW_L / 2 / 256), dim3(256), 0, st, p);
        hipLaunchKernelGGL(fill_stw_kernel, dim3((STW_TOTAL + 255) / 256), dim3(256), 0, st, q);
        e = note(hipGetLastError(), "fill tables");
        if (e != hipSuccess) return e;
        e = note(rows_fill_tables(&g_tab[dev].rtab, st), "fill row tables");
        if (e != hipSuccess) return e;
        e = note(long_fill_tables(&g_tab[dev].ltab, st), "fill long-row tables");
        if (e != hipSuccess) return e;
        e = note(chunk_fill_tables(&g_tab[dev].chtab, st), "fill chunk tables");
        if (e != hipSuccess) return e;
        e = note(coop_fill_tables(&g_tab[dev].ctab, st), "fill coop tables");
        if (e != hipSuccess) return e;
        e = note(valu_fill_twist(q, st), "fill twists");
        if (e != hipSuccess) return e;
        e = note(valu_fill_tables(&g_tab[dev].ftw, st), "fill fp32 tables");
        if (e != hipSuccess) return e;
        void* sp = nullptr;
        e = note(hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
        if (e != hipSuccess) return e;
        e = note(sync_device ? hipDeviceSynchronize() : hipStreamSynchronize(st), "table sync");
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = sp;
        g_tab[dev].stw = q;
        g_tab[dev].tw = p;
    }
    *out = g_tab[dev];
    if (scratch_out) *scratch_out = g_scratch_ptr[dev];
    return hipSuccess;
}

static int ilog2(int64_t x)
{
    int l = 0;
    while ((int64_t(1) << l) < x) ++l;
    return l;
}

static int env_int(const char* name, int dflt)
{
    const char* v = getenv(name);
    return (v && *v) ? atoi(v) : dflt;
}

// The switches: defaults, overridden once from the environment, then only by longconv_set_option().
static Options g_opt = {0, 0, 0, 1, 1};
static std::once_flag g_opt_once;
static void load_options_from_env()
{
    if (const char* e = getenv("LONGCONV_ENGINE")) {
        if (!strcmp(e, "valu")) g_opt.engine = 1;
        if (!strcmp(e, "mfma")) g_opt.engine = 2;
    }
    g_opt.inner_log2 = env_int("LONGCONV_INNER_LOG2", 0);
    if (const char* e = getenv("LONGCONV_MFMA_KERNEL")) g_opt.staged = !strcmp(e, "staged");
    g_opt.fuse_pass_a = env_int("LONGCONV_FUSE_PASS_A", 1) != 0;
    g_opt.fuse_bwd = env_int("LONGCONV_FUSE_BWD", 1) != 0;
}
const Options& options()
{
    std::call_once(g_opt_once, load_options_from_env);
    return g_opt;
}

// Plan for (N, io).  fp32 I/O runs the fp32 vector-ALU engine; fp16/bf16 I/O runs the fp16
// matrix-core engine, unless the debug switches say otherwise.
Plan make_plan(int64_t N, int io)
{
    const Options& opt = options();
    Plan pl{};
    pl.log2L = ilog2(2 * N);
    pl.engine = (io == LONGCONV_F32) ? ENGINE_VALU : ENGINE_MFMA;
    if (opt.engine == 1) pl.engine = ENGINE_VALU;
    if (opt.engine == 2 && io != LONGCONV_F32) pl.engine = ENGINE_MFMA;
    int cap = pl.engine == ENGINE_VALU ? VALU_INNER_MAX_LOG2 : MFMA_INNER_MAX_LOG2;
    const int forced = opt.inner_log2;
    if (forced >= 8 && forced < cap) cap = forced;
    pl.log2L2 = pl.log2L < cap ? pl.log2L : cap;
    pl.log2R = pl.log2L - pl.log2L2;
    if (pl.log2R > 5) { pl.log2R = 5; pl.log2L2 = pl.log2L - 5; }   // not reachable for supported N
    // fp32 rows whose N points fit where a pair's 2N would (or, unless a split is forced, N = 16384: twice as fast as in chunks);
    // N <= 1024 stays with pairs: a wave or two per row would leave them nothing to hide behind
    if (pl.engine == ENGINE_VALU && io == LONGCONV_F32 && pl.log2L > VALU_ROWS_MIN_LOG2 &&
        (pl.log2R == 0 || (cap == VALU_INNER_MAX_LOG2 && pl.log2L == VALU_ROWS_MAX_LOG2 + 1))) {
        pl.vrow = pl.log2L - 1;
        pl.log2R = 0;
        pl.log2L2 = pl.log2L;
    }
    if (pl.engine == ENGINE_VALU) valu_fill_plan(pl);
    else mfma_fill_plan(pl);
    return pl;
}

static size_t cw_bytes(const Plan& pl) { return pl.engine == ENGINE_VALU ? sizeof(float2) : sizeof(__half2); }
// bytes per stored spectrum bin: fp16 complex for the wave and cooperative matrix-core kernels, fp32 complex otherwise
static size_t spec_bytes(const Plan& pl)
{
    return (pl.engine == ENGINE_MFMA && (pl.order.wave_lg || pl.order.long_lg || pl.order.coop_lg)) ? sizeof(__half2) : sizeof(float2);
}
static size_t up256(size_t x) { return (x + 255) & ~size_t(255); }
// the stored spectrum of H heads: the bins, and for fp16 storage a trailer of H per-head exponents (spec_exponent)
static bool spec_is_f16(const Plan& pl) { return spec_bytes(pl) == sizeof(__half2); }
static size_t spec_total_bytes(int64_t H, size_t L, const Plan& pl)
{
    return (size_t)H * L * spec_bytes(pl) + (spec_is_f16(pl) ? (((size_t)H * sizeof(int) + 15) & ~size_t(15)) : 0);
}
static const int* spec_exp_ptr(const float2* kspec, int64_t H, size_t L, const Plan& pl)
{
    return spec_is_f16(pl) ? reinterpret_cast<const int*>(reinterpret_cast<const uint32_t*>(kspec) + (size_t)H * L) : nullptr;
}

struct WsLayout {
    size_t kspec, kscratch, hscale, ws1, ws2, wsA, dpart, chunk, zbuf, dkpart, ddpart, rowmx, total;
    int nblk;
};

// Single-pass plans: the backward kernels run one workgroup per head; with few heads the rows (pairs) of a head are dealt
// to `nsplit` workgroups, whose partial dk and dD are then summed in a fixed order.
static int dk_nsplit(int64_t B, int64_t H, const Plan& pl, bool gated)
{
    if (pl.engine == ENGINE_VALU) return valu_bwd_nsplit(B, H, pl);
    if (pl.engine == ENGINE_MFMA && pl.order.wave_lg) return rows_bwd_nsplit(B, H, pl.order.wave_lg, gated);
    if (pl.engine == ENGINE_MFMA && pl.order.long_lg) return long_bwd_nsplit(B, H);
    return 1;
}
// the most of them that a call of up to B rows takes (the numbers above need not grow with B, the workspace has to)
static int dk_room(int64_t B, int64_t H, const Plan& pl)
{
    if (pl.engine == ENGINE_MFMA && pl.order.wave_lg) return rows_bwd_room(B, H, pl.order.wave_lg);
    if (pl.engine == ENGINE_MFMA && pl.order.long_lg) return long_bwd_room(B, H);
    if (pl.engine == ENGINE_VALU) return valu_bwd_room(B, H, pl);
    return 1;
}

// bf16 rows of the multi-pass plans that take pass A inside the inner kernels are scaled per head (see rows_absmax)
static bool rows_rescaled(const Plan& pl, int io)
{
    return io == LONGCONV_BF16 && pl.engine == ENGINE_MFMA && pl.log2R > 0 && pl.fuse_a;
}

static WsLayout carve(int64_t B, int64_t H, int64_t N, const Plan& pl, bool backward, int io)
{
    WsLayout w{};
    const size_t L = size_t(1) << pl.log2L;
    const size_t npairs = (size_t)((B + 1) / 2);
    size_t off = 0;
    w.kspec = off; off += up256(spec_total_bytes(H, L, pl));
    // pass-A output of k, for the spectrum routes that run pass A as a kernel of its own
    const bool mc = pl.engine == ENGINE_MFMA && (pl.order.wave_lg || pl.order.coop_lg);
    const bool kscr = mc && pl.log2R && !pl.fuse_a;
    w.kscratch = off; if (kscr) off += up256((size_t)H * L * sizeof(float2));
    w.hscale = off; off += up256(head_stats_floats(H, N) * sizeof(float));
    // rows that go from memory to memory (row1) have no chunks to keep; pass A's outputs for dk, and what goes with them,
    // belong to plans that run it as a kernel of its own (not the fp32 engine, and not where dk comes straight from the rows)
    const bool chunks = pl.engine == ENGINE_MFMA && chunk_dk_plan(pl);
    const bool outer_a = pl.engine == ENGINE_MFMA && !chunks;
    w.ws1 = off; if (pl.log2R && !pl.row1) off += up256((size_t)H * npairs * L * cw_bytes(pl));
    w.ws2 = off; if (pl.log2R && backward && outer_a) off += up256((size_t)H * npairs * L * cw_bytes(pl));
    w.wsA = off; if (pl.log2R && backward) off += up256((size_t)H * L * cw_bytes(pl));
    w.nblk = (int)(npairs * ((size_t(1) << pl.log2L2) / 256));
    const size_t npart = (size_t)w.nblk > (size_t(1) << pl.log2R) ? (size_t)w.nblk : (size_t(1) << pl.log2R);
    w.dpart = off; if (pl.log2R && backward && outer_a) off += up256((size_t)H * npart * sizeof(float));
    w.chunk = off; if (backward && chunks) off += up256((size_t)chunk_bwd_shares(B, H, pl.log2R, false) * (H << pl.log2R) * 2 * sizeof(float));
    const size_t shares = backward ? dk_room(B, H, pl) : 1;
    w.zbuf = off;
    if (backward && pl.order.coop_lg && outer_a) off += up256((size_t)H * L * sizeof(__half2));
    if (backward && pl.engine == ENGINE_VALU) off += up256(valu_zbuf_bytes(B, H, (int)shares, pl));
    // partial dk rows, or (fp32 engine, multi-pass) partial sets of pass C's complex chunks
    w.dkpart = off; if (shares > 1) off += up256(shares * H * (pl.log2R ? 2 * L : L / 2) * sizeof(float));
    w.ddpart = off; if (shares > 1) off += up256(shares * H * sizeof(float));
    // bf16 rows of the multi-pass plans with pass A inside the inner kernels: per-head maxima of u and dy
    w.rowmx = off; if (rows_rescaled(pl, io)) off += up256((size_t)2 * H * sizeof(uint32_t));
    w.total = off;
    return w;
}

static size_t io_bytes(int io) { return io == LONGCONV_F32 ? 4 : 2; }
static size_t gated_dz_bytes(int64_t B, int64_t H, int64_t N, int io)
{
    return up256((size_t)B * H * N * io_bytes(io));
}

static bool pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }
static int check_shape(int64_t B, int64_t H, int64_t N, int io)
{
    if (io != LONGCONV_F32 && io != LONGCONV_F16 && io != LONGCONV_BF16) return LONGCONV_ERR_DTYPE;
    if (B < 1 || H < 1 || !pow2(N) || N < 256 || N > 131072) return LONGCONV_ERR_SHAPE;
    if (B > (int64_t(1) << 24) || H > 65535) return LONGCONV_ERR_SHAPE;
    if (((B + 1) / 2) * H > (int64_t(1) << 22)) return LONGCONV_ERR_SHAPE;   // (head, pair) items index 1-D grids
    return LONGCONV_OK;
}
static bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

// Spectrum of all heads into `kspec` (storage order and scale of plan `pl`).
static hipError_t run_kspec(const float* k, const float* D, float2* kspec, float2* kscratch, float* hscale,
                            int64_t H, int64_t N, const Plan& pl, const Tables& tb, hipStream_t st, uint32_t pad = 0)
{
    const float2* tw = tb.tw;
    if (pl.engine == ENGINE_MFMA && pl.order.long_lg) return long_kspec(k, D, kspec, H, pl, tb, st);
    if (pl.engine == ENGINE_MFMA && (pl.order.wave_lg || pl.order.coop_lg)) {
        // matrix-core route: per-head power-of-two pre-scale, (pass A,) forward half of the fused kernel
        if (pl.order.wave_lg) return rows_kspec(k, D, kspec, H, pl, pad, tb, st);
        // the kernel reads k itself and finds the maxima
        // (N = 131072: eight chunks per head would each scan 512 KB, so the maxima are found once, in front)
        if (pl.row1) return coop_kspec(k, nullptr, D, nullptr, kspec, H, N, pl, tb, st);
        if (chunk_plan(pl) && pl.log2R == 2) return chunk_kspec(k, D, nullptr, kspec, H, pl, tb, st);
        hipError_t e = head_stats(k, D, hscale, H, N, st);
        if (e != hipSuccess) return e;
        if (chunk_plan(pl)) return chunk_kspec(k, D, hscale, kspec, H, pl, tb, st);
        if (pl.log2R) {
            Problem pk{1, H, N, LONGCONV_F32, 1};
            e = outer_fwd(k, nullptr, kscratch, nullptr, nullptr, pk, pl.log2R, pl.log2L2, 1.0f, tw, st, hscale);
            if (e != hipSuccess) return e;
        }
        return coop_kspec(k, (const __half2*)kscratch, D, hscale, kspec, H, N, pl, tb, st);
    }
    if (pl.engine == ENGINE_VALU && pl.vrow) return valu_rows_kspec(k, D, kspec, H, pl, tb, st);
    if (pl.engine == ENGINE_VALU) return valu_kspec(k, D, kspec, H, N, nullptr, pl.kscale, tb, pl.log2R, pl.log2L2, st);
    // staged matrix-core kernel: fp32 spectrum in that kernel's digit-reversed order
    const int lg2 = pl.log2L < VALU_INNER_MAX_LOG2 ? pl.log2L : VALU_INNER_MAX_LOG2;
    return valu_kspec(k, D, kspec, H, N, &pl.order, pl.kscale, tb, pl.log2L - lg2, lg2, st);
}

// y = conv(in, spectrum) (or correlation when conj): all passes of the plan.
static hipError_t run_conv(const void* in, const float2* kspec, void* out, void* ws1, bool conj,
                           const Problem& pr, const Plan& pl, const Tables& tb, hipStream_t st,
                           bool ws1_ready)
{
    hipError_t e;
    const float2* tw = tb.tw;
    const bool f16ws = pl.engine == ENGINE_MFMA;
    if (pl.engine == ENGINE_MFMA && chunk_plan(pl)) {
        Problem pc = pr;
        pc.spec_exp = spec_exp_ptr(kspec, pr.H, size_t(1) << pl.log2L, pl);
        return chunk_conv(in, kspec, out, ws1, conj, pc, pl, tb, st);
    }
    if (pl.engine == ENGINE_MFMA && pl.log2R && !ws1_ready && !pl.row1) {
        e = outer_fwd(in, nullptr, ws1, nullptr, nullptr, pr, pl.log2R, pl.log2L2, 1.0f, tw, st);
        if (e != hipSuccess) return e;
    }
    if (pl.engine == ENGINE_VALU)
        e = valu_conv(in, kspec, out, (float2*)ws1, conj, pr, pl, tb, st);
    else
        e = mfma_conv(in, kspec, out, (__half2*)ws1, conj, pr, pl, tb, st);
    if (e != hipSuccess) return e;
    if (pl.log2R && !pl.row1) {
        Problem pc = pr;     // pass C gives the output the power of two that the stored spectrum left out
        pc.spec_exp = spec_exp_ptr(kspec, pr.H, size_t(1) << pl.log2L, pl);
        e = outer_inv(ws1, out, pc, pl.log2R, pl.log2L2, 1.0f, f16ws, tw, st);
    }
    return e;
}

}  // namespace lc

using namespace lc;

extern "C" {

int longconv_init(void)
{
    Tables tb;
    return get_tables(&tb, nullptr, true) == hipSuccess ? LONGCONV_OK : LONGCONV_ERR_HIP;
}

size_t longconv_kspec_bytes(int64_t H, int64_t N, int io)
{
    if (check_shape(1, H, N, io) != LONGCONV_OK) return 0;
    return spec_total_bytes(H, (size_t)(2 * N), make_plan(N, io));
}

size_t longconv_workspace_bytes(int64_t B, int64_t H, int64_t N, int io, int backward)
{
    if (check_shape(B, H, N, io) != LONGCONV_OK) return 0;
    const Plan pl = make_plan(N, io);
    const size_t base = carve(B, H, N, pl, backward != 0, io).total;
    // gated backward: room for dz = dy * g behind the backward pass's own workspace
    return backward == 2 ? base + gated_dz_bytes(B, H, N, io) : base;
}

int longconv_kspec_compute(const float* k, const float* D, void* kspec, int64_t H, int64_t N, int io,
                           void* workspace, size_t workspace_bytes, void* stream)
{
    int s = check_shape(1, H, N, io);
    if (s != LONGCONV_OK) return s;
    if (!k || !D || !kspec) return LONGCONV_ERR_NULL;
    if (misaligned(k) || misaligned(kspec) || misaligned(workspace)) return LONGCONV_ERR_ALIGN;
    const Plan pl = make_plan(N, io);
    const WsLayout w = carve(1, H, N, pl, false, io);
    const size_t need = w.ws1 - w.kscratch;   // producer scratch and per-head scales
    if (need && (!workspace || workspace_bytes < w.kscratch + need)) return LONGCONV_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    Tables tb;
    if (get_tables(&tb, st, false) != hipSuccess) return LONGCONV_ERR_HIP;
    float2* scratch = (float2*)((char*)workspace + w.kscratch);
    if (note(run_kspec(k, D, (float2*)kspec, scratch, (float*)((char*)workspace + w.hscale), H, N, pl, tb, st),
             "kspec") != hipSuccess)
        return LONGCONV_ERR_HIP;
    return LONGCONV_OK;
}

// Forward pass.  own_scratch: the workspace is the library's static device array (longconv_fwd_noalloc);
// otherwise the caller's.
static int fwd_impl(const void* u, const float* k, const float* D, const void* kspec, void* y, int64_t B,
                    int64_t H, int64_t N, int io, void* workspace, size_t workspace_bytes, void* stream,
                    bool own_scratch, const void* gate = nullptr, uint32_t pad = 0)
{
    int s = check_shape(B, H, N, io);
    if (s != LONGCONV_OK) return s;
    if (!u || !y || (!kspec && (!k || !D))) return LONGCONV_ERR_NULL;
    if (misaligned(u) || misaligned(y) || misaligned(k) || misaligned(kspec) || misaligned(workspace))
        return LONGCONV_ERR_ALIGN;
    const Plan pl = make_plan(N, io);
    const WsLayout w = carve(B, H, N, pl, false, io);
    if (own_scratch) {
        if (w.total > (size_t)LONGCONV_STATIC_SCRATCH_BYTES) return LONGCONV_ERR_WORKSPACE;
    } else if (!workspace || workspace_bytes < w.total) {
        return LONGCONV_ERR_WORKSPACE;
    }
    hipStream_t st = (hipStream_t)stream;
    Tables tb;
    if (get_tables(&tb, st, false, own_scratch ? &workspace : nullptr) != hipSuccess) return LONGCONV_ERR_HIP;
    char* base = (char*)workspace;
    const float2* ks = (const float2*)kspec;
    if (!ks) {
        if (note(run_kspec(k, D, (float2*)(base + w.kspec), (float2*)(base + w.kscratch), (float*)(base + w.hscale),
                           H, N, pl, tb, st, pad), "kspec") != hipSuccess)
            return LONGCONV_ERR_HIP;
        ks = (const float2*)(base + w.kspec);
    }
    Problem pr{B, H, N, io, (int)((B + 1) / 2)};
    pr.pad = pad;
    if (rows_rescaled(pl, io) && !pl.row1) {      // (row1: the kernel measures the rows itself)
        uint32_t* mx = (uint32_t*)(base + w.rowmx);
        if (note(rows_absmax(u, mx, pr, st), "rows max") != hipSuccess) return LONGCONV_ERR_HIP;
        pr.max_a = mx;
    }
    // output gate (y = g * z): inside the convolution's store where the plan's kernel has that form, otherwise a
    // pass of its own over y
    const bool fused_gate = gate && conv_applies_gate(pl);
    if (fused_gate) pr.gate = gate;
    if (note(run_conv(u, ks, y, base + w.ws1, false, pr, pl, tb, st, false), "fwd") != hipSuccess)
        return LONGCONV_ERR_HIP;
    if (gate && !fused_gate && note(ew_mul(y, gate, y, (size_t)B * H * N, io, st), "gate") != hipSuccess)
        return LONGCONV_ERR_HIP;
    return LONGCONV_OK;
}

int longconv_fwd(const void* u, const float* k, const float* D, const void* kspec, void* y, int64_t B,
                 int64_t H, int64_t N, int io, void* workspace, size_t workspace_bytes, void* stream)
{
    return fwd_impl(u, k, D, kspec, y, B, H, N, io, workspace, workspace_bytes, stream, false);
}

int longconv_fwd_noalloc(const void* u, const float* k, const float* D, const void* kspec, void* y, int64_t B,
                         int64_t H, int64_t N, int io, void* stream)
{
    return fwd_impl(u, k, D, kspec, y, B, H, N, io, nullptr, 0, stream, true);
}

int longconv_fwd_gated(const void* u, const float* k, const float* D, const void* kspec, const void* g, void* y,
                       int64_t B, int64_t H, int64_t N, int io, void* workspace, size_t workspace_bytes,
                       void* stream)
{
    if (!g) return LONGCONV_ERR_NULL;
    if (misaligned(g)) return LONGCONV_ERR_ALIGN;
    int s = fwd_impl(u, k, D, kspec, y, B, H, N, io, workspace, workspace_bytes, stream, false, g);
    return s;
}

static int bwd_impl(const void* dy, const void* u, const float* k, const float* D, const void* kspec, void* du,
                    float* dk, float* dD, int64_t B, int64_t H, int64_t N, int io, void* workspace,
                    size_t workspace_bytes, void* stream, uint32_t pad, const void* gate = nullptr, void* dg = nullptr);

int longconv_bwd_gated(const void* dy, const void* g, const void* u, const float* k, const float* D,
                       const void* kspec, void* du, float* dk, float* dD, void* dg, int64_t B, int64_t H,
                       int64_t N, int io, void* workspace, size_t workspace_bytes, void* stream)
{
    int s = check_shape(B, H, N, io);
    if (s != LONGCONV_OK) return s;
    if (!dy || !g || (dg && (!u || (!kspec && (!k || !D))))) return LONGCONV_ERR_NULL;
    if (misaligned(dy) || misaligned(g) || misaligned(dg) || misaligned(workspace)) return LONGCONV_ERR_ALIGN;
    const size_t base = longconv_workspace_bytes(B, H, N, io, 1);
    if (!workspace || workspace_bytes < base + gated_dz_bytes(B, H, N, io)) return LONGCONV_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const size_t n = (size_t)B * H * N;
    const Plan pl = make_plan(N, io);
    if (pl.engine == ENGINE_MFMA && pl.fuse_bwd && pl.order.wave_lg && du && dg && (dk || dD))      // all of it from one kernel
        return bwd_impl(dy, u, k, D, kspec, du, dk, dD, B, H, N, io, workspace, base, stream, 0, g, dg);
    if (du || dk || dD) {
        // dz = dy * g is what the convolution's backward pass receives.  dD = sum dy g u comes from the same reads, straight from
        // the three tensors: the rounding of dz to the I/O dtype stays out of it.  Its partial sums lie where the backward pass
        // puts its spectrum (2N numbers a head), if it has to make one, later.
        void* dz = du || dk ? (char*)workspace + base : nullptr;
        Problem pr{B, H, N, io, (int)((B + 1) / 2)};
        static_assert(GATE_SHARES <= 2 * 256, "the partial sums fit the spectrum of the shortest rows");
        if (dD && u) {
            if (note(gate_bwd(dy, g, u, dz, dD, (float*)workspace, pr, st), "gate dD") != hipSuccess) return LONGCONV_ERR_HIP;
        } else if (dz && note(ew_mul(dy, g, dz, n, io, st), "gate") != hipSuccess) {
            return LONGCONV_ERR_HIP;
        }
        if (dz) {
            s = longconv_bwd(dz, u, k, D, kspec, du, dk, nullptr, B, H, N, io, workspace, base, stream);
            if (s != LONGCONV_OK) return s;
        }
        if (dD && !u) return LONGCONV_ERR_NULL;
    }
    if (dg) {
        // dg = dy * z, z the ungated output recomputed: the gated forward with dy in the gate's place
        s = fwd_impl(u, k, D, kspec, dg, B, H, N, io, workspace, base, stream, false, dy);
        if (s != LONGCONV_OK) return s;
    }
    return LONGCONV_OK;
}

static int bwd_impl(const void* dy, const void* u, const float* k, const float* D, const void* kspec, void* du,
                    float* dk, float* dD, int64_t B, int64_t H, int64_t N, int io, void* workspace,
                    size_t workspace_bytes, void* stream, uint32_t pad, const void* gate, void* dg)
{
    int s = check_shape(B, H, N, io);
    if (s != LONGCONV_OK) return s;
    const bool want_dkD = dk || dD;
    if (!dy || (want_dkD && !u) || (du && !kspec && (!k || !D))) return LONGCONV_ERR_NULL;
    if (misaligned(dy) || misaligned(u) || misaligned(k) || misaligned(kspec) || misaligned(du) ||
        misaligned(dk) || misaligned(workspace))
        return LONGCONV_ERR_ALIGN;
    const Plan pl = make_plan(N, io);
    const WsLayout w = carve(B, H, N, pl, true, io);
    if (!workspace || workspace_bytes < w.total) return LONGCONV_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    Tables tb;
    if (get_tables(&tb, st, false) != hipSuccess) return LONGCONV_ERR_HIP;
    const float2* tw = tb.tw;
    char* base = (char*)workspace;
    Problem pr{B, H, N, io, (int)((B + 1) / 2)};
    pr.pad = pad;
    pr.gate = gate;
    const bool f16ws = pl.engine == ENGINE_MFMA;
    bool dy_ready = false;   // multi-pass: pass A of dy already in ws1
    uint32_t* mx_u = nullptr;      // bf16 rows of these multi-pass plans: per-head maxima of u and dy
    uint32_t* mx_dy = nullptr;
    if (rows_rescaled(pl, io) && (want_dkD || !pl.row1)) {
        mx_u = (uint32_t*)(base + w.rowmx);
        mx_dy = mx_u + H;
        hipError_t e = hipSuccess;
        if (want_dkD) e = rows_absmax(u, mx_u, pr, st);
        if (e == hipSuccess) e = rows_absmax(dy, mx_dy, pr, st);
        if (note(e, "rows max") != hipSuccess) return LONGCONV_ERR_HIP;
    }

    if (want_dkD && du && pl.engine == ENGINE_MFMA && pl.fuse_bwd) {
        // everything from one kernel: dy and u are read once, dy is transformed once
        const float2* ks = (const float2*)kspec;
        if (!ks) {
            if (note(run_kspec(k, D, (float2*)(base + w.kspec), (float2*)(base + w.kscratch),
                               (float*)(base + w.hscale), H, N, pl, tb, st, pad), "kspec") != hipSuccess)
                return LONGCONV_ERR_HIP;
            ks = (const float2*)(base + w.kspec);
        }
        const int ns = dk_nsplit(B, H, pl, gate != nullptr);
        float* dkp = (float*)(base + w.dkpart);
        float* ddp = (float*)(base + w.ddpart);
        float *dk1 = ns > 1 ? (dk ? dkp : nullptr) : dk, *dD1 = ns > 1 ? (dD ? ddp : nullptr) : dD;
        hipError_t e = pl.order.long_lg ? long_bwd(dy, u, ks, du, dk1, dD1, ns, pr, pl, tb, st)
                                        : rows_bwd(dy, u, ks, du, dk1, dD1, dg, ns, pr, pl, tb, st);
        if (e == hipSuccess && ns > 1) e = sum_partials(dkp, dk, (size_t)H * (pad ? N / 2 : N), ddp, dD, (size_t)H, ns, st);
        if (note(e, "bwd") != hipSuccess) return LONGCONV_ERR_HIP;
        return LONGCONV_OK;
    }
    if (want_dkD && pl.engine == ENGINE_VALU) {
        // one kernel for what is asked for (du alone: the convolution kernel, below)
        const float2* ks = (const float2*)kspec;
        if (du && !ks) {
            if (note(run_kspec(k, D, (float2*)(base + w.kspec), nullptr, nullptr, H, N, pl, tb, st), "kspec") != hipSuccess)
                return LONGCONV_ERR_HIP;
            ks = (const float2*)(base + w.kspec);
        }
        const int ns = dk_nsplit(B, H, pl, gate != nullptr);
        const bool multi = pl.log2R != 0;
        float* dkp = (float*)(base + w.dkpart);
        float* ddp = (float*)(base + w.ddpart);
        float* acc = multi ? (float*)(base + w.wsA) : dk;         // where the (summed) dk rows or chunks belong
        const size_t n_acc = dk ? (size_t)H * (multi ? 4 * N : N) : 0;
        float* to = dk ? (ns > 1 ? dkp : acc) : nullptr;
        hipError_t e = valu_bwd(dy, u, ks, du, du ? (float2*)(base + w.ws1) : nullptr, multi ? nullptr : to,
                                multi ? (float2*)to : nullptr, dD ? (ns > 1 ? ddp : dD) : nullptr, base + w.zbuf, ns, pr, pl,
                                tb, st);
        if (e == hipSuccess && ns > 1) e = sum_partials(dkp, n_acc ? acc : nullptr, n_acc, ddp, dD, (size_t)H, ns, st);
        if (e == hipSuccess && multi && dk)
            e = outer_inv(base + w.wsA, dk, Problem{1, H, N, LONGCONV_F32, 1}, pl.log2R, pl.log2L2, pl.dkscale, false, tw, st);
        if (e == hipSuccess && multi && du) e = outer_inv(base + w.ws1, du, pr, pl.log2R, pl.log2L2, 1.0f, false, tw, st);
        return note(e, "bwd") == hipSuccess ? LONGCONV_OK : LONGCONV_ERR_HIP;
    }
    if (want_dkD && pl.engine == ENGINE_MFMA && chunk_dk_plan(pl)) {
        // one walk over the rows for all that is asked for (switch fuse_bwd = 0, and N = 32768: du by itself, below)
        void* du1 = chunk_plan(pl) && options().fuse_bwd ? du : nullptr;
        const float2* ks = (const float2*)kspec;
        if (du1 && !ks) {
            if (note(run_kspec(k, D, (float2*)(base + w.kspec), nullptr, (float*)(base + w.hscale), H, N, pl, tb, st), "kspec") !=
                hipSuccess)
                return LONGCONV_ERR_HIP;
            ks = (const float2*)(base + w.kspec);
        }
        Problem prc = pr;
        prc.max_a = mx_u;
        prc.max_b = mx_dy;
        prc.spec_exp = du1 ? spec_exp_ptr(ks, H, size_t(1) << pl.log2L, pl) : nullptr;
        // The workspace has room for the results of two shares of a head's rows, 4 H N bytes each.  More of them, and the numbers that
        // go with them (at most 2 KB), wait in the 2 B H N bytes of du, which is written behind them from start to end.
        const int ns = chunk_bwd_shares(B, H, pl.log2R, du != nullptr);
        char* parts = ns > 2 ? (char*)du : base + w.wsA;
        int* exps = (int*)(ns > 2 ? parts + (size_t)ns * H * N * 4 : base + w.chunk);
        float* dD_part = (float*)exps + (size_t)ns * (H << pl.log2R);
        if (note(chunk_bwd(dy, u, ks, du1, base + w.ws1, dk, dD, parts, exps, dD_part, ns, prc, pl, tb, st), "bwd") != hipSuccess)
            return LONGCONV_ERR_HIP;
        if (du1) return LONGCONV_OK;
    } else if (want_dkD) {
        hipError_t e = hipSuccess;
        float* dpart = (float*)(base + w.dpart);
        if (pl.log2R) {
            // pass A for u and dy in one launch; its blocks also leave dD's partial dot products
            e = outer_fwd(dy, u, base + w.ws1, base + w.ws2, dD ? dpart : nullptr, pr, pl.log2R, pl.log2L2, 1.0f, tw, st);
            dy_ready = true;
            if (e == hipSuccess && dD) e = reduce_dD(dpart, dD, H, w.nblk, st);
        }
        if (e == hipSuccess && (dk || !pl.log2R)) {
            const int ns = dk_nsplit(B, H, pl, false);
            float* dkp = (float*)(base + w.dkpart);
            float* ddp = (float*)(base + w.ddpart);
            float* dD1 = pl.log2R ? nullptr : dD;
            e = mfma_dk(dy, u, ns > 1 ? (dk ? dkp : nullptr) : dk, ns > 1 ? (dD1 ? ddp : nullptr) : dD1, ns,
                        (const __half2*)(base + w.ws2), (const __half2*)(base + w.ws1), (__half2*)(base + w.wsA), nullptr,
                        base + w.zbuf, pr, pl, tb, st);
            if (e == hipSuccess && ns > 1) e = sum_partials(dkp, dk, (size_t)H * (pad ? N / 2 : N), ddp, dD1, (size_t)H, ns, st);
        }
        if (e == hipSuccess && pl.log2R && dk)           // heads as single rows, real part only
            e = outer_inv(base + w.wsA, dk, Problem{1, H, N, LONGCONV_F32, 1}, pl.log2R, pl.log2L2, pl.dkscale, f16ws, tw, st);
        if (note(e, "bwd dk/dD") != hipSuccess) return LONGCONV_ERR_HIP;
    }
    if (du) {
        const float2* ks = (const float2*)kspec;
        if (!ks) {
            if (note(run_kspec(k, D, (float2*)(base + w.kspec), (float2*)(base + w.kscratch),
                               (float*)(base + w.hscale), H, N, pl, tb, st, pad), "kspec") != hipSuccess)
                return LONGCONV_ERR_HIP;
            ks = (const float2*)(base + w.kspec);
        }
        Problem prd = pr;
        prd.max_a = dy_ready ? nullptr : mx_dy;
        if (note(run_conv(dy, ks, du, base + w.ws1, true, prd, pl, tb, st, dy_ready), "bwd du") != hipSuccess)
            return LONGCONV_ERR_HIP;
    }
    return LONGCONV_OK;
}

int longconv_bwd(const void* dy, const void* u, const float* k, const float* D, const void* kspec, void* du,
                 float* dk, float* dD, int64_t B, int64_t H, int64_t N, int io, void* workspace,
                 size_t workspace_bytes, void* stream)
{
    return bwd_impl(dy, u, k, D, kspec, du, dk, dD, B, H, N, io, workspace, workspace_bytes, stream, 0);
}

// ---- 2-D long convolution: rows padded to twice their width, then the 1-D path on the row-major sequence -------
// The single-row kernels pad while they load and drop the padding while they store; for the other plans padded copies
// are made in the workspace.
static bool pads_itself(const Plan& pl) { return pl.engine == ENGINE_MFMA && pl.order.wave_lg; }

struct Ws2d {
    size_t base, kp, up, yp, dup, dkp, total;     // byte offsets; base = size of the 1-D call's own workspace
};
static int check_shape2d(int64_t B, int64_t H, int64_t N1, int64_t N2, int io)
{
    if (io != LONGCONV_F32 && io != LONGCONV_F16 && io != LONGCONV_BF16) return LONGCONV_ERR_DTYPE;
    if (!pow2(N1) || !pow2(N2) || N2 < 8 || N1 > 131072 || N2 > 65536) return LONGCONV_ERR_SHAPE;
    return check_shape(B, H, 2 * N1 * N2, io);
}
static Ws2d carve2d(int64_t B, int64_t H, int64_t N, int io, bool backward)
{
    Ws2d w{};
    const size_t rows = up256((size_t)B * H * N * io_bytes(io)), heads = up256((size_t)H * N * sizeof(float));
    size_t off = up256(longconv_workspace_bytes(B, H, N, io, backward ? 1 : 0));
    w.base = off;
    w.total = off + (backward ? 256 : 0);          // (a backward size is above the forward one of its shape at every length)
    if (pads_itself(make_plan(N, io))) return w;   // no copies
    w.kp = off;  off += heads;
    w.up = off;  off += rows;
    w.yp = off;  off += rows;                      // y of the forward pass, dy of the backward pass
    if (backward) {
        w.dup = off; off += rows;
        w.dkp = off; off += heads;
    }
    w.total = off;
    return w;
}

size_t longconv2d_workspace_bytes(int64_t B, int64_t H, int64_t N1, int64_t N2, int io, int backward)
{
    if (check_shape2d(B, H, N1, N2, io) != LONGCONV_OK) return 0;
    return carve2d(B, H, 2 * N1 * N2, io, backward != 0).total;
}

int longconv2d_fwd(const void* u, const float* k, const float* D, void* y, int64_t B, int64_t H, int64_t N1,
                   int64_t N2, int io, void* workspace, size_t workspace_bytes, void* stream)
{
    int s = check_shape2d(B, H, N1, N2, io);
    if (s != LONGCONV_OK) return s;
    if (!u || !k || !D || !y) return LONGCONV_ERR_NULL;
    if (misaligned(u) || misaligned(k) || misaligned(y) || misaligned(workspace)) return LONGCONV_ERR_ALIGN;
    const int64_t N = 2 * N1 * N2;
    const Ws2d w = carve2d(B, H, N, io, false);
    if (!workspace || workspace_bytes < w.total) return LONGCONV_ERR_WORKSPACE;
    if (pads_itself(make_plan(N, io)))
        return fwd_impl(u, k, D, nullptr, y, B, H, N, io, workspace, w.base, stream, false, nullptr, (uint32_t)N2);
    hipStream_t st = (hipStream_t)stream;
    char* ws = (char*)workspace;
    if (note(pad_rows(k, ws + w.kp, (size_t)H * N1, (size_t)N2 * sizeof(float), st), "pad k") != hipSuccess ||
        note(pad_rows(u, ws + w.up, (size_t)B * H * N1, (size_t)N2 * io_bytes(io), st), "pad u") != hipSuccess)
        return LONGCONV_ERR_HIP;
    s = longconv_fwd(ws + w.up, (const float*)(ws + w.kp), D, nullptr, ws + w.yp, B, H, N, io, ws, w.base, stream);
    if (s != LONGCONV_OK) return s;
    if (note(unpad_rows(ws + w.yp, y, (size_t)B * H * N1, (size_t)N2 * io_bytes(io), st), "unpad y") != hipSuccess)
        return LONGCONV_ERR_HIP;
    return LONGCONV_OK;
}

int longconv2d_bwd(const void* dy, const void* u, const float* k, const float* D, void* du, float* dk, float* dD,
                   int64_t B, int64_t H, int64_t N1, int64_t N2, int io, void* workspace, size_t workspace_bytes,
                   void* stream)
{
    int s = check_shape2d(B, H, N1, N2, io);
    if (s != LONGCONV_OK) return s;
    if (!dy || ((dk || dD) && !u) || (du && (!k || !D))) return LONGCONV_ERR_NULL;
    if (misaligned(dy) || misaligned(u) || misaligned(k) || misaligned(du) || misaligned(dk) || misaligned(workspace))
        return LONGCONV_ERR_ALIGN;
    const int64_t N = 2 * N1 * N2;
    const Ws2d w = carve2d(B, H, N, io, true);
    if (!workspace || workspace_bytes < w.total) return LONGCONV_ERR_WORKSPACE;
    if (!du && !dk && !dD) return LONGCONV_OK;
    if (pads_itself(make_plan(N, io)))
        return bwd_impl(dy, u, k, D, nullptr, du, dk, dD, B, H, N, io, workspace, w.base, stream, (uint32_t)N2);
    hipStream_t st = (hipStream_t)stream;
    char* ws = (char*)workspace;
    const size_t rows = (size_t)B * H * N1, rb = (size_t)N2 * io_bytes(io);
    if (note(pad_rows(dy, ws + w.yp, rows, rb, st), "pad dy") != hipSuccess) return LONGCONV_ERR_HIP;
    if ((dk || dD) && note(pad_rows(u, ws + w.up, rows, rb, st), "pad u") != hipSuccess) return LONGCONV_ERR_HIP;
    if (du && note(pad_rows(k, ws + w.kp, (size_t)H * N1, (size_t)N2 * sizeof(float), st), "pad k") != hipSuccess)
        return LONGCONV_ERR_HIP;
    s = longconv_bwd(ws + w.yp, ws + w.up, (const float*)(ws + w.kp), D, nullptr, du ? ws + w.dup : nullptr,
                     dk ? (float*)(ws + w.dkp) : nullptr, dD, B, H, N, io, ws, w.base, stream);
    if (s != LONGCONV_OK) return s;
    // the gradient with respect to the padding columns of the image and of the filter is dropped: they are
    // constants of the construction, not parameters
    if (du && note(unpad_rows(ws + w.dup, du, rows, rb, st), "unpad du") != hipSuccess) return LONGCONV_ERR_HIP;
    if (dk && note(unpad_rows(ws + w.dkp, dk, (size_t)H * N1, (size_t)N2 * sizeof(float), st), "unpad dk") != hipSuccess)
        return LONGCONV_ERR_HIP;
    return LONGCONV_OK;
}

// ---- learned Butterfly extension -----------------------------------------------------------------------------------

static int check_shape_lb(int64_t B, int64_t H, int64_t N, int io)
{
    if (io != LONGCONV_F16 && io != LONGCONV_BF16) return LONGCONV_ERR_DTYPE;
    if (B < 1 || B > (int64_t(1) << 24) || H < 1 || H > 65535) return LONGCONV_ERR_SHAPE;
    if (!pow2(N) || N < 256 || N > 2048) return LONGCONV_ERR_SHAPE;
    return LONGCONV_OK;
}

size_t longconv_lbfly_workspace_bytes(int64_t B, int64_t H, int64_t N, int io)
{
    if (check_shape_lb(B, H, N, io) != LONGCONV_OK) return 0;
    return up256(lbfly_partial_bytes(B, H, N));
}

// the spectrum helpers also serve the block-size study: up to N = 4096
static int check_shape_spectrum(int64_t H, int64_t N)
{
    if (H < 1 || H > 65535 || !pow2(N) || N < 256 || N > 4096) return LONGCONV_ERR_SHAPE;
    return LONGCONV_OK;
}

int longconv_lbfly_spectrum(const float* k, const float* D, float* shat, int64_t H, int64_t N, void* stream)
{
    int s = check_shape_spectrum(H, N);
    if (s != LONGCONV_OK) return s;
    if (!k || !D || !shat) return LONGCONV_ERR_NULL;
    if (misaligned(k) || misaligned(shat)) return LONGCONV_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    Tables tb;
    if (get_tables(&tb, st, false) != hipSuccess) return LONGCONV_ERR_HIP;
    return note(spectrum_natural(k, D, shat, H, N, tb, st), "lbfly spectrum") == hipSuccess ? LONGCONV_OK
                                                                                            : LONGCONV_ERR_HIP;
}

int longconv_lbfly_spectrum_bwd(const float* dshat, float* dk, float* dD, int64_t H, int64_t N, void* stream)
{
    int s = check_shape_spectrum(H, N);
    if (s != LONGCONV_OK) return s;
    if (!dshat) return LONGCONV_ERR_NULL;
    if (misaligned(dshat) || misaligned(dk)) return LONGCONV_ERR_ALIGN;
    if (!dk && !dD) return LONGCONV_OK;
    hipStream_t st = (hipStream_t)stream;
    Tables tb;
    if (get_tables(&tb, st, false) != hipSuccess) return LONGCONV_ERR_HIP;
    return note(spectrum_natural_bwd(dshat, dk, dD, H, N, tb, st), "lbfly spectrum bwd") == hipSuccess
               ? LONGCONV_OK
               : LONGCONV_ERR_HIP;
}

int longconv_lbfly_fwd(const void* u, const float* shat, const float* Af, const float* Ai, void* y, int64_t B,
                       int64_t H, int64_t N, int io, void* stream)
{
    int s = check_shape_lb(B, H, N, io);
    if (s != LONGCONV_OK) return s;
    if (!u || !shat || !Af || !Ai || !y) return LONGCONV_ERR_NULL;
    if (misaligned(u) || misaligned(shat) || misaligned(Af) || misaligned(Ai) || misaligned(y))
        return LONGCONV_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    Tables tb;
    if (get_tables(&tb, st, false) != hipSuccess) return LONGCONV_ERR_HIP;
    return note(lbfly_fwd(u, shat, Af, Ai, y, B, H, N, io, tb, st), "lbfly fwd") == hipSuccess ? LONGCONV_OK
                                                                                                : LONGCONV_ERR_HIP;
}

int longconv_lbfly_bwd(const void* dy, const void* u, const float* shat, const float* Af, const float* Ai, void* du,
                       float* dshat, float* dAf, float* dAi, int64_t B, int64_t H, int64_t N, int io, void* workspace,
                       size_t workspace_bytes, void* stream)
{
    int s = check_shape_lb(B, H, N, io);
    if (s != LONGCONV_OK) return s;
    if (!dy || !u || !shat || !Af || !Ai) return LONGCONV_ERR_NULL;
    if (misaligned(dy) || misaligned(u) || misaligned(shat) || misaligned(Af) || misaligned(Ai) || misaligned(du) ||
        misaligned(dshat) || misaligned(dAf) || misaligned(dAi) || misaligned(workspace))
        return LONGCONV_ERR_ALIGN;
    if (!workspace || workspace_bytes < up256(lbfly_partial_bytes(B, H, N))) return LONGCONV_ERR_WORKSPACE;
    if (!du && !dshat && !dAf && !dAi) return LONGCONV_OK;
    hipStream_t st = (hipStream_t)stream;
    Tables tb;
    if (get_tables(&tb, st, false) != hipSuccess) return LONGCONV_ERR_HIP;
    return note(lbfly_bwd(dy, u, shat, Af, Ai, du, dshat, dAf, dAi, workspace, B, H, N, io, tb, st), "lbfly bwd") ==
                   hipSuccess
               ? LONGCONV_OK
               : LONGCONV_ERR_HIP;
}

// ---- block-size study ------------------------------------------------------------------------------------------------

int longconv_blocksize_fwd(const void* u, const float* shat, void* y, int64_t B, int64_t H, int64_t N, int io, int log2r,
                           void* stream)
{
    if (io != LONGCONV_F16) return LONGCONV_ERR_DTYPE;
    if (B < 1 || B > (int64_t(1) << 24) || H < 1 || H > 65535 || (N != 1024 && N != 4096) || log2r < 1 ||
        (log2r > 6 && !(log2r == 8 && N == 4096)))
        return LONGCONV_ERR_SHAPE;
    if (!u || !shat || !y) return LONGCONV_ERR_NULL;
    if (misaligned(u) || misaligned(shat) || misaligned(y)) return LONGCONV_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    Tables tb;
    if (get_tables(&tb, st, false) != hipSuccess) return LONGCONV_ERR_HIP;
    return note(blocksize_fwd(u, shat, y, B, H, N, log2r, tb, st), "blocksize fwd") == hipSuccess ? LONGCONV_OK
                                                                                                   : LONGCONV_ERR_HIP;
}

static int kreg_check(const float* k, const void* a, const void* b, int64_t H, int64_t N, int p, float lambda)
{
    int s = check_shape(1, H, N, LONGCONV_F32);
    if (s != LONGCONV_OK) return s;
    if (!k || !a || !b) return LONGCONV_ERR_NULL;
    if (p < 0 || p > KREG_MAX_P || !(lambda >= 0.f) || !(lambda < 3.0e38f)) return LONGCONV_ERR_SHAPE;
    return LONGCONV_OK;
}

int longconv_kreg_fwd(const float* k, const float* drop_mask, float* kbar, int64_t H, int64_t N, int p, float lambda,
                      void* stream)
{
    int s = kreg_check(k, kbar, kbar, H, N, p, lambda);
    if (s != LONGCONV_OK) return s;
    if (note(kreg_fwd(k, drop_mask, kbar, H, N, p, lambda, (hipStream_t)stream), "kreg fwd") != hipSuccess)
        return LONGCONV_ERR_HIP;
    return LONGCONV_OK;
}

int longconv_kreg_bwd(const float* k, const float* drop_mask, const float* dkbar, float* dk, int64_t H, int64_t N,
                      int p, float lambda, void* stream)
{
    int s = kreg_check(k, dkbar, dk, H, N, p, lambda);
    if (s != LONGCONV_OK) return s;
    if (note(kreg_bwd(k, drop_mask, dkbar, dk, H, N, p, lambda, (hipStream_t)stream), "kreg bwd") != hipSuccess)
        return LONGCONV_ERR_HIP;
    return LONGCONV_OK;
}

int longconv_set_option(const char* name, int value)
{
    if (!name) return LONGCONV_ERR_NULL;
    options();                                   // the environment is read first, once
    if (!strcmp(name, "engine")) { if (value < 0 || value > 2) return LONGCONV_ERR_SHAPE; g_opt.engine = value; }
    else if (!strcmp(name, "inner_log2")) { if (value < 0 || value > 31) return LONGCONV_ERR_SHAPE; g_opt.inner_log2 = value; }
    else if (!strcmp(name, "staged_kernel")) g_opt.staged = value != 0;
    else if (!strcmp(name, "fuse_pass_a")) g_opt.fuse_pass_a = value != 0;
    else if (!strcmp(name, "fuse_bwd")) g_opt.fuse_bwd = value != 0;
    else return LONGCONV_ERR_SHAPE;
    return LONGCONV_OK;
}

const char* longconv_status_string(int status)
{
    switch (status) {
        case LONGCONV_OK: return "ok";
        case LONGCONV_ERR_NULL: return "a required pointer is NULL";
        case LONGCONV_ERR_SHAPE: return "bad shape: need B,H >= 1 and N a power of two in [256, 131072]";
        case LONGCONV_ERR_DTYPE: return "unsupported dtype";
        case LONGCONV_ERR_ALIGN: return "pointer not 16-byte aligned";
        case LONGCONV_ERR_WORKSPACE: return "workspace missing or too small";
        case LONGCONV_ERR_HIP: return "HIP call failed";
        default: return "unknown status";
    }
}

const char* longconv_last_hip_error(void) { return t_hip_err; }

const char* longconv_plan_string(int64_t N, int io)
{
    static thread_local char buf[256];
    if (check_shape(1, 1, N, io) != LONGCONV_OK) { snprintf(buf, sizeof(buf), "invalid"); return buf; }
    const Plan pl = make_plan(N, io);
    const bool mfma = pl.engine == ENGINE_MFMA, wave = mfma && pl.order.wave_lg, lng = mfma && pl.order.long_lg;
    const bool chunks = mfma && chunk_plan(pl);
    // what the convolutions transform: N twisted points of each row, or 2N zero-padded points of a row pair; rows above 32768
    // samples in chunks of 16384 points
    const bool rows = wave || lng || chunks || (mfma && pl.row1) || pl.vrow;
    const int lgL = pl.log2L - rows, lgL2 = chunks ? lgL - pl.log2R : rows ? lgL : pl.log2L2, lgR = lgL - lgL2;
    int bits[20], nd = 0;
    if (lgR) bits[nd++] = lgR;
    if (wave || lng || chunks) {
        for (int left = lgL2; left > 0; left -= 4) bits[nd++] = left < 4 ? left : 4;
    } else {
        for (int i = pl.log2R != 0; i < pl.order.ndig; ++i) bits[nd++] = pl.order.bits[i];
    }
    int n = snprintf(buf, sizeof(buf), "engine=%s L=2^%d of %s outer_radix=%d inner=2^%d passes=%d digits=",
                     mfma ? "mfma-fp16" : "valu-fp32", lgL, rows ? "rows" : "pairs", 1 << lgR, lgL2, lgR ? 3 : 1);
    for (int i = 0; i < nd; ++i) n += snprintf(buf + n, sizeof(buf) - n, "%s%d", i ? "x" : "", 1 << bits[i]);
    if (wave) n += snprintf(buf + n, sizeof(buf) - n, " kernel=wave");
    if (mfma && !wave && (lng || pl.order.coop_lg)) n += snprintf(buf + n, sizeof(buf) - n, " kernel=chained");
    if (!mfma || pl.fuse_bwd || (chunks && options().fuse_bwd)) snprintf(buf + n, sizeof(buf) - n, " backward=one");
    else if (mfma && chunk_dk_plan(pl)) snprintf(buf + n, sizeof(buf) - n, " backward=dk(rows,%dx2^14),du", 1 << pl.log2R);
    else snprintf(buf + n, sizeof(buf) - n, " backward=dk,du");
    return buf;
}

}  // extern "C"
