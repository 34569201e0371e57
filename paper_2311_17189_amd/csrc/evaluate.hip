// Runtime side of the evaluators: table upload, launch shapes, kernel
// dispatch, deterministic reductions, and the evaluate entry points of the C
// ABI (include/amigpu.h).
//
// The evaluation (Burke & LeBlanc, arXiv 2311.17189, Sec. 2.3) maps one lane
// to one energy sample; the kernels are in kernels_packed.hpp (bit-mask tables,
// specialized per self-energy shape, forward and adjoint) and kernel_generic.hpp
// (double tables, forward only, any coefficients).  Sums over samples (the
// Monte-Carlo row sums of Sec. 2.3 and the reductions of the adjoint) are done
// per block with a fixed shuffle tree and then across blocks in a fixed order,
// so repeated calls are bitwise identical.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "ami_internal.hpp"
#include "device_common.hpp"
#include "kernel_generic.hpp"
#include "jit.hpp"
#include "kernels_packed.hpp"
#include "runtime.hpp"

namespace ami {

AmiStatus hip_fail(hipError_t e, const char *what) {
    return fail(AMI_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

namespace {

// out[j] = sum over rows of column j.  One block per column.
__global__ __launch_bounds__(kRedThreads) void ami_colsum_kernel(const double *partial, int64_t rows, int64_t rs,
                                                                 int64_t cs, double *out) {
    __shared__ double sh[kRedThreads / 64];
    const double r = column_sum(partial + blockIdx.x * cs, rows, rs, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = r;
}

// Same reduction for the adjoint partials, routing each column to its output:
// column 0 dL/dbeta, 1 dL/dmu, 2 dL/dt, 4.. dL/dw (complex [n_f][n_ext]).
// Blocks past the gradient columns reduce the forward values' row sums
// (partial sums of nval columns stored after the ncols gradient ones, in the
// same layout: column-major when colmajor, else row-major).
__global__ __launch_bounds__(kRedThreads) void ami_adj_finalize_kernel(const double *partial, int64_t rows, int ncols,
                                                                       int colmajor, double *gbeta, double *gmu,
                                                                       double *gt, double *gw, int nval,
                                                                       double *vsum) {
    __shared__ double sh[kRedThreads / 64];
    int j = blockIdx.x;
    double *dst = nullptr;
    const double *src = partial;
    int64_t width = ncols;
    if (j == 0) dst = gbeta;
    else if (j == 1) dst = gmu;
    else if (j == 2) dst = gt;
    else if (j >= kAdjScalars && j < ncols && gw) dst = gw + (j - kAdjScalars);
    else if (j >= ncols && vsum) {
        j -= ncols;
        dst = vsum + j;
        src = partial + rows * ncols;
        width = nval;
    }
    if (!dst) return;
    const double r = colmajor ? column_sum(src + j * rows, rows, 1, sh) : column_sum(src + j, rows, width, sh);
    if (threadIdx.x == 0) *dst = r;
}

__global__ void ami_fill_kernel(double *p, int64_t n, double v) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

}  // namespace

AmiStatus fill(double *p, int64_t n, hipStream_t stream) {
    if (!p || n <= 0) return AMI_OK;
    hipLaunchKernelGGL(ami_fill_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream, p, n,
                       0.0);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? AMI_OK : hip_fail(e, "fill launch");
}

// Upload (once per device) every table of a handle in one allocation.
AmiStatus upload(AmiTerms *t, DeviceTables **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> lk(t->dev_mu);
    for (auto &d : t->dev)
        if (d.device == dev) {
            *out = &d;
            return AMI_OK;
        }
    const Tables &tb = t->tab;
    struct Piece {
        const void *src;
        size_t bytes;
        size_t off;
    };
    Piece pieces[13] = {
        {tb.leaf_coef.data(), tb.leaf_coef.size() * sizeof(double), 0},
        {tb.leaf_sigma.data(), tb.leaf_sigma.size() * sizeof(double), 0},
        {tb.den_coef.data(), tb.den_coef.size() * sizeof(double), 0},
        {tb.group_dens.data(), tb.group_dens.size() * sizeof(int32_t), 0},
        {tb.group_start.data(), tb.group_start.size() * sizeof(int32_t), 0},
        {tb.term_sign.data(), tb.term_sign.size() * sizeof(double), 0},
        {tb.term_leaf.data(), tb.term_leaf.size() * sizeof(int32_t), 0},
        {tb.line_alpha.data(), tb.line_alpha.size() * sizeof(double), 0},
        {tb.p_leaf.data(), tb.p_leaf.size() * sizeof(uint64_t), 0},
        {tb.p_den.data(), tb.p_den.size() * sizeof(uint64_t), 0},
        {tb.p_line.data(), tb.p_line.size() * sizeof(uint32_t), 0},
        {tb.p_term.data(), tb.p_term.size() * sizeof(uint64_t), 0},
        {tb.p_group.data(), tb.p_group.size() * sizeof(uint64_t), 0},
    };
    size_t total = 0;
    for (auto &pc : pieces) {
        pc.off = total;
        total += align256(std::max<size_t>(pc.bytes, 8));
    }
    std::vector<unsigned char> host(total, 0);
    for (auto &pc : pieces)
        if (pc.bytes) std::memcpy(host.data() + pc.off, pc.src, pc.bytes);
    void *blob = nullptr;
    e = hipMalloc(&blob, total);
    if (e != hipSuccess) return fail(AMI_E_OOM, std::string("hipMalloc of tables: ") + hipGetErrorString(e));
    e = hipMemcpy(blob, host.data(), total, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(blob);
        return hip_fail(e, "hipMemcpy of tables");
    }
    DeviceTables d;
    d.device = dev;
    d.blob = blob;
    auto at = [&](int i) { return static_cast<unsigned char *>(blob) + pieces[i].off; };
    d.leaf_coef = reinterpret_cast<const double *>(at(0));
    d.leaf_sigma = reinterpret_cast<const double *>(at(1));
    d.den_coef = reinterpret_cast<const double *>(at(2));
    d.group_dens = reinterpret_cast<const int32_t *>(at(3));
    d.group_start = reinterpret_cast<const int32_t *>(at(4));
    d.term_sign = reinterpret_cast<const double *>(at(5));
    d.term_leaf = reinterpret_cast<const int32_t *>(at(6));
    d.line_alpha = reinterpret_cast<const double *>(at(7));
    d.p_leaf = reinterpret_cast<const uint64_t *>(at(8));
    d.p_den = reinterpret_cast<const uint64_t *>(at(9));
    d.p_line = reinterpret_cast<const uint32_t *>(at(10));
    d.p_term = reinterpret_cast<const uint64_t *>(at(11));
    d.p_group = reinterpret_cast<const uint64_t *>(at(12));
    t->dev.push_back(d);
    *out = &t->dev.back();
    return AMI_OK;
}

AmiStatus pick_shape(int slots, LaunchShape &ls) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    int max_lds = 0;
    e = hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
    ls.slots = slots;
    const size_t per_lane = static_cast<size_t>(slots) * sizeof(double);
    // 256 lanes while a block stays within a quarter of the CU's LDS, else fewer
    const int blocks[3] = {256, 128, 64};
    for (int b : blocks) {
        const size_t lds = per_lane * b + 2 * sizeof(double) * (b / 64);
        if (lds <= static_cast<size_t>(max_lds) && (lds <= 40 * 1024 || b == 64)) {
            ls.block = b;
            ls.lds = lds;
            return AMI_OK;
        }
    }
    return fail(AMI_E_UNSUPPORTED, "solution too large for the LDS-resident evaluator (" +
                                       std::to_string(per_lane) + " B per sample)");
}

PackedTabs packed_tabs(const AmiTerms *t, const DeviceTables *dt) {
    const Tables &tb = t->tab;
    PackedTabs p;
    p.leaf = dt->p_leaf;
    p.den = dt->p_den;
    p.line = dt->p_line;
    p.term = dt->p_term;
    p.term_sign = dt->term_sign;
    p.group_start = dt->group_start;
    p.group = dt->p_group;
    p.L = tb.L;
    p.D = tb.D;
    p.G = tb.G;
    p.T = tb.T;
    p.n_eps = t->n_eps;
    p.n_int = t->n_int;
    p.n_ext = t->n_ext;
    p.n_freq = t->n_freq;
    p.n_g = t->n_g;
    p.dpt = tb.dpt;
    p.fermi_used = tb.fermi_used;
    p.use_products = tb.use_products ? 1 : 0;
    return p;
}

namespace {

template <bool ADJ, int NE, int NI, int DPT, bool EXACT, bool HUB>
void launch_packed_one(dim3 grid, dim3 block, size_t lds, hipStream_t stream, const KArgs &a) {
    if constexpr (ADJ)
        hipLaunchKernelGGL((ami_adj_packed<NE, NI, DPT, EXACT, HUB>), grid, block, lds, stream, a);
    else
        hipLaunchKernelGGL((ami_fwd_packed<NE, NI, DPT, EXACT, HUB>), grid, block, lds, stream, a);
}

// Self-energy shapes (order n: 2n-1 energies, n leaves and n-1 denominators
// per term) get exact instances; anything else the bounded generic one.
template <bool ADJ, bool HUB>
const char *launch_packed(const AmiTerms *t, dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                          const KArgs &a) {
    const int ne = t->n_eps, ni = t->n_int, dpt = t->tab.dpt;
    const bool se = (ne == 2 * ni - 1) && (dpt == ni - 1) && (!HUB || t->n_g == ne);
#define AMI_SE(N)                                                                                 \
    if (se && ni == N) {                                                                          \
        launch_packed_one<ADJ, 2 * N - 1, N, N - 1, true, HUB>(grid, block, lds, stream, a);      \
        return "self-energy order " #N;                                                           \
    }
    AMI_SE(1)
    AMI_SE(2)
    AMI_SE(3)
    AMI_SE(4)
    AMI_SE(5)
    AMI_SE(6)
    AMI_SE(7)
#undef AMI_SE
    launch_packed_one<ADJ, 16, 8, 8, false, HUB>(grid, block, lds, stream, a);
    return "bounded generic";
}

}  // namespace

int fwd_slots(const Tables &tb) { return std::max(tb.L, 2 * tb.D) + tb.G; }

namespace {
int adj_slots(const Tables &tb) { return tb.L + 2 * tb.G + std::max(2 * tb.D, tb.L); }

AmiStatus launch_generic_forward(AmiTerms *t, DeviceTables *dt, bool hub, const KArgs &ka, double *partial,
                                 const LaunchShape &ls, dim3 grid, hipStream_t stream) {
    const Tables &tb = t->tab;
    FwdParams p;
    std::memset(&p, 0, sizeof(p));
    p.leaf_coef = dt->leaf_coef;
    p.leaf_sigma = dt->leaf_sigma;
    p.den_coef = dt->den_coef;
    p.group_dens = dt->group_dens;
    p.group_start = dt->group_start;
    p.term_sign = dt->term_sign;
    p.term_leaf = dt->term_leaf;
    p.line_alpha = dt->line_alpha;
    p.n_eps = t->n_eps;
    p.n_ext = t->n_ext;
    p.n_int = t->n_int;
    p.n_g = t->n_g;
    p.n_freq = t->n_freq;
    p.L = tb.L;
    p.D = tb.D;
    p.G = tb.G;
    p.dpt = tb.dpt;
    p.region_a = std::max(tb.L, 2 * tb.D);
    p.energies = ka.energies;
    p.stride_s = ka.stride_s;
    p.stride_i = ka.stride_i;
    p.k = ka.k;
    p.stride_k = ka.stride_k;
    for (int x = 0; x < 2 * kMaxExt; ++x) p.q[x] = ka.q[x];
    p.hop_t = ka.hop_t;
    p.mu = ka.mu;
    p.ext_freqs = ka.ext_freqs;
    p.n_f = ka.n_f;
    p.beta = ka.beta;
    p.e_reg = ka.e_reg;
    p.n_e = ka.n_e;
    p.out = ka.out;
    p.partial = partial;
    const int maxe = t->n_eps <= 4 ? 4 : (t->n_eps <= 8 ? 8 : 16);
    const dim3 block(ls.block);
#define AMI_LAUNCH(ME, H) hipLaunchKernelGGL((ami_fwd_kernel<ME, H>), grid, block, ls.lds, stream, p)
    if (hub) {
        if (maxe == 4) AMI_LAUNCH(4, true);
        else if (maxe == 8) AMI_LAUNCH(8, true);
        else AMI_LAUNCH(16, true);
    } else {
        if (maxe == 4) AMI_LAUNCH(4, false);
        else if (maxe == 8) AMI_LAUNCH(8, false);
        else AMI_LAUNCH(16, false);
    }
#undef AMI_LAUNCH
    return AMI_OK;
}

thread_local std::string g_last_variant;

// Optional HIP-event timing of the main evaluation kernel of each call on
// this thread (amiKernelTimerStart / amiKernelTimerStop).  The specialized
// kernels carry the events on their own dispatch (hipExtModuleLaunchKernel),
// so the pair brackets the kernel alone; the table-driven ones are bracketed
// by events recorded on the stream around the launch.
struct KernelTimer {
    bool on = false;
    std::vector<hipEvent_t> ev;      // start/stop pairs
    int used = 0;
};
thread_local KernelTimer g_timer;

void timer_mark(hipStream_t stream, bool stop) {
    if (!g_timer.on || g_timer.used >= static_cast<int>(g_timer.ev.size()) / 2) return;
    (void)hipEventRecord(g_timer.ev[2 * g_timer.used + (stop ? 1 : 0)], stream);
    if (stop) ++g_timer.used;
}

// The next start/stop pair for a dispatch, or false when the timer is off or full.
bool timer_pair(hipEvent_t &start, hipEvent_t &stop) {
    if (!g_timer.on || g_timer.used >= static_cast<int>(g_timer.ev.size()) / 2) return false;
    start = g_timer.ev[2 * g_timer.used];
    stop = g_timer.ev[2 * g_timer.used + 1];
    ++g_timer.used;
    return true;
}

enum class Path { TABLES, PACKED, SPECIALIZED, TWO_PASS, ADJ_PASSES, ADJ_BLOCK, FWD_BLOCK };

// Workspace of one chunk of the two-pass forward and of the adjoint in passes
// (group sums, energies and their cotangents): 1 GiB unless
// amiSetTwoPassChunkBytes set another bound (a chunk never exceeds what the
// call's samples need).
std::atomic<int64_t> g_two_pass_chunk_bytes{int64_t(1) << 30};
// Frequency rows of one two-pass launch (its second kernel runs a block per
// tile and frequency row; the bound keeps that grid below 2^31 blocks).
constexpr int kTwoPassMaxFreqs = 65535;

// Which kernels serve a call (AMI_VARIANT_* of the handle); for the
// specialized path also loads them.  AUTO falls back and records why.
// With no_load the specialized kernels must already be loaded on the device
// (jit_loaded): nothing is compiled, loaded or allocated, and a kernel that
// the call would use but that is not loaded yet is an error, not a fallback.
// The forward of a solution too large for one pass takes the block kernel under
// AUTO (Path::FWD_BLOCK), else two kernels over a workspace (Path::TWO_PASS).
// The adjoint of a large solution takes the block kernel under AUTO where the
// solution splits over the waves of a block (Path::ADJ_BLOCK), else three
// kernels over a workspace (Path::ADJ_PASSES): jit_fn (sums pass), jit_fn2
// (frequency pass), jit_fn3 (leaf pass).
AmiStatus choose_path(AmiTerms *t, bool hub, bool adjoint, Path &p, void **jit_fn, std::string &note,
                      void **jit_fn2 = nullptr, int n_f = 1, int variant = -1, bool no_load = false,
                      void **jit_fn3 = nullptr) {
    const int v = variant >= 0 ? variant : t->variant;
    note.clear();
    auto get = [&](int kind, void **fn) {
        return no_load ? jit_loaded(t, hub, kind, fn) : jit_get(t, hub, kind, fn);
    };
    // the forward of a large solution: two passes (AUTO and SPECIALIZED when the
    // one-pass kernel would not fit its registers; TWO_PASS always)
    const bool two = !adjoint && jit_fn2 && n_f <= kTwoPassMaxFreqs &&
                     (v == AMI_VARIANT_TWO_PASS ||
                      ((v == AMI_VARIANT_AUTO || v == AMI_VARIANT_SPECIALIZED) && jit_prefers_two_pass(t)));
    const bool passes = adjoint && jit_fn2 && jit_fn3 &&
                        (v == AMI_VARIANT_TWO_PASS || (v == AMI_VARIANT_AUTO && t->tab.T > kJitAutoAdjointTerms));
    if (v == AMI_VARIANT_TWO_PASS && !two && !passes)
        return fail(AMI_E_UNSUPPORTED, adjoint ? "the two-pass variant of the adjoint runs in passes only"
                                               : "the two-pass variant takes at most 65535 frequency rows");
    if (adjoint && jit_fn3 && v == AMI_VARIANT_AUTO && jit_prefers_block_adjoint(t) &&
        jit_block_waves(t, hub) > 0) {
        // one row's kernel and several rows' are ready together
        AmiStatus st = get(kJitBlockAdjoint, jit_fn);
        if (st == AMI_OK && jit_block_rows_apart(t)) {
            void *rows = nullptr;
            st = get(kJitBlockAdjointRows, &rows);
            if (n_f > 1) *jit_fn = rows;
        }
        if (st == AMI_OK) {
            p = Path::ADJ_BLOCK;
            return AMI_OK;
        }
        if (no_load && st != AMI_E_UNSUPPORTED) return st;
        note = std::string(" (not in a block: ") + amiLastError() + ")";
        clear_error();
    }
    if (passes) {
        std::string why;
        AmiStatus st = AMI_OK;
        if (!jit_adjoint_passes_supported(t, hub, &why)) st = fail(AMI_E_UNSUPPORTED, "no adjoint in passes: " + why);
        if (st == AMI_OK) st = get(kJitSumsPass, jit_fn);
        if (st == AMI_OK) st = get(kJitAdjFreq, jit_fn2);
        if (st == AMI_OK) st = get(kJitAdjLeaf, jit_fn3);
        if (st == AMI_OK) {
            p = Path::ADJ_PASSES;
            return AMI_OK;
        }
        if (v != AMI_VARIANT_AUTO || (no_load && st != AMI_E_UNSUPPORTED)) return st;
        note = std::string(" (not in passes: ") + amiLastError() + ")";
        clear_error();
    }
    if (two && v == AMI_VARIANT_AUTO && jit_block_forward_waves(t) > 0) {
        const AmiStatus st = get(kJitBlockForward, jit_fn);
        if (st == AMI_OK) {
            p = Path::FWD_BLOCK;
            return AMI_OK;
        }
        note = std::string(" (not in a block: ") + amiLastError() + ")";
        clear_error();
    }
    if (two) {
        AmiStatus st = get(kJitSumsPass, jit_fn);
        if (st == AMI_OK) st = get(kJitFreqPass, jit_fn2);
        if (st == AMI_OK) {
            p = Path::TWO_PASS;
            return AMI_OK;
        }
        if (v != AMI_VARIANT_AUTO || (no_load && st != AMI_E_UNSUPPORTED)) return st;
        note = std::string(" (not two-pass: ") + amiLastError() + ")";
        clear_error();
    }
    const bool auto_skip = v == AMI_VARIANT_AUTO && adjoint && t->tab.T > kJitAutoAdjointTerms;
    if (auto_skip && note.empty())
        note = " (adjoint specialized in one pass up to " + std::to_string(kJitAutoAdjointTerms) + " terms)";
    if (v == AMI_VARIANT_SPECIALIZED || (v == AMI_VARIANT_AUTO && !auto_skip && !two)) {
        const AmiStatus st = get(adjoint ? kJitAdjoint : kJitForward, jit_fn);
        if (st == AMI_OK) {
            p = Path::SPECIALIZED;
            return AMI_OK;
        }
        if (v == AMI_VARIANT_SPECIALIZED || (no_load && st != AMI_E_UNSUPPORTED)) return st;
        note = std::string(" (not specialized: ") + amiLastError() + ")";
        clear_error();
    }
    if (!t->tab.uniform)
        return fail(AMI_E_UNSUPPORTED, "poles of higher order are evaluated by the specialized kernels only" + note);
    if (v == AMI_VARIANT_TABLES) {
        if (adjoint) return fail(AMI_E_UNSUPPORTED, "the double-table variant has no adjoint");
        p = Path::TABLES;
        return AMI_OK;
    }
    if (t->tab.packable) {
        p = Path::PACKED;
        return AMI_OK;
    }
    if (v == AMI_VARIANT_PACKED || adjoint)
        return fail(AMI_E_UNSUPPORTED,
                    "the packed kernels need +-1 coefficients and at most 255 leaves/denominators" + note);
    p = Path::TABLES;
    return AMI_OK;
}

// Partial-sum workspace of (handle, device, stream), at least `bytes` long:
// steady-state calls allocate nothing (and can be captured in a graph once a
// first call on the stream has sized it).
AmiStatus workspace(AmiTerms *t, DeviceTables *dt, hipStream_t stream, size_t bytes, double **out) {
    std::lock_guard<std::mutex> lk(t->dev_mu);
    DeviceTables::Workspace *w = nullptr;
    for (auto &x : dt->ws)
        if (x.stream == static_cast<void *>(stream)) w = &x;
    if (!w) {
        dt->ws.emplace_back();
        w = &dt->ws.back();
        w->stream = static_cast<void *>(stream);
    }
    if (w->bytes < bytes) {
        const size_t want = align256(std::max(bytes, 2 * w->bytes));
        void *p = nullptr;
        const hipError_t e = hipMalloc(&p, want + (w->ptr ? 0 : 256));   // the first holds the ticket
        if (e != hipSuccess) return fail(AMI_E_OOM, std::string("workspace: ") + hipGetErrorString(e));
        if (!w->ptr) w->ticket = reinterpret_cast<unsigned *>(static_cast<char *>(p) + want);
        if (w->ptr) dt->retired.push_back(w->ptr);     // a launch already queued may still read it
        w->ptr = p;
        w->bytes = want;
    }
    *out = static_cast<double *>(w->ptr);
    return AMI_OK;
}

// Whether a capture of the stream is under way (or that is not known).
bool capturing(hipStream_t stream) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return cap != hipStreamCaptureStatusNone;
}

// Where the totals of a call's partial sums go (finish_small): a's gradient
// columns, then the row sums of the values.
struct AdjOut {
    double *grad_beta = nullptr, *grad_mu = nullptr, *grad_t = nullptr, *grad_freqs = nullptr;
    double *out_sum = nullptr;   // forward row sums computed on the way (optional)
};

// Has the kernel's last block add the partial sums (a.nrows rows of ncols columns
// of gradients and nval of values) instead of a second launch, where that is
// cheaper: the launch takes 3 us of the host, the last block's work some 30 ns
// of the GPU per block (each releases its rows) and 1 us per 16 loads of 64 rows
// by a wave.  The limits keep that below the launch it replaces, so that a caller
// who waits for every call loses nothing either; a kernel whose blocks run long
// takes fewer.  At most 1024 rows, the reduction kernel's one pass.  Per call,
// with two launches and with one: forwards of momenta 14.4 and 11.3 us, adjoints
// 21.5 and 18.5 (waited for: 23.7 and 23.7, 31.5 and 31); past the limits, waited
// for: 32 and 35 (order 2 adjoint, 130 blocks), and 22 and 28 (2804 terms, 3 rows,
// 500 blocks).
// Needs the stream's workspace (call workspace() first).  Not under capture,
// whose replays may run on other streams beside this one's calls, nor on the
// per-thread default stream, one handle of many streams: both would share the
// counter.
struct FinishLimits {
    int64_t blocks, loads;
};
constexpr FinishLimits kFinishOnePass{64, 16}, kFinishBlockForward{64, 16}, kFinishBlockAdjoint{32, 4};
constexpr FinishLimits kFinishComplex{32, 8}, kFinishComplexAdjoint{32, 4};
bool finish_small(AmiTerms *t, DeviceTables *dt, hipStream_t stream, KArgs &a, const FinishLimits &lim, int64_t blocks,
                  int waves, int ncols, int nval, const AdjOut &o) {
    const int64_t chunks = (a.nrows + 63) / 64;
    if (chunks > 16 || blocks > lim.blocks || (ncols + nval + waves - 1) / waves * chunks > lim.loads) return false;
    if (stream == hipStreamPerThread) return false;
    if (capturing(stream)) return false;
    {
        std::lock_guard<std::mutex> lk(t->dev_mu);
        DeviceTables::Workspace *w = nullptr;
        for (auto &x : dt->ws)
            if (x.stream == static_cast<void *>(stream)) w = &x;
        if (!w || !w->ticket) return false;
        if (!w->counting) {
            if (fill(reinterpret_cast<double *>(w->ticket), 32, stream) != AMI_OK) {
                clear_error();
                return false;
            }
            w->counting = true;
        }
        a.fin_ticket = w->ticket;
    }
    a.fin_cols = ncols + nval;
    a.fin_grad = ncols;
    a.fin_beta = o.grad_beta;
    a.fin_mu = o.grad_mu;
    a.fin_t = o.grad_t;
    a.fin_w = o.grad_freqs;
    a.fin_sum = o.out_sum;
    return true;
}

// Launch of a specialized kernel on a grid of nblocks x gy blocks (timed by
// the kernel timer when it runs).
hipError_t launch_jit(void *fn, int64_t nblocks, int block, hipStream_t stream, KArgs &a, int gy = 1) {
    void *params[] = {&a};
    const hipFunction_t f = static_cast<hipFunction_t>(fn);
    hipEvent_t t0 = nullptr, t1 = nullptr;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (g_timer.on) (void)hipStreamIsCapturing(stream, &cap);   // no timer events inside a capture
    if (nblocks * block <= 0xffffffffLL && cap == hipStreamCaptureStatusNone && timer_pair(t0, t1))
        return hipExtModuleLaunchKernel(f, static_cast<uint32_t>(nblocks * block), static_cast<uint32_t>(gy), 1,
                                        static_cast<uint32_t>(block), 1, 1, 0, stream, params, nullptr, t0, t1, 0);
    return hipModuleLaunchKernel(f, static_cast<unsigned>(nblocks), static_cast<unsigned>(gy), 1,
                                 static_cast<unsigned>(block), 1, 1, 0, stream, params, nullptr);
}

// Launches of a block kernel (`waves` waves share 64 samples) over all `tiles`:
// more than one where its threads, up to eight per sample, pass the 2^32 of a
// grid.
hipError_t launch_block(void *fn, int64_t tiles, int waves, hipStream_t stream, KArgs &a, int gy = 1) {
    const int64_t most = 0xffffffffLL / (64 * waves);
    hipError_t e = hipSuccess;
    for (int64_t t0 = 0; t0 < tiles && e == hipSuccess; t0 += most) {
        a.s0 = 64 * t0;
        e = launch_jit(fn, std::min(most, tiles - t0), 64 * waves, stream, a, gy);
    }
    return e;
}

// Rows of a part where n_f rows are split in `parts`: an even number of them
// (AMI_JIT_ROW_PART); and the parts of those that hold a row.
int64_t rows_per_part(int64_t n_f, int64_t parts) {
    return parts <= 1 ? n_f : ((n_f + parts - 1) / parts + 1) & ~int64_t(1);
}

int nonempty_parts(int64_t n_f, int64_t parts) {
    const int64_t per = std::max<int64_t>(rows_per_part(n_f, parts), 1);
    return parts <= 1 ? 1 : static_cast<int>((n_f + per - 1) / per);
}

// Parts of the frequency rows of a one-pass forward, each a grid of its own over
// the samples that forms the leaves and group sums again: the number whose waves
// finish first.  A SIMD's time is its waves' instructions (estimated from the
// sizes), 1.3 times that for a wave alone, 1.1 for two at a time, 1.03 for three;
// the waves the registers do not hold side by side follow as others end.  (From the
// times of six diagrams at 3000 to 10^6 samples, 4 to 256 rows and one to 32 parts,
// real and complex: what this picks takes 1% more than the best on average.  Two
// waves per SIMD taken for free, as before, took 4 to 8% more, and lost where a row
// is cheap beside the leaves: 5 10^4 samples, four rows, 264 terms 9.4 us in one
// part and 11.5 in two, at complex energies 14.3 and 20.4.  The gains: order 4, 52
// terms, 256 rows of 10^5 samples 140 us in one part, 117 in five, of 10^4 samples
// 96 and 21.)
int forward_row_parts(const AmiTerms *t, bool hub, bool cplx, int64_t n_waves, int64_t n_f) {
    if (n_f < 4) return 1;
    const Tables &tb = t->tab;
    const double once = cplx ? 85.0 * tb.L + 4.0 * tb.T + 2.0 * tb.D : 30.0 * tb.L + tb.T + (hub ? 34.0 * t->n_g : 0.0);
    const double per_row = (cplx ? 22.0 * tb.D + 16.0 * tb.G : 18.0 * tb.D + 12.0 * tb.G) + 40.0;
    const double vgprs = cplx ? 1.5 * (4.0 * tb.G + 6.0 * tb.D) : 2.2 * (2.0 * tb.G + 4.0 * tb.D);
    const int64_t side_by_side = std::max(1, std::min(8, static_cast<int>(512.0 / std::max(vgprs, 40.0))));
    auto rate = [](int64_t waves) {
        return waves <= 1 ? 1.3 : waves == 2 ? 1.1 : waves == 3 ? 1.03 : waves <= 5 ? 1.015 : 1.0;
    };
    auto time = [&](int64_t parts) {
        const int64_t waves = (std::max<int64_t>(n_waves, 1) * parts + 1023) / 1024;      // of a SIMD
        const int64_t full = waves / side_by_side, rest = waves % side_by_side;
        const double issue = static_cast<double>(full * side_by_side) * rate(side_by_side) +
                             static_cast<double>(rest) * (full ? 1.0 : rate(rest));
        return issue * (once + per_row * static_cast<double>(rows_per_part(n_f, parts)));
    };
    // the fewest parts within 2% of the least time, one within 3%
    const int64_t most = std::min<int64_t>(n_f / 2, 1024);
    auto next = [](int64_t p) { return p + (p < 16 ? 1 : p & (p - 1) ? p / 3 : p / 2); };
    double least = 0.97 * time(1);
    bool split = false;
    for (int64_t p = 2; p <= most; p = next(p)) {
        const double v = time(p);
        if (v >= least) continue;
        least = v;
        split = true;
    }
    if (!split) return 1;
    int64_t p = 2;
    while (time(p) > 1.02 * least) p = next(p);
    return nonempty_parts(n_f, p);
}

// Row parts of the block forward: as many as fill the chip's 512 resident blocks
// of four waves (256 of eight), a row per wave at least.  Beyond that the leaves
// and sums formed again cost more than they hide.  560 terms, 256 rows of 4000
// samples: 40 us in two passes, 29 here; 2804 terms, 200 samples: 41 and 15.
int block_row_parts(int waves, int64_t tiles, int64_t n_f) {
    const int64_t fill = (2048 / waves) / std::max<int64_t>(tiles, 1);
    return nonempty_parts(n_f, std::min<int64_t>(fill, n_f / waves));
}

// The two-pass forward: the samples in chunks whose group sums and energies
// fit the chunk workspace; per chunk the sums pass (one lane per sample) and
// the frequency pass (a block per tile and frequency row), then one column reduction
// of the per-wave partial sums for the row sums.
// cplx: the complex-energy passes, whose group sums and energies take two
// columns each.
AmiStatus launch_two_pass(AmiTerms *t, DeviceTables *dt, bool hub, KArgs &a, double *out_sum, void *fn_sums,
                          void *fn_freq, hipStream_t stream, bool cplx = false, RowSums *sums = nullptr) {
    const int B = jit_block(t, hub);
    const int64_t tiles = (a.n_e + B - 1) / B;
    if (tiles > 0x7fffffffLL) return fail(AMI_E_ARG, "n_e too large");
    const int64_t rows = tiles * (B / 64);
    const int64_t cols = (cplx ? 2 : 1) * (static_cast<int64_t>(t->tab.G) + t->n_eps);
    const int64_t chunk_bytes = g_two_pass_chunk_bytes.load();
    int64_t ld = chunk_bytes / (cols * static_cast<int64_t>(sizeof(double))) / B * B;
    ld = std::max<int64_t>(B, std::min<int64_t>(ld, tiles * B));
    ld = std::min<int64_t>(ld, int64_t(1) << 28);   // the kernels address a chunk with 32-bit byte offsets
    double *ws = nullptr;
    const int ncols = a.mc ? 4 * a.n_f : 2 * a.n_f;   // per-wave sums (Monte Carlo: with squares)
    const size_t n_part = out_sum && !sums ? static_cast<size_t>(rows) * ncols : 0;
    AmiStatus st = workspace(t, dt, stream, (static_cast<size_t>(cols) * ld + n_part) * sizeof(double), &ws);
    if (st != AMI_OK) return st;
    a.work = ws;
    a.ld = ld;
    a.partial = sums ? sums->partial : out_sum ? ws + static_cast<size_t>(cols) * ld : nullptr;
    a.nrows = rows;
    // the largest chunk's frequency pass: a block per tile and frequency row
    if ((std::min<int64_t>(ld, a.n_e) + B - 1) / B * a.n_f + 7 * a.n_f > 0x7fffffffLL)
        return fail(AMI_E_ARG, "two-pass chunk too large for its frequency rows");
    hipError_t e = hipSuccess;
    for (int64_t s0 = 0; s0 < a.n_e && e == hipSuccess; s0 += ld) {
        a.s0 = s0;
        a.n_chunk = std::min<int64_t>(ld, a.n_e - s0);
        const int64_t nb = (a.n_chunk + B - 1) / B;
        e = launch_jit(fn_sums, nb, B, stream, a);
        // (tile, frequency) blocks, tiles rounded up to a multiple of the 8 XCDs
        if (e == hipSuccess) e = launch_jit(fn_freq, (nb + 7) / 8 * 8 * a.n_f, B, stream, a);
    }
    if (e == hipSuccess) e = hipGetLastError();
    g_last_variant = cplx ? "specialized complex two-pass" : "specialized two-pass";
    if (e != hipSuccess) return hip_fail(e, "two-pass launch");
    if (sums) *sums = RowSums{a.partial, rows, ncols};
    else if (out_sum) {
        hipLaunchKernelGGL(ami_colsum_kernel, dim3(ncols), dim3(kRedThreads), 0, stream, a.partial, rows,
                           static_cast<int64_t>(1), rows, out_sum);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "row-sum launch");
    }
    return AMI_OK;
}

AmiStatus launch_forward(AmiTerms *t, bool hub, KArgs &a, double *out_sum, hipStream_t stream, int variant = -1,
                         RowSums *sums = nullptr) {
    DeviceTables *dt = nullptr;
    AmiStatus st = upload(t, &dt);
    if (st != AMI_OK) return st;
    const Tables &tb = t->tab;
    if (a.n_e == 0) return fill(out_sum, 2 * static_cast<int64_t>(a.n_f), stream);
    Path path;
    void *jit_fn = nullptr, *jit_fn2 = nullptr;
    std::string note;
    st = choose_path(t, hub, false, path, &jit_fn, note, &jit_fn2, a.n_f, variant);
    if (st != AMI_OK) return st;
    if (path == Path::TWO_PASS) {
        st = launch_two_pass(t, dt, hub, a, out_sum, jit_fn, jit_fn2, stream, false, sums);
        g_last_variant += note;
        return st;
    }
    const bool block_fwd = path == Path::FWD_BLOCK;   // one row of partial sums per 64 samples
    if (block_fwd) path = Path::SPECIALIZED;
    LaunchShape ls;
    if (block_fwd) {
        ls.block = 64;
    } else if (path == Path::SPECIALIZED) {
        ls.block = jit_block(t, hub);
    } else {
        st = pick_shape(fwd_slots(tb), ls);
        if (st != AMI_OK) return st;
    }
    const int64_t nblocks = (a.n_e + ls.block - 1) / ls.block;
    if (nblocks > 0x7fffffffLL) return fail(AMI_E_ARG, "n_e too large");
    // partial-sum rows: one per wave for the specialized kernels, per block otherwise
    const int64_t rows = path == Path::SPECIALIZED ? nblocks * (ls.block / 64) : nblocks;
    double *partial = nullptr;
    hipError_t e;
    if (sums && path == Path::SPECIALIZED) {
        partial = sums->partial;
    } else if (out_sum) {
        st = workspace(t, dt, stream, static_cast<size_t>(rows) * a.n_f * 2 * sizeof(double), &partial);
        if (st != AMI_OK) return st;
    }
    const dim3 grid(static_cast<unsigned>(nblocks)), block(ls.block);
    if (path != Path::SPECIALIZED) timer_mark(stream, false);
    if (path == Path::SPECIALIZED) {
        a.partial = partial;
        a.nrows = rows;
        const int waves = block_fwd ? jit_block_forward_waves(t) : ls.block / 64;
        const int parts = block_fwd ? block_row_parts(waves, nblocks, a.n_f) : forward_row_parts(t, hub, false, rows, a.n_f);
        if (out_sum && !sums) {
            AdjOut o;
            o.out_sum = out_sum;
            const FinishLimits &lim = block_fwd ? kFinishBlockForward : kFinishOnePass;
            if (finish_small(t, dt, stream, a, lim, nblocks * parts, waves, 0, 2 * a.n_f, o)) out_sum = nullptr;
        }
        if (block_fwd) e = launch_block(jit_fn, nblocks, waves, stream, a, parts);
        else e = launch_jit(jit_fn, nblocks, ls.block, stream, a, parts);
        // the block forward is named as the two passes it stands for; those name
        // why it did not run where AUTO falls back to them
        g_last_variant = block_fwd ? "specialized two-pass" : "specialized";
        if (e == hipSuccess) e = hipGetLastError();
    } else if (path == Path::PACKED) {
        a.tb = packed_tabs(t, dt);
        a.slots = ls.slots;
        a.partial = partial;
        g_last_variant = std::string("packed ") +
                         (hub ? launch_packed<false, true>(t, grid, block, ls.lds, stream, a)
                              : launch_packed<false, false>(t, grid, block, ls.lds, stream, a)) + note;
        e = hipGetLastError();
    } else {
        launch_generic_forward(t, dt, hub, a, partial, ls, grid, stream);
        g_last_variant = "double tables" + note;
        e = hipGetLastError();
    }
    if (path != Path::SPECIALIZED) timer_mark(stream, true);
    if (e != hipSuccess) return hip_fail(e, "forward launch");
    if (sums && path == Path::SPECIALIZED) {
        *sums = RowSums{partial, rows, 2 * a.n_f};
    } else if (out_sum) {
        const bool cm = path == Path::SPECIALIZED;
        hipLaunchKernelGGL(ami_colsum_kernel, dim3(2 * a.n_f), dim3(kRedThreads), 0, stream, partial, rows,
                           static_cast<int64_t>(cm ? 1 : 2 * a.n_f), cm ? rows : static_cast<int64_t>(1), out_sum);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "row-sum launch");
    }
    return AMI_OK;
}

// Scratch of the allocation-free entry point (amiEvaluateHubbardAdjointNoAlloc):
// the partial sums of one call.  Every device the library runs on holds its
// own copy until the process ends.  In host code `scratch` names a host-side
// stand-in, not device memory: kernels get the address hipGetSymbolAddress
// returns for the current device (scratch_address).
constexpr size_t kScratchBytes = AMI_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];

constexpr int kScratchMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kScratchMaxDevices] = {};

// The device address of `scratch` on the current device, looked up on the
// first call there.
AmiStatus scratch_address(double **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kScratchMaxDevices) return fail(AMI_E_UNSUPPORTED, "device index beyond 63");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress (scratch)");
        if (!p) return fail(AMI_E_HIP, "hipGetSymbolAddress (scratch) returned NULL");
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return AMI_OK;
}

// The handle's tables on the current device when amiTermsUpload (or an
// earlier evaluate call) has put them there; uploads nothing.
AmiStatus find_uploaded(AmiTerms *t, DeviceTables **out) {
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> lk(t->dev_mu);
    for (auto &d : t->dev)
        if (d.device == dev) {
            *out = &d;
            return AMI_OK;
        }
    return fail(AMI_E_ARG, "the tables are not on this device: call amiTermsUpload first");
}

// Whether the adjoint of n_e samples with ncols columns of per-wave partial sums
// fits the allocation-free scratch: alone up to the one-pass kernel's automatic
// size, above it beside one chunk of samples of the passes (in *chunk, if given,
// the samples of the chunk that is left), whichever kernel then runs.
AmiStatus adjoint_scratch_fits(const AmiTerms *t, bool hub, int64_t n_e, int ncols, int64_t *chunk = nullptr) {
    const int B = jit_block(t, hub);
    const int64_t rows = (n_e + B - 1) / B * (B / 64);
    const int64_t left = static_cast<int64_t>(kScratchBytes / sizeof(double)) - rows * ncols;
    if (!chunk && t->tab.T <= kJitAutoAdjointTerms) {
        if (left >= 0) return AMI_OK;
        return fail(AMI_E_ARG, "the partial sums need " + std::to_string(rows * ncols * sizeof(double)) +
                                   " bytes, more than the " + std::to_string(kScratchBytes) +
                                   "-byte scratch of the allocation-free entry point: split the samples");
    }
    const int64_t cols = 2 * static_cast<int64_t>(t->tab.G) + 2 * t->n_eps;
    const int64_t ld = left > 0 ? left / cols / B * B : 0;
    if (chunk) *chunk = ld;
    if (ld >= B) return AMI_OK;
    return fail(AMI_E_ARG, "the partial sums and one chunk of samples do not fit the " + std::to_string(kScratchBytes) +
                               "-byte scratch of the allocation-free entry point: split the samples");
}

// The adjoint of a large solution in passes, per chunk of samples: the
// two-pass forward's sums pass (FT_g and E_j into the workspace), the
// frequency pass (values, FTB_g and the denominators' energy cotangents into
// the workspace, wave sums of dL/dw and of the values), the leaf pass (leaf
// cotangents, per-sample gradients, wave sums of dL/dbeta, dL/dmu, dL/dt);
// then one reduction of the wave sums.  Workspace: the partial sums (rows x
// columns), then the chunk's 2 G + 2 NE columns of ld samples each.
// fixed_ws: both in the allocation-free scratch (the chunk sized to what is
// left), nothing allocated.
// cplx: the passes at complex energies, whose workspace columns are complex
// (4 G + 4 NE of them).
AmiStatus launch_adjoint_passes(AmiTerms *t, DeviceTables *dt, bool hub, KArgs &a, const AdjOut &o, void *fn_sums,
                                void *fn_freq, void *fn_leaf, hipStream_t stream, double *fixed_ws,
                                bool cplx = false) {
    const int B = jit_block(t, hub);
    const int64_t tiles = (a.n_e + B - 1) / B;
    if (tiles > 0x7fffffffLL) return fail(AMI_E_ARG, "n_e too large");
    const int64_t rows = tiles * (B / 64);
    const int ncols = kAdjScalars + 2 * a.n_f * t->n_ext;
    const int nval = o.out_sum ? 2 * a.n_f : 0;
    const int64_t cols = (cplx ? 2 : 1) * (2 * static_cast<int64_t>(t->tab.G) + 2 * t->n_eps);
    const size_t n_part = static_cast<size_t>(rows) * (ncols + nval);
    int64_t ld = 0;
    double *ws = nullptr;
    if (fixed_ws) {
        const AmiStatus st = adjoint_scratch_fits(t, hub, a.n_e, ncols + nval, &ld);
        if (st != AMI_OK) return st;
        ld = std::min<int64_t>(ld, tiles * B);
        ws = fixed_ws;
    } else {
        ld = g_two_pass_chunk_bytes.load() / (cols * static_cast<int64_t>(sizeof(double))) / B * B;
        ld = std::max<int64_t>(B, std::min<int64_t>(ld, tiles * B));
    }
    ld = std::min<int64_t>(ld, int64_t(1) << 28);   // the kernels address a chunk with 32-bit byte offsets
    if (!fixed_ws) {
        const AmiStatus st = workspace(t, dt, stream, (n_part + static_cast<size_t>(cols) * ld) * sizeof(double), &ws);
        if (st != AMI_OK) return st;
    }
    a.gpartial = ws;
    a.partial = o.out_sum ? ws + static_cast<size_t>(rows) * ncols : nullptr;
    a.nrows = rows;
    a.work = ws + n_part;
    a.ld = ld;
    a.mc = 0;
    hipError_t e = hipSuccess;
    for (int64_t s0 = 0; s0 < a.n_e && e == hipSuccess; s0 += ld) {
        a.s0 = s0;
        a.n_chunk = std::min<int64_t>(ld, a.n_e - s0);
        const int64_t nb = (a.n_chunk + B - 1) / B;
        e = launch_jit(fn_sums, nb, B, stream, a);
        if (e == hipSuccess) e = launch_jit(fn_freq, nb, B, stream, a);
        if (e == hipSuccess) e = launch_jit(fn_leaf, nb, B, stream, a);
    }
    if (e == hipSuccess) e = hipGetLastError();
    g_last_variant = cplx ? "specialized complex passes" : "specialized passes";
    if (e != hipSuccess) return hip_fail(e, "adjoint passes launch");
    hipLaunchKernelGGL(ami_adj_finalize_kernel, dim3(ncols + nval), dim3(kRedThreads), 0, stream, a.gpartial, rows,
                       ncols, 1, o.grad_beta, o.grad_mu, o.grad_t, o.grad_freqs, 2 * a.n_f, o.out_sum);
    e = hipGetLastError();
    return e == hipSuccess ? AMI_OK : hip_fail(e, "adjoint reduction launch");
}

// The adjoint of a large solution in one launch: blocks of 64 samples whose
// waves split the solution, each block one row of the partial sums.  fixed_ws:
// the partial sums in the allocation-free scratch, under the size limit of the
// passes (the entry point's documented one).
AmiStatus launch_adjoint_block(AmiTerms *t, DeviceTables *dt, bool hub, KArgs &a, const AdjOut &o, void *fn,
                               hipStream_t stream, double *fixed_ws, bool cplx = false) {
    const int64_t rows = (a.n_e + 63) / 64;
    if (rows > 0x7fffffffLL) return fail(AMI_E_ARG, "n_e too large");
    const int ncols = kAdjScalars + 2 * a.n_f * t->n_ext;
    const int nval = o.out_sum ? 2 * a.n_f : 0;
    double *ws = fixed_ws;
    if (fixed_ws) {
        const AmiStatus st = adjoint_scratch_fits(t, hub, a.n_e, ncols + nval);
        if (st != AMI_OK) return st;
    } else {
        const AmiStatus st = workspace(t, dt, stream, static_cast<size_t>(rows) * (ncols + nval) * sizeof(double), &ws);
        if (st != AMI_OK) return st;
    }
    a.gpartial = ws;
    a.partial = o.out_sum ? ws + static_cast<size_t>(rows) * ncols : nullptr;
    a.nrows = rows;
    const int waves = jit_block_waves(t, hub, cplx, a.n_f > 1);
    const bool fin = !fixed_ws && finish_small(t, dt, stream, a, kFinishBlockAdjoint, rows, waves, ncols, nval, o);
    hipError_t e = launch_block(fn, rows, waves, stream, a);
    if (e == hipSuccess) e = hipGetLastError();
    // named by the size, as the kernels it stands for (one pass or passes)
    if (cplx) g_last_variant = t->tab.T > kJitAutoComplexAdjointTerms ? "specialized complex passes" : "specialized complex";
    else g_last_variant = t->tab.T > kJitAutoAdjointTerms ? "specialized passes" : "specialized";
    if (e != hipSuccess) return hip_fail(e, "block adjoint launch");
    if (fin) return AMI_OK;
    hipLaunchKernelGGL(ami_adj_finalize_kernel, dim3(ncols + nval), dim3(kRedThreads), 0, stream, a.gpartial, rows,
                       ncols, 1, o.grad_beta, o.grad_mu, o.grad_t, o.grad_freqs, 2 * a.n_f, o.out_sum);
    e = hipGetLastError();
    return e == hipSuccess ? AMI_OK : hip_fail(e, "adjoint reduction launch");
}

// fixed_ws: the partial sums go there (at most kScratchBytes), and nothing is
// uploaded, compiled, loaded or allocated (the allocation-free entry point);
// NULL: the handle's per-stream workspace.
AmiStatus launch_adjoint(AmiTerms *t, bool hub, KArgs &a, const AdjOut &o, hipStream_t stream,
                         double *fixed_ws = nullptr) {
    DeviceTables *dt = nullptr;
    AmiStatus st = fixed_ws ? find_uploaded(t, &dt) : upload(t, &dt);
    if (st != AMI_OK) return st;
    const Tables &tb = t->tab;
    const int nx = t->n_ext;
    const int ncols = kAdjScalars + 2 * a.n_f * nx;
    if (a.n_e == 0) {
        for (double *p : {o.grad_beta, o.grad_mu, o.grad_t}) {
            st = fill(p, 1, stream);
            if (st != AMI_OK) return st;
        }
        st = fill(o.out_sum, 2 * static_cast<int64_t>(a.n_f), stream);
        if (st != AMI_OK) return st;
        return fill(o.grad_freqs, 2 * static_cast<int64_t>(a.n_f) * nx, stream);
    }
    Path path;
    void *jit_fn = nullptr, *jit_fn2 = nullptr, *jit_fn3 = nullptr;
    std::string note;
    st = choose_path(t, hub, true, path, &jit_fn, note, &jit_fn2, a.n_f, -1, fixed_ws != nullptr, &jit_fn3);
    if (st != AMI_OK) return st;
    if (path == Path::ADJ_PASSES) {
        st = launch_adjoint_passes(t, dt, hub, a, o, jit_fn, jit_fn2, jit_fn3, stream, fixed_ws);
        g_last_variant += note;
        return st;
    }
    if (path == Path::ADJ_BLOCK) return launch_adjoint_block(t, dt, hub, a, o, jit_fn, stream, fixed_ws);
    LaunchShape ls;
    if (path == Path::SPECIALIZED) {
        ls.block = jit_block(t, hub);
    } else {
        st = pick_shape(adj_slots(tb), ls);
        if (st != AMI_OK) return st;
    }
    const int64_t nblocks = (a.n_e + ls.block - 1) / ls.block;
    if (nblocks > 0x7fffffffLL) return fail(AMI_E_ARG, "n_e too large");
    // partial-sum rows: one per wave for the specialized kernels, per block otherwise
    const int64_t rows = path == Path::SPECIALIZED ? nblocks * (ls.block / 64) : nblocks;
    double *partial = nullptr;
    const size_t n_grad = static_cast<size_t>(rows) * ncols;
    const size_t n_val = o.out_sum ? static_cast<size_t>(rows) * a.n_f * 2 : 0;
    const size_t ws_bytes = (n_grad + n_val) * sizeof(double);
    if (fixed_ws) {
        if (ws_bytes > kScratchBytes)
            return fail(AMI_E_ARG, "the partial sums need " + std::to_string(ws_bytes) +
                                       " bytes, more than the " + std::to_string(kScratchBytes) +
                                       "-byte scratch of the allocation-free entry point: split the samples");
        partial = fixed_ws;
    } else {
        st = workspace(t, dt, stream, ws_bytes, &partial);
        if (st != AMI_OK) return st;
    }
    hipError_t e;
    bool fin = false;
    a.gpartial = partial;
    a.partial = o.out_sum ? partial + n_grad : nullptr;
    const dim3 grid(static_cast<unsigned>(nblocks)), block(ls.block);
    if (path == Path::SPECIALIZED) {
        a.nrows = rows;
        fin = !fixed_ws && finish_small(t, dt, stream, a, kFinishOnePass, nblocks, ls.block / 64, ncols,
                                       o.out_sum ? 2 * a.n_f : 0, o);
        e = launch_jit(jit_fn, nblocks, ls.block, stream, a);
        g_last_variant = "specialized" + note;
        if (e == hipSuccess) e = hipGetLastError();
    } else {
        a.tb = packed_tabs(t, dt);
        a.slots = ls.slots;
        timer_mark(stream, false);
        g_last_variant = std::string("packed ") +
                         (hub ? launch_packed<true, true>(t, grid, block, ls.lds, stream, a)
                              : launch_packed<true, false>(t, grid, block, ls.lds, stream, a)) + note;
        e = hipGetLastError();
        timer_mark(stream, true);
    }
    if (e != hipSuccess) return hip_fail(e, "adjoint launch");
    if (fin) return AMI_OK;
    // one launch for every reduction: gradient columns, then the value row sums
    const int n_red = ncols + (o.out_sum ? 2 * a.n_f : 0);
    hipLaunchKernelGGL(ami_adj_finalize_kernel, dim3(n_red), dim3(kRedThreads), 0, stream, partial, rows, ncols,
                       path == Path::SPECIALIZED ? 1 : 0, o.grad_beta, o.grad_mu, o.grad_t, o.grad_freqs, 2 * a.n_f,
                       o.out_sum);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "adjoint reduction launch");
    return AMI_OK;
}

AmiStatus check_common(const AmiTerms *t, int64_t n_e, const double *ext_freqs, int64_t n_f, double beta) {
    if (!t) return fail(AMI_E_ARG, "terms is NULL");
    if (n_e < 0) return fail(AMI_E_ARG, "n_e < 0");
    if (n_f < 1 || n_f > (1 << 24)) return fail(AMI_E_ARG, "n_f must be in 1..2^24");
    if (!ext_freqs && t->n_ext > 0) return fail(AMI_E_ARG, "ext_freqs is NULL");
    if (!(beta > 0.0)) return fail(AMI_E_ARG, "beta must be > 0");
    if (t->n_eps > kMaxEpsDev) return fail(AMI_E_UNSUPPORTED, "more than 16 energy placeholders");
    if (t->n_ext > kMaxExt) return fail(AMI_E_UNSUPPORTED, "more than 4 external frequency slots");
    return AMI_OK;
}

AmiStatus check_energies(const AmiTerms *, int64_t n_e, const double *energies, int64_t stride_s,
                         int64_t stride_i) {
    if (n_e > 0 && !energies) return fail(AMI_E_ARG, "energies is NULL");
    if (n_e > 0 && (stride_i < 1 || stride_s < 1)) return fail(AMI_E_ARG, "strides must be >= 1");
    return AMI_OK;
}

AmiStatus check_momenta(const AmiTerms *t, int64_t n_e, const double *k, int64_t stride_k, const double *q) {
    if (t->n_eps != t->n_g) return fail(AMI_E_ARG, "the momentum path needs one energy per propagator");
    if (t->n_int > kMaxInt) return fail(AMI_E_UNSUPPORTED, "more than 12 summed frequencies on the momentum path");
    if (n_e > 0 && !k) return fail(AMI_E_ARG, "k is NULL");
    if (n_e > 0 && stride_k < 2 * t->n_int) return fail(AMI_E_ARG, "stride_k < 2*n_int");
    if (t->n_ext > 0 && !q) return fail(AMI_E_ARG, "q is NULL");
    return AMI_OK;
}

void set_momenta(KArgs &a, const AmiTerms *t, const double *k, int64_t stride_k, const double *q, double hop_t,
                 double mu) {
    a.k = k;
    a.stride_k = stride_k;
    a.q_big = 0;
    if (k && (reinterpret_cast<uintptr_t>(k) & 15u) == 0 && (stride_k & 1) == 0) a.vec_io |= 1;
    for (int x = 0; x < t->n_ext && x < kMaxExtDev; ++x)
        for (int c = 0; c < 2; ++c) {
            const double r = std::remainder(q[2 * x + c], 2.0 * M_PI);
            a.q[2 * x + c] = r;
            a.qs[2 * x + c] = std::sin(r);
            a.qc[2 * x + c] = std::cos(r);
        }
    a.hop_t = hop_t;
    a.mu = mu;
}

void set_common(KArgs &a, const double *ext_freqs, int64_t n_f, double beta, double e_reg, int64_t n_e) {
    a.ext_freqs = ext_freqs;
    a.n_f = static_cast<int>(n_f);
    a.beta = beta;
    a.e_reg = e_reg;
    a.n_e = n_e;
}

// The kernels that amiTermsSpecialize makes ready for this input under a variant:
// AUTO's, or what a forced variant takes beside them -- the passes and one-pass
// adjoints that AUTO leaves to the block kernels where a solution splits (their
// compilation is as long as the block kernels').
std::vector<int> kernels_of(const AmiTerms *t, bool hub, int variant) {
    const bool forced = variant != AMI_VARIANT_AUTO;
    const bool one_pass = variant == AMI_VARIANT_SPECIALIZED, passes = variant == AMI_VARIANT_TWO_PASS;
    const int T = t->tab.T;
    const bool small = T <= kJitMaxTerms;
    bool taylor = false;                    // Taylor-coefficient leaves: no complex energies
    for (int o : t->tab.leaf_order) taylor = taylor || o > 0;
    std::vector<int> kinds;
    if (!forced) {
        if (jit_prefers_two_pass(t)) {      // the passes: Monte Carlo, and persistent batches
            kinds.push_back(kJitSumsPass);
            kinds.push_back(kJitFreqPass);
            if (jit_block_forward_waves(t) > 0) kinds.push_back(kJitBlockForward);
        } else {
            kinds.push_back(kJitForward);
        }
    }
    if ((one_pass || passes) && jit_prefers_two_pass(t)) {
        kinds.push_back(kJitSumsPass);
        kinds.push_back(kJitFreqPass);
    }
    const bool block = jit_prefers_block_adjoint(t) && jit_block_waves(t, hub) > 0;
    if (!forced && block) {
        kinds.push_back(kJitBlockAdjoint);
        if (jit_block_rows_apart(t)) kinds.push_back(kJitBlockAdjointRows);
    }
    if (T <= kJitAutoAdjointTerms) {
        if (forced ? one_pass : !block) kinds.push_back(kJitAdjoint);
    } else if ((forced ? passes : !block) && jit_adjoint_passes_supported(t, hub, nullptr)) {
        if (!jit_prefers_two_pass(t)) kinds.push_back(kJitSumsPass);
        kinds.push_back(kJitAdjFreq);
        kinds.push_back(kJitAdjLeaf);
    }
    if (taylor || hub || T > kJitTwoPassMaxTerms) return kinds;
    // complex energies: the forward in one pass up to 1024 terms, in two above; the
    // adjoint in a block, in one pass up to 512 terms, or in passes above
    if (!forced) {
        if (small) {
            kinds.push_back(kJitComplex);
        } else {
            kinds.push_back(kJitComplexSums);
            kinds.push_back(kJitComplexFreq);
        }
    }
    const bool cblock = jit_block_waves(t, false, true) > 0;
    if (!forced && cblock && jit_prefers_complex_block(t, true)) kinds.push_back(kJitComplexBlockAdjoint);
    const bool all_rows = cblock && jit_prefers_complex_block(t, false);      // the block for any number of rows
    if (T <= kJitAutoComplexAdjointTerms) {
        if (forced ? one_pass : !all_rows) kinds.push_back(kJitComplexAdj);
    } else if (forced ? passes : !all_rows) {
        if (forced || small) kinds.push_back(kJitComplexSums);
        kinds.push_back(kJitComplexAdjFreq);
        kinds.push_back(kJitComplexAdjLeaf);
    }
    return kinds;
}

// After amiSetVariant: loads what the new variant takes in place of AUTO's block
// kernels, on the devices of the handle's kernels, so that no later call (under
// capture, or the allocation-free one) finds it missing: for the inputs that
// amiTermsSpecialize has made ready, else where a call has loaded the block kernel
// that it stands for.  A kernel that is not to be had is reported by the call that needs it.
void specialize_variant(AmiTerms *t) {
    if (t->variant == AMI_VARIANT_AUTO) return;
    for (int h = 0; h < 2; ++h) {
        const bool hub = h != 0, all = t->specialized[h].load();
        const bool fwd = all || jit_has_module(t, hub, kJitBlockForward);
        const bool adj = all || jit_has_module(t, hub, kJitBlockAdjoint);
        const bool cadj = !hub && (all || jit_has_module(t, hub, kJitComplexBlockAdjoint));
        if (!fwd && !adj && !cadj) continue;
        for (int k : kernels_of(t, hub, t->variant))
            if (jit_kind_complex(k) ? cadj : k == kJitFreqPass ? fwd : k == kJitSumsPass ? fwd || adj : adj)
                (void)jit_load_everywhere(t, hub, k);
    }
    clear_error();
}

}  // namespace

AmiStatus launch_forward_as(AmiTerms *t, bool hub, KArgs &a, double *out_sum, hipStream_t stream, int variant,
                            RowSums *sums) {
    return launch_forward(t, hub, a, out_sum, stream, variant, sums);
}

int64_t row_sum_rows(const AmiTerms *t, bool hub, int64_t n_e) {
    const int B = jit_block(t, hub);      // the block forward's tiles of 64 samples are no more
    return (n_e + B - 1) / B * (B / 64);
}

bool specialized_forward_ready(AmiTerms *t, bool hub, int n_f, int variant) {
    Path p;
    void *f1 = nullptr, *f2 = nullptr;
    std::string note;
    const AmiStatus st = choose_path(t, hub, false, p, &f1, note, &f2, n_f, variant);
    clear_error();
    return st == AMI_OK && (p == Path::SPECIALIZED || p == Path::TWO_PASS || p == Path::FWD_BLOCK);
}

void set_inputs(KArgs &a, const AmiTerms *t, const double *k, int64_t stride_k, const double *q, double hop_t,
                double mu, const double *energies, int64_t stride_s, int64_t stride_i, const double *ext_freqs,
                int64_t n_f, double beta, double e_reg, int64_t n_e) {
    if (k) set_momenta(a, t, k, stride_k, q, hop_t, mu);
    a.energies = energies;
    a.stride_s = stride_s;
    a.stride_i = stride_i;
    set_common(a, ext_freqs, n_f, beta, e_reg, n_e);
}

}  // namespace ami

extern "C" {

AmiStatus amiTermsUpload(AmiTerms *t) {
    ami::clear_error();
    if (!t) return ami::fail(AMI_E_ARG, "terms is NULL");
    ami::DeviceTables *dt = nullptr;
    return ami::upload(t, &dt);
}

void amiFree(AmiTerms *t) {
    if (!t) return;
    int cur = 0;
    const bool have_cur = hipGetDevice(&cur) == hipSuccess;
    for (auto &d : t->dev)
        if (hipSetDevice(d.device) == hipSuccess) {
            if (d.blob) (void)hipFree(d.blob);
            for (auto &w : d.ws) (void)hipFree(w.ptr);
            for (void *p : d.retired) (void)hipFree(p);
        }
    if (have_cur) (void)hipSetDevice(cur);
    ami::jit_release(t);
    delete t;
}

AmiStatus amiEvaluate(AmiTerms *t, const double *energies, int64_t n_e, int64_t stride_s, int64_t stride_i,
                      const double *ext_freqs, int64_t n_f, double beta, double e_reg, double *out,
                      double *out_sum, void *hip_stream) {
    using namespace ami;
    clear_error();
    AmiStatus st = check_common(t, n_e, ext_freqs, n_f, beta);
    if (st == AMI_OK) st = check_energies(t, n_e, energies, stride_s, stride_i);
    if (st != AMI_OK) return st;
    if (!out && !out_sum) return fail(AMI_E_ARG, "out and out_sum are both NULL");
    KArgs a;
    std::memset(&a, 0, sizeof(a));
    a.energies = energies;
    a.stride_s = stride_s;
    a.stride_i = stride_i;
    set_common(a, ext_freqs, n_f, beta, e_reg, n_e);
    a.out = out;
    return launch_forward(t, false, a, out_sum, static_cast<hipStream_t>(hip_stream));
}

AmiStatus amiEvaluateComplex(AmiTerms *t, const double *energies, int64_t n_e, int64_t stride_s, int64_t stride_i,
                             const double *ext_freqs, int64_t n_f, double beta, double e_reg, double *out,
                             double *out_sum, void *hip_stream) {
    using namespace ami;
    clear_error();
    AmiStatus st = check_common(t, n_e, ext_freqs, n_f, beta);
    if (st == AMI_OK) st = check_energies(t, n_e, energies, stride_s, stride_i);
    if (st != AMI_OK) return st;
    if (!out && !out_sum) return fail(AMI_E_ARG, "out and out_sum are both NULL");
    const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    DeviceTables *dt = nullptr;
    st = upload(t, &dt);
    if (st != AMI_OK) return st;
    // solutions above the one-pass size (or the forced two-pass variant): the
    // complex group sums stored per sample, then evaluated per frequency row
    if (t->tab.T > kJitMaxTerms || t->variant == AMI_VARIANT_TWO_PASS) {
        void *fs = nullptr, *ff = nullptr;
        st = jit_get(t, false, kJitComplexSums, &fs);
        if (st == AMI_OK) st = jit_get(t, false, kJitComplexFreq, &ff);
        if (st != AMI_OK) return st;
        if (n_e == 0) return fill(out_sum, 2 * n_f, stream);
        if (n_f > kTwoPassMaxFreqs) return fail(AMI_E_ARG, "the two-pass variant takes at most 65535 frequency rows");
        KArgs a;
        std::memset(&a, 0, sizeof(a));
        a.energies = energies;
        a.stride_s = stride_s;
        a.stride_i = stride_i;
        set_common(a, ext_freqs, n_f, beta, e_reg, n_e);
        a.out = out;
        return launch_two_pass(t, dt, false, a, out_sum, fs, ff, stream, true);
    }
    void *fn = nullptr;
    st = jit_get(t, false, kJitComplex, &fn);
    if (st != AMI_OK) return st;
    if (n_e == 0) return fill(out_sum, 2 * n_f, stream);
    const int block = jit_block(t, false);
    const int64_t nblocks = (n_e + block - 1) / block;
    if (nblocks > 0x7fffffffLL) return fail(AMI_E_ARG, "n_e too large");
    const int64_t rows = nblocks * (block / 64);   // partial sums per wave
    KArgs a;
    std::memset(&a, 0, sizeof(a));
    a.energies = energies;
    a.stride_s = stride_s;
    a.stride_i = stride_i;
    set_common(a, ext_freqs, n_f, beta, e_reg, n_e);
    a.out = out;
    a.nrows = rows;
    if (out_sum) {
        st = workspace(t, dt, stream, static_cast<size_t>(rows) * n_f * 2 * sizeof(double), &a.partial);
        if (st != AMI_OK) return st;
    }
    const int parts = forward_row_parts(t, false, true, rows, n_f);
    AdjOut o;
    o.out_sum = out_sum;
    const bool fin = out_sum && finish_small(t, dt, stream, a, kFinishComplex, nblocks * parts, block / 64, 0,
                                             static_cast<int>(2 * n_f), o);
    hipError_t e = launch_jit(fn, nblocks, block, stream, a, parts);
    if (e == hipSuccess) e = hipGetLastError();
    g_last_variant = "specialized complex";
    if (e != hipSuccess) return hip_fail(e, "complex-energy launch");
    if (out_sum && !fin) {
        hipLaunchKernelGGL(ami_colsum_kernel, dim3(static_cast<unsigned>(2 * n_f)), dim3(kRedThreads), 0, stream,
                           a.partial, rows, static_cast<int64_t>(1), rows, out_sum);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "row-sum launch");
    }
    return AMI_OK;
}

AmiStatus amiEvaluateComplexAdjoint(AmiTerms *t, const double *energies, int64_t n_e, int64_t stride_s,
                                    int64_t stride_i, const double *ext_freqs, int64_t n_f, double beta, double e_reg,
                                    const double *grad_out, const double *grad_sum, double *grad_energies,
                                    double *grad_beta, double *grad_freqs, double *out, double *out_sum,
                                    void *hip_stream) {
    using namespace ami;
    clear_error();
    AmiStatus st = check_common(t, n_e, ext_freqs, n_f, beta);
    if (st == AMI_OK) st = check_energies(t, n_e, energies, stride_s, stride_i);
    if (st != AMI_OK) return st;
    if (!grad_out && !grad_sum) return fail(AMI_E_ARG, "grad_out and grad_sum are both NULL");
    const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    DeviceTables *dt = nullptr;
    st = upload(t, &dt);
    if (st != AMI_OK) return st;
    KArgs ba;
    std::memset(&ba, 0, sizeof(ba));
    ba.energies = energies;
    ba.stride_s = stride_s;
    ba.stride_i = stride_i;
    set_common(ba, ext_freqs, n_f, beta, e_reg, n_e);
    ba.g_out = grad_out;
    ba.g_sum = grad_sum;
    ba.grad_e = grad_energies;
    ba.out = out;
    AdjOut bo;
    bo.grad_beta = grad_beta;
    bo.grad_freqs = grad_freqs;
    bo.out_sum = out_sum;
    std::string note;
    // AUTO: the block adjoint where the solution splits over the waves of a block
    bool to_block = t->variant == AMI_VARIANT_AUTO && n_e > 0 && jit_prefers_complex_block(t, n_f == 1) &&
                    jit_block_waves(t, false, true) > 0;
    // where the number of rows decides, earlier calls with other rows may have left
    // this call's kernel unloaded: under capture, which is no place to compile, the
    // one that is loaded serves
    if (t->variant == AMI_VARIANT_AUTO && n_e > 0 && jit_prefers_complex_block(t, true) &&
        !jit_prefers_complex_block(t, false) && capturing(stream)) {
        void *fn = nullptr;
        const bool block = jit_loaded(t, false, kJitComplexBlockAdjoint, &fn) == AMI_OK;
        if (block != (jit_loaded(t, false, kJitComplexAdj, &fn) == AMI_OK)) to_block = block;
        clear_error();
    }
    if (to_block) {
        void *fb = nullptr;
        st = jit_get(t, false, kJitComplexBlockAdjoint, &fb);
        if (st == AMI_OK) return launch_adjoint_block(t, dt, false, ba, bo, fb, stream, nullptr, true);
        note = std::string(" (not in a block: ") + amiLastError() + ")";
        clear_error();
    }
    // above the one-pass complex adjoint's automatic size (unless the handle
    // forces the specialized variant), or under the forced two-pass variant:
    // the adjoint in passes at complex energies
    if (t->variant == AMI_VARIANT_TWO_PASS ||
        (t->variant != AMI_VARIANT_SPECIALIZED && t->tab.T > kJitAutoComplexAdjointTerms)) {
        void *fs = nullptr, *ff = nullptr, *fl = nullptr;
        st = jit_get(t, false, kJitComplexSums, &fs);
        if (st == AMI_OK) st = jit_get(t, false, kJitComplexAdjFreq, &ff);
        if (st == AMI_OK) st = jit_get(t, false, kJitComplexAdjLeaf, &fl);
        if (st != AMI_OK) return st;
        if (n_e == 0) {
            st = fill(grad_beta, 1, stream);
            if (st == AMI_OK) st = fill(out_sum, 2 * n_f, stream);
            if (st == AMI_OK) st = fill(grad_freqs, 2 * n_f * t->n_ext, stream);
            return st;
        }
        st = launch_adjoint_passes(t, dt, false, ba, bo, fs, ff, fl, stream, nullptr, true);
        g_last_variant += note;
        return st;
    }
    void *fn = nullptr;
    st = jit_get(t, false, kJitComplexAdj, &fn);
    if (st != AMI_OK) return st;
    const int nx = t->n_ext;
    const int ncols = kAdjScalars + 2 * static_cast<int>(n_f) * nx;
    if (n_e == 0) {
        st = fill(grad_beta, 1, stream);
        if (st == AMI_OK) st = fill(out_sum, 2 * n_f, stream);
        if (st == AMI_OK) st = fill(grad_freqs, 2 * n_f * nx, stream);
        return st;
    }
    const int block = jit_block(t, false);
    const int64_t nblocks = (n_e + block - 1) / block;
    if (nblocks > 0x7fffffffLL) return fail(AMI_E_ARG, "n_e too large");
    const int64_t rows = nblocks * (block / 64);   // partial sums per wave
    const size_t n_grad = static_cast<size_t>(rows) * ncols;
    const size_t n_val = out_sum ? static_cast<size_t>(rows) * n_f * 2 : 0;
    double *partial = nullptr;
    st = workspace(t, dt, stream, (n_grad + n_val) * sizeof(double), &partial);
    if (st != AMI_OK) return st;
    KArgs a;
    std::memset(&a, 0, sizeof(a));
    a.energies = energies;
    a.stride_s = stride_s;
    a.stride_i = stride_i;
    set_common(a, ext_freqs, n_f, beta, e_reg, n_e);
    a.g_out = grad_out;
    a.g_sum = grad_sum;
    a.grad_e = grad_energies;
    a.out = out;
    a.nrows = rows;
    a.gpartial = partial;
    a.partial = out_sum ? partial + n_grad : nullptr;
    const int nval = out_sum ? 2 * static_cast<int>(n_f) : 0;
    const bool fin = finish_small(t, dt, stream, a, kFinishComplexAdjoint, nblocks, block / 64, ncols, nval, bo);
    hipError_t e = launch_jit(fn, nblocks, block, stream, a);
    if (e == hipSuccess) e = hipGetLastError();
    g_last_variant = "specialized complex" + note;
    if (e != hipSuccess) return hip_fail(e, "complex-energy adjoint launch");
    if (fin) return AMI_OK;
    const int n_red = ncols + nval;
    hipLaunchKernelGGL(ami_adj_finalize_kernel, dim3(n_red), dim3(kRedThreads), 0, stream, partial, rows, ncols, 1,
                       grad_beta, static_cast<double *>(nullptr), static_cast<double *>(nullptr), grad_freqs,
                       2 * static_cast<int>(n_f), out_sum);
    e = hipGetLastError();
    return e == hipSuccess ? AMI_OK : hip_fail(e, "adjoint reduction launch");
}

AmiStatus amiEvaluateHubbard(AmiTerms *t, const double *k, int64_t n_e, int64_t stride_k, const double *q,
                             double hop_t, double mu, const double *ext_freqs, int64_t n_f, double beta,
                             double e_reg, double *out, double *out_sum, void *hip_stream) {
    using namespace ami;
    clear_error();
    AmiStatus st = check_common(t, n_e, ext_freqs, n_f, beta);
    if (st == AMI_OK) st = check_momenta(t, n_e, k, stride_k, q);
    if (st != AMI_OK) return st;
    if (!out && !out_sum) return fail(AMI_E_ARG, "out and out_sum are both NULL");
    KArgs a;
    std::memset(&a, 0, sizeof(a));
    set_momenta(a, t, k, stride_k, q, hop_t, mu);
    set_common(a, ext_freqs, n_f, beta, e_reg, n_e);
    a.out = out;
    return launch_forward(t, true, a, out_sum, static_cast<hipStream_t>(hip_stream));
}

AmiStatus amiEvaluateAdjoint(AmiTerms *t, const double *energies, int64_t n_e, int64_t stride_s,
                             int64_t stride_i, const double *ext_freqs, int64_t n_f, double beta, double e_reg,
                             const double *grad_out, const double *grad_sum, double *grad_energies,
                             double *grad_beta, double *grad_freqs, double *out, double *out_sum,
                             void *hip_stream) {
    using namespace ami;
    clear_error();
    AmiStatus st = check_common(t, n_e, ext_freqs, n_f, beta);
    if (st == AMI_OK) st = check_energies(t, n_e, energies, stride_s, stride_i);
    if (st != AMI_OK) return st;
    if (!grad_out && !grad_sum) return fail(AMI_E_ARG, "grad_out and grad_sum are both NULL");
    KArgs a;
    std::memset(&a, 0, sizeof(a));
    a.energies = energies;
    a.stride_s = stride_s;
    a.stride_i = stride_i;
    set_common(a, ext_freqs, n_f, beta, e_reg, n_e);
    a.g_out = grad_out;
    a.g_sum = grad_sum;
    a.grad_e = grad_energies;
    a.out = out;
    AdjOut o;
    o.grad_beta = grad_beta;
    o.grad_freqs = grad_freqs;
    o.out_sum = out_sum;
    return launch_adjoint(t, false, a, o, static_cast<hipStream_t>(hip_stream));
}

}  // extern "C"

namespace ami {
namespace {

AmiStatus hubbard_adjoint(AmiTerms *t, const double *k, int64_t n_e, int64_t stride_k, const double *q,
                          double hop_t, double mu, const double *ext_freqs, int64_t n_f, double beta, double e_reg,
                          const double *grad_out, const double *grad_sum, double *grad_k, double *grad_mu,
                          double *grad_t, double *grad_beta, double *grad_freqs, double *out, double *out_sum,
                          void *hip_stream, bool no_alloc) {
    clear_error();
    AmiStatus st = check_common(t, n_e, ext_freqs, n_f, beta);
    if (st == AMI_OK) st = check_momenta(t, n_e, k, stride_k, q);
    if (st != AMI_OK) return st;
    if (!grad_out && !grad_sum) return fail(AMI_E_ARG, "grad_out and grad_sum are both NULL");
    KArgs a;
    std::memset(&a, 0, sizeof(a));
    set_momenta(a, t, k, stride_k, q, hop_t, mu);
    set_common(a, ext_freqs, n_f, beta, e_reg, n_e);
    a.g_out = grad_out;
    a.g_sum = grad_sum;
    a.grad_k = grad_k;
    if (grad_k && (reinterpret_cast<uintptr_t>(grad_k) & 15u) == 0) a.vec_io |= 2;
    a.out = out;
    AdjOut o;
    o.grad_beta = grad_beta;
    o.grad_mu = grad_mu;
    o.grad_t = grad_t;
    o.grad_freqs = grad_freqs;
    o.out_sum = out_sum;
    double *ws = nullptr;
    if (no_alloc) {
        st = scratch_address(&ws);
        if (st != AMI_OK) return st;
    }
    return launch_adjoint(t, true, a, o, static_cast<hipStream_t>(hip_stream), ws);
}

}  // namespace
}  // namespace ami

extern "C" {

AmiStatus amiEvaluateHubbardAdjoint(AmiTerms *t, const double *k, int64_t n_e, int64_t stride_k, const double *q,
                                    double hop_t, double mu, const double *ext_freqs, int64_t n_f, double beta,
                                    double e_reg, const double *grad_out, const double *grad_sum, double *grad_k,
                                    double *grad_mu, double *grad_t, double *grad_beta, double *grad_freqs,
                                    double *out, double *out_sum, void *hip_stream) {
    return ami::hubbard_adjoint(t, k, n_e, stride_k, q, hop_t, mu, ext_freqs, n_f, beta, e_reg, grad_out, grad_sum,
                                grad_k, grad_mu, grad_t, grad_beta, grad_freqs, out, out_sum, hip_stream, false);
}

AmiStatus amiEvaluateHubbardAdjointNoAlloc(AmiTerms *t, const double *k, int64_t n_e, int64_t stride_k,
                                           const double *q, double hop_t, double mu, const double *ext_freqs,
                                           int64_t n_f, double beta, double e_reg, const double *grad_out,
                                           const double *grad_sum, double *grad_k, double *grad_mu, double *grad_t,
                                           double *grad_beta, double *grad_freqs, double *out, double *out_sum,
                                           void *hip_stream) {
    return ami::hubbard_adjoint(t, k, n_e, stride_k, q, hop_t, mu, ext_freqs, n_f, beta, e_reg, grad_out, grad_sum,
                                grad_k, grad_mu, grad_t, grad_beta, grad_freqs, out, out_sum, hip_stream, true);
}

AmiStatus amiIntegrateHubbard(AmiTerms *t, int64_t n_samples, uint64_t seed, const double *q, double hop_t,
                              double mu, const double *ext_freqs, int64_t n_f, double beta, double e_reg,
                              double *sums, void *hip_stream) {
    using namespace ami;
    clear_error();
    AmiStatus st = check_common(t, n_samples, ext_freqs, n_f, beta);
    if (st != AMI_OK) return st;
    if (n_f > kMcMaxFreqs) return fail(AMI_E_ARG, "at most 8 frequency rows per Monte-Carlo call");
    if (!sums) return fail(AMI_E_ARG, "sums is NULL");
    if (t->n_eps != t->n_g) return fail(AMI_E_ARG, "the momentum path needs one energy per propagator");
    if (t->n_ext > 0 && !q) return fail(AMI_E_ARG, "q is NULL");
    const hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    DeviceTables *dt = nullptr;
    st = upload(t, &dt);
    if (st != AMI_OK) return st;
    if (jit_prefers_two_pass(t)) {
        // large solutions: the two-pass kernels, momenta drawn in the first
        void *f1 = nullptr, *f2 = nullptr;
        st = jit_get(t, true, kJitSumsPass, &f1);
        if (st == AMI_OK) st = jit_get(t, true, kJitFreqPass, &f2);
        if (st != AMI_OK) return st;
        if (n_samples == 0) return fill(sums, 4 * n_f, stream);
        KArgs a;
        std::memset(&a, 0, sizeof(a));
        set_momenta(a, t, nullptr, 0, q, hop_t, mu);
        set_common(a, ext_freqs, n_f, beta, e_reg, n_samples);
        a.seed = seed;
        a.mc = 1;
        return launch_two_pass(t, dt, true, a, sums, f1, f2, stream);
    }
    void *fn = nullptr;
    st = jit_get(t, true, kJitMonteCarlo, &fn);
    if (st != AMI_OK) return st;
    if (n_samples == 0) return fill(sums, 4 * n_f, stream);
    int dev = 0, n_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
    // a fixed grid per device (the sums are reduced in a fixed order for it):
    // eight blocks per CU, or fewer when there are fewer samples
    const int block = jit_block(t, true);
    const int64_t grid = std::min<int64_t>((n_samples + block - 1) / block, 8 * static_cast<int64_t>(n_cu));
    const int64_t rows = grid * (block / 64);   // partial sums per wave
    double *partial = nullptr;
    st = workspace(t, dt, stream, static_cast<size_t>(rows) * n_f * 4 * sizeof(double), &partial);
    if (st != AMI_OK) return st;
    KArgs a;
    std::memset(&a, 0, sizeof(a));
    set_momenta(a, t, nullptr, 0, q, hop_t, mu);
    set_common(a, ext_freqs, n_f, beta, e_reg, n_samples);
    a.seed = seed;
    a.partial = partial;
    a.nrows = rows;
    e = launch_jit(fn, grid, block, stream, a);
    if (e == hipSuccess) e = hipGetLastError();
    g_last_variant = "specialized";
    if (e != hipSuccess) return hip_fail(e, "Monte-Carlo launch");
    hipLaunchKernelGGL(ami_colsum_kernel, dim3(static_cast<unsigned>(4 * n_f)), dim3(kRedThreads), 0, stream, partial,
                       rows, static_cast<int64_t>(1), rows, sums);
    e = hipGetLastError();
    return e == hipSuccess ? AMI_OK : hip_fail(e, "Monte-Carlo reduction launch");
}

AmiStatus amiSetTwoPassChunkBytes(int64_t bytes) {
    ami::clear_error();
    if (bytes < (int64_t(1) << 16)) return ami::fail(AMI_E_ARG, "the chunk bound must be at least 64 KiB");
    ami::g_two_pass_chunk_bytes.store(bytes);
    return AMI_OK;
}

AmiStatus amiSetVariant(AmiTerms *t, int32_t variant) {
    ami::clear_error();
    if (!t) return ami::fail(AMI_E_ARG, "terms is NULL");
    if (variant < AMI_VARIANT_AUTO || variant > AMI_VARIANT_TWO_PASS)
        return ami::fail(AMI_E_ARG, "variant must be one of AMI_VARIANT_*");
    t->variant = variant;
    ami::specialize_variant(t);
    return AMI_OK;
}

AmiStatus amiTermsSpecialize(AmiTerms *t, int32_t momentum) {
    ami::clear_error();
    if (!t) return ami::fail(AMI_E_ARG, "terms is NULL");
    using namespace ami;
    const bool hub = momentum != 0;
    std::vector<int> kinds = kernels_of(t, hub, AMI_VARIANT_AUTO);
    for (int k : kernels_of(t, hub, t->variant))
        if (std::find(kinds.begin(), kinds.end(), k) == kinds.end()) kinds.push_back(k);
    // all compiled before any device is touched
    for (int k : kinds) {
        const AmiStatus st = jit_compile(t, hub, k);
        if (st != AMI_OK) return st;
    }
    for (int k : kinds) {
        void *fn = nullptr;
        const AmiStatus st = jit_get(t, hub, k, &fn);
        if (st != AMI_OK) return st;
    }
    t->specialized[hub ? 1 : 0].store(true);
    return AMI_OK;
}

const char *amiLastVariant(void) { return ami::g_last_variant.c_str(); }

AmiStatus amiKernelTimerStart(int32_t capacity) {
    using namespace ami;
    clear_error();
    if (capacity < 1 || capacity > (1 << 20)) return fail(AMI_E_ARG, "capacity must be in 1..2^20");
    if (g_timer.on) return fail(AMI_E_ARG, "the kernel timer is already running on this thread");
    g_timer.ev.assign(2 * static_cast<size_t>(capacity), nullptr);
    for (size_t i = 0; i < g_timer.ev.size(); ++i) {
        const hipError_t e = hipEventCreate(&g_timer.ev[i]);
        if (e != hipSuccess) {
            for (size_t j = 0; j < i; ++j) (void)hipEventDestroy(g_timer.ev[j]);
            g_timer.ev.clear();
            return hip_fail(e, "hipEventCreate");
        }
    }
    g_timer.used = 0;
    g_timer.on = true;
    return AMI_OK;
}

AmiStatus amiKernelTimerStop(float *ms, int32_t cap, int32_t *count) {
    using namespace ami;
    clear_error();
    if (!g_timer.on) return fail(AMI_E_ARG, "the kernel timer is not running on this thread");
    AmiStatus st = AMI_OK;
    int n = 0;
    for (int i = 0; i < g_timer.used; ++i) {
        hipError_t e = hipEventSynchronize(g_timer.ev[2 * i + 1]);
        float v = 0.0f;
        if (e == hipSuccess) e = hipEventElapsedTime(&v, g_timer.ev[2 * i], g_timer.ev[2 * i + 1]);
        if (e != hipSuccess) {
            st = hip_fail(e, "kernel timer events");
            break;
        }
        if (ms && n < cap) ms[n] = v;
        ++n;
    }
    for (hipEvent_t ev : g_timer.ev) (void)hipEventDestroy(ev);
    g_timer.ev.clear();
    g_timer.used = 0;
    g_timer.on = false;
    if (count) *count = n;
    return st;
}

}  // extern "C"
