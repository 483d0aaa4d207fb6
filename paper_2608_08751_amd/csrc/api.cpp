// C ABI of the gfx950 IVF routing / construction library (declared in
// include/ivf.h). Validates arguments, sizes and carves the caller's
// workspace, and enqueues the kernels on the context's stream. No call
// synchronises with the host except ivf_sync and ivf_last_stats.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "ivf.h"
#include "ivf_internal.h"

using namespace ivf;

struct ivf_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    int num_cus = 1;
    void *ws = nullptr;
    size_t ws_bytes = 0;
    std::string err;
    int force_fallback = 0;
    int sample_rank = 0;
    int build_blocks = 0;
    int screen_waves = 8;
    int fp32_screen = 0;  // 1: uint8 rows also take the fp32 MFMA screen
    int two_plane_only = 0;  // 1: no single-plane int8 pre-screen
    int s1_id_order = 0;     // 1: the single plane visits centroids in id order
    int force_rescreen = 0;  // 1: the single-plane screen lists every row
    int64_t rescreen_cap = 0;  // > 0: smaller capacity of that list (tests)
    int64_t assign_slice = 0;  // > 0: shorter assignment slices (tests)
    unsigned long long *last_stats = nullptr;  // device, inside the workspace
    int64_t last_sample = 0;
    // kernel timing (IVF_OPT_PROFILE): an event pair per launch of the last call
    int profile = 0;
    std::vector<hipEvent_t> events;
    std::vector<std::string> knames;
    std::vector<std::string> retired;  // names handed out by the last read
    size_t kused = 0;
    const char *cur_call = "";
    ~ivf_ctx()
    {
        for (hipEvent_t e : events) (void)hipEventDestroy(e);
    }
};

namespace {

constexpr size_t kAlign = 256;
constexpr int64_t kRouteBatch = 16384;
constexpr int64_t kDirectMaxQ = 32;
constexpr int kMaxNprobe = 1024;
constexpr int kMaxD = 256;
constexpr int kMaxHops = 1024;  // greedy moves of ivf_assign_cells
// Rows per assignment slice (row ids inside a slice fit int32).
constexpr int64_t kAssignSlice = (int64_t)1 << 28;

// Scratch memory of ivf_route_noalloc, for callers that cannot allocate
// device memory: one copy per device, held while the library is loaded. In
// host code `scratch` names a host-side stand-in; kernels get the device
// address that hipGetSymbolAddress returns for each device.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Looks up (once per device, with that device current) the device address of
// `scratch`; nullptr on failure.
void *static_scratch(int device)
{
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int prev = -1;
        if (hipGetDevice(&prev) != hipSuccess) return nullptr;
        if (prev != device && hipSetDevice(device) != hipSuccess) return nullptr;
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (prev != device) (void)hipSetDevice(prev);
        if (e != hipSuccess) return nullptr;
        g_scratch_ptr[device] = ptr;
    }
    return g_scratch_ptr[device];
}

ivf_status fail(ivf_ctx *ctx, ivf_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (ctx) ctx->err = buf;
    return st;
}

// Bump allocator over the workspace (base == nullptr: sizing only).
struct Carver {
    char *base;
    size_t off = 0;
    explicit Carver(void *b) : base((char *)b) {}
    template <typename T> T *take(size_t count)
    {
        off = (off + kAlign - 1) / kAlign * kAlign;
        T *p = base ? (T *)(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

// Workspace of ivf_adc_scan for B queries, P probes, handoff k (layout only
// when base is null); returns the bytes used.
size_t layout_adc(void *base, int64_t B, int64_t P, int64_t k, AdcScratch *w)
{
    Carver c(base);
    AdcScratch s;
    s.handoff = c.take<uint64_t>((size_t)B * 2 * P * k);
    s.hcnt = c.take<int32_t>((size_t)B * 2 * P);
    s.dl = c.take<int32_t>((size_t)B * 2 * P);
    s.dpos = c.take<longlong2>((size_t)B * 2 * P);
    s.gcnt = c.take<int32_t>((size_t)B);
    if (w) *w = s;
    return c.off + kAlign;
}

// Scalar area at the start of every workspace: [0] max centroid norm bits,
// [1] worklist counter, [2] nonzero when some centroid does not quantise for
// the int8 screen, [3] the same for its single plane, [4] the single plane's
// largest coordinate residual (float bits), [5] counter of the rows the
// single plane leaves to the two planes, [6] nonzero when
// the int8 planes do not take a routing call, [7] the
// single plane's largest residual norm (float bits), [8] counter of the rows
// with two candidates, [9] counter of the rows with too many, [10] and [11] see
// ScalarWord, then (from word 16) kNumStats uint64 counters.
struct Scalars {
    uint32_t *mc2_bits;
    uint32_t *wl_cnt;
    unsigned long long *stats;
};

Scalars take_scalars(Carver &c)
{
    uint32_t *p = c.take<uint32_t>(64);
    Scalars s;
    s.mc2_bits = p;
    s.wl_cnt = p ? p + 1 : nullptr;
    s.stats = p ? (unsigned long long *)(p + 16) : nullptr;
    return s;
}

int padded_dim(int D)
{
    static const int dps[] = {32, 64, 96, 128, 192, 256};
    for (int dp : dps)
        if (D <= dp) return dp;
    return 0;
}

// Padded dimension of the quantised centroids kept for the int8 screen (the
// largest when D is not a supported size: such calls fail validation anyway).
int quant_dim(int D)
{
    const int dp = padded_dim(D);
    return dp > 0 ? dp : 256;
}

double bound_coef(int DP)
{
    const double u = 0x1p-23;  // one fp32 ulp relative: covers any rounding mode
    const double n = DP + 2;
    return n * u / (1.0 - n * u);
}

int pow2_ceil(int64_t v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

struct RoutePlan {
    int64_t QB;   // queries per internal batch
    int64_t Cs;   // threshold sample size, 0 = none
    int64_t Ss;   // the sample: chunks j * Ss of kChunk centroids, j < Cs / kChunk
    int L;        // candidate capacity per query
    int rank_j;
    int qdp;      // padded dimension of the int8 and f16 route planes; 0 = fp32 kernels only
    int rank_safe, rank_max;  // f16 plane: see RouteArgs
    bool f16;     // the f16 plane is laid out for what the int8 planes do not take
};

// The f16 plane takes the queries that are not uint8-valued from 10 GFLOP per
// call on: building the plane and the filter's flushes cost 40-80 us however small the call,
// against 8 us per GFLOP on fp32 MFMA (1,656 queries on 20,438 x 64: 242 us in f16,
// 181 in fp32; 1,280 on 83,435 x 64: 157 and 214).
bool f16_route(int64_t Q, int64_t C, int D) { return 2.0 * (double)Q * (double)C * (double)D >= 1e10; }

RoutePlan plan_route(int64_t Q, int64_t C, int k, int rank_override, int D)
{
    RoutePlan p;
    p.QB = std::max<int64_t>(1, std::min<int64_t>(Q, kRouteBatch));
    p.qdp = quant_dim(D);
    p.f16 = C > 2048 && f16_route(Q, C, D);
    if (C <= 2048) {
        p.Cs = 0;
        p.Ss = 1;
        p.L = pow2_ceil(std::max<int64_t>(C, k));
        p.rank_j = 0;
        p.rank_safe = p.rank_max = 0;
        return p;
    }
    // sizes depend only on (Q, C, k); a rank override (a test knob) moves the
    // threshold but never the buffers, so ivf_workspace_bytes stays valid
    const int r = 32;
    const int64_t mu = std::max<int64_t>(4 * (int64_t)k, 256);
    int64_t f = mu / r;
    f = std::min<int64_t>(std::max<int64_t>(f, 4), 64);
    int64_t Cs = (C / f) / kChunk * kChunk;
    Cs = std::max<int64_t>(Cs, (int64_t)2 * r * 16);
    Cs = std::min<int64_t>(Cs, (C / 2) / kChunk * kChunk);
    Cs = std::min<int64_t>(Cs, 65536);
    Cs = std::max<int64_t>(Cs, kChunk);
    p.Cs = Cs;
    // spread over the table (a table sorted by position or by list would
    // bias a contiguous sample); Cs <= C / 2 gives a stride of at least 2
    p.Ss = (C / kChunk) / (Cs / kChunk);
    p.rank_j = (int)std::min<int64_t>(r, Cs / 16);
    const double expected = (double)p.rank_j * (double)C / (double)Cs;
    if (rank_override > 0) p.rank_j = (int)std::min<int64_t>(rank_override, Cs / 16);
    int L = pow2_ceil((int64_t)(2.5 * expected) + 1);
    L = std::max(L, std::max(512, pow2_ceil(k)));
    p.L = std::min(L, 4096);
    // the k-th smallest key has sample rank k Cs / C on average: five standard
    // deviations above that are safe; up to three quarters of a candidate list
    // are expected below the last minimum the f16 window may reach
    const double rk = (double)k * (double)Cs / (double)C;
    p.rank_safe = (int)std::min<double>(r - 1, ceil(rk + 5.0 * sqrt(rk) + 3.0));
    p.rank_max = (int)std::min<double>(64, floor(0.75 * p.L * (double)Cs / (double)C));
    p.rank_max = std::max(p.rank_max, r);
    return p;
}

struct RouteLayout {
    Scalars sc;
    float *cnorm;
    double *qn2;
    float *tau;
    uint32_t *cand_cnt;
    uint2 *cand;
    float *keys;
    float *kmin;
    int32_t *wl;
    // int8 route planes (plan.qdp > 0): two planes [quantized_pad(C)][2 qdp],
    // biases, per-query bounds
    int8_t *qc;
    int32_t *negb;
    float *qbound;
    size_t bytes;
};

RouteLayout layout_route(void *base, const RoutePlan &p, int64_t C)
{
    Carver c(base);
    RouteLayout l;
    l.sc = take_scalars(c);
    l.cnorm = c.take<float>(C);
    l.qn2 = c.take<double>(p.QB);
    l.tau = c.take<float>(p.QB);
    l.cand_cnt = c.take<uint32_t>(p.QB);
    l.cand = c.take<uint2>((size_t)p.QB * p.L);
    l.keys = c.take<float>((size_t)p.QB * p.Cs);
    l.kmin = c.take<float>((size_t)p.QB * (p.Cs / 16));
    l.wl = c.take<int32_t>(p.QB);
    l.qc = nullptr;
    l.negb = nullptr;
    l.qbound = nullptr;
    if (p.qdp > 0) {
        // the two int8 planes or the f16 plane: one call uses one of them
        const int64_t pad = p.f16 ? quantized_pad1(C) : quantized_pad(C);
        l.qc = c.take<int8_t>((size_t)pad * 2 * p.qdp);
        l.negb = c.take<int32_t>(pad);
        l.qbound = c.take<float>(p.QB);
    }
    l.bytes = c.off + kAlign;
    return l;
}

// The direct route (two launches: every key, then one workgroup per query)
// in place of sample, threshold, filter, select and fallback (up to 16
// launches of 3-5 us each, most of them idle on any one call): tables small
// enough to be candidates whole, at any number of queries, and the smallest
// batches on tables of up to kDirectMaxC centroids, whose key matrix fits
// where the planes would lie (D / 2 queries). Past half a workgroup of
// neighbours (k > 512) every key of a large table would have to enter the
// selection. Measured against the general path: 1,000 queries on 1,024 x 128
// 25 us instead of 61, 16,384 on 2,048 x 128 403 instead of 657, one query on
// 65,536 x 128 46 instead of 88, 32 queries 53 instead of 101.
bool direct_route(const RoutePlan &p, int64_t Q, int64_t C, int k)
{
    if (p.Cs == 0) return true;
    return C <= kDirectMaxC && k <= 512 && Q <= p.QB && Q <= kDirectMaxQ && 2 * Q <= p.qdp;
}

// fp32 rows are screened on f16 where the table is long enough that a tile's
// scan of it, or the call large enough that the whole, outweighs the four more
// launches (5 us each): 300 rows x 100 x 32 60 us in f16 and 45 on fp32 MFMA alone,
// 3,000 x 300 x 96 102-121 and 98-104, 50,000 x 50 x 64 60-82 and 44-67; 5,000 x 500 x
// 64 104 and 104, 1,000 x 1,000 x 64 108 and 132, 20,000 x 500 x 128 134 and 157.
bool f16_assign(int64_t N, int64_t C, int D, int DP)
{
    return C * DP >= 32000 || 2.0 * (double)N * (double)C * (double)D >= 8e8;
}

int64_t worklist_cap(int64_t N) { return std::min<int64_t>(N, 4096 + N / 64); }
// Rows a one-pass screen may list before the next screen takes every row: a
// quarter of a call of up to 2^24 rows (a 131,072 x 100 table of close centroids
// lists 16 %; past a quarter a full second screen costs about as much as
// collecting), 2^22 rows up to 2^26, a sixteenth past that: the lists' 48 bytes
// per entry would grow into gigabytes.
int64_t rescreen_cap(int64_t N)
{
    return std::min<int64_t>(N, 4096 + std::max<int64_t>(N / 16, std::min<int64_t>(N / 4, (int64_t)1 << 22)));
}
// two-candidate rows left to the resolving kernel (12 bytes each; more are
// decided inside the screen)
int64_t duel_cap(int64_t N)
{
    return std::min<int64_t>(N, 4096 + std::max<int64_t>(N / 8, std::min<int64_t>(N / 2, (int64_t)1 << 23)));
}

struct AssignLayout {
    Scalars sc;
    float *cnorm;
    // quantised centroids of the int8 screen (uint8 rows)
    int8_t *qc;
    int32_t *negb;
    // single plane (padded dimension <= 128) and the rows it leaves
    int8_t *qc1;
    int32_t *negb1;
    // its visiting order: keys, column sums and mean, counting-sort scratch,
    // bucket counts and offsets, order (plane row -> id) and positions
    int32_t *okeys;
    double *opart;
    float *omean;
    void *oradix;
    int64_t *ocounts;
    int64_t *ooffsets;
    uint32_t *ord1;
    int32_t *pos1;
    int32_t *list;
    int64_t list_cap;
    ResolveLists rs;
    bool lean;
    int32_t *wl;
    int64_t wl_cap;
    double *fb_d;   // split fallback partial results
    int32_t *fb_i;
    // build
    uint32_t *cntmat;
    int64_t *counts;
    int64_t *offsets;
    uint32_t *perm;
    double *jpart;
    size_t bytes;
};

// Product-quantisation training step over M subspaces: labels [M][n], the
// list build of all subspaces' labels (256 lists each; block counts),
// counts [M][256], offsets [M][257], permutations [M][n] and the update's
// objective parts [M][256].
struct PqLayout {
    int32_t *labels;
    uint32_t *cnt;
    int64_t *counts;
    int64_t *offsets;
    uint32_t *perm;
    double *jpart;
    size_t bytes;
};

PqLayout layout_pq(void *base, int64_t n, int M, int num_cus)
{
    Carver c(base);
    PqLayout l{};
    l.labels = c.take<int32_t>((size_t)n * M);
    const size_t cnt = single_scratch_bytes(plan_single(n, kPqK, M, num_cus));
    const bool shared = cnt <= (size_t)kPqK * M * sizeof(double);  // the list build ends before the update begins
    if (!shared) l.cnt = c.take<uint32_t>(cnt / 4);
    l.counts = c.take<int64_t>((size_t)kPqK * M);
    l.offsets = c.take<int64_t>((size_t)(kPqK + 1) * M);
    l.perm = c.take<uint32_t>((size_t)n * M);
    l.jpart = c.take<double>((size_t)kPqK * M);
    if (shared) l.cnt = (uint32_t *)l.jpart;
    l.bytes = c.off;
    return l;
}

// need_lists: counts/offsets/perm live in the workspace (k-means step);
// need_build: count matrix for the list build; qdp > 0: quantised centroids
// of padded dimension qdp for the int8 screen.
// lean: without the f16 plane and the lists of rows to resolve (the fp32 screen
// takes fp32 rows, the two-plane screen the rows that the single plane leaves).
AssignLayout layout_assign(void *base, int64_t N, int64_t C, int qdp, bool need_build, bool need_lists,
                           int num_cus, bool lean = false)
{
    Carver c(base);
    AssignLayout l{};
    l.sc = take_scalars(c);
    l.cnorm = c.take<float>(C);
    if (qdp > 0) {
        // the two int8 planes (uint8 rows) or the f16 plane (fp32 rows)
        const int64_t pad = lean ? quantized_pad(C) : quantized_pad1(C);
        l.qc = c.take<int8_t>((size_t)pad * 2 * qdp);
        l.negb = c.take<int32_t>(pad);
        if (qdp <= 128) {
            l.qc1 = c.take<int8_t>((size_t)quantized_pad1(C) * qdp);
            l.negb1 = c.take<int32_t>(quantized_pad1(C));
            l.okeys = c.take<int32_t>(C);
            l.opart = c.take<double>((size_t)order1_parts(C) * qdp);
            l.omean = c.take<float>(qdp);
            l.oradix = c.take<unsigned char>(radix_scratch_bytes(plan_radix(C, kOrder1Keys, num_cus)));
            l.ocounts = c.take<int64_t>(kOrder1Keys);
            l.ooffsets = c.take<int64_t>(kOrder1Keys + 1);
            l.ord1 = c.take<uint32_t>(C);
            l.pos1 = c.take<int32_t>(C);
        }
        const int64_t n = std::min(N, kAssignSlice);
        l.lean = lean;
        if (!lean || qdp <= 128) {
            l.list_cap = lean ? std::min<int64_t>(n, 4096 + n / 16) : rescreen_cap(n);
            l.list = c.take<int32_t>(l.list_cap);
        }
        if (!lean) {
            l.rs.duel_cap = duel_cap(n);
            l.rs.duel = c.take<uint2>(l.rs.duel_cap);
            l.rs.duel2 = c.take<int32_t>(l.rs.duel_cap);
            l.rs.list_thr = c.take<int32_t>(l.list_cap);
            l.rs.cand_cnt = c.take<uint32_t>(l.list_cap);
            l.rs.cand = c.take<int32_t>((size_t)l.list_cap * kResolveCand);
            l.rs.list2 = c.take<int32_t>(l.list_cap);
            l.rs.duel_cnt = l.sc.mc2_bits ? l.sc.mc2_bits + 8 : nullptr;
            l.rs.list2_cnt = l.sc.mc2_bits ? l.sc.mc2_bits + 9 : nullptr;
        }
    }
    l.wl_cap = worklist_cap(std::min(N, kAssignSlice));
    l.wl = c.take<int32_t>(l.wl_cap);
    l.fb_d = c.take<double>(kFbSplitEntries);
    l.fb_i = c.take<int32_t>(kFbSplitEntries);
    if (need_build) {
        if (C <= kSingleMaxLists)
            l.cntmat = c.take<uint32_t>(single_scratch_bytes(plan_single(N, C, 1, num_cus)) / 4);
        else if (C <= kRadixMaxLists)
            l.cntmat = (uint32_t *)c.take<unsigned char>(radix_scratch_bytes(plan_radix(N, C, num_cus)));
        else
            l.cntmat = c.take<uint32_t>(build_scratch_bytes(plan_build(N, C, num_cus)) / 4);
    }
    if (need_lists) {
        l.counts = c.take<int64_t>(C);
        l.offsets = c.take<int64_t>(C + 1);
        l.perm = c.take<uint32_t>(N);
        l.jpart = c.take<double>(C);
    }
    l.bytes = c.off + kAlign;
    return l;
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    if (!a || !b || na == 0 || nb == 0) return false;
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + nb && b0 < a0 + na;
}

struct DeviceGuard {
    int prev = -1;
    bool ok = true;
    explicit DeviceGuard(int dev)
    {
        if (dev < 0) {  // validation-only context
            ok = false;
            return;
        }
        if (hipGetDevice(&prev) != hipSuccess) {
            ok = false;
            return;
        }
        if (prev != dev && hipSetDevice(dev) != hipSuccess) ok = false;
    }
    ~DeviceGuard()
    {
        int cur;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

// least: what the call can do with; need: what ivf_workspace_bytes asks for
ivf_status check_ws(ivf_ctx *ctx, size_t least, size_t need)
{
    if (!ctx->ws || ctx->ws_bytes < least)
        return fail(ctx, IVF_ENOMEM, "workspace too small: %zu bytes required, %zu provided", need,
                    ctx->ws ? ctx->ws_bytes : (size_t)0);
    return IVF_OK;
}
ivf_status check_ws(ivf_ctx *ctx, size_t need) { return check_ws(ctx, need, need); }

// The layout of an assignment with its list build in the context's workspace:
// lean when the whole one does not fit.
ivf_status fit_assign(ivf_ctx *ctx, int64_t N, int64_t C, int D, bool need_lists, AssignLayout &l)
{
    const int qdp = quant_dim(D), cus = ctx->num_cus;
    const size_t need = layout_assign(nullptr, N, C, qdp, true, need_lists, cus).bytes;
    const bool lean = ctx->ws_bytes < need;
    const size_t least = lean ? layout_assign(nullptr, N, C, qdp, true, need_lists, cus, true).bytes : need;
    const ivf_status st = check_ws(ctx, least, need);
    if (st == IVF_OK) l = layout_assign(ctx->ws, N, C, qdp, true, need_lists, cus, lean);
    return st;
}

#define HIP_TRY(expr)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return fail(ctx, IVF_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));  \
    } while (0)

// Drops the recorded kernel timeline.
void prof_reset(ivf_ctx *ctx) { ctx->kused = 0; ctx->knames.clear(); }

// Records the start event of a kernel launch; returns its slot or -1.
int prof_start(ivf_ctx *ctx, const char *name)
{
    if (!ctx->profile) return -1;
    const size_t i = ctx->kused++;
    while (ctx->events.size() < 2 * ctx->kused) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) {
            --ctx->kused;
            return -1;
        }
        ctx->events.push_back(e);
    }
    ctx->knames.push_back(std::string(ctx->cur_call) + "/" + name);
    (void)hipEventRecord(ctx->events[2 * i], ctx->stream);
    return (int)i;
}

void prof_stop(ivf_ctx *ctx, int slot)
{
    if (slot >= 0) (void)hipEventRecord(ctx->events[2 * slot + 1], ctx->stream);
}

// Launch with optional event timing around it.
#define TIMED(name, expr)                        \
    do {                                         \
        const int slot_ = prof_start(ctx, name); \
        HIP_TRY(expr);                           \
        prof_stop(ctx, slot_);                   \
    } while (0)

ivf_status check_common(ivf_ctx *ctx, int64_t C, int32_t D)
{
    if (C < 1) return fail(ctx, IVF_EINVAL, "C must be >= 1 (got %lld)", (long long)C);
    if (C > INT32_MAX) return fail(ctx, IVF_EUNSUPPORTED, "C must fit int32 ids");
    if (D < 4 || D > kMaxD || D % 4 != 0)
        return fail(ctx, IVF_EUNSUPPORTED, "D must be a multiple of 4 in [4, %d] (got %d)", kMaxD, D);
    return IVF_OK;
}

// Assignment of N rows (top-1 with certification and fallback) into labels.
// The centroid preparation (norms, quantised planes) runs once; the rows are
// then screened in slices of at most `slice` rows, each with its own
// worklists, so that the row ids the screens and the fallback pass around
// (int32, relative to the slice) stay below 2^31 for any N <= 2^32 - 1.
ivf_status enqueue_assign(ivf_ctx *ctx, const void *rows, int rowtype, int64_t N,
                          const float *cent, int64_t C, int D, int32_t *labels,
                          const AssignLayout &l, const int32_t *hint = nullptr)
{
    hipStream_t s = ctx->stream;
    const int DP = padded_dim(D);
    const size_t rb = (size_t)D * (rowtype == kRowU8 ? 1 : 4);
    const int64_t slice = ctx->assign_slice > 0 ? std::min<int64_t>(ctx->assign_slice, kAssignSlice) : kAssignSlice;
    TIMED("fill", launch_fill_u32(l.sc.mc2_bits, 64, 0u, s));
    TIMED("centroid_norms", launch_centroid_norms(cent, C, D, l.cnorm, l.sc.mc2_bits, s));
    const bool int8 = rowtype == kRowU8 && !ctx->fp32_screen;
    const bool f16 = rowtype == kRowF32 && !ctx->fp32_screen && !l.lean && f16_assign(N, C, D, DP);
    const bool single = int8 && l.qc1 && !ctx->two_plane_only;
    uint32_t *q_bad = l.sc.mc2_bits + 2;
    uint32_t *q_bad1 = l.sc.mc2_bits + 3;
    uint32_t *e_bits = l.sc.mc2_bits + 4;
    uint32_t *list_cnt = l.sc.mc2_bits + 5;
    uint32_t *r2_bits = l.sc.mc2_bits + 7;
    uint32_t *rc_bits = l.sc.mc2_bits + kWordF16Rc;
    const uint32_t *ord1 = nullptr;
    const int32_t *pos1 = nullptr;
    if (int8) {
        // int8 MFMA screens; the fp32 kernel runs only if some centroid does not quantise
        TIMED("quantize", launch_quantize_centroids(cent, C, D, DP, l.qc, l.negb, q_bad, s));
        if (single) {
            const bool ordered = !ctx->s1_id_order;
            if (ordered) {
                // the plane's visiting order: a stable counting sort of the
                // centroids by their distance bucket
                TIMED("order1_keys", launch_order1_keys(cent, C, D, l.opart, l.omean, l.okeys, s));
                const RadixPlan rp = plan_radix(C, kOrder1Keys, ctx->num_cus);
                const RadixScratch rs = carve_radix(rp, l.oradix);
                TIMED("order1_level0", launch_radix_level0(rp, l.okeys, rs, s));
                TIMED("order1_counts", launch_radix_level1_counts(rp, rs, l.ocounts, s));
                TIMED("order1_offsets", launch_offsets(l.ocounts, kOrder1Keys, l.ooffsets, s));
                TIMED("order1_scatter", launch_radix_level1_scatter(rp, rs, l.ooffsets, l.ord1, s));
            }
            TIMED("quantize1", launch_quantize_centroids1(cent, C, D, DP, l.qc1, l.negb1, q_bad1, e_bits, r2_bits,
                                                          s, ordered ? l.ord1 : nullptr, ordered ? l.pos1 : nullptr));
            ord1 = ordered ? l.ord1 : nullptr;
            pos1 = ordered ? l.pos1 : nullptr;
        }
    }
    uint16_t *plane16 = (uint16_t *)l.qc;
    float *bias16 = (float *)l.negb;
    if (f16) TIMED("quantize_f16", launch_quantize_f16(cent, C, D, DP, l.sc.mc2_bits, plane16, bias16, rc_bits, s));
    for (int64_t r0 = 0; r0 < N; r0 += slice) {
        const int64_t n = std::min(slice, N - r0);
        const void *xr = (const char *)rows + (size_t)r0 * rb;
        int32_t *lab = labels + r0;
        if (r0 > 0) {
            // the worklist and the single plane's list start empty for every slice
            TIMED("fill", launch_fill_u32(l.sc.wl_cnt, 1, 0u, s));
            if (single || f16) {
                TIMED("fill", launch_fill_u32(list_cnt, 1, 0u, s));
                if (!l.lean) TIMED("fill", launch_fill_u32(l.rs.duel_cnt, 2, 0u, s));
            }
        }
        ScreenArgs a{};
        a.rows = xr;
        a.nrows = n;
        a.D = D;
        a.cent = cent;
        a.cnorm = l.cnorm;
        a.c_begin = 0;
        a.c_end = C;
        a.nchunks = (C + kChunk - 1) / kChunk;
        a.mc2_bits = l.sc.mc2_bits;
        a.bound_coef = bound_coef(DP);
        a.labels = lab;
        a.wl = l.wl;
        a.wl_cnt = l.sc.wl_cnt;
        a.wl_cap = l.wl_cap;
        a.stats = l.sc.stats;
        a.force_fallback = ctx->force_fallback;
        auto resolve_args = [&](const ResolveLists &rs, int64_t cap, const uint32_t *ord) {
            ResolveArgs ra{};
            ra.rows = xr;
            ra.nrows = n;
            ra.D = D;
            ra.cent = cent;
            ra.C = C;
            ra.ord = ord;
            ra.list = l.list;
            ra.list_cnt = list_cnt;
            ra.list_cap = cap;
            ra.rs = rs;
            ra.labels = lab;
            return ra;
        };
        if (f16) {
            ScreenF16Args q{};
            q.rows = (const float *)xr;
            q.nrows = n;
            q.D = D;
            q.cent = cent;
            q.plane = plane16;
            q.nbias = bias16;
            q.mc2_bits = l.sc.mc2_bits;
            q.rc_bits = rc_bits;
            q.acc_coef = f16_acc_coef(DP);
            q.ncent = C;
            q.cpad = quantized_pad1(C);
            q.labels = lab;
            q.stats = l.sc.stats;
            q.list = l.list;
            q.list_cnt = list_cnt;
            q.list_cap = ctx->rescreen_cap > 0 ? std::min<int64_t>(ctx->rescreen_cap, l.list_cap) : l.list_cap;
            q.rs = l.rs;
            // a forced fallback passes every row on to the fp32 screen, which sends it on
            q.force_list = ctx->force_rescreen || ctx->force_fallback;
            const bool collect = !q.force_list && ctx->rescreen_cap == 0;
            if (!collect) q.rs.list_thr = nullptr;
            TIMED("screen_top1_f16", launch_screen_f16(DP, q, ctx->num_cus, s));
            if (collect) TIMED("collect_f16", launch_collect_f16(DP, q, ctx->num_cus, s));
            TIMED("resolve", launch_resolve(rowtype, resolve_args(q.rs, q.list_cap, nullptr), ctx->num_cus, s));
            a.list = l.list;
            a.list_cnt = list_cnt;
            a.list_cap = q.list_cap;
            a.rs = q.rs;
        }
        if (int8) {
            ScreenI8Args q{};
            q.rows = (const uint8_t *)xr;
            q.nrows = n;
            q.D = D;
            q.cent = cent;
            q.qc = l.qc;
            q.negb = l.negb;
            q.cpad = quantized_pad(C);
            q.nchunks = q.cpad / 64;
            q.q_bad = q_bad;
            q.labels = lab;
            q.wl = l.wl;
            q.wl_cnt = l.sc.wl_cnt;
            q.wl_cap = l.wl_cap;
            q.stats = l.sc.stats;
            q.force_fallback = ctx->force_fallback;
            q.ncent = C;
            if (single) {
                // single plane first; the two planes then screen the rows it leaves
                q.qc1 = l.qc1;
                q.negb1 = l.negb1;
                q.e_bits = e_bits;
                q.r2_bits = r2_bits;
                q.q_bad1 = q_bad1;
                q.list = l.list;
                q.list_cnt = list_cnt;
                q.list_cap = ctx->rescreen_cap > 0 ? std::min<int64_t>(ctx->rescreen_cap, l.list_cap) : l.list_cap;
                // a forced fallback passes every row on to the two planes, which send it on
                q.force_rescreen = ctx->force_rescreen || ctx->force_fallback;
                q.hint = hint ? hint + r0 : nullptr;
                q.ord1 = ord1;
                q.pos1 = pos1;
                // near ties: decided from collected candidates (a forced
                // rescreen or a test's list capacity keeps the two-plane
                // screen of the listed rows)
                const bool collect = !q.force_rescreen && ctx->rescreen_cap == 0 && !l.lean;
                q.rs = l.rs;
                if (!collect) q.rs.list_thr = nullptr;
                TIMED("screen_top1_i8s", launch_screen_i8_single(DP, q, ctx->num_cus, s));
                if (collect) TIMED("collect_i8", launch_collect_i8(DP, q, ctx->num_cus, s));
                if (!l.lean)
                    TIMED("resolve", launch_resolve(rowtype, resolve_args(q.rs, q.list_cap, ord1), ctx->num_cus, s));
            }
            TIMED("screen_top1_i8", launch_screen_i8(DP, q, ctx->num_cus, s));
            a.gate = q_bad;
        }
        TIMED("screen_top1", launch_screen(kModeTop1, rowtype, DP, a, ctx->screen_waves, ctx->num_cus, s));
        TIMED("assign_fallback", launch_assign_fallback(xr, rowtype, n, D, cent, C, lab, l.wl, l.sc.wl_cnt,
                                                        l.wl_cap, l.fb_d, l.fb_i, 2 * ctx->num_cus, s));
    }
    ctx->last_stats = l.sc.stats;
    ctx->last_sample = 0;
    return IVF_OK;
}

// List build: one partition by the label for C <= 256 lists, the two-level
// radix partition for C <= 65,536, the single-pass per-block build otherwise.
// `scratch` is the build area of the workspace.
ivf_status enqueue_build(ivf_ctx *ctx, int64_t N, int64_t C, const int32_t *labels, void *scratch,
                         int64_t *counts, int64_t *offsets, uint32_t *perm)
{
    if (C <= kRadixMaxLists) {
        if (N == 0) {
            TIMED("fill", launch_fill_u32((uint32_t *)counts, 2 * C, 0u, ctx->stream));
            TIMED("build_offsets", launch_offsets(counts, C, offsets, ctx->stream));
            return IVF_OK;
        }
        if (C <= kSingleMaxLists) {
            TIMED("build_single", launch_single_build(plan_single(N, C, 1, ctx->num_cus), labels, (uint32_t *)scratch,
                                                      counts, offsets, perm, ctx->stream));
            return IVF_OK;
        }
        const RadixPlan rp = plan_radix(N, C, ctx->num_cus);
        const RadixScratch rs = carve_radix(rp, scratch);
        TIMED("build_level0", launch_radix_level0(rp, labels, rs, ctx->stream));
        TIMED("build_level1_counts", launch_radix_level1_counts(rp, rs, counts, ctx->stream));
        TIMED("build_offsets", launch_offsets(counts, C, offsets, ctx->stream));
        TIMED("build_level1_scatter", launch_radix_level1_scatter(rp, rs, offsets, perm, ctx->stream));
        return IVF_OK;
    }
    const BuildPlan bp = plan_build(N, C, ctx->num_cus, ctx->build_blocks);
    uint32_t *cntmat = (uint32_t *)scratch;
    TIMED("build_hist", launch_build_hist(bp, labels, cntmat, ctx->stream));
    TIMED("build_scan", launch_build_scan(bp, cntmat, counts, offsets, ctx->stream));
    TIMED("build_scatter", launch_build_scatter(bp, labels, cntmat, offsets, perm, ctx->stream));
    return IVF_OK;
}

}  // namespace

extern "C" {

ivf_status ivf_create(int device, void *hip_stream, ivf_ctx **out)
{
    if (!out) return IVF_EINVAL;
    *out = nullptr;
    if (device == -1) {  // validation-only context: checks arguments, enqueues nothing
        ivf_ctx *c = new ivf_ctx();
        c->device = -1;
        c->num_cus = 256;
        *out = c;
        return IVF_OK;
    }
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess) return IVF_EDEVICE;
    if (device < 0 || device >= n) return IVF_EINVAL;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) return IVF_EDEVICE;
    // the static scratch of ivf_route_noalloc: its address on this device
    if (!static_scratch(device)) return IVF_EDEVICE;
    ivf_ctx *c = new ivf_ctx();
    c->device = device;
    c->stream = (hipStream_t)hip_stream;
    c->num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 1;
    *out = c;
    return IVF_OK;
}

void ivf_destroy(ivf_ctx *ctx) { delete ctx; }

const char *ivf_last_error(const ivf_ctx *ctx) { return ctx ? ctx->err.c_str() : "null context"; }

ivf_status ivf_set_stream(ivf_ctx *ctx, void *hip_stream)
{
    if (!ctx) return IVF_EINVAL;
    ctx->stream = (hipStream_t)hip_stream;
    return IVF_OK;
}

size_t ivf_workspace_bytes(int op, int64_t rows, int64_t C, int32_t D, int32_t k)
{
    if (C < 1 || rows < 0) return 0;
    int num_cus = 256;
    int dev;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess &&
        prop.multiProcessorCount > 0)
        num_cus = prop.multiProcessorCount;
    switch (op) {
    case IVF_OP_ROUTE:
        if (k < 1) return 0;
        return layout_route(nullptr, plan_route(rows, C, k, 0, D), C).bytes;
    case IVF_OP_KMEANS_STEP:
        return layout_assign(nullptr, std::max<int64_t>(rows, 1), C, quant_dim(D), true, true, num_cus).bytes;
    case IVF_OP_ASSIGN_BUILD:
        return layout_assign(nullptr, std::max<int64_t>(rows, 1), C, quant_dim(D), true, false, num_cus).bytes;
    case IVF_OP_BUILD_LISTS:
        return layout_assign(nullptr, std::max<int64_t>(rows, 1), C, 0, true, false, num_cus).bytes;
    case IVF_OP_ADC_SCAN:  // rows = B, C = P (probes per query), k = handoff
        if (k < 1 || k > kAdcMaxK || C < 1 || C > kMaxAdcProbes) return 0;
        return layout_adc(nullptr, rows, C, k, nullptr);
    case IVF_OP_PQ_TRAIN_STEP:  // C = M
        if (C > kMaxD) return 0;
        return layout_pq(nullptr, std::max<int64_t>(rows, 1), (int)C, num_cus).bytes;
    default:
        return 0;
    }
}

ivf_status ivf_set_workspace(ivf_ctx *ctx, void *dev_ptr, size_t bytes)
{
    if (!ctx) return IVF_EINVAL;
    if (dev_ptr && ((uintptr_t)dev_ptr % kAlign) != 0)
        return fail(ctx, IVF_EINVAL, "workspace must be %zu-byte aligned", kAlign);
    ctx->ws = dev_ptr;
    ctx->ws_bytes = dev_ptr ? bytes : 0;
    return IVF_OK;
}

ivf_status ivf_sync(ivf_ctx *ctx)
{
    if (!ctx) return IVF_EINVAL;
    if (ctx->device < 0) return IVF_OK;
    DeviceGuard g(ctx->device);
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return fail(ctx, IVF_EDEVICE, "device error: %s", hipGetErrorString(e));
    return IVF_OK;
}

ivf_status ivf_set_option(ivf_ctx *ctx, int option, int64_t value)
{
    if (!ctx) return IVF_EINVAL;
    switch (option) {
    case IVF_OPT_FORCE_FALLBACK: ctx->force_fallback = value ? 1 : 0; return IVF_OK;
    case IVF_OPT_SAMPLE_RANK:
        if (value < 0 || value > 4096) return fail(ctx, IVF_EINVAL, "sample rank out of range");
        ctx->sample_rank = (int)value;
        return IVF_OK;
    case IVF_OPT_PROFILE: ctx->profile = value ? 1 : 0; return IVF_OK;
    case IVF_OPT_SCREEN_WAVES:
        if (value != 4 && value != 8) return fail(ctx, IVF_EINVAL, "screen waves must be 4 or 8");
        ctx->screen_waves = (int)value;
        return IVF_OK;
    case IVF_OPT_FP32_SCREEN: ctx->fp32_screen = value ? 1 : 0; return IVF_OK;
    case IVF_OPT_I8_TWO_PLANE_ONLY: ctx->two_plane_only = value ? 1 : 0; return IVF_OK;
    case IVF_OPT_FORCE_RESCREEN: ctx->force_rescreen = value ? 1 : 0; return IVF_OK;
    case IVF_OPT_RESCREEN_CAP:
        if (value < 0) return fail(ctx, IVF_EINVAL, "rescreen capacity must be >= 0");
        ctx->rescreen_cap = value;
        return IVF_OK;
    case IVF_OPT_S1_ID_ORDER: ctx->s1_id_order = value ? 1 : 0; return IVF_OK;
    case IVF_OPT_ASSIGN_SLICE:
        if (value < 0) return fail(ctx, IVF_EINVAL, "assignment slice must be >= 0");
        ctx->assign_slice = value;
        return IVF_OK;
    case IVF_OPT_BUILD_BLOCKS:
        if (value < 0 || value > 65536) return fail(ctx, IVF_EINVAL, "build blocks out of range");
        ctx->build_blocks = (int)value;
        return IVF_OK;
    default: return fail(ctx, IVF_EINVAL, "unknown option %d", option);
    }
}

ivf_status ivf_last_stats(ivf_ctx *ctx, int64_t out[8])
{
    if (!ctx || !out) return IVF_EINVAL;
    for (int i = 0; i < 8; ++i) out[i] = 0;
    if (!ctx->last_stats) return IVF_OK;
    DeviceGuard g(ctx->device);
    unsigned long long h[kNumStats];
    HIP_TRY(hipMemcpyAsync(h, ctx->last_stats, sizeof h, hipMemcpyDeviceToHost, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    for (int i = 0; i < 8; ++i) out[i] = (int64_t)h[i];
    out[kStatSample] = ctx->last_sample;
    return IVF_OK;
}

int ivf_kernel_times(ivf_ctx *ctx, int max, const char **names, float *ms)
{
    if (!ctx || max < 0) return -1;
    if (ctx->device < 0) return 0;
    DeviceGuard g(ctx->device);
    if (hipStreamSynchronize(ctx->stream) != hipSuccess) return -1;
    const int n = (int)ctx->kused;
    for (int i = 0; i < n && i < max; ++i) {
        if (names) names[i] = ctx->knames[i].c_str();
        if (ms) {
            float t = 0.f;
            if (hipEventElapsedTime(&t, ctx->events[2 * i], ctx->events[2 * i + 1]) != hipSuccess) t = -1.f;
            ms[i] = t;
        }
    }
    if (max > 0 && max >= n) {
        // every entry delivered: start a new timeline (names stay valid until
        // the next recorded launch)
        ctx->kused = 0;
        ctx->retired.swap(ctx->knames);
        ctx->knames.clear();
    }
    return n;
}

}  // extern "C"

namespace {

// Times one probe launch (after an untimed one that loads the kernel) and
// reports its duration and rate in units of 1e12 operations per second.
ivf_status run_probe(ivf_ctx *ctx, int32_t iters, hipError_t (*launch)(int, int, hipStream_t, double *),
                     const char *what, float *out_ms, double *out_rate)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    if (iters < 1 || iters > (1 << 20)) return fail(ctx, IVF_EINVAL, "iters must be in [1, 2^20]");
    if (!out_ms && !out_rate) return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (ctx->device < 0) return fail(ctx, IVF_EUNSUPPORTED, "validation-only context");
    DeviceGuard g(ctx->device);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return fail(ctx, IVF_EDEVICE, "hipEventCreate failed");
    }
    double ops = 0.0;
    float ms = 0.f;
    hipError_t e = launch(1, ctx->num_cus, ctx->stream, &ops);
    if (e == hipSuccess) e = hipEventRecord(e0, ctx->stream);
    if (e == hipSuccess) e = launch(iters, ctx->num_cus, ctx->stream, &ops);
    if (e == hipSuccess) e = hipEventRecord(e1, ctx->stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) return fail(ctx, IVF_EDEVICE, "%s: %s", what, hipGetErrorString(e));
    if (out_ms) *out_ms = ms;
    if (out_rate) *out_rate = ms > 0.f ? ops / (ms * 1e-3) / 1e12 : 0.0;
    return IVF_OK;
}

}  // namespace

extern "C" {

ivf_status ivf_mfma_probe(ivf_ctx *ctx, int32_t iters, float *out_ms, double *out_tflops)
{
    return run_probe(ctx, iters, launch_mfma_probe, "fp32 MFMA probe", out_ms, out_tflops);
}

ivf_status ivf_mfma_probe_i8(ivf_ctx *ctx, int32_t iters, float *out_ms, double *out_tops)
{
    return run_probe(ctx, iters, launch_mfma_probe_i8, "int8 MFMA probe", out_ms, out_tops);
}

}  // extern "C"

namespace {

// Argument checks shared by ivf_route and ivf_route_noalloc (nothing is
// enqueued). *done is set when Q == 0 (a no-op).
ivf_status check_route(ivf_ctx *ctx, const float *queries, int64_t Q, const float *centroids, int64_t C,
                       int32_t D, int32_t nprobe, int32_t *out_ids, float *out_dist, bool *done)
{
    *done = false;
    if (Q < 0) return fail(ctx, IVF_EINVAL, "Q must be >= 0");
    ivf_status st = check_common(ctx, C, D);
    if (st != IVF_OK) return st;
    if (nprobe < 1 || nprobe > C)
        return fail(ctx, IVF_EINVAL, "nprobe must be in [1, C] (got %d, C = %lld)", nprobe, (long long)C);
    if (nprobe > kMaxNprobe) return fail(ctx, IVF_EUNSUPPORTED, "nprobe > %d", kMaxNprobe);
    if (Q == 0) {
        *done = true;
        return IVF_OK;
    }
    if (!queries || !centroids || !out_ids) return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(queries) || !aligned16(centroids) || !aligned16(out_ids) ||
        (out_dist && !aligned16(out_dist)))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const size_t qb = (size_t)Q * D * 4, cb = (size_t)C * D * 4, ob = (size_t)Q * nprobe * 4;
    if (overlap(out_ids, ob, queries, qb) || overlap(out_ids, ob, centroids, cb) ||
        overlap(out_dist, ob, queries, qb) || overlap(out_dist, ob, centroids, cb) ||
        overlap(out_ids, ob, out_dist, ob))
        return fail(ctx, IVF_EINVAL, "outputs overlap inputs or each other");
    return IVF_OK;
}

// Enqueues the routing kernels, queries in batches of p.QB, with the scratch
// memory laid out by layout_route at `ws`.
ivf_status enqueue_route(ivf_ctx *ctx, const float *queries, int64_t Q, const float *centroids, int64_t C,
                         int32_t D, int32_t nprobe, int32_t *out_ids, float *out_dist, const RoutePlan &p,
                         void *ws)
{
    const RouteLayout l = layout_route(ws, p, C);
    hipStream_t s = ctx->stream;
    const int DP = padded_dim(D);
    if (direct_route(p, Q, C, nprobe)) {
        for (int64_t q0 = 0; q0 < Q; q0 += p.QB) {
            DirectArgs a{};
            a.queries = queries + q0 * D;
            a.nq = std::min(p.QB, Q - q0);
            a.cent = centroids;
            a.C = C;
            a.D = D;
            a.k = nprobe;
            // no planes and no candidate lists are in use: a list's L pairs
            // hold the row's 2L >= C keys, and 2 Q <= qdp rows fit the planes
            a.keys = p.Cs == 0 ? (float *)l.cand : (float *)l.qc;
            a.stride = p.Cs == 0 ? 2 * (int64_t)p.L : (C + 3) / 4 * 4;
            a.mc2_part = l.cnorm;
            a.zero = q0 == 0 ? l.sc.mc2_bits : nullptr;
            const uint64_t total = (uint64_t)Q * (uint64_t)C;
            a.total_word = (int)((uint32_t *)(l.sc.stats + kStatCandidates) - l.sc.mc2_bits);
            a.total_lo = (uint32_t)total;
            a.total_hi = (uint32_t)(total >> 32);
            a.bound_coef = bound_coef(DP);
            a.force_fallback = ctx->force_fallback;
            a.out_ids = out_ids + q0 * nprobe;
            a.out_dist = out_dist ? out_dist + q0 * nprobe : nullptr;
            a.stats = l.sc.stats;
            TIMED("direct_keys", launch_direct_keys(DP, a, s));
            TIMED("direct_select", launch_direct_select(a, s));
        }
        ctx->last_stats = l.sc.stats;
        ctx->last_sample = 0;
        return IVF_OK;
    }
    TIMED("fill", launch_fill_u32(l.sc.mc2_bits, 64, 0u, s));
    TIMED("centroid_norms", launch_centroid_norms(centroids, C, D, l.cnorm, l.sc.mc2_bits, s));
    // uint8-valued queries are routed on the two int8 planes, other queries on
    // the f16 plane; the fp32 kernels run instead (device words, no host
    // synchronisation) when a centroid does not fit the int8 planes or the f16
    // window is too wide.
    const bool planes = p.qdp > 0 && !ctx->fp32_screen;
    const bool f16 = planes && p.f16;
    uint32_t *w = l.sc.mc2_bits;
    if (planes) {
        TIMED("route_i8_check", launch_route_i8_check(queries, Q, D, w + kWordNotI8, s));
        TIMED("quantize", launch_quantize_centroids(centroids, C, D, p.qdp, l.qc, l.negb, w + kWordQBad, s,
                                                    w + kWordNotI8, f16 ? w : nullptr));
    }
    for (int64_t q0 = 0; q0 < Q; q0 += p.QB) {
        const int64_t nb = std::min(p.QB, Q - q0);
        const float *qrows = queries + q0 * D;
        TIMED("route_bound", launch_route_i8_bound(qrows, nb, D, planes ? w + kWordQBad : nullptr,
                                                   planes ? w + kWordNotI8 : nullptr, planes ? l.qbound : nullptr, s,
                                                   w, f16 || !planes ? f16_acc_coef(DP) : -1.0, l.qn2));
        ScreenArgs a{};
        a.rows = qrows;
        a.nrows = nb;
        a.D = D;
        a.cent = centroids;
        a.cnorm = l.cnorm;
        a.route_w = planes ? w : nullptr;
        RouteI8Args ra{};
        ra.queries = qrows;
        ra.nq = nb;
        ra.D = D;
        ra.qc = l.qc;
        ra.negb = l.negb;
        ra.cpad = quantized_pad(C);
        ra.off = w + kWordNotI8;
        ra.stats = l.sc.stats;
        RouteF16Args rf{};
        rf.queries = qrows;
        rf.nq = nb;
        rf.D = D;
        rf.plane = (const uint16_t *)l.qc;
        rf.nbias = (const float *)l.negb;
        rf.mc2_bits = l.sc.mc2_bits;
        rf.w = w;
        rf.cpad = quantized_pad1(C);
        rf.stats = l.sc.stats;
        RouteArgs r{};
        r.queries = qrows;
        r.nq = nb;
        r.cent = centroids;
        r.C = C;
        r.D = D;
        r.k = nprobe;
        r.L = p.L;
        r.Cs = p.Cs;
        r.sstride = p.Ss;
        r.rank_j = p.rank_j;
        r.rank_safe = p.rank_safe;
        r.rank_max = p.rank_max;
        r.keys = l.keys;
        r.kmin = l.kmin;
        r.tau = l.tau;
        r.cand_cnt = l.cand_cnt;
        r.cand = l.cand;
        r.qn2 = l.qn2;
        r.mc2_bits = l.sc.mc2_bits;
        r.bound_coef = bound_coef(DP);
        r.force_fallback = ctx->force_fallback;
        r.out_ids = out_ids + q0 * nprobe;
        r.out_dist = out_dist ? out_dist + q0 * nprobe : nullptr;
        r.wl = l.wl;
        r.wl_cnt = l.sc.wl_cnt;
        r.stats = l.sc.stats;
        r.w = planes ? w : nullptr;
        r.qbound = l.qbound;
        r.f16 = f16;
        if (planes) {
            // the planes' sample minima (in the keys buffer), threshold and
            // filter over every centroid
            ra.c_begin = 0;
            ra.c_end = p.Cs;
            ra.nchunks = p.Cs / kQuantChunk;
            ra.cstride = p.Ss;
            ra.keys = l.keys;
            TIMED("route_i8_keys", launch_route_i8(kRouteKeys, p.qdp, ra, ctx->num_cus, s));
            rf.nsub = p.Cs / kQuantChunk;
            rf.cstride = p.Ss;
            rf.kmin = l.keys;
            if (f16) TIMED("route_f16_keys", launch_route_f16(kRouteKeys, p.qdp, rf, ctx->num_cus, s));
            TIMED("route_threshold_min", launch_route_threshold_min(r, s));
            ra.c_end = C;
            ra.nchunks = (C + kQuantChunk - 1) / kQuantChunk;
            ra.cstride = 1;
            ra.keys = nullptr;
            ra.tau = l.tau;
            ra.cand_cnt = l.cand_cnt;
            ra.cand = l.cand;
            ra.L = p.L;
            TIMED("route_i8_filter", launch_route_i8(kRouteFilter, p.qdp, ra, ctx->num_cus, s));
            rf.nsub = rf.cpad / kQuantChunk;
            rf.cstride = 1;
            rf.kmin = nullptr;
            rf.tau = l.tau;
            rf.cand_cnt = l.cand_cnt;
            rf.cand = l.cand;
            rf.L = p.L;
            if (f16) TIMED("route_f16_filter", launch_route_f16(kRouteFilter, p.qdp, rf, ctx->num_cus, s));
        }
        a.c_begin = 0;
        a.c_end = C;
        a.nchunks = p.Cs / kChunk;
        a.cstride = p.Ss;
        a.keys = l.keys;
        a.kmin = l.kmin;
        TIMED("screen_keys", launch_screen(kModeKeys, kRowF32, DP, a, ctx->screen_waves, ctx->num_cus, s));
        TIMED("route_threshold", launch_route_threshold(r, s));
        // every chunk the sample left
        a.nchunks = (C + kChunk - 1) / kChunk - p.Cs / kChunk;
        a.cstride = 1;
        a.skip_n = p.Cs / kChunk;
        a.skip_s = p.Ss;
        a.keys = nullptr;
        a.tau = l.tau;
        a.cand_cnt = l.cand_cnt;
        a.cand = l.cand;
        a.L = p.L;
        TIMED("screen_filter", launch_screen(kModeFilter, kRowF32, DP, a, ctx->screen_waves, ctx->num_cus, s));
        TIMED("route_select", launch_route_select(r, s));
        TIMED("route_fallback", launch_route_fallback(r, 2 * ctx->num_cus, s));
    }
    ctx->last_stats = l.sc.stats;
    ctx->last_sample = p.Cs;
    return IVF_OK;
}

}  // namespace

extern "C" {

ivf_status ivf_route(ivf_ctx *ctx, const float *queries, int64_t Q, const float *centroids,
                     int64_t C, int32_t D, int32_t nprobe, int32_t *out_ids, float *out_dist)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "route";
    bool done = false;
    ivf_status st = check_route(ctx, queries, Q, centroids, C, D, nprobe, out_ids, out_dist, &done);
    if (st != IVF_OK || done) return st;
    RoutePlan p = plan_route(Q, C, nprobe, ctx->sample_rank, D);
    const size_t need = layout_route(nullptr, p, C).bytes;
    // without room for the f16 plane's padding the fp32 kernels take its place
    if (p.f16 && ctx->ws_bytes < need) p.f16 = false;
    if ((st = check_ws(ctx, layout_route(nullptr, p, C).bytes, need)) != IVF_OK) return st;
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    return enqueue_route(ctx, queries, Q, centroids, C, D, nprobe, out_ids, out_dist, p, ctx->ws);
}

ivf_status ivf_route_noalloc(ivf_ctx *ctx, const float *queries, int64_t Q, const float *centroids,
                             int64_t C, int32_t D, int32_t nprobe, int32_t *out_ids, float *out_dist)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "route_noalloc";
    bool done = false;
    ivf_status st = check_route(ctx, queries, Q, centroids, C, D, nprobe, out_ids, out_dist, &done);
    if (st != IVF_OK || done) return st;
    // the batch of queries shrinks until the layout fits the static scratch;
    // sizes that do not fit with a single query are refused
    RoutePlan p = plan_route(Q, C, nprobe, ctx->sample_rank, D);
    auto one_query = [&] {
        RoutePlan q1 = p;
        q1.QB = 1;
        return layout_route(nullptr, q1, C).bytes;
    };
    // the f16 plane, then the int8 route planes are left out (fp32 kernels
    // only) when they do not fit beside one query
    if (one_query() > kStaticScratchBytes) p.f16 = false;
    if (one_query() > kStaticScratchBytes) p.qdp = 0;
    const size_t one = one_query();
    if (one > kStaticScratchBytes)
        return fail(ctx, IVF_EUNSUPPORTED,
                    "route_noalloc: C = %lld, nprobe = %d need %zu bytes of scratch for one query; the static "
                    "scratch holds %zu", (long long)C, nprobe, one, kStaticScratchBytes);
    RoutePlan two = p;
    two.QB = 2;
    const size_t per_query = layout_route(nullptr, two, C).bytes - one;
    const int64_t fit = 1 + (int64_t)((kStaticScratchBytes - one) / std::max<size_t>(per_query, 1));
    if (p.QB > fit) p.QB = fit >= 64 ? fit / 32 * 32 : fit;
    while (p.QB > 1 && layout_route(nullptr, p, C).bytes > kStaticScratchBytes) --p.QB;
    if (ctx->device < 0) return fail(ctx, IVF_EDEVICE, "no usable device (validation-only context)");
    void *scratch_ptr = static_scratch(ctx->device);
    if (!scratch_ptr) return fail(ctx, IVF_EDEVICE, "static scratch of device %d is not available", ctx->device);
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    // no event objects are created for this call, even when profiling is on
    const int prof = ctx->profile;
    ctx->profile = 0;
    st = enqueue_route(ctx, queries, Q, centroids, C, D, nprobe, out_ids, out_dist, p, scratch_ptr);
    ctx->profile = prof;
    return st;
}

static ivf_status check_rows(ivf_ctx *ctx, const void *rows, int dt, int64_t N, int32_t D,
                             size_t *row_bytes)
{
    if (dt != IVF_F32 && dt != IVF_U8) return fail(ctx, IVF_EINVAL, "dtype must be IVF_F32 or IVF_U8");
    if (N < 0) return fail(ctx, IVF_EINVAL, "N must be >= 0");
    if (N > (int64_t)UINT32_MAX) return fail(ctx, IVF_EUNSUPPORTED, "N must be < 2^32");
    if (N > 0 && !rows) return fail(ctx, IVF_EINVAL, "null data pointer");
    if (rows && !aligned16(rows)) return fail(ctx, IVF_EINVAL, "data must be 16-byte aligned");
    *row_bytes = (size_t)D * (dt == IVF_U8 ? 1 : 4);
    return IVF_OK;
}

ivf_status ivf_kmeans_step(ivf_ctx *ctx, const void *train, int dt, int64_t N,
                           const float *centroids, int64_t C, int32_t D, uint64_t seed,
                           int32_t iter, int32_t *out_labels, float *out_centroids,
                           int64_t *out_counts, double *out_objective, const int32_t *hint_labels)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "kmeans_step";
    ivf_status st = check_common(ctx, C, D);
    if (st != IVF_OK) return st;
    size_t rb;
    if ((st = check_rows(ctx, train, dt, N, D, &rb)) != IVF_OK) return st;
    if (N == 0) return IVF_OK;
    if (!centroids || !out_labels || !out_centroids) return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(centroids) || !aligned16(out_labels) || !aligned16(out_centroids) ||
        (out_counts && !aligned16(out_counts)) || (out_objective && !aligned16(out_objective)) ||
        (hint_labels && !aligned16(hint_labels)))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const size_t xb = (size_t)N * rb, cb = (size_t)C * D * 4, lb = (size_t)N * 4, nb = (size_t)C * 8;
    const void *outs[4] = {out_labels, out_centroids, out_counts, out_objective};
    const size_t osz[4] = {lb, cb, nb, 8};
    for (int i = 0; i < 4; ++i) {
        if (overlap(outs[i], osz[i], train, xb) || overlap(outs[i], osz[i], centroids, cb) ||
            overlap(outs[i], osz[i], hint_labels, hint_labels ? lb : 0))
            return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
        for (int j = i + 1; j < 4; ++j)
            if (overlap(outs[i], osz[i], outs[j], osz[j])) return fail(ctx, IVF_EINVAL, "outputs overlap");
    }
    AssignLayout l;
    if ((st = fit_assign(ctx, N, C, D, true, l)) != IVF_OK) return st;
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);

    const int rowtype = dt == IVF_U8 ? kRowU8 : kRowF32;
    if ((st = enqueue_assign(ctx, train, rowtype, N, centroids, C, D, out_labels, l, hint_labels)) != IVF_OK)
        return st;
    int64_t *counts = out_counts ? out_counts : l.counts;
    if ((st = enqueue_build(ctx, N, C, out_labels, l.cntmat, counts, l.offsets, l.perm)) != IVF_OK) return st;
    TIMED("kmeans_update", launch_kmeans_update(train, rowtype, N, D, D, centroids, C, counts, l.offsets, l.perm, seed,
                                 iter, out_centroids, l.jpart, out_objective, ctx->stream));
    return IVF_OK;
}

ivf_status ivf_assign_build(ivf_ctx *ctx, const void *base, int dt, int64_t N,
                            const float *centroids, int64_t C, int32_t D, int32_t *out_labels,
                            int64_t *out_counts, int64_t *out_offsets, uint32_t *out_perm)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "assign_build";
    ivf_status st = check_common(ctx, C, D);
    if (st != IVF_OK) return st;
    size_t rb;
    if ((st = check_rows(ctx, base, dt, N, D, &rb)) != IVF_OK) return st;
    if (!centroids || !out_counts || !out_offsets || (N > 0 && (!out_labels || !out_perm)))
        return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(centroids) || !aligned16(out_counts) || !aligned16(out_offsets) ||
        (out_labels && !aligned16(out_labels)) || (out_perm && !aligned16(out_perm)))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const size_t xb = (size_t)N * rb, cb = (size_t)C * D * 4;
    const void *outs[4] = {out_labels, out_counts, out_offsets, out_perm};
    const size_t osz[4] = {(size_t)N * 4, (size_t)C * 8, (size_t)(C + 1) * 8, (size_t)N * 4};
    for (int i = 0; i < 4; ++i) {
        if (overlap(outs[i], osz[i], base, xb) || overlap(outs[i], osz[i], centroids, cb))
            return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
        for (int j = i + 1; j < 4; ++j)
            if (overlap(outs[i], osz[i], outs[j], osz[j])) return fail(ctx, IVF_EINVAL, "outputs overlap");
    }
    AssignLayout l;
    if ((st = fit_assign(ctx, std::max<int64_t>(N, 1), C, D, false, l)) != IVF_OK) return st;
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);

    const int rowtype = dt == IVF_U8 ? kRowU8 : kRowF32;
    if (N > 0 && (st = enqueue_assign(ctx, base, rowtype, N, centroids, C, D, out_labels, l)) != IVF_OK)
        return st;
    if ((st = enqueue_build(ctx, N, C, out_labels, l.cntmat, out_counts, out_offsets, out_perm)) != IVF_OK)
        return st;
    return IVF_OK;
}

ivf_status ivf_build_lists(ivf_ctx *ctx, const int32_t *labels, int64_t N, int64_t C,
                           int64_t *out_counts, int64_t *out_offsets, uint32_t *out_perm)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "build_lists";
    if (C < 1) return fail(ctx, IVF_EINVAL, "C must be >= 1");
    if (C > INT32_MAX) return fail(ctx, IVF_EUNSUPPORTED, "C must fit int32 ids");
    if (N < 0) return fail(ctx, IVF_EINVAL, "N must be >= 0");
    if (N > (int64_t)UINT32_MAX) return fail(ctx, IVF_EUNSUPPORTED, "N must be < 2^32");
    if (!out_counts || !out_offsets || (N > 0 && (!labels || !out_perm)))
        return fail(ctx, IVF_EINVAL, "null pointer argument");
    if ((labels && !aligned16(labels)) || !aligned16(out_counts) || !aligned16(out_offsets) ||
        (out_perm && !aligned16(out_perm)))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const void *outs[3] = {out_counts, out_offsets, out_perm};
    const size_t osz[3] = {(size_t)C * 8, (size_t)(C + 1) * 8, (size_t)N * 4};
    for (int i = 0; i < 3; ++i) {
        if (overlap(outs[i], osz[i], labels, (size_t)N * 4)) return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
        for (int j = i + 1; j < 3; ++j)
            if (overlap(outs[i], osz[i], outs[j], osz[j])) return fail(ctx, IVF_EINVAL, "outputs overlap");
    }
    const size_t need = layout_assign(nullptr, std::max<int64_t>(N, 1), C, 0, true, false, ctx->num_cus).bytes;
    ivf_status st;
    if ((st = check_ws(ctx, need)) != IVF_OK) return st;
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    const AssignLayout l = layout_assign(ctx->ws, std::max<int64_t>(N, 1), C, 0, true, false, ctx->num_cus);
    if ((st = enqueue_build(ctx, N, C, labels, l.cntmat, out_counts, out_offsets, out_perm)) != IVF_OK) return st;
    ctx->last_stats = nullptr;
    return IVF_OK;
}

ivf_status ivf_list_major(ivf_ctx *ctx, const void *base, int dt, int64_t N, const float *centroids,
                          int64_t C, int32_t D, const int64_t *offsets, const uint32_t *perm,
                          int64_t pos0, int64_t n, void *out_rows, float *out_residuals)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "list_major";
    ivf_status st = check_common(ctx, C, D);
    if (st != IVF_OK) return st;
    size_t rb;
    if ((st = check_rows(ctx, base, dt, N, D, &rb)) != IVF_OK) return st;
    if (pos0 < 0 || n < 0 || pos0 > N || n > N - pos0)
        return fail(ctx, IVF_EINVAL, "positions [pos0, pos0 + n) must lie in [0, N)");
    if (n == 0) return IVF_OK;
    if (!out_rows && !out_residuals) return fail(ctx, IVF_EINVAL, "no output requested");
    if (!centroids || !offsets || (N > 0 && !perm)) return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(centroids) || !aligned16(offsets) || (perm && !aligned16(perm)) ||
        (out_rows && !aligned16(out_rows)) || (out_residuals && !aligned16(out_residuals)))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const size_t ob[2] = {(size_t)n * rb, (size_t)n * D * 4};
    const void *outs[2] = {out_rows, out_residuals};
    const void *ins[4] = {base, centroids, offsets, perm};
    const size_t ib[4] = {(size_t)N * rb, (size_t)C * D * 4, (size_t)(C + 1) * 8, (size_t)N * 4};
    for (int i = 0; i < 2; ++i)
        for (int k = 0; k < 4; ++k)
            if (overlap(outs[i], ob[i], ins[k], ib[k])) return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
    if (overlap(out_rows, ob[0], out_residuals, ob[1])) return fail(ctx, IVF_EINVAL, "outputs overlap");
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    const int rowtype = dt == IVF_U8 ? kRowU8 : kRowF32;
    TIMED("list_major", launch_list_major(base, rowtype, N, centroids, C, D, offsets, perm, pos0, n,
                                          out_rows, out_residuals, ctx->stream));
    ctx->last_stats = nullptr;
    return IVF_OK;
}

ivf_status ivf_assign_graph(ivf_ctx *ctx, const void *rows, int dt, int64_t N, const float *centroids,
                            int64_t C, int32_t D, const int32_t *graph, int32_t S, const int32_t *prev,
                            const uint32_t *order, int32_t *out_labels, float *out_dist)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "assign_graph";
    ivf_status st = check_common(ctx, C, D);
    if (st != IVF_OK) return st;
    size_t rb;
    if ((st = check_rows(ctx, rows, dt, N, D, &rb)) != IVF_OK) return st;
    if (S < 1 || S > kMaxGraphDegree)
        return fail(ctx, IVF_EINVAL, "S must be in [1, %d] (got %d)", kMaxGraphDegree, S);
    if (N == 0) return IVF_OK;
    if (!centroids || !graph || !prev || !out_labels) return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(centroids) || !aligned16(graph) || !aligned16(prev) || (order && !aligned16(order)) ||
        !aligned16(out_labels) || (out_dist && !aligned16(out_dist)))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const void *ins[5] = {rows, centroids, graph, prev, order};
    const size_t ib[5] = {(size_t)N * rb, (size_t)C * D * 4, (size_t)C * S * 4, (size_t)N * 4,
                          order ? (size_t)N * 4 : 0};
    const void *outs[2] = {out_labels, out_dist};
    const size_t ob[2] = {(size_t)N * 4, (size_t)N * 4};
    for (int i = 0; i < 2; ++i)
        for (int k = 0; k < 5; ++k)
            if (overlap(outs[i], ob[i], ins[k], ib[k])) return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
    if (overlap(out_labels, ob[0], out_dist, ob[1])) return fail(ctx, IVF_EINVAL, "outputs overlap");
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    const int rowtype = dt == IVF_U8 ? kRowU8 : kRowF32;
    TIMED("assign_graph", launch_assign_graph(rows, rowtype, N, centroids, C, D, graph, S, prev, order,
                                              out_labels, out_dist, ctx->stream));
    ctx->last_stats = nullptr;
    return IVF_OK;
}

ivf_status ivf_assign_cells(ivf_ctx *ctx, const void *rows, int dt, int64_t N, const float *centroids,
                            int64_t C, int32_t D, const int32_t *cell, int64_t G, const int64_t *cell_offsets,
                            const uint32_t *cell_members, int64_t M, const int32_t *graph, int32_t S,
                            int32_t hops, const uint32_t *order, int32_t *out_labels, float *out_dist)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "assign_cells";
    ivf_status st = check_common(ctx, C, D);
    if (st != IVF_OK) return st;
    size_t rb;
    if ((st = check_rows(ctx, rows, dt, N, D, &rb)) != IVF_OK) return st;
    if (G < 1 || G > INT32_MAX) return fail(ctx, IVF_EINVAL, "G must be in [1, 2^31 - 1] (got %lld)", (long long)G);
    if (M < 0) return fail(ctx, IVF_EINVAL, "M must be >= 0");
    if (hops < 0 || hops > kMaxHops) return fail(ctx, IVF_EINVAL, "hops must be in [0, %d] (got %d)", kMaxHops, hops);
    if (graph && (S < 1 || S > kMaxGraphDegree))
        return fail(ctx, IVF_EINVAL, "S must be in [1, %d] (got %d)", kMaxGraphDegree, S);
    if (N == 0) return IVF_OK;
    if (!centroids || !cell || !cell_offsets || (M > 0 && !cell_members) || !out_labels)
        return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(centroids) || !aligned16(cell) || !aligned16(cell_offsets) ||
        (cell_members && !aligned16(cell_members)) || (graph && !aligned16(graph)) || (order && !aligned16(order)) ||
        !aligned16(out_labels) || (out_dist && !aligned16(out_dist)))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const void *ins[7] = {rows, centroids, cell, cell_offsets, cell_members, graph, order};
    const size_t ib[7] = {(size_t)N * rb, (size_t)C * D * 4, (size_t)N * 4, (size_t)(G + 1) * 8, (size_t)M * 4,
                          graph ? (size_t)C * S * 4 : 0, order ? (size_t)N * 4 : 0};
    const void *outs[2] = {out_labels, out_dist};
    const size_t ob[2] = {(size_t)N * 4, (size_t)N * 4};
    for (int i = 0; i < 2; ++i)
        for (int k = 0; k < 7; ++k)
            if (overlap(outs[i], ob[i], ins[k], ib[k])) return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
    if (overlap(out_labels, ob[0], out_dist, ob[1])) return fail(ctx, IVF_EINVAL, "outputs overlap");
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    const int rowtype = dt == IVF_U8 ? kRowU8 : kRowF32;
    TIMED("assign_cells", launch_assign_cells(rows, rowtype, N, centroids, C, D, cell, G, cell_offsets, cell_members,
                                              M, graph, graph ? S : 0, hops, order, out_labels, out_dist,
                                              ctx->num_cus, ctx->stream));
    ctx->last_stats = nullptr;
    return IVF_OK;
}

ivf_status ivf_adc_scan(ivf_ctx *ctx, const float *queries, int64_t B, int32_t D, const float *centroids,
                        int64_t C, const int32_t *probes, int32_t P, const int64_t *offsets,
                        const uint32_t *perm, int64_t N, const uint8_t *codes, int32_t M,
                        const float *codebooks, int32_t k, uint32_t *out_ids, float *out_dist)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "adc_scan";
    ivf_status st = check_common(ctx, C, D);
    if (st != IVF_OK) return st;
    if (B < 0 || N < 0) return fail(ctx, IVF_EINVAL, "B and N must be >= 0");
    if (N > (int64_t)UINT32_MAX) return fail(ctx, IVF_EUNSUPPORTED, "N must be < 2^32");
    if (M < 1 || D % M != 0) return fail(ctx, IVF_EINVAL, "M must divide D (D = %d, M = %d)", D, M);
    if (M > kAdcMaxM) return fail(ctx, IVF_EUNSUPPORTED, "at most %d subspaces", kAdcMaxM);
    if (P < 1 || P > kMaxAdcProbes) return fail(ctx, IVF_EINVAL, "P must be in [1, %d]", kMaxAdcProbes);
    if (k < 1 || k > kAdcMaxK) return fail(ctx, IVF_EINVAL, "k must be in [1, %d]", kAdcMaxK);
    if (B == 0) return IVF_OK;
    if (!queries || !centroids || !probes || !offsets || !codebooks || !out_ids || !out_dist ||
        (N > 0 && (!perm || !codes)))
        return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(queries) || !aligned16(centroids) || !aligned16(probes) || !aligned16(offsets) ||
        (perm && !aligned16(perm)) || (codes && !aligned16(codes)) || !aligned16(codebooks) ||
        !aligned16(out_ids) || !aligned16(out_dist))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const void *ins[7] = {queries, centroids, probes, offsets, perm, codes, codebooks};
    const size_t ib[7] = {(size_t)B * D * 4, (size_t)C * D * 4, (size_t)B * P * 4, (size_t)(C + 1) * 8,
                          (size_t)N * 4, (size_t)N * M, (size_t)kPqK * D * 4};
    const void *outs[2] = {out_ids, out_dist};
    const size_t ob = (size_t)B * k * 4;
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 7; ++j)
            if (overlap(outs[i], ob, ins[j], ib[j])) return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
    if (overlap(out_ids, ob, out_dist, ob)) return fail(ctx, IVF_EINVAL, "outputs overlap");
    const size_t need = layout_adc(nullptr, B, P, k, nullptr);
    if ((st = check_ws(ctx, need)) != IVF_OK) return st;
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    AdcScratch w;
    layout_adc(ctx->ws, B, P, k, &w);
    TIMED("adc_scan", launch_adc_scan(queries, B, D, centroids, C, probes, P, offsets, perm, N, codes, M,
                                      codebooks, k, w, out_ids, out_dist, ctx->num_cus, ctx->stream));
    ctx->last_stats = nullptr;
    return IVF_OK;
}

static ivf_status check_pq(ivf_ctx *ctx, int32_t D, int32_t M, int *dsub)
{
    ivf_status st = check_common(ctx, kPqK, D);
    if (st != IVF_OK) return st;
    if (M < 1 || D % M != 0) return fail(ctx, IVF_EINVAL, "M must divide D (D = %d, M = %d)", D, M);
    *dsub = D / M;
    if (*dsub > kPqMaxSubDims)
        return fail(ctx, IVF_EUNSUPPORTED, "at most %d dims per subspace (D / M = %d)", kPqMaxSubDims, *dsub);
    return IVF_OK;
}

ivf_status ivf_pq_encode(ivf_ctx *ctx, const float *x, int64_t n, int32_t D, int32_t M,
                         const float *codebooks, uint8_t *out_codes)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "pq_encode";
    int dsub = 0;
    ivf_status st = check_pq(ctx, D, M, &dsub);
    if (st != IVF_OK) return st;
    if (n < 0) return fail(ctx, IVF_EINVAL, "n must be >= 0");
    if (n == 0) return IVF_OK;
    if (!x || !codebooks || !out_codes) return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(x) || !aligned16(codebooks) || !aligned16(out_codes))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const size_t ob = (size_t)n * M;
    if (overlap(out_codes, ob, x, (size_t)n * D * 4) || overlap(out_codes, ob, codebooks, (size_t)kPqK * D * 4))
        return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    TIMED("pq_assign", launch_pq_assign(x, n, D, dsub, M, codebooks, out_codes, nullptr, ctx->num_cus, ctx->stream));
    ctx->last_stats = nullptr;
    return IVF_OK;
}

ivf_status ivf_pq_train_step(ivf_ctx *ctx, const float *x, int64_t n, int32_t D, int32_t M,
                             const float *codebooks, uint64_t seed, int32_t iter, float *out_codebooks,
                             int64_t *out_counts, double *out_objective)
{
    if (!ctx) return IVF_EINVAL;
    ctx->err.clear();
    ctx->cur_call = "pq_train_step";
    int dsub = 0;
    ivf_status st = check_pq(ctx, D, M, &dsub);
    if (st != IVF_OK) return st;
    if (n < 1) return fail(ctx, IVF_EINVAL, "n must be >= 1");
    if (n > (int64_t)UINT32_MAX) return fail(ctx, IVF_EUNSUPPORTED, "n must be < 2^32");
    if (!x || !codebooks || !out_codebooks) return fail(ctx, IVF_EINVAL, "null pointer argument");
    if (!aligned16(x) || !aligned16(codebooks) || !aligned16(out_codebooks) ||
        (out_counts && !aligned16(out_counts)) || (out_objective && !aligned16(out_objective)))
        return fail(ctx, IVF_EINVAL, "arrays must be 16-byte aligned");
    const size_t xb = (size_t)n * D * 4, cb = (size_t)kPqK * D * 4;
    const void *outs[3] = {out_codebooks, out_counts, out_objective};
    const size_t osz[3] = {cb, (size_t)M * kPqK * 8, (size_t)M * 8};
    for (int i = 0; i < 3; ++i) {
        if (overlap(outs[i], osz[i], x, xb) || overlap(outs[i], osz[i], codebooks, cb))
            return fail(ctx, IVF_EINVAL, "outputs overlap inputs");
        for (int j = i + 1; j < 3; ++j)
            if (overlap(outs[i], osz[i], outs[j], osz[j])) return fail(ctx, IVF_EINVAL, "outputs overlap");
    }
    const size_t need = layout_pq(nullptr, n, M, ctx->num_cus).bytes;
    if ((st = check_ws(ctx, need)) != IVF_OK) return st;
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, IVF_EDEVICE, "no usable device (context device %d)", ctx->device);
    const PqLayout l = layout_pq(ctx->ws, n, M, ctx->num_cus);
    int64_t *counts = out_counts ? out_counts : l.counts;
    // every subspace's labels, then all subspaces' lists, then one update
    // launch over all M x 256 codewords (group m = subspace m, seed + m)
    TIMED("pq_assign", launch_pq_assign(x, n, D, dsub, M, codebooks, nullptr, l.labels, ctx->num_cus, ctx->stream));
    TIMED("build_single", launch_single_build(plan_single(n, kPqK, M, ctx->num_cus), l.labels, l.cnt, counts, l.offsets,
                                              l.perm, ctx->stream));
    TIMED("pq_update", launch_kmeans_update(x, kRowF32, n, dsub, D, codebooks, kPqK, counts, l.offsets, l.perm,
                                            seed, iter, out_codebooks, l.jpart, out_objective, ctx->stream, M,
                                            dsub));
    ctx->last_stats = nullptr;
    return IVF_OK;
}

}  // extern "C"
