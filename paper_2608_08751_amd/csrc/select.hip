// Norms, routing threshold, certified top-k selection with fp64 refinement,
// and the exact fp64 fallback scan of queries (gfx950).
//
// Coarse search returns, per query, the nprobe centroids of smallest squared
// L2 distance (Eq. 1), selected on the device so that only O(B*P) ids and
// distances leave the GPU ("On-device list selection", Sec. "GPU coarse
// search"). The screening keys from the MFMA kernel carry a rounding error of
// at most B per key; the selection below only trusts them as far as B allows
// and decides the final order with exact fp64 distances.
#include "ivf_internal.h"
#include "exact.h"

#include <float.h>
#include <math.h>

namespace ivf {
namespace {

constexpr float kInfF = __builtin_huge_valf();
constexpr double kInfD = __builtin_huge_val();

__device__ __forceinline__ bool key_lt(float ka, int ia, float kb, int ib)
{
    return ka < kb || (ka == kb && ia < ib);
}

__device__ __forceinline__ double key_bound(double coef, uint32_t mc2_bits, double xn2)
{
    const double M = (double)__uint_as_float(mc2_bits) * (1.0 + 0x1p-20);
    return coef * (M + 2.0 * sqrt(xn2 * (1.0 + 0x1p-40)) * sqrt(M)) + 0x1p-100;
}

__device__ __forceinline__ int pow2_at_least(int n)
{
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

// Bitonic sort of P (power of two) entries in LDS by (key, id) ascending.
template <typename K, typename LT>
__device__ void bitonic_sort(K *key, int *id, int P, LT lt)
{
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < P; i += blockDim.x) {
                const int ixj = i ^ j;
                if (ixj > i) {
                    const bool up = (i & k) == 0;
                    const K ka = key[i], kb = key[ixj];
                    const int ia = id[i], ib = id[ixj];
                    const bool swap = up ? lt(kb, ib, ka, ia) : lt(ka, ia, kb, ib);
                    if (swap) {
                        key[i] = kb;
                        key[ixj] = ka;
                        id[i] = ib;
                        id[ixj] = ia;
                    }
                }
            }
            __syncthreads();
        }
    }
}

__global__ void fill_u32_kernel(uint32_t *p, int64_t n, uint32_t v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// fl32(||c||^2) per centroid (fp64 accumulation in dimension order, one
// thread per row, 16-byte loads; D % 4 == 0) and the maximum over all rows
// (as float bits; floats >= 0 order like their bits).
__global__ __launch_bounds__(256) void centroid_norms_kernel(const float *__restrict__ cent,
                                                             int64_t C, int D,
                                                             float *__restrict__ cnorm,
                                                             uint32_t *__restrict__ mc2_bits)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    __shared__ uint32_t wmax[4];
    uint32_t mx = 0;
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < C; r += (int64_t)gridDim.x * 256) {
        const float4 *p = reinterpret_cast<const float4 *>(cent + r * D);
        double s = 0.0;
        for (int d4 = 0; d4 < D / 4; d4 += 8) {
            float4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (d4 + u < D / 4) v[u] = p[d4 + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (d4 + u < D / 4) {
                    s = fma((double)v[u].x, (double)v[u].x, s);
                    s = fma((double)v[u].y, (double)v[u].y, s);
                    s = fma((double)v[u].z, (double)v[u].z, s);
                    s = fma((double)v[u].w, (double)v[u].w, s);
                }
            }
        }
        const float n = (float)s;
        cnorm[r] = n;
        mx = max(mx, __float_as_uint(n));
    }
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
    if (lane == 0) wmax[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t m = max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3]));
        atomicMax(mc2_bits, m);
    }
}

// Order-preserving map between non-NaN floats and uint32 keys.
__device__ __forceinline__ uint32_t f2o(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float o2f(uint32_t u)
{
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}

// k-th smallest (1-based, k <= number of values) of the values spread over
// the workgroup (thread t holds v[e] for e < nv): MSD radix select, four
// passes of 8 bits with a 256-bin LDS histogram each; one wave locates the
// bin that contains rank k with a prefix scan. Returns the exact value.
template <int V>
__device__ uint32_t block_select(const uint32_t (&v)[V], int nv, int k, uint32_t *hist,
                                 uint32_t *sh)
{
    uint32_t prefix = 0, mask = 0, krem = (uint32_t)k;
    const int lane = threadIdx.x & 63;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        for (int i = threadIdx.x; i < 256; i += blockDim.x) hist[i] = 0;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (e < nv && (v[e] & mask) == prefix) atomicAdd(&hist[(v[e] >> shift) & 0xFFu], 1u);
        __syncthreads();
        if (threadIdx.x < 64) {
            const uint32_t c0 = hist[4 * lane], c1 = hist[4 * lane + 1];
            const uint32_t c2 = hist[4 * lane + 2], c3 = hist[4 * lane + 3];
            const uint32_t own = c0 + c1 + c2 + c3;
            uint32_t incl = own;
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t up = __shfl_up(incl, o);
                if (lane >= o) incl += up;
            }
            const uint32_t before = incl - own;
            if (before < krem && krem <= incl) {
                uint32_t r = krem - before;
                int bin = 4 * lane;
                if (r > c0) { r -= c0; ++bin;
                    if (r > c1) { r -= c1; ++bin;
                        if (r > c2) { r -= c2; ++bin; } } }
                sh[0] = (uint32_t)bin;
                sh[1] = r;
            }
        }
        __syncthreads();
        prefix |= sh[0] << shift;
        mask |= 0xFFu << shift;
        krem = sh[1];
        __syncthreads();
    }
    return prefix;
}

// Routing threshold from the Cs sample keys of one query: the keys are cut
// into groups of 16 consecutive sample centroids, tau = the rank_j-th smallest group
// minimum (so about rank_j sample keys lie at or below tau), and every sample
// key <= tau is emitted as a candidate. Cs is at most 65,536.
constexpr int kMaxGroups = 4096;
constexpr int kGroupsPerThread = kMaxGroups / 256;

// true when a plane's route kernels produce this batch's keys (group minima)
__device__ __forceinline__ bool plane_keys(const RouteArgs &a) { return a.w && route_mode(a.w) != kModeF32; }

// Centroid id of sample key s: the sample is the chunks j * sstride of kChunk
// centroids, its keys in that order.
__device__ __forceinline__ uint32_t sample_id(const RouteArgs &a, int64_t s)
{
    const int64_t st = a.sstride > 1 ? a.sstride : 1;
    return (uint32_t)((s / kChunk) * st * kChunk + s % kChunk);
}

// The threshold from the group minima the fp32 keys pass wrote: tau = the
// rank_j-th smallest minimum, then only the groups whose minimum is <= tau
// (about rank_j of them) are read for their keys <= tau, which become
// candidates (a group whose minimum exceeds tau holds none).
__global__ __launch_bounds__(256) void route_threshold_gmin_kernel(RouteArgs a)
{
    if (plane_keys(a)) return;
    const int64_t q = blockIdx.x;
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sh[2];
    __shared__ uint32_t s_cnt;
    const int G = (int)(a.Cs / 16);
    const float *gmin = a.kmin + q * G;
    uint32_t v[kGroupsPerThread];
    int nv = 0;
#pragma unroll
    for (int e = 0; e < kGroupsPerThread; ++e) {
        const int g = threadIdx.x + 256 * e;
        v[e] = 0xFFFFFFFFu;
        if (g < G) {
            v[e] = f2o(gmin[g]);
            nv = e + 1;
        }
    }
    if (threadIdx.x == 0) s_cnt = 0;
    const uint32_t tho = block_select(v, nv, min(a.rank_j, G), hist, sh);
    const float th = o2f(tho);
    const float4 *k4 = reinterpret_cast<const float4 *>(a.keys + q * a.Cs);
#pragma unroll
    for (int e = 0; e < kGroupsPerThread; ++e) {
        const int g = threadIdx.x + 256 * e;
        if (g < G && v[e] <= tho) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 w = k4[4 * (int64_t)g + i];
                const float kk[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (kk[c] <= th) {
                        const uint32_t slot = atomicAdd(&s_cnt, 1u);
                        if (slot < (uint32_t)a.L)
                            a.cand[q * a.L + slot] = make_uint2(__float_as_uint(kk[c]), sample_id(a, 16 * g + 4 * i + c));
                    }
                }
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.tau[q] = th;
        a.cand_cnt[q] = s_cnt;
    }
}

// The threshold when a plane's route kernels ran: the keys buffer holds the
// sample's group minima [nq, Cs / 16] directly, tau = the rank_j-th smallest,
// and the sample's centroids are left to the filter, which then covers every
// centroid (the candidate list starts empty). The f16 plane's window 2 B is
// part of the spacing of the minima, so tau is at least the window above the
// rank_safe-th minimum (the k-th smallest key lies below that minimum but for
// a five-sigma draw of the sample); a query for which that lies above the
// rank_max-th minimum would keep too many candidates, and its batch goes to
// the fp32 kernels. A rank above rank_max (IVF_OPT_SAMPLE_RANK) is selected
// from all minima. tau stays below infinity: the filter keeps v >= -tau, and
// what lies outside the table (padding rows, the scan's start block) scores
// -infinity.
constexpr int kRankMax = 64;

__global__ __launch_bounds__(256) void route_threshold_min_kernel(RouteArgs a)
{
    // (kWordF16Off, zero before this kernel, is raised by it and not read)
    const bool i8 = a.w[kWordNotI8] == 0u;
    if (!i8 && !a.f16) return;
    const int64_t q = blockIdx.x;
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sh[2];
    __shared__ uint32_t s_n;
    __shared__ uint32_t s_v[2 * kRankMax];
    __shared__ float s_rank[2];
    const int G = (int)(a.Cs / 16);
    const float *kr = a.keys + q * G;
    uint32_t v[kGroupsPerThread];
    int nv = 0;
#pragma unroll
    for (int e = 0; e < kGroupsPerThread; ++e) {
        const int g = threadIdx.x + 256 * e;
        v[e] = 0xFFFFFFFFu;
        if (g < G) {
            v[e] = f2o(kr[g]);
            nv = e + 1;
        }
    }
    const int rank = min(a.rank_j, G);
    if (i8) {
        const float th = o2f(block_select(v, nv, rank, hist, sh));
        if (threadIdx.x == 0) {
            a.tau[q] = th;
            a.cand_cnt[q] = 0;
        }
        return;
    }
    // the rank_max smallest minima, then two ranks among them
    if (threadIdx.x == 0) s_n = 0;
    const int rmax = min(a.rank_max, G);
    const uint32_t top = block_select(v, nv, rmax, hist, sh);
#pragma unroll
    for (int e = 0; e < kGroupsPerThread; ++e) {
        if (e < nv && v[e] <= top) {
            const uint32_t at = atomicAdd(&s_n, 1u);
            if (at < 2 * kRankMax) s_v[at] = v[e];
        }
    }
    __syncthreads();
    const int n = min((int)s_n, 2 * kRankMax);  // rmax but for equal minima
    if ((int)threadIdx.x < n) {
        const uint32_t m = s_v[threadIdx.x];
        int less = 0, same = 0;
        for (int i = 0; i < n; ++i) {
            less += s_v[i] < m ? 1 : 0;
            same += s_v[i] == m ? 1 : 0;
        }
        if (less < rank && rank <= less + same) s_rank[0] = o2f(m);
        const int rs = min(a.rank_safe, rmax);
        if (less < rs && rs <= less + same) s_rank[1] = o2f(m);
    }
    __syncthreads();
    const float th = rank <= rmax ? s_rank[0] : o2f(block_select(v, nv, rank, hist, sh));
    if (threadIdx.x == 0) {
        const float cover = __double2float_ru((double)s_rank[1] + 2.0 * (double)a.qbound[q]);
        const bool wide = !(cover <= o2f(top));
        a.tau[q] = fminf(fmaxf(th, cover), FLT_MAX);
        a.cand_cnt[q] = 0;
        if (wide) a.w[kWordF16Off] = 1u;
    }
}

// Ranks nr re-evaluated candidates (distances and ids in LDS) by (distance, id)
// and writes the first k: every thread counts, for R of its candidates at a
// time, the ones before them, so a pass over the list serves R (16,384 queries on
// 2,048 x 32 centroids, k = 1,024: 5.6 -> 2.4 ms; every centroid a candidate: 20.6 ->
// 8.4).
template <int R>
__device__ __forceinline__ void rank_some(const double *__restrict__ bd, const int *__restrict__ bi, int nr, int k, int i0,
                                          int32_t *__restrict__ ids, float *__restrict__ dist)
{
    double d[R];
    int id[R], rank[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = min(i0 + r * (int)blockDim.x, nr - 1);
        d[r] = bd[i];
        id[r] = bi[i];
        rank[r] = 0;
    }
#pragma unroll 4
    for (int j = 0; j < nr; ++j) {
        const double dj = bd[j];
        const int ij = bi[j];
#pragma unroll
        for (int r = 0; r < R; ++r) rank[r] += dist_lt(dj, ij, d[r], id[r]) ? 1 : 0;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (i0 + r * (int)blockDim.x < nr && rank[r] < k) {
            ids[rank[r]] = id[r];
            if (dist) dist[rank[r]] = (float)d[r];
        }
    }
}

__device__ __forceinline__ void write_ranked(const double *__restrict__ bd, const int *__restrict__ bi, int nr, int k,
                                             int32_t *__restrict__ ids, float *__restrict__ dist)
{
    int i = threadIdx.x;
    for (; i + (int)blockDim.x < nr; i += 4 * (int)blockDim.x) rank_some<4>(bd, bi, nr, k, i, ids, dist);
    if (i < nr) rank_some<1>(bd, bi, nr, k, i, ids, dist);
}

// Certified selection of one query's top-k from its screened candidates.
// Candidates = every centroid with key <= tau. Let kth = the k-th smallest key
// (radix select). If tau >= kth + 2B, every centroid outside
// R = {key <= kth + 2B} is strictly farther (exactly) than k candidates, so the
// exact top-k lies in R; R's members are re-evaluated in fp64 and ranked by
// (distance, id). Otherwise (or on overflow / underflow) the query goes to
// the fallback scan.
constexpr int kMaxCand = 4096;
constexpr int kCandPerThread = kMaxCand / 256;

__device__ __forceinline__ void push_fallback(const RouteArgs &a, int64_t q, bool overflow)
{
    const uint32_t slot = atomicAdd(a.wl_cnt, 1u);
    a.wl[slot] = (int32_t)q;
    atomicAdd(a.stats + kStatFallback, 1ull);
    if (overflow) atomicAdd(a.stats + kStatOverflow, 1ull);
}

__global__ __launch_bounds__(256) void route_select_kernel(RouteArgs a)
{
    const int64_t q = blockIdx.x;
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sh[2];
    __shared__ __attribute__((aligned(16))) float qrow[256];
    __shared__ int s_nr;
    // R (at most L <= kMaxCand entries): fp64 distances, then ids
    extern __shared__ __attribute__((aligned(16))) unsigned char sel_lds[];
    double *rd = reinterpret_cast<double *>(sel_lds);
    int *rid = reinterpret_cast<int *>(rd + a.L);
    const uint32_t n = a.cand_cnt[q];
    const bool overflow = n > (uint32_t)a.L;
    if (a.force_fallback || overflow || n < (uint32_t)a.k) {
        if (threadIdx.x == 0) push_fallback(a, q, overflow);
        return;
    }
    uint32_t v[kCandPerThread];
    int cid[kCandPerThread];
    int nv = 0;
#pragma unroll
    for (int e = 0; e < kCandPerThread; ++e) {
        const int i = threadIdx.x + 256 * e;
        v[e] = 0xFFFFFFFFu;
        cid[e] = 0;
        if (i < (int)n) {
            const uint2 c = a.cand[q * a.L + i];
            v[e] = f2o(__uint_as_float(c.x));
            cid[e] = (int)c.y;
            nv = e + 1;
        }
    }
    for (int d = threadIdx.x; d < a.D; d += blockDim.x) qrow[d] = a.queries[q * a.D + d];
    if (threadIdx.x == 0) s_nr = 0;
    const double kth = (double)o2f(block_select(v, nv, a.k, hist, sh));
    const double B2 = plane_keys(a) ? 2.0 * (double)a.qbound[q]
                                    : 2.0 * key_bound(a.bound_coef, *a.mc2_bits, a.qn2[q]);
    if (!((double)a.tau[q] >= kth + B2)) {
        if (threadIdx.x == 0) push_fallback(a, q, false);
        return;
    }
    const double thr = kth + B2;
#pragma unroll
    for (int e = 0; e < kCandPerThread; ++e)
        if (e < nv && (double)o2f(v[e]) <= thr) rid[atomicAdd(&s_nr, 1)] = cid[e];
    __syncthreads();
    const int nr = s_nr;  // >= k
    for (int i = threadIdx.x; i < nr; i += blockDim.x)
        rd[i] = exact_dist(qrow, a.cent + (int64_t)rid[i] * a.D, a.D);
    __syncthreads();
    write_ranked(rd, rid, nr, a.k, a.out_ids + q * a.k, a.out_dist ? a.out_dist + q * a.k : nullptr);
}

// Exact fp64 scan of all centroids for one query (its row staged in LDS): a
// running best list of K2 entries plus a buffer of new entries that beat its
// k-th element; the union is re-sorted whenever the buffer fills. bd, bi:
// 2 K2 entries, K2 the first power of two from max(k, workgroup) on.
__device__ void exact_topk(const float *__restrict__ cent, int64_t C, int D, int k, const float *qrow, double *bd,
                           int *bi, uint32_t &s_cnt, int32_t *out_ids, float *out_dist)
{
    int K2 = blockDim.x;
    while (K2 < k) K2 <<= 1;
    for (int i = threadIdx.x; i < 2 * K2; i += blockDim.x) {
        bd[i] = kInfD;
        bi[i] = 0x7fffffff;
    }
    if (threadIdx.x == 0) s_cnt = 0;
    __syncthreads();
    double wd = kInfD;
    int wi = 0x7fffffff;
    for (int64_t base = 0; base < C; base += blockDim.x) {
        const int64_t c = base + threadIdx.x;
        if (c < C) {
            const double d = exact_dist(qrow, cent + c * D, D);
            if (dist_lt(d, (int)c, wd, wi)) {
                const uint32_t slot = atomicAdd(&s_cnt, 1u);
                bd[K2 + slot] = d;
                bi[K2 + slot] = (int)c;
            }
        }
        __syncthreads();
        const bool last = base + blockDim.x >= C;
        if (s_cnt > (uint32_t)(K2 - blockDim.x) || last) {
            bitonic_sort(bd, bi, 2 * K2, dist_lt);
            for (int i = K2 + threadIdx.x; i < 2 * K2; i += blockDim.x) {
                bd[i] = kInfD;
                bi[i] = 0x7fffffff;
            }
            if (threadIdx.x == 0) s_cnt = 0;
            __syncthreads();
            wd = bd[k - 1];
            wi = bi[k - 1];
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < k; i += blockDim.x) {
        out_ids[i] = bi[i];
        if (out_dist) out_dist[i] = (float)bd[i];
    }
}

// The queries on the worklist.
__global__ __launch_bounds__(256) void route_fallback_kernel(RouteArgs a)
{
    __shared__ double bd[2048];
    __shared__ int bi[2048];
    __shared__ float qrow[256];
    __shared__ uint32_t s_cnt;
    __shared__ unsigned long long s_sum[4];
    {
        // the candidate total of the batch for the statistics (one atomic
        // per workgroup instead of one per query)
        unsigned long long sum = 0;
        for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < a.nq; q += (int64_t)gridDim.x * blockDim.x)
            sum += a.cand_cnt[q];
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long t = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
            if (t) atomicAdd(a.stats + kStatCandidates, t);
        }
    }
    const uint32_t total = *a.wl_cnt;
    for (uint32_t w = blockIdx.x; w < total; w += gridDim.x) {
        const int64_t q = a.wl[w];
        for (int d = threadIdx.x; d < a.D; d += blockDim.x) qrow[d] = a.queries[q * a.D + d];
        exact_topk(a.cent, a.C, a.D, a.k, qrow, bd, bi, s_cnt, a.out_ids + q * a.k,
                   a.out_dist ? a.out_dist + q * a.k : nullptr);
        __syncthreads();
    }
}

// Direct route: one workgroup of T threads selects a query's k nearest from
// its row of keys, V of them per thread in registers. tau = the k-th smallest
// of the threads' minima (k of the keys are no larger, so it is no smaller than
// the k-th key, and with many keys per thread only a few more lie below it), or
// the k-th key itself where k is over half the threads or the minima let too
// many keys through; every centroid that can be among the k nearest has a key
// of at most tau + 2B and is re-evaluated in fp64. A query whose window holds
// more than kDirectCand, or whose bound is not finite, is scanned here in
// fp64: no worklist and no further launch.
// Rounds of latency bound this kernel (a selection of four passes, a gather,
// a count), not bytes: 12 us for 1,000 queries on 1,024 x 128 with k = 16, 28
// for 8 queries on 65,536 x 128 with k = 64.
constexpr int kDirectCand = 2048;

template <int T, int V>
constexpr int direct_cand()  // also the scan's 2 K2 entries with k <= T V
{
    return 2 * T * V < kDirectCand ? 2 * T * V : kDirectCand;
}

template <int T, int V>
__global__ __launch_bounds__(T) void direct_select_kernel(DirectArgs a)
{
    static_assert(V % 4 == 0, "keys are read in fours");
    constexpr int kCand = direct_cand<T, V>();
    __shared__ double bd[kCand];
    __shared__ int bi[kCand];
    __shared__ __attribute__((aligned(16))) float qrow[256];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sh[2];
    __shared__ uint32_t s_cnt;
    __shared__ double s_x2;
    __shared__ uint32_t s_m[T / 64];
    const int64_t q = blockIdx.x;
    const int t = threadIdx.x;
    const float *kr = a.keys + q * a.stride;
    uint32_t v[V];
    uint32_t mn = 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < V / 4; ++e) {
        const int i = 4 * (t + T * e);
        float4 w = make_float4(kInfF, kInfF, kInfF, kInfF);
        if (i + 4 <= a.stride && i < a.C)
            w = *reinterpret_cast<const float4 *>(kr + i);
        else if (i < a.C)
            w.x = kr[i];
        v[4 * e] = f2o(w.x);
        v[4 * e + 1] = f2o(w.y);
        v[4 * e + 2] = f2o(w.z);
        v[4 * e + 3] = f2o(w.w);
        mn = min(min(mn, min(v[4 * e], v[4 * e + 1])), min(v[4 * e + 2], v[4 * e + 3]));
    }
    // the largest norm; NaN and infinities order above the finite ones
    uint32_t m = 0;
    for (int i = t; i < (int)((a.C + 31) / 32); i += T)
        m = max(m, __float_as_uint(a.mc2_part[i]) & 0x7FFFFFFFu);
    for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o));
    if ((t & 63) == 0) s_m[t >> 6] = m;
    for (int d = t; d < a.D; d += T) qrow[d] = a.queries[q * a.D + d];
    if (t < 64) {
        double s = 0.0;
        for (int d = t; d < a.D; d += 64) {
            const double x = (double)a.queries[q * a.D + d];
            s = fma(x, x, s);
        }
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (t == 0) {
            s_x2 = s;
            s_cnt = 0;
        }
    }
    __syncthreads();
    for (int i = 0; i < T / 64; ++i) m = max(m, s_m[i]);
    const double x2 = s_x2, B2 = 2.0 * key_bound(a.bound_coef, m, x2);
    const double M = (double)__uint_as_float(m);
    bool exact = a.force_fallback || !(M + 2.0 * sqrt(x2) * sqrt(M) < 1e37);  // sums of finite keys
    bool over = false;
    int nr = 0;
    if (!exact) {
        const bool by_min = a.k <= T / 2 && V > 4;
#pragma unroll 1
        for (int pass = by_min ? 0 : 1; pass < 2; ++pass) {
            uint32_t tau;
            if (pass == 0) {
                const uint32_t vm[1] = {mn};
                tau = block_select(vm, 1, a.k, hist, sh);
            } else {
                tau = block_select(v, V, a.k, hist, sh);
            }
            const double thr = (double)o2f(tau) + B2;
            // the keys are compared as floats no smaller than thr
            float tf = (float)thr;
            if ((double)tf < thr) tf = nextafterf(tf, kInfF);
            const uint32_t to = f2o(tf);
            if (mn <= to) {
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const int id = 4 * (t + T * (e / 4)) + e % 4;
                    if (v[e] <= to && id < a.C) {
                        const uint32_t slot = atomicAdd(&s_cnt, 1u);
                        if (slot < kCand) bi[slot] = id;
                    }
                }
            }
            __syncthreads();
            nr = (int)s_cnt;
            over = nr > kCand;
            if (!over) break;
            __syncthreads();
            if (t == 0) s_cnt = 0;
            __syncthreads();
        }
        exact = over;
    }
    if (exact) {
        if (t == 0) {
            atomicAdd(a.stats + kStatFallback, 1ull);
            if (over) atomicAdd(a.stats + kStatOverflow, 1ull);
        }
        __syncthreads();
        exact_topk(a.cent, a.C, a.D, a.k, qrow, bd, bi, s_cnt, a.out_ids + q * a.k,
                   a.out_dist ? a.out_dist + q * a.k : nullptr);
        return;
    }
    for (int i = t; i < nr; i += T) bd[i] = exact_dist_lds4(qrow, a.cent + (int64_t)bi[i] * a.D, a.D);
    __syncthreads();
    write_ranked(bd, bi, nr, a.k, a.out_ids + q * a.k, a.out_dist ? a.out_dist + q * a.k : nullptr);
}

int grid_for(int64_t n, int per_block, int cap)
{
    int64_t g = (n + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

}  // namespace

hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_centroid_norms(const float *cent, int64_t C, int D, float *cnorm,
                                 uint32_t *mc2_bits, hipStream_t s)
{
    hipLaunchKernelGGL(centroid_norms_kernel, dim3(grid_for(C, 256, 4096)), dim3(256), 0, s, cent, C, D,
                       cnorm, mc2_bits);
    return hipGetLastError();
}

hipError_t launch_route_threshold(const RouteArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(route_threshold_gmin_kernel, dim3((unsigned)a.nq), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_route_threshold_min(const RouteArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(route_threshold_min_kernel, dim3((unsigned)a.nq), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_route_select(const RouteArgs &a, hipStream_t s)
{
    const size_t lds = (size_t)a.L * (sizeof(double) + sizeof(int));
    hipLaunchKernelGGL(route_select_kernel, dim3((unsigned)a.nq), dim3(256), lds, s, a);
    return hipGetLastError();
}

// Threads by table size: up to 512 centroids one wave holds the row and needs
// no barrier (a call of 16,384 queries on 256 x 256: 162 us, 291 with four
// waves; on 300 x 256 162 and 264);
// a workgroup of 256 keeps up to 2,048 keys, eight per thread, and several
// share a CU; past that 1,024 threads read the row.
hipError_t launch_direct_select(const DirectArgs &a, hipStream_t s)
{
    const dim3 grid((unsigned)a.nq);
    if (a.C <= 64 * 4)
        hipLaunchKernelGGL((direct_select_kernel<64, 4>), grid, dim3(64), 0, s, a);
    else if (a.C <= 64 * 8)
        hipLaunchKernelGGL((direct_select_kernel<64, 8>), grid, dim3(64), 0, s, a);
    else if (a.C <= 256 * 4)
        hipLaunchKernelGGL((direct_select_kernel<256, 4>), grid, dim3(256), 0, s, a);
    else if (a.C <= 256 * 8)
        hipLaunchKernelGGL((direct_select_kernel<256, 8>), grid, dim3(256), 0, s, a);
    else if (a.C <= 1024 * 16)
        hipLaunchKernelGGL((direct_select_kernel<1024, 16>), grid, dim3(1024), 0, s, a);
    else
        hipLaunchKernelGGL((direct_select_kernel<1024, 64>), grid, dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_route_fallback(const RouteArgs &a, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(route_fallback_kernel, dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
}


}  // namespace ivf
