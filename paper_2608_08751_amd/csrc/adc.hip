// Residual-PQ approximate-distance scan on gfx950 (Sec. "Residual-PQ
// Candidate Reduction": lookup tables and ADC sums; Sec. "Compact PQ-Code
// Offloading": GPU-side task setup, chunked scan with local top-K, fused
// first merge, hierarchical merge to a bounded per-query handoff of N_rerank
// candidates).
//
// For query b and probed list l: r = q - c_l (fp32), LUT[m][j] = the fp64
// distance of the contract between r^(m) and codeword j of subspace m,
// rounded to fp32, and for every position p of list l
//     d~ = ((0 + LUT[0][a_0]) + LUT[1][a_1]) + ... ,   a = codes[p],
// with candidate id perm[p]. Candidates are ordered by (d~, id) through one
// 64-bit key: (order-preserving bits of d~) << 32 | id.
//
// Work decomposition. Every probed list is cut into chunks of kAdcChunk
// codes (the last one partial); the chunks of a list are taken in runs of
// G_b (the group size of query b, max(kAdcMinGroup, ceil(chunks_b / P))), so a
// short list is one group and a long one is spread over several groups, and a
// query has at most 2P groups. The groups of a query are dealt to S_b parts
// (part s takes groups s, s + S_b, ...): one part per query when the batch fills
// the chip, several when it does not, more for a query far heavier than the
// others.
//   adc_setup_kernel   one workgroup per query: the chunk counts of its
//                      probed lists, G_b, the groups of every list and their
//                      exclusive scan over the probes (each group's slot),
//                      and one descriptor per group (list, code range);
//   adc_extra_kernel   one workgroup, where lists may be skewed: the parts of
//                      the heavy queries beyond those every query has;
//   adc_scan_kernel    one workgroup of 16 waves per part: a few groups at a
//                      time it builds their lists' LUTs in LDS, scans their
//                      codes and keeps the k smallest keys of the part in an
//                      LDS pool (an exact radix select trims it when the next
//                      codes might not fit; later codes enter only below the
//                      k-th key of the last trim). The part of a whole query
//                      sorts its keys into the results, the others hand over
//                      their k keys;
//   adc_merge_kernel   one workgroup per query merges its parts' keys the same
//                      way and sorts them.
// What bounds it is the LUT arithmetic: 256 D fp64 subtractions and fmas per
// probed list, whatever its length. With one workgroup per group every group
// read the 1,024 D bytes of codebooks from L2 and converted them, and handed
// all its codes to the merge; here a thread holds its codewords of the usual
// widths (see scan_kernel) in registers in fp64 for all the groups of its part,
// the other widths are read once for the lists of a step, and one threshold serves
// a whole query. 2,048 queries x 96 probed lists of 122 codes, M = 16, k = 512:
// 1.86 -> 1.12 ms; 8 queries x 64 lists: 98 -> 45 us.
// Ids are unique within a query (lists are disjoint), so "the k smallest
// keys" is exact whatever the grouping.
#include "ivf_internal.h"

#include <math.h>

#include <algorithm>

namespace ivf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSetupThreads = 256;
constexpr int kAdcThreads = 1024;
constexpr int kAdcWaves = kAdcThreads / 64;
constexpr int kAdcChunk = 1024;      // codes per chunk
constexpr int kAdcMinGroup = 8;      // chunks per group at least
constexpr int kAdcPool = 4096;       // LDS pool capacity (keys): trimmed when fewer than kAdcThreads places are left
constexpr int kAdcMaxLists = 8;      // lists whose LUTs are built at a time, as many as fit
constexpr int kAdcLutBytes = 73728;  // LUTs
constexpr int kAdcPadD = 512;        // dims of a list's residual, its subspaces padded to 4, 8 or 16 dims
constexpr int kAdcBins = 2048;       // 11-bit digits
constexpr uint64_t kNoKey = ~0ull;
static_assert(kAdcMaxK + kAdcThreads <= kAdcPool, "a trimmed pool takes another round of keys");

__device__ __forceinline__ uint32_t f2o(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float o2f(uint32_t u)
{
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}

struct PoolLds {
    uint64_t key[kAdcPool];
    uint32_t hist[kAdcBins];
    uint32_t wsum[kAdcWaves];
    uint64_t thr;  // keys above it are not among the k smallest seen
    uint32_t digit, below, count;  // the selected bin of a pass
    uint32_t n;    // keys in the pool
};

__device__ __forceinline__ void pool_init(PoolLds &P)
{
    if (threadIdx.x == 0) {
        P.n = 0;
        P.thr = kNoKey;
    }
}

// Appends this thread's key (every thread of the workgroup calls it).
__device__ __forceinline__ void pool_add(PoolLds &P, uint64_t key, bool have, uint64_t thr)
{
    const int lane = threadIdx.x & 63;
    const bool keep = have && key <= thr;
    const uint64_t want = __ballot(keep);
    if (want != 0) {
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&P.n, (uint32_t)__popcll(want));
        base = __shfl(base, 0);
        if (keep) P.key[base + __popcll(want & ((1ull << lane) - 1))] = key;
    }
}

// Leaves exactly the k smallest of the pool's n (> k) unique keys in it. The
// select takes 11 bits a pass and stops as soon as the bin of the k-th key ends
// at rank k (usually after the second or third pass).
__device__ void pool_trim(PoolLds &P, int k)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int n = (int)P.n;
    uint64_t mine[kAdcPool / kAdcThreads];
#pragma unroll
    for (int e = 0; e < kAdcPool / kAdcThreads; ++e) {
        const int i = t + e * kAdcThreads;
        mine[e] = i < n ? P.key[i] : kNoKey;
    }
    uint64_t prefix = 0, mask = 0;
    uint32_t kk = (uint32_t)k;  // rank of the target inside the current prefix
    for (int top = 64; top > 0;) {
        const int width = min(top, 11), shift = top - width;
        top = shift;
        P.hist[t] = 0;
        P.hist[t + kAdcThreads] = 0;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kAdcPool / kAdcThreads; ++e)
            if (t + e * kAdcThreads < n && (mine[e] & mask) == prefix)
                atomicAdd(&P.hist[(mine[e] >> shift) & ((1u << width) - 1u)], 1u);
        __syncthreads();
        const uint32_t h0 = P.hist[2 * t], h1 = P.hist[2 * t + 1];
        uint32_t incl = h0 + h1;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t up = __shfl_up(incl, o);
            if (lane >= o) incl += up;
        }
        if (lane == 63) P.wsum[wave] = incl;
        __syncthreads();
        uint32_t before = incl - h0 - h1;
        for (int w = 0; w < wave; ++w) before += P.wsum[w];
        if (before < kk && kk <= before + h0 + h1) {
            const bool second = before + h0 < kk;
            P.digit = 2 * t + (second ? 1 : 0);
            P.below = before + (second ? h0 : 0u);
            P.count = second ? h1 : h0;
        }
        __syncthreads();
        prefix |= (uint64_t)P.digit << shift;
        mask |= ((1ull << width) - 1ull) << shift;
        kk -= P.below;
        if (P.count == kk) break;  // (uniform) the whole bin belongs to the k smallest
    }
    if (t == 0) {
        P.n = 0;
        P.thr = prefix | ~mask;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kAdcPool / kAdcThreads; ++e)
        pool_add(P, mine[e], t + e * kAdcThreads < n && (mine[e] & mask) <= prefix, kNoKey);
    __syncthreads();
    // with unique keys exactly k remain; repeated ids (not a valid list
    // layout) must not let the pool outgrow its capacity
    if (t == 0 && P.n > (uint32_t)k) P.n = (uint32_t)k;
    __syncthreads();
}

// Room for one more round of keys, after every thread's last append.
__device__ __forceinline__ void pool_room(PoolLds &P, int k)
{
    __syncthreads();
    const int n = (int)P.n;
    __syncthreads();  // every thread has read n before anyone appends again
    if (n > kAdcPool - kAdcThreads) pool_trim(P, k);
}

// The pool's k smallest keys, ascending, into the results of query b: one key
// per thread, exchanged by shuffles inside a wave and through LDS across.
__device__ void pool_finish(PoolLds &P, int k, int64_t b, uint32_t *__restrict__ ids, float *__restrict__ dist)
{
    const int t = threadIdx.x;
    const int n = (int)P.n;  // <= k <= kAdcThreads
    int np = 64;
    while (np < n) np <<= 1;
    uint64_t v = t < n ? P.key[t] : kNoKey;
    for (int size = 2; size <= np; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            uint64_t o;
            if (stride < 64) {
                o = (uint64_t)__shfl_xor((unsigned long long)v, stride);
            } else {
                __syncthreads();
                P.key[t] = v;
                __syncthreads();
                o = P.key[t ^ stride];
            }
            const bool up = (t & size) == 0, low = (t & stride) == 0;
            v = (up == low) == (o < v) ? o : v;
        }
    }
    if (t < k) {
        const bool have = t < n;
        ids[b * k + t] = have ? (uint32_t)v : 0xFFFFFFFFu;
        dist[b * k + t] = have ? o2f((uint32_t)(v >> 32)) : __builtin_huge_valf();
    }
}

// Positions [o0, o1) of list l, kept inside [0, N) whatever the offsets hold;
// an id outside [0, C) is an empty list.
__device__ __forceinline__ void list_range(const int64_t *__restrict__ offsets, int64_t C, int64_t N, int32_t l,
                                           int64_t &o0, int64_t &o1)
{
    if (l < 0 || l >= C) {
        o0 = o1 = 0;
        return;
    }
    o0 = min(max(offsets[l], (int64_t)0), N);
    o1 = min(max(offsets[l + 1], o0), N);
}

// What the parts of a query are decided by, in units of one ordinary list
// (1.2 us): a table, a chunk of codes, the work a part is meant to have; parts:
// per query where lists are of about the same length.
struct AdcCost {
    float list, chunk, part;
    int parts;
};

// gcnt[b]: groups (at most 2P <= 8,192) and parts (at most P) of query b.
__device__ __forceinline__ int32_t pack_groups(int groups, int parts) { return groups | parts << 14; }
__device__ __forceinline__ int groups_of(int32_t g) { return g & 0x3FFF; }
__device__ __forceinline__ int parts_of(int32_t g) { return g >> 14; }
static_assert(2 * kMaxAdcProbes < 1 << 14 && kMaxAdcProbes < 1 << 16, "both fit a word");

// Parts beyond the `S` that every query has, for queries that cost more than
// twice the usual (skewed lists): x.list[e] = (query, part) of extra part e,
// *x.n of them; x.split[i] = query of which some are, *x.nsplit of them. One
// workgroup; the extra parts are scaled down to x.cap where more are asked for.
struct AdcExtra {
    uint64_t *list;
    int32_t *n;
    int32_t *split;
    int32_t *nsplit;
    int cap;  // 0: no extra parts
};

__global__ __launch_bounds__(kAdcThreads) void adc_extra_kernel(int64_t B, int S, int32_t *__restrict__ gcnt,
                                                               AdcExtra x)
{
    __shared__ int64_t wsum[kAdcWaves];
    __shared__ int32_t s_split;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int64_t sum = 0;
    for (int64_t b = t; b < B; b += kAdcThreads) sum += parts_of(gcnt[b]) - S;
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor((long long)sum, o);
    if (lane == 0) wsum[wave] = sum;
    if (t == 0) s_split = 0;
    __syncthreads();
    int64_t total = 0;
    for (int w = 0; w < kAdcWaves; ++w) total += wsum[w];
    __syncthreads();
    int64_t first = 0;  // extra parts of the queries before this round's
    for (int64_t b0 = 0; b0 < B; b0 += kAdcThreads) {
        const int64_t b = b0 + t;
        const int32_t g = b < B ? gcnt[b] : 0;
        int64_t ex = b < B ? parts_of(g) - S : 0;
        if (total > x.cap) ex = ex * x.cap / total;
        int64_t incl = ex;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t up = __shfl_up((long long)incl, o);
            if (lane >= o) incl += up;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        int64_t at = first + incl - ex;
        for (int w = 0; w < kAdcWaves; ++w) {
            if (w < wave) at += wsum[w];
            first += wsum[w];
        }
        if (b < B) gcnt[b] = pack_groups(groups_of(g), S + (int)ex);
        for (int e = 0; e < (int)ex; ++e) x.list[at + e] = (uint64_t)b << 32 | (uint32_t)(S + e);
        if (ex > 0) x.split[atomicAdd(&s_split, 1)] = (int32_t)b;
        __syncthreads();
    }
    if (t == 0) {
        *x.n = (int32_t)first;
        *x.nsplit = s_split;
    }
}

// Task setup of query b: the group size, the groups of each probed list
// (prefix over the probes gives each group's slot j < 2P), and for every
// group its list and code range: dl[b][j], dpos[b][j] = (first, end). gcnt[b]
// holds the groups and the parts that the query's cost asks for (see AdcCost).
__global__ __launch_bounds__(kSetupThreads) void adc_setup_kernel(const int32_t *__restrict__ probes, int P,
                                                                const int64_t *__restrict__ offsets, int64_t C,
                                                                int64_t N, AdcCost cost, int32_t *__restrict__ gcnt,
                                                                int32_t *__restrict__ dl,
                                                                longlong2 *__restrict__ dpos)
{
    __shared__ int32_t wsum[kSetupThreads / 64];
    __shared__ int32_t s_g, s_n;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t b = blockIdx.x;
    // thread t takes the contiguous probes [t * per, (t + 1) * per)
    const int per = (P + kSetupThreads - 1) / kSetupThreads;  // <= 16
    int32_t nch[16];
    int64_t o0s[16], o1s[16];
    int32_t tot = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int p = t * per + e;
        nch[e] = 0;
        o0s[e] = o1s[e] = 0;
        if (e < per && p < P) {
            list_range(offsets, C, N, probes[b * P + p], o0s[e], o1s[e]);
            nch[e] = (int32_t)((o1s[e] - o0s[e] + kAdcChunk - 1) / kAdcChunk);
        }
        tot += nch[e];
    }
    // chunks of the query -> group size
    int32_t s = tot;
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) wsum[wave] = s;
    __syncthreads();
    if (t == 0) {
        int32_t n = 0;
        for (int w = 0; w < kSetupThreads / 64; ++w) n += wsum[w];
        s_n = n;
        s_g = max(kAdcMinGroup, (n + P - 1) / P);
    }
    __syncthreads();
    const int32_t G = s_g;
    // groups per list and their exclusive scan over the probes
    int32_t ng = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) ng += (nch[e] + G - 1) / G;
    int32_t incl = ng;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int32_t j = incl - ng;
    for (int w = 0; w < wave; ++w) j += wsum[w];
    const int64_t base = b * 2 * (int64_t)P;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        if (nch[e] == 0) continue;
        const int32_t l = probes[b * P + t * per + e];
        for (int64_t f = o0s[e]; f < o1s[e]; f += (int64_t)G * kAdcChunk, ++j) {
            dl[base + j] = l;
            dpos[base + j] = make_longlong2(f, min(o1s[e], f + (int64_t)G * kAdcChunk));
        }
    }
    if (t == kSetupThreads - 1) {  // the last thread ends past every group
        const float c = (float)j * cost.list + (float)s_n * cost.chunk;
        const float want = fminf(ceilf(c / cost.part), (float)min(P, j));
        gcnt[b] = pack_groups(j, c > 2.0f * (float)cost.parts * cost.part ? max(cost.parts, (int)want) : cost.parts);
    }
}

struct Desc {
    int64_t from, end;  // code positions
    int32_t list;       // -1: none
};

// A wave's SL slices lie in one subspace or, from six on, in two; they cover
// this many dims: so many lanes hold a list's residuals, 64 of them those of a
// step's lists
constexpr int slice_dims(int DS, int SL) { return (SL >= 6 ? 2 : 1) * DS; }

// Part s of the S_b of query b (grid: B * S, then the extra parts): its groups
// s, s + S_b, ..., `lists` of them at a time. DS, SL: dims of a subspace and codeword slices per wave held in
// registers (slice 4 m + q is codewords 64 q .. 64 q + 63 of subspace m, one per
// lane; wave w holds slices SL w .. SL w + SL - 1). SL = 0: codewords of DS dims
// (of 9 to 16 with DS = 16) are read from memory, SL = -1: of more than 16.
template <int DS, int SL>
__global__ __launch_bounds__(kAdcThreads) void adc_scan_kernel(
    const float *__restrict__ Q, int D, const float *__restrict__ cent, int P, const uint32_t *__restrict__ perm,
    const uint8_t *__restrict__ codes, int M, const float *__restrict__ codebooks, int k, int64_t B, int S0, int lists,
    AdcExtra extra, const int32_t *__restrict__ gcnt, const int32_t *__restrict__ dl, const longlong2 *__restrict__ dpos,
    uint64_t *__restrict__ handoff, int32_t *__restrict__ hcnt, uint32_t *__restrict__ ids, float *__restrict__ dist)
{
    __shared__ __attribute__((aligned(16))) float lut[kAdcLutBytes / 4];  // [lists][M][256]
    __shared__ PoolLds pool;
    __shared__ Desc ring[4][kAdcMaxLists];  // descriptors of the steps around the current one
    __shared__ __attribute__((aligned(16))) double res[SL > 0 ? 1 : kAdcMaxLists * kAdcPadD];  // [lists][M][pd]
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    int64_t b = blockIdx.x / S0;
    int part = (int)(blockIdx.x - b * S0);
    if (b >= B) {
        const int64_t e = blockIdx.x - B * S0;
        if (e >= *extra.n) return;
        b = (int64_t)(extra.list[e] >> 32);
        part = (int)(uint32_t)extra.list[e];
    }
    const int S = parts_of(gcnt[b]);
    const int ng = (groups_of(gcnt[b]) - part + S - 1) / S;  // groups of this part
    const int steps = (ng + lists - 1) / lists;
    const int64_t g_first = b * 2 * (int64_t)P + part;
    const float *qb = Q + b * D;
    constexpr int NS = SL > 0 ? SL : 1;
    const int dsub = SL == 0 && DS <= 8 ? DS : D / M;
    const int pd = (dsub + DS - 1) / DS * DS;  // (SL <= 0, from 9 dims on: padded with zeros)
    // dims of the subspaces a wave's slices lie in, from dim wd on
    constexpr int W = slice_dims(DS, SL);
    const int m_lo = wave * NS >> 2;
    const int wd = m_lo * DS + lane % W;
    double w[NS][DS];
    if constexpr (SL > 0) {
        // (16 bytes at a time: single floats, 4 DS bytes apart between lanes, took
        // each line of the codebooks out of L2 once per dim, 14 of a part's 29 us)
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            const int sl = wave * SL + i;
            const f32x4 *src = reinterpret_cast<const f32x4 *>(codebooks + ((int64_t)min(sl, 4 * M - 1) * 64 + lane) * DS);
#pragma unroll
            for (int q = 0; q < DS / 4; ++q) {
                const f32x4 v = src[q];
#pragma unroll
                for (int e = 0; e < 4; ++e) w[i][4 * q + e] = (double)v[e];
            }
        }
    }
    // the residual dims this thread forms for a step's lists: lane W u + d holds
    // dim wd of list u, or (SL = 0) dims of the lists' rows laid end to end
    constexpr int NR = SL > 0 ? 1 : kAdcMaxLists * 256 / kAdcThreads;
    int ru[NR], rd[NR];
    float ql[NR];
#pragma unroll
    for (int e = 0; e < NR; ++e) {
        const int i = t + e * kAdcThreads;
        ru[e] = SL > 0 ? lane / W : i / D;
        rd[e] = SL > 0 ? wd : i % D;
        if (ru[e] >= lists || rd[e] >= D) ru[e] = -1;
        ql[e] = ru[e] >= 0 ? qb[rd[e]] : 0.0f;
    }
    if constexpr (SL <= 0) {
        for (int i = t; i < lists * M * pd; i += kAdcThreads) res[i] = 0.0;
    }
    pool_init(pool);
    auto load_desc = [&](int step) __attribute__((always_inline)) {
        Desc v{0, 0, -1};
        if (t < lists && step * lists + t < ng) {
            const int64_t slot = g_first + (int64_t)(step * lists + t) * S;
            const longlong2 rg = dpos[slot];
            v = Desc{rg.x, rg.y, dl[slot]};
        }
        return v;
    };
    // this thread's centroid dims of a step's lists (their descriptors are in the ring)
    struct Dims {
        float v[NR];
    };
    auto load_cent = [&](int step) __attribute__((always_inline)) {
        Dims c;
#pragma unroll
        for (int e = 0; e < NR; ++e) {
            const int32_t l = ru[e] >= 0 ? ring[step & 3][ru[e]].list : -1;
            c.v[e] = l >= 0 ? cent[(int64_t)l * D + rd[e]] : 0.0f;
        }
        return c;
    };
    // The tables of one step from its lanes' centroid dims. The residual r = q -
    // c (fp32, as defined) is the same for every lane: it is formed once per
    // list and dim, in the lane that holds the dim, and read from there into
    // scalar registers (LDS broadcasts of it took the whole LDS bandwidth).
    auto build = [&](int step, const Dims &cl, float *buf) __attribute__((always_inline)) {
        const int nl = min(lists, ng - step * lists);
        const double rl = (double)(ql[0] - cl.v[0]);
        const int rlo = (int)(uint32_t)__double_as_longlong(rl), rhi = (int)(uint32_t)(__double_as_longlong(rl) >> 32);
        for (int u = 0; u < nl; ++u) {
            float *lt = buf + (size_t)u * M * kPqK;
            if constexpr (SL > 0) {
                double r[DS];
                int m_of = -1;
#pragma unroll
                for (int i = 0; i < SL; ++i) {
                    const int sl = wave * SL + i;
                    if (sl < 4 * M) {
                        const int m = (sl >> 2) - m_lo;
                        if (SL != 6 ? i % 4 == 0 : m != m_of) {  // (uniform) the slice's subspace
                            m_of = m;
#pragma unroll
                            for (int d = 0; d < DS; ++d) {
                                const int from = W * u + m * DS + d;
                                r[d] = __hiloint2double(__builtin_amdgcn_readlane(rhi, from),
                                                        __builtin_amdgcn_readlane(rlo, from));
                            }
                        }
                        double acc = 0.0;
#pragma unroll
                        for (int d = 0; d < DS; ++d) {
                            const double v = r[d] - w[i][d];
                            acc = fma(v, v, acc);
                        }
                        lt[sl * 64 + lane] = (float)acc;
                    }
                }
            }
        }
    };
    // The same from memory, for the widths without a register layout: the
    // residuals of the step's lists lie in LDS in fp64, padded to DS dims a
    // subspace, and a wave reads U slices' codewords (the next ones while these
    // are in use) and converts them once for all of the lists. Bound by the LDS
    // broadcasts of the residuals, which U slices share. 512 queries x 32 lists
    // of 244 codes, 32 subspaces of 8: 1.93 -> 0.34 ms (a
    // float a load, the residual formed anew by every lane).
    auto build_memory = [&](int step, const Dims &cl) __attribute__((always_inline)) {
        constexpr int U = DS <= 4 ? 4 : DS <= 8 ? 2 : 1;
        constexpr bool BLOCKS = SL < 0;  // subspaces of more than 16 dims go through in blocks of 16
        const int nl = min(lists, ng - step * lists);
#pragma unroll
        for (int e = 0; e < NR; ++e)
            if (ru[e] >= 0) res[(ru[e] * M + rd[e] / dsub) * pd + rd[e] % dsub] = (double)(ql[e] - cl.v[e]);
        __syncthreads();
        auto load = [&](int un, int blk, float(&c)[U][DS]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const float *w0 = codebooks + ((int64_t)(un * U + j) * 64 + lane) * dsub;
#pragma unroll
                for (int q = 0; q < (DS + 3) / 4; ++q) {
                    const int d0 = blk * DS + 4 * q;
                    if (DS % 4 == 0 && (DS <= 8 || (dsub & 3) == 0)) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(w0 + min(d0, dsub - 4));
#pragma unroll
                        for (int e = 0; e < 4; ++e) c[j][4 * q + e] = d0 < dsub ? v[e] : 0.0f;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (4 * q + e < DS) {
                                const float v = w0[min(d0 + e, dsub - 1)];
                                c[j][4 * q + e] = d0 + e < dsub ? v : 0.0f;
                            }
                        }
                    }
                }
            }
        };
        const int nu = 4 * M / U, nb = pd / DS;
        float c[U][DS];
        if (wave < nu) load(wave, 0, c);
        double acc[BLOCKS ? kAdcMaxLists : 1];
        for (int un = wave, blk = 0; un < nu;) {
            double w[U][DS];
#pragma unroll
            for (int j = 0; j < U; ++j)
#pragma unroll
                for (int d = 0; d < DS; ++d) w[j][d] = (double)c[j][d];
            const bool last = !BLOCKS || blk + 1 == nb;
            const int nun = last ? un + kAdcWaves : un, nblk = last ? 0 : blk + 1;
            if (nun < nu) load(nun, nblk, c);
            const int m = un * U >> 2;
            const double *r0 = res + m * pd + blk * DS;
            float *l0 = lut + m * kPqK + (un * U & 3) * 64 + lane;
            auto one = [&](int u, double &a) __attribute__((always_inline)) {
                double r[DS];
#pragma unroll
                for (int d = 0; d < DS; ++d) r[d] = r0[u * M * pd + d];
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    double s = BLOCKS && blk > 0 ? a : 0.0;
#pragma unroll
                    for (int d = 0; d < DS; ++d) {  // (the padding adds exact zeros)
                        const double v = r[d] - w[j][d];
                        s = fma(v, v, s);
                    }
                    if (BLOCKS) a = s;
                    if (last) l0[u * M * kPqK + 64 * j] = (float)s;
                }
            };
            if constexpr (BLOCKS) {
#pragma unroll
                for (int u = 0; u < kAdcMaxLists; ++u)
                    if (u < nl) one(u, acc[u]);
            } else {
#pragma unroll 1
                for (int u = 0; u < nl; ++u) one(u, acc[0]);
            }
            un = nun;
            blk = nblk;
        }
    };
    // a code is SL words, or whole words of which NW are loaded at a time
    constexpr int NW = SL > 0 ? SL : 8;
    const bool words = SL > 0 ? M == 4 * SL : (M & 3) == 0;
    auto load_code = [&](int64_t pos, uint32_t(&cw)[NW]) __attribute__((always_inline)) {
        const uint32_t *a = reinterpret_cast<const uint32_t *>(codes + pos * M);
#pragma unroll
        for (int e = 0; e < NW; ++e) cw[e] = a[SL > 0 || 4 * e < M ? e : 0];
    };
    // Loads are issued a table build ahead of their use: a step's descriptors
    // three steps, its centroid dims one step, its codes one build. (Two table
    // buffers of half as many lists, a build beside the scan before it, were
    // slower: 1.31 against 1.20 ms.)
    for (int i = 0; i < 3; ++i) {
        const Desc v = load_desc(i);
        if (t < lists) ring[i][t] = v;
    }
    Desc ahead = load_desc(3);
    __syncthreads();
    Dims cl = load_cent(0);
    int room = kAdcPool;  // places the pool has at least
    for (int step = 0; step < steps; ++step) {
        const Desc *ds = ring[step & 3];
        const int nl = min(lists, ng - step * lists);
        if (t < lists) ring[(step + 3) & 3][t] = ahead;  // (read from the next barrier on)
        ahead = load_desc(step + 4);
        // code i of the step's groups laid end to end: list u, position
        int64_t total = 0;
        for (int u = 0; u < nl; ++u) total += ds[u].end - ds[u].from;
        auto locate = [&](int64_t i, int &u) __attribute__((always_inline)) {
            for (u = 0;; ++u) {
                const int64_t from = ds[u].from, len = ds[u].end - from;
                if (i < len) return from + i;
                i -= len;
            }
        };
        int cu = 0;
        uint32_t cw[NW], id = 0;
        if (t < total) {
            const int64_t pos = locate(t, cu);
            id = perm[pos];
            // (the number of words is known at compile time: a branch per word
            // would wait for each load before the next)
            if (words) load_code(pos, cw);
        }
        const Dims cc = cl;
        cl = load_cent(step + 1);
        if constexpr (SL > 0)
            build(step, cc, lut);
        else
            build_memory(step, cc);
        __syncthreads();
        for (int64_t c0 = 0; c0 < total; c0 += kAdcThreads) {
            if (room < kAdcThreads) {  // (uniform)
                pool_room(pool, k);
                room = kAdcPool - (int)pool.n;
                __syncthreads();  // every thread has read n before anyone appends
            }
            room -= (int)min((int64_t)kAdcThreads, total - c0);
            uint64_t key = kNoKey;
            const bool have = c0 + t < total;
            if (have) {
                const float *lt;
                float acc = 0.0f;
                if (words) {
                    int64_t pos = 0;
                    if (c0 > 0 || SL <= 0) pos = locate(c0 + t, cu);
                    if (c0 > 0) {
                        id = perm[pos];
                        load_code(pos, cw);
                    }
                    lt = lut + (size_t)cu * M * kPqK;
#pragma unroll
                    for (int e = 0; e < NW; ++e) {
                        if (SL > 0 || 4 * e < M) {
                            const float *l4 = lt + 4 * e * kPqK;
                            acc = acc + l4[0 * kPqK + (cw[e] & 0xFFu)];
                            acc = acc + l4[1 * kPqK + ((cw[e] >> 8) & 0xFFu)];
                            acc = acc + l4[2 * kPqK + ((cw[e] >> 16) & 0xFFu)];
                            acc = acc + l4[3 * kPqK + (cw[e] >> 24)];
                        }
                    }
                    if constexpr (SL <= 0) {
                        const uint32_t *a = reinterpret_cast<const uint32_t *>(codes + pos * M);
                        for (int m = 4 * NW; m < M; m += 4) {
                            const uint32_t x = a[m / 4];
                            acc = acc + lt[(m + 0) * kPqK + (x & 0xFFu)];
                            acc = acc + lt[(m + 1) * kPqK + ((x >> 8) & 0xFFu)];
                            acc = acc + lt[(m + 2) * kPqK + ((x >> 16) & 0xFFu)];
                            acc = acc + lt[(m + 3) * kPqK + (x >> 24)];
                        }
                    }
                } else {
                    const int64_t pos = locate(c0 + t, cu);
                    lt = lut + (size_t)cu * M * kPqK;
                    const uint8_t *a = codes + pos * M;
                    if (c0 > 0) id = perm[pos];
                    int m = 0;
                    if ((M & 3) == 0) {
                        for (; m < M; m += 4) {
                            const uint32_t x = *reinterpret_cast<const uint32_t *>(a + m);
                            acc = acc + lt[(m + 0) * kPqK + (x & 0xFFu)];
                            acc = acc + lt[(m + 1) * kPqK + ((x >> 8) & 0xFFu)];
                            acc = acc + lt[(m + 2) * kPqK + ((x >> 16) & 0xFFu)];
                            acc = acc + lt[(m + 3) * kPqK + (x >> 24)];
                        }
                    }
                    for (; m < M; ++m) acc = acc + lt[m * kPqK + a[m]];
                }
                key = ((uint64_t)f2o(acc) << 32) | id;
            }
            pool_add(pool, key, have, pool.thr);
        }
        __syncthreads();
    }
    const int n = (int)pool.n;
    __syncthreads();
    if (n > k) pool_trim(pool, k);
    if (S == 1) {
        pool_finish(pool, k, b, ids, dist);
        return;
    }
    const int64_t slot = b * P + part;
    const int m = min(n, k);
    if (t < m) handoff[slot * k + t] = pool.key[t];
    if (t == 0) hcnt[slot] = m;
}

// Query b's parts, 16 at a time: wave w takes the keys of part p0 + w. Every
// query, or (split given) those that have extra parts.
__global__ __launch_bounds__(kAdcThreads) void adc_merge_kernel(const uint64_t *__restrict__ handoff,
                                                               const int32_t *__restrict__ hcnt,
                                                               const int32_t *__restrict__ gcnt, int P,
                                                               const int32_t *__restrict__ split,
                                                               const int32_t *__restrict__ nsplit, int k,
                                                               uint32_t *__restrict__ ids, float *__restrict__ dist)
{
    __shared__ PoolLds pool;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (split && (int)blockIdx.x >= *nsplit) return;
    const int64_t b = split ? split[blockIdx.x] : blockIdx.x;
    const int S = parts_of(gcnt[b]);
    pool_init(pool);
    for (int p0 = 0; p0 < S; p0 += kAdcWaves) {
        int most = 0;
        for (int p = p0; p < min(S, p0 + kAdcWaves); ++p) most = max(most, hcnt[b * P + p]);
        const int p = p0 + wave;
        const int n = p < S ? hcnt[b * P + p] : 0;
        const uint64_t *in = handoff + (b * P + min(p, S - 1)) * (int64_t)k;
        for (int i0 = 0; i0 < most; i0 += 64) {
            const int i = i0 + lane;
            const uint64_t key = i < n ? in[i] : kNoKey;
            pool_room(pool, k);
            pool_add(pool, key, i < n, pool.thr);
        }
    }
    __syncthreads();
    const int n = (int)pool.n;
    __syncthreads();
    if (n > k) pool_trim(pool, k);
    pool_finish(pool, k, b, ids, dist);
}

using ScanKernel = decltype(&adc_scan_kernel<8, 4>);

// The kernel for a width: codebooks in registers where a wave's slices are at
// most 32 doubles a thread (more spill) and share their subspaces evenly, from memory
// otherwise. 2,048 queries x 96 lists of 122 codes, registers against memory:
// 16 subspaces of 8 dims 1.12 and 1.46 ms, 32 of 4 1.41 and 2.30, 24 of 4 1.16 and
// 1.41; 12 of 8 (slices in threes) 1.24 and 1.05, 20 of 8 (fives) 1.92 and 1.73, 10
// of 16 (48 floats) 2.98 and 1.78.
ScanKernel scan_kernel(int dsub, int M, int &held)
{
    const int sl = (M + 3) / 4;
    held = 64 / slice_dims(dsub, sl);
    if (dsub == 8) {
        switch (sl) {
        case 1: return adc_scan_kernel<8, 1>;
        case 2: return adc_scan_kernel<8, 2>;
        case 4: return adc_scan_kernel<8, 4>;
        }
    } else if (dsub == 4) {
        switch (sl) {
        case 2: return adc_scan_kernel<4, 2>;
        case 4: return adc_scan_kernel<4, 4>;
        case 6: return adc_scan_kernel<4, 6>;
        case 8: return adc_scan_kernel<4, 8>;
        }
    } else if (dsub == 16) {
        switch (sl) {
        case 1: return adc_scan_kernel<16, 1>;
        case 2: return adc_scan_kernel<16, 2>;
        }
    }
    held = kAdcMaxLists;
    switch (dsub) {
    case 1: return adc_scan_kernel<1, 0>;
    case 2: return adc_scan_kernel<2, 0>;
    case 3: return adc_scan_kernel<3, 0>;
    case 4: return adc_scan_kernel<4, 0>;
    case 5: return adc_scan_kernel<5, 0>;
    case 6: return adc_scan_kernel<6, 0>;
    case 7: return adc_scan_kernel<7, 0>;
    case 8: return adc_scan_kernel<8, 0>;
    }
    return dsub <= 16 ? adc_scan_kernel<16, 0> : adc_scan_kernel<16, -1>;
}

// Parts per query: the number for which the rounds of workgroups (one per CU)
// end soonest. A part costs about 15 us whatever it holds (codebooks, pool, final
// trim) and 1.2 us per list of ordinary length (more where a step holds fewer
// than four), that is 12 lists; lists of thousands of codes cost their scan;
// several parts cost the merge, about five lists. 8 queries x 64 lists: 32 parts
// of two lists, 45 us (98 with a workgroup per group of a list); 149 queries x 7:
// one part, 28 us (49).
constexpr double kPartCost = 12.0;     // lists
constexpr double kCodesCost = 2048.0;  // codes scanned in the time of a list's table

int adc_parts(int64_t B, int P, double list, int num_cus)
{
    int best = 1;
    double cost = 0.0;
    for (int s = 1; s <= P; ++s) {
        const double rounds = (double)((B * s + num_cus - 1) / num_cus);
        const double t = rounds * (kPartCost + ((P + s - 1) / s) * list) + (s > 1 ? 5.0 : 0.0);
        if (s == 1 || t < cost) {
            best = s;
            cost = t;
        }
        if (B * s > 4 * (int64_t)num_cus) break;  // more rounds of less only add the fixed cost
    }
    return best;
}

}  // namespace

hipError_t launch_adc_scan(const float *Q, int64_t B, int D, const float *cent, int64_t C,
                           const int32_t *probes, int P, const int64_t *offsets, const uint32_t *perm,
                           int64_t N, const uint8_t *codes, int M, const float *codebooks, int k,
                           const AdcScratch &w, uint32_t *ids, float *dist, int num_cus, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    // lists whose tables are built at a time: as many as fit LDS, and whose
    // residuals a wave's lanes hold
    int held = 0;
    const ScanKernel scan = scan_kernel(D / M, M, held);
    const int lists = std::max(1, std::min(std::min(held, kAdcMaxLists), kAdcLutBytes / (M * kPqK * 4)));
    if ((size_t)lists * M * kPqK * 4 > (size_t)kAdcLutBytes) return hipErrorInvalidValue;
    const double table = std::max(1.0, 4.0 / held), chunk = kAdcChunk / kCodesCost;
    const double list = table + (double)(N / C) / kCodesCost;
    const int S = adc_parts(B, P, list, num_cus);
    // Extra parts: where lists are skewed, one query may hold many times the
    // others' codes, and the workgroup that scans them ends long after the rest
    // (256 queries x 64 of 16,384 Zipf lists of 10M codes: 1.48 ms, 0.73 with a
    // workgroup per group of a list, 0.37 with extra parts). The lengths are on
    // the device, so the extra parts are decided there, wherever the codes are
    // enough to make a query twice as heavy as its parts are meant for; the two
    // launches take 5 us where no query is.
    const double part = std::max(kPartCost, (double)P / S * list);
    AdcExtra x{};
    if (S < P && (double)N / kCodesCost > 2.0 * S * part) {
        x.cap = (int)std::min<int64_t>(2 * (int64_t)num_cus, B * (P - S));
        x.list = w.handoff + B * P * k;  // parts hand over below B * P slots of the 2 B * P
        x.split = (int32_t *)(x.list + x.cap);  // at most B, after at most B (P - 1) of B P k entries
        x.n = w.hcnt + B * P;                   // (P >= 2 here)
        x.nsplit = w.hcnt + B * P + 1;
    }
    const AdcCost cost{(float)table, (float)chunk, x.cap > 0 ? (float)part : INFINITY, S};
    hipLaunchKernelGGL(adc_setup_kernel, dim3((unsigned)B), dim3(kSetupThreads), 0, s, probes, P, offsets, C, N, cost,
                       w.gcnt, w.dl, w.dpos);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (x.cap > 0) {
        hipLaunchKernelGGL(adc_extra_kernel, dim3(1), dim3(kAdcThreads), 0, s, B, S, w.gcnt, x);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(scan, dim3((unsigned)(B * S + x.cap)), dim3(kAdcThreads), 0, s, Q, D, cent, P, perm,
                       codes, M, codebooks, k, B, S, lists, x, w.gcnt, w.dl, w.dpos, w.handoff, w.hcnt, ids, dist);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (S > 1 || x.cap > 0)
        hipLaunchKernelGGL(adc_merge_kernel, dim3((unsigned)(S > 1 ? B : std::min<int64_t>(B, x.cap))), dim3(kAdcThreads),
                           0, s, w.handoff, w.hcnt, w.gcnt, P, S > 1 ? nullptr : x.split, x.nsplit, k, ids, dist);
    return hipGetLastError();
}

}  // namespace ivf
