// Screening of fp32 rows and queries on f16 MFMA (gfx950).
//
// The results stay those of the fp64 definition; what f16 does here is only to
// discard centroids that a bound shows to be too far (the int8 planes do the
// same for uint8 data). Rows and centroids are scaled by one power of two
// per call and rounded to f16, X = s x, C = s c, and the screening value of a
// centroid is
//     v(c) = Xh.Ch - ||C||^2 / 2          (f16 products, fp32 accumulation),
// which orders the centroids like -||x - c||^2. With the residuals
// rx = ||X - Xh||_2 (measured per row) and rc = max_c ||C - Ch||_2 (measured
// by the quantisation) Cauchy-Schwarz gives
//     |v(c) - (X.C - ||C||^2 / 2)| <= B = rx M + ||Xh|| rc
//                                       + g (M^2 / 2 + ||Xh|| (M + rc)),
// M >= max ||C||, g = the rounding of DP products added in fp32 in any order
// (gamma_n with n = 2 (DP + 2) and u = 2^-23: twice the standard bound at
// twice the unit roundoff, which also covers truncating adders). Values an f16
// cannot hold as a normal number are rounded to zero here, so the bound does
// not depend on how the unit treats subnormals, and a row with a value beyond
// f16's range is never settled here.
//
// Assignment keeps the three best values per row like the other one-pass
// screens: a gap above T >= 2 B settles the row, two candidates are compared in
// fp64, more are collected by a second pass and compared in fp64, and the fp32
// screen takes the rows (or the call) for which that is too much. Routing takes
// its threshold from sample values, keeps every centroid within the window and
// ranks by fp64 distance as before.
//
// v_mfma_f32_32x32x16_f16 runs at 16 times the rate of the fp32 instruction
// (2.5 PFLOP/s against 157 TFLOP/s), and vector instructions issue beside it
// where the fp32 MFMA blocks them. 500,000 x 96 rows against 16,384 centroids:
// 12.1 ms on fp32 MFMA, 1.65 here (950 TFLOP/s); 10,000 x 96 queries against 262,144: filter
// 3.89 ms, 0.80 here.
#include "exact.h"
#include "f16_bound.h"
#include "ivf_internal.h"
#include "qstage.h"
#include "tile_lists.h"
#include "wave_ops.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace ivf {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kInf = __builtin_huge_valf();

// A tile: W waves of RB blocks of 32 rows. Each staged centroid fragment feeds
// RB MFMAs (a fragment read per MFMA would take the CU's whole LDS bandwidth);
// two blocks of rows fit the register file up to 128 dims. A staged chunk holds
// SUB sub-chunks of 64 centroids, two chunks in LDS.
template <int DP>
struct Geo {
    static constexpr int KS = DP / 16;  // K-steps
    static constexpr int RB = DP <= 128 ? 2 : 1;
    static constexpr int SUB = DP <= 64 ? 4 : DP <= 128 ? 2 : 1;
    static constexpr int CHUNK = SUB * kQChunk;
    static constexpr int NB = 2 * SUB;  // 32-centroid blocks per chunk
    static constexpr int W = 8;
    static constexpr int NT = W * 64;
    static constexpr int ROWS = W * 32 * RB;
    using St = QStager<2 * DP, NT, 1>;
    static constexpr int CS = (St::kBytes + 15) / 16 * 16;
    static constexpr int LDS = 2 * SUB * CS;
};

// ------------------------------------------------------------ quantisation
__global__ __launch_bounds__(256) void quantize_f16_kernel(const float *__restrict__ cent, int64_t C, int D, int DP,
                                                           int64_t Cpad, const uint32_t *__restrict__ mc2_bits,
                                                           uint16_t *__restrict__ plane, float *__restrict__ nbias,
                                                           uint32_t *__restrict__ rc_bits)
{
    quantize_f16_rows(cent, C, D, DP, Cpad, mc2_bits, plane, nbias, rc_bits);
}

// ------------------------------------------------------------ rows
// This lane's half of a row (row < 0: none) as B fragments: K-step k of lane
// half h holds dims 16 k + 8 h .. + 7. The norms are summed over both halves;
// a row with a value beyond f16's range gets an infinite residual.
template <int DP>
__device__ __forceinline__ RowNorms load_row_f16(const float *__restrict__ X, int64_t row, int D, int h, float sc,
                                                 f16x8 (&x)[DP / 16])
{
    const float *p = X + (row < 0 ? 0 : row) * (int64_t)D + 8 * h;
    RowAcc acc;
#pragma unroll
    for (int k = 0; k < DP / 16; ++k) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int d = 16 * k + 8 * h + 4 * q;
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (row >= 0 && d < D) v = *reinterpret_cast<const float4 *>(p + 16 * k + 4 * q);
            const float va[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) x[k][4 * q + e] = acc.add(va[e] * sc);
        }
    }
    acc.r2 += __shfl_xor(acc.r2, 32);
    acc.n2 += __shfl_xor(acc.n2, 32);
    acc.over = (__shfl_xor((int)acc.over, 32) != 0) | acc.over;
    return acc.norms();
}

// ------------------------------------------------------------ epilogues
__device__ __forceinline__ float max3f(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

__device__ __forceinline__ float max16f(const f32x16 &p)
{
    return fmaxf(fmaxf(max3f(max3f(p[0], p[1], p[2]), max3f(p[3], p[4], p[5]), max3f(p[6], p[7], p[8])),
                       max3f(max3f(p[9], p[10], p[11]), max3f(p[12], p[13], p[14]), p[15])),
                 -kInf);
}

// Largest value over the two half-lanes of a row (a VALU lane swap).
__device__ __forceinline__ float halves_max(float v)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float med3f(float a, float b, float c) { return __builtin_amdgcn_fmed3f(a, b, c); }

struct NoCtx {};

// Assignment: the three largest values a lane has kept for its row, the ids of
// two, the keep threshold t3 (values at or below it cannot change the
// certificate's decision) and the window T.
struct Top3f {
    static constexpr int kPieces = 1;
    float k1, k2, k3;
    int i1, i2;
    float t3, T;
};

__device__ __forceinline__ void top3_push(Top3f &t, float v, int id)
{
    const bool gt1 = v > t.k1;
    const bool gt2 = v > t.k2;
    t.k3 = med3f(v, t.k2, t.k3);
    t.k2 = med3f(v, t.k1, t.k2);
    t.k1 = gt1 ? v : t.k1;
    const int j2 = gt2 ? id : t.i2;
    t.i2 = gt1 ? t.i1 : j2;
    t.i1 = gt1 ? id : t.i1;
}

__device__ __forceinline__ void top3_raise(Top3f &t) { t.t3 = fmaxf(t.k3, halves_max(t.k1) - t.T); }

template <int g>
__device__ __forceinline__ void top3_group(const f32x16 &p, int idp, Top3f &st)
{
    const float v0 = p[4 * g], v1 = p[4 * g + 1], v2 = p[4 * g + 2], v3 = p[4 * g + 3];
    const float m = fmaxf(max3f(v0, v1, v2), v3);
    if (__builtin_expect(__any(m > st.t3), 0)) {
        // the group's best (the lowest id among equal values) first
        const int e1 = v0 == m ? 0 : v1 == m ? 1 : v2 == m ? 2 : 3;
        top3_push(st, m, idp + 8 * g + e1);
        top3_raise(st);
        // the other three only when some lane still needs one of them
        const float r0 = e1 == 0 ? -kInf : v0, r1 = e1 == 1 ? -kInf : v1;
        const float r2 = e1 == 2 ? -kInf : v2, r3 = e1 == 3 ? -kInf : v3;
        if (__builtin_expect(__any(fmaxf(max3f(r0, r1, r2), r3) > st.t3), 0)) {
            top3_push(st, r0, idp + 8 * g);
            top3_push(st, r1, idp + 8 * g + 1);
            top3_push(st, r2, idp + 8 * g + 2);
            top3_push(st, r3, idp + 8 * g + 3);
            top3_raise(st);
        }
    }
}

template <int piece>
__device__ __forceinline__ void tile_test(const f32x16 &p, int idp, Top3f &st, NoCtx &)
{
    if (__builtin_expect(__any(max16f(p) > st.t3), 0)) {
        top3_group<0>(p, idp, st);
        top3_group<1>(p, idp, st);
        top3_group<2>(p, idp, st);
        top3_group<3>(p, idp, st);
    }
}

// Collecting pass over listed rows: plane rows with a value of at least thr,
// at most kResolveCand queued per lane (LDS), all counted.
struct CollectF {
    static constexpr int kPieces = 1;
    float thr;
    int qn;
    int32_t *q;
    int stride;
};

template <int piece>
__device__ __forceinline__ void tile_test(const f32x16 &p, int idp, CollectF &st, NoCtx &)
{
    if (__builtin_expect(__any(max16f(p) >= st.thr), 0)) {
        uint32_t hit = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) hit |= p[r] >= st.thr ? 1u << r : 0u;
        while (__any(hit != 0)) {
            if (hit != 0) {
                const int r = __builtin_ctz(hit);
                if (st.qn < kResolveCand) st.q[st.qn * st.stride] = idp + 8 * (r >> 2) + (r & 3);
                ++st.qn;
                hit &= hit - 1u;
            }
        }
    }
}

// Threshold sample: the smallest key (-v) of every 16 visited centroids, the
// two half-lanes of a row holding 8 of them each.
struct KeysF {
    static constexpr int kPieces = 1;
    float *krow;     // the row's group minima; null: no row
    int lo, hi;      // visited positions of this range
};

template <int piece>
__device__ __forceinline__ void tile_test(const f32x16 &p, int idp, KeysF &st, NoCtx &)
{
    float m[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        const int r = 8 * g;
        m[g] = halves_max(fmaxf(max3f(p[r], p[r + 1], p[r + 2]), fmaxf(max3f(p[r + 3], p[r + 4], p[r + 5]), fmaxf(p[r + 6], p[r + 7]))));
    }
    const int id0 = idp & ~31;  // a block's 32 positions are all in the range or all outside
    if (st.krow && (threadIdx.x & 32) == 0 && id0 >= st.lo && id0 < st.hi)
        *reinterpret_cast<float2 *>(st.krow + (id0 >> 4)) = make_float2(-m[0], -m[1]);
}

// Candidate filter: every group of four values with one at or above the row's
// threshold goes, whole, to a queue in LDS that the wave's lanes share (the
// lanes that pass take consecutive places, so a full queue is full of groups
// that pass); a flush looks at the four values and reserves their places in
// the query's list with one atomic per entry. About 0.2 % of the values are
// candidates, so some lane passes in 40 % of the groups: a queue per lane had
// to be flushed as soon as one lane's was full.
constexpr int kWaveQueue = 128;

template <int RB>
struct FilterCtx {
    float4 *v;         // this wave's queue: four values,
    uint2 *meta;       // first id and row of the wave (0 .. 32 RB - 1)
    const float *tv;   // the wave's thresholds by row
    int n;             // entries (wave-uniform)
    int64_t row0;      // the wave's first row
    uint32_t *cand_cnt;
    uint2 *cand;
    int L;
};

struct FilterF {
    static constexpr int kPieces = 4;
    float tv;   // keep v >= tv (+inf: no row)
    int r;      // row of the wave
};

template <int RB>
__device__ __forceinline__ void filter_flush(FilterCtx<RB> &c)
{
    // the queue is this wave's own: its LDS accesses stay in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int lane = threadIdx.x & 63;
    for (int i = lane; i < c.n; i += 64) {
        const float4 v4 = c.v[i];
        const uint2 mt = c.meta[i];
        const float tv = c.tv[mt.y];
        const float va[4] = {v4.x, v4.y, v4.z, v4.w};
        const uint32_t n = (va[0] >= tv) + (va[1] >= tv) + (va[2] >= tv) + (va[3] >= tv);
        const int64_t row = c.row0 + mt.y;
        uint32_t slot = atomicAdd(c.cand_cnt + row, n);
        uint2 *dst = c.cand + row * c.L;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (va[e] >= tv) {
                if (slot < (uint32_t)c.L) dst[slot] = make_uint2(__float_as_uint(-va[e]), mt.x + e);
                ++slot;
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    c.n = 0;
}

template <int g, int RB>
__device__ __forceinline__ void tile_test(const f32x16 &p, int idp, FilterF &st, FilterCtx<RB> &c)
{
    const float m = fmaxf(max3f(p[4 * g], p[4 * g + 1], p[4 * g + 2]), p[4 * g + 3]);
    const bool pass = m >= st.tv;
    const uint64_t mask = __ballot(pass);
    if (mask) {
        if (c.n > kWaveQueue - 64) filter_flush(c);
        if (pass) {
            const int at = c.n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
            c.v[at] = make_float4(p[4 * g], p[4 * g + 1], p[4 * g + 2], p[4 * g + 3]);
            c.meta[at] = make_uint2((uint32_t)(idp + 8 * g), (uint32_t)st.r);
        }
        c.n += (int)__popcll(mask);
    }
}

// ------------------------------------------------------------ the scan
// Piece i of n test pieces of the previous block runs after this K-step: an
// even spread, one step late (the last MFMA's result is then ready).
constexpr int test_step(int i, int n, int KS)
{
    return i * KS / n + 1 < KS ? i * KS / n + 1 : KS - 1;
}

template <int I, int T, int KS, int RB, class S, class X>
__device__ __forceinline__ void tests_at(const f32x16 (&p)[RB], int idp, S (&st)[RB], X &ctx)
{
    constexpr int P = S::kPieces;
    if constexpr (I < RB * P) {
        if constexpr (test_step(I, RB * P, KS) == T) tile_test<I % P>(p[I / P], idp, st[I / P], ctx);
        tests_at<I + 1, T, KS, RB>(p, idp, st, ctx);
    }
}

template <int I, int RB, class S, class X>
__device__ __forceinline__ void drain(const f32x16 (&p)[RB], int idp, S (&st)[RB], X &ctx)
{
    constexpr int P = S::kPieces;
    if constexpr (I < RB * P) {
        tile_test<I % P>(p[I / P], idp, st[I / P], ctx);
        drain<I + 1, RB>(p, idp, st, ctx);
    }
}

__device__ __forceinline__ f32x16 load_bias(const float *B)
{
    f32x16 b;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f32x4 u = *reinterpret_cast<const f32x4 *>(B + 8 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) b[4 * g + e] = u[e];
    }
    return b;
}

// K-steps T .. KS-1 of one 32-centroid block against the wave's row blocks,
// starting from the biases; the tests of the block before run between them,
// and each fragment register is refilled from the next block (nA, nB) right
// after its last MFMA.
template <int DP, int RB, int T, class S, class X>
__device__ __forceinline__ void f16_block(f16x8 (&f)[DP / 16], const f16x8 (&x)[RB][DP / 16], f32x16 &bias,
                                          f32x16 (&c)[RB], const f32x16 (&p)[RB], int idp, S (&st)[RB], X &ctx,
                                          const char *nA, const float *nB)
{
    constexpr int KS = DP / 16;
    if constexpr (T < KS) {
        if constexpr (T == 0) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) c[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[0], x[rb][0], bias, 0, 0, 0);
            asm volatile("" ::"v"(bias));  // no MFMA is the biases' last reader: no copy of them first
            bias = load_bias(nB);
        } else {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) c[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[T], x[rb][T], c[rb], 0, 0, 0);
        }
        f[T] = *reinterpret_cast<const f16x8 *>(nA + 32 * T);
        tests_at<0, T, KS, RB>(p, idp, st, ctx);
        __builtin_amdgcn_sched_barrier(0);
        f16_block<DP, RB, T + 1>(f, x, bias, c, p, idp, st, ctx, nA, nB);
    }
}

template <class F, int... I>
__device__ __forceinline__ void for_each_index(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// nch staged chunks from visited sub-chunk v0 on (visited sub-chunk u is plane
// sub-chunk u * cst) against the wave's rows. The ids handed to the tests are
// visited positions 64 u + i. The barrier before the last block of a chunk
// makes the next chunk visible, and the one after next is then fetched into
// the buffer no wave reads any more.
template <int DP, class S, class X>
__device__ __forceinline__ void f16_scan(const uint16_t *__restrict__ plane, const float *__restrict__ nbias,
                                         int64_t cpad, int64_t v0, int64_t cst, int nch,
                                         const f16x8 (&xf)[Geo<DP>::RB][DP / 16], S (&st)[Geo<DP>::RB], X &ctx,
                                         char *__restrict__ lds)
{
    using G = Geo<DP>;
    using St = typename G::St;
    constexpr int RB = G::RB, NB = G::NB, CS = G::CS, SB = G::SUB * G::CS;
    constexpr int BLK = 32 * St::kPitch;
    const int lane = threadIdx.x & 63;
    const int h = lane >> 5;
    const int jl = lane & 31;
    const char *A0 = lds + jl * St::kPitch + 16 * h;
    const char *B0 = lds + St::kBias + 16 * h;
    const int idh = 4 * h + (int)(v0 * kQChunk);
    auto abuf = [&](int jj, int b) { return A0 + (jj & 1) * SB + (b >> 1) * CS + (b & 1) * BLK; };
    auto bbuf = [&](int jj, int b) {
        return reinterpret_cast<const float *>(B0 + (jj & 1) * SB + (b >> 1) * CS) + 32 * (b & 1);
    };
    St q;
    q.init();
    auto fetch = [&](int jj) {
        char *buf = lds + (jj & 1) * SB;
#pragma unroll
        for (int u = 0; u < G::SUB; ++u)
            q.fetch(reinterpret_cast<const int8_t *>(plane), reinterpret_cast<const int32_t *>(nbias),
                    (v0 + (int64_t)jj * G::SUB + u) * cst * kQChunk, cpad, buf + u * CS);
    };
    fetch(0);
    __syncthreads();
    fetch(1);

    // set B starts as a block of lowest values: the first tests keep nothing
    f32x16 sa[RB], sb[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) sb[rb][r] = -kInf;
    f32x16 bias = load_bias(bbuf(0, 0));
    f16x8 f[DP / 16];
#pragma unroll
    for (int k = 0; k < DP / 16; ++k) f[k] = *reinterpret_cast<const f16x8 *>(abuf(0, 0) + 32 * k);

    auto block = [&](int jj, auto bc) {
        constexpr int b = decltype(bc)::value;
        const char *nA = b + 1 < NB ? abuf(jj, b + 1) : abuf(jj + 1, 0);
        const float *nB = b + 1 < NB ? bbuf(jj, b + 1) : bbuf(jj + 1, 0);
        const int idp = idh + jj * G::CHUNK + 32 * b - 32;
        if constexpr (b % 2 == 0)
            f16_block<DP, RB, 0>(f, xf, bias, sa, sb, idp, st, ctx, nA, nB);
        else
            f16_block<DP, RB, 0>(f, xf, bias, sb, sa, idp, st, ctx, nA, nB);
    };
    for (int j = 0;; ++j) {
        for_each_index([&](auto bc) { block(j, bc); }, std::make_integer_sequence<int, NB - 1>{});
        __syncthreads();
        fetch(j + 2);
        block(j, std::integral_constant<int, NB - 1>{});
        if (j + 1 == nch) break;
    }
    drain<0, RB>(sb, idh + (nch - 1) * G::CHUNK + 32 * (NB - 1), st, ctx);
}

// ------------------------------------------------------------ assignment
__device__ __forceinline__ bool val_gt(float ka, int ia, float kb, int ib)
{
    return ka > kb || (ka == kb && ia < ib);
}

// Merges the two half-lanes of a row and certifies with the window T.
__device__ __forceinline__ RowVerdict f16_finish(const ScreenF16Args &a, int64_t row, bool rvalid, int h,
                                                 const Top3f &st, TileLists &tl)
{
    Top3f x = st, y;
    y.k1 = __shfl_xor(st.k1, 32);
    y.k2 = __shfl_xor(st.k2, 32);
    y.k3 = __shfl_xor(st.k3, 32);
    y.i1 = __shfl_xor(st.i1, 32);
    y.i2 = __shfl_xor(st.i2, 32);
    if (val_gt(y.k1, y.i1, x.k1, x.i1)) {
        const Top3f t = x;
        x = y;
        y = t;
    }
    const bool second = val_gt(y.k1, y.i1, x.k2, x.i2);
    const float k2 = second ? y.k1 : x.k2;
    const int i2 = second ? y.i1 : x.i2;
    const float k3 = second ? fmaxf(x.k2, y.k2) : fmaxf(x.k3, y.k1);
    RowVerdict v{-1, 0, 0, 0, 0};
    if (rvalid && h == 0) {
        // a centroid id is used only when it names a real centroid; any other
        // state collects nothing and goes on to the next screen
        const bool ok1 = x.i1 >= 0 && x.i1 < a.ncent;
        const bool ok2 = i2 >= 0 && i2 < a.ncent;
        v.thr = __float_as_int(ok1 && st.T < kInf ? x.k1 - st.T : kInf);
        v.kind = 1;
        if (!a.force_list && ok1) {
            v.c1 = x.i1;
            v.c2 = i2;
            // (differences of fp32 values are formed in double: exact enough
            // that T's margin covers them; an infinite T settles nothing)
            if ((double)x.k1 - (double)k2 > (double)st.T) {
                v.kind = -1;
                a.labels[row] = x.i1;
            } else if ((double)x.k1 - (double)k3 > (double)st.T && ok2) {
                v.kind = 0;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t at = wave_append(&tl.cnt[k], v.kind == k);
        v.at = v.kind == k ? at : v.at;
    }
    return v;
}

template <int DP>
__global__ __launch_bounds__(512, 2) void screen_f16_kernel(ScreenF16Args a)
{
    using G = Geo<DP>;
    constexpr int RB = G::RB;
    __shared__ __attribute__((aligned(16))) char lds[G::LDS];
    __shared__ TileLists tl;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, jl = lane & 31;
    if (threadIdx.x == 0) tl.cnt[0] = tl.cnt[1] = tl.base[1] = 0;  // (a tile's barriers come before their first use)
    const uint32_t mc2 = *a.mc2_bits, rc = *a.rc_bits;
    const float sc = f16_scale(mc2);
    const int64_t ntiles = (a.nrows + G::ROWS - 1) / G::ROWS;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        f16x8 xf[RB][DP / 16];
        Top3f st[RB];
        int64_t row[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            row[rb] = tile * G::ROWS + (wave * RB + rb) * 32 + jl;
            const RowNorms n = load_row_f16<DP>(a.rows, row[rb] < a.nrows ? row[rb] : -1, a.D, h, sc, xf[rb]);
            st[rb] = Top3f{-kInf, -kInf, -kInf, -1, -1, -kInf, f16_window(n, mc2, rc, a.acc_coef)};
        }
        NoCtx none;
        f16_scan<DP>(a.plane, a.nbias, a.cpad, 0, 1, (int)(a.cpad / G::CHUNK), xf, st, none, lds);
        RowVerdict v[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) v[rb] = f16_finish(a, row[rb], row[rb] < a.nrows, h, st[rb], tl);
        list_tile<float, RB>(a, row, v, tl);
        // a list past its capacity hands every row to the fp32 screen: the
        // tiles that are left would be screened for nothing (500,000 x 96 rows
        // that f16 cannot tell apart, 16,384 centroids: 14.3 -> 13.3 ms)
        const bool full = (int64_t)tl.base[1] >= a.list_cap && !a.force_list;
        __syncthreads();
        if (full) break;
    }
}

// (tile, chunk) units of `ntiles` tiles over the grid, in tile-major order:
// calls body(tile, first chunk, end chunk) for this workgroup's share.
template <class F>
__device__ __forceinline__ void for_units(int64_t ntiles, int64_t nchunks, F &&body)
{
    const int64_t units = ntiles * nchunks;
    int64_t u = units * blockIdx.x / gridDim.x;
    const int64_t u1 = units * (blockIdx.x + 1) / gridDim.x;
    while (u < u1) {
        const int64_t tile = u / nchunks;
        const int64_t ch = u - tile * nchunks;
        const int64_t ch_end = min(nchunks, ch + (u1 - u));
        body(tile, (int)ch, (int)ch_end);
        u += ch_end - ch;
        __syncthreads();
    }
}

template <int DP>
__global__ __launch_bounds__(512, 2) void collect_f16_kernel(ScreenF16Args a)
{
    using G = Geo<DP>;
    constexpr int RB = G::RB;
    __shared__ __attribute__((aligned(16))) char lds[G::LDS];
    __shared__ int32_t queue[RB * kResolveCand * G::NT];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, jl = lane & 31;
    const int64_t n = *a.list_cnt;
    if (n > a.list_cap) return;  // the fp32 screen takes every row
    const float sc = f16_scale(*a.mc2_bits);
    for_units((n + G::ROWS - 1) / G::ROWS, a.cpad / G::CHUNK, [&](int64_t tile, int lo, int hi) {
        f16x8 xf[RB][DP / 16];
        CollectF st[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int64_t pos = tile * G::ROWS + (wave * RB + rb) * 32 + jl;
            const int64_t r = pos < n ? (int64_t)a.list[pos] : -1;
            const bool ok = r >= 0 && r < a.nrows;
            load_row_f16<DP>(a.rows, ok ? r : -1, a.D, h, sc, xf[rb]);
            st[rb] = CollectF{ok ? __int_as_float(a.rs.list_thr[pos]) : kInf, 0,
                              queue + rb * kResolveCand * G::NT + threadIdx.x, G::NT};
        }
        NoCtx none;
        f16_scan<DP>(a.plane, a.nbias, a.cpad, (int64_t)lo * G::SUB, 1, hi - lo, xf, st, none, lds);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (st[rb].qn > 0) {  // thr < inf: a listed row
                const int64_t pos = tile * G::ROWS + (wave * RB + rb) * 32 + jl;
                const uint32_t slot = atomicAdd(a.rs.cand_cnt + pos, (uint32_t)st[rb].qn);
                for (int i = 0; i < st[rb].qn && i < kResolveCand && slot + i < (uint32_t)kResolveCand; ++i)
                    a.rs.cand[pos * kResolveCand + slot + i] = st[rb].q[i * G::NT];
            }
        }
    });
}

// ------------------------------------------------------------ routing
template <int DP, int MODE>
__global__ __launch_bounds__(512, 2) void route_f16_kernel(RouteF16Args a)
{
    using G = Geo<DP>;
    constexpr int RB = G::RB;
    constexpr bool KEYS = MODE == kRouteKeys;
    __shared__ __attribute__((aligned(16))) char lds[G::LDS];
    __shared__ __attribute__((aligned(16))) float4 qv[KEYS ? 1 : G::W * kWaveQueue];
    __shared__ uint2 qm[KEYS ? 1 : G::W * kWaveQueue];
    __shared__ float tvs[KEYS ? 1 : G::ROWS];
    if (route_mode(a.w) != kModeF16) return;
    if (!KEYS && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(a.stats + kStatScreenF16, 1ull);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, h = lane >> 5, jl = lane & 31;
    const float sc = f16_scale(*a.mc2_bits);
    const int64_t nchunks = (a.nsub + G::SUB - 1) / G::SUB;
    for_units((a.nq + G::ROWS - 1) / G::ROWS, nchunks, [&](int64_t tile, int lo, int hi) {
        f16x8 xf[RB][DP / 16];
        using S = typename std::conditional<KEYS, KeysF, FilterF>::type;
        S st[RB];
        const int64_t row0 = tile * G::ROWS + wave * RB * 32;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int64_t row = row0 + rb * 32 + jl;
            const bool ok = row < a.nq;
            load_row_f16<DP>(a.queries, ok ? row : -1, a.D, h, sc, xf[rb]);
            if constexpr (KEYS) {
                st[rb].krow = ok ? a.kmin + row * (a.nsub * (kQChunk / 16)) : nullptr;
                st[rb].lo = lo * G::CHUNK;
                st[rb].hi = (int)min((int64_t)hi * G::CHUNK, a.nsub * kQChunk);
            } else {
                st[rb].tv = ok ? -a.tau[row] : kInf;
                st[rb].r = rb * 32 + jl;
                if (h == 0) tvs[wave * RB * 32 + rb * 32 + jl] = st[rb].tv;
            }
        }
        if constexpr (KEYS) {
            NoCtx none;
            f16_scan<DP>(a.plane, a.nbias, a.cpad, (int64_t)lo * G::SUB, a.cstride, hi - lo, xf, st, none, lds);
        } else {
            FilterCtx<RB> c{qv + wave * kWaveQueue, qm + wave * kWaveQueue, tvs + wave * RB * 32, 0, row0,
                            a.cand_cnt, a.cand, a.L};
            f16_scan<DP>(a.plane, a.nbias, a.cpad, (int64_t)lo * G::SUB, 1, hi - lo, xf, st, c, lds);
            filter_flush(c);
        }
    });
}

template <template <int> class L, class A>
hipError_t by_dim(int DP, const A &a, int num_cus, hipStream_t s)
{
    switch (DP) {
    case 32: return L<32>::go(a, num_cus, s);
    case 64: return L<64>::go(a, num_cus, s);
    case 96: return L<96>::go(a, num_cus, s);
    case 128: return L<128>::go(a, num_cus, s);
    case 192: return L<192>::go(a, num_cus, s);
    case 256: return L<256>::go(a, num_cus, s);
    default: return hipErrorInvalidValue;
    }
}

template <int DP>
struct LaunchTop1 {
    static hipError_t go(const ScreenF16Args &a, int num_cus, hipStream_t s)
    {
        const int64_t ntiles = (a.nrows + Geo<DP>::ROWS - 1) / Geo<DP>::ROWS;
        hipLaunchKernelGGL((screen_f16_kernel<DP>), dim3((unsigned)std::min<int64_t>(ntiles, num_cus)), dim3(512), 0, s, a);
        return hipGetLastError();
    }
};

template <int DP>
struct LaunchCollect {
    static hipError_t go(const ScreenF16Args &a, int num_cus, hipStream_t s)
    {
        hipLaunchKernelGGL((collect_f16_kernel<DP>), dim3(num_cus), dim3(512), 0, s, a);
        return hipGetLastError();
    }
};

template <int DP>
struct LaunchKeys {
    static hipError_t go(const RouteF16Args &a, int num_cus, hipStream_t s)
    {
        hipLaunchKernelGGL((route_f16_kernel<DP, kRouteKeys>), dim3(num_cus), dim3(512), 0, s, a);
        return hipGetLastError();
    }
};

template <int DP>
struct LaunchFilter {
    static hipError_t go(const RouteF16Args &a, int num_cus, hipStream_t s)
    {
        hipLaunchKernelGGL((route_f16_kernel<DP, kRouteFilter>), dim3(num_cus), dim3(512), 0, s, a);
        return hipGetLastError();
    }
};

}  // namespace

double f16_acc_coef(int DP)
{
    const double n = 2.0 * (DP + 2) * 0x1p-23;
    return n / (1.0 - n);
}

hipError_t launch_quantize_f16(const float *cent, int64_t C, int D, int DP, const uint32_t *mc2_bits, uint16_t *plane,
                               float *nbias, uint32_t *rc_bits, hipStream_t s)
{
    const int64_t cpad = quantized_pad1(C);
    const int64_t blocks = std::min<int64_t>((cpad + 7) / 8, 2048);
    hipLaunchKernelGGL(quantize_f16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, cent, C, D, DP, cpad, mc2_bits,
                       plane, nbias, rc_bits);
    return hipGetLastError();
}

hipError_t launch_screen_f16(int DP, const ScreenF16Args &a, int num_cus, hipStream_t s)
{
    if (a.nrows <= 0) return hipSuccess;
    return by_dim<LaunchTop1>(DP, a, num_cus, s);
}

hipError_t launch_collect_f16(int DP, const ScreenF16Args &a, int num_cus, hipStream_t s)
{
    if (a.nrows <= 0) return hipSuccess;
    return by_dim<LaunchCollect>(DP, a, num_cus, s);
}

hipError_t launch_route_f16(int mode, int DP, const RouteF16Args &a, int num_cus, hipStream_t s)
{
    if (a.nq <= 0 || a.nsub <= 0) return hipSuccess;
    return mode == kRouteKeys ? by_dim<LaunchKeys>(DP, a, num_cus, s) : by_dim<LaunchFilter>(DP, a, num_cus, s);
}

}  // namespace ivf
