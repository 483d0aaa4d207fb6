// Product quantisation on gfx950: the PQ encoding equation (Sec. "ANN Search
// and IVF") applied to residuals (Sec. "Residual-PQ Candidate Reduction").
// For every row and subspace m, the nearest of the K = 256 codewords of
// subspace m by (distance, index), with the distance evaluated in fp64 as
// everywhere in this library:
//     t = (double)x_d - (double)c_d; s = fma(t, t, s), d ascending.
//
// The 256 distances of a sub-vector are a contraction, so the matrix cores
// screen them: with X = s (x - mu), C = s (c - mu) (mu the subspace's mean
// codeword, s a power of two) split into two f16 parts each, the value
//     v(j) = Xh.Ch + Xh.Cl + Xl.Ch (+ Xl.Cl) - ||C_j||^2 / 2
// orders the codewords like the distance up to
//     B = ||rX|| M + ||X|| rC + g (M^2 / 2 + ||X|| M),
// rX what the two parts and the subtraction leave of X (at most 2^-21 of each
// coordinate and 2^-14, the smallest normal f16), rC the same of C (measured),
// M the largest ||C||, g the rounding of the fp32 sums (one 2^-23 per product
// and then some) and, at 16 dims, the term left out (2^-21). Each value's six low
// mantissa bits are replaced by the codeword's place (2^-17 of the value), so
// the largest carries its index, and the row is settled when it beats the
// second largest by T >= 2 B plus that. Codes are those of the fp64 definition
// either way:
//   - a few undecided rows of a tile (0.07 % of the sub-vectors of Gaussian
//     residuals) get the wave's four codewords per lane, one row after another;
//   - a tile with more is left for the dense evaluation: one row per lane,
//     several tiles at a time, every codeword read once for them. The window
//     follows the largest ||C||, so one codeword far from the others, equal
//     codewords or narrow subspaces can leave most rows undecided; where two
//     tiles in a row were left, the following ones skip the screen;
//   - a subspace whose codewords all but coincide, or whose values the fp32
//     terms of the bound cannot hold, is dense from the start.
//
// f16 parts share one v_mfma_f32_32x32x16_f16 where the subspace leaves room:
// 4 dims: [Ch Cl | Ch Cl] x [Xh Xh | Xl Xl], one instruction for 32 x 32
// values; 8 dims: [Ch | Cl] x [Xh | Xh] and x [Xl | Xl], two; 16 dims: three.
// What bounds it are the vector instructions of the selection, five per two
// values (place the indices; med3, max and max3 keep the two largest; this file
// is compiled without NaN semantics, which would add one per value), 1,280
// cycles of a SIMD per 32 sub-vectors against 512 of the matrix core; the fp64 evaluation of
// every distance took 16 fp64 instructions per value at 8 dims. 2M x 128 rows,
// 16 subspaces: 5.1 -> 1.1 ms.
//
// A persistent workgroup of eight waves per CU holds the split codebooks of as
// many subspaces as fit LDS (16 of 8 dims) in the order the fragments are
// read, and walks tiles of 64 rows per wave; the tile's rows are read once from
// memory (a 128-byte line serves the next subspaces from L1 and L2).
#include "ivf_internal.h"
#include "f16_bound.h"

#include <algorithm>
#include <type_traits>

namespace ivf {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kPqThreads = 512;
constexpr int kPqWaves = kPqThreads / 64;
constexpr int kPqTile = 64;  // rows per wave and step: two blocks of 32 share the biases read from LDS
constexpr int kPqEpoch = 32;  // tiles between two rounds of dense evaluation (a bit each)
constexpr int kPqFew = 20;    // undecided rows of a tile evaluated one by one; see pq_few

// DS: dims per subspace, padded with zeros.
template <int DS>
struct PqGeo {
    static constexpr int NF = DS == 16 ? 2 : 1;            // A fragments per tile of 32 codewords
    static constexpr int FRAG = DS == 4 ? 512 : 1024;      // bytes of one (4 dims: both lane halves read the same)
    static constexpr int BIAS = 8 * NF * FRAG;             // offset of the 256 biases
    static constexpr int BYTES = BIAS + 1024;              // LDS image of one subspace
    static constexpr float GAMMA = (DS == 4 ? 24 : DS == 8 ? 40 : 56 + 4) * 0x1p-23f;
    static constexpr int MAXM = DS == 4 ? 28 : DS == 8 ? 16 : 8;
};

struct PqSub {
    float mu[16];
    float sc, M, rc;  // scale, largest ||C||, largest residual norm (over-estimates)
    int dense;        // nothing above holds: every row is evaluated exactly
};

struct Split {
    _Float16 h, l;
};

// Two f16 parts of t. Whether the matrix unit keeps or flushes parts below the
// smallest normal number, the pair is off by at most 2^-14 more.
__device__ __forceinline__ Split split16(float t)
{
    Split s;
    s.h = (_Float16)t;
    s.l = (_Float16)(t - (float)s.h);
    return s;
}

__device__ __forceinline__ float wave_max(float v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// Dim d of a sub-vector, zero past its end (without a branch per dim)
__device__ __forceinline__ float sub_dim(const float *__restrict__ p, int d, int dsub)
{
    const float v = p[min(d, dsub - 1)];
    return d < dsub ? v : 0.0f;
}

// One wave builds the LDS image of a subspace: lane l owns codewords l, l + 64,
// l + 128, l + 192.
template <int DS>
__device__ __forceinline__ void pq_stage(const float *__restrict__ cb, int dsub, char *__restrict__ img, PqSub &sub)
{
    using G = PqGeo<DS>;
    const int lane = threadIdx.x & 63;
    float c[4][DS];
    float big = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int d = 0; d < DS; ++d) {
            c[q][d] = sub_dim(cb + (lane + 64 * q) * dsub, d, dsub);
            big = fmaxf(big, fabsf(c[q][d]));
        }
    big = wave_max(big);
    float mu[DS];
#pragma unroll
    for (int d = 0; d < DS; ++d) {
        float s = c[0][d] + c[1][d] + c[2][d] + c[3][d];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        mu[d] = s * (1.0f / 256.0f);  // any value serves: both sides subtract the same
    }
    float n2 = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float s = 0.0f;
#pragma unroll
        for (int d = 0; d < DS; ++d) {
            c[q][d] = c[q][d] - mu[d];  // rounded: 2^-24 of the difference
            s = fmaf(c[q][d], c[q][d], s);
        }
        n2 = fmaxf(n2, s);
    }
    n2 = wave_max(n2) * (1.0f + 0x1p-18f);  // >= every ||c - mu||^2
    // values from 2^60 on could overflow the sums of squares, and squares this
    // small lose more to underflow than the bound allows for
    const bool dense = big >= 0x1p60f || n2 < 0x1p-120f;
    // M below 2^10: rows up to 64 times as long, and what f16 cannot hold
    // (2^-14) is small beside the rounding of the sums
    const float sc = 4.0f * f16_scale(__float_as_uint(n2));
    float r2 = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = lane + 64 * q;
        double b = 0.0;
        float r = 0.0f;
        _Float16 h[DS], l[DS];
#pragma unroll
        for (int d = 0; d < DS; ++d) {
            const float t = c[q][d] * sc;
            const Split s = split16(t);
            h[d] = s.h;
            l[d] = s.l;
            const float rem = (t - (float)s.h) - (float)s.l;
            r = fmaf(rem, rem, r);
            b = fma((double)t, (double)t, b);
        }
        r2 = fmaxf(r2, r);
        // fragment order: tile j / 32, row j % 32; the halves of a lane pair
        // 16 bytes of 32 lanes apart
        char *row = img + (j >> 5) * G::NF * G::FRAG + (j & 31) * 16;
        if constexpr (DS == 4) {
            _Float16 f[8] = {h[0], h[1], h[2], h[3], l[0], l[1], l[2], l[3]};
            __builtin_memcpy(row, f, 16);
        } else if constexpr (DS == 8) {
            __builtin_memcpy(row, h, 16);        // half 0: Ch
            __builtin_memcpy(row + 512, l, 16);  // half 1: Cl
        } else {
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                __builtin_memcpy(row + 512 * hf, h + 8 * hf, 16);
                __builtin_memcpy(row + G::FRAG + 512 * hf, l + 8 * hf, 16);
            }
        }
        // accumulator register r of lane half hf holds codeword 8 (r / 4) + 4 hf + r % 4 of the tile
        const int i = j & 31, hf = (i >> 2) & 1, reg = 4 * (i >> 3) + (i & 3);
        reinterpret_cast<float *>(img + G::BIAS)[(j >> 5) * 32 + 16 * hf + reg] = -(float)(0.5 * b);
    }
    r2 = wave_max(r2);
    if (lane >= DS && lane < 16) sub.mu[lane] = 0.0f;
#pragma unroll
    for (int d = 0; d < DS; ++d)
        if (lane == 0) sub.mu[d] = mu[d];
    if (lane == 0) {
        sub.sc = sc;
        sub.M = sqrtf(n2) * sc * (1.0f + 0x1p-18f);
        // the two parts' remainder, plus the rounding of c - mu
        sub.rc = sqrtf(r2) * (1.0f + 0x1p-18f) + 0x1p-22f * sub.M;
        sub.dense = dense ? 1 : 0;
    }
}

// This lane's dims of a sub-vector (row < n): both halves the same dims for 4
// and 8, dims 8 h .. 8 h + 7 for 16. EXACT: dsub == DS, whose rows take 16-byte
// loads (every subspace starts at a multiple of four floats).
template <int DS, bool EXACT>
__device__ __forceinline__ void pq_load(const float *__restrict__ p, int dsub, int h, bool ok,
                                        float (&x)[DS == 4 ? 4 : 8])
{
    constexpr int ND = DS == 4 ? 4 : 8;
    const int d0 = DS == 16 ? 8 * h : 0;
    if constexpr (EXACT) {
#pragma unroll
        for (int q = 0; q < ND / 4; ++q) {
            f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
            if (ok) v = *reinterpret_cast<const f32x4 *>(p + d0 + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * q + e] = v[e];
        }
    } else {
#pragma unroll
        for (int d = 0; d < ND; ++d) x[d] = ok && d0 + d < dsub ? p[d0 + d] : 0.0f;
    }
}

constexpr double kInfD = __builtin_huge_val();

// The exact nearest codewords of the rows in `left` (bit 32 rb + s: row s of
// block rb of the tile, xm its first row's dims), one after another by the whole wave, lane l with
// codewords l, l + 64, l + 128, l + 192. About 0.75 us a row (8 dims), of
// which the reduction over the lanes is most; a tile's share of the dense
// evaluation is 20 us, so up to kPqFew rows come here (2M x 128, 16 subspaces,
// one codeword at 30 times the others' radius: 5.2 ms with at most 3 rows, 3.0
// with 8, 2.2 with 16).
template <int DS>
__device__ __forceinline__ void pq_few(const float *__restrict__ xm, int D, const float *__restrict__ cb, int dsub,
                                       uint64_t left, int (&code)[2])
{
    const int lane = threadIdx.x & 63;
    float c[4][DS];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int d = 0; d < DS; ++d) c[q][d] = sub_dim(cb + (lane + 64 * q) * dsub, d, dsub);
    while (left) {
        const int at = __builtin_ctzll(left);
        left &= left - 1;
        const float *x = xm + at * D;
        float xv[DS];
#pragma unroll
        for (int d = 0; d < DS; ++d) xv[d] = sub_dim(x, d, dsub);
        double best = kInfD;
        int bj = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            double s = 0.0;
#pragma unroll
            for (int d = 0; d < DS; ++d) {  // (the padding adds exact zeros)
                const double t = (double)xv[d] - (double)c[q][d];
                s = fma(t, t, s);
            }
            if (s < best) {  // strict, ascending j: the lower index wins a tie
                best = s;
                bj = lane + 64 * q;
            }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const double ob = __shfl_xor(best, o);
            const int oj = __shfl_xor(bj, o);
            if (ob < best || (ob == best && oj < bj)) {
                best = ob;
                bj = oj;
            }
        }
        if (lane == (at & 31)) {
            if (at < 32)
                code[0] = bj;
            else
                code[1] = bj;
        }
    }
}

// The exact nearest codewords of R tiles' rows in one subspace, a row of each
// tile per lane; the codeword is the same for every lane (scalar loads, one
// conversion each) and serves R chains. Bound by the fp64 instructions, 16 a
// codeword and row at 8 dims: 2M x 128 rows, 16 subspaces, all of them
// here, 5.2 ms (116 with every row by the whole wave).
template <int DS, bool EXACT, int R>
__device__ __forceinline__ void pq_dense(const float *__restrict__ X, int64_t n, int D, const float *__restrict__ cb,
                                         int dsub, int m, int M, const int64_t (&tile)[R], uint8_t *__restrict__ codes,
                                         int32_t *__restrict__ labels)
{
    const int lane = threadIdx.x & 63;
    double x[R][DS];
    int64_t row[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        row[r] = tile[r] * kPqTile + lane;
        const float *p = X + (row[r] < n ? row[r] : 0) * (int64_t)D + (int64_t)m * dsub;
        if constexpr (EXACT) {
#pragma unroll
            for (int q = 0; q < DS / 4; ++q) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(p + 4 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[r][4 * q + e] = (double)v[e];
            }
        } else {
#pragma unroll
            for (int d = 0; d < DS; ++d) x[r][d] = d < dsub ? (double)p[d] : 0.0;
        }
    }
    double best[R];
    int bj[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        best[r] = kInfD;
        bj[r] = 0;
    }
    // codeword j + 1 is on its way during codeword j's chains
    float c[DS];
    if constexpr (EXACT) {
#pragma unroll
        for (int d = 0; d < DS; ++d) c[d] = cb[d];
    }
#pragma unroll EXACT ? 2 : 1
    for (int j = 0; j < kPqK; ++j) {
        const float *next = cb + (EXACT ? min(j + 1, kPqK - 1) : j) * dsub;
        float cn[DS];
        if constexpr (EXACT) {
#pragma unroll
            for (int d = 0; d < DS; ++d) cn[d] = next[d];
        }
        double s[R];
#pragma unroll
        for (int r = 0; r < R; ++r) s[r] = 0.0;
#pragma unroll
        for (int d = 0; d < DS; ++d) {
            if (EXACT || d < dsub) {
                const double cd = (double)(EXACT ? c[d] : next[d]);
                double t[R];
#pragma unroll
                for (int r = 0; r < R; ++r) t[r] = x[r][d] - cd;
                if constexpr (EXACT) __builtin_amdgcn_sched_barrier(0);  // an fma right behind its difference would wait
#pragma unroll
                for (int r = 0; r < R; ++r) s[r] = fma(t[r], t[r], s[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            bj[r] = s[r] < best[r] ? j : bj[r];  // strict: the lower index wins a tie
            best[r] = fmin(s[r], best[r]);
        }
        if constexpr (EXACT) {
#pragma unroll
            for (int d = 0; d < DS; ++d) c[d] = cn[d];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (row[r] < n) {
            if (codes) codes[row[r] * M + m] = (uint8_t)bj[r];
            if (labels) labels[(int64_t)m * n + row[r]] = bj[r];
        }
    }
}

template <int DS, bool EXACT>
__global__ __launch_bounds__(kPqThreads, 2) void pq_assign_kernel(
    const float *__restrict__ X, int64_t n, int D, int dsub_arg, int M, int per, int ngroups,
    const float *__restrict__ codebooks, uint8_t *__restrict__ codes, int32_t *__restrict__ labels)
{
    using G = PqGeo<DS>;
    constexpr int ND = DS == 4 ? 4 : 8;
    const int dsub = EXACT ? DS : dsub_arg;
    __shared__ __attribute__((aligned(16))) char img[G::MAXM * G::BYTES];
    __shared__ PqSub subs[G::MAXM];
    const int lane = threadIdx.x & 63, h = lane >> 5, jl = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int group = blockIdx.x % ngroups;
    const int m0 = group * per, nm = min(M, m0 + per) - m0;
    if (nm <= 0) return;
    for (int i = wave; i < nm; i += kPqWaves)
        pq_stage<DS>(codebooks + (int64_t)(m0 + i) * kPqK * dsub, dsub, img + i * G::BYTES, subs[i]);
    __syncthreads();

    const int64_t ntiles = (n + kPqTile - 1) / kPqTile;
    const int64_t step = (int64_t)(gridDim.x / ngroups) * kPqWaves;
    for (int64_t tile0 = (int64_t)(blockIdx.x / ngroups) * kPqWaves + wave; tile0 < ntiles; tile0 += kPqEpoch * step) {
        // bit e of lane i: subspace i of tile tile0 + e * step waits for its dense evaluation
        uint32_t waiting = 0;
        int e = 0;
        for (int64_t tile = tile0; e < kPqEpoch && tile < ntiles; ++e, tile += step) {
            // (scalar bases of the tile and 32-bit offsets in it)
            const int64_t row0 = tile * kPqTile;
            const float *xt = X + row0 * D + (int64_t)m0 * dsub;
            const int in = (int)min(n - row0, (int64_t)kPqTile);
            int at[2], xo[2];
            bool ok[2];
            uint32_t packed[2] = {0u, 0u};
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                at[rb] = rb * 32 + jl;
                ok[rb] = at[rb] < in;
                xo[rb] = ok[rb] ? at[rb] * D : 0;
            }
            float x[2][ND];
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) pq_load<DS, EXACT>(xt + xo[rb], dsub, h, ok[rb], x[rb]);
            for (int i = 0; i < nm; ++i) {
                const PqSub &sub = subs[i];
                const int m = m0 + i;
                const float sc = sub.sc;
                // (e > 0: shifts below 32; the tiles before this one in the epoch)
                const uint32_t before = __builtin_amdgcn_readlane((int)waiting, i);
                const bool skip = sub.dense || (e >= 2 && (before >> (e - 2)) == 3u);
                int code[2] = {0, 0};
                bool defer = skip;
                auto next_dims = [&]() __attribute__((always_inline)) {
                    if (i + 1 < nm) {
#pragma unroll
                        for (int rb = 0; rb < 2; ++rb)
                            pq_load<DS, EXACT>(xt + (i + 1) * dsub + xo[rb], dsub, h, ok[rb], x[rb]);
                    }
                };
                if (skip) {
                    next_dims();
                } else {
                    // B fragments: the first parts, the second parts
                    f16x8 bh[2], bl[2];
                    float xn[2];
                    bool over[2];
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb) {
                        float n2 = 0.0f;
                        _Float16 ph[ND], pl[ND];
#pragma unroll
                        for (int d = 0; d < ND; ++d) {
                            // a value beyond f16's range takes its end, and the norm then shows it
                            const float t = __builtin_amdgcn_fmed3f((x[rb][d] - sub.mu[(DS == 16 ? 8 * h : 0) + d]) * sc,
                                                                    -kF16Max, kF16Max);
                            n2 = fmaf(t, t, n2);
                            const Split s = split16(t);
                            ph[d] = s.h;
                            pl[d] = s.l;
                        }
                        if constexpr (DS == 16) n2 += __shfl_xor(n2, 32);
                        over[rb] = !(n2 < 0.99f * kF16Max * kF16Max);
                        xn[rb] = n2;
                        if constexpr (DS == 4) {
#pragma unroll
                            for (int d = 0; d < 4; ++d) bh[rb][d] = bh[rb][4 + d] = h ? pl[d] : ph[d];
                        } else {
#pragma unroll
                            for (int d = 0; d < 8; ++d) {
                                bh[rb][d] = ph[d];
                                bl[rb][d] = pl[d];
                            }
                        }
                    }
                    // the next subspace's dims, in flight during this one's tiles
                    next_dims();
                    const char *fa = img + i * G::BYTES + (DS == 4 ? jl : lane) * 16;
                    const f32x4 *bi = reinterpret_cast<const f32x4 *>(img + i * G::BYTES + G::BIAS) + 4 * h;
                    // the two largest of the first and the last four tiles: a place
                    // below 64 is an inline constant, and one and-or puts it into the
                    // value
                    const float ninf = -__builtin_huge_valf();
                    float v1[2][2] = {{ninf, ninf}, {ninf, ninf}}, v2[2][2] = {{ninf, ninf}, {ninf, ninf}};
                    // tile t's fragments and biases are read while tile t - 2 is
                    // selected from, and tile t - 1's values are selected from while
                    // the matrix core works on tile t
                    f16x8 a0, a1;
                    f32x16 bias, acc[2][2];
                    auto fetch = [&](int t) __attribute__((always_inline)) {
                        a0 = *reinterpret_cast<const f16x8 *>(fa + t * G::NF * G::FRAG);
                        if constexpr (G::NF == 2) a1 = *reinterpret_cast<const f16x8 *>(fa + (t * G::NF + 1) * G::FRAG);
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const f32x4 u = bi[8 * t + g];
#pragma unroll
                            for (int e = 0; e < 4; ++e) bias[4 * g + e] = u[e];
                        }
                    };
                    auto select = [&](const f32x16 (&c)[2], int t) __attribute__((always_inline)) {
#pragma unroll
                        for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
                            for (int r = 0; r < 16; r += 2) {
                                const float a = __uint_as_float((__float_as_uint(c[rb][r]) & ~63u) | (uint32_t)(16 * (t & 3) + r));
                                const float b = __uint_as_float((__float_as_uint(c[rb][r + 1]) & ~63u) | (uint32_t)(16 * (t & 3) + r + 1));
                                float &w1 = v1[rb][t >> 2], &w2 = v2[rb][t >> 2];
                                w2 = fmaxf(w2, __builtin_amdgcn_fmed3f(w1, a, b));  // the second largest of w1, a, b
                                w1 = fmaxf(fmaxf(w1, a), b);
                            }
                        }
                    };
                    fetch(0);
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        f32x16(&c)[2] = acc[t & 1];
#pragma unroll
                        for (int rb = 0; rb < 2; ++rb) c[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, bh[rb], bias, 0, 0, 0);
                        if constexpr (DS >= 8) {
#pragma unroll
                            for (int rb = 0; rb < 2; ++rb) c[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, bl[rb], c[rb], 0, 0, 0);
                        }
                        if constexpr (DS == 16) {
#pragma unroll
                            for (int rb = 0; rb < 2; ++rb) c[rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, bh[rb], c[rb], 0, 0, 0);
                        }
                        if (t + 1 < 8) fetch(t + 1);
                        __builtin_amdgcn_sched_barrier(0);
                        if (t > 0) select(acc[(t - 1) & 1], t - 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    select(acc[1], 7);
                    bool todo[2];
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb) {
                        // the halves of the tiles, then of the lanes (equal values leave a gap of zero)
                        const bool late = v1[rb][1] > v1[rb][0];
                        const float b1 = late ? v1[rb][1] : v1[rb][0];
                        const float b2 = fmaxf(late ? v1[rb][0] : v1[rb][1], fmaxf(v2[rb][0], v2[rb][1]));
                        int place = (int)(__float_as_uint(b1) & 63u);
                        place = ((place >> 4) + (late ? 4 : 0)) * 32 + 8 * ((place & 15) >> 2) + (place & 3) + 4 * h;
                        const float o1 = __shfl_xor(b1, 32), o2 = __shfl_xor(b2, 32);
                        const int op = __shfl_xor(place, 32);
                        const float best = fmaxf(b1, o1);
                        const float second = fmaxf(fminf(b1, o1), fmaxf(b2, o2));
                        code[rb] = b1 >= o1 ? place : op;
                        // T (see the top): 2^-11 covers the fp32 arithmetic of the terms themselves
                        const float xl = sqrtf(xn[rb]) * (1.0f + 0x1p-18f);
                        const float B = (0x1p-21f * xl + 0x1p-12f) * sub.M + xl * sub.rc +
                                        G::GAMMA * (0.5f * sub.M * sub.M + xl * sub.M);
                        const float T = (2.0f * B + 0x1p-17f * (fabsf(best) + fabsf(second))) * (1.0f + 0x1p-11f);
                        todo[rb] = ok[rb] && h == 0 && (over[rb] || !(best - second > T));
                    }
                    const uint64_t left = __ballot(todo[0]) | (__ballot(todo[1]) << 32);
                    defer = __popcll(left) > kPqFew;
                    if (left != 0 && !defer)
                        pq_few<DS>(xt + i * dsub, D, codebooks + (int64_t)m * kPqK * dsub, dsub, left, code);
                }
                if (defer && lane == i) waiting |= 1u << e;
                const bool words = (M & 3) == 0 && (per & 3) == 0;
#pragma unroll
                for (int rb = 0; rb < 2; ++rb) {
                    if (ok[rb] && h == 0) {
                        if (labels && !defer) (labels + (int64_t)m * n + row0)[at[rb]] = code[rb];
                        if (codes && words) {
                            // four subspaces' codes in one store where the row's codes are words
                            // (a byte that waits is written later)
                            packed[rb] = (packed[rb] >> 8) | ((uint32_t)code[rb] << 24);
                            if ((i & 3) == 3)
                                *reinterpret_cast<uint32_t *>(codes + row0 * M + (m - 3) + at[rb] * M) = packed[rb];
                        } else if (codes && !defer) {
                            (codes + row0 * M + m)[at[rb] * M] = (uint8_t)code[rb];
                        }
                    }
                }
            }
        }
        if (__any(waiting != 0)) {
            // the words above are written before their bytes
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_s_waitcnt(0);
            for (int i = 0; i < nm; ++i) {
                uint32_t left = __builtin_amdgcn_readlane((int)waiting, i);
                const float *cb = codebooks + (int64_t)(m0 + i) * kPqK * dsub;
                auto some = [&](auto rc) __attribute__((always_inline)) {
                    constexpr int R = decltype(rc)::value;
                    int64_t t[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        t[r] = left ? tile0 + __builtin_ctz(left) * step : t[0];  // (or its rows once more)
                        left &= left - 1;
                    }
                    pq_dense<DS, EXACT, R>(X, n, D, cb, dsub, m0 + i, M, t, codes, labels);
                };
                constexpr int R = DS == 16 ? 4 : 8;  // 128 registers of dims
                while (left) {
                    const int w = __popc(left);
                    if (w > R / 2)
                        some(std::integral_constant<int, R>{});
                    else if (w > 1)
                        some(std::integral_constant<int, R / 2>{});
                    else
                        some(std::integral_constant<int, 1>{});
                }
            }
        }
    }
}

template <int DS, bool EXACT>
hipError_t launch_ds(const float *X, int64_t n, int D, int dsub, int M, const float *codebooks, uint8_t *codes,
                     int32_t *labels, int num_cus, hipStream_t s)
{
    // groups of subspaces of about equal size (whole words of codes where they can be)
    const int ngroups = (M + PqGeo<DS>::MAXM - 1) / PqGeo<DS>::MAXM;
    int per = (M + ngroups - 1) / ngroups;
    if ((M & 3) == 0) per = (per + 3) & ~3;
    const int64_t ntiles = (n + kPqTile - 1) / kPqTile;
    const int64_t wgs = std::min<int64_t>((ntiles + kPqWaves - 1) / kPqWaves, std::max(1, num_cus / ngroups));
    hipLaunchKernelGGL((pq_assign_kernel<DS, EXACT>), dim3((unsigned)(wgs * ngroups)), dim3(kPqThreads), 0, s, X, n, D,
                       dsub, M, per, ngroups, codebooks, codes, labels);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_pq_assign(const float *X, int64_t n, int D, int dsub, int M, const float *codebooks, uint8_t *codes,
                            int32_t *labels, int num_cus, hipStream_t s)
{
    if (n <= 0 || M <= 0) return hipSuccess;
    if (dsub == 4) return launch_ds<4, true>(X, n, D, dsub, M, codebooks, codes, labels, num_cus, s);
    if (dsub == 8) return launch_ds<8, true>(X, n, D, dsub, M, codebooks, codes, labels, num_cus, s);
    if (dsub == 16) return launch_ds<16, true>(X, n, D, dsub, M, codebooks, codes, labels, num_cus, s);
    if (dsub < 4) return launch_ds<4, false>(X, n, D, dsub, M, codebooks, codes, labels, num_cus, s);
    if (dsub < 8) return launch_ds<8, false>(X, n, D, dsub, M, codebooks, codes, labels, num_cus, s);
    return launch_ds<16, false>(X, n, D, dsub, M, codebooks, codes, labels, num_cus, s);
}

}  // namespace ivf
