// Near ties of the one-pass assignment screens (gfx950): rows with two
// candidates (duels) and listed rows with their collected candidates take the
// nearest by exact fp64 distance and (distance, id), as the definition states.
// Evaluating the two candidates inside the screening kernel cost 1.6 of its
// 2.0 ms on 2M rows x 256 centroids (few lanes of a wave at work, two waves
// per SIMD to hide the scattered loads): here every lane has a distance and
// the chip is full.
#include "ivf_internal.h"
#include "exact.h"
#include "wave_ops.h"

#include <algorithm>

namespace ivf {
namespace {

constexpr double kInfD = __builtin_huge_val();

template <typename XT>
__device__ __forceinline__ double cand_dist(const ResolveArgs &a, int64_t row, int c)
{
    if (c < 0 || c >= a.C || row < 0 || row >= a.nrows) return kInfD;
    return exact_dist(reinterpret_cast<const XT *>(a.rows) + row * (int64_t)a.D, a.cent + (int64_t)c * a.D, a.D);
}

// Two lanes per duel and eight (kResolveCand) per listed row: latency of the
// scattered row reads bounds it, so one distance per lane and as many waves
// as the registers of a 32-dim load block allow.
template <typename XT>
__global__ __launch_bounds__(256) void resolve_kernel(ResolveArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t nt = (int64_t)gridDim.x * 256;
    const int64_t nl = *a.list_cnt;
    if (nl > a.list_cap) return;  // another screen takes every row
    const int64_t nd = min((int64_t)*a.rs.duel_cnt, a.rs.duel_cap);
    // whole waves stay in step (nt and the wave's first item are multiples of
    // 64 lanes), so the shuffles always find their partners
    for (int64_t w = t0 - lane; w < 2 * nd; w += nt) {
        const int64_t t = w + lane;
        const bool on = t < 2 * nd;
        const uint2 rc = on ? a.rs.duel[t >> 1] : make_uint2(0u, 0u);
        const int c = !on ? -1 : (t & 1) ? a.rs.duel2[t >> 1] : (int)rc.y;
        const double d = cand_dist<XT>(a, (int64_t)rc.x, c);
        const double od = __shfl_xor(d, 1);
        const int oc = __shfl_xor(c, 1);
        if (on && !(t & 1)) a.labels[rc.x] = dist_lt(od, oc, d, c) ? oc : c;
    }
    if (!a.rs.list_thr) return;  // another screen takes the listed rows
    for (int64_t w = t0 - lane; w < kResolveCand * nl; w += nt) {
        const int64_t t = w + lane;
        const int64_t i = t / kResolveCand;
        const int j = (int)(t % kResolveCand);
        const bool on = i < nl;
        const int64_t row = on ? (int64_t)a.list[i] : -1;
        const uint32_t n = on ? a.rs.cand_cnt[i] : 0u;
        const bool fits = n >= 1u && n <= (uint32_t)kResolveCand;
        int c = -1;
        if (fits && j < (int)n) {
            c = a.rs.cand[i * kResolveCand + j];
            if (c >= 0 && c < a.C && a.ord) c = (int)a.ord[c];
        }
        double d = cand_dist<XT>(a, row, c);
#pragma unroll
        for (int o = 1; o < kResolveCand; o <<= 1) {
            const double od = __shfl_xor(d, o);
            const int oc = __shfl_xor(c, o);
            if (oc >= 0 && oc < a.C && (c < 0 || c >= a.C || dist_lt(od, oc, d, c))) {
                d = od;
                c = oc;
            }
        }
        const bool good = fits && c >= 0 && c < a.C;
        if (on && j == 0 && good) a.labels[row] = c;
        const bool rest = on && j == 0 && !good;
        const uint32_t slot = wave_append(a.rs.list2_cnt, rest);
        if (rest) a.rs.list2[slot] = (int32_t)row;  // at most list_cap rows in all
    }
}

}  // namespace

hipError_t launch_resolve(int rowtype, const ResolveArgs &a, int num_cus, hipStream_t s)
{
    if (a.nrows <= 0) return hipSuccess;
    const int64_t most = (std::min<int64_t>(a.nrows, a.rs.duel_cap) * 2 + std::min<int64_t>(a.nrows, a.list_cap) *
                          kResolveCand + 255) / 256;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(most, 8 * (int64_t)num_cus));
    if (rowtype == kRowU8)
        hipLaunchKernelGGL(resolve_kernel<uint8_t>, dim3(grid), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(resolve_kernel<float>, dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace ivf
