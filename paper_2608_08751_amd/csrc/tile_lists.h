// What a one-pass screen does with the rows it cannot settle by scores alone
// (gfx950): per tile, the rows with two candidates and the rows with more are
// counted in LDS and appended to the call's lists; the next screen picks the
// rows that are left.
#pragma once

#include "exact.h"
#include "ivf_internal.h"
#include "wave_ops.h"

namespace ivf {

// Counters of one tile's unsettled rows (LDS) and their places in the call's
// lists. One atomic per tile and list: with one per wave and row block, 250K
// atomics on four neighbouring words bound an assignment against few
// centroids (2M x 128 rows, 256 centroids: 1.86 ms, 0.45 with these).
struct TileLists {
    uint32_t cnt[2];   // duels, listed rows of this tile
    uint32_t base[2];  // their first slots in the lists
};

// What a row's three best scores decide.
struct RowVerdict {
    int kind;      // -1: nothing to list, 0: duel of c1 and c2, 1: listed
    int c1, c2;
    int thr;       // listed: scores >= thr can belong to the nearest centroid
    uint32_t at;   // place among the tile's rows of this kind
};

template <typename XT, class A>
__device__ __forceinline__ int duel_here(const A &a, int64_t row, int c1, int c2)
{
    const XT *x = reinterpret_cast<const XT *>(a.rows) + row * (int64_t)a.D;
    const double d1 = exact_dist(x, a.cent + (int64_t)c1 * a.D, a.D);
    const double d2 = exact_dist(x, a.cent + (int64_t)c2 * a.D, a.D);
    return dist_lt(d2, c2, d1, c1) ? c2 : c1;
}

// After every row block of the tile has its verdicts: the workgroup reserves
// the list slots of its rows and writes them.
template <typename XT, int RB, class A>
__device__ __forceinline__ void list_tile(const A &a, const int64_t (&row)[RB], const RowVerdict (&v)[RB], TileLists &tl)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t nd = tl.cnt[0], nl = tl.cnt[1];
        if (nd) {
            if (a.rs.duel_cnt) tl.base[0] = atomicAdd(a.rs.duel_cnt, nd);
            atomicAdd(a.stats + kStatRefine2, (unsigned long long)nd);
        }
        if (nl) {
            tl.base[1] = atomicAdd(const_cast<uint32_t *>(a.list_cnt), nl);
            atomicAdd(a.stats + kStatRescreen, (unsigned long long)nl);
        }
        tl.cnt[0] = 0;
        tl.cnt[1] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (v[rb].kind == 0) {
            const uint64_t slot = (uint64_t)tl.base[0] + v[rb].at;
            if (a.rs.duel_cnt && slot < (uint64_t)a.rs.duel_cap) {
                a.rs.duel[slot] = make_uint2((uint32_t)row[rb], (uint32_t)v[rb].c1);
                a.rs.duel2[slot] = v[rb].c2;
            } else {
                a.labels[row[rb]] = duel_here<XT>(a, row[rb], v[rb].c1, v[rb].c2);
            }
        } else if (v[rb].kind == 1) {
            // past the list's capacity the next screen takes every row
            const uint64_t slot = (uint64_t)tl.base[1] + v[rb].at;
            if (slot < (uint64_t)a.list_cap) {
                const_cast<int32_t *>(a.list)[slot] = (int32_t)row[rb];
                if (a.rs.list_thr) {
                    a.rs.list_thr[slot] = v[rb].thr;
                    a.rs.cand_cnt[slot] = 0;
                }
            }
        }
    }
}

// The rows a screen after a one-pass screen takes: every row when the list
// overflowed; the listed rows; or, where their candidates were collected, the
// rows with too many candidates. A tile's scan of the whole table takes as
// long for one row as for 512 (1.6 ms at 65,536 x 128 on two int8 planes), the
// split fp64 scan 0.1 ms for 30 rows and 1 ms for 500: at most
// kResolveScanRows rows go straight to that. Returns false when there is
// nothing left for the screen.
template <class A>
__device__ __forceinline__ bool pick_rows(const A &a, const int32_t *&ids, int64_t &n)
{
    const uint32_t c = *a.list_cnt;
    if (c > (uint64_t)a.list_cap) return true;
    ids = a.list;
    n = c;
    if (a.rs.list_thr) {
        ids = a.rs.list2;
        n = *a.rs.list2_cnt;
        if (n <= kResolveScanRows) {
            if (blockIdx.x == 0) {
                for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
                    const int32_t r = ids[i];
                    a.labels[r] = -1;
                    const uint32_t slot = atomicAdd(a.wl_cnt, 1u);
                    if (slot < (uint64_t)a.wl_cap) a.wl[slot] = r;
                }
                if (threadIdx.x == 0 && n) atomicAdd(a.stats + kStatFallback, (unsigned long long)n);
            }
            return false;
        }
    }
    return n > 0;
}

}  // namespace ivf
