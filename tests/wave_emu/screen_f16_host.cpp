// Runs the f16 kernels of screen_f16.hip and the resolving kernel of resolve.hip
// on the host emulation, with every array in an allocation of its own.
//   usage: screen_f16_host in.bin out.bin num_cus
//   in:  int64 N, C, D, list_cap, duel_cap, collect, Cs, stride, L; float rows [N][D];
//        float centroids [C][D]; float largest squared norm; float tau [N]
//   out: int32 labels [N]; uint32 listed, duels, left; int32 left rows
//        [list_cap]; float sample minima [N][Cs / 16]; uint32 candidates [N];
//        uint2 candidate lists [N][L]
#include "hip/hip_runtime.h"
namespace emu {
thread_local dim3 tid, bid;
dim3 bdim, gdim;
Block *blk;
unsigned char *dyn_lds;
}  // namespace emu
#include "screen_f16_host_src.hip"
namespace ivf {
// (screen_i8.hip is not part of this build)
int64_t quantized_pad1(int64_t C) { return (C + 255) / 256 * 256; }
}  // namespace ivf
#include "resolve_host_src.hip"
using namespace ivf;

template <typename T>
static T *alloc(size_t n, FILE *f = nullptr)
{
    const size_t b = std::max<size_t>(n, 1) * sizeof(T);
    T *p = (T *)aligned_alloc(16, (b + 15) / 16 * 16);
    memset(p, 0x7f, b);
    if (f && n && fread(p, sizeof(T), n, f) != n) exit(2);
    return p;
}
template <typename T>
static T *zero(size_t n)
{
    T *p = alloc<T>(n);
    memset(p, 0, n * sizeof(T));
    return p;
}

int main(int argc, char **argv)
{
    if (argc != 4) return 2;
    FILE *f = fopen(argv[1], "rb");
    int64_t h[9];
    if (!f || fread(h, 8, 9, f) != 9) return 2;
    const int64_t N = h[0], C = h[1], Cs = h[6], L = h[8];
    const int D = (int)h[2], num_cus = atoi(argv[3]);
    const float *rows = alloc<float>(N * D, f), *cent = alloc<float>(C * D, f);
    uint32_t *w = zero<uint32_t>(64);
    if (fread(w + kWordMc2, 4, 1, f) != 1) return 2;
    const float *tau = alloc<float>(N, f);
    fclose(f);
    int DP = 0;
    for (int dp : {32, 64, 96, 128, 192, 256})
        if (!DP && D <= dp) DP = dp;
    const int64_t cpad = quantized_pad1(C);
    uint16_t *plane = alloc<uint16_t>(cpad * DP);
    float *nbias = alloc<float>(cpad);
    launch_quantize_f16(cent, C, D, DP, w + kWordMc2, plane, nbias, w + kWordF16Rc, nullptr);

    ScreenF16Args q{};
    q.rows = rows;
    q.nrows = N;
    q.D = D;
    q.cent = cent;
    q.plane = plane;
    q.nbias = nbias;
    q.mc2_bits = w + kWordMc2;
    q.rc_bits = w + kWordF16Rc;
    q.acc_coef = f16_acc_coef(DP);
    q.cpad = cpad;
    q.ncent = C;
    q.labels = alloc<int32_t>(N);
    q.stats = zero<unsigned long long>(kNumStats);
    q.list_cap = h[3];
    q.list = alloc<int32_t>(q.list_cap);
    uint32_t *cnt = zero<uint32_t>(3);
    q.list_cnt = cnt;
    q.rs.duel_cap = h[4];
    q.rs.duel = alloc<uint2>(h[4]);
    q.rs.duel2 = alloc<int32_t>(h[4]);
    q.rs.duel_cnt = cnt + 1;
    q.rs.list_thr = h[5] ? alloc<int32_t>(q.list_cap) : nullptr;
    q.rs.cand_cnt = alloc<uint32_t>(q.list_cap);
    q.rs.cand = alloc<int32_t>(q.list_cap * kResolveCand);
    q.rs.list2 = alloc<int32_t>(q.list_cap);
    q.rs.list2_cnt = cnt + 2;
    launch_screen_f16(DP, q, num_cus, nullptr);
    if (h[5]) launch_collect_f16(DP, q, num_cus, nullptr);
    ResolveArgs r{};
    r.rows = rows;
    r.nrows = N;
    r.D = D;
    r.cent = cent;
    r.C = C;
    r.list = q.list;
    r.list_cnt = cnt;
    r.list_cap = q.list_cap;
    r.rs = q.rs;
    r.labels = q.labels;
    launch_resolve(kRowF32, r, num_cus, nullptr);

    // routing: the rows as queries
    w[kWordNotI8] = 1u;
    RouteF16Args a{};
    a.queries = rows;
    a.nq = N;
    a.D = D;
    a.plane = plane;
    a.nbias = nbias;
    a.mc2_bits = w + kWordMc2;
    a.w = w;
    a.cpad = cpad;
    a.stats = q.stats;
    a.nsub = Cs / 64;
    a.cstride = h[7];
    a.kmin = alloc<float>(N * (Cs / 16));
    launch_route_f16(kRouteKeys, DP, a, num_cus, nullptr);
    a.nsub = cpad / 64;
    a.cstride = 1;
    a.tau = tau;
    a.cand_cnt = zero<uint32_t>(N);
    a.cand = alloc<uint2>(N * L);
    a.L = (int)L;
    launch_route_f16(kRouteFilter, DP, a, num_cus, nullptr);

    f = fopen(argv[2], "wb");
    if (!f) return 2;
    fwrite(q.labels, 4, N, f);
    fwrite(cnt, 4, 3, f);
    fwrite(q.rs.list2, 4, q.list_cap, f);
    fwrite(a.kmin, 4, N * (Cs / 16), f);
    fwrite(a.cand_cnt, 4, N, f);
    fwrite(a.cand, 8, N * L, f);
    fclose(f);
    return 0;
}
