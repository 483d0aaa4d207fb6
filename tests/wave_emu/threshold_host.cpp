// Runs the planes' routing threshold kernel of select.hip on the host
// emulation: tau of every query from given group minima and window bounds.
//   usage: threshold_host in.bin out.bin
//   in:  int64 Q, G, rank_j, rank_safe, rank_max, f16; float minima [Q][G];
//        float qbound [Q]
//   out: float tau [Q]; uint32 cand_cnt [Q]; uint32 the batch's f16-off word
#include "hip/hip_runtime.h"
namespace emu {
thread_local dim3 tid, bid;
dim3 bdim, gdim;
Block *blk;
unsigned char *dyn_lds;
}  // namespace emu
#include "select_host_src.hip"
using namespace ivf;

int main(int argc, char **argv)
{
    if (argc != 3) return 2;
    FILE *f = fopen(argv[1], "rb");
    int64_t h[6];
    if (!f || fread(h, 8, 6, f) != 6) return 2;
    const int64_t Q = h[0], G = h[1];
    if (G > kMaxGroups) return 2;
    std::vector<float> minima(Q * G), qbound(Q), tau(Q, -1.0f);
    std::vector<uint32_t> cnt(Q, 7u), w(64, 0u);
    if (fread(minima.data(), 4, Q * G, f) != (size_t)(Q * G) || fread(qbound.data(), 4, Q, f) != (size_t)Q) return 2;
    fclose(f);
    w[kWordNotI8] = h[5] ? 1u : 0u;
    RouteArgs a{};
    a.nq = Q;
    a.Cs = 16 * G;
    a.rank_j = (int)h[2];
    a.rank_safe = (int)h[3];
    a.rank_max = (int)h[4];
    a.f16 = h[5] != 0;
    a.keys = minima.data();
    a.qbound = qbound.data();
    a.tau = tau.data();
    a.cand_cnt = cnt.data();
    a.w = w.data();
    launch_route_threshold_min(a, nullptr);
    f = fopen(argv[2], "wb");
    if (!f) return 2;
    fwrite(tau.data(), 4, Q, f);
    fwrite(cnt.data(), 4, Q, f);
    fwrite(&w[kWordF16Off], 4, 1, f);
    fclose(f);
    return 0;
}
