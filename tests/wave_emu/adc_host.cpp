// Runs the ADC scan of adc.hip (setup, extra parts, scan, merge, as the library
// enqueues them) on the host emulation, with every array in an allocation of its
// own.
//   usage: adc_host in.bin out.bin num_cus
//   in:  int64 B, D, C, P, N, M, k; float queries [B][D]; float centroids [C][D];
//        int32 probes [B][P]; int64 offsets [C + 1]; uint32 perm [N];
//        uint8 codes [N][M]; float codebooks [M][256][D / M]
//   out: uint32 ids [B][k]; float dist [B][k]; int32 parts of each query [B]
#include "hip/hip_runtime.h"
namespace emu {
thread_local dim3 tid, bid;
dim3 bdim, gdim;
Block *blk;
unsigned char *dyn_lds;
}  // namespace emu
#include "adc_host_src.hip"
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

int main(int argc, char **argv)
{
    if (argc != 4) return 2;
    FILE *f = fopen(argv[1], "rb");
    int64_t h[7];
    if (!f || fread(h, 8, 7, f) != 7) return 2;
    const int64_t B = h[0], D = h[1], C = h[2], P = h[3], N = h[4], M = h[5], k = h[6];
    const float *q = alloc<float>(B * D, f), *cent = alloc<float>(C * D, f);
    const int32_t *probes = alloc<int32_t>(B * P, f);
    const int64_t *off = alloc<int64_t>(C + 1, f);
    const uint32_t *perm = alloc<uint32_t>(N, f);
    const uint8_t *codes = alloc<uint8_t>(N * M, f);
    const float *cb = alloc<float>(256 * D, f);
    fclose(f);
    AdcScratch w;
    w.handoff = alloc<uint64_t>(B * 2 * P * k);
    w.hcnt = alloc<int32_t>(B * 2 * P);
    w.dl = alloc<int32_t>(B * 2 * P);
    w.dpos = alloc<longlong2>(B * 2 * P);
    w.gcnt = alloc<int32_t>(B);
    uint32_t *ids = alloc<uint32_t>(B * k);
    float *dist = alloc<float>(B * k);
    if (launch_adc_scan(q, B, (int)D, cent, C, probes, (int)P, off, perm, N, codes, (int)M, cb, (int)k, w, ids, dist,
                        atoi(argv[3]), nullptr) != hipSuccess)
        return 3;
    f = fopen(argv[2], "wb");
    if (!f) return 2;
    fwrite(ids, 4, B * k, f);
    fwrite(dist, 4, B * k, f);
    for (int64_t b = 0; b < B; ++b) {
        const int32_t s = parts_of(w.gcnt[b]);
        fwrite(&s, 4, 1, f);
    }
    fclose(f);
    return 0;
}
