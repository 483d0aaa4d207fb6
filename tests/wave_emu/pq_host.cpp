// Runs the PQ assignment of pq.hip on the host emulation, with every array in an
// allocation of its own.
//   usage: pq_host in.bin out.bin num_cus
//   in:  int64 n, D, M; float x [n][D]; float codebooks [M][256][D / M]
//   out: uint8 codes [n][M]; int32 labels [M][n]
#include "hip/hip_runtime.h"
namespace emu {
thread_local dim3 tid, bid;
dim3 bdim, gdim;
Block *blk;
unsigned char *dyn_lds;
}  // namespace emu
#include "pq_host_src.hip"
using namespace ivf;

template <typename T>
static T *alloc(size_t n, FILE *f = nullptr)
{
    const size_t b = n * sizeof(T);
    T *p = (T *)aligned_alloc(16, (b + 15) / 16 * 16);
    memset(p, 0x7f, b);
    if (f && fread(p, sizeof(T), n, f) != n) exit(2);
    return p;
}

int main(int argc, char **argv)
{
    if (argc != 4) return 2;
    FILE *f = fopen(argv[1], "rb");
    int64_t h[3];
    if (!f || fread(h, 8, 3, f) != 3) return 2;
    const int64_t n = h[0], D = h[1], M = h[2];
    const float *x = alloc<float>(n * D, f), *cb = alloc<float>(256 * D, f);
    fclose(f);
    uint8_t *codes = alloc<uint8_t>(n * M);
    int32_t *labels = alloc<int32_t>(n * M);
    if (launch_pq_assign(x, n, (int)D, (int)(D / M), (int)M, cb, codes, nullptr, atoi(argv[3]), nullptr) != hipSuccess ||
        launch_pq_assign(x, n, (int)D, (int)(D / M), (int)M, cb, nullptr, labels, atoi(argv[3]), nullptr) != hipSuccess)
        return 3;
    f = fopen(argv[2], "wb");
    if (!f) return 2;
    fwrite(codes, 1, n * M, f);
    fwrite(labels, 4, n * M, f);
    fclose(f);
    return 0;
}
