// The scale and the largest-norm bound of f16_bound.h for given squared norms.
//   usage: f16_bound_host in.bin out.bin
//   in: float n2 []   out: double (f16_scale, f16_max_norm) []
#include "hip/hip_runtime.h"
namespace emu {
thread_local dim3 tid, bid;
dim3 bdim, gdim;
Block *blk;
unsigned char *dyn_lds;
}  // namespace emu
#include "f16_bound.h"

int main(int argc, char **argv)
{
    if (argc != 3) return 2;
    FILE *f = fopen(argv[1], "rb"), *o = fopen(argv[2], "wb");
    if (!f || !o) return 2;
    uint32_t bits;
    while (fread(&bits, 4, 1, f) == 1) {
        const double v[2] = {(double)ivf::f16_scale(bits), ivf::f16_max_norm(bits)};
        fwrite(v, 8, 2, o);
    }
    fclose(f);
    fclose(o);
    return 0;
}
