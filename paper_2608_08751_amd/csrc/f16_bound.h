// Scale, rounding and error bound of the f16 screening values (gfx950); the
// argument is at the top of screen_f16.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace ivf {

constexpr float kF16Max = 65504.0f;
constexpr float kF16MinNormal = 0x1p-14f;

// The power of two that brings the largest centroid norm below 2^8: f16 keeps
// 11 bits of every coordinate down to 2^-22 of that norm, and rows may be 255
// times as long.
__device__ __forceinline__ float f16_scale(uint32_t mc2_bits)
{
    if (mc2_bits == 0u) return 1.0f;
    const int e = (int)(mc2_bits >> 23) - 127;  // max ||c||^2 < 2^(e + 1)
    return ldexpf(1.0f, 8 - ((e + 2) >> 1));
}

__device__ __forceinline__ _Float16 to_f16(float t)
{
    return fabsf(t) < kF16MinNormal ? (_Float16)0.0f : (_Float16)t;
}

// What the bound needs of a row: its f16 norm and residual norm (over-estimates)
struct RowNorms {
    float xh, rx;
};

// A row's scaled values, one at a time: the f16 value of each, the sums of
// squares of these and of the residuals, and whether some value is beyond
// f16's range (it then counts as zero).
struct RowAcc {
    float r2 = 0.0f, n2 = 0.0f;
    bool over = false;
    __device__ __forceinline__ _Float16 add(float t)
    {
        const bool big = !(fabsf(t) <= kF16Max);  // also true for NaN
        over |= big;
        const _Float16 hv = big ? (_Float16)0.0f : to_f16(t);
        const float f = (float)hv;
        const float r = big ? 0.0f : t - f;  // exact
        r2 = fmaf(r, r, r2);
        n2 = fmaf(f, f, n2);
        return hv;
    }
    // over-estimates of the norms: 2^-14 covers the fp32 sums of at most 256
    // squares and the roots; a row beyond f16's range has no bound
    __device__ __forceinline__ RowNorms norms() const
    {
        RowNorms o;
        o.xh = sqrtf(n2) * (1.0f + 0x1p-14f);
        o.rx = over ? __builtin_huge_valf() : sqrtf(r2) * (1.0f + 0x1p-14f) + 0x1p-40f;
        return o;
    }
};

// M >= the largest scaled centroid norm: 2^-20 covers the rounding of the
// squared norm to fp32 and of the sums and roots, 2^-149 that of a subnormal
// one.
__device__ __forceinline__ double f16_max_norm(uint32_t mc2_bits)
{
    return sqrt((double)__uint_as_float(mc2_bits) * (1.0 + 0x1p-20) + 0x1p-149) * (double)f16_scale(mc2_bits);
}

// B for a row, in the scaled units, as a double.
__device__ __forceinline__ double f16_bound(const RowNorms &r, uint32_t mc2_bits, uint32_t rc_bits, double acc)
{
    const double M = f16_max_norm(mc2_bits);
    const double rc = (double)__uint_as_float(rc_bits);
    return (double)r.rx * M + (double)r.xh * rc + acc * (0.5 * M * M + (double)r.xh * (M + rc)) + 0x1p-60;
}

// Window of the certificate and of the keep threshold: at least 2 B plus what
// fp32 loses in (value - window).
__device__ __forceinline__ float f16_window(const RowNorms &r, uint32_t mc2_bits, uint32_t rc_bits, double acc)
{
    const double M = f16_max_norm(mc2_bits);
    return __double2float_ru(2.0 * f16_bound(r, mc2_bits, rc_bits, acc) + 0x1p-21 * (M * M + (double)r.xh * M));
}

// The f16 plane, by every thread of a grid of 256-thread workgroups: half a
// wave per plane row (zero beyond D), -||C||^2 / 2 (-inf for the padding rows
// C .. Cpad-1, below every value), and the largest residual norm over the
// table (float bits, rounded up). Memory bound: reads 4 and writes 2 bytes per
// element (262,144 x 96: 40 us, 3.8 TB/s).
__device__ __forceinline__ void quantize_f16_rows(const float *__restrict__ cent, int64_t C, int D, int DP,
                                                  int64_t Cpad, const uint32_t *__restrict__ mc2_bits,
                                                  uint16_t *__restrict__ plane, float *__restrict__ nbias,
                                                  uint32_t *__restrict__ rc_bits)
{
    const int l = threadIdx.x & 31;
    const float sc = f16_scale(*mc2_bits);
    const int64_t w0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 5;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 5;
    double rmax = 0.0;
    for (int64_t j0 = w0 & ~1ll; j0 < Cpad; j0 += nw) {  // Cpad and nw are even: both halves stay in step
        const int64_t j = j0 + (w0 & 1);
        double n2 = 0.0, r2 = 0.0;
        for (int d = 4 * l; d < DP; d += 128) {
            _Float16 q[4] = {0, 0, 0, 0};
            if (j < C && d < D) {
                const float4 v = *reinterpret_cast<const float4 *>(cent + j * D + d);
                const float va[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float t = va[e] * sc;  // exact: a power of two
                    q[e] = to_f16(t);
                    const double r = (double)t - (double)(float)q[e];
                    r2 = fma(r, r, r2);
                    n2 = fma((double)t, (double)t, n2);
                }
            }
            uint2 w;
            __builtin_memcpy(&w, q, 8);
            *reinterpret_cast<uint2 *>(plane + j * DP + d) = w;
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) {
            n2 += __shfl_xor(n2, o);
            r2 += __shfl_xor(r2, o);
        }
        rmax = fmax(rmax, r2);
        if (l == 0) nbias[j] = j < C ? -(float)(0.5 * n2) : -__builtin_huge_valf();
    }
    // the norm of the largest residual, rounded up (2^-40 covers the sum and
    // the root); one atomic per workgroup
    __shared__ uint32_t smax;
    if (threadIdx.x == 0) smax = 0;
    __syncthreads();
    if (l == 0) atomicMax(&smax, __float_as_uint(__double2float_ru(sqrt(rmax) * (1.0 + 0x1p-40))));
    __syncthreads();
    if (threadIdx.x == 0 && smax > __atomic_load_n(rc_bits, __ATOMIC_RELAXED)) atomicMax(rc_bits, smax);
}

}  // namespace ivf
