// Staging of quantised centroids from memory into LDS, shared by the int8 and
// f16 screens (gfx950).
#pragma once

#include "ivf_internal.h"

namespace ivf {

constexpr int kQChunk = kQuantChunk;  // centroids per staged chunk (sub-chunk of the one-plane screens)

// A chunk of kQChunk quantised centroids (both planes) and their biases is
// copied from the padded global arrays straight into LDS by buffer loads with
// an LDS destination (16 bytes per lane, a wave writes 1 KiB of consecutive
// LDS per instruction): no register staging and no LDS stores by the vector
// unit. LDS layout of a chunk: centroid rows of PL planes with a pitch of
// PL DP + 16 bytes (the 16 spread the rows over the banks), then the 64
// biases. Slot s (16 bytes) of the row area holds unit s % (PL DP / 16 + 1)
// of row s / (PL DP / 16 + 1); the pad unit and the bias instruction's lanes past the
// biases read beyond the buffer range and receive zeros. Loads go through
// buffer resources over the chunk's valid rows, so a ragged last chunk and
// the chunk after the last one read zeros and every load is unconditional.
// The loads of a chunk are complete (and visible to every wave) after the
// next workgroup barrier, which waits for all outstanding vector memory
// operations.
template <int DP, int NT, int PL = 2>
struct QStager {
    static constexpr int kRowB = PL * DP;                // bytes per centroid
    static constexpr int kRowU = kRowB / 16;             // 16-byte units per centroid
    static constexpr int kPitch = kRowB + 16;
    static constexpr int kRowInst = kRowU + 1;           // 64 rows x (kRowU + 1) slots / 64 lanes
    static constexpr int kInst = kRowInst + 1;           // plus one for the biases
    static constexpr int kBias = kQChunk * kPitch;       // byte offset of the biases (= kRowInst KiB)
    static constexpr int kBytes = kInst * 1024;
    static constexpr int kW = NT / 64;
    static constexpr int kIPW = (kInst + kW - 1) / kW;   // load instructions per wave
    int voff[kIPW];
    int wave;  // wave-uniform

    __device__ __forceinline__ void init()
    {
        const int lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
        for (int i = 0; i < kIPW; ++i) {
            const int inst = wave + i * kW;
            int off = 1 << 30;  // beyond any buffer range: reads zero
            if (inst < kRowInst) {
                const int slot = 64 * inst + lane;
                const int r = slot / (kRowU + 1), u = slot % (kRowU + 1);
                if (u < kRowU) off = r * kRowB + 16 * u;
            } else if (inst == kRowInst && lane < kQChunk / 4) {
                off = 16 * lane;
            }
            voff[i] = off;
        }
    }

    // Enqueues the loads of the chunk starting at centroid cbase into the LDS
    // buffer buf.
    __device__ __forceinline__ void fetch(const int8_t *__restrict__ qc, const int32_t *__restrict__ negb,
                                          int64_t cbase, int64_t cpad, char *buf) const
    {
        const int64_t left = cpad - cbase;
        const int valid = (int)(left < 0 ? 0 : left < kQChunk ? left : kQChunk);
        const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<int8_t *>(qc + cbase * kRowB), (short)0, valid * kRowB, 0x00020000);
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<int32_t *>(negb + cbase), (short)0, valid * 4, 0x00020000);
#pragma unroll
        for (int i = 0; i < kIPW; ++i) {
            const int inst = wave + i * kW;
            if (inst < kInst)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(inst < kRowInst ? rq : rb,
                                                         (__attribute__((address_space(3))) void *)(buf + inst * 1024),
                                                         16, voff[i], 0, 0, 0);
        }
    }
};

}  // namespace ivf
