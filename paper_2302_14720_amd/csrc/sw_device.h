// sw_device.h -- device helpers shared by the tile and brick kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swmi {

// Workgroup b runs on XCD b % 8; give each XCD a contiguous band of tiles so
// that neighbouring tiles (which share halo rows and cache lines) meet in
// the same L2 (the last n mod 8 blocks keep their own index).
__device__ __forceinline__ uint32_t tile_of_block(uint32_t b, uint32_t n) {
    const uint32_t n8 = n & ~7u;
    if (b < n8) return (b & 7u) * (n8 >> 3) + (b >> 3);
    return b;
}

// m shifted left by one, with w < T as the bit below: a compare and an add
// with carry (the compiler makes a compare, a select and a shift-or of it).
__device__ __forceinline__ uint32_t shift_in_below(uint32_t m, uint32_t w, uint32_t T) {
    asm("v_cmp_gt_u32 vcc, %2, %1\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(m) : "v"(w), "s"(T) : "vcc");
    return m;
}

// Equal-neighbour masks of 16 sites from their bit planes and those of the
// E and N neighbours; equal pairs and the population of every value 0..7
// (two 16-bit counts per word).  M: the sites of the masks.
template <uint32_t M>
__device__ __forceinline__ void potts_counts(const uint32_t pl[3], uint32_t cpk[4]) {
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
        uint32_t c[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int v = k + h;
            const uint32_t m = ~((pl[0] ^ ((v & 1) ? 0xFFFFu : 0u)) | (pl[1] ^ ((v & 2) ? 0xFFFFu : 0u)) |
                                 (pl[2] ^ ((v & 4) ? 0xFFFFu : 0u))) & M;
            c[h] = (uint32_t)__popc(m);
        }
        cpk[k >> 1] = c[0] | (c[1] << 16);
    }
}

}  // namespace swmi
