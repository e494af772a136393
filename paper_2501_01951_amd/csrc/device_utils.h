// Small device-side helpers: wave/block prefix sums for 256-thread blocks of 64-wide waves.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mixgcn.h"

namespace mixgcn {

constexpr int kBlock = 256;  // threads per block used by the integer kernels
constexpr int kWave = 64;

__device__ inline uint64_t wave_inclusive_scan_u64(uint64_t v)
{
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        unsigned long long t = __shfl_up((unsigned long long)v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive prefix sum over the 256 threads of a block; *total receives the block sum.
// lds must hold 4 uint64.  Contains two __syncthreads().
__device__ inline uint64_t block_exclusive_scan_u64(uint64_t v, uint64_t* total, uint64_t* lds)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x >> 6;
    const uint64_t inc = wave_inclusive_scan_u64(v);
    if (lane == kWave - 1) lds[w] = inc;
    __syncthreads();
    uint64_t woff = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) {
        const uint64_t x = lds[i];
        if (i < w) woff += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return woff + inc - v;
}

// Stable ranks of the keys of a tile by an 8-bit digit.  Wave w of the block's four owns ITEMS * 64
// consecutive keys of the tile and walks them 64 at a time (key r of a lane is number r * 64 + lane
// of the wave).  whist[w][d] must be zero on entry and holds the wave's count of digit d on return;
// rank[r] is the number of earlier keys of the wave with the same digit.
template <int ITEMS>
__device__ inline void wave_digit_ranks(const uint32_t (&digit)[ITEMS], const bool (&valid)[ITEMS],
                                        uint32_t (*whist)[256], uint32_t (&rank)[ITEMS])
{
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x >> 6;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = digit[r];
        uint64_t m = __ballot(valid[r]);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            m &= bit ? bal : ~bal;
        }
        // m: valid lanes of this round with my digit (includes me when valid)
        const int leader = m ? (__ffsll((unsigned long long)m) - 1) : 0;
        uint32_t prior = 0;
        if (valid[r] && lane == leader) prior = atomicAdd(&whist[w][d], (uint32_t)__popcll(m));
        prior = __shfl(prior, leader, kWave);
        rank[r] = prior + (uint32_t)__popcll(m & lt_mask);
    }
}

// Value of the stored entry (row, c) of the CSR at hand under a normalisation mode.  `swapped`: the
// CSR holds the transpose of the aggregation matrix, so the entry carries the value of (c, row).
//   symmetric: dinv[row] * dinv[c] - a single fp32 multiply, so val(u,v) == val(v,u) bit for bit;
//   mean:      dinv[row of the aggregation matrix] = 1 / deg;
//   sum:       1, and 1 + eps on the diagonal.
// drow = dinv[row] (unused in sum mode).
__device__ inline float entry_value(int mode, float eps, int swapped, uint32_t row, uint32_t c,
                                    float drow, const float* __restrict__ dinv)
{
    if (mode == MIXGCN_NORM_MEAN) return swapped ? dinv[c] : drow;
    if (mode == MIXGCN_NORM_SUM) return c == row ? 1.0f + eps : 1.0f;
    return drow * dinv[c];
}

}  // namespace mixgcn
