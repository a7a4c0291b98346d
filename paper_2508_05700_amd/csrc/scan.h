// Wavefront and workgroup prefix sums used by the offsets builder and by the
// sort / run-length stages of the backward.
#pragma once
#include "emb_internal.h"

// One step of a scan by data-parallel moves of the vector unit (the lane shuffles of __shfl go through LDS: some 100
// cycles each, one behind the other).  A lane that the move gives nothing gets 0.  What bounds these scans is latency: the
// workgroups of the small steps and the set-up launches do little else between their loads (a training step of 30 720
// lookups 34.0 us with shuffles, 32.8 so; of 148 700 67.9 and 66.3).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t scan_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS, typename V>
__device__ __forceinline__ V scan_step(V v)
{
    static_assert(sizeof(V) == 4 || sizeof(V) == 8, "scans of 32- and 64-bit integers");
    if constexpr (sizeof(V) == 4) {
        return v + (V)scan_move<CTRL, ROWS>((uint32_t)v);
    } else {
        const uint32_t lo = scan_move<CTRL, ROWS>((uint32_t)(uint64_t)v), hi = scan_move<CTRL, ROWS>((uint32_t)((uint64_t)v >> 32));
        return v + (V)(((uint64_t)hi << 32) | lo);
    }
}

// Every lane of the wavefront must be there.
template <typename V>
__device__ __forceinline__ V wave_inclusive_scan(V v)
{
    v = scan_step<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8: within the rows of 16 lanes
    v = scan_step<0x112, 0xF>(v);
    v = scan_step<0x114, 0xF>(v);
    v = scan_step<0x118, 0xF>(v);
    v = scan_step<0x142, 0xA>(v);   // row_bcast:15: the ends of rows 0 and 2 to rows 1 and 3
    return scan_step<0x143, 0xC>(v);   // row_bcast:31: the end of row 1 to rows 2 and 3
}

// Inclusive scan of one value per thread over a workgroup of BLOCK threads
// (a multiple of 64, at most 1024).  `wave_sums` is LDS scratch of BLOCK/64
// entries.  Returns the inclusive value; `total` receives the workgroup sum.
// Ends with a barrier, so the scratch can be reused at once.
template <typename V, int BLOCK>
__device__ __forceinline__ V block_inclusive_scan(V v, V *wave_sums, V &total)
{
    constexpr int WAVES = BLOCK / EMB_WAVE;
    static_assert(BLOCK % EMB_WAVE == 0 && WAVES <= EMB_WAVE, "unsupported workgroup size");
    const int lane = threadIdx.x & (EMB_WAVE - 1);
    const int wave = threadIdx.x / EMB_WAVE;
    V inc = wave_inclusive_scan(v);
    if (lane == EMB_WAVE - 1) wave_sums[wave] = inc;
    __syncthreads();
    // every wavefront adds up the sums before its own itself: one barrier less than one of them doing it for all
    V before = V(0), all = V(0);
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const V x = wave_sums[w];
        if (w < wave) before += x;
        all += x;
    }
    total = all;
    __syncthreads();
    return inc + before;
}
