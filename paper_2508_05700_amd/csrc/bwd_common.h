// Constants and the device control block shared by the stages of the backward.
#pragma once
#include "emb_internal.h"

struct BwdCtrl {
    uint32_t abort;        // offsets are not a partition of [0, nnz): do nothing
    uint32_t reserved[2];
    uint32_t num_unique;   // U
    unsigned long long task_and_multi_count;  // low half: chunk tasks; high half: queued runs of several chunks
    uint32_t pad[58];
};
static_assert(sizeof(BwdCtrl) == 256, "control block is one 256-byte line");

// Whether the backward is aborted, for kernels whose own launch may abort it: one thread reads the word, and every thread of
// the workgroup gets its answer.  Wavefronts that each read it for themselves could part before a barrier.  Other kernels
// find the word settled.
__device__ __forceinline__ bool workgroup_aborted(const BwdCtrl *ctrl)
{
    __shared__ uint32_t word;
    if (threadIdx.x == 0) word = __hip_atomic_load(&ctrl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return word != 0;
}

constexpr int RADIX_BITS = 8;
constexpr int RADIX = 1 << RADIX_BITS;
constexpr int SORT_BLOCK = 512;
constexpr int SORT_WAVES = SORT_BLOCK / EMB_WAVE;
constexpr int SORT_ITEMS = 8;
constexpr int SORT_TILE = SORT_BLOCK * SORT_ITEMS;  // 4096 records per workgroup
constexpr int SORT_PAD = 320;                       // records of slack after the key / payload arrays

constexpr int UPD_BLOCK = 128;       // two wavefronts: measured better than four for the update kernels
constexpr int UPD_SPAN = 256;        // sorted records per wavefront in the update
constexpr int UPD_LOOK = 32;         // records of look-ahead after a span
constexpr int UPD_SHORT_MAX = 32;    // longest run the short-run kernel sums itself
constexpr int UPD_QSLOTS = UPD_SPAN / (UPD_SHORT_MAX + 1) + 1;  // runs longer than that which can start in one span
constexpr int LONG_CHUNK = 256;     // records of a queued run summed by one wavefront
constexpr int PREP_BLOCK = 1024;     // workgroup of the kernel that turns queued runs into tasks
constexpr int UPD_LDS_TABLES = 512; // table directories up to this size are staged in LDS

// Small steps (32-bit keys, at most UPD_LDS_TABLES tables) are sorted by tile_merge_sort.h (small_step) and updated by
// update_spans.h, on the caller's stream alone (spans_step); larger ones by radix_sort.h and update.h.  What ends the first
// is the merge, whose work is the number of records times the records of a table, of which the host knows the average:
// SMALL_STEP_MERGE_MAX is where even tables lose.  But a batch may have all its records in one of its tables:
// SMALL_STEP_MAX is where such a batch takes as long as it does without either route.  Whole steps of 256-byte rows with
// popular heads in us, merged / sorted by radix_sort.h / that in its earlier form (wave_rank_digits) and update.h, in turn on
// one card:
//   even tables: one 92 000 records 68 / 71 / 105, 110 000 75 / 73 / 106, 150 000 111 / 81 / 113; two 130 000 68 / 76 / 106,
//   150 000 83 / 79 / 112; four 160 000 73 / 83 / 114, 262 000 94 / 94 / 121; seven 150 000 65 / 81 / 114; sixteen 160 000
//   65 / 87 / 122, 262 000 81 / 100 / 127;
//   all records in one of two 150 000 115 / 82 / 115, of seven 131 / 98 / 131, of twenty-four 140 / 107 / 141, of sixteen
//   185 000 160 / 113 / 147, 262 000 211 / 134 / 162; four fifths in one of sixteen 160 000 113 / 103 / 140, 262 000
//   186 / 127 / 160.
constexpr int64_t SMALL_STEP_MAX = 150'000;
constexpr int64_t SMALL_STEP_MERGE_MAX = (int64_t)9 << 30;   // records times average records of a table
static inline bool small_step(int32_t T, int64_t nnz, int key_bytes)
{
    return key_bytes == 4 && nnz > 0 && nnz <= SMALL_STEP_MAX && T <= UPD_LDS_TABLES && nnz * nnz / T <= SMALL_STEP_MERGE_MAX;
}

// What ends the second is the start and the staging of a wavefront per 32 records, which the fork to a second stream and
// the join cost less than in the end, and sooner for bf16 rows, whose accumulators leave two wavefronts on a SIMD where
// update.h has four.  Updates alone of the same sorted records in us, update_spans.h / update.h:
//   fp32, one table of 128-byte rows that hardly repeat, 1 040 000 records 70 / 54; of 256 bytes 850 000 57 / 56,
//   1 040 000 73 / 61; three tables with popular heads 850 000 70 / 75, 1 040 000 82 / 85; sixteen 850 000 88 / 92;
//   bf16, one table of 128-byte rows that hardly repeat 500 000 45 / 55, 700 000 68 / 56; three of 256 bytes with popular
//   heads 500 000 70 / 71, 700 000 91 / 86; sixteen 500 000 81 / 82, 700 000 106 / 101, of 384 bytes 850 000 181 / 156.
// Wider rows gain up to the same lines (fp32 of 4 KB 300 000 336 / 415, of 16 KB 1245 / 1348; bf16 of 8 KB 1014 / 1115), except
// bf16 rows beyond 8 KB: the sums of a chunk of 16 KB do not fit the registers (410 spilled a lane), and a row with many
// lookups is many such chunks.  Rows of 16 KB with popular heads, 10 000 records 695 / 1026, 12 000 815 / 1021, 16 000
// 1078 / 1005, 60 000 1738 / 989; of 9 KB 16 000 979 / 836.
constexpr int64_t SPANS_STEP_MAX = 3 << 18, SPANS_STEP_MAX_BF16 = 1 << 19, SPANS_STEP_MAX_BF16_WIDEST = 3 << 12;
constexpr int32_t SPANS_BF16_WIDEST = 4096;   // values of a row; wider ones have 16 chunks a lane
static inline bool spans_step(int32_t T, int64_t nnz, int key_bytes, int32_t D, bool bf16)
{
    const int64_t most = !bf16 ? SPANS_STEP_MAX : D <= SPANS_BF16_WIDEST ? SPANS_STEP_MAX_BF16 : SPANS_STEP_MAX_BF16_WIDEST;
    return key_bytes == 4 && nnz > 0 && nnz <= most && T <= UPD_LDS_TABLES;
}

struct LongSeg {
    uint32_t lo, hi;       // records [lo, hi) of the sorted arrays
    uint32_t chunk_base;   // first chunk-sum slot (runs of several chunks)
    uint32_t n_chunks;
};
