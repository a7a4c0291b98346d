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

// Small steps (32-bit keys, at most UPD_LDS_TABLES tables) are sorted by tile_merge_sort.h and updated by update_spans.h,
// on the caller's stream alone; larger ones by radix_sort.h and update.h.  What ends the first is the merge, whose work
// is the number of records times the records of a table, of which the host knows the average.  Whole steps of 256-byte
// rows in us, with both / neither, in turn on one card: one table 60 000 records 54 / 100, 120 000 83 / 108, 240 000
// 160 / 119; four tables 120 000 57 / 107, 240 000 87 / 118, 480 000 177 / 139; sixteen 128 000 53 / 105, 256 000 74 / 118,
// 512 000 126 / 145, 1 024 000 255 / 200.  Up to SMALL_STEP_MAX a batch that has all its records in one of its tables
// loses 40 % at most; sixteen even tables would still gain at twice as many.
constexpr int64_t SMALL_STEP_MAX = 1 << 18;
constexpr int64_t SMALL_STEP_MERGE_MAX = (int64_t)1 << 35;   // records times average records of a table
static inline bool small_step(int32_t T, int64_t nnz, int key_bytes)
{
    return key_bytes == 4 && nnz > 0 && nnz <= SMALL_STEP_MAX && T <= UPD_LDS_TABLES && nnz * nnz / T <= SMALL_STEP_MERGE_MAX;
}
// What ends the second is the start and the staging of a wavefront per 32 records, which the fork to a second stream and
// the join cost less than in the end.  Sorted the same way, in us, update_spans.h / update.h: one table 343 000 records of
// 224 bytes 117 / 140, 480 000 of 64 80 / 106, of 256 127 / 147, 960 000 179 / 200; four 480 000 122 / 139, 960 000
// 185 / 189; sixteen 512 000 130 / 145, 1 024 000 197 / 200, 2 049 000 339 / 315, 2 623 000 439 / 410.
constexpr int64_t SPANS_STEP_MAX = 1 << 20;
static inline bool spans_step(int32_t T, int64_t nnz, int key_bytes)
{
    return key_bytes == 4 && nnz > 0 && nnz <= SPANS_STEP_MAX && T <= UPD_LDS_TABLES;
}

struct LongSeg {
    uint32_t lo, hi;       // records [lo, hi) of the sorted arrays
    uint32_t chunk_base;   // first chunk-sum slot (runs of several chunks)
    uint32_t n_chunks;
};
