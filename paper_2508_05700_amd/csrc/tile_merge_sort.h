// The sort of a small step (small_step, bwd_common.h) in two launches without a wait between
// workgroups: tiles of MERGE_TILE records are sorted inside LDS, a workgroup each (tile_sort_kernel), then
// every record counts the records that come before it in the other tiles of its table (tile_merge_kernel).
//
// What bounds the passes of radix_sort.h at these sizes is not work but steps that depend on each other: five
// launches (count, scan, three scatters), every scatter with an exchange between its workgroups, 7 to 8 us each
// with up to 4 us between them for 30 720 records.  Here the passes of a tile are barriers inside a workgroup.
// Tiles are small so that many CUs rank at once (a wavefront instruction of the ranking takes its SIMD four
// cycles, whatever else the chip does): three tables of 10 240 records with 18-bit keys are sorted and merged in
// 13 + 5 us with tiles of 4096 records, in 8 + 7 us with these; seven of 21 000 with 20 bits in 15 + 9, here 10 + 15.
// The passes over memory took 50.
//
// Tiles are numbered table after table, none straddles two tables; a workgroup finds its own from the tables'
// record ranges (table_start), so the launches before it need not describe them.
#pragma once
#include "bwd_common.h"
#include "radix_sort.h"
#include "scan.h"

constexpr int MERGE_ITEMS = 4;                         // records of a thread of the tile sort
constexpr int MERGE_BLOCK = 256;
constexpr int MERGE_WAVES = MERGE_BLOCK / EMB_WAVE;
constexpr int MERGE_TILE = MERGE_BLOCK * MERGE_ITEMS;
constexpr int MERGE_BITS_MIN = 7, MERGE_BITS_MAX = 10; // of a pass: tables of 2^20 rows take two passes, 2^30 three
constexpr int PLACE_BLOCK = 512;                       // records (and threads) of a workgroup of the merge
constexpr int PLACE_TILES = 4;                         // tiles a thread bisects side by side

struct MergePart {
    uint32_t index;                   // number among the table's parts
    uint32_t seg_start, seg_count;    // records of its table; the part has records index * SIZE ... of them
    uint32_t table;
};

// Part `b` of the tables' records cut into SIZE records each, table after table; false: there is none.  Every thread of
// the workgroup calls this.  table_start: [T + 1], a partition of [0, nnz) in order unless ctrl->abort is set.
template <int SIZE, int BLOCK>
__device__ __forceinline__ bool merge_part_of(const int64_t *__restrict__ table_start, int32_t T, uint32_t b, const BwdCtrl *ctrl,
                                              MergePart &part)
{
    __shared__ uint32_t wave_sums[BLOCK / EMB_WAVE];
    __shared__ MergePart found;
    __shared__ uint32_t is_there;
    const uint32_t abort = ctrl->abort;   // (asked for together with the ranges)
    if (threadIdx.x == 0) is_there = 0;
    uint32_t before = 0;
    for (int32_t t0 = 0; t0 < T; t0 += BLOCK) {
        const int32_t t = t0 + (int32_t)threadIdx.x;
        uint32_t s = 0, e = 0;
        if (t < T) {
            s = (uint32_t)table_start[t];
            e = (uint32_t)table_start[t + 1];
        }
        const uint32_t parts = (e - s + SIZE - 1) / SIZE;
        uint32_t total;
        const uint32_t inc = before + block_inclusive_scan<uint32_t, BLOCK>(parts, wave_sums, total);   // (has barriers)
        before += total;
        if (b >= inc - parts && b < inc) {   // one thread at most
            found.index = b - (inc - parts);
            found.seg_start = s;
            found.seg_count = e - s;
            found.table = (uint32_t)t;
            is_there = 1;
        }
    }
    __syncthreads();
    part = found;
    return !abort && is_there;   // uniform
}

// Sorts every tile by its key, stably: `passes` passes of BITS bits inside LDS.  LAST: there is nothing to merge (no
// table has more than one tile), the keys are written as positions in the concatenation of the tables, as the last
// pass of radix_sort.h does.
// Also clears what the launches after it count in: the words of the list of distinct rows (list_flags, [list_tiles],
// optional) and the flags of update_spans_kernel ([n_flags]).
template <int BITS, bool LAST>
__global__ __launch_bounds__(MERGE_BLOCK) void tile_sort_kernel(const uint32_t *__restrict__ keys_in,
                                                                const uint32_t *__restrict__ pay_in,
                                                                uint32_t *__restrict__ keys_out,
                                                                uint32_t *__restrict__ pay_out,
                                                                const int64_t *__restrict__ table_start, int32_t T,
                                                                int passes, const emb_table *__restrict__ tables,
                                                                uint32_t local_sentinel, uint32_t global_sentinel,
                                                                unsigned long long *__restrict__ list_flags,
                                                                uint32_t list_tiles, uint32_t *__restrict__ span_flags,
                                                                uint32_t n_flags, const BwdCtrl *ctrl)
{
    constexpr uint32_t DIGITS = 1u << BITS;
    constexpr int PER = DIGITS > (uint32_t)MERGE_BLOCK ? DIGITS / MERGE_BLOCK : 1;   // digits a thread looks after
    __shared__ uint32_t cnt[MERGE_WAVES][DIGITS];   // per-wavefront digit counts, then offsets inside the tile
    __shared__ uint32_t sk[MERGE_TILE], sp[MERGE_TILE];
    __shared__ uint32_t wave_sums[MERGE_WAVES];
    const uint32_t gid = blockIdx.x * MERGE_BLOCK + threadIdx.x;   // a grid has at least one workgroup per MERGE_TILE records
    if (list_flags && gid < list_tiles) list_flags[gid] = 0ull;
    if (gid < n_flags) span_flags[gid] = 0u;
    MergePart tile;
    if (!merge_part_of<MERGE_TILE, MERGE_BLOCK>(table_start, T, blockIdx.x, ctrl, tile)) return;
    const uint32_t start = tile.seg_start + tile.index * MERGE_TILE;
    const uint32_t left = tile.seg_count - tile.index * MERGE_TILE;
    const uint32_t count = left < (uint32_t)MERGE_TILE ? left : MERGE_TILE;
    const int lane = threadIdx.x & (EMB_WAVE - 1);
    const int wave = threadIdx.x / EMB_WAVE;
    const uint32_t wbase = wave * (MERGE_ITEMS * EMB_WAVE);
    uint32_t key[MERGE_ITEMS], pay[MERGE_ITEMS], rank[MERGE_ITEMS];
#pragma unroll
    for (int k = 0; k < MERGE_ITEMS; ++k) {
        const uint32_t i = wbase + k * EMB_WAVE + lane;
        key[k] = i < count ? keys_in[start + i] : 0u;
        pay[k] = i < count ? pay_in[start + i] : 0u;
    }
    for (int p = 0; p < passes; ++p) {
        const int shift = p * BITS;
        for (uint32_t i = lane; i < DIGITS; i += EMB_WAVE) cnt[wave][i] = 0;
        __builtin_amdgcn_wave_barrier();   // (the wavefront's own counters: no other touches them before the next barrier)
        wave_rank_digits<uint32_t, BITS, MERGE_ITEMS>(key, wbase, count, shift, BITS, cnt[wave], rank);
        __syncthreads();
        // thread d: PER consecutive digits; their starts inside the tile, and the wavefronts' within them
        {
            uint32_t c[PER][MERGE_WAVES], total = 0, all;
            const uint32_t d0 = threadIdx.x * PER;
            const bool owner = d0 < DIGITS;
#pragma unroll
            for (int j = 0; j < PER; ++j)
#pragma unroll
                for (int w = 0; w < MERGE_WAVES; ++w) {
                    c[j][w] = owner ? cnt[w][d0 + j] : 0u;
                    total += c[j][w];
                }
            uint32_t run = block_inclusive_scan<uint32_t, MERGE_BLOCK>(total, wave_sums, all) - total;
            if (owner) {
#pragma unroll
                for (int j = 0; j < PER; ++j)
#pragma unroll
                    for (int w = 0; w < MERGE_WAVES; ++w) {
                        cnt[w][d0 + j] = run;
                        run += c[j][w];
                    }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MERGE_ITEMS; ++k) {
            if (wbase + k * EMB_WAVE + lane < count) {
                const uint32_t at = cnt[wave][(key[k] >> shift) & (DIGITS - 1)] + rank[k];
                sk[at] = key[k];
                sp[at] = pay[k];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MERGE_ITEMS; ++k) {   // the records of the next pass, or of the way out
            const uint32_t i = wbase + k * EMB_WAVE + lane;
            if (i < count) {
                key[k] = sk[i];
                pay[k] = sp[i];
            }
        }
    }
    uint32_t row_base = 0;
    if (LAST) row_base = (uint32_t)tables[tile.table].row_base;
#pragma unroll
    for (int k = 0; k < MERGE_ITEMS; ++k) {
        const uint32_t i = wbase + k * EMB_WAVE + lane;
        if (i < count) {
            keys_out[start + i] = LAST ? (key[k] == local_sentinel ? global_sentinel : key[k] + row_base) : key[k];
            pay_out[start + i] = pay[k];
        }
    }
}

// Every record's place in its table: its place in its own tile and, for each other tile of the table, the number
// of that tile's records that come before it (smaller keys; equal ones of earlier tiles too, which keeps the
// order stable).  The tiles' keys go through LDS, PLACE_TILES tiles a round, and a thread bisects those for its record
// side by side: a bisection is a chain of LDS reads that wait for each other (one in 4096 keys for eight records
// a thread, one after the other, made 6 us of every 4096 records of the table).  The next round's keys are requested
// while the current ones are searched.
__global__ __launch_bounds__(PLACE_BLOCK) void tile_merge_kernel(const uint32_t *__restrict__ keys_in,
                                                                 const uint32_t *__restrict__ pay_in,
                                                                 uint32_t *__restrict__ keys_out,
                                                                 uint32_t *__restrict__ pay_out,
                                                                 const int64_t *__restrict__ table_start, int32_t T,
                                                                 const emb_table *__restrict__ tables,
                                                                 uint32_t local_sentinel, uint32_t global_sentinel,
                                                                 const BwdCtrl *ctrl)
{
    constexpr int ROUND = PLACE_TILES * MERGE_TILE;       // keys in LDS at a time
    constexpr int PER = ROUND / PLACE_BLOCK;              // of them a thread fetches
    static_assert(MERGE_TILE % PLACE_BLOCK == 0, "a part lies in one tile");
    __shared__ uint32_t other[2][PLACE_TILES][MERGE_TILE];
    MergePart part;
    if (!merge_part_of<PLACE_BLOCK, PLACE_BLOCK>(table_start, T, blockIdx.x, ctrl, part)) return;
    const uint32_t mine = part.index * PLACE_BLOCK + threadIdx.x;   // place among the table's records as they are now
    const bool live = mine < part.seg_count;
    const uint32_t my_tile = part.index * PLACE_BLOCK / MERGE_TILE;   // uniform
    const uint32_t *const seg = keys_in + part.seg_start;
    const uint32_t key = live ? seg[mine] : 0u;
    const uint32_t pay = live ? pay_in[part.seg_start + mine] : 0u;
    // the keys of a round, made up to whole tiles with a value that no key has (keys are at most local_sentinel < 2^32 - 1)
    uint32_t next[PER];
    auto ask = [&](uint32_t at) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const uint32_t i = at + e * PLACE_BLOCK + threadIdx.x;
            next[e] = i < part.seg_count ? seg[i] : 0xFFFFFFFFu;
        }
    };
    uint32_t place = mine % MERGE_TILE;
    if (part.seg_count > (uint32_t)MERGE_TILE) ask(0);   // uniform; else the table is one tile, in order already
    for (uint32_t at = 0, buf = 0; part.seg_count > (uint32_t)MERGE_TILE && at < part.seg_count; at += ROUND, buf ^= 1) {   // uniform
#pragma unroll
        for (int e = 0; e < PER; ++e) (&other[buf][0][0])[e * PLACE_BLOCK + threadIdx.x] = next[e];
        if (at + ROUND < part.seg_count) ask(at + ROUND);
        __syncthreads();   // one barrier a round: the buffer written next is the one read a round ago
        uint32_t lo[PLACE_TILES], below[PLACE_TILES];
#pragma unroll
        for (int j = 0; j < PLACE_TILES; ++j) {
            lo[j] = 0;
            below[j] = key + (at / MERGE_TILE + j < my_tile ? 1u : 0u);   // what is smaller than this comes before the record
        }
#pragma unroll
        for (uint32_t step = MERGE_TILE / 2; step >= 1; step /= 2)
#pragma unroll
            for (int j = 0; j < PLACE_TILES; ++j) lo[j] += other[buf][j][lo[j] + step - 1] < below[j] ? step : 0u;
#pragma unroll
        for (int j = 0; j < PLACE_TILES; ++j) {
            const uint32_t n = lo[j] + (other[buf][j][lo[j]] < below[j] ? 1u : 0u);
            place += at / MERGE_TILE + j == my_tile ? 0u : n;
        }
    }
    if (live) {
        const uint32_t dst = part.seg_start + place;
        keys_out[dst] = key == local_sentinel ? global_sentinel : key + (uint32_t)tables[part.table].row_base;
        pay_out[dst] = pay;
    }
}
