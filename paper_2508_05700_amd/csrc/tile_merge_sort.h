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
#include "gather.h"
#include "radix_sort.h"
#include "scan.h"
#include "u64mod.h"

constexpr int MERGE_ITEMS = 4;                         // records of a thread of the tile sort
constexpr int MERGE_BLOCK = 256;
constexpr int MERGE_WAVES = MERGE_BLOCK / EMB_WAVE;
constexpr int MERGE_TILE = MERGE_BLOCK * MERGE_ITEMS;
constexpr int MERGE_BITS_MAX = 10;                     // of a pass: tables of 2^20 rows take two passes, 2^30 three
constexpr int PLACE_BLOCK = 512;                       // records (and threads) of a workgroup of the merge
constexpr int PLACE_TILES = 4;                         // tiles a thread bisects side by side

struct MergePart {
    uint32_t index;                   // number among the table's parts
    uint32_t seg_start, seg_count;    // records of its table; the part has records index * SIZE ... of them
    uint32_t table;
};

// Part `b` of the tables' records cut into SIZE records each, table after table; false: there is none.  Every thread of
// the workgroup calls this and gets the same answer.  range(t, s, e): table t has records [s, e), a partition of [0, nnz)
// in order, unless `ctrl` (nullable) says that the backward is aborted: then there is no part.  That is read once for the
// workgroup: the lookup that a tile is sorted beside may abort meanwhile, and wavefronts that each read it for themselves
// could part before a barrier.
template <int SIZE, int BLOCK, typename Range>
__device__ __forceinline__ bool merge_part_in(int32_t T, uint32_t b, const Range &range, MergePart &part, const BwdCtrl *ctrl = nullptr)
{
    __shared__ uint32_t wave_sums[BLOCK / EMB_WAVE];
    __shared__ MergePart found;
    __shared__ uint32_t is_there, aborted;
    if (threadIdx.x == 0) {
        is_there = 0;
        aborted = ctrl ? __hip_atomic_load(&ctrl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    }
    uint32_t before = 0;
    for (int32_t t0 = 0; t0 < T; t0 += BLOCK) {
        const int32_t t = t0 + (int32_t)threadIdx.x;
        uint32_t s = 0, e = 0;
        if (t < T) range(t, s, e);
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
    return is_there && !aborted;   // uniform
}

// The same from table_start ([T + 1], a partition unless ctrl->abort is set); there is no part of an aborted backward.
template <int SIZE, int BLOCK>
__device__ __forceinline__ bool merge_part_of(const int64_t *__restrict__ table_start, int32_t T, uint32_t b, const BwdCtrl *ctrl,
                                              MergePart &part)
{
    return merge_part_in<SIZE, BLOCK>(T, b, [&](int32_t t, uint32_t &s, uint32_t &e) {
        s = (uint32_t)table_start[t];
        e = (uint32_t)table_start[t + 1];
    }, part, ctrl);
}

constexpr uint32_t MERGE_DIGITS = 1u << MERGE_BITS_MAX;
struct alignas(sizeof(uint4)) TileSortLds {
    uint32_t cnt[MERGE_WAVES][MERGE_DIGITS];   // per-wavefront digit counts, then offsets inside the tile
    uint32_t sk[MERGE_TILE], sp[MERGE_TILE];
    uint32_t wave_sums[MERGE_WAVES];
};
// the counts are cleared, and offsets that stand in their place written, 16 bytes at a time
static_assert(alignof(TileSortLds) % alignof(uint4) == 0 && offsetof(TileSortLds, cnt) % alignof(uint4) == 0 &&
                  sizeof(TileSortLds::cnt[0]) % sizeof(uint4) == 0, "16-byte accesses of LDS");

// How the tiles of a small step are sorted and where they go.
struct TileSortArgs {
    uint32_t *keys_out, *pay_out;
    int passes, bits;                 // passes of `bits` (at most MERGE_BITS_MAX) bits each
    bool last;                        // there is nothing to merge: no table has more than one tile
    uint32_t local_sentinel, global_sentinel;
    uint32_t *span_flags;             // [n_flags] flags of update_spans_kernel, cleared here: a tile has more threads than flags
    uint32_t n_flags;
};

// Sorts a tile by its key, stably: `passes` passes of `bits` bits inside LDS.  load(i, count, key, pay): the records
// i of the tile, those below count.  With nothing to merge the keys are written as positions in the concatenation of the tables, as the last pass of
// radix_sort.h does.  BITS: a.bits where that is known to the compiler, else 0.
template <int BITS, typename Load>
__device__ __forceinline__ void tile_sort(const TileSortArgs &a, const MergePart &tile, uint32_t row_base, TileSortLds &lds,
                                          const Load &load)
{
    constexpr uint32_t DIGITS = BITS ? 1u << BITS : MERGE_DIGITS;   // (with fewer bits than that the others count nothing)
    constexpr int PER = DIGITS > (uint32_t)MERGE_BLOCK ? DIGITS / MERGE_BLOCK : 1;   // digits a thread looks after
    const int bits = BITS ? BITS : a.bits;
    const uint32_t start = tile.seg_start + tile.index * MERGE_TILE;
    const uint32_t left = tile.seg_count - tile.index * MERGE_TILE;
    const uint32_t count = left < (uint32_t)MERGE_TILE ? left : MERGE_TILE;
    const int lane = threadIdx.x & (EMB_WAVE - 1);
    const int wave = threadIdx.x / EMB_WAVE;
    const uint32_t wbase = wave * (MERGE_ITEMS * EMB_WAVE);
    const uint32_t digit_mask = (1u << bits) - 1;
    uint32_t at[MERGE_ITEMS], key[MERGE_ITEMS], pay[MERGE_ITEMS], rank[MERGE_ITEMS];
#pragma unroll
    for (int k = 0; k < MERGE_ITEMS; ++k) {
        at[k] = wbase + k * EMB_WAVE + lane;
        key[k] = pay[k] = 0u;
    }
    load(at, count, key, pay);
    __syncthreads();   // (it may have read what is counted in from here on)
    for (int p = 0; p < a.passes; ++p) {
        const int shift = p * bits;
        // (the wavefront's own counters: no other touches them before the next barrier)
        for (uint32_t i = lane; i < DIGITS / 4; i += EMB_WAVE)
            reinterpret_cast<uint4 *>(lds.cnt[wave])[i] = make_uint4(0u, 0u, 0u, 0u);
        __builtin_amdgcn_wave_barrier();
        wave_rank_digits<uint32_t, BITS, MERGE_ITEMS>(key, wbase, count, shift, bits, lds.cnt[wave], rank);
        __syncthreads();
        // thread d: PER consecutive digits; their starts inside the tile, and the wavefronts' within them
        {
            uint32_t c[PER][MERGE_WAVES], total = 0, all;
            const uint32_t d0 = threadIdx.x * PER;
            const bool owner = d0 < DIGITS;
#pragma unroll
            for (int w = 0; w < MERGE_WAVES; ++w)
#pragma unroll
                for (int j = 0; j < PER; ++j) {
                    c[j][w] = owner ? lds.cnt[w][d0 + j] : 0u;
                    total += c[j][w];
                }
            uint32_t run = block_inclusive_scan<uint32_t, MERGE_BLOCK>(total, lds.wave_sums, all) - total;
#pragma unroll
            for (int j = 0; j < PER; ++j)
#pragma unroll
                for (int w = 0; w < MERGE_WAVES; ++w) {
                    const uint32_t n = c[j][w];
                    c[j][w] = run;
                    run += n;
                }
            if (owner) {
#pragma unroll
                for (int w = 0; w < MERGE_WAVES; ++w)
#pragma unroll
                    for (int j = 0; j < PER; ++j) lds.cnt[w][d0 + j] = c[j][w];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MERGE_ITEMS; ++k) {
            if (wbase + k * EMB_WAVE + lane < count) {
                const uint32_t to = lds.cnt[wave][(key[k] >> shift) & digit_mask] + rank[k];
                lds.sk[to] = key[k];
                lds.sp[to] = pay[k];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MERGE_ITEMS; ++k) {   // the records of the next pass, or of the way out
            const uint32_t i = wbase + k * EMB_WAVE + lane;
            if (i < count) {
                key[k] = lds.sk[i];
                pay[k] = lds.sp[i];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < MERGE_ITEMS; ++k) {
        const uint32_t i = wbase + k * EMB_WAVE + lane;
        if (i < count) {
            a.keys_out[start + i] = a.last ? (key[k] == a.local_sentinel ? a.global_sentinel : key[k] + row_base) : key[k];
            a.pay_out[start + i] = pay[k];
        }
    }
}

// The records are in memory (emb_bag_backward_sort's).
template <int BITS>
__global__ __launch_bounds__(MERGE_BLOCK) void tile_sort_kernel(const uint32_t *__restrict__ keys_in,
                                                                const uint32_t *__restrict__ pay_in,
                                                                const int64_t *__restrict__ table_start, int32_t T,
                                                                const emb_table *__restrict__ tables, TileSortArgs a,
                                                                const BwdCtrl *ctrl)
{
    __shared__ TileSortLds lds;
    const uint32_t gid = blockIdx.x * MERGE_BLOCK + threadIdx.x;
    if (gid < a.n_flags) a.span_flags[gid] = 0u;
    MergePart tile;
    if (!merge_part_of<MERGE_TILE, MERGE_BLOCK>(table_start, T, blockIdx.x, ctrl, tile)) return;
    const uint32_t start = tile.seg_start + tile.index * MERGE_TILE;
    tile_sort<BITS>(a, tile, a.last ? (uint32_t)tables[tile.table].row_base : 0u, lds,
              [&](const uint32_t (&i)[MERGE_ITEMS], uint32_t count, uint32_t (&key)[MERGE_ITEMS], uint32_t (&pay)[MERGE_ITEMS]) {
#pragma unroll
                  for (int k = 0; k < MERGE_ITEMS; ++k) {
                      if (i[k] < count) {
                          key[k] = keys_in[start + i[k]];
                          pay[k] = pay_in[start + i[k]];
                      }
                  }
              });
}

// ---------------------------------------------------------------------------
// tiles straight from raw IDs, for the launch that does the lookup beside it
// ---------------------------------------------------------------------------
// The tile's workgroup needs the tables' record ranges and the bag of every record before any launch has written them: both
// come from the bag offsets, which it makes itself in one of three forms.  Bags of the tile are found by bisection, first
// in LDS.
constexpr int TILE_SAMPLES = MERGE_BLOCK;
static_assert((EMB_LENGTHS_DIRECT_BAGS + 1) * 4 <= sizeof(TileSortLds) && (2 * TILE_SAMPLES + 1) * 4 <= sizeof(TileSortLds),
              "the offsets stand where the sort counts afterwards");

// Offsets of up to EMB_LENGTHS_DIRECT_BAGS bags from their lengths, all of them, to LDS ([n + 1]); a negative length counts
// as 0.  False (uniform): they do not add up to nnz.
__device__ __forceinline__ bool tile_offsets_from_lengths(const int32_t *__restrict__ lengths, uint32_t n, int64_t nnz,
                                                          uint32_t *off /*LDS*/, int64_t *wave_sums /*LDS*/)
{
    constexpr int PER = EMB_LENGTHS_DIRECT_BAGS / MERGE_BLOCK;
    static_assert(PER * MERGE_BLOCK == EMB_LENGTHS_DIRECT_BAGS && PER % 4 == 0, "a thread's lengths are 16-byte accesses of LDS");
    int32_t v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const uint32_t i = u * MERGE_BLOCK + threadIdx.x;
        v[u] = i < n ? lengths[i] : 0;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) off[u * MERGE_BLOCK + threadIdx.x] = v[u] < 0 ? 0u : (uint32_t)v[u];
    __syncthreads();
    uint4 *const own = reinterpret_cast<uint4 *>(off + threadIdx.x * PER);
    uint4 x[PER / 4];
    int64_t mine = 0, total;
#pragma unroll
    for (int u = 0; u < PER / 4; ++u) {
        x[u] = own[u];
        mine += (int64_t)x[u].x + x[u].y + x[u].z + x[u].w;
    }
    const int64_t before = block_inclusive_scan<int64_t, MERGE_BLOCK>(mine, wave_sums, total) - mine;   // (has barriers)
    if (total != nnz) return false;
    uint32_t run = (uint32_t)before;   // nnz is below 2^31
#pragma unroll
    for (int u = 0; u < PER / 4; ++u) {
        const uint4 l = x[u];
        own[u] = make_uint4(run, run + l.x, run + l.x + l.y, run + l.x + l.y + l.z);
        run += l.x + l.y + l.z + l.w;
    }
    if (threadIdx.x == MERGE_BLOCK - 1) off[EMB_LENGTHS_DIRECT_BAGS] = run;   // (entries after the last bag hold nnz)
    __syncthreads();
    return true;
}

// For MERGE_ITEMS places j at once: the last of n ascending values, from lo on, that is at most j (lo itself if none is; the
// number is counted from lo).  value(i) may be asked for i < n.
template <typename Value>
__device__ __forceinline__ void last_at_most(uint32_t n, const uint32_t (&j)[MERGE_ITEMS], uint32_t (&found)[MERGE_ITEMS],
                                             const Value &value)
{
#pragma unroll
    for (int k = 0; k < MERGE_ITEMS; ++k) found[k] = 0;
    for (uint32_t step = 1u << (31 - __clz((int)n)); step >= 1; step >>= 1) {   // uniform
#pragma unroll
        for (int k = 0; k < MERGE_ITEMS; ++k) {
            const uint32_t next = found[k] + step;
            if (next < n && value(k, next) <= j[k]) found[k] = next;
        }
    }
}

// Tile `number` of a small step, from raw IDs (hashed here as the lookup does).  lengths != NULL: up to
// EMB_LENGTHS_DIRECT_BAGS bags, given by their lengths; else MAKE_OFFSETS: `offsets` are sums within tiles
// (emb_offsets_tile_sums) of at most MERGE_BLOCK tiles, whose prefix sums are taken here; else offsets as
// emb_offset_at takes them, and table_start and ctrl are set up already.
template <bool MAKE_OFFSETS>
__device__ __forceinline__ void tile_sort_raw(const TileSortArgs &a, uint32_t number, const emb_table *__restrict__ tables,
                                              int32_t T, int64_t B, int64_t nnz, const int64_t *__restrict__ raw,
                                              const int32_t *__restrict__ lengths, const int64_t *__restrict__ offsets,
                                              const int64_t *__restrict__ tile_prefix, const int64_t *__restrict__ table_start,
                                              const BwdCtrl *ctrl)
{
    __shared__ TileSortLds lds;
    __shared__ int64_t wave_sums[MERGE_WAVES];
    uint32_t *const off = reinterpret_cast<uint32_t *>(&lds);
    uint32_t *const prefix = off + TILE_SAMPLES;
    const uint32_t gid = number * MERGE_BLOCK + threadIdx.x;
    if (gid < a.n_flags) a.span_flags[gid] = 0u;
    // first record of bag i, where it is not in LDS already (sums that are no offsets give a number like any other: the
    // backward is aborted then)
    auto bag_start = [&](int64_t i) -> uint32_t {
        if (MAKE_OFFSETS) return (uint32_t)offsets[i] + (i > 0 ? prefix[(i - 1) / EMB_OFFSETS_TILE] : 0u);
        return (uint32_t)emb_offset_at(offsets, tile_prefix, i);
    };
    MergePart tile;
    bool there;
    if (MAKE_OFFSETS && lengths) {   // uniform
        if (!tile_offsets_from_lengths(lengths, (uint32_t)(T * B), nnz, off, wave_sums)) return;
        there = merge_part_in<MERGE_TILE, MERGE_BLOCK>(T, number, [&](int32_t t, uint32_t &s, uint32_t &e) {
            s = off[t * (uint32_t)B];
            e = off[(t + 1) * (uint32_t)B];
        }, tile);
    } else if (MAKE_OFFSETS) {
        const int64_t n = (int64_t)T * B, k = threadIdx.x;
        int64_t end = (k + 1) * EMB_OFFSETS_TILE, total;
        if (end > n) end = n;
        const int64_t v = k * EMB_OFFSETS_TILE < n ? offsets[end] : 0;   // the tile's total stands at its end
        const int64_t inc = block_inclusive_scan<int64_t, MERGE_BLOCK>(v, wave_sums, total);
        if (total != nnz) return;   // uniform; the lookup aborts the backward
        prefix[k] = (uint32_t)(inc - v);
        __syncthreads();
        there = merge_part_in<MERGE_TILE, MERGE_BLOCK>(T, number, [&](int32_t t, uint32_t &s, uint32_t &e) {
            s = bag_start(t * B);
            e = bag_start((t + 1) * B);
        }, tile);
    } else {
        there = merge_part_of<MERGE_TILE, MERGE_BLOCK>(table_start, T, number, ctrl, tile);
    }
    if (!there) return;   // uniform
    const emb_table tb = tables[tile.table];
    const uint32_t first_bag = tile.table * (uint32_t)B, n_bags = (uint32_t)B;   // (T * B fits 32 bits)
    const uint32_t step = (n_bags + TILE_SAMPLES - 1) / TILE_SAMPLES;
    if (!(MAKE_OFFSETS && lengths)) {
        const uint64_t at = (uint64_t)threadIdx.x * step;
        off[threadIdx.x] = at < n_bags ? bag_start((int64_t)first_bag + (int64_t)at) : 0xFFFFFFFFu;
        __syncthreads();
    }
    const uint32_t start = tile.seg_start + tile.index * MERGE_TILE;
    tile_sort<0>(a, tile, a.last ? (uint32_t)tb.row_base : 0u, lds,
              [&](const uint32_t (&i)[MERGE_ITEMS], uint32_t count, uint32_t (&key)[MERGE_ITEMS], uint32_t (&pay)[MERGE_ITEMS]) {
        uint64_t id[MERGE_ITEMS];
        uint32_t j[MERGE_ITEMS], bag[MERGE_ITEMS];
#pragma unroll
        for (int k = 0; k < MERGE_ITEMS; ++k) {
            j[k] = start + i[k];
            id[k] = i[k] < count ? (uint64_t)raw[j[k]] : 0ull;
        }
        if (MAKE_OFFSETS && lengths) {
            last_at_most(n_bags, j, bag, [&](int, uint32_t b) { return off[first_bag + b]; });
        } else {
            uint32_t part[MERGE_ITEMS];
            last_at_most(TILE_SAMPLES, j, part, [&](int, uint32_t b) { return off[b]; });
            last_at_most(step, j, bag, [&](int k, uint32_t b) {
                const uint32_t at = part[k] * step + b;
                return at < n_bags ? bag_start((int64_t)first_bag + at) : 0xFFFFFFFFu;
            });
#pragma unroll
            for (int k = 0; k < MERGE_ITEMS; ++k) bag[k] += part[k] * step;
        }
#pragma unroll
        for (int k = 0; k < MERGE_ITEMS; ++k) {
            key[k] = (uint32_t)emb_fast_mod(emb_splitmix64(id[k] ^ tb.salt), (uint64_t)tb.num_rows, tb.mod_magic);
            pay[k] = first_bag + bag[k];
        }
    });
}

// Every record's place in its table: its place in its own tile and, for each other tile of the table, the number
// of that tile's records that come before it (smaller keys; equal ones of earlier tiles too, which keeps the
// order stable).  The tiles' keys go through LDS, PLACE_TILES tiles a round, and a thread bisects those for its record
// side by side: a bisection is a chain of LDS reads that wait for each other (one in 4096 keys for eight records
// a thread, one after the other, made 6 us of every 4096 records of the table).  The next round's keys are requested
// while the current ones are searched.  Also clears the words of the list of distinct rows (list_flags, [list_tiles],
// optional), which is the next launch (a step that is not merged has one such word, and nobody waits for it).
__global__ __launch_bounds__(PLACE_BLOCK) void tile_merge_kernel(const uint32_t *__restrict__ keys_in,
                                                                 const uint32_t *__restrict__ pay_in,
                                                                 uint32_t *__restrict__ keys_out,
                                                                 uint32_t *__restrict__ pay_out,
                                                                 const int64_t *__restrict__ table_start, int32_t T,
                                                                 const emb_table *__restrict__ tables,
                                                                 uint32_t local_sentinel, uint32_t global_sentinel,
                                                                 unsigned long long *__restrict__ list_flags,
                                                                 uint32_t list_tiles, const BwdCtrl *ctrl)
{
    const uint32_t gid = blockIdx.x * PLACE_BLOCK + threadIdx.x;
    if (list_flags && gid < list_tiles) list_flags[gid] = 0ull;
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
