// Which rows the HBM hot-row cache of a host-resident table holds (paper
// Section 3.3 for the hosted table; Section 6 names better caching strategies
// as open work and gives no policy, so this one is a stated choice):
// frequency-based admission with batched refresh.
//
//   observe   one u32 counter per table row counts the lookups of that row;
//   select    at a refresh the cache takes the num_hot rows with the largest
//             counters (a tie goes to the smaller row number), and the
//             counters are aged by a right shift.
//
// The selection is an exact top-k without a sort.  One pass over the counters
// counts every value below SEL_EXACT in a bin of its own; the bin in which the
// num_hot-th row in preference order falls is the threshold.  Only if that row
// lies among the larger values (a small cache refreshed after very much traffic)
// do three more passes find it digit by digit; they return at once otherwise.
// Then a pass counts the selected rows per tile, a scan places the tiles, and a
// last pass writes the rows in ascending order, the order the cache index needs,
// and ages the counters.  A refresh (emb_cache_refresh) lets that last pass write
// the index and fetch the rows of the new cache as well, all but those of tiles
// with very many chosen rows (sel_wide_copy_kernel).  Everything is integer work:
// results are exact.
//
// What bounds it: 80 MB of counters (2e7 rows) are read three times (16 us each
// at the rate of a large copy; the second and third time from the memory-side
// cache) and written only where they are not zero.  With one histogram pass per
// 8-bit digit, each ending in 4096 workgroups adding to the same few words (such
// adds are served one at a time, about 24 ns each), a selection took 395 us.
#include <mutex>

#include "cache_index.h"
#include "emb_internal.h"
#include "scan.h"
#include "u64mod.h"

namespace {

constexpr int CP_BLOCK = 256;
constexpr int SEL_PER_THREAD = 16;                         // consecutive rows per thread in count/write
constexpr int SEL_TILE = CP_BLOCK * SEL_PER_THREAD;        // rows per workgroup in count/write
constexpr int SEL_BLOCK = 1024;                            // workgroups of the histogram passes, the pick and the scan
constexpr int SEL_BINS = 2048;
constexpr uint32_t SEL_EXACT = SEL_BINS - 1;               // values below have a bin each, the others share the last one
constexpr int SEL_REPLICAS = 8;                            // of the first histogram: fewer adds per word
constexpr int SEL_HIST_BLOCKS = 256;                       // one workgroup per CU: 64 KB of loads in flight each
constexpr int SEL_GROUPS = 64;                             // words that collect the kept rows of a refresh
constexpr int64_t SEL_TILE_CHUNKS = 4 * SEL_TILE;          // chunks that a tile's workgroup copies itself, or, where that is
constexpr int64_t SEL_TILE_SHARE = 256;                    // more, this part of all chunks (sel_wide_copy_kernel)
constexpr int SEL_WIDE_GRID = 256;                         // with two loads a lane 2 MB in flight
constexpr int SEL_WIDE_UNROLL = 2;
constexpr int SEL_WIDE_CHUNKS = 512;                       // a wavefront's share of rows: at most so many chunks, or one row
// digits of the threshold where it is not below SEL_EXACT: bits 21.., 10..20, 0..9
constexpr int SEL_SHIFT1 = 21, SEL_SHIFT2 = 10;

struct SelCtrl {
    uint32_t exact;      // the threshold is below SEL_EXACT: thr0, take0
    uint32_t thr0;
    uint64_t take0;      // rows to take among those at the threshold (exact) / among those not below SEL_EXACT
    uint32_t digit1, pad0;
    uint64_t need1;      // after the first digit
    uint32_t prefix2, pad1;
    uint64_t need2;      // after the second
    uint32_t thr;        // the threshold and the number of rows to take at it
    uint32_t wide;       // a tile has left its rows to sel_wide_copy_kernel
    uint64_t take;
};
static_assert(sizeof(SelCtrl) <= 256, "the control block has 256 bytes");

// Workspace: SelCtrl | hist u64[SEL_REPLICAS + 3][SEL_BINS] | groups u64[SEL_GROUPS] | base u64[tiles] | counts u32[tiles] | ties u32[tiles]
struct SelLayout {
    size_t ctrl, hist, groups, base, counts, ties, total;
    int64_t tiles;
};
constexpr int SEL_HIST_WORDS = (SEL_REPLICAS + 3) * SEL_BINS;

SelLayout sel_layout(int64_t num_rows)
{
    SelLayout L;
    L.tiles = (num_rows + SEL_TILE - 1) / SEL_TILE;
    size_t o = 0;
    L.ctrl = o;
    o += 256;
    L.hist = o;
    o += sizeof(uint64_t) * SEL_HIST_WORDS;
    L.groups = o;      // cleared together with the histograms: must follow them
    o += sizeof(uint64_t) * SEL_GROUPS;
    L.base = o;
    o += ((size_t)L.tiles * sizeof(uint64_t) + 255) / 256 * 256;
    L.counts = o;
    o += ((size_t)L.tiles * sizeof(uint32_t) + 255) / 256 * 256;
    L.ties = o;
    o += ((size_t)L.tiles * sizeof(uint32_t) + 255) / 256 * 256;
    L.total = o;
    return L;
}

// Popular rows repeat: under a Zipf law the most popular row alone takes a tenth of all lookups, and
// atomics on one address are served one at a time by the L2.  A workgroup therefore first merges its
// OBS_TILE lookups in a small LDS hash table (row -> count, open addressing) and then adds each distinct
// row's count to its counter once.  A lookup that finds no slot within a few probes goes to its counter
// directly, so the result is the exact count either way.  Tiles are as large as a full CU takes at once:
// a row that every tile holds is added to once per tile.  SlotT: 32 bits where every row number fits,
// which halves the table.
constexpr int OBS_BLOCK = 1024;
constexpr int OBS_ITEMS = 4;                       // lookups per thread
constexpr int OBS_TILE = OBS_BLOCK * OBS_ITEMS;    // lookups per workgroup
constexpr int OBS_SLOTS = 2 * OBS_TILE;            // load factor at most one half
constexpr int OBS_PROBES = 8;

template <bool HASHED, typename SlotT>
__global__ __launch_bounds__(OBS_BLOCK) void cache_observe_kernel(const int64_t *__restrict__ ids, int64_t nnz,
                                                                  uint64_t num_rows, uint64_t salt, uint64_t magic,
                                                                  uint32_t *freq, uint32_t *status)
{
    constexpr SlotT EMPTY = ~(SlotT)0;             // not a row number: the host picks SlotT accordingly
    __shared__ SlotT keys[OBS_SLOTS];
    __shared__ uint32_t counts[OBS_SLOTS];
    const int64_t base = (int64_t)blockIdx.x * OBS_TILE + threadIdx.x;
    uint64_t r[OBS_ITEMS];
#pragma unroll
    for (int k = 0; k < OBS_ITEMS; ++k) {
        const int64_t j = base + (int64_t)k * OBS_BLOCK;
        r[k] = j < nnz ? (uint64_t)ids[j] : 0ull;
    }
    for (int i = threadIdx.x; i < OBS_SLOTS; i += OBS_BLOCK) {
        keys[i] = EMPTY;
        counts[i] = 0u;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < OBS_ITEMS; ++k) {
        if (base + (int64_t)k * OBS_BLOCK >= nnz) continue;
        uint64_t row = r[k];
        if (HASHED) row = emb_fast_mod(emb_splitmix64(row ^ salt), num_rows, magic);
        if (row >= num_rows) {  // negative row numbers are huge as unsigned
            emb_flag(status, EMB_STATUS_BAD_INDEX);
            continue;
        }
        uint32_t slot = (uint32_t)((row * UINT64_C(0x9E3779B97F4A7C15)) >> 32) & (OBS_SLOTS - 1);
        bool placed = false;
        for (int p = 0; p < OBS_PROBES && !placed; ++p) {
            const SlotT prev = atomicCAS(&keys[slot], EMPTY, (SlotT)row);
            if (prev == EMPTY || prev == (SlotT)row) {
                atomicAdd(&counts[slot], 1u);
                placed = true;
            } else {
                slot = (slot + 1) & (OBS_SLOTS - 1);
            }
        }
        if (!placed) atomicAdd(freq + row, 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < OBS_SLOTS; i += OBS_BLOCK) {
        const uint32_t c = counts[i];
        if (c) atomicAdd(freq + keys[i], c);
    }
}

// Clears the histograms and the words after them (SelLayout); `words` is their number.
__global__ __launch_bounds__(CP_BLOCK) void sel_init_kernel(unsigned long long *hist, int words)
{
    for (int i = blockIdx.x * CP_BLOCK + threadIdx.x; i < words; i += gridDim.x * CP_BLOCK) hist[i] = 0ull;
}

// The counters of one grid-stride trip of a thread: four, `valid` of them inside the array.
__device__ __forceinline__ void sel_load4(const uint32_t *__restrict__ freq, int64_t q, int64_t num_rows, uint32_t (&v)[4],
                                          int &valid)
{
    const int64_t r0 = q * 4;
    v[0] = v[1] = v[2] = v[3] = 0u;
    valid = 0;
    if (r0 + 4 <= num_rows) {
        const uint4 x = *reinterpret_cast<const uint4 *>(freq + r0);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        valid = 4;
    } else if (r0 < num_rows) {
        valid = (int)(num_rows - r0);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c < valid) v[c] = freq[r0 + c];
    }
}

// Histogram of the counters with a bin for each value below SEL_EXACT.  Most counters are zero and most of
// the others small: the values 0 to 3 are counted in registers (four 16-bit fields of one word, flushed
// before they can overflow), those of the last bin in another, the rest by LDS adds.  A workgroup adds its bins to
// one of SEL_REPLICAS copies.
__global__ __launch_bounds__(SEL_BLOCK) void sel_values_kernel(const uint32_t *__restrict__ freq, int64_t num_rows,
                                                               unsigned long long *__restrict__ hist)
{
    __shared__ uint32_t lds[SEL_BINS];   // a workgroup counts num_rows / 256 values: below 2^32 for any array a GPU holds
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_BLOCK) lds[i] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & (EMB_WAVE - 1);
    const int64_t quads = (num_rows + 3) / 4;
    const int64_t stride = (int64_t)gridDim.x * SEL_BLOCK;
    constexpr int UNROLL = 4;
    constexpr int FLUSH = 65535 / (4 * UNROLL);   // trips until a 16-bit field may be full
    int64_t q = (int64_t)blockIdx.x * SEL_BLOCK + threadIdx.x;
    const int64_t trips = (quads + UNROLL * stride - 1) / (UNROLL * stride);   // the same for every thread
    uint32_t large = 0u;
    for (int64_t t0 = 0; t0 < trips; t0 += FLUSH) {
        unsigned long long small = 0ull;
        const int64_t t1 = t0 + FLUSH < trips ? t0 + FLUSH : trips;
        for (int64_t t = t0; t < t1; ++t) {
            uint32_t v[UNROLL][4];
            int valid[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) sel_load4(freq, q + u * stride, num_rows, v[u], valid[u]);
            q += UNROLL * stride;
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t x = v[u][c];
                    if (c >= valid[u]) continue;
                    if (x < 4u) small += 1ull << (16 * x);
                    else if (x < SEL_EXACT) atomicAdd(&lds[x], 1u);
                    else ++large;
                }
        }
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            uint32_t c = (uint32_t)(small >> (16 * f)) & 0xFFFFu;
#pragma unroll
            for (int d = EMB_WAVE >> 1; d >= 1; d >>= 1) c += __shfl_xor(c, d, EMB_WAVE);
            if (lane == 0 && c) atomicAdd(&lds[f], c);
        }
    }
#pragma unroll
    for (int d = EMB_WAVE >> 1; d >= 1; d >>= 1) large += __shfl_xor(large, d, EMB_WAVE);
    if (lane == 0 && large) atomicAdd(&lds[SEL_EXACT], large);
    __syncthreads();
    unsigned long long *mine = hist + (size_t)(blockIdx.x % SEL_REPLICAS) * SEL_BINS;
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_BLOCK) {
        const uint32_t n = lds[i];
        if (n) atomicAdd(mine + i, (unsigned long long)n);
    }
}

// The largest bin such that the bins above it hold fewer than `need` entries (1 <= need <= all of them),
// and how many of its own entries are needed.  Every thread of the workgroup calls this.
template <int BLOCK, int BINS, int REPLICAS>
__device__ __forceinline__ void sel_pick(const unsigned long long *__restrict__ hist, uint64_t need, uint32_t &bin,
                                         uint64_t &left)
{
    constexpr int PER = BINS / BLOCK;
    static_assert(PER * BLOCK == BINS, "whole bins per thread");
    __shared__ unsigned long long wave_sums[BLOCK / EMB_WAVE];
    __shared__ unsigned long long s_left;
    __shared__ uint32_t s_bin;
    unsigned long long c[PER], mine = 0ull;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int b = BINS - 1 - ((int)threadIdx.x * PER + i);   // descending
        c[i] = 0ull;
#pragma unroll
        for (int k = 0; k < REPLICAS; ++k) c[i] += hist[(size_t)k * SEL_BINS + b];
        mine += c[i];
    }
    unsigned long long all;
    unsigned long long above = block_inclusive_scan<unsigned long long, BLOCK>(mine, wave_sums, all) - mine;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (above < need && above + c[i] >= need) {              // one bin of one thread
            s_bin = (uint32_t)(BINS - 1 - ((int)threadIdx.x * PER + i));
            s_left = need - above;
        }
        above += c[i];
    }
    __syncthreads();
    bin = s_bin;
    left = s_left;
}

__global__ __launch_bounds__(SEL_BLOCK) void sel_pick_kernel(const unsigned long long *__restrict__ hist, int64_t num_hot,
                                                             SelCtrl *ctrl)
{
    uint32_t bin;
    uint64_t left;
    sel_pick<SEL_BLOCK, SEL_BINS, SEL_REPLICAS>(hist, (uint64_t)num_hot, bin, left);
    if (threadIdx.x == 0) {
        ctrl->exact = bin < SEL_EXACT ? 1u : 0u;
        ctrl->thr0 = bin;
        ctrl->take0 = left;
        ctrl->wide = 0u;
    }
}

// Adds one to the bin of every lane that has one.  Counters of like size share their upper digits, and an LDS add of
// 64 lanes to one word is served lane by lane: where the wavefront has one bin, one lane adds for all (2.5e8 counters
// of 3000: the three digits 3130 us with an add per lane, 780 so).
__device__ __forceinline__ void sel_add(uint32_t *lds, bool counted, uint32_t bin)
{
    const unsigned long long lanes = __ballot(counted);
    if (lanes == 0ull) return;
    const int first = __ffsll(lanes) - 1;
    const uint32_t bin0 = (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
    if (__ballot(counted && bin == bin0) == lanes) {
        if ((int)(threadIdx.x & (EMB_WAVE - 1)) == first) atomicAdd(&lds[bin0], (uint32_t)__popcll(lanes));
    } else if (counted) {
        atomicAdd(&lds[bin], 1u);
    }
}

// Where the threshold is not below SEL_EXACT: histogram of digit DIGIT (1, 2, 3 from the top) over the
// counters not below SEL_EXACT whose digits above it are those of the threshold.  Every workgroup picks the
// digit before from the finished histogram; the first one leaves it for the next launch.
template <int DIGIT>
__global__ __launch_bounds__(SEL_BLOCK) void sel_digit_kernel(const uint32_t *__restrict__ freq, int64_t num_rows,
                                                              SelCtrl *ctrl, const unsigned long long *__restrict__ before,
                                                              unsigned long long *__restrict__ hist)
{
    if (ctrl->exact) return;   // uniform
    __shared__ uint32_t lds[SEL_BINS];
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_BLOCK) lds[i] = 0u;
    uint32_t prefix = 0u;
    if (DIGIT == 2) {
        uint64_t left;
        sel_pick<SEL_BLOCK, SEL_BINS, 1>(before, ctrl->take0, prefix, left);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            ctrl->digit1 = prefix;
            ctrl->need1 = left;
        }
    }
    if (DIGIT == 3) {
        uint64_t left;
        uint32_t d;
        sel_pick<SEL_BLOCK, SEL_BINS, 1>(before, ctrl->need1, d, left);
        prefix = (ctrl->digit1 << (SEL_SHIFT1 - SEL_SHIFT2)) | d;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            ctrl->prefix2 = prefix;
            ctrl->need2 = left;
        }
    }
    __syncthreads();
    const int64_t quads = (num_rows + 3) / 4;
    const int64_t stride = (int64_t)gridDim.x * SEL_BLOCK;
    constexpr int UNROLL = 4;
    for (int64_t q0 = (int64_t)blockIdx.x * SEL_BLOCK; q0 < quads; q0 += UNROLL * stride) {   // the same for every thread
        uint32_t v[UNROLL][4];
        int valid[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) sel_load4(freq, q0 + threadIdx.x + u * stride, num_rows, v[u], valid[u]);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t x = v[u][c];   // counters past the array read as zero
                const bool large = x >= SEL_EXACT;
                if (DIGIT == 1) sel_add(lds, large, x >> SEL_SHIFT1);
                if (DIGIT == 2) sel_add(lds, large && (x >> SEL_SHIFT1) == prefix, (x >> SEL_SHIFT2) & (SEL_BINS - 1));
                if (DIGIT == 3) sel_add(lds, large && (x >> SEL_SHIFT2) == prefix, x & ((1u << SEL_SHIFT2) - 1));
            }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_BLOCK) {
        const uint32_t n = lds[i];
        if (n) atomicAdd(hist + i, (unsigned long long)n);
    }
}

__device__ __forceinline__ void sel_load16(const uint32_t *__restrict__ freq, int64_t r0, int64_t num_rows, uint32_t (&v)[SEL_PER_THREAD],
                                           int &valid)
{
    if (r0 + SEL_PER_THREAD <= num_rows) {
#pragma unroll
        for (int i = 0; i < SEL_PER_THREAD / 4; ++i) {
            const uint4 x = *reinterpret_cast<const uint4 *>(freq + r0 + 4 * i);
            v[4 * i] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
        }
        valid = SEL_PER_THREAD;
    } else {
        valid = r0 < num_rows ? (int)(num_rows - r0) : 0;
#pragma unroll
        for (int i = 0; i < SEL_PER_THREAD; ++i) v[i] = i < valid ? freq[r0 + i] : 0u;
    }
}

// A tile's counts travel as (above-threshold count | at-threshold count << 16): neither exceeds SEL_TILE = 4096.
__device__ __forceinline__ uint32_t sel_counts(const uint32_t (&v)[SEL_PER_THREAD], int valid, uint32_t thr)
{
    uint32_t mine = 0u;
#pragma unroll
    for (int i = 0; i < SEL_PER_THREAD; ++i)
        if (i < valid) mine += v[i] > thr ? 1u : (v[i] == thr ? 0x10000u : 0u);
    return mine;
}

// Per tile of SEL_TILE rows: how many counters lie above the threshold, how many equal it.  Settles the
// threshold first (the last digit's pick, where digits were needed) and leaves it in the control block.
__global__ __launch_bounds__(CP_BLOCK) void sel_count_kernel(const uint32_t *__restrict__ freq, int64_t num_rows,
                                                             SelCtrl *ctrl, const unsigned long long *__restrict__ hist3,
                                                             uint32_t *__restrict__ counts)
{
    __shared__ uint32_t wave_sum[CP_BLOCK / EMB_WAVE];
    const int64_t r0 = (int64_t)blockIdx.x * SEL_TILE + (int64_t)threadIdx.x * SEL_PER_THREAD;
    uint32_t v[SEL_PER_THREAD];
    int valid;
    sel_load16(freq, r0, num_rows, v, valid);
    uint32_t thr = ctrl->thr0;
    uint64_t take = ctrl->take0;
    if (!ctrl->exact) {   // uniform
        uint32_t d;
        sel_pick<CP_BLOCK, 1 << SEL_SHIFT2, 1>(hist3, ctrl->need2, d, take);
        thr = (ctrl->prefix2 << SEL_SHIFT2) | d;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctrl->thr = thr;
        ctrl->take = take;
    }
    uint32_t mine = sel_counts(v, valid, thr);
#pragma unroll
    for (int d = EMB_WAVE >> 1; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, EMB_WAVE);
    if ((threadIdx.x & (EMB_WAVE - 1)) == 0) wave_sum[threadIdx.x / EMB_WAVE] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t all = 0u;
#pragma unroll
        for (int w = 0; w < CP_BLOCK / EMB_WAVE; ++w) all += wave_sum[w];
        counts[blockIdx.x] = all;
    }
}

// One workgroup: where every tile's rows go.  base = selected rows before the tile; ties = at-threshold rows
// that may still be taken in the tile (SEL_TILE: all of them).
__global__ __launch_bounds__(SEL_BLOCK) void sel_scan_kernel(const uint32_t *__restrict__ counts, int64_t tiles,
                                                             const SelCtrl *__restrict__ ctrl,
                                                             unsigned long long *__restrict__ base,
                                                             uint32_t *__restrict__ ties, uint64_t *info)
{
    constexpr int PER = 4;
    __shared__ unsigned long long wave_sums[SEL_BLOCK / EMB_WAVE];
    const uint64_t take = ctrl->take;
    if (info && threadIdx.x == 0) {
        info[0] = ctrl->thr;
        info[1] = take;
    }
    uint64_t gt_carry = 0, eq_carry = 0;
    for (int64_t t0 = 0; t0 < tiles; t0 += SEL_BLOCK * PER) {
        const int64_t at = t0 + (int64_t)threadIdx.x * PER;
        uint32_t c[PER];
        unsigned long long mine = 0ull;   // low half: above, high half: at the threshold (at most 2^24 each)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            c[i] = at + i < tiles ? counts[at + i] : 0u;
            mine += (unsigned long long)(c[i] & 0xFFFFu) | ((unsigned long long)(c[i] >> 16) << 32);
        }
        unsigned long long all;
        const unsigned long long excl = block_inclusive_scan<unsigned long long, SEL_BLOCK>(mine, wave_sums, all) - mine;
        uint64_t gt = gt_carry + (uint32_t)excl, eq = eq_carry + (uint32_t)(excl >> 32);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (at + i < tiles) {
                const uint64_t used = eq < take ? eq : take;
                base[at + i] = gt + used;
                ties[at + i] = (uint32_t)(take - used < SEL_TILE ? take - used : SEL_TILE);
            }
            gt += c[i] & 0xFFFFu;
            eq += c[i] >> 16;
        }
        gt_carry += (uint32_t)all;
        eq_carry += (uint32_t)(all >> 32);
    }
}

// What the last pass of a refresh needs beside the selection.
struct RefreshArgs {
    const char *table;            // the hosted table
    const char *old_rows;         // the cache in use
    const CacheEntry *old_index;
    int64_t old_num_hot;
    char *new_rows;               // the cache being made
    CacheEntry *new_index;
    int32_t chunks;               // 16-byte chunks per row
    uint32_t chunk_magic;         // floor(2^32 / chunks) + 1: i / chunks for i < SEL_TILE * 1024 (0: one chunk)
    unsigned long long *moved;    // nullable
    unsigned long long *groups;   // [SEL_GROUPS], zero
    uint32_t tile_chunks;         // a tile with more chunks than this leaves them to sel_wide_copy_kernel
    uint32_t *wide;               // SelCtrl::wide
};

// Write the selected rows in ascending order and age the counters.  A row is selected if its counter is above
// the threshold, or equals it and fewer than `take` rows with that counter precede it.  The rows of a tile are
// put in order in LDS and written out with consecutive lanes.  A counter that is zero needs no store.
//
// REFRESH: the pass has the new cache's index in its hands (a thread's 16 rows are a quarter of an entry, and
// a row's place in the cache is its place in the list), so it writes the entries, and fetches the rows: those
// the old cache holds from there, the others from the table.  The reads over the link are what bounds it (one
// 128-byte line per 3 ns in ascending order: 1.66e5 new rows of 48 bytes 585 us); copying inside this pass
// they start with the first tile.  Before, clearing the index, marking it with one atomic per row (62 us) and
// copying with two same-address adds per wavefront were launches of their own (830 us together).
template <bool REFRESH>
__global__ __launch_bounds__(CP_BLOCK) void sel_write_kernel(uint32_t *freq, int64_t num_rows, const SelCtrl *__restrict__ ctrl,
                                                             const unsigned long long *__restrict__ base,
                                                             const uint32_t *__restrict__ ties, int64_t num_hot,
                                                             int decay_shift, int64_t *__restrict__ hot_out, RefreshArgs f)
{
    __shared__ uint32_t wave_sums[CP_BLOCK / EMB_WAVE];
    __shared__ uint16_t list[SEL_TILE];
    __shared__ uint4 old_entry[REFRESH ? SEL_TILE / 64 : 1];
    __shared__ uint32_t s_kept;
    const int64_t tile0 = (int64_t)blockIdx.x * SEL_TILE;
    const int64_t r0 = tile0 + (int64_t)threadIdx.x * SEL_PER_THREAD;
    uint32_t v[SEL_PER_THREAD];
    int valid;
    sel_load16(freq, r0, num_rows, v, valid);
    const uint32_t thr = ctrl->thr;
    const uint64_t tile_base = base[blockIdx.x];
    const uint32_t take = ties[blockIdx.x];
    if (REFRESH) {
        if (threadIdx.x < SEL_TILE / 64) {
            const int64_t e = tile0 / 64 + threadIdx.x;
            old_entry[threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
            // clipped, so that the rows counted as kept are the rows copied from the old cache
            if (e * 64 < num_rows)
                old_entry[threadIdx.x] = cache_clip(*reinterpret_cast<const uint4 *>(f.old_index + e), (uint64_t)f.old_num_hot);
        }
        if (threadIdx.x == 0) s_kept = 0u;
    }
    const uint32_t mine = sel_counts(v, valid, thr);
    uint32_t total;
    const uint32_t excl = block_inclusive_scan<uint32_t, CP_BLOCK>(mine, wave_sums, total) - mine;
    // places inside the tile
    uint32_t eq = excl >> 16;
    uint32_t pos = (excl & 0xFFFFu) + (eq < take ? eq : take);
    const uint32_t first = pos;
    const uint32_t tile_eq = total >> 16;
    const uint32_t selected = (total & 0xFFFFu) + (tile_eq < take ? tile_eq : take);
    uint32_t bits = 0u;
#pragma unroll
    for (int i = 0; i < SEL_PER_THREAD; ++i) {
        if (i >= valid) continue;
        const bool above = v[i] > thr, tied = v[i] == thr;
        if (above || (tied && eq < take)) {
            list[pos++] = (uint16_t)(threadIdx.x * SEL_PER_THREAD + i);
            bits |= 1u << i;
        }
        eq += tied ? 1u : 0u;
    }
    if (decay_shift > 0) {
        if (valid == SEL_PER_THREAD) {
#pragma unroll
            for (int i = 0; i < SEL_PER_THREAD / 4; ++i)
                if (v[4 * i] | v[4 * i + 1] | v[4 * i + 2] | v[4 * i + 3])
                    *reinterpret_cast<uint4 *>(freq + r0 + 4 * i) =
                        make_uint4(v[4 * i] >> decay_shift, v[4 * i + 1] >> decay_shift, v[4 * i + 2] >> decay_shift,
                                   v[4 * i + 3] >> decay_shift);
        } else {
            for (int i = 0; i < valid; ++i) freq[r0 + i] = v[i] >> decay_shift;
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < selected; i += CP_BLOCK) {
        const uint64_t at = tile_base + i;
        if (at < (uint64_t)num_hot) hot_out[at] = tile0 + list[i];   // always true; keeps a corrupted workspace from writing outside
    }
    if (!REFRESH) return;

    // ---- index: four threads hold the 64 rows of an entry
    {
        const int part = threadIdx.x & 3;
        uint32_t lo = part == 0 ? bits : (part == 1 ? bits << 16 : 0u);
        uint32_t hi = part == 2 ? bits : (part == 3 ? bits << 16 : 0u);
#pragma unroll
        for (int d = 1; d < 4; d <<= 1) {
            lo |= (uint32_t)__shfl_xor((int)lo, d, EMB_WAVE);
            hi |= (uint32_t)__shfl_xor((int)hi, d, EMB_WAVE);
        }
        const int64_t e = r0 / 64;
        uint32_t kept = 0u;
        if (part == 0 && e * 64 < num_rows) {
            const uint32_t before = (lo | hi) ? (uint32_t)(tile_base + first) : 0u;   // an entry without rows is all zero
            *reinterpret_cast<uint4 *>(f.new_index + e) = make_uint4(lo, hi, before, 0u);
            const uint4 old = old_entry[threadIdx.x / 4];
            kept = (uint32_t)(__popc(lo & old.x) + __popc(hi & old.y));
        }
#pragma unroll
        for (int d = EMB_WAVE >> 1; d >= 1; d >>= 1) kept += __shfl_xor(kept, d, EMB_WAVE);
        if (f.moved && (threadIdx.x & (EMB_WAVE - 1)) == 0 && kept) atomicAdd(&s_kept, kept);
    }
    // ---- rows: consecutive lanes copy consecutive chunks of the tile's part of the cache
    const uint32_t chunks = (uint32_t)f.chunks;
    uint32_t items = selected * chunks;
    if (items > f.tile_chunks) {   // uniform; sel_wide_copy_kernel tells such tiles by the same test
        items = 0u;
        if (threadIdx.x == 0) *f.wide = 1u;
    }
    constexpr int UNROLL = 4;
    for (uint32_t i0 = threadIdx.x; i0 < items; i0 += CP_BLOCK * UNROLL) {
        uint4 x[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint32_t i = i0 + u * CP_BLOCK;
            if (i < items) {
                const uint32_t k = f.chunk_magic ? __umulhi(i, f.chunk_magic) : i;
                const uint32_t c = i - k * chunks;
                const uint32_t row = list[k];
                const uint4 old = old_entry[row >> 6];
                const int64_t slot = cache_slot(old, (int)(row & 63u), (uint64_t)f.old_num_hot);
                const char *src = slot >= 0 ? f.old_rows + slot * (int64_t)chunks * 16
                                            : f.table + (tile0 + row) * (int64_t)chunks * 16;
                x[u] = load_chunk(src + (int64_t)c * 16);
            }
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint32_t i = i0 + u * CP_BLOCK;
            if (i < items && tile_base + selected <= (uint64_t)num_hot)   // the second is always true, as above
                *reinterpret_cast<uint4 *>(f.new_rows + (int64_t)(tile_base * chunks + i) * 16) = x[u];
        }
    }
    // ---- how many rows were kept: tiles report in groups, the last tile of a group adds the group's sum (a
    // count that travels in one word with the number of reports needs no fence)
    if (f.moved) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t g = blockIdx.x % SEL_GROUPS;
            const uint32_t members = (gridDim.x - g + SEL_GROUPS - 1) / SEL_GROUPS;
            const unsigned long long one = (1ull << 40) | s_kept;   // kept rows of a group: below 2^40
            const unsigned long long sum = atomicAdd(f.groups + g, one) + one;
            if ((uint32_t)(sum >> 40) == members) {
                const unsigned long long kept = sum & ((1ull << 40) - 1ull);
                if (kept) {
                    atomicAdd(&f.moved[0], kept);
                    atomicAdd(&f.moved[1], 0ull - kept);
                }
            }
            if (blockIdx.x == 0) atomicAdd(&f.moved[1], (unsigned long long)num_hot);   // all rows, less the kept ones
        }
    }
}

// The rows of the tiles that hold more than tile_chunks chunks of the new cache.  Left to the tile's one workgroup they
// are a serial chain of 1.5 us per 1024 chunks while the rest of the chip is idle: of 10 000 rows of 4096 bytes side by
// side a refresh took 1590 us with all of them in the old cache and 2455 with none.  Copied from the finished list,
// which is what this kernel does, it takes 61 and 776.  Tiles up to the line are the faster for being copied in the
// pass: 75 000 of 1.5e6 rows of 512 bytes, 6550 chunks a tile, 54 us, emb_cache_rebuild's copy 62; at 32 768 chunks a
// tile the two are even (95 us in the pass, 89 here).  And where no tile holds more than one part in SEL_TILE_SHARE of
// the cache, the chain of the fullest is no longer than the whole chip needs for all of it, and copying in the pass
// lets rows from the old cache pass beside those from the link: 1.25e7 rows of 256 bytes, 1.1e7 of them kept and most
// side by side, 7.8 ms in the pass, 9.1 with this kernel for every tile of more than 16 384 chunks.
// A wavefront takes a share of consecutive rows of the list: a lane each finds where a row comes from, then all
// lanes copy the share's chunks.  unit: rows of a share (at most EMB_WAVE).  2 MB in flight are what the two places
// that rows come from agree on: 4096-byte rows, 2, 4 and 8 MB: 771, 792 and 819 us over the link, 65, 57 and 56 from
// the old cache.
__global__ __launch_bounds__(CP_BLOCK) void sel_wide_copy_kernel(const SelCtrl *__restrict__ ctrl,
                                                                 const unsigned long long *__restrict__ base, int64_t tiles,
                                                                 int64_t num_rows, int64_t num_hot,
                                                                 const int64_t *__restrict__ hot, int unit, RefreshArgs f)
{
    if (!ctrl->wide) return;   // uniform
    const int lane = threadIdx.x & (EMB_WAVE - 1);
    const int64_t wave = (int64_t)blockIdx.x * (CP_BLOCK / EMB_WAVE) + threadIdx.x / EMB_WAVE;
    const int64_t step = (int64_t)gridDim.x * (CP_BLOCK / EMB_WAVE) * unit;
    const uint32_t chunks = (uint32_t)f.chunks;
    const uint32_t items = (uint32_t)unit * chunks;
    for (int64_t k0 = wave * unit; k0 < num_hot; k0 += step) {   // the same for every lane
        uint64_t src = 0ull;
        if (lane < unit && k0 + lane < num_hot) {
            const int64_t row = hot[k0 + lane];
            if (row >= 0 && row < num_rows) {   // always true, as in sel_write_kernel
                const int64_t tile = row / SEL_TILE;
                const uint64_t end = tile + 1 < tiles ? base[tile + 1] : (uint64_t)num_hot;
                if ((end - base[tile]) * chunks > f.tile_chunks) {
                    const int64_t slot = cache_probe(f.old_index, (uint64_t)row, (uint64_t)f.old_num_hot);
                    src = reinterpret_cast<uint64_t>(slot >= 0 ? f.old_rows + slot * (int64_t)chunks * 16
                                                               : f.table + row * (int64_t)chunks * 16);
                }
            }
        }
        if (__ballot(src != 0ull) == 0ull) continue;
        for (uint32_t i0 = 0; i0 < items; i0 += EMB_WAVE * SEL_WIDE_UNROLL) {
            uint4 x[SEL_WIDE_UNROLL];
            bool mine[SEL_WIDE_UNROLL];
#pragma unroll
            for (int u = 0; u < SEL_WIDE_UNROLL; ++u) {
                const uint32_t i = i0 + u * EMB_WAVE + lane;
                const uint32_t k = f.chunk_magic ? __umulhi(i, f.chunk_magic) : i;
                const uint64_t p = (uint64_t)shfl_i64((int64_t)src, (int)(k < (uint32_t)unit ? k : 0u), EMB_WAVE);
                mine[u] = i < items && p != 0ull;
                if (mine[u]) x[u] = load_chunk(reinterpret_cast<const char *>(p) + (int64_t)(i - k * chunks) * 16);
            }
#pragma unroll
            for (int u = 0; u < SEL_WIDE_UNROLL; ++u)
                if (mine[u])
                    *reinterpret_cast<uint4 *>(f.new_rows + (k0 * chunks + i0 + u * EMB_WAVE + lane) * 16) = x[u];
        }
    }
}

// Aging alone (a refresh that keeps no rows).
__global__ __launch_bounds__(CP_BLOCK) void sel_age_kernel(uint32_t *freq, int64_t num_rows, int decay_shift)
{
    const int64_t r0 = (int64_t)blockIdx.x * SEL_TILE + (int64_t)threadIdx.x * SEL_PER_THREAD;
    for (int i = 0; i < SEL_PER_THREAD; ++i)
        if (r0 + i < num_rows) freq[r0 + i] >>= decay_shift;
}

int observe_entry(int64_t num_rows, const int64_t *ids, int64_t nnz, uint32_t *freq_dev, uint32_t *status_dev, void *stream,
                  bool hashed, uint64_t salt)
{
    if (num_rows <= 0 || nnz < 0) return EMB_ERR_INVALID_ARG;
    if (nnz == 0) return EMB_OK;
    if (!ids || !freq_dev) return EMB_ERR_INVALID_ARG;
    const int64_t blocks = (nnz + OBS_TILE - 1) / OBS_TILE;
    if (blocks > 0x7FFFFFFF) return EMB_ERR_UNSUPPORTED;
    const uint64_t magic = emb_mod_magic((uint64_t)num_rows);
    const bool narrow = (uint64_t)num_rows <= 0xFFFFFFFFull;   // row numbers below 2^32 - 1
    hipStream_t s = emb_stream(stream);
#define EMB_OBS(HASHED, SlotT)                                                                                  \
    hipLaunchKernelGGL((cache_observe_kernel<HASHED, SlotT>), dim3((unsigned)blocks), dim3(OBS_BLOCK), 0, s, ids, nnz, \
                       (uint64_t)num_rows, salt, magic, freq_dev, status_dev)
    if (hashed) {
        if (narrow) EMB_OBS(true, uint32_t); else EMB_OBS(true, unsigned long long);
    } else {
        if (narrow) EMB_OBS(false, uint32_t); else EMB_OBS(false, unsigned long long);
    }
#undef EMB_OBS
    EMB_RETURN_IF_LAUNCH_FAILED();
    return EMB_OK;
}

}  // namespace

extern "C" int emb_cache_observe(int64_t num_rows, const int64_t *rows_dev, int64_t nnz, uint32_t *freq_dev,
                                 uint32_t *status_dev, void *stream)
{
    return observe_entry(num_rows, rows_dev, nnz, freq_dev, status_dev, stream, false, 0);
}

extern "C" int emb_cache_observe_hashed(int64_t num_rows, uint64_t salt, const uint64_t *raw_dev, int64_t nnz,
                                        uint32_t *freq_dev, uint32_t *status_dev, void *stream)
{
    return observe_entry(num_rows, reinterpret_cast<const int64_t *>(raw_dev), nnz, freq_dev, status_dev, stream, true,
                         salt);
}

extern "C" int emb_cache_select_workspace_bytes(int64_t num_rows, size_t *bytes)
{
    if (num_rows <= 0 || !bytes) return EMB_ERR_INVALID_ARG;
    *bytes = sel_layout(num_rows).total;
    return EMB_OK;
}

namespace {

// The launches of a selection over counters freq_dev, with the scratch memory at `ws` (laid out by
// sel_layout, at least that large, 256-byte aligned).  Nothing in `ws` has to be zero on entry:
// sel_init_kernel clears the histograms and the group words, every other word is written before it is
// read.  refresh (nullable): the last pass makes the cache too.
int select_run(uint32_t *freq_dev, int64_t num_rows, int64_t num_hot, int32_t decay_shift, const SelLayout &L, char *ws,
               int64_t *hot_rows_out_dev, uint64_t *info_out_dev, hipStream_t s, const RefreshArgs *refresh = nullptr)
{
    if (num_hot == 0) {   // with nothing to take there is no threshold: the counters only age
        if (decay_shift > 0) {
            hipLaunchKernelGGL(sel_age_kernel, dim3((unsigned)L.tiles), dim3(CP_BLOCK), 0, s, freq_dev, num_rows,
                               (int)decay_shift);
            EMB_RETURN_IF_LAUNCH_FAILED();
        }
        return EMB_OK;
    }
    SelCtrl *ctrl = reinterpret_cast<SelCtrl *>(ws + L.ctrl);
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(ws + L.hist);
    unsigned long long *base = reinterpret_cast<unsigned long long *>(ws + L.base);
    uint32_t *counts = reinterpret_cast<uint32_t *>(ws + L.counts);
    uint32_t *ties = reinterpret_cast<uint32_t *>(ws + L.ties);
    unsigned long long *digit[3];
    for (int i = 0; i < 3; ++i) digit[i] = hist + (size_t)(SEL_REPLICAS + i) * SEL_BINS;

    const int words = SEL_HIST_WORDS + SEL_GROUPS;
    hipLaunchKernelGGL(sel_init_kernel, dim3((words + CP_BLOCK - 1) / CP_BLOCK), dim3(CP_BLOCK), 0, s, hist, words);
    EMB_RETURN_IF_LAUNCH_FAILED();
    const int64_t want = ((num_rows + 3) / 4 + SEL_BLOCK - 1) / SEL_BLOCK;
    const dim3 hgrid((unsigned)(want < SEL_HIST_BLOCKS ? want : SEL_HIST_BLOCKS));
    hipLaunchKernelGGL(sel_values_kernel, hgrid, dim3(SEL_BLOCK), 0, s, freq_dev, num_rows, hist);
    EMB_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(sel_pick_kernel, dim3(1), dim3(SEL_BLOCK), 0, s, hist, num_hot, ctrl);
    EMB_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(sel_digit_kernel<1>, hgrid, dim3(SEL_BLOCK), 0, s, freq_dev, num_rows, ctrl,
                       (const unsigned long long *)nullptr, digit[0]);
    EMB_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(sel_digit_kernel<2>, hgrid, dim3(SEL_BLOCK), 0, s, freq_dev, num_rows, ctrl, digit[0], digit[1]);
    EMB_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(sel_digit_kernel<3>, hgrid, dim3(SEL_BLOCK), 0, s, freq_dev, num_rows, ctrl, digit[1], digit[2]);
    EMB_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(sel_count_kernel, dim3((unsigned)L.tiles), dim3(CP_BLOCK), 0, s, freq_dev, num_rows, ctrl, digit[2],
                       counts);
    EMB_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(sel_scan_kernel, dim3(1), dim3(SEL_BLOCK), 0, s, counts, L.tiles, ctrl, base, ties,
                       info_out_dev);
    EMB_RETURN_IF_LAUNCH_FAILED();
    if (refresh) {
        RefreshArgs f = *refresh;
        f.groups = reinterpret_cast<unsigned long long *>(ws + L.groups);
        f.wide = &ctrl->wide;
        hipLaunchKernelGGL(sel_write_kernel<true>, dim3((unsigned)L.tiles), dim3(CP_BLOCK), 0, s, freq_dev, num_rows, ctrl,
                           base, ties, num_hot, (int)decay_shift, hot_rows_out_dev, f);
        // only where the rows chosen from one tile can be so many
        if ((num_hot < SEL_TILE ? num_hot : SEL_TILE) * f.chunks > (int64_t)f.tile_chunks) {
            EMB_RETURN_IF_LAUNCH_FAILED();
            int unit = SEL_WIDE_CHUNKS / f.chunks;
            unit = unit < 1 ? 1 : (unit > EMB_WAVE ? EMB_WAVE : unit);
            const int64_t per_block = (int64_t)unit * (CP_BLOCK / EMB_WAVE);
            const int64_t blocks = (num_hot + per_block - 1) / per_block;
            hipLaunchKernelGGL(sel_wide_copy_kernel, dim3((unsigned)(blocks < SEL_WIDE_GRID ? blocks : SEL_WIDE_GRID)),
                               dim3(CP_BLOCK), 0, s, ctrl, base, L.tiles, num_rows, num_hot, hot_rows_out_dev, unit, f);
        }
    } else {
        hipLaunchKernelGGL(sel_write_kernel<false>, dim3((unsigned)L.tiles), dim3(CP_BLOCK), 0, s, freq_dev, num_rows, ctrl,
                           base, ties, num_hot, (int)decay_shift, hot_rows_out_dev, RefreshArgs{});
    }
    EMB_RETURN_IF_LAUNCH_FAILED();
    return EMB_OK;
}

int select_check(const uint32_t *freq_dev, int64_t num_rows, int64_t num_hot, int32_t decay_shift,
                 const int64_t *hot_rows_out_dev)
{
    if (num_rows <= 0 || num_hot < 0 || num_hot > num_rows || decay_shift < 0 || decay_shift > 31)
        return EMB_ERR_INVALID_ARG;
    if (!freq_dev || !emb_aligned(freq_dev, 16) || (num_hot > 0 && !hot_rows_out_dev)) return EMB_ERR_INVALID_ARG;
    return EMB_OK;
}

}  // namespace

extern "C" int emb_cache_select(uint32_t *freq_dev, int64_t num_rows, int64_t num_hot, int32_t decay_shift,
                                void *workspace_dev, size_t workspace_bytes, int64_t *hot_rows_out_dev,
                                uint64_t *info_out_dev, void *stream)
{
    const int rc = select_check(freq_dev, num_rows, num_hot, decay_shift, hot_rows_out_dev);
    if (rc != EMB_OK) return rc;
    const SelLayout L = sel_layout(num_rows);
    if (L.tiles > 0x7FFFFFFF) return EMB_ERR_UNSUPPORTED;
    if (!workspace_dev || !emb_aligned(workspace_dev, 256) || workspace_bytes < L.total) return EMB_ERR_WORKSPACE;
    return select_run(freq_dev, num_rows, num_hot, decay_shift, L, reinterpret_cast<char *>(workspace_dev),
                      hot_rows_out_dev, info_out_dev, emb_stream(stream));
}

extern "C" int emb_cache_refresh(uint32_t *freq_dev, int64_t num_rows, int64_t num_hot, int32_t decay_shift,
                                 void *workspace_dev, size_t workspace_bytes, const void *table_dev, int32_t D,
                                 int32_t dtype, const void *old_cache_rows_dev, const void *old_cache_index_dev,
                                 int64_t old_num_hot, int64_t *hot_rows_out_dev, void *cache_rows_dev,
                                 void *cache_index_dev, uint64_t *moved_dev, uint64_t *info_out_dev, uint32_t *status_dev,
                                 void *stream)
{
    int rc = select_check(freq_dev, num_rows, num_hot, decay_shift, hot_rows_out_dev);
    if (rc != EMB_OK) return rc;
    if (!old_cache_index_dev) return EMB_ERR_INVALID_ARG;
    rc = emb_check_cache_build(table_dev, num_rows, D, dtype, old_cache_rows_dev, old_cache_index_dev, old_num_hot,
                               hot_rows_out_dev, num_hot, cache_rows_dev, cache_index_dev);
    if (rc != EMB_OK) return rc;
    const SelLayout L = sel_layout(num_rows);
    if (L.tiles > 0x7FFFFFFF) return EMB_ERR_UNSUPPORTED;
    if (!workspace_dev || !emb_aligned(workspace_dev, 256) || workspace_bytes < L.total) return EMB_ERR_WORKSPACE;
    const int64_t row_bytes = emb_row_bytes(D, dtype);
    RefreshArgs f;
    f.table = static_cast<const char *>(table_dev);
    f.old_rows = static_cast<const char *>(old_cache_rows_dev);
    f.old_index = static_cast<const CacheEntry *>(old_cache_index_dev);
    f.old_num_hot = old_num_hot;
    f.new_rows = static_cast<char *>(cache_rows_dev);
    f.new_index = static_cast<CacheEntry *>(cache_index_dev);
    f.chunks = (int32_t)(row_bytes / 16);   // rows of every storage type are whole 16-byte chunks
    f.chunk_magic = f.chunks == 1 ? 0u : (uint32_t)((UINT64_C(1) << 32) / (uint32_t)f.chunks) + 1u;
    f.moved = reinterpret_cast<unsigned long long *>(moved_dev);
    const int64_t share = num_hot * f.chunks / SEL_TILE_SHARE;
    const int64_t limit = share < SEL_TILE_CHUNKS ? SEL_TILE_CHUNKS : share;
    f.tile_chunks = (uint32_t)(limit < 0xFFFFFFFFll ? limit : 0xFFFFFFFFll);   // (no tile holds 2^32)
    f.groups = nullptr;   // these two: select_run
    f.wide = nullptr;
    rc = select_run(freq_dev, num_rows, num_hot, decay_shift, L, static_cast<char *>(workspace_dev), hot_rows_out_dev,
                    info_out_dev, emb_stream(stream), &f);
    if (rc != EMB_OK || num_hot > 0) return rc;
    // an empty cache: the index alone
    return emb_cache_rebuild(table_dev, num_rows, D, dtype, old_cache_rows_dev, old_cache_index_dev, old_num_hot,
                             hot_rows_out_dev, 0, cache_rows_dev, cache_index_dev, moved_dev, status_dev, stream);
}

// ---------------------------------------------------------------------------
// the selection for callers that cannot allocate
// ---------------------------------------------------------------------------
// The scratch memory of emb_cache_select_static: one array per device, part of the
// loaded code object, held until the process ends.  In host code the name `scratch`
// is only a handle for hipGetSymbolAddress: the device address it stands for on a
// given device is looked up once per device (sel_static_address) and that address,
// never the name, is what the kernels are given.
constexpr size_t SEL_STATIC_BYTES = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[SEL_STATIC_BYTES];

namespace {

constexpr int SEL_MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
char *g_scratch_ptr[SEL_MAX_DEVICES];   // by device ordinal; null until that device's first call

// Device address of `scratch` on the current device; null if the runtime refuses.
char *sel_static_address()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= SEL_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        g_scratch_ptr[dev] = reinterpret_cast<char *>(p);
    }
    return g_scratch_ptr[dev];
}

}  // namespace

static_assert(EMB_CACHE_SELECT_STATIC_MAX_ROWS / SEL_TILE + 1 <=
                  (SEL_STATIC_BYTES - 256 - 8 * (SEL_HIST_WORDS + SEL_GROUPS) - 3 * 256) / 16,
              "the static scratch array holds the selection's tile tables up to the stated maximum");

extern "C" int emb_cache_select_static(uint32_t *freq_dev, int64_t num_rows, int64_t num_hot, int32_t decay_shift,
                                       int64_t *hot_rows_out_dev, uint64_t *info_out_dev, void *stream)
{
    const int rc = select_check(freq_dev, num_rows, num_hot, decay_shift, hot_rows_out_dev);
    if (rc != EMB_OK) return rc;
    if (num_rows > EMB_CACHE_SELECT_STATIC_MAX_ROWS) return EMB_ERR_UNSUPPORTED;   // beyond the scratch array
    const SelLayout L = sel_layout(num_rows);
    if (L.total > SEL_STATIC_BYTES) return EMB_ERR_UNSUPPORTED;
    char *ws = sel_static_address();
    if (!ws) return EMB_ERR_HIP;
    return select_run(freq_dev, num_rows, num_hot, decay_shift, L, ws, hot_rows_out_dev, info_out_dev,
                      emb_stream(stream));
}
