// Device helpers shared by the gather-pool kernels: 16-byte row chunks of fp32
// or bf16 rows, accumulated in fp32.
#pragma once
#include <type_traits>

#include "emb_internal.h"
#include "scan.h"
#include "u64mod.h"

// Per-lane accumulator for one 16-byte chunk of a row.
template <bool BF16>
struct ChunkAcc;

template <>
struct ChunkAcc<false> {
    static constexpr int FLOATS = 4;
    float a[4];
    __device__ __forceinline__ void zero() { a[0] = a[1] = a[2] = a[3] = 0.f; }
    __device__ __forceinline__ void add(const uint4 &v)
    {
        a[0] += __uint_as_float(v.x);
        a[1] += __uint_as_float(v.y);
        a[2] += __uint_as_float(v.z);
        a[3] += __uint_as_float(v.w);
    }
};

template <>
struct ChunkAcc<true> {
    static constexpr int FLOATS = 8;
    float a[8];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = 0.f;
    }
    // a bf16 value is the high half of an fp32: widening is a shift / a mask
    __device__ __forceinline__ void add(const uint4 &v)
    {
        a[0] += __uint_as_float(v.x << 16);
        a[1] += __uint_as_float(v.x & 0xFFFF0000u);
        a[2] += __uint_as_float(v.y << 16);
        a[3] += __uint_as_float(v.y & 0xFFFF0000u);
        a[4] += __uint_as_float(v.z << 16);
        a[5] += __uint_as_float(v.z & 0xFFFF0000u);
        a[6] += __uint_as_float(v.w << 16);
        a[7] += __uint_as_float(v.w & 0xFFFF0000u);
    }
};

// Table rows, accumulators and gradients live in device (or mapped host) memory, never in LDS: the
// accesses below say so (global address space), so that they are not generic ("flat") operations,
// which count against both the memory and the LDS counters of a wavefront and make waits on one
// wait for the other.
#define EMB_GLOBAL __attribute__((address_space(1)))
typedef uint32_t emb_u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_chunk(const char *p)
{
    const emb_u4 v = *(const EMB_GLOBAL emb_u4 *)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Streaming variants for data that is touched once (the rows and accumulators the update
// rewrites): they are marked non-temporal so that they do not push reusable lines (hot
// rows, gradient rows) out of L2 and the memory-side cache.
__device__ __forceinline__ uint4 load_chunk_nt(const char *p)
{
    const emb_u4 v = __builtin_nontemporal_load((const EMB_GLOBAL emb_u4 *)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float load_f32_nt(const float *p) { return __builtin_nontemporal_load((const EMB_GLOBAL float *)p); }
__device__ __forceinline__ void store_f32_nt(float *p, float v) { __builtin_nontemporal_store(v, (EMB_GLOBAL float *)p); }
__device__ __forceinline__ void store_chunk_nt(char *p, const uint4 &x)
{
    emb_u4 v;
    v.x = x.x; v.y = x.y; v.z = x.z; v.w = x.w;
    __builtin_nontemporal_store(v, (EMB_GLOBAL emb_u4 *)p);
}


__device__ __forceinline__ int64_t shfl_i64(int64_t v, int src, int width)
{
    int lo = __shfl((int)(uint32_t)(uint64_t)v, src, width);
    int hi = __shfl((int)(uint32_t)((uint64_t)v >> 32), src, width);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// The value that lane k of every group of LPR lanes holds, in all lanes of the group (up to 16 lanes k is a
// constant once the caller's loop is unrolled).  Inside 16 lanes this is a data-parallel move of the vector
// unit, which neither waits for nor loads the LDS pipe that a general lane shuffle goes through.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_upper_half(uint32_t low, uint32_t v)   // lanes 8..15 of every 16 move, the others keep low
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)low, (int)v, CTRL, 0xF, 0xC, false);
}
template <int LPR>
__device__ __forceinline__ uint32_t group_bcast(uint32_t v, int k)
{
    if constexpr (LPR == 1) return v;
    if constexpr (LPR == 2) return k == 0 ? dpp_move<0xA0>(v) : dpp_move<0xF5>(v);   // quad_perm
    if constexpr (LPR == 4) {
        switch (k) {   // quad_perm [k, k, k, k]
            case 0: return dpp_move<0x00>(v);
            case 1: return dpp_move<0x55>(v);
            case 2: return dpp_move<0xAA>(v);
            default: return dpp_move<0xFF>(v);
        }
    }
#define EMB_BC8(K) dpp_upper_half<0x158 + K>(dpp_move<0x150 + K>(v), v)   // row_newbcast, one for each half of a row
    if constexpr (LPR == 8) {
        switch (k) {
            case 0: return EMB_BC8(0);
            case 1: return EMB_BC8(1);
            case 2: return EMB_BC8(2);
            case 3: return EMB_BC8(3);
            case 4: return EMB_BC8(4);
            case 5: return EMB_BC8(5);
            case 6: return EMB_BC8(6);
            default: return EMB_BC8(7);
        }
    }
#undef EMB_BC8
#define EMB_BC16(K) case K: return dpp_move<0x150 + K>(v)   // row_newbcast
    if constexpr (LPR == 16) {
        switch (k) {
            EMB_BC16(0); EMB_BC16(1); EMB_BC16(2); EMB_BC16(3); EMB_BC16(4); EMB_BC16(5); EMB_BC16(6); EMB_BC16(7);
            EMB_BC16(8); EMB_BC16(9); EMB_BC16(10); EMB_BC16(11); EMB_BC16(12); EMB_BC16(13); EMB_BC16(14);
            default: return dpp_move<0x15F>(v);
        }
    }
#undef EMB_BC16
    if constexpr (LPR == 32) return (uint32_t)__shfl((int)v, k, LPR);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, k);   // the whole wavefront: a scalar
}
template <int LPR>
__device__ __forceinline__ const char *group_bcast_ptr(uint64_t p, int k)
{
    const uint32_t lo = group_bcast<LPR>((uint32_t)p, k), hi = group_bcast<LPR>((uint32_t)(p >> 32), k);
    return reinterpret_cast<const char *>(((uint64_t)hi << 32) | lo);
}

// A row of zeros as long as the largest row: what an entry that is skipped reads, so that the row loads need
// no test of their own (adding +0 to a sum that started at +0 changes no bit).
static __device__ uint4 emb_zero_row[1024];

// Bounds of bag `bag` (clamped to bag 0 where the caller's lane group has no bag) from offsets kept in two
// levels: `local` holds the sums of the bag lengths within tiles of EMB_OFFSETS_TILE lengths
// (emb_offsets_tile_sums), the tile totals standing at the tile ends; the prefix sums of the totals are
// taken here.  Up to 64 tiles every wavefront does that by itself: lane k loads tile k's total together
// with the loads of its bag's own two sums, one scan over the wavefront, and the two prefixes a bag needs
// come by lane shuffles (no LDS, no barrier).  Up to BLOCK tiles the workgroup scans the totals in LDS
// (tile_prefix: BLOCK entries, wave_sums: BLOCK / 64).  Every thread of the workgroup calls this.
template <int BLOCK>
__device__ __forceinline__ void emb_two_level_bounds(const int64_t *__restrict__ local, int64_t n_bags, bool live,
                                                     int64_t bag, int64_t *tile_prefix, int64_t *wave_sums,
                                                     int64_t &s, int64_t &e)
{
    const int64_t n_tiles = (n_bags + EMB_OFFSETS_TILE - 1) / EMB_OFFSETS_TILE;   // <= BLOCK (checked by the host)
    const int64_t bc = live ? bag : 0;
    const int64_t ts = (bc > 0 ? bc - 1 : 0) / EMB_OFFSETS_TILE, te = bc / EMB_OFFSETS_TILE;
    int64_t ps, pe;
    if (n_tiles <= EMB_WAVE) {   // uniform
        const int lane = threadIdx.x & (EMB_WAVE - 1);
        int64_t end = (int64_t)(lane + 1) * EMB_OFFSETS_TILE;
        if (end > n_bags) end = n_bags;
        const int64_t total = lane < n_tiles ? local[end] : 0;
        const int64_t a0 = local[bc], a1 = local[bc + 1];
        const int64_t prefix = wave_inclusive_scan(total) - total;
        ps = shfl_i64(prefix, (int)ts, EMB_WAVE);
        pe = shfl_i64(prefix, (int)te, EMB_WAVE);
        s = a0 + (bc > 0 ? ps : 0);
        e = a1 + pe;
        return;
    }
    const int64_t k = threadIdx.x;
    int64_t end = (k + 1) * EMB_OFFSETS_TILE;
    if (end > n_bags) end = n_bags;
    const int64_t v = k < n_tiles ? local[end] : 0;
    const int64_t a0 = local[bc], a1 = local[bc + 1];
    int64_t total;
    const int64_t inc = block_inclusive_scan<int64_t, BLOCK>(v, wave_sums, total);
    tile_prefix[k] = inc - v;
    __syncthreads();
    ps = tile_prefix[ts];
    pe = tile_prefix[te];
    s = a0 + (bc > 0 ? ps : 0);
    e = a1 + pe;
}

// Bounds of the workgroup's bags straight from the bag lengths, for batches of up to EMB_LENGTHS_DIRECT_BAGS
// bags: every workgroup adds up the lengths before its first bag itself (at most 16 KB, from the L2), which
// saves the launch that would make sums within tiles (about 3 us of a call in a full queue).  The reads grow with
// the square of the number of bags, and with the row width (up to 4 bags a workgroup).  Calls in us, lengths here /
// sums within tiles, one fixed-length table of fp32 rows, bags of 1: 4096 bags 7.5 / 9.4 (D = 16), 7.6 / 10.6 (64),
// 7.4 / 10.6 (256), 9.8 / 13.1 (1024); 8192 bags 7.4 / 9.5, 7.7 / 10.6, 10.1 / 11.1, 16.6 / 19.2; 16 384 bags 7.5 / 9.4,
// 8.7 / 10.5, 22.6 / 14.8, 33.4 / 28.0.  The line is the last size at which the widest rows lose nothing of the gain.
// first: the workgroup's first bag; bags: how many it has (at most BLOCK / LPR); g: the calling thread's.  Every thread
// of the workgroup calls this.
constexpr int64_t EMB_LENGTHS_DIRECT_BAGS = 4096;
template <int BLOCK, int GROUPS>
__device__ __forceinline__ void emb_bounds_from_lengths(const int32_t *__restrict__ lengths, int64_t first, int bags, int g,
                                                        int64_t *own /*LDS [GROUPS + 1]*/,
                                                        int64_t *wave_sums /*LDS [2 * BLOCK / 64]*/, uint32_t *status,
                                                        int64_t &s, int64_t &e)
{
    constexpr int WAVES = BLOCK / EMB_WAVE;
    constexpr int UNROLL = 8;
    const int tid = threadIdx.x, lane = tid & (EMB_WAVE - 1), wave = tid / EMB_WAVE;
    int64_t before = 0, mine = 0;
    bool bad = false;
    if (tid < bags) mine = lengths[first + tid];
    for (int64_t i0 = tid; i0 < first; i0 += BLOCK * UNROLL) {
        int32_t v[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) v[u] = i0 + u * BLOCK < first ? lengths[i0 + u * BLOCK] : 0;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            bad |= v[u] < 0;
            before += v[u] < 0 ? 0 : v[u];
        }
    }
    if (mine < 0) {
        bad = true;
        mine = 0;
    }
    if (bad) emb_flag(status, EMB_STATUS_BAD_OFFSETS);
    before = wave_inclusive_scan(before);   // (the last lane has the sum)
    int64_t inc = mine;
    if (wave * EMB_WAVE < GROUPS) inc = wave_inclusive_scan(mine);   // uniform over the wavefront
    if (lane == EMB_WAVE - 1) {
        wave_sums[wave] = before;
        wave_sums[WAVES + wave] = inc;
    }
    __syncthreads();
    int64_t base = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        base += wave_sums[w];
        if (w < wave) inc += wave_sums[WAVES + w];
    }
    if (tid < GROUPS) own[tid + 1] = base + inc;
    if (tid == 0) own[0] = base;
    __syncthreads();
    s = own[g];
    e = own[g + 1];
}

// Lanes per row (a power of two <= 64) and chunks per lane for a row of
// `chunks` 16-byte chunks.
static inline void emb_row_split(int chunks, int &lpr, int &cpl)
{
    lpr = 1;
    while (lpr < chunks && lpr < 64) lpr <<= 1;
    int need = (chunks + lpr - 1) / lpr;
    cpl = 1;
    while (cpl < need) cpl <<= 1;
}

// ---------------------------------------------------------------------------
// The gather-pool loop shared by the plain and the cached pooled lookup.
//
// A row of chunks_per_row 16-byte chunks is covered by LPR lanes (CPL chunks
// per lane when a row is wider than a wavefront).  Each group of LPR lanes owns
// one bag and walks its lookups UNROLL rows at a time, issuing all UNROLL row
// loads before the first add, so a wavefront keeps 64/LPR * UNROLL independent
// row reads in flight.  The group's lanes fetch the bag's row indices with one
// coalesced load; the lane that fetched an index resolves it to the address of
// the row (Source::resolve: bounds check, and for the cached table the cache
// probe) and the address is handed round (group_bcast), so every index is
// read and resolved exactly once.  No cross-lane reduction is needed: a lane
// only ever adds the chunks it owns.
//
// What bounds it: on narrow rows the instructions around a row load, on wide ones
// the rate of scattered lines.  So a row costs two moves, one address add, the load
// and the adds: entries past the bag's end and skipped ones read a row of zeros,
// lanes past the row read its first chunk and store nothing, and a batch that no
// bag of the wavefront fills is done at half its length (a short bag would pay for
// eight loads otherwise).
//
// Source must provide
//   __device__ uint64_t resolve(int64_t v, int64_t j)   address of the row that entry j of
//                                                       `rows` (value v) selects, 0 = skip it
// ---------------------------------------------------------------------------
// STREAM: the rows are read with non-temporal loads (see EMB_ROWS_STREAMING in the header).
template <int LPR, int CPL, int N, bool BF16, bool STREAM, int IPL>
__device__ __forceinline__ void gather_rows(ChunkAcc<BF16> (&acc)[CPL], const uint64_t (&mine)[IPL], int k0, const uint32_t (&off)[CPL])
{
    uint4 v[N][CPL];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const char *p = group_bcast_ptr<LPR>(mine[IPL == 1 ? 0 : (k0 + i) / LPR], (k0 + i) % LPR);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            if constexpr (STREAM) {
                // the row of zeros is not asked for here: a non-temporal load of it does not stay in the caches
                // (uniform IDs, 16 x 8192 bags of 20 rows of 256 bytes: 134 to 137 us with it, 130 to 134 without)
                v[i][c] = make_uint4(0, 0, 0, 0);
                if (p != reinterpret_cast<const char *>(emb_zero_row)) v[i][c] = load_chunk_nt(p + off[c]);
            } else {
                v[i][c] = load_chunk(p + off[c]);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);   // every load of the batch before its first add
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c].add(v[i][c]);
}

// A Source whose entries are raw IDs: the row is splitmix64(raw XOR salt) mod num_rows (Section 2.2), computed
// by the lane that fetched the ID, so hashing costs no pass of its own.  The row numbers can be
// written out for the backward.
struct HashedTableSource {
    const char *weights;
    uint64_t num_rows, salt, magic;
    int64_t row_bytes;
    int64_t *rows_out;   // nullable
    __device__ __forceinline__ uint64_t resolve(int64_t raw, int64_t j) const
    {
        const uint64_t r = emb_fast_mod(emb_splitmix64((uint64_t)raw ^ salt), num_rows, magic);
        if (rows_out) rows_out[j] = (int64_t)r;
        return reinterpret_cast<uint64_t>(weights + (int64_t)r * row_bytes);
    }
};

// Does `left` entries' worth of a batch of UNROLL at its full length, a half or a quarter: do_rows(n) with n a
// compile-time constant.  The longest of the wavefront's bags decides (uniform).
template <int UNROLL, typename Rows>
__device__ __forceinline__ void gather_batch(int64_t left, const Rows &do_rows)
{
    if constexpr (UNROLL >= 4) {
        if (__ballot(left > UNROLL / 2) != 0) do_rows(std::integral_constant<int, UNROLL>());
        else if (__ballot(left > UNROLL / 4) != 0) do_rows(std::integral_constant<int, UNROLL / 2>());
        else do_rows(std::integral_constant<int, UNROLL / 4>());
    } else {
        do_rows(std::integral_constant<int, UNROLL>());
    }
}

// The bag is given by its bounds: lookups [s, e) of `rows` (ignored unless live).
template <int LPR, int CPL, int UNROLL, bool BF16, bool STREAM = false, typename Source>
__device__ __forceinline__ void gather_pool_range(Source &src, bool live, int64_t s, int64_t e, int l, int64_t nnz,
                                                  const int64_t *__restrict__ rows, int32_t chunks_per_row,
                                                  int32_t mode, float *__restrict__ out_row, uint32_t *status)
{
    // out_row is where the bag's pooled row goes (not touched unless live)
    constexpr int IPL = (UNROLL > LPR) ? UNROLL / LPR : 1;  // indices fetched per lane per batch
    constexpr int IB = IPL * LPR;                           // indices per batch
    static_assert(IB % UNROLL == 0, "index batch must be whole unroll groups");

    if (!live) {
        s = e = 0;
    } else if (s < 0 || e < s || e > nnz) {
        if (l == 0) emb_flag(status, EMB_STATUS_BAD_OFFSETS);
        s = e = 0;
    }

    ChunkAcc<BF16> acc[CPL];
    uint32_t off[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        acc[c].zero();
        off[c] = l + c * LPR < chunks_per_row ? (uint32_t)(l + c * LPR) * 16u : 0u;
    }

    const uint64_t zero_row = reinterpret_cast<uint64_t>(emb_zero_row);
    // the entries of the batch after the current one are asked for before the current one's rows
    int64_t next[IPL];
#pragma unroll
    for (int m = 0; m < IPL; ++m) {
        const int64_t j = s + m * LPR + l;
        next[m] = j < e ? rows[j] : 0;
    }
    for (int64_t base = s; base < e; base += IB) {
        uint64_t mine[IPL];
#pragma unroll
        for (int m = 0; m < IPL; ++m) {
            const int64_t j = base + m * LPR + l;
            mine[m] = 0ull;
            if (j < e) mine[m] = src.resolve(next[m], j);
            if (mine[m] == 0ull) mine[m] = zero_row;
            if (j + IB < e) next[m] = rows[j + IB];
        }
        // (lane numbers of a group of up to 16 must be constants)
#pragma unroll(LPR <= 16 ? IB / UNROLL : 1)
        for (int u = 0; u < IB / UNROLL; ++u) {
            const int64_t left = e - base - u * UNROLL;
            if (left > 0)   // the group's lanes agree
                gather_batch<UNROLL>(left, [&](auto n) {
                    gather_rows<LPR, CPL, decltype(n)::value, BF16, STREAM>(acc, mine, u * UNROLL, off);
                });
        }
    }

    if (!live) return;
    const int64_t len = e - s;
    const bool mean = (mode == EMB_POOL_MEAN) && len > 0;
    const float flen = (float)len;
    constexpr int F = ChunkAcc<BF16>::FLOATS;
    float *obase = out_row;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int chunk = l + c * LPR;
        if (chunk < chunks_per_row) {
            float r[F];
#pragma unroll
            for (int i = 0; i < F; ++i) r[i] = mean ? acc[c].a[i] / flen : acc[c].a[i];
            float4 *o = reinterpret_cast<float4 *>(obase + (int64_t)chunk * F);
#pragma unroll
            for (int i = 0; i < F / 4; ++i) o[i] = make_float4(r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]);
        }
    }
}

// The bag is number `bag` of `offsets`.  tile_prefix: the offsets are sums within tiles and these are the
// tiles' prefix sums (emb_bag_bounds).
template <int LPR, int CPL, int UNROLL, bool BF16, bool STREAM = false, typename Source>
__device__ __forceinline__ void gather_pool_bag(Source &src, bool live, int64_t bag, int l, int64_t nnz,
                                                const int64_t *__restrict__ rows,
                                                const int64_t *__restrict__ offsets, int32_t chunks_per_row,
                                                int32_t mode, float *__restrict__ out_row, uint32_t *status,
                                                const int64_t *__restrict__ tile_prefix = nullptr)
{
    int64_t s = 0, e = 0;
    if (live) emb_bag_bounds(offsets, tile_prefix, bag, s, e);
    gather_pool_range<LPR, CPL, UNROLL, BF16, STREAM>(src, live, s, e, l, nnz, rows, chunks_per_row, mode, out_row,
                                                      status);
}
