// Bag-offset (CSR) builder: exclusive prefix sum of int32 bag lengths into
// int64 offsets, in the output array alone: no scratch memory and no inter-block waiting.
//
// Up to DIRECT_TILES tiles of 4096 lengths (the last may take more), two launches:
//   1. every tile but the last adds its lengths up and leaves the sum in each later tile's part of the output, one
//      entry per sum, where nothing else has been written yet,
//   2. every tile adds up the sums it finds in its part, and then overwrites that part with the offsets.
// One tile (n < 8192) needs the second only.  These launches are shorter than the way from one to the next: 196 608
// lengths take 10.5 us with the three below, 7.8 with these; 1e6 17.6 and 10.4, 4e6 40 and 29.  More tiles than that, three:
//   1. every tile of 4096 lengths writes its local inclusive sums to
//      offsets[i+1] (so the last entry of a tile holds the tile total),
//   2. one block turns the tile totals into global inclusive sums,
//   3. every tile but the first adds the global sum at the end of the tile
//      before it to all its entries except its last.
#include "emb_internal.h"
#include "scan.h"

namespace {

constexpr int SCAN_BLOCK = 1024;
constexpr int SCAN_ITEMS = 4;
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;
static_assert(SCAN_TILE == EMB_OFFSETS_TILE, "callers of emb_offsets_tile_sums index the tile totals by this size");
constexpr int SCAN_WAVES = SCAN_BLOCK / EMB_WAVE;

__global__ __launch_bounds__(SCAN_BLOCK) void offsets_tile_scan_kernel(const int32_t *__restrict__ lengths, int64_t n,
                                                                       int64_t *__restrict__ offsets, uint32_t *status)
{
    __shared__ int64_t wave_sums[SCAN_WAVES];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int64_t v[SCAN_ITEMS];
    bool bad = false;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        int32_t len = (base + k < n) ? lengths[base + k] : 0;
        if (len < 0) {
            bad = true;
            len = 0;
        }
        v[k] = len;
    }
    if (bad) emb_flag(status, EMB_STATUS_BAD_OFFSETS);
    int64_t mine = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        mine += v[k];
        v[k] = mine;
    }
    int64_t total;
    int64_t inc = block_inclusive_scan<int64_t, SCAN_BLOCK>(mine, wave_sums, total);
    int64_t before = inc - mine;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k)
        if (base + k < n) offsets[base + k + 1] = before + v[k];
    if (blockIdx.x == 0 && threadIdx.x == 0) offsets[0] = 0;
}

constexpr int64_t DIRECT_TILES = SCAN_BLOCK;   // a tile has a thread and (more than) an entry for every tile before it

// grid: tiles - 1.  Sum of tile k goes to entry 1 + k of the parts of the tiles after it.
__global__ __launch_bounds__(SCAN_BLOCK) void offsets_tile_sums_kernel(const int32_t *__restrict__ lengths, int64_t tiles,
                                                                       int64_t *__restrict__ offsets)
{
    __shared__ int64_t wave_sums[SCAN_WAVES];
    const int64_t tile = blockIdx.x;
    int64_t mine = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        const int32_t len = lengths[tile * SCAN_TILE + k * SCAN_BLOCK + threadIdx.x];
        mine += len < 0 ? 0 : len;
    }
#pragma unroll
    for (int d = EMB_WAVE >> 1; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, EMB_WAVE);
    if (threadIdx.x % EMB_WAVE == 0) wave_sums[threadIdx.x / EMB_WAVE] = mine;
    __syncthreads();
    int64_t total = 0;
#pragma unroll
    for (int w = 0; w < SCAN_WAVES; ++w) total += wave_sums[w];
    const int64_t later = tile + 1 + threadIdx.x;
    if (later < tiles) offsets[later * SCAN_TILE + 1 + tile] = total;
}

// grid: tiles.
__global__ __launch_bounds__(SCAN_BLOCK) void offsets_tile_write_kernel(const int32_t *__restrict__ lengths, int64_t n,
                                                                        int64_t tiles, int64_t *__restrict__ offsets,
                                                                        uint32_t *status)
{
    __shared__ int64_t wave_sums[SCAN_WAVES];
    const int64_t tile = blockIdx.x, first = tile * SCAN_TILE;
    int64_t carry = 0;
    if (tile > 0) {   // uniform
        int64_t mine = threadIdx.x < tile ? offsets[first + 1 + threadIdx.x] : 0;
#pragma unroll
        for (int d = EMB_WAVE >> 1; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, EMB_WAVE);
        if (threadIdx.x % EMB_WAVE == 0) wave_sums[threadIdx.x / EMB_WAVE] = mine;
        __syncthreads();   // every sum has been read: the part may be overwritten
#pragma unroll
        for (int w = 0; w < SCAN_WAVES; ++w) carry += wave_sums[w];
        __syncthreads();
    }
    const int64_t end = tile + 1 < tiles ? first + SCAN_TILE : n;
    bool bad = false;
    for (int64_t base0 = first; base0 < end; base0 += SCAN_TILE) {   // once, in the last tile perhaps twice
        const int64_t base = base0 + (int64_t)threadIdx.x * SCAN_ITEMS;
        int64_t v[SCAN_ITEMS], mine = 0, total;
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            const int32_t len = base + k < end ? lengths[base + k] : 0;
            bad |= len < 0;
            mine += len < 0 ? 0 : len;
            v[k] = mine;
        }
        const int64_t before = carry + block_inclusive_scan<int64_t, SCAN_BLOCK>(mine, wave_sums, total) - mine;
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k)
            if (base + k < end) offsets[base + k + 1] = before + v[k];
        carry += total;
    }
    if (bad) emb_flag(status, EMB_STATUS_BAD_OFFSETS);
    if (tile == 0 && threadIdx.x == 0) offsets[0] = 0;
}

// Entry "end of tile k" is offsets[min((k+1)*SCAN_TILE, n)].
__device__ __forceinline__ int64_t tile_end(int64_t k, int64_t n)
{
    int64_t e = (k + 1) * SCAN_TILE;
    return e < n ? e : n;
}

__global__ __launch_bounds__(SCAN_BLOCK) void offsets_tile_totals_kernel(int64_t *__restrict__ offsets, int64_t n,
                                                                         int64_t num_tiles)
{
    __shared__ int64_t wave_sums[SCAN_WAVES];
    int64_t carry = 0;
    for (int64_t k0 = 0; k0 < num_tiles; k0 += SCAN_BLOCK) {
        int64_t k = k0 + threadIdx.x;
        int64_t v = k < num_tiles ? offsets[tile_end(k, n)] : 0;
        int64_t total;
        int64_t inc = block_inclusive_scan<int64_t, SCAN_BLOCK>(v, wave_sums, total);
        if (k < num_tiles) offsets[tile_end(k, n)] = carry + inc;
        carry += total;
    }
}

__global__ __launch_bounds__(SCAN_BLOCK) void offsets_add_prefix_kernel(int64_t *__restrict__ offsets, int64_t n)
{
    const int64_t tile = (int64_t)blockIdx.x + 1;                 // tile 0 needs nothing
    const int64_t prefix = offsets[tile * SCAN_TILE];             // global sum at the end of tile-1
    const int64_t last = tile_end(tile, n);                       // already global
    const int64_t base = tile * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        int64_t i = base + k + 1;
        if (i < last) offsets[i] += prefix;
    }
}

}  // namespace

// The first launch alone: sums within tiles (for callers that add the tiles' prefix themselves).
int emb_offsets_tile_sums(const int32_t *lengths_dev, int64_t n, int64_t *local_dev, uint32_t *status_dev, hipStream_t s)
{
    const int64_t tiles = n == 0 ? 1 : (n + SCAN_TILE - 1) / SCAN_TILE;
    if (tiles > 0x7FFFFFFF) return EMB_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(offsets_tile_scan_kernel, dim3((unsigned)tiles), dim3(SCAN_BLOCK), 0, s, lengths_dev, n, local_dev,
                       status_dev);
    EMB_RETURN_IF_LAUNCH_FAILED();
    return EMB_OK;
}

extern "C" int emb_lengths_to_offsets(const int32_t *lengths_dev, int64_t n, int64_t *offsets_dev,
                                      uint32_t *status_dev, void *stream)
{
    if (n < 0 || !offsets_dev || (n > 0 && !lengths_dev)) return EMB_ERR_INVALID_ARG;
    int64_t tiles = n == 0 ? 1 : (n + SCAN_TILE - 1) / SCAN_TILE;
    if (tiles > 0x7FFFFFFF) return EMB_ERR_UNSUPPORTED;
    hipStream_t s = emb_stream(stream);
    // whole tiles; what is left is a tile of its own if it has an entry for each tile before it, else the last one's
    // (and up to 8191 lengths are one tile and one launch: 4097 lengths 9.0 us with three, 4.7 with one, 8000 9.1 and 6.2)
    int64_t parts = n < SCAN_TILE ? 1 : n / SCAN_TILE;
    if (parts > 1 && n - parts * SCAN_TILE >= parts) ++parts;
    if (parts <= DIRECT_TILES) {
        if (parts > 1) {
            hipLaunchKernelGGL(offsets_tile_sums_kernel, dim3((unsigned)(parts - 1)), dim3(SCAN_BLOCK), 0, s, lengths_dev, parts,
                               offsets_dev);
            EMB_RETURN_IF_LAUNCH_FAILED();
        }
        hipLaunchKernelGGL(offsets_tile_write_kernel, dim3((unsigned)parts), dim3(SCAN_BLOCK), 0, s, lengths_dev, n, parts,
                           offsets_dev, status_dev);
        EMB_RETURN_IF_LAUNCH_FAILED();
        return EMB_OK;
    }
    hipLaunchKernelGGL(offsets_tile_scan_kernel, dim3((unsigned)tiles), dim3(SCAN_BLOCK), 0, s, lengths_dev, n,
                       offsets_dev, status_dev);
    EMB_RETURN_IF_LAUNCH_FAILED();
    if (tiles > 1) {
        hipLaunchKernelGGL(offsets_tile_totals_kernel, dim3(1), dim3(SCAN_BLOCK), 0, s, offsets_dev, n, tiles);
        EMB_RETURN_IF_LAUNCH_FAILED();
        hipLaunchKernelGGL(offsets_add_prefix_kernel, dim3((unsigned)(tiles - 1)), dim3(SCAN_BLOCK), 0, s,
                           offsets_dev, n);
        EMB_RETURN_IF_LAUNCH_FAILED();
    }
    return EMB_OK;
}
