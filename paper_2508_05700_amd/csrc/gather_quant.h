// Device code of the pooled lookup over row-quantised tables (storage described
// in quant.hip), shared by the plain and the cached lookup.
#pragma once
#include "emb_internal.h"
#include "gather.h"

constexpr int Q_ELEMS = 16;   // elements per lane
constexpr int Q_BLOCK = 256;

typedef uint32_t emb_u2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint2 load_u2(const char *p)   // rows are in device (or mapped host) memory
{
    const emb_u2 v = *(const EMB_GLOBAL emb_u2 *)p;
    return make_uint2(v.x, v.y);
}

// 16 bytes of an INT4 row, from a lane's place on: lanes are 8 bytes apart, so every other address is a multiple of 8 only.
// (Still one request: the vector unit loads 16 bytes from any multiple of 4.)
constexpr int Q4_LANE_BYTES = Q_ELEMS / 2;
typedef uint32_t emb_u4_codes __attribute__((ext_vector_type(4), aligned(8)));
static_assert(Q4_LANE_BYTES % alignof(emb_u4_codes) == 0, "the type promises no more than a lane's address keeps");
__device__ __forceinline__ uint4 load_codes(const char *p)
{
    const emb_u4_codes v = *(const EMB_GLOBAL emb_u4_codes *)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// 16 codes of a lane -> fp32.  INT4: masking every other nibble leaves one code per
// byte, which converts with the byte-to-float instructions.
template <int BITS>
__device__ __forceinline__ void codes_to_float(const uint32_t (&w)[BITS == 8 ? 4 : 2], float (&f)[Q_ELEMS])
{
    if (BITS == 8) {
#pragma unroll
        for (int i = 0; i < Q_ELEMS; ++i) f[i] = (float)((w[i / 4] >> (8 * (i % 4))) & 0xFFu);
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t even = w[h] & 0x0F0F0F0Fu, odd = (w[h] >> 4) & 0x0F0F0F0Fu;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f[8 * h + 2 * i] = (float)((even >> (8 * i)) & 0xFFu);
                f[8 * h + 2 * i + 1] = (float)((odd >> (8 * i)) & 0xFFu);
            }
        }
    }
}

// N rows of a group's batch, from entry k0 on.  INT4: a lane asks for 16 bytes, its own 8
// of codes and the 8 before them, which for the first lane are the header; that is handed round by
// data-parallel moves.  One request instead of two a row: 2.6e6 lookups of 48-byte rows 68.7 -> 67.3 us (handing the
// codes round as well, by shuffles through LDS, lost 10).  INT8: the 8-byte header, one request
// for the group, and the lane's 16 code bytes.  Each element
// is dequantised (one fused multiply-add) and then added, so the rounding behaviour
// is that of summing fp32 rows; a row of zeros has scale and bias 0.
template <int LPR, int BITS, int N, int IPL>
__device__ __forceinline__ void gather_dequant_rows(float (&acc)[Q_ELEMS], const uint64_t (&mine)[IPL], int k0, uint32_t code_off)
{
    constexpr int CW = BITS == 8 ? 4 : 2;                   // code words per lane and row
    uint2 hdr[N];
    uint32_t w[N][CW];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const char *row = group_bcast_ptr<LPR>(mine[IPL == 1 ? 0 : (k0 + i) / LPR], (k0 + i) % LPR);
        if (BITS == 4) {
            const uint4 v = load_codes(row + code_off - Q4_LANE_BYTES);
            hdr[i] = make_uint2(v.x, v.y);
            w[i][0] = v.z;
            w[i][1] = v.w;
        } else {
            hdr[i] = load_u2(row);
            const uint2 c0 = load_u2(row + code_off), c1 = load_u2(row + code_off + 8);
            w[i][0] = c0.x;
            w[i][1] = c0.y;
            w[i][CW - 2] = c1.x;
            w[i][CW - 1] = c1.y;
        }
    }
    __builtin_amdgcn_sched_barrier(0);   // every load of the batch before its first add
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (BITS == 4) hdr[i] = make_uint2(group_bcast<LPR>(hdr[i].x, 0), group_bcast<LPR>(hdr[i].y, 0));
        const float scale = __uint_as_float(hdr[i].x), bias = __uint_as_float(hdr[i].y);
        float f[Q_ELEMS];
        codes_to_float<BITS>(w[i], f);
#pragma unroll
        for (int x = 0; x < Q_ELEMS; ++x) acc[x] += __builtin_fmaf(scale, f[x], bias);
    }
}

// The loop has the shape of gather_pool_range (gather.h): a group of LPR lanes owns a
// bag, fetches its indices with one coalesced load (the next batch's ahead of the
// current one's rows), the fetching lane resolves an index to the row's address
// (Source::resolve, 0 = skip: a row of zeros), addresses are handed round, UNROLL
// rows are requested before the first add.  `bag` indexes offsets and out.
// The bag is given by its bounds: lookups [s, e) of `rows` (ignored unless live).
template <int LPR, int BITS, int UNROLL, typename Source>
__device__ __forceinline__ void gather_dequant_pool_range(Source &src, bool live, int64_t bag, int64_t s, int64_t e, int l,
                                                          int64_t nnz, const int64_t *__restrict__ rows, int32_t D,
                                                          int32_t mode, float *__restrict__ out, uint32_t *status)
{
    constexpr int IPL = (UNROLL > LPR) ? UNROLL / LPR : 1;  // indices fetched per lane per batch
    constexpr int IB = IPL * LPR;                           // indices per batch
    static_assert(IB % UNROLL == 0, "index batch must be whole unroll groups");
    const bool mine_elems = l * Q_ELEMS < D;         // lanes past the row (D/16 not a power of two) read its first codes
    const uint32_t code_off = 8u + (mine_elems ? (uint32_t)l * (BITS == 8 ? 16u : (uint32_t)Q4_LANE_BYTES) : 0u);

    if (!live) {
        s = e = 0;
    } else if (s < 0 || e < s || e > nnz) {
        if (l == 0) emb_flag(status, EMB_STATUS_BAD_OFFSETS);
        s = e = 0;
    }
    float acc[Q_ELEMS];
#pragma unroll
    for (int i = 0; i < Q_ELEMS; ++i) acc[i] = 0.f;

    const uint64_t zero_row = reinterpret_cast<uint64_t>(emb_zero_row);
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
#pragma unroll(LPR <= 16 ? IB / UNROLL : 1)
        for (int u = 0; u < IB / UNROLL; ++u) {
            const int64_t left = e - base - u * UNROLL;
            if (left > 0)
                gather_batch<UNROLL>(left, [&](auto n) {
                    gather_dequant_rows<LPR, BITS, decltype(n)::value>(acc, mine, u * UNROLL, code_off);
                });
        }
    }

    if (!live || !mine_elems) return;
    const int64_t len = e - s;
    const bool mean = (mode == EMB_POOL_MEAN) && len > 0;
    const float flen = (float)len;
    float4 *o = reinterpret_cast<float4 *>(out + bag * (int64_t)D + l * Q_ELEMS);
#pragma unroll
    for (int i = 0; i < Q_ELEMS / 4; ++i) {
        float4 v = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
        if (mean) v = make_float4(v.x / flen, v.y / flen, v.z / flen, v.w / flen);
        o[i] = v;
    }
}

// The bag is number `bag` of `offsets`.
template <int LPR, int BITS, int UNROLL, typename Source>
__device__ __forceinline__ void gather_dequant_pool_bag(Source &src, bool live, int64_t bag, int l, int64_t nnz,
                                                        const int64_t *__restrict__ rows,
                                                        const int64_t *__restrict__ offsets, int32_t D, int32_t mode,
                                                        float *__restrict__ out, uint32_t *status)
{
    int64_t s = 0, e = 0;
    if (live) {
        s = offsets[bag];
        e = offsets[bag + 1];
    }
    gather_dequant_pool_range<LPR, BITS, UNROLL>(src, live, bag, s, e, l, nnz, rows, D, mode, out, status);
}

// Lanes per row: D/16 rounded up to a power of two.
static inline int emb_quant_lanes(int32_t D)
{
    int lpr = 1;
    while (lpr * Q_ELEMS < D) lpr <<= 1;
    return lpr;
}
