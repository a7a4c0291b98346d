// Segment reduce and row-wise Adagrad of a step of few records (spans_step, bwd_common.h) in one launch.
//
// What bounds the arrangement of update.h at these sizes is latency: a wavefront that owns 256 sorted records
// deals some 32 dependent rounds (gradients, row, update) to its lane groups, 32 us for 30 720 records on a
// sixteenth of the chip, and the rows with many lookups take four more launches on a second stream, which with
// the two event pairs are 45 us of host time.  Here a wavefront owns `span` records, a few rounds, and the rows with many lookups are summed by the same launch.
//
// Every sum is taken in the order of update.h, so results are the same bit for bit: runs of up to UPD_SHORT_MAX
// records in ascending order by a lane group; longer ones cut into LONG_CHUNK records from the run's start, a
// chunk summed by a wavefront (chunk_sum), the chunk sums added as long_combine_kernel does.
//
// A run belongs to the wavefront in whose span it starts, a chunk of a long run to the one in whose span the chunk
// starts.  The owner of a run's last chunk finishes the run: it waits for the other chunk sums, all of which belong to
// spans before its own, i.e. to wavefronts that were started earlier (as the waits of radix_sort.h).  The wait is
// bounded, and needs no second outcome: a wavefront that gives up sums the missing chunks itself, in the same order.
//
// A launch leaves every flag as it found it, zero, so that the records can serve another update.  A flag has one writer and
// one reader; whoever comes second clears it.  That is the reader, unless it gave up before the sum was there: it leaves
// SPAN_GIVEN_UP then, and the writer, which finds that in the place of zero, clears it.
//
// A chunk sum goes to memory with stores that are visible to the whole device once complete (relaxed atomics of
// device scope are not held back by the die's L2); the flag follows when they are.  No fence: a fence of device
// scope writes back every dirty line of the L2.
#pragma once
#include "bwd_common.h"
#include "update.h"

constexpr int SPAN_MAX = EMB_WAVE - UPD_LOOK;      // sorted records per wavefront at most: with the look-ahead one a lane
constexpr uint32_t SPAN_COUNT_RECORDS = 2048;      // records whose distinct rows a counting workgroup counts
constexpr uint32_t SPAN_SUMMED = 1, SPAN_GIVEN_UP = 2;   // a chunk's flag: its sum is in memory; its reader will not look at it

__device__ __forceinline__ void span_store(float *p, float v)
{
    __hip_atomic_store(reinterpret_cast<uint32_t *>(p), __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float span_load(const float *p)
{
    return __uint_as_float(__hip_atomic_load(reinterpret_cast<const uint32_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// What the writer of a flag (mine: SPAN_SUMMED) and a reader that gives up (mine: SPAN_GIVEN_UP) do with it.
__device__ __forceinline__ void span_flag_put(uint32_t *flag, uint32_t mine)
{
    const uint32_t found = __hip_atomic_exchange(flag, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (found != 0u) __hip_atomic_store(flag, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // the other has been here
}

// First record of the run that record i0 belongs to, by the whole wavefront.  `key` is its key; records of other runs
// differ, wherever they are.  Strides of 4096 and 64 records, 64 at a time, then single records: three dependent loads
// for a run of up to 2^18 records.
__device__ __forceinline__ uint32_t span_run_start(const uint32_t *__restrict__ keys, uint32_t i0, uint32_t key)
{
    const int lane = threadIdx.x & (EMB_WAVE - 1);
    uint32_t in = i0;   // a record of the run, the earliest known
    for (uint32_t stride = EMB_WAVE * EMB_WAVE; stride >= 1; stride /= EMB_WAVE) {
        for (;;) {
            const uint32_t back = (uint32_t)(lane + 1) * stride;
            const bool same = back <= in && keys[in - back] == key;
            // the records of a run are consecutive: the lanes that see it are the first ones
            const uint32_t n = (uint32_t)__popcll(__ballot(same));
            in -= n * stride;
            if (n < (uint32_t)EMB_WAVE) break;   // uniform
        }
    }
    return in;
}

// chunk_sum (update.h) of `count` records whose bags and gradient scales are in LDS.  Twice as many gradient rows are in
// flight: here a chunk is on the way that the whole launch waits for.
template <int LPR, int CPL, bool BF16>
__device__ __forceinline__ void span_chunk_sum(GradAcc<BF16> (&acc)[CPL], const uint32_t *bags /*LDS*/, const float *scales /*LDS*/,
                                               int count, const float *__restrict__ dout, int32_t chunks_per_row, int32_t D)
{
    constexpr int GPW = EMB_WAVE / LPR;
    constexpr int F = GradAcc<BF16>::F;
    constexpr int V = GradAcc<BF16>::V;
    constexpr int CU = 16 / (CPL * V) > 1 ? 16 / (CPL * V) : 1;   // gradient rows in flight: 64 registers a lane
    const int lane = threadIdx.x & (EMB_WAVE - 1);
    const int l = lane % LPR;
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc[c].zero();
    for (int i0 = lane / LPR; i0 < count; i0 += GPW * CU) {
        float4 v[CU][CPL][V];
        float sc[CU];
#pragma unroll
        for (int u = 0; u < CU; ++u) {
            const int i = i0 + u * GPW;
            sc[u] = 0.f;
#pragma unroll
            for (int c = 0; c < CPL; ++c)
#pragma unroll
                for (int x = 0; x < V; ++x) v[u][c][x] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (i < count) {
                sc[u] = scales[i];
                const float *grow = dout + (int64_t)bags[i] * D;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    const int chunk = l + c * LPR;
                    if (chunk < chunks_per_row) load_grad<BF16>(grow + (int64_t)chunk * F, v[u][c]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < CU; ++u)
#pragma unroll
            for (int c = 0; c < CPL; ++c) acc[c].fma(sc[u], v[u][c]);
    }
    group_butterfly<LPR, CPL, BF16>(acc);
}

template <int LPR, int CPL, int EU, bool BF16>
__global__ __launch_bounds__(UPD_BLOCK) void update_spans_kernel(
    const emb_table *__restrict__ tables, int32_t T, const uint32_t *__restrict__ keys, const uint32_t *__restrict__ pay,
    uint32_t n, uint32_t sentinel, const float *__restrict__ bag_scale, const float *__restrict__ dout,
    int32_t chunks_per_row, int32_t D, float inv_D, float lr, float eps, BagDiv bdiv, uint32_t span, uint32_t count_blocks,
    uint32_t *flags, float *partials, uint32_t poll_limit, BwdCtrl *ctrl, int64_t *num_unique_out)
{
    if (ctrl->abort) return;
    constexpr int WAVES = UPD_BLOCK / EMB_WAVE;
    constexpr int GPW = EMB_WAVE / LPR;
    constexpr int F = GradAcc<BF16>::F;
    const int wave = threadIdx.x / EMB_WAVE;
    const int lane = threadIdx.x & (EMB_WAVE - 1);

    // ---- the first workgroups count the distinct rows, beside the others' updates
    if (blockIdx.x < count_blocks) {   // uniform
        __shared__ uint32_t wave_heads[WAVES];
        constexpr int PER = SPAN_COUNT_RECORDS / UPD_BLOCK;
        const uint32_t at = blockIdx.x * SPAN_COUNT_RECORDS + threadIdx.x;
        uint32_t k[PER], k_before[PER];   // all asked for at once: with a test in between, 16 us of loads one after the other
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const uint32_t i = at + e * UPD_BLOCK;
            k[e] = i < n ? keys[i] : sentinel;
            k_before[e] = i < n && i > 0 ? keys[i - 1] : sentinel;
        }
        uint32_t heads = 0;
#pragma unroll
        for (int e = 0; e < PER; ++e) heads += k[e] != sentinel && k[e] != k_before[e] ? 1u : 0u;
#pragma unroll
        for (int d = EMB_WAVE >> 1; d >= 1; d >>= 1) heads += __shfl_xor(heads, d, EMB_WAVE);
        if (lane == 0) wave_heads[wave] = heads;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long mine = 1ull << 32;   // high half: workgroups that have counted
#pragma unroll
            for (int w = 0; w < WAVES; ++w) mine += wave_heads[w];
            const unsigned long long all = atomicAdd(&ctrl->task_and_multi_count, mine) + mine;
            if ((uint32_t)(all >> 32) == count_blocks) {   // the last one; the next update of these records counts from nothing
                ctrl->task_and_multi_count = 0ull;
                if (num_unique_out) *num_unique_out = (int64_t)(uint32_t)all;
            }
        }
        return;
    }

    EMB_STAGE_TABLE_DIR_T(dir, tables, T, UPD_BLOCK, true)   // T <= UPD_LDS_TABLES
    __shared__ uint32_t lk[WAVES][EMB_WAVE], lp[WAVES][EMB_WAVE];   // keys and bags of the window
    __shared__ uint32_t cb[WAVES][LONG_CHUNK];                      // bags and gradient scales of a chunk
    __shared__ float cw[WAVES][LONG_CHUNK];
    __shared__ uint8_t lh[WAVES][SPAN_MAX + 1];                     // positions of the run starts in the span, ascending
    __syncthreads();
    const int g = lane / LPR;
    const int l = lane % LPR;
    const uint32_t i0 = ((blockIdx.x - count_blocks) * WAVES + wave) * span;   // (no renumbering by die: see the waits below)
    if (i0 >= n) return;   // whole wavefronts; no barrier follows

    // ---- stage the window, a record a lane (the span and at least UPD_LOOK records after it), and the keys of the
    // UPD_LOOK records before it
    const uint32_t i = i0 + lane;
    const uint32_t key = i < n ? keys[i] : sentinel;
    const bool behind = lane < UPD_LOOK && i >= (uint32_t)UPD_LOOK;
    const uint32_t key_behind = behind ? keys[i - UPD_LOOK] : sentinel;
    lk[wave][lane] = key;
    lp[wave][lane] = i < n ? pay[i] : 0u;

    // ---- where runs start in the window (the end of the records counts), and whether one starts among the UPD_LOOK - 1
    // records before it
    const uint32_t before_span = (uint32_t)__builtin_amdgcn_readlane((int)key_behind, UPD_LOOK - 1);   // key of record i0 - 1
    const uint32_t first_key = (uint32_t)__builtin_amdgcn_readlane((int)key, 0);
    uint32_t prev = (uint32_t)__shfl_up((int)key, 1, EMB_WAVE);
    if (lane == 0) prev = before_span;
    const bool start = i == 0 || i >= n || key != prev;
    const uint64_t starts = __ballot(start);
    const uint64_t own = __ballot(start && i < n && lane < (int)span);   // the runs that belong to this wavefront
    const uint32_t prev_b = (uint32_t)__shfl_up((int)key_behind, 1, EMB_WAVE);
    const bool starts_behind = __ballot(behind && lane > 0 && (i == (uint32_t)UPD_LOOK || key_behind != prev_b)) != 0;
    constexpr uint32_t NONE = EMB_WAVE;
    const uint32_t runs = (uint32_t)__popcll(own);
    if ((own >> lane) & 1ull) lh[wave][__popcll(own & ((1ull << lane) - 1))] = (uint8_t)lane;
    // where the last of them ends, as far as the window shows (NONE is more than UPD_SHORT_MAX records after any start)
    const uint64_t later = starts & ~own;
    const uint32_t last_end = later ? (uint32_t)__ffsll((unsigned long long)later) - 1 : NONE;
    if (lane == 0) lh[wave][runs] = (uint8_t)last_end;
    __builtin_amdgcn_wave_barrier();   // (one wavefront's LDS accesses are in order)

    // ---- chunks of longer runs that start in the span (others may wait for them, so they come before the short runs):
    // first of the run that was there before it, then of those that start here
    uint32_t cand = NONE, lo = 0;   // the next chunk start to look at (position in the span) and the start of its run
    if ((starts & 1ull) == 0 && first_key != sentinel && !starts_behind) {   // (else it is short, or its first chunk covers the span)
        lo = span_run_start(keys, i0, first_key);
        const uint32_t at = lo + (i0 - lo + LONG_CHUNK - 1) / LONG_CHUNK * LONG_CHUNK - i0;
        const uint32_t over = starts ? (uint32_t)__ffsll((unsigned long long)starts) - 1 : NONE;   // the run goes at least this far
        if (at < over && at < span) cand = at;
    }
    // (of the runs that start here only the last can be longer than UPD_SHORT_MAX: a span has no more records than that)
    static_assert(SPAN_MAX <= UPD_SHORT_MAX, "a run that ends in the span it starts in is short");
    const uint32_t last_start = own ? (uint32_t)(EMB_WAVE - 1 - __clzll((long long)own)) : NONE;
    bool tail = own != 0 && last_end - last_start > (uint32_t)UPD_SHORT_MAX && lk[wave][last_start] != sentinel;
    for (;;) {   // uniform
        if (cand == NONE) {
            if (!tail) break;
            tail = false;
            cand = last_start;
            lo = i0 + last_start;
        }
        const uint32_t cs = i0 + cand;   // the chunk's first record
        const uint32_t rkey = lk[wave][cand];
        cand = NONE;
        // how many of the chunk's records there are, and whether the run goes on after them; their bags and scales go to LDS
        constexpr int PER = LONG_CHUNK / EMB_WAVE;
        uint32_t k[PER], b[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const uint32_t j = cs + e * EMB_WAVE + lane;
            k[e] = j < n ? keys[j] : sentinel;
            b[e] = j < n ? pay[j] : 0u;
        }
        const uint32_t k_after = cs + LONG_CHUNK < n ? keys[cs + LONG_CHUNK] : sentinel;
        uint32_t count = 0;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            count += (uint32_t)__popcll(__ballot(k[e] == rkey));
            cb[wave][e * EMB_WAVE + lane] = b[e];
            cw[wave][e * EMB_WAVE + lane] = bag_scale[b[e]];
        }
        const bool last = count < (uint32_t)LONG_CHUNK || k_after != rkey;
        __builtin_amdgcn_wave_barrier();
        const uint32_t n_before = (cs - lo) / LONG_CHUNK;   // chunks of this run before this one
        // the row is asked for with the gradients
        const int t = bdiv.table(cb[wave][0]);
        const int64_t r = (int64_t)rkey - dir.base(t);
        char *wrow = dir.weights(t) + r * ((int64_t)chunks_per_row * 16);
        float *aptr = dir.accum(t) + r;
        uint4 w[CPL];
        float s_old = 0.f;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int chunk = l + c * LPR;
            w[c] = make_uint4(0, 0, 0, 0);
            if (last && chunk < chunks_per_row) w[c] = load_chunk_nt(wrow + (int64_t)chunk * 16);
        }
        if (last) s_old = load_f32_nt(aptr);
        GradAcc<BF16> sum[CPL];
        span_chunk_sum<LPR, CPL, BF16>(sum, cb[wave], cw[wave], (int)count, dout, chunks_per_row, D);
        __builtin_amdgcn_wave_barrier();
        if (!last) {   // one such chunk at most starts in any LONG_CHUNK records: it has slot cs / LONG_CHUNK to itself
            const uint32_t slot = cs / LONG_CHUNK;
            float *to = partials + (int64_t)slot * ((int64_t)chunks_per_row * F);
            if (g == 0) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    const int chunk = l + c * LPR;
                    if (chunk < chunks_per_row) {
#pragma unroll
                        for (int f = 0; f < F; ++f) span_store(to + (int64_t)chunk * F + f, sum[c].a[f]);
                    }
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the sum is in memory before the flag is
            if (lane == 0) span_flag_put(flags + slot, SPAN_SUMMED);
            continue;
        }
        if (n_before > 0) {
            // the sums of the chunks before, each added by lane group (chunk mod GPW) in ascending order, this
            // one's last: the order of long_combine_kernel
            bool ready = poll_limit > 0;
            for (uint32_t c0 = 0; c0 < n_before && ready; c0 += EMB_WAVE) {   // uniform
                const uint32_t c = c0 + lane;
                bool have = c >= n_before;
                for (uint32_t polls = 0; polls < poll_limit; ++polls) {
                    if (!have) have = __hip_atomic_load(flags + (lo + c * LONG_CHUNK) / LONG_CHUNK, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) != 0;
                    if (__ballot(!have) == 0) break;   // uniform
                    __builtin_amdgcn_s_sleep(2);
                }
                ready = __ballot(!have) == 0;
            }
            asm volatile("" ::: "memory");
            for (uint32_t c = lane; c < n_before; c += EMB_WAVE) {
                uint32_t *flag = flags + (lo + c * LONG_CHUNK) / LONG_CHUNK;
                if (ready) __hip_atomic_store(flag, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else span_flag_put(flag, SPAN_GIVEN_UP);
            }
            GradAcc<BF16> acc[CPL];
#pragma unroll
            for (int c = 0; c < CPL; ++c) acc[c].zero();
            if (ready) {
                constexpr int CU = 2;   // chunk sums a group requests together
                for (uint32_t c0 = g; c0 < n_before; c0 += GPW * CU) {
                    float v[CU][CPL][F];
#pragma unroll
                    for (int u = 0; u < CU; ++u) {
                        const uint32_t cc = c0 + u * GPW;
                        const float *from = partials + (int64_t)((lo + cc * LONG_CHUNK) / LONG_CHUNK) * ((int64_t)chunks_per_row * F);
#pragma unroll
                        for (int c = 0; c < CPL; ++c) {
                            const int chunk = l + c * LPR;
#pragma unroll
                            for (int f = 0; f < F; ++f)
                                v[u][c][f] = cc < n_before && chunk < chunks_per_row ? span_load(from + (int64_t)chunk * F + f) : 0.f;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < CU; ++u)
#pragma unroll
                        for (int c = 0; c < CPL; ++c)
#pragma unroll
                            for (int f = 0; f < F; ++f) acc[c].a[f] += v[u][c][f];
                }
            } else {
                for (uint32_t cc = 0; cc < n_before; ++cc) {
                    GradAcc<BF16> one[CPL];
                    chunk_sum<LPR, CPL, EU, BF16>(one, pay, bag_scale, dout, lo + cc * LONG_CHUNK, lo + (cc + 1) * LONG_CHUNK,
                                                  chunks_per_row, D);
                    if ((cc % GPW) == (uint32_t)g) {
#pragma unroll
                        for (int c = 0; c < CPL; ++c)
#pragma unroll
                            for (int f = 0; f < F; ++f) acc[c].a[f] += one[c].a[f];
                    }
                }
            }
            if ((n_before % GPW) == (uint32_t)g) {
#pragma unroll
                for (int c = 0; c < CPL; ++c)
#pragma unroll
                    for (int f = 0; f < F; ++f) acc[c].a[f] += sum[c].a[f];
            }
            group_butterfly<LPR, CPL, BF16>(acc);
#pragma unroll
            for (int c = 0; c < CPL; ++c) sum[c] = acc[c];
        }
        if (g == 0) adagrad_apply<LPR, CPL, BF16>(sum, w, s_old, wrow, aptr, l, chunks_per_row, inv_D, lr, eps);
    }

    // ---- rows with up to UPD_SHORT_MAX lookups: as in update_kernel
    for (uint32_t k = g; k < runs; k += GPW) {
        const int pos = lh[wave][k];
        const int end = lh[wave][k + 1];
        const uint32_t rkey = lk[wave][pos];
        if (rkey == sentinel || end - pos > UPD_SHORT_MAX) continue;   // (a run not over after the look-ahead is longer)
        update_short_run<uint32_t, LPR, CPL, EU, BF16>(dir, bdiv, lp[wave], pos, end, rkey, bag_scale, dout, l, chunks_per_row, D,
                                                       inv_D, lr, eps);
    }
}
