// Cuts numbered workgroups into one stretch of equal cost per die.  Host code without HIP, so that it can be checked on
// the CPU at sizes that no test would launch.
#pragma once
#include <cstdint>

// Table t's workgroups are numbered from first(t) on (first(T): how many there are in all), each costs cost(t) > 0.
// Stretch d is workgroups cut[d] .. cut[d + 1] - 1.  Returns the largest number of workgroups in a stretch.
// A launch has room for `most_allowed` workgroups in every stretch: where equal costs need more, the stretches get equal
// numbers.
template <uint32_t DIES, typename First, typename Cost>
uint32_t emb_die_shares(int32_t T, First first, Cost cost, uint32_t most_allowed, uint32_t (&cut)[DIES + 1])
{
    const uint32_t blocks_all = first(T);
    uint64_t total = 0;   // fewer than 2^31 workgroups of less than 2^13 each
    for (int32_t t = 0; t < T; ++t) total += (uint64_t)(first(t + 1) - first(t)) * cost(t);
    uint64_t before = 0;  // cost of the tables before t
    uint32_t d = 1;
    cut[0] = 0;
    for (int32_t t = 0; t < T; ++t) {
        const uint64_t blocks = first(t + 1) - first(t), per = cost(t);
        // the cuts that fall into this table: the first workgroup that starts at or after d shares of the cost
        for (; d < DIES && total * d <= (before + blocks * per) * DIES; ++d) {
            const uint64_t at = (total * d + DIES - 1) / DIES;
            cut[d] = first(t) + (uint32_t)(((at > before ? at - before : 0) + per - 1) / per);   // (the cost does not fit 32 bits)
        }
        before += blocks * per;
    }
    for (; d <= DIES; ++d) cut[d] = blocks_all;
    uint32_t most = 0;
    for (d = 0; d < DIES; ++d)
        if (cut[d + 1] - cut[d] > most) most = cut[d + 1] - cut[d];
    if (most > most_allowed) {
        most = (uint32_t)(((uint64_t)blocks_all + DIES - 1) / DIES);
        for (d = 0; d <= DIES; ++d) {
            const uint64_t at = (uint64_t)d * most;
            cut[d] = at < blocks_all ? (uint32_t)at : blocks_all;
        }
    }
    return most;
}
