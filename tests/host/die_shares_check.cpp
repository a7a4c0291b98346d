// Host check of the cuts that share the workgroups of a mixed-width lookup among the dies, against cuts found by
// bisection: a stretch ends at the first workgroup that starts at or after its share of the cost.  Costs beyond 32 bits
// are among them (477e6 bags of 16-byte rows cost 4.3e9), and cuts with more workgroups in a stretch than a launch has
// room for, in whose place equal numbers are wanted.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "die_shares.h"

constexpr uint32_t DIES = 8, ROOM = 0xFFFFFFFFu / 256 / DIES;

static bool check(const std::vector<uint32_t> &blocks, const std::vector<uint64_t> &cost)
{
    const int T = (int)blocks.size();
    std::vector<uint32_t> first(T + 1, 0);
    for (int t = 0; t < T; ++t) first[t + 1] = first[t] + blocks[t];
    const uint32_t all = first[T];
    auto before = [&](uint32_t w) {   // cost of the workgroups before w
        uint64_t c = 0;
        for (int t = 0; t < T; ++t) c += (uint64_t)(w < first[t] ? 0 : w > first[t + 1] ? blocks[t] : w - first[t]) * cost[t];
        return c;
    };
    uint32_t want[DIES + 1], most = 0;
    for (uint32_t d = 0; d <= DIES; ++d) {
        uint32_t lo = 0, hi = all;
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2;
            if (before(mid) * DIES >= before(all) * d) hi = mid;
            else lo = mid + 1;
        }
        want[d] = d == DIES ? all : lo;
        if (d > 0 && want[d] - want[d - 1] > most) most = want[d] - want[d - 1];
    }
    if (most > ROOM) {
        most = (all + DIES - 1) / DIES;
        for (uint32_t d = 0; d <= DIES; ++d) want[d] = (uint64_t)d * most < all ? d * most : all;
    }
    uint32_t cut[DIES + 1];
    const uint32_t got = emb_die_shares<DIES>(T, [&](int32_t t) { return first[t]; }, [&](int32_t t) { return cost[t]; }, ROOM, cut);
    bool ok = got == most;
    for (uint32_t d = 0; d <= DIES; ++d) ok = ok && cut[d] == want[d];
    if (!ok) {
        std::printf("FAIL T=%d blocks=%u cuts", T, all);
        for (uint32_t d = 0; d <= DIES; ++d) std::printf(" %u (%u)", cut[d], want[d]);
        std::printf("\n");
    }
    return ok;
}

int main()
{
    // costs of a workgroup: rows of 16 bytes 256 * 9, of 64 64 * 12, of 256 16 * 24, of 1024 4 * 72
    const std::vector<std::vector<uint32_t>> blocks = {
        {1}, {7}, {9}, {0}, {0, 5, 0}, {3, 1, 1}, {128, 128, 512, 1024}, {1000, 1, 1, 1}, {1, 1, 1, 1000},
        {1863000}, {4000000, 300000}, {16000000}, {16000000 - 7}, {2000000, 12000000}, {13000000, 700000},
        {6000000, 6000000, 4000000}, {8000000, 0, 8000000, 1}, {100000, 100000, 100000, 14000000}};
    const uint64_t costs[] = {256 * 9, 64 * 12, 16 * 24, 4 * 72};
    long checked = 0;
    for (const auto &b : blocks)
        for (int turn = 0; turn < 4; ++turn) {
            std::vector<uint64_t> c;
            for (size_t t = 0; t < b.size(); ++t) c.push_back(costs[(t + turn) % 4]);
            if (!check(b, c)) return 1;
            ++checked;
        }
    std::printf("OK %ld\n", checked);
    return 0;
}
