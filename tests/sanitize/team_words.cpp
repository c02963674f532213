// Two members of a team meet at exchanges in plain memory; then one of them
// stops.  The other's wait gives up on its words, and what it then takes may
// hold no key of an earlier exchange: its buffer has room for the step's own
// candidates only.  (Test infrastructure: the rules are team.hpp's, the
// buffers here are sized as the kernel sizes its own.)
#include "team.hpp"

#include <cstdio>
#include <vector>

using namespace vie;

namespace {

constexpr int kTeam = 2, kLine = 8, kShift = 3, kThreads = 4, kWordsEach = kTeam * kLine / kThreads;
uint64_t lines[2][kTeam][kLine];  // two sets, zero before the first exchange

void publish(uint32_t e, int member, const std::vector<uint64_t> &keys, uint32_t fresh)
{
    for (int w = 0; w < kLine; ++w) {
        const uint64_t v = w == 0 ? ((uint64_t)fresh << 32) | keys.size()
                                  : w <= (int)keys.size() ? keys[(size_t)w - 1] & ~kTeamMark : 0ull;
        lines[e & 1u][member][w] = v | team_mark(e);
    }
}

struct Took {
    std::vector<uint64_t> keys;
    uint32_t fresh = 0, kept = 0;
    bool gave_up = false;
};

// what member 0's threads take at exchange e, waiting `looks` times at most
Took take(uint32_t e, int looks)
{
    Took t;
    for (int tid = 0; tid < kThreads; ++tid) {
        uint64_t v[kWordsEach] = {};
        uint32_t need = 0;
        for (int i = 0; i < kWordsEach; ++i)
            if ((tid + i * kThreads) >> kShift != 0) need |= 1u << i;
        for (int n = 0; need && n < looks; ++n)
            need = team_poll(need, team_mark(e), v, [&](int i) { return (&lines[e & 1u][0][0])[tid + i * kThreads]; });
        if (need) t.gave_up = true;
        team_sift(
            v, need, tid, kThreads, kTeam * kLine, kShift,
            [&](int o, uint32_t fresh, uint32_t kept) {
                if (o == 0) return;
                t.fresh += fresh;
                t.kept += kept;
            },
            [&](uint64_t key) { t.keys.push_back(key); });
    }
    return t;
}

int fail(const char *what)
{
    std::printf("failed: %s\n", what);
    return 1;
}

}  // namespace

int main()
{
    const uint64_t id = 0xFFFFFFFFull;  // ~id, bit 31 set as in every key
    for (uint32_t e = 0; e < 6; ++e) {
        std::vector<uint64_t> keys;
        for (uint32_t i = 0; i < 1 + e % 7; ++i) keys.push_back(((uint64_t)(100 * e + i) << 32) | (id - i));
        if (!take(e, 3).gave_up) return fail("a wait that ended before the other member wrote");
        publish(e, 1, keys, 10 + e);
        const Took t = take(e, 3);
        if (t.gave_up || t.fresh != 10 + e || t.kept != keys.size()) return fail("a header");
        if (t.keys.size() != keys.size()) return fail("the number of keys");
        for (const uint64_t k : keys) {
            bool found = false;
            for (const uint64_t g : t.keys) found |= g == k;
            if (!found) return fail("a key");
        }
    }
    // the other member stops: its lines hold the keys of exchanges 4 and 5
    const Took none = take(6, 3);
    if (!none.gave_up) return fail("a wait that should have given up");
    if (!none.keys.empty() || none.kept || none.fresh) return fail("words of an earlier exchange taken after a wait that gave up");
    // or stops half way through its line: the written half counts, no more
    for (int w = 0; w < kLine / 2; ++w)
        lines[0][1][w] = ((w == 0 ? 7ull : ((uint64_t)w << 32) | (id - (uint32_t)w)) & ~kTeamMark) | team_mark(6);
    const Took half = take(6, 3);
    if (!half.gave_up || half.keys.size() != (size_t)kLine / 2 - 1) return fail("half a line");
    std::printf("all checks passed\n");
    return 0;
}
