// What a team member takes from the lines the other members write at an
// exchange (the protocol is described at TeamArgs in kernels.hip).  Plain
// templates (constexpr functions compile for host and device), so that the
// rules run on the host too.
#pragma once

#include <cstdint>

namespace vie {

constexpr uint64_t kTeamMark = 1ull << 31;

// The mark every word of exchange e carries: it changes with every use of a
// set of lines (sets alternate), and lines are zero before the first.
constexpr uint64_t team_mark(uint32_t e) { return e & 2u ? 0ull : kTeamMark; }

// One look at a reader's words: loads those that are still awaited (the bits
// of `need`) and returns the bits of those that do not carry the mark yet.
template <int N, typename Load>
constexpr uint32_t team_poll(uint32_t need, uint64_t mark, uint64_t (&v)[N], Load load)
{
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (need & (1u << i)) v[i] = load(i);
#pragma unroll
    for (int i = 0; i < N; ++i)
        if ((v[i] & kTeamMark) == mark) need &= ~(1u << i);
    return need;
}

// Hands out a reader's words (word i is number first + i * step of `words`, in
// lines of 2^line_shift): the headers by member, new nodes and kept keys, and
// the keys.  A word that a wait gave up on (the bits of `missed`) still holds
// an earlier exchange's and is left out: the keys of one exchange fit the
// step's candidates, keys of two need not.
template <int N, typename Header, typename Key>
constexpr void team_sift(const uint64_t (&v)[N], uint32_t missed, int first, int step, int words, int line_shift,
                         Header header, Key key)
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int w = first + i * step;
        if (w >= words || (missed & (1u << i))) continue;
        const uint32_t low = (uint32_t)v[i] & 0x7FFFFFFFu;
        if ((w & ((1 << line_shift) - 1)) == 0) header(w >> line_shift, (uint32_t)(v[i] >> 32), low);
        else if (low) key(v[i] | kTeamMark);
    }
}

}  // namespace vie
