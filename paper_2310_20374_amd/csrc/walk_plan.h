// The parts of the walk that are plain arithmetic: how its hand-down lists share the
// space set aside for them.  No HIP here, so that a host program can check them.
#pragma once

#include <stdint.h>

namespace ncorp {

// The hardware deals the workgroups of a launch to the 8 XCDs in turn (workgroup b
// runs on XCD b mod 8), and each XCD has its own L2.
constexpr int kXcds = 8;
// hand-down entries a cell keeps in a slot of its own
constexpr int64_t kWalkInline = 64;

// The space of a walk's hand-down lists: the 2 queue_cap words set aside for its open
// pairs, or those of p2p_cap pairs where a caller asked for a smaller queue than that, as a
// slot of `inl` entries a cell and kXcds equal regions for longer lists.
struct ListSpace {
    bool own;                  // in the queue's buffer, else in that of the pair list
    int64_t words;             // 32-bit words of the space
    int inl;                   // entries of a cell's own slot
    int64_t shared0, shared_n; // start of the first region, words of each
};

// A list's place is kept as a 32-bit offset, negative for none, so a larger buffer (more
// than 2^30 pairs) is used up to there.  A pair is handed down at most once, so queue_cap
// words hold what a walk of queue_cap visits leaves to be opened; the cells' own slots are
// taken where that leaves as much, and the rest is room for segment heads and for the
// direct-sum pairs that leaves inherit.
constexpr ListSpace list_space(int64_t queue_cap, int64_t p2p_cap, int64_t cell_cap) {
    ListSpace s{};
    s.own = queue_cap >= p2p_cap;
    const int64_t pairs = s.own ? queue_cap : p2p_cap;
    s.words = pairs > INT32_MAX / 2 ? INT32_MAX : 2 * pairs;
    s.inl = s.words / 2 >= kWalkInline * cell_cap &&
                    s.words - kWalkInline * cell_cap >= queue_cap
                ? (int)kWalkInline : 0;
    s.shared0 = (int64_t)s.inl * cell_cap;
    s.shared_n = (s.words - s.shared0) / kXcds;
    return s;
}

}  // namespace ncorp
