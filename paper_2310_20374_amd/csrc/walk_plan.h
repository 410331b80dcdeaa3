// The parts of the walk that are plain arithmetic: how its hand-down lists share the
// space set aside for them, and which cell a wave takes next.  No HIP here, so that a host
// program can check them.
#pragma once

#include <stdint.h>

namespace ncorp {

// The hardware deals the workgroups of a launch to the 8 XCDs in turn (workgroup b
// runs on XCD b mod 8), and each XCD has its own L2.
constexpr int kXcds = 8;
// hand-down entries a cell keeps in a slot of its own
constexpr int64_t kWalkInline = 64;

// The space of a walk's hand-down lists: a slot of `inl` entries a cell and kXcds equal
// regions for longer lists.
struct ListSpace {
    int64_t words;             // 32-bit words in use
    int inl;                   // entries of a cell's own slot
    int64_t shared0, shared_n; // start of the first region, words of each
};

// Of the `words` words of the workspace that a walk may use, at least 2 (queue_cap +
// m2l_cap + p2p_cap) of them.  A list's place is kept as a 32-bit offset, negative for
// none, so a larger buffer is used up to there.
//
// A walk of V visits lists at most V entries and as many again: a pair to be opened in one
// cell's list, a direct-sum pair in those of both its cells if they are internal.  (What a
// cell inherits takes no more than its own slot.)  A list beyond its slot has segments, the
// first without a head, the next ones with two words for some 200 entries; the unused ends
// of the regions are lost, less than 300 words each.  So 2 queue_cap words for them and
// what m2l_cap and p2p_cap leave beside the cells' slots (both carry 2^17 entries and more
// on top of what the caller asked for) hold every walk of up to queue_cap visits, and
// without slots too; slots are taken where that is so with them.
constexpr ListSpace list_space(int64_t words, int64_t queue_cap, int64_t cell_cap) {
    ListSpace s{};
    s.words = words < INT32_MAX ? words : INT32_MAX;
    const int64_t lists = 2 * queue_cap + queue_cap / 16 + 4096;
    s.inl = s.words - kWalkInline * cell_cap >= lists ? (int)kWalkInline : 0;
    s.shared0 = (int64_t)s.inl * cell_cap;
    s.shared_n = (s.words - s.shared0) / kXcds;
    return s;
}

// ---------------------------------------------------------------- turns
// A walk deals its cells in runs of kWalkRun to kWalkClasses classes of waves; turn i of
// a class is its i-th cell in breadth-first order.
constexpr int kWalkRun = 8;
constexpr int kWalkClasses = 64;
constexpr int cell_class(int c) { return c / kWalkRun % kWalkClasses; }
constexpr int cell_turn(int c) {
    return c / (kWalkRun * kWalkClasses) * kWalkRun + c % kWalkRun;
}
constexpr int64_t turn_cell(int cls, int turn) {
    return ((int64_t)(turn / kWalkRun) * kWalkClasses + cls) * kWalkRun + turn % kWalkRun;
}

// The cells of one wave.  It takes those of its own class, and one that waits for a parent
// which nobody has taken (no wave of the parent's class may be running yet) puts its cell
// aside and takes the parent's class's lowest cell first.  That one is the parent or comes
// before it, so it lies on a higher level than the cell put aside: a wave holds a cell a
// level at most.  Of the cells that waves have taken and not finished, take the lowest: its
// parent is not among them, so it is finished or nobody has taken it, and either way that
// wave goes on.  So the walk ends with a single wave running as well.
//
// M holds the classes' counters: take(cls) adds one and returns the turn before (value()
// makes it known to the wave), taken(cls) reads the counter, claim(cls, t) moves it from t to
// t + 1 or returns false.
// Polls for a parent, a power of two, before a wave looks whether it is taken (some 90 us,
// longer than most waits of a whole chip), and once it has helped: waves are missing.
constexpr int kHelpPolls = 64, kHelpAgain = 4;
constexpr int kWalkHeld = 24;      // more than the levels of a tree
struct WaveTurns {
    int cls = 0, next = 0, nheld = 0, patience = kHelpPolls;

    template <class M> constexpr void start(M &m, int own) {
        cls = own;
        next = m.take(cls);
    }
    // the wave's next cell, or false: its class has none left
    template <class M> constexpr bool get(M &m, const int *held, int nc, int &c) {
        if (nheld > 0) {
            c = m.value(held[--nheld]);
            return true;
        }
        const int i = m.value(next);
        const int64_t t = turn_cell(cls, i);
        if (i < 0 || t >= nc) return false;
        next = m.take(cls);        // in flight while the cell is worked on
        c = (int)t;
        return true;
    }
    // Cell c waits for its parent.  True: c is put aside, get() returns another one first.
    template <class M> constexpr bool help(M &m, int *held, int c, int parent) {
        const int k = cell_class(parent), t = m.taken(k);
        if (t > cell_turn(parent) || nheld + 2 > kWalkHeld || !m.claim(k, t)) return false;
        held[nheld++] = c;
        held[nheld++] = (int)turn_cell(k, t);
        patience = kHelpAgain;
        return true;
    }
};

}  // namespace ncorp
