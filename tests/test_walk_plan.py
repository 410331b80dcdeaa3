"""The walk's plain arithmetic (csrc/walk_plan.h), compiled for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2310_20374_amd", "csrc")


def host_program(tmp_path, source):
    """Compiles `source` (a main) with the host compiler; returns a function that runs it."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(source)
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    return lambda *a: subprocess.run([str(exe), *map(str, a)], check=True, capture_output=True,
                                     text=True, timeout=300).stdout


SPACE = r"""
#include <cstdio>
#include <cstdlib>
#include "walk_plan.h"
int main(int argc, char **argv) {
    for (int i = 1; i + 2 < argc; i += 3) {
        const auto s = ncorp::list_space(atoll(argv[i]), atoll(argv[i + 1]), atoll(argv[i + 2]));
        printf("%lld %d %lld %lld\n", (long long)s.words, s.inl, (long long)s.shared0,
               (long long)s.shared_n);
    }
}
"""

# (queue_cap, m2l_cap, p2p_cap, cell_cap): small, usual and tight sizes; the queue's limit;
# pair lists around and beyond 2^30 and 2^32 pairs
SLACK = 1 << 17
CASES = [(1, SLACK + 1, SLACK + 1, 1024), (15047, SLACK + 1, SLACK + 1, 49024),
         (800_000, 400_000, 270_000, 2024), (70_000_000, 40_000_000, 20_000_000, 300_000),
         (100_000_000, 99_999_999, 99_999_999, (1 << 24) - 2),
         (100_000_000, 1_080_000_000, 537_000_000, (1 << 24) - 2)]
CASES += [(q, m, p, c) for q in (1, 100_000_000) for c in (1, 200_000, (1 << 24) - 2)
          for m in (SLACK + 1, 1 << 30)
          for p in ((1 << 30) - 1, 1 << 30, (1 << 30) + 1, 1_230_000_000, (1 << 31) + 7,
                    (1 << 33) + 5)]


def test_list_offsets_fit_32_bits(tmp_path):
    """Every offset into the hand-down lists' space is a non-negative 32-bit number
    (negative means no list) inside the buffer, whatever the capacities, and the regions
    hold two entries a visit, the segments' heads and the regions' unused ends: as long as
    the offsets allow, for any queue_cap that the library takes."""
    run = host_program(tmp_path, SPACE)
    buffers = [2 * (q + m + p) for q, m, p, _ in CASES]
    out = run(*[v for w, (q, _, _, c) in zip(buffers, CASES) for v in (w, q, c)]).split("\n")
    for (q, m, p, c), buffer, line in zip(CASES, buffers, out):
        words, inl, shared0, shared_n = map(int, line.split())
        assert words == min(buffer, 2 ** 31 - 1)
        assert shared0 == inl * c and inl in (0, 64)
        assert shared_n >= 0 and shared0 + 8 * shared_n <= words
        assert 8 * (shared_n - 300) >= 2 * q * (1 + 2 / 128), (q, m, p, c)


# Waves in blocks of four, block b of class b mod 64, of which `room` blocks run at a time;
# the next one starts when one has ended.  A scheduler picks a running wave at random; it
# does one thing: get a cell, finish it if its parent is finished, or poll once more.  No
# wave leaves for a full round of polls of all of them without a cell finished in between:
# then the walk is stuck.
TURNS = r"""
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "walk_plan.h"
using namespace ncorp;
struct Mem {
    std::vector<int> ctr = std::vector<int>(kWalkClasses, 0);
    int take(int k) { return ctr[k]++; }
    int value(int v) { return v; }
    int taken(int k) { return ctr[k]; }
    bool claim(int k, int t) { if (ctr[k] != t) return false; ctr[k]++; return true; }
};
struct Wave { WaveTurns t; int held[kWalkHeld]; int c = -1, polls = 0; bool begun = false; };
int main(int, char **a) {
    const int nc = atoi(a[1]), depth = atoi(a[2]), blocks = atoi(a[3]), room = atoi(a[4]);
    const bool help = atoi(a[5]) != 0;
    std::mt19937 rng(atoi(a[6]));
    // a breadth-first tree: levels of growing size, children of consecutive cells in order
    std::vector<int> par(nc, -1);
    int lo = 0, hi = 1;
    for (int l = 1; l < depth && hi < nc; l++) {
        const int left = depth - l, want = l == depth - 1 ? nc - hi : 1 + (int)(rng() % (1 + (nc - hi) / left));
        const int n = want < nc - hi ? want : nc - hi;
        for (int q = 0; q < n; q++) par[hi + q] = lo + (int)((long long)q * (hi - lo) / n);
        lo = hi;
        hi += n;
    }
    const int cells = hi;
    Mem m;
    std::vector<int> done(cells, 0);
    std::vector<Wave> waves(4 * blocks);
    std::vector<int> run;
    int started = 0, most = 0;
    long long finished = 0, idle = 0;
    std::vector<int> left(blocks, 4);
    auto admit = [&]() {
        int running = 0;
        for (int b = 0; b < started; b++) running += left[b] > 0;
        while (started < blocks && running < room) {
            for (int w = 0; w < 4; w++) run.push_back(4 * started + w);
            started++;
            running++;
        }
    };
    admit();
    while (!run.empty()) {
        const int at = (int)(rng() % run.size()), id = run[at];
        Wave &w = waves[id];
        if (!w.begun) { w.t.start(m, id / 4 % kWalkClasses); w.begun = true; }
        if (w.c < 0) {
            if (!w.t.get(m, w.held, cells, w.c)) {
                run[at] = run.back();
                run.pop_back();
                if (--left[id / 4] == 0) admit();
                idle = 0;
                continue;
            }
            w.polls = 0;
        }
        if (par[w.c] < 0 || done[par[w.c]]) {
            if (done[w.c]++) { printf("twice %d\n", w.c); return 0; }
            finished++;
            idle = 0;
            w.c = -1;
        } else {
            if (++w.polls % w.t.patience == 0 && help && w.t.help(m, w.held, w.c, par[w.c])) w.c = -1;
            if (w.t.nheld > most) most = w.t.nheld;
            if (++idle > 400ll * (long long)run.size() + 100000) { printf("stuck %lld\n", finished); return 0; }
        }
    }
    printf("%s %lld %d %d\n", finished == cells ? "all" : "missing", finished, cells, most);
}
"""


def test_walk_ends_with_few_workgroups_running(tmp_path):
    """Every cell is walked once however few of the walk's workgroups run at a time; with
    fewer than the classes and no helping, the walk would be stuck."""
    run = host_program(tmp_path, TURNS)
    for seed in range(6):
        for nc, depth in ((1, 1), (9, 3), (700, 5), (5000, 12), (30000, 21), (600, 21)):
            for blocks, room in ((64, 1), (64, 3), (128, 17), (256, 63), (256, 256)):
                word, finished, cells, most = run(nc, depth, blocks, room, 1, seed).split()
                assert word == "all" and finished == cells, (nc, depth, blocks, room, seed)
                assert int(most) <= depth + 1
    assert run(30000, 12, 64, 3, 0, 1).startswith("stuck")
    assert run(30000, 12, 64, 64, 0, 1).startswith("all")
