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
        printf("%d %lld %d %lld %lld\n", s.own ? 1 : 0, (long long)s.words, s.inl,
               (long long)s.shared0, (long long)s.shared_n);
    }
}
"""

# (queue_cap, p2p_cap, cell_cap): small and usual sizes; the queue's limit; pair lists
# around 2^30 (a space of 2^31 words), beyond it, and beyond 2^32 pairs
CASES = [(1, 131073, 1024), (262145, 262145, 2024), (70_000_000, 12_000_000, 300_000),
         (100_000_000, 99_999_999, (1 << 24) - 2), (100_000_000, 537_000_000, (1 << 24) - 2)]
CASES += [(q, p, c) for q in (1, 100_000_000) for c in (1, 200_000, (1 << 24) - 2)
          for p in ((1 << 30) - 1, 1 << 30, (1 << 30) + 1, 1_230_000_000, (1 << 31) + 7,
                    (1 << 33) + 5)]


def test_list_offsets_fit_32_bits(tmp_path):
    """Every offset into the hand-down lists' space is a non-negative 32-bit number
    (negative means no list) inside the buffer, whatever the capacities."""
    run = host_program(tmp_path, SPACE)
    out = run(*[v for c in CASES for v in c]).split("\n")
    for (q, p, c), line in zip(CASES, out):
        own, words, inl, shared0, shared_n = map(int, line.split())
        assert own == (q >= p)
        buffer = 2 * (q if own else p)
        assert words <= buffer and words <= 2 ** 31 - 1
        assert words == min(buffer, 2 ** 31 - 1)           # and no less than that
        assert shared0 == inl * c and inl in (0, 64)
        assert shared_n >= 0 and shared0 + 8 * shared_n <= words
        assert inl == 0 or (shared0 <= words // 2 and words - shared0 >= q)
