"""Which matrices share a launch of the fused block elimination (host code,
compiled here with the host compiler): the ranges are a partition in order, the
one with the most rows is named, and classes are joined exactly where those
before or after it are at most 256 together."""
import random
import shutil
import subprocess

import pytest

from paper_2101_01763_amd import build

SRC = """
#include "elim_launches.h"
#include <cstdio>
int main() {
  int na;
  while (std::scanf("%d", &na) == 1) {
    std::vector<int> n(static_cast<size_t>(na));
    for (auto &x : n) if (std::scanf("%d", &x) != 1) return 1;
    size_t big;
    const auto r = spand::elim_launches(na, [&](int i) { return n[static_cast<size_t>(i)]; }, &big);
    std::printf("%zu", big);
    for (const auto &q : r) std::printf(" %d %d", q.first, q.second);
    std::printf("\\n");
  }
}
"""
UNITS = 256


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    cxx = shutil.which("g++") or build._hipcc()
    d = tmp_path_factory.mktemp("elim")
    (d / "m.cpp").write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(d / "m"), str(d / "m.cpp")], check=True)

    def run(lists):
        text = "\n".join(" ".join(map(str, [len(n), *n])) for n in lists)
        out = subprocess.run([str(d / "m")], input=text, capture_output=True, text=True, check=True).stdout
        rows = [list(map(int, ln.split())) for ln in out.splitlines()]
        return [(r[0], list(zip(r[1::2], r[2::2]))) for r in rows]
    return run


def _rows(counts):
    """counts[c] matrices of 64-row class c (c = 1: 1 to 64 rows), descending."""
    return [64 * c for c in sorted(counts, reverse=True) for _ in range(counts[c])]


@pytest.mark.parametrize("counts,want,big", [
    ({9: 1}, [1], 0),
    ({9: 1, 5: 3, 1: 252}, [256], 0),                               # 256: one launch
    ({9: 1, 5: 3, 1: 253}, [4, 253], 1),                            # 257: two of them joined before the rest
    ({16: 1, 12: 125, 9: 3906}, [126, 3906], 1),
    ({16: 1, 9: 300, 4: 200, 2: 50, 1: 6}, [1, 300, 256], 1),       # biggest in the middle, both sides joined
    ({16: 1, 9: 300, 4: 200, 2: 50, 1: 7}, [1, 300, 200, 50, 7], 1),
    ({16: 1, 12: 255, 9: 2000, 4: 256}, [256, 2000, 256], 1),
    ({16: 2, 12: 255, 9: 2000, 4: 257, 1: 1}, [2, 255, 2000, 257, 1], 2),
    ({9: 300, 4: 3, 1: 4}, [300, 7], 0),
    ({9: 1, 4: 3, 1: 4000}, [4, 4000], 1),
    ({4: 300}, [300], 0),
])
def test_expected(launches, counts, want, big):
    (got_big, got), = launches([_rows(counts)])
    assert got_big == big and [b - a for a, b in got] == want


def test_partition(launches):
    rng = random.Random(5)
    lists = []
    for _ in range(300):
        counts = {}
        for _ in range(rng.randint(1, 7)):
            counts[rng.randint(1, 16)] = rng.choice([1, 2, 7, 60, 128, 255, 256, 257, 500])
        n = [64 * c - rng.randint(0, 63) for c, k in counts.items() for _ in range(k)]
        lists.append(sorted(n, reverse=True))
    for n, (big, got) in zip(lists, launches(lists)):
        assert got[0][0] == 0 and got[-1][1] == len(n) and all(a < b for a, b in got)
        assert all(got[i][1] == got[i + 1][0] for i in range(len(got) - 1)) and big < len(got)
        cls = lambda q: {-(-x // 64) for x in n[q[0]:q[1]]}  # noqa: E731
        for q in got:
            assert len(cls(q)) == 1 or q[1] - q[0] <= UNITS
        for side in (got[:big], got[big + 1:]):
            if side and side[-1][1] - side[0][0] <= UNITS:
                assert len(side) == 1
        if len(n) <= UNITS:
            assert len(got) == 1
        else:                       # the named range is a whole class, and none has more rows
            assert len(cls(got[big])) == 1
            work = {}
            for x in n:
                work.setdefault(-(-x // 64), []).append(x)
            assert len(n[slice(*got[big])]) * n[got[big][0]] == max(len(v) * v[0] for v in work.values())
