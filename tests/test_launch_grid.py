"""Launch geometry of the hub tier and of the light classes together
(csrc/slg_grid.h), compiled and run on the host: a device takes workgroups *
threads < 2^32 per launch, and every pair of a row group and a window, and
every light row, is visited once."""
import os
import shutil
import subprocess

import pytest

from paper_2201_11326_amd import build

CXX = shutil.which("g++") or shutil.which("c++")
WINDOW_BITS, THREADS = 14, 512

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "slg_grid.h"
int main(int argc, char **argv) {
    if (argc == 9) {  // rows of seven classes, and the limit
        int64_t n[7];
        for (int t = 0; t < 7; ++t) n[t] = atoll(argv[1 + t]);
        slg::ClassRuns<7> r;
        while (unsigned grid = r.next(n, 256, 4, slg::max_workgroups(256, atoll(argv[8])))) {
            std::printf("%u", grid);
            for (int t = 0; t < 7; ++t)
                std::printf(" %lld %lld %u", (long long)r.begin[t], (long long)r.count[t], r.first[t]);
            std::printf("\n");
        }
        return 0;
    }
    int64_t a[7];
    for (int t = 0; t < 7; ++t) a[t] = atoll(argv[1 + t]);
    const slg::HubGrid g(a[0], a[1], (int)a[2], a[3], (int)a[4], a[5], 512, a[6]);
    std::printf("%lld %lld\n", (long long)g.groups, (long long)g.total);
    for (int64_t base = 0; base < g.total; base += g.cap)
        std::printf("%lld %lld\n", (long long)base, (long long)g.count(base));
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not CXX:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("grid")
    (d / "g.cpp").write_text(PROGRAM)
    subprocess.run([CXX, "-std=c++17", "-I", build.CSRC, str(d / "g.cpp"), "-o", str(d / "g")], check=True)

    def run(*args):
        out = subprocess.run([str(d / "g"), *map(str, args)], check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


@pytest.fixture(scope="module")
def grid(program):
    def run(lo, hi, rows, kept, first_window=0, limit=0):
        head, *launches = program(lo, hi, rows, kept, WINDOW_BITS, first_window, limit)
        return head, launches
    return grid_check(run)


def grid_check(run):
    def check(lo, hi, rows, kept, first_window=0, limit=0):
        (groups, total), launches = run(lo, hi, rows, kept, first_window, limit)
        assert groups == -(-(hi - lo) // rows)
        assert total == groups * ((kept >> WINDOW_BITS) + 1 - first_window)
        at = 0
        for base, count in launches:
            assert base == at and count > 0
            assert count * THREADS < 1 << 32
            assert limit == 0 or count <= limit
            at += count
        assert at == total
        return launches
    return check


# 3.03e6 kept rows (186 windows) of which a block holds 1.45e6, 2.05e6 or all;
# the emit pass takes groups of 16
@pytest.mark.parametrize("hub_rows", [1_450_000, 2_050_000, 3_030_000])
@pytest.mark.parametrize("rows", [32, 16])
def test_whole_graph_of_ten_million_hyperedges(grid, hub_rows, rows):
    launches = grid(0, hub_rows, rows, 3_030_000)
    assert len(launches) == -(-(-(-hub_rows // rows) * 185) // ((1 << 32) // THREADS - 1))
    assert len(launches) >= (2 if hub_rows * 185 // rows >= 1 << 23 else 1)


def test_at_and_above_the_limit(grid):
    most = ((1 << 32) - 1) // THREADS
    assert len(grid(0, most * 32, 32, 1)) == 1
    assert len(grid(0, most * 32 + 1, 32, 1)) == 2
    assert len(grid(5, 5 + most * 16, 16, 1 << WINDOW_BITS, first_window=1)) == 1


@pytest.mark.parametrize("limit", [1, 2, 7, 1 << 40])
def test_lowered_limit_and_first_window(grid, limit):
    launches = grid(40, 171, 32, 3 << WINDOW_BITS, first_window=2, limit=limit)  # 5 groups, 2 windows
    assert len(launches) == -(-10 // min(limit, 10))


@pytest.mark.parametrize("rows, limit, launches", [
    ([0, 0, 0, 0, 0, 0, 0], 0, 0),
    ([1, 0, 0, 0, 0, 0, 0], 0, 1),
    ([7, 5, 4, 0, 9, 0, 1], 0, 1),
    ([600, 5, 4, 0, 9, 0, 1], 2, 5),    # 3 + 2 + 1 + 3 + 1 workgroups
    ([600, 5, 4, 0, 9, 0, 1], 1, 10),
    # under 2^26 rows in every class, more in all
    ([10**8, 3 * 10**7, 3 * 10**7, 10**7, 0, 0, 1], 0, 2),
    ([2**31 - 1, 0, 0, 0, 0, 0, 0], 0, 1),
    ([256 * 5, 4 * (2**24 - 6), 0, 0, 0, 0, 0], 0, 1),   # 2^24 - 1 workgroups
    ([256 * 5 + 1, 4 * (2**24 - 6), 0, 0, 0, 0, 0], 0, 2),
])
def test_light_classes_together(program, rows, limit, launches):
    lines = program(*rows, limit)
    assert len(lines) == launches
    done = [0] * 7
    for line in lines:
        grid, parts = line[0], [line[1 + 3 * t:4 + 3 * t] for t in range(7)]
        assert 0 < grid * 256 < 1 << 32 and (limit == 0 or grid <= limit)
        first = 0
        for c in range(6, -1, -1):  # the last class first, each from its own workgroup on
            begin, count, _ = parts[c]
            assert begin == done[c] and count >= 0
            assert parts[6 - c][2] == first
            done[c] += count
            first += -(-count // (4 if c else 256))
        assert first == grid
    assert done == rows
