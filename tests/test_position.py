"""Search midpoints and aligned blocks (csrc/slg_position.h) over the positions that lists of
fewer than 2^31 entries have, compiled and run on the host."""
import shutil
import subprocess

import pytest

from paper_2201_11326_amd import build

CXX = shutil.which("g++") or shutil.which("c++")

PROGRAM = r"""
#include <climits>
#include <cstdio>
#include "slg_position.h"
int main() {
    const int at[] = {0, 1, 2, (1 << 30) - 1, 1 << 30, (1 << 30) + 1, INT_MAX - 2, INT_MAX - 1, INT_MAX};
    for (int lo : at)
        for (int hi : at) {
            if (lo > hi) continue;
            const long long want = ((long long)lo + hi) / 2;
            if (slg::middle(lo, hi) != want || (lo < hi && slg::middle(lo, hi) >= hi)) {
                std::printf("%d %d: %d, not %lld\n", lo, hi, slg::middle(lo, hi), want);
                return 1;
            }
        }
    // a list's last position: its own block begins inside the list, the next ones past its end
    for (int end : at) {
        if (end < 1) continue;
        const unsigned last = (unsigned)end - 1u, own = slg::block_at(last);
        if (own > last || own + 7u < last || own % 8u) return 2;
        for (unsigned ahead = 1; ahead < 8; ++ahead)
            if (slg::block_at(last, ahead) != own + 8u * ahead || slg::block_at(last, ahead) <= last) return 3;
    }
    return 0;
}
"""


@pytest.mark.skipif(not CXX, reason="no host C++ compiler")
def test_middle_and_blocks(tmp_path):
    (tmp_path / "p.cpp").write_text(PROGRAM)
    subprocess.run([CXX, "-std=c++17", "-I", build.CSRC, str(tmp_path / "p.cpp"), "-o", str(tmp_path / "p")],
                   check=True)
    out = subprocess.run([str(tmp_path / "p")], capture_output=True, text=True)
    assert out.returncode == 0, (out.returncode, out.stdout)
