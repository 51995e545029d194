"""The workgroups of a batch reach every tile once, and no place in the images falls to
one XCD throughout (workgroups go to the 8 of them by turns)."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "isaac_internal.h"
int main() {
    const int sizes[] = {1, 2, 7, 8, 9, 16, 24, 64, 100};
    for (int n : sizes) {
        std::vector<std::vector<int>> on(n, std::vector<int>(8, 0));
        int begin = 0;
        for (int job = 0; job < 256; ++job, begin += n) {
            std::vector<int> seen(n, 0);
            for (int t = 0; t < n; ++t) {
                const int tile = isaac::job_tile(t, job, n);
                if (tile < 0 || tile >= n || seen[tile]++) return std::printf("tile %d of %d twice\n", tile, n), 1;
                ++on[tile][(begin + t) % 8];
            }
        }
        for (int p = 0; p < n; ++p)
            for (int x = 0; x < 8; ++x)
                if (on[p][x] > 2 * 256 / 8) return std::printf("%d tiles: place %d on XCD %d %d times\n", n, p, x, on[p][x]), 1;
    }
    return 0;
}
"""


def test_tiles_of_a_batch(tmp_path):
    src, exe = str(tmp_path / "t.cpp"), str(tmp_path / "t")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1611_09048_amd", "csrc"), src, "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
