"""The order of work items over a launch's workgroups (csrc/items.hpp), run on the CPU: every item is taken exactly once, in
grids of one row and of several with a ragged last row."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2212_01317_amd", "csrc")
PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "items.hpp"
int main(int argc, char** argv)
{
    for (int i = 1; i + 1 < argc; i += 2) {
        const uint32_t row = (uint32_t)atol(argv[i]), n = (uint32_t)atol(argv[i + 1]);
        const uint32_t nx = n < row ? (n + 7u) / 8u * 8u : row, ny = (n + row - 1u) / row;
        std::vector<unsigned char> taken(n, 0);
        for (uint32_t y = 0; y < ny; ++y)
            for (uint32_t x = 0; x < nx; ++x) {
                const uint32_t w = mpr::item_of(x, y, row, n);
                if (w != mpr::kNoItem) {
                    if (w >= n) return printf("item %u of %u (row %u)\\n", w, n, row), 1;
                    ++taken[w];
                }
            }
        for (uint32_t w = 0; w < n; ++w)
            if (taken[w] != 1) return printf("item %u of %u taken %d times (row %u)\\n", w, n, taken[w], row), 1;
    }
    return 0;
}
"""


@pytest.mark.parametrize("row,counts", [
    (8, (1, 7, 8, 9, 15, 16, 17, 23, 24, 25)), (64, (1, 8, 63, 64, 65, 72, 100, 127, 128, 129, 200, 1000)),
    (1 << 22, (1, 4095, (1 << 22) - 1, 1 << 22, (1 << 22) + 1, (1 << 22) + (1 << 19), (1 << 23) + 77, 3 << 22))])
def test_every_item_is_taken_once(tmp_path, row, counts):
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", str(exe), str(src)])
    args = [str(v) for n in counts for v in (row, n)]
    r = subprocess.run([str(exe), *args], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
