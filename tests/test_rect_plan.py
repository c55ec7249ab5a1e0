"""The rectangles of the portfolio rebuild: the header that sizes them, compiled for the host and asked over row
lengths on both sides of the number of weights from which they are whole."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_06973_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include "rect_plan.h"
using namespace shifter;
int main() {
    int bad = 0;
    for (double weights : {100.0, RECT_FEW_WEIGHTS, RECT_FEW_WEIGHTS + 1.0, 1e9})
        for (uint32_t row = 1; row <= 1024; ++row) {
            const uint32_t rows = rect_rows(weights, row), padded = (row + 127u) / 128u * 128u;
            const uint32_t whole = 8192u / padded < 64u ? 8192u / padded : 64u;
            bool ok = rows >= 1u && rows <= 64u && rows * padded <= RECT_ELEMS;
            if (weights > RECT_FEW_WEIGHTS) ok = ok && rows == whole;
            // in a small network a quarter of that, but not for a few dozen weights
            else ok = ok && (rows == 64u || (rows + 1u) * row > 1024u) && (rows * padded <= 2048u || rows * row <= 1024u);
            if (!ok && ++bad < 20) printf("%.0f weights, rows of %u: %u\n", weights, row, rows);
        }
    printf("%d bad\n", bad);
    return bad != 0;
}
"""


def test_rows(tmp_path):
    src = tmp_path / "rect.cpp"
    src.write_text("#include <initializer_list>\n" + PROGRAM)
    exe = str(tmp_path / "rect")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
