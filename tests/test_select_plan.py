"""Sizes of the multi-pass select that its state and histograms are laid out for: the header
that computes them, compiled for the host and asked over the numbers of weights and ranks."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_06973_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include "sel_plan.h"
using namespace shifter;
static int bad = 0;
static void check(uint64_t n, uint32_t k, uint64_t list_pairs) {
    const uint32_t bits = sel_bits(k), g_bits = sel_g_bits(n), cap = sel_list_cap(list_pairs, k);
    const uint32_t stages = sel_stages(n, k, list_pairs);
    // a stage's histograms fit the counters; lists start on 16 bytes and do not overlap
    bool ok = (k << bits) <= SEL_BINS && bits >= 8 && stages >= 1 && stages <= SEL_STAGES;
    ok = ok && cap % 2 == 0 && cap > 0 && (uint64_t)cap * k <= list_pairs;
    ok = ok && (g_bits == 32 ? n >> 32 == 0 : n >> g_bits == 0);
    // every split yields at most 2^bits bins, and the last stage's windows fit the lists
    uint32_t width = SEL_MAX_WIDTH;
    for (uint32_t s = 1; s < stages; ++s) {
        const uint32_t from = width == 32 ? g_bits : width;
        width = sel_shift(width, bits, g_bits);
        ok = ok && (from <= width || from - width <= bits);
    }
    ok = ok && (n <= cap || (1ull << width) <= cap);
    if (!ok && ++bad < 20) printf("n %llu k %u pairs %llu: stages %u cap %u\n", (unsigned long long)n, k,
                                  (unsigned long long)list_pairs, stages, cap);
}
int main() {
    for (uint32_t k = 1; k <= 64; ++k)
        for (int e = 0; e < 32; ++e)
            for (uint64_t m = 8; m < 16; ++m)
                for (int d = -1; d <= 1; ++d) {
                    const uint64_t n = ((m << e) >> 3) + d;
                    if (n == 0 || n >= 0xffffffffull) continue;
                    // a model's candidate buffer: a quarter of its weights, at least 8192 pairs in each of 256 parts
                    const uint64_t part = n / 4 / 256 > 8192 ? n / 4 / 256 : 8192;
                    check(n, k, part * 256);
                    if (n <= 1ull << 28) check(n, k, 1ull << 19);       // a flat run's lists
                }
    printf("%d bad\n", bad);
    return bad != 0;
}
"""


# The top bins cut all keys above zero into stretches in order, each within its window, and hold no more than 1/64 of a binade
# from 2^-46 to 2^13, 1/512 from 2^-24 to 2^4.
BINS = r"""
#include <initializer_list>
#include <stdio.h>
#include "sel_plan.h"
using namespace shifter;
int main() {
    int bad = 0;
    for (uint32_t bin = 0; bin < SEL_BINS; ++bin) {
        const uint32_t first = sel_bin_first_key(bin), end = bin + 1 < SEL_BINS ? sel_bin_first_key(bin + 1) : 0x80000000u;
        const uint32_t width = sel_bin_width(bin);
        bool ok = first < end && (uint64_t)(end - first) << 32 <= 1ull << width && width <= SEL_MAX_WIDTH;
        for (uint32_t d : {0u, 1u, (end - first) / 2, end - first - 1}) ok = ok && sel_top_bin(first + d) == bin;
        auto power = [](int e) { return (uint32_t)(127 + e) << 23; };
        const uint32_t most = first < power(-46) || bin + 1 == SEL_BINS ? 0x40000000u : first < power(-24) || first >= power(4) ? 1u << 17 : 1u << 14;
        ok = ok && end - first <= most;
        if (!ok && ++bad < 20) printf("bin %u: %08x to %08x, width %u\n", bin, first, end, width);
    }
    if (sel_top_bin((127u - 46u) << 23) == 0 || sel_top_bin(((127u + 13u) << 23) - (1u << 18)) == SEL_BINS - 1) { ++bad; printf("range\n"); }
    return bad != 0;
}
"""


def test_top_bins(tmp_path):
    run(tmp_path, BINS)


def test_stages_fit_the_state(tmp_path):
    run(tmp_path, PROGRAM)


def run(tmp_path, program):
    src = tmp_path / "plan.cpp"
    src.write_text(program)
    exe = str(tmp_path / "plan")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
