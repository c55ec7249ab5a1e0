"""The encoder's chained offsets: blocks that draw tickets, store their segment's size and walk back
over their predecessors' words, played step by step on the host in random orders with few
polls allowed.  Whatever the order: every block ends, and a call in which some wait ran out says so;
one in which none did has every offset right."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_06973_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <random>
#include <vector>
#include "chain.h"
using namespace shifter;

struct Block {
    ChainWalk walk{0};
    bool placed = false, done = false;
};

int main() {
    std::mt19937 rng(1);
    int broke = 0, silent = 0, wrong = 0, whole = 0;
    for (int game = 0; game < 60000; ++game) {
        const uint32_t n = 1 + rng() % (game % 3 ? 8 : 150), limit = 1 + rng() % (game % 2 ? 4 : 400);
        const uint32_t resident = 1 + rng() % 8;
        std::vector<uint64_t> word(n, 0), size(n), off(n, ~0ull);
        uint64_t result[4] = {77, 0, 0, 0}, total = 0;      // cleared by the call's first kernel but for the bytes
        for (auto& s : size) { s = 5 + rng() % 40000; total += s; }
        std::vector<Block> blocks(n);
        auto put = [](uint64_t* p, uint64_t v) { *p = v; };
        std::vector<uint32_t> live;
        uint32_t ticket = 0, left = n;
        while (left) {
            if (ticket < n && (live.empty() || (live.size() < resident && rng() % 3 == 0))) {
                blocks[ticket].walk = ChainWalk(ticket);
                live.push_back(ticket++);
                continue;
            }
            const size_t at = rng() % 2 ? live.size() - 1 : rng() % live.size();      // the young run ahead
            const uint32_t c = live[at];
            Block& b = blocks[c];
            if (!b.placed) {
                word[c] = chain_size(c, size[c]);
                b.placed = true;
            } else if (b.walk.waits()) {
                uint64_t known = 0, here = 0, bad = 0;
                for (int l = 0; l < 64; ++l) {
                    const int64_t i = b.walk.last - l;
                    const uint64_t x = i >= 0 ? word[i] : 2ull << 62;
                    known |= (uint64_t)(x >> 62 == 2) << l;
                    here |= (uint64_t)(x >> 62 != 0) << l;
                    bad |= (uint64_t)(x >> 62 == 3) << l;
                }
                const int64_t last = b.walk.last;
                const uint64_t need = b.walk.look(known, here, bad, limit);
                for (int l = 0; l < 64; ++l)
                    if ((need >> l & 1) && last - l >= 0) b.walk.sum += word[last - l] & CHAIN_VALUE;
            } else {
                chain_leave(b.walk, c, c + 1 == n, size[c], &word[c], result, put);
                if (!b.walk.broken) off[c] = b.walk.sum;
                live.erase(live.begin() + at);
                --left;
            }
        }
        uint64_t sum = 0;
        bool missing = false, bad_off = false;
        for (uint32_t c = 0; c < n; ++c) {
            missing |= off[c] == ~0ull;
            bad_off |= off[c] != ~0ull && off[c] != sum;
            sum += size[c];
        }
        const bool told = (result[CHAIN_STATUS] | result[CHAIN_BROKE]) != 0;
        broke += missing;
        silent += missing && !told;
        wrong += bad_off || (!missing && (told || result[CHAIN_BYTES] != total));
        whole += !missing;
    }
    printf("%d with a wait that ran out, %d of them silent; %d wrong; %d whole\n", broke, silent, wrong, whole);
    return silent != 0 || wrong != 0 || broke < 1000 || whole < 1000;
}
"""


def test_a_wait_that_runs_out_is_told(tmp_path):
    src = tmp_path / "chain.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "chain")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout
