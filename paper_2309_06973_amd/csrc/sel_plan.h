// Sizes of the multi-pass select (select.hip) that follow from the number of weights, of ranks
// and of list pairs alone.  Plain C++: host, device and tests share it.
#pragma once

#include <stdint.h>

namespace shifter {

constexpr uint32_t SEL_BINS = 16384;      // counters of one histogram: the top bins, or all windows' of a stage
constexpr uint32_t SEL_STAGES = 8;        // at most this many stages for any N < 2^32 and K <= MAXK
constexpr uint32_t SEL_MAX_WIDTH = 62;    // of a window: 2^30 keys of the bins at both ends of the binning
// A list is ranked by one block, in two walks of about 16 us each for this many pairs of one key: a window
// with more weights is split by a further stage, one read of the arena by all blocks, while there
// is one.
constexpr uint32_t SEL_LIST_GOOD = 1u << 16;

// log2 of the bins of one window's histogram: what k of them may share SEL_BINS counters.
constexpr uint32_t sel_bits(uint32_t k) {
    uint32_t b = 12;
    while (b > 8 && (k << b) > SEL_BINS) --b;
    return b;
}

// Bits of an index below n.
constexpr uint32_t sel_g_bits(uint64_t n) {
    uint32_t b = 0;
    while (b < 32 && (n >> b) != 0) ++b;
    return b;
}

// A window of 2^width composites is split into bins of 2^shift: by key until it holds a single
// one (width 32), then by index, of which the lowest g_bits can be set.
constexpr uint32_t sel_shift(uint32_t width, uint32_t bits, uint32_t g_bits) {
    if (width > 32u) return width - 32u > bits ? width - bits : 32u;
    const uint32_t w = width == 32u ? g_bits : width;
    return w > bits ? w - bits : 0u;
}

// Room of one rank's list in pairs: an even number, so that every list starts on 16 bytes.
constexpr uint32_t sel_list_cap(uint64_t list_pairs, uint32_t k) {
    const uint64_t share = list_pairs / k;
    return (uint32_t)(share < 1u << 20 ? share : 1u << 20) & ~1u;
}

// Stages that certainly suffice: a window of the widest kind is split until no more weights
// than a list holds can lie in it, and listed.  Where a list would hold them all from the
// start, but more than is good, three: equal weights are told from others by the first, split by
// index in the second and listed in the third.
constexpr uint32_t sel_stages(uint64_t n, uint32_t k, uint64_t list_pairs) {
    const uint32_t bits = sel_bits(k), g_bits = sel_g_bits(n), list_cap = sel_list_cap(list_pairs, k);
    uint32_t width = SEL_MAX_WIDTH, stages = 1;
    while ((n < (1ull << width) ? n : 1ull << width) > list_cap) {
        width = sel_shift(width, bits, g_bits);
        ++stages;
    }
    return n > SEL_LIST_GOOD && stages < 3u ? 3u : stages;
}

}  // namespace shifter
