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

// The top bins: 1/512 of a binade from 2^-24 to 2^4, where nearly all thresholds of networks lie, 1/64 below down to 2^-47 and above
// up to 2^13; the keys below share the first bin with its own, those above the last one.  Against 1/256 from 2^-50 to 2^14
// lists are half as long, and twice as many bins are added up by the blocks: us a call 10 counts of 14.7 M normal weights 51.6 ->
// 45.8, half precision 83 -> 62, one of 100 M 225 -> 159, but of 14.7 M weights of many magnitudes 45.8 -> 47.6 (one count 34.2
// -> 38.2), where nearly all bins hold some.
constexpr uint32_t SEL_FINE_SHIFT = 14, SEL_WIDE_SHIFT = 17;
constexpr uint32_t SEL_KEY_FIRST = (127u - 47u) << 23, SEL_KEY_FINE = (127u - 24u) << 23, SEL_KEY_ABOVE = (127u + 4u) << 23,
                   SEL_KEY_END = (127u + 13u) << 23;
constexpr uint32_t SEL_BIN_FINE = (SEL_KEY_FINE - SEL_KEY_FIRST) >> SEL_WIDE_SHIFT;           // first fine bin
constexpr uint32_t SEL_FINE_BINS = (SEL_KEY_ABOVE - SEL_KEY_FINE) >> SEL_FINE_SHIFT;
constexpr uint32_t SEL_BIN_ABOVE = SEL_BIN_FINE + SEL_FINE_BINS;
static_assert(SEL_BIN_ABOVE + ((SEL_KEY_END - SEL_KEY_ABOVE) >> SEL_WIDE_SHIFT) == SEL_BINS, "all bins are used");
// A key's bin among the fine ones; SEL_FINE_BINS or more where it is in none.
constexpr uint32_t sel_fine_bin(uint32_t key) { return (key - SEL_KEY_FINE) >> SEL_FINE_SHIFT; }
// Any key's bin: of three lines through two corners, of which the fine one is the steepest, the middle one.  No branches.
constexpr uint32_t sel_top_bin(uint32_t key) {
    constexpr uint32_t first = SEL_KEY_FIRST >> SEL_FINE_SHIFT, last = (SEL_KEY_END >> SEL_FINE_SHIFT) - 1u;
    constexpr uint32_t zero = (SEL_KEY_FINE >> SEL_FINE_SHIFT) - SEL_BIN_FINE;
    constexpr uint32_t below_0 = (SEL_KEY_FINE >> SEL_FINE_SHIFT) - (SEL_KEY_FINE >> SEL_WIDE_SHIFT);
    constexpr uint32_t above_0 = (SEL_KEY_ABOVE >> SEL_FINE_SHIFT) - (SEL_KEY_ABOVE >> SEL_WIDE_SHIFT);
    const uint32_t raised = (key >> SEL_FINE_SHIFT) < first ? first : key >> SEL_FINE_SHIFT, fine = raised < last ? raised : last;
    const uint32_t wide = fine >> (SEL_WIDE_SHIFT - SEL_FINE_SHIFT), below = wide + below_0, above = wide + above_0;
    const uint32_t low = fine > below ? fine : below;
    return (low < above ? low : above) - zero;
}
// First key of a bin (zeros are in none), and the bits of a window that is a whole bin: those at both ends span up to 2^30
// keys.
constexpr uint32_t sel_bin_first_key(uint32_t bin) {
    return bin == 0u ? 1u
         : bin < SEL_BIN_FINE ? SEL_KEY_FIRST + (bin << SEL_WIDE_SHIFT)
         : bin < SEL_BIN_ABOVE ? SEL_KEY_FINE + ((bin - SEL_BIN_FINE) << SEL_FINE_SHIFT)
                               : SEL_KEY_ABOVE + ((bin - SEL_BIN_ABOVE) << SEL_WIDE_SHIFT);
}
constexpr bool sel_bin_is_fine(uint32_t bin) { return bin >= SEL_BIN_FINE && bin < SEL_BIN_ABOVE; }
constexpr uint32_t sel_bin_width(uint32_t bin) {
    return bin == 0u || bin == SEL_BINS - 1u ? SEL_MAX_WIDTH
         : 32u + (sel_bin_is_fine(bin) ? SEL_FINE_SHIFT : SEL_WIDE_SHIFT);
}

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
