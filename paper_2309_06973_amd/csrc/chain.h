// Rules of the chained offsets of the encoder's segments (codec.hip): what a chunk's block
// makes of its predecessors' words, and what it leaves behind.  Plain C++: the kernel and the
// test that plays every order of events share it.
#pragma once

#include <stdint.h>

namespace shifter {

// A link's word (a link is what one block encodes: one chunk, or two where blocks take pairs; "chunk"
// below means a link): 0 nothing yet, bits 62-63 = 1 the size of its segments alone, 2 the size of all
// segments up to and including them, 3 its wait ran out.
constexpr uint64_t CHAIN_VALUE = (1ull << 62) - 1ull;
constexpr uint64_t chain_size(uint32_t c, uint64_t size) { return ((c == 0 ? 2ull : 1ull) << 62) | size; }
constexpr uint64_t CHAIN_BROKEN = 3ull << 62;
// The call's outcome in its result words: bytes, status, and whether some chunk's wait ran out.
enum : uint32_t { CHAIN_BYTES = 0, CHAIN_STATUS = 1, CHAIN_BROKE = 2 };

// The walk back over a chunk's predecessors, 64 words at a time, to the nearest one whose sum is known.
struct ChainWalk {
    int64_t last;           // nearest predecessor not added yet; below 0: all are
    uint64_t sum = 0;
    uint32_t polls = 0;
    bool broken = false;
    constexpr explicit ChainWalk(uint32_t c) : last((int64_t)c - 1) {}
    constexpr bool waits() const { return last >= 0 && !broken; }
    // One look at the words last, last - 1, ... (bit 0, bit 1, ...; those before the first chunk are
    // known sums of nothing): which hold a sum, which hold anything, which are broken.  Returns
    // the words whose values are to be added; none: look again.
    constexpr uint64_t look(uint64_t known, uint64_t here, uint64_t bad, uint32_t limit) {
        if (bad != 0ull || ++polls > limit) { broken = true; return 0; }
        const uint64_t nearest = known & (~known + 1ull);
        const uint64_t need = known ? (nearest << 1) - 1ull : ~0ull;
        if ((here & need) != need) return 0;
        last = known ? -1 : last - 64;
        return need;
    }
};

// What a chunk's block leaves when its walk has ended.  Every block whose wait ran out says so in a
// result word that nothing but the next call clears: blocks behind it may have added its size
// before, the last one among them, and end with a sum as if nothing had happened.
template <class Put>
constexpr void chain_leave(const ChainWalk& walk, uint32_t c, bool is_last, uint64_t size, uint64_t* word, uint64_t* result,
                           Put&& put) {
    if (walk.broken) {
        put(word, CHAIN_BROKEN);
        put(result + CHAIN_BROKE, 1ull);
    } else if (c != 0) {
        put(word, (2ull << 62) | (walk.sum + size));
    }
    if (is_last) {
        put(result + CHAIN_BYTES, walk.sum + size);
        put(result + CHAIN_STATUS, 0ull);
    }
}

}  // namespace shifter
