// Sizes of the rectangles in which the portfolio rebuild takes a source tensor (gather_rect_kernel).  Plain C++: the
// host and the test that holds them to their limits share it.
#pragma once

#include <stdint.h>

namespace shifter {

constexpr uint32_t RECT_ELEMS = 8192;    // floats of a rectangle staged in LDS, rows rounded up to RECT_ROW
constexpr uint32_t RECT_ROW = 128;
constexpr uint32_t RECT_BAND = 64;       // most rows (filters) of one
// A network of up to this many weights is cut into rectangles of a quarter of that: whole ones are too few to keep 256
// compute units busy.  us a step of ten variants, whole / quarters: 12 k weights 82.8 / 82.6, 61 k 91.7 / 87.2, 0.18 M 96.4 / 90.3,
// 0.24 M 94.0 / 87.7, 0.4 M 100.1 / 91.3, 0.44 M 95.0 / 90.6; 0.93 M 100.0 / 102.5, 3.7 M 144 / 153, 8.1 M 197 / 219.
constexpr double RECT_FEW_WEIGHTS = 524288.0;
// But for at least this many weights a rectangle takes more rows: those that are short are rounded up, and a block each for
// a few dozen weights costs more than it spreads.  us a step of ten variants, whole / quarters / now: 1x1 layers of 3 and 2000
// filters in turn, 0.48 M weights, 140 / 177 / 137; of 16 and 900, 0.39 M, 111 / 108 / 102; 160000 filters of one weight 402 / 485 / 401.
constexpr uint32_t RECT_LEAST = 1024;

// Rows of a rectangle whose rows hold `row` weights, in a network of `weights`.
constexpr uint32_t rect_rows(double weights, uint32_t row) {
    const uint32_t padded = (row + RECT_ROW - 1u) / RECT_ROW * RECT_ROW, wide = padded ? padded : RECT_ROW;
    const uint32_t whole = RECT_ELEMS / wide, quarter = RECT_ELEMS / 4u / wide, least = row ? RECT_LEAST / row : RECT_BAND;
    uint32_t rows = whole;
    if (weights <= RECT_FEW_WEIGHTS) rows = quarter > least ? quarter : (least < whole ? least : whole);
    return rows == 0u ? 1u : (rows < RECT_BAND ? rows : RECT_BAND);
}

}  // namespace shifter
