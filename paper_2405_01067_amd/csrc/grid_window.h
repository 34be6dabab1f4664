// Host arithmetic behind the 32-bit offsets of the gathered kernels (plain C++, no device code).
#pragma once

#include <stdint.h>

namespace abt {

// Rows are the pixels of a grid RH x RW per image; row (image, y, x) stands for pixel (mul y, mul x) of an image of
// H x W pixels.  The number of pixels from the first to the last pixel that `rows` consecutive rows stand for, whole
// grid lines included (from x = 0 of the first line to x = RW - 1 of the last): the largest over all rows to start from.
inline int64_t grid_window(int64_t rows, int64_t RH, int64_t RW, int64_t mul, int64_t H, int64_t W) {
    if (rows < 1 || RH < 1 || RW < 1) return 0;
    const int64_t steps = (rows + RW - 2) / RW;              // line to line, from the first row's line to the last row's
    // a step within an image is mul lines of the image, one to the next image H - mul (RH - 1): more than mul where the
    // grid leaves lines out (one parity of an odd height), fewer where mul RH exceeds H
    const int64_t extra = H - mul * RH;
    const int64_t crossings = extra > 0 ? (steps + RH - 1) / RH : steps / RH;
    return (steps * mul + crossings * extra) * W + mul * (RW - 1) + 1;
}

}  // namespace abt
