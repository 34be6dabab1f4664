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

// The gathered chain through a window of the image in LDS: bytes of a work-group at rank R whose window has `pixels` pixels (two
// slabs of 64 columns of the factor; 64 channels of each pixel, eight pixels at a time, and of a row of zeros).
inline int64_t window_lds_bytes(int R, int64_t pixels) { return 2 * R * 128 + ((pixels + 7) / 8 * 8 + 1) * 128; }
constexpr int kMaxWindow = 256;                          // 16-byte pieces that 256 threads load, eight each
// Two work-groups have to share the 160 KB of a compute unit.  At R = 192 they do up to 248 pixels (forward of 60 x 60, 250 pixels, r = 192, 64800
// rows, through the window / gathered, us: C = 64 35 / 30, 128 50 / 43, 192 66 / 57; 59 x 59, 248 pixels: 26 / 30, 39 / 42, 55 / 57).
inline bool window_fits(int R, int64_t pixels) { return pixels <= kMaxWindow && 2 * window_lds_bytes(R, pixels) <= 160 * 1024; }

}  // namespace abt
