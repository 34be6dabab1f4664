// C ABI of the library: argument validation, workspace carving and the launch sequences.
// Every operation is documented in include/abtrain.h.
#include <atomic>
#include <cmath>
#include <initializer_list>
#include <new>
#include <vector>

#include "common.h"

using namespace abt;

namespace {

std::atomic<int> g_max_sweeps{30};

// Chain kernel choice: one launch of few_fwd_kernel where few_rows says so, two products where wide_products or two_products do; else the narrow-rank kernel where use_narrow / narrow_gather do; else
// by choose_chain_shape work-groups of 128 rows (r = 32, 64, 96, 128, and 192 to 384 in the kernel of eight equal waves; from an image 192 and
// 384 too) or of 64 rows with loader and MFMA waves (r = 32, 64, 96, 128, 160, 192, 256, 320, 384).
std::atomic<int> g_chain_rows{0};    // 0: automatic; 64 or 128: force that work-group height where the rank allows it
std::atomic<int> g_chain_parts{0};   // 0: automatic; n: force n column parts for 128-row work-groups

// Launch shape of the chain kernel.  Measured on gfx950 (forward of configs 2 and 3 and four other
// shapes): a 128-row work-group takes 1.58 times as long as a 64-row one on the same factors (its
// LDS traffic per slab, not its loaders, sets the pace), so it only pays through the rounds the
// grid needs on the 256 compute units: 4 rounds of 64-row work-groups against 2 of 128-row ones at
// M = 50432 (148 -> 127 us), 2 against 1 at M = 25216.  Column parts (several work-groups per row
// block) never paid in those measurements and are only used when forced.
struct ChainShape { int rows, parts; };

ChainShape choose_chain_shape(int64_t M, int p, int q, int R, bool second_stage, bool allow_parts) {
    const ChainShape small{64, 1};
    const int rows_forced = g_chain_rows.load(), parts_forced = g_chain_parts.load();
    if (!chain2_tall_supports(R, p, q) || (rows_forced == 64 && chain2_supports(R, p, q))) return small;
    int parts = 1;
    if (allow_parts && second_stage && parts_forced > 1) {
        const int ntile = (int)ceil_div(q, 128);
        parts = parts_forced < ntile ? parts_forced : ntile;
    }
    if (rows_forced == 128 || !chain2_supports(R, p, q)) return ChainShape{128, parts};
    const double cost64 = (double)ceil_div(ceil_div(M, 64), 256);
    const double cost128 = 1.58 * (double)ceil_div(ceil_div(M, 128) * parts, 256);
    return cost128 < cost64 ? ChainShape{128, parts} : small;
}

// Work-groups per row block of the narrow-rank kernel: as many as find an idle compute unit, while one more
// saves a tenth of the slabs (each repeats the p / 64 slabs of stage 1).
int narrow_parts(int64_t row_blocks, int p, int q, bool second_stage) {
    if (!second_stage) return 1;
    const int ns1 = p / 64, ntile = q / 64;
    int best = 1;
    for (int parts = 2; parts <= ntile && row_blocks * parts <= 256; ++parts) {
        const int now = ns1 + (ntile + best - 1) / best, then = ns1 + (ntile + parts - 1) / parts;
        if (10 * then <= 9 * now) best = parts;
    }
    return best;
}
// Rows per work-group of the narrow-rank kernel: the smallest whole number of work-groups per compute unit with at
// most 128 rows each, and the rows shared out evenly among them (39597 rows as 512 work-groups of 80 rows instead of
// 310 of 128: 82 us instead of 89, 69 instead of 75, at 3072 x 768, r = 96).  A small batch keeps 128 rows: its
// row blocks are shared by output tiles instead.
int narrow_rows(int64_t M) {
    if (M <= 8192) return 128;
    const int64_t per_cu = ceil_div(M, 256 * 128);
    return (int)(ceil_div(ceil_div(M, 256 * per_cu), 4) * 4);
}
// Where the narrow-rank kernel is taken for a matrix operand (times of a forward in us, this kernel / the better of the
// others, inputs not in the last-level cache):
//   At most 8192 rows: its work-groups can share a row block's output tiles, the more of them the better, so p <= q.
//     768 -> 3072: 197 rows 12 / 25 at r = 96, 18 / 30 at r = 192; 6304 rows 24 / 32, 33 / 38.  With 2 p <= q it pays
//     at any rank, until the p / 64 slabs that each of them repeats are too many (2048 -> 4096, 8192 rows: 48 / 41 at
//     r = 128, 59 / 48 at r = 192; 1536 -> 3072, 8000 rows, r = 32: 29 / 30, but T alone 4 us the slower).  Below that
//     only at r <= 96 (768 -> 768, r = 192: 19 / 15): 768 -> 768 with 197 rows 12 / 13 at r = 96, 8 / 10 at r = 32; with 8192
//     rows 18 / 19, 15 / 14; 1536 -> 1536 with 8192 rows 29 / 28, 27 / 25 at r = 64, 25 / 22 at r = 32.
//   8192 to 32768 rows: one work-group alone on a compute unit waits for its loads (12608 rows, r = 96: 44 / 28, 45 / 36,
//     23 / 20).  Only at r = 160, where the others have 64-row work-groups: 17000 rows, 3072 -> 768 60 / 85, 768 -> 768
//     29 / 41, but 768 -> 3072 59 / 47, from 45000 rows on 106 / 107; 3072 -> 3072 103 / 94, but 25000 rows 100 / 117.
//   More than 32768 rows, at least two work-groups per compute unit, r <= 128.  768 -> 3072 / 3072 -> 768 / 768 -> 768
//     with 39597 rows: r = 64 66 / 68, 79 / 89, 33 / 46; r = 96 68 / 76, 82 / 95, 34 / 44.  With 100864 rows: r = 64
//     164 / 176, 168 / 176; r = 96 186 / 175, 179 / 194 and, 1536 -> 1536, 155 / 146: not for the widest layers there.
//     r = 128, where the others are better at long contractions and wide outputs: 33000 rows 82 / 69, 88 / 114, 42 / 56,
//     3072 -> 3072 137 / 132; 65536 rows 120 / 115, 124 / 118, 50 / 52.  r = 32 only with p >= q: 50432 rows 91 / 86,
//     75 / 80, 31 / 36.  (r = 192, 100000 rows: 241 / 213, 246 / 226, 104 / 100.)
// (The rule does not ask for the second stage: a T that the backward computes again comes from the same kernel.)
bool use_narrow(int64_t rows, int p, int q, int R) {
    if (g_chain_rows.load() != 0 || g_chain_parts.load() != 0 || !chain4_supports(R, p, q)) return false;
    if (rows <= 8192) {
        if (2 * p <= q) return p <= 768 || rows <= 4096 || (p <= 1536 && R >= 96);
        if (p > q || R > 96) return false;
        if (p <= 512 || (R == 96 && rows <= 2048)) return true;
        return p <= 1024 && rows <= (R == 32 ? 1024 : R == 64 ? 4096 : 8192);
    }
    if (R == 160) return rows > 16384 && (q <= 1536 || rows > 45056 || (p >= q && rows > 24576));
    if (rows <= 32768) return false;
    switch (R) {
        case 32: return p >= q;
        case 64: return true;
        case 96: return rows <= 65536 || q <= 1024 || p + q < 3072;
        case 128: return p >= q ? p <= 1024 || (rows <= 49152 && q <= 1536) : q <= 1024;
        default: return false;
    }
}

// Columns of T per work-group where only T is wanted: nothing shares a row block's output tiles then, and at wide ranks
// a slab of the whole P takes longer than the other kernels' loaders (T of 197 rows, p = 1536, r = 192, and dA: 36 us,
// 22 with 32 columns each, 26 in the other kernels; p = 768, r = 96: 18.6, 16.2, 18.8).  The sums of a column do not change.
int narrow_cols(int n, int64_t row_blocks, int R) {
    for (int c : {32, 64, 96})
        if (R % c == 0 && n * (R / c) <= kChainMaxGroups && row_blocks * (R / c) <= 256) return c;
    return R;
}

// Runs n problems of one shape, all with a second stage or none, in the narrow-rank kernel if the rule above says so for `of`
// problems (n, or the groups of a call of which n compute T again: the order of the sums is then that of the forward).
// Work-groups that share a row block all read its rows of Xin, and the first of them to finish writes: not with an output
// over Xin (the other kernels have one reader per row block, which reads before it writes).
bool narrow_chain(const ChainProblem* problems, int n, int of, int64_t M, int p, int q, int R, hipStream_t s, hipError_t* e) {
    if (!use_narrow(of * M, p, q, R)) return false;
    const bool second = problems[0].Yout != nullptr;
    const int rows = narrow_rows(of * M);
    const int64_t blocks = n * ceil_div(M, rows);
    const int parts = narrow_parts(blocks, p, q, second);
    int cols = second || n * M > 8192 ? R : narrow_cols(n, blocks, R);
    bool in_place = false;
    for (int g = 0; g < n; ++g)
        in_place |= overlap(problems[g].Xin, M * p * 2, problems[g].Yout, M * q * 2) ||
                    overlap(problems[g].Xin, M * p * 2, problems[g].Tout, M * R * 2);
    if (in_place && parts > 1) return false;
    if (in_place) cols = R;
    ChainProblem share[kChainMaxGroups];
    int k = 0;
    for (int g = 0; g < n; ++g) {
        const ChainProblem& c = problems[g];
        share[k++] = c;
        for (int c0 = cols; c0 < R; c0 += cols)
            share[k++] = ChainProblem{c.Xin, (const char*)c.P + (size_t)c0 * p * 2, nullptr, nullptr, (char*)c.Tout + (size_t)c0 * 2};
    }
    *e = launch_chain4_bf16(share, k, M, p, q, cols, R, rows, parts, s);
    return true;
}

// Where the chain runs as two products, T and then Y (lr_small.hip), by the rows of all problems together.  Forward, us, the fused kernels /
// two products.
//   Too few row blocks for the chip, rows up to 4096, and 8192 where the fused kernel's row block takes longest (r = 256; above where Y is the wide
//   side; from an image):
//                               197 rows     4000         8192                                197 rows     4000       8192
//     768 -> 2304   r = 32     8.2 / 7.1   14.0 / 14.3                3072 -> 768  r = 96   19.3 / 10.5   22 / 17   24 / 25
//                   r = 96    11.7 / 7.3   16.3 / 15.4  20.4 / 23.2                r = 192               31 / 22   31 / 33
//                   r = 192                  24 / 21      28 / 26                  r = 256                         36 / 35
//                   r = 384   37.7 / 9.1     39 / 25      42 / 39                  r = 320                         42 / 47
//     768 -> 3072   r = 320                               46 / 42                  r = 384    39 / 12    43 / 33   48 / 48
//     3 x 3 on 14 x 14 x 256: r = 64 3920 rows 23 / 13, 8036 23 / 14, 12544 24 / 20;  r = 192 26 / 13, 27 / 25, 28 / 35.
//   Not where the fused kernel is soon done, since a second launch costs the host 3.5 us: limits on the rank and on p r that fall with the rows.
//     Forward and backward together, fused / two products:
//     768 -> 2304  197 rows   r = 32 25.8 / 29.6, r = 96 26.6 / 30.4, r = 128 30.3 / 30.2 (p r = 98304), r = 192 33.0 / 30.2 (147456)
//                  2000 rows  r = 64 34 / 33, r = 96 37.6 / 35.3 (73728), r = 128 40 / 34
//     3072 -> 768  197 rows   r = 32 25 / 30, r = 64 27 / 30, r = 96 30 / 30, r = 128 34 / 30
//                  2000 rows  r = 32 32 / 30 (98304), r = 64 35 / 30
//     Above r = 192 the fused kernel takes long at any size but the smallest (forward, 64 -> 64, r = 384 10.7 / 7.6; 64 -> 1920, r = 256 25 / 7).
//   Not for many rows of a short contraction and a very wide Y, which one work-group per row block writes from a T that it has at once:
//     1088 -> 16320, 4096 rows, r = 96 43 / 48;  640 -> 8832, 8108 rows, r = 256 103 / 108;  384 -> 10432, 4096 rows, r = 96 23.5 / 23.1
//     (1984 -> 15040, 4096 rows, r = 128 61 / 53;  832 -> 15808, 2048 rows, r = 128 36 / 31;  64 -> 16384, 4096 rows, r = 384 185 / 88).
//   r = 224, 288 and 352, whose fused kernel is that of the next wider rank in 128-row work-groups, up to 10240 rows:
//                             3000 rows   8192      12608     16384
//     768 -> 2304  r = 224     45 / 20   45 / 31   48 / 44   48 / 54
//     3072 -> 768  r = 352     70 / 32   71 / 48   73 / 74   76 / 78
//     64 -> 1920   r = 288     39 / 17   40 / 29   41 / 39   39 / 46
bool two_products(int64_t rows, int p, int q, int R, bool image) {
    if (g_chain_rows.load() != 0 || g_chain_parts.load() != 0) return false;
    const int64_t least = image ? (rows >= 2048 ? 36864 : rows >= 1024 ? 73728 : 147456) : (rows >= 2048 ? 73728 : rows >= 1024 ? 98304 : 147456);
    const bool small = R > 192 ? p + q >= 1024 : (int64_t)p * R >= least && (image || R >= 96 || rows >= 1024);
    const bool wide = R == 256 || (R > 256 && q >= 2 * p);
    const bool padded = R == 224 || R == 288 || R == 352;
    if (!padded && !image && R <= 256 && rows > 2048 && q > 8192 && q >= 8 * p) return false;
    return small && rows <= (padded ? 10240 : image || wide ? 8192 : 4096);
}
// Where the chain runs as the two products for many rows (lr_pair.hip), by the rows of all problems together.  Forward, us, the other kernels /
// these, on a card that keeps what fits in the last-level cache between the calls:
//   More than 32768 rows, where the fused kernels' 128-row work-groups need a second round:
//                          r = 64         r = 96         r = 128        r = 192         r = 384
//     768 -> 3072  36000   58.1 / 57.9    66.9 / 57.2    73.7 / 57.6    89.5 / 65.0     133 / 115
//                  50432   80.0 / 77.4    82.2 / 77.8    95.4 / 75.8    116 / 82.4      176 / 154
//     3072 -> 768  36000                  72.0 / 56.2    87.2 / 62.0    99.0 / 78.1     155 / 126
//                  50432                  91.0 / 75.0    97.6 / 79.6    107 / 95.2      175 / 157
//     768 -> 768   36000                  32.5 / 28.9                   49.8 / 37.3     66.7 / 56.3
//     Narrow ranks and layers gain least, and lose below the limits here (64 -> 1600, 57148 rows, r = 96 44.9 / 48.1; 1472 -> 832, 37521 rows, r = 96
//     41.0 / 45.5).  The more rows the last round of the fused work-groups has, the less there is to gain, and nothing for a narrow result, whose T is
//     read for few columns each: beyond 49152 rows from 768 columns on (1024 -> 640, 50460 rows, r = 256 57 / 62; r = 160, with its rounds of 16384 rows,
//     beyond 40960 too: 320 -> 640, 47971 rows 27 / 31), beyond 57344 only at ranks up to 192, from 1088 columns on and not where the last round is
//     all but full (768 -> 3072, 150000 rows, r = 96 240 / 217; 2816 -> 1984, 92516 rows, r = 256 251 / 290; 1920 -> 384, 61160 rows, r = 192 74 / 82),
//     and up to r = 224 where a third round has just begun (65537 to 73728 rows: 0.98 to 1.54 times as fast).
//   r = 288 and 352 above 10752 rows, where the fused kernel is that of the next wider rank in 128-row work-groups (768 -> 3072, 12000
//     rows, r = 288 72.6 / 41.2; even with it from 16384 on; not r = 352 into few columns: 1152 -> 128, 13406 rows 29 / 32); r = 160, whose fused
//     kernel has 64-row work-groups (768 -> 3072, 25000 rows 62.7 / 44.4), until a second round of those is three fifths full (1280 -> 640, 30343 rows 33 / 36).
//   Wide results of short contractions, where a fused work-group's time is the stores of Y (768 -> 3072, r = 192): 4608 to 10240 rows (6000
//     rows 31.1 / 23.3), 16384 to 22528 (20000 rows 52.8 / 40.6) and, at r = 160 and 192, up to 12800 (12608 rows 32.0 / 30.7; over 116
//     shapes 0.98 to 1.18 times as fast, mean 1.06).  Above that one round of 64-row work-groups fills the chip (14500 rows, r = 160 33.5 / 34.6,
//     r = 128 28.7 / 33.4).  Of contractions so short that X and P are soon there a second launch is the longer way (256 -> 2496, 7237 rows, r = 64
//     14.9 / 16.5; 256 -> 1536, 6018 rows, r = 160 14.8 / 16.2; 384 -> 1408, 22481 rows, r = 320 38 / 41), sooner at one rank than at another.
//   Forwards of 8800 shapes inside these limits: 1.2 times as fast in the mean, 1 in 280 of them more than 3 % slower, 0.84 at worst; of 3100 outside
//   that went this way up to wider limits, 1 in 8 were.
//   The two lower limits lie 512 rows above those of the products for few rows (4096 and 10240): next to these a forward asks for no place for T,
//   as before.
//   Groups share launches of 64- or 128-row work-groups that split no tail and have no form of eight equal waves, so that they gain more: of 800 calls
//   outside the limits for one problem 577 are more than 3 % faster as two products (8 x 2255 rows, 320 -> 2112, r = 160 52.9 / 29.4), 64 slower, of these most
//   below 8192 rows, which keep them, and at r = 224, 256, 352 and 384 where a third round is full to more than a half (5 x 17187 rows, 1472 -> 1792, r = 256 177 / 214).
bool wide_products(int64_t rows, int p, int q, int R, bool groups) {
    if (g_chain_rows.load() != 0 || g_chain_parts.load() != 0 || rows <= 4608 || p < 256 || q < 128) return false;
    if (rows > 32768) {
        const int64_t last = (rows - 1) % 32768 + 1;      // rows of the last round
        if (R >= 160) {
            if (rows > 114688 || p + q < (rows <= 49152 ? 704 : 1536)) return false;
            if (groups) return R == 160 || R == 192 || R == 288 || R == 320 || rows <= 81920 || rows > 98304;
            if (rows <= 49152) return (R != 224 || p + q >= 960) && (R != 160 || rows <= 40960 || q >= 768);
            if (rows <= 57344) return q >= 768;
            if (rows > 65536 && rows <= 73728 && R <= 224) return true;
            return R <= 192 && last <= 28672 && q >= 1088;
        }
        if (R == 128) return rows <= 49152 ? p >= 1024 || q > 1024 : p + q >= 3072 && (groups || q >= 768 || last <= 24576);
        if (R == 96) return q >= 2304 || (p >= 3072 && (groups || q >= 512)) ||
                            (rows <= 40960 && p >= 512 && q >= 512 && p + q >= 1280 && (groups || q >= 1024 || p <= 1024));
        return R == 64 && q >= 2304 && (groups || p <= q);
    }
    if ((R == 288 || R == 352) && rows > 10752 && rows <= 16384) return p + q >= 1280 && (groups || R == 288 || q >= 640);
    if (R == 160 && rows > 16384) return q >= 512 && p + q >= 1472 && (groups || (rows <= 26624 && p >= 576));
    if (rows <= 8192 && R >= 96 && R <= 192) return q >= 1024 && p <= 1920 && p >= (R == 128 ? 256 : R == 96 ? 320 : 384);
    if (rows <= 10240)
        return q >= 1344 && q >= 2 * p && (R == 64 ? p >= 640 || (groups && rows > 8192) : R == 288 ? groups || rows > 5632 : R >= 96 && R <= 192);
    if (rows <= 12800) return (R == 160 || (R == 192 && (groups || p >= 640))) && q >= 2304 && q >= 2 * p;
    return rows > 16384 && rows <= 22528 && R >= 64 && q >= 1344 && 2 * q >= 5 * p && (groups || p >= 512 || R == 384);
}
// Where a few rows go through both products in one launch whose work-groups make the rows of T themselves (lr_few.hip), a round of work-groups of
// 32 rows and 256 columns of Y (128 above r = 96).  Forward, GPU time in us, the other kernels / this one:
//                             1 row        197         512          1024         2048
//     768 -> 2304   r = 32   7.7 / 3.5   8.0 / 4.1   8.2 / 4.3    8.5 / 6.0   10.5 / 8.8
//                   r = 96    11 / 5.4    12 / 5.9    12 / 6.2   12.2 / 11.0                  (288 work-groups)
//                   r = 128   14 / 6.2    15 / 6.6  14.6 / 12.2                               (288 work-groups)
//                   r = 192  7.0 / 7.6   7.7 / 8.3   8.4 / 15.7                               (two launches / one; 288 work-groups)
//     3072 -> 768   r = 32    13 / 5.3    14 / 5.8    14 / 5.9     10 / 6.2     11 / 7.3
//                   r = 64    16 / 7.4    16 / 7.9    17 / 8.1     10 / 8.4    11.5 / 10
//                   r = 96   9.6 / 9.1  10.3 / 9.7  10.5 / 9.9                               (two launches / one)
//     64 -> 64      r = 64   4.3 / 2.7   4.6 / 3.0   4.7 / 3.0    4.7 / 3.1    4.7 / 3.1
// Over 300 shapes of 16 to 4096 rows 1.4 times as fast in the mean, none slower.  T alone at r = 32 and 64, a work-group per 32 rows, is as fast as the two
// products' (a backward of T again and dA, 3072 -> 64: r = 32 1024 rows 16.2 / 14.4, 4096 rows 26.7 / 26.3; r = 64 16.5 / 16.1, 29.7 / 29.4).  From r = 96 on, and from an image, not where two_products holds: T alone, which shares its
// contraction among more work-groups there, took up to 1.4 us longer (3072 columns, r = 96, 10.7 -> 12.1 with dA).
// From an image over 165 layers and batches 1.5 times as fast in the mean, none slower: 28 x 28 x 128, stride 2, r = 32, 3 images 14.6 / 5.5;
// 7 x 7 x 64, r = 160, 9 images 19.7 / 7.7.
// Groups of a call, each with factors of its own, over 450 shapes 1.47 times as fast in the mean: four of 40 rows, 640 -> 768, r = 160 15.9 / 6.6; where
// two_products holds they stay with it at any rank (eight of 197 rows, 3072 -> 768, r = 64 12.7 / 13.6).
// At r = 32 two work-groups share a compute unit (768 -> 3072, 1024 rows 8.7 / 6.4; 3072 -> 768, 3200 rows 12.4 / 11.9).
bool few_rows(int G, int64_t M, int p, int q, int R, bool image) {
    const int64_t rows = G * M;
    if (g_chain_rows.load() != 0 || g_chain_parts.load() != 0 || rows > 4096 || p > 3072 || R > 192) return false;
    const int64_t groups = G * ceil_div(M, 32) * ceil_div(q, R <= 96 ? 256 : 128);
    return groups <= (R == 32 ? 512 : 256) && ((R <= 64 && !image && G == 1) || !two_products(rows, p, q, R, image));
}
// Several work-groups read the rows of X and the factors: no output may lie over them.
bool no_output_over(const ChainProblem& c, int64_t x_bytes, int64_t M, int p, int q, int R) {
    const void* out[2] = {c.Yout, c.Tout};
    const int64_t bytes[2] = {M * q * 2, M * R * 2};
    for (int i = 0; i < 2; ++i)
        if (overlap(out[i], bytes[i], c.Xin, x_bytes) || overlap(out[i], bytes[i], c.P, (int64_t)R * p * 2) || overlap(out[i], bytes[i], c.Q, (int64_t)q * R * 2))
            return false;
    return true;
}
// (n of the G problems of a call: the rule is that of all of them)
bool few_rows(const ChainProblem* problems, int n, int G, int64_t M, int p, int q, int R) {
    if (!few_rows(G, M, p, q, R, false) || !few_supports(M, p, q, R)) return false;
    for (int g = 0; g < n; ++g)
        if (!no_output_over(problems[g], M * p * 2, M, p, q, R)) return false;
    return true;
}
// T needs a place, and not over the first operand, whose rows several work-groups read.
bool place_for_T(const ChainProblem* problems, int n, int64_t M, int p, int R) {
    for (int g = 0; g < n; ++g)
        if (!problems[g].Tout || overlap(problems[g].Xin, M * p * 2, problems[g].Tout, M * R * 2)) return false;
    return true;
}
bool two_products(const ChainProblem* problems, int n, int of, int64_t M, int p, int q, int R) {
    if (!two_products(of * M, p, q, R, false) || !lr_small_supports(M, q, p, R)) return false;
    return place_for_T(problems, n, M, p, R);
}
// Does a forward of these rows go faster with a place for T?
bool place_pays(int64_t rows, int64_t M, int p, int q, int R) {
    if (few_rows((int)(rows / M), M, p, q, R, false) && few_supports(M, p, q, R)) return false;
    return (wide_products(rows, p, q, R, rows > M) && pair_supports(M, p, q, R)) || (two_products(rows, p, q, R, false) && lr_small_supports(M, q, p, R));
}

// From an image: a lane has one pixel for the whole kernel, while the loader waves of the other kernels compute
// a range check per 16 bytes.  Forward, us, this kernel / the better of the others, r = 64: 56 x 56 x 64
// (200704 rows) 50 / 110, 28 x 28 x 128 (50176 rows) 29 / 43; with few row blocks the other kernels' deeper prefetch
// wins back (14 x 14 x 256, 12544 rows: 28 / 26, r = 192 45 / 32) except where the patches are strided
// (28 x 28 x 128, stride 2: 17 / 20; r = 192 27 / 24) and not too many for one row block (7 x 7 x 512, 3 x 3, stride 2,
// r = 96: 1 image 42 / 38, 4 images 43 / 44; r = 64 34 / 35).
// Through a window in LDS (stride 1) also for few rows at r <= 64, where one block of channels keeps the order of the sums that the plain
// kernels have on an explicit patch matrix (56 x 56 x 64, batch 1 17 / 15; with more blocks it would be 23 / 20 for 14 x 14 x 256,
// batch 1 to 32, at r = 128 26 / 29).
bool narrow_gather(int64_t row_blocks, bool window, int mul, int p, int q, int R) {
    if (g_chain_rows.load() != 0 || g_chain_parts.load() != 0 || !chain4_supports(R, p, q)) return false;
    return (window && R <= 64) || row_blocks > 128 || (mul == 2 && (R <= 64 || (R == 96 && (p <= 4096 || row_blocks > 1))));
}

// the gathered chain (factored convolution): same choice of work-group height, no column parts
hipError_t chain_gather(const void* image, const PatchGeom& g, const void* P, const void* Q, void* Yout, void* Tout,
                        int t_pitch, int64_t M, int q, int R, hipStream_t s) {
    const int p = g.kh * g.kw * ((g.Cin + 63) / 64) * 64;
    if (Tout && t_pitch == R && two_products(M, p, q, R, true) && lr_small_gather_supports(g, M, q, R) &&
        !overlap(image, (M / (g.RH * g.RW)) * g.H * g.W * g.Cin * 2, Tout, M * R * 2))
        return launch_lr_small_fwd_gather(image, g, P, Q, Yout, Tout, M, q, R, s);
    const ChainProblem c{image, P, Q, Yout, Tout};
    if ((!Tout || t_pitch == R) && few_rows(1, M, p, q, R, true) && few_gather_supports(g, M, q, R) &&
        no_output_over(c, (M / ((int64_t)g.RH * g.RW)) * g.H * g.W * g.Cin * 2, M, p, q, R))
        return launch_few_fwd_gather(c, g, M, q, R, s);
    const ChainGather cg{g.H, g.W, g.Cin, 0, g.kh, g.kw, g.sign, g.kh / 2, g.kw / 2, g.RH, g.RW, g.mul, 1, 0, 0, g.RH, g.RW};
    if (g.sign > 0 && narrow_gather(ceil_div(M, 128), g.Cin <= 64 && chain4_window(cg, R, narrow_rows(M)), g.mul, p, q, R)) {
        const GatherProblem one{image, P, Q, Yout, Tout, M, cg};
        const hipError_t e = launch_chain4_gather_bf16(&one, 1, q, R, t_pitch, narrow_rows(M), narrow_parts(ceil_div(M, narrow_rows(M)), p, q, Yout != nullptr), s);
        if (e != hipErrorInvalidValue) return e;
        (void)hipGetLastError();
    }
    const ChainShape sh = choose_chain_shape(M, p, q, R, Yout != nullptr, false);
    if (sh.rows == 128) {
        // the tall launcher checks the image window of a 128-row block before it launches anything and
        // reports an invalid value when it does not fit 32-bit offsets: take the 64-row kernel then
        const hipError_t e = launch_chain2_tall_gather_bf16(image, g, P, Q, Yout, Tout, t_pitch, M, q, R, s);
        if (e != hipErrorInvalidValue) return e;
        (void)hipGetLastError();
    }
    return launch_chain2_gather_bf16(image, g, P, Q, Yout, Tout, t_pitch, M, q, R, s);
}

hipError_t chain(const void* Xin, const void* P, const void* Q, void* Yout, void* Tout,
                 int64_t M, int p, int q, int R, hipStream_t s) {
    const ChainProblem one{Xin, P, Q, Yout, Tout};
    if (wide_products(M, p, q, R, false) && pair_supports(M, p, q, R) && place_for_T(&one, 1, M, p, R))
        return launch_pair_bf16(&one, 1, 1, M, p, q, R, s);
    if (few_rows(&one, 1, 1, M, p, q, R)) return launch_few_fwd(&one, 1, M, p, q, R, s);
    if (two_products(&one, 1, 1, M, p, q, R)) return launch_lr_small_fwd(&one, 1, 1, M, p, q, R, s);
    hipError_t e;
    if (narrow_chain(&one, 1, 1, M, p, q, R, s, &e)) return e;
    const ChainShape sh = choose_chain_shape(M, p, q, R, Yout != nullptr, true);
    if (sh.rows == 128) return launch_chain2_tall_bf16(Xin, P, Q, Yout, Tout, M, p, q, R, sh.parts, s);
    return launch_chain2_bf16(Xin, P, Q, Yout, Tout, M, p, q, R, s);
}

// The entry points promise not to throw: what the host-side tables of a call may throw (allocation
// failure of a std::vector) becomes a status.
template <class F>
int guarded(F&& f) {
    try { return f(); }
    catch (const std::bad_alloc&) { return ABT_ENOMEM; }
    catch (...) { return ABT_EHIP; }
}
template <class F>
size_t guarded_size(F&& f) {
    try { return f(); }
    catch (...) { return 0; }
}

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline size_t esize(int dt) { return dt == ABT_BF16 ? 2 : 4; }

int check_lr_shapes(int64_t M, int64_t m, int64_t n, int64_t r, int dt) {
    if (dt != ABT_F32 && dt != ABT_BF16) return ABT_EDTYPE;
    if (M < 1 || m < 1 || n < 1 || r < 1) return ABT_ESHAPE;
    if (M > 0x7fffffff || m > 0x7fffffff || n > 0x7fffffff || r > 0x7fffffff) return ABT_ESHAPE;
    if (dt == ABT_BF16) {
        if (m % 64 || n % 64 || r % 32 || r > 384) return ABT_ESHAPE;
        if (m > (1 << 20) || n > (1 << 20)) return ABT_ESHAPE;   // 32-bit byte offsets inside row blocks
    }
    return ABT_OK;
}

GemmF32 gemm(const float* A, const float* B, float* C, int64_t P, int64_t Q, int64_t K,
             int64_t lda, int64_t ldb, int64_t ldc, int tA, int tB, int acc) {
    GemmF32 g{};
    g.A = A; g.B = B; g.C = C; g.P = (int)P; g.Q = (int)Q; g.K = (int)K;
    g.lda = (int)lda; g.ldb = (int)ldb; g.ldc = (int)ldc;
    g.transA = tA; g.transB = tB; g.accumulate = acc; g.alpha = 1.0f;
    return g;
}

// The smallest fp32 layers go in one launch each way, in which no output may lie over what another work-group reads.
struct Place { const void* at; int64_t count; };
bool tiny_f32(int64_t M, int64_t m, int64_t n, int64_t r, std::initializer_list<Place> in, std::initializer_list<Place> out) {
    if (!tiny_f32_supports(M, m, n, r)) return false;
    for (const Place& o : out)
        for (const Place& i : in)
            if (overlap(o.at, o.count * 4, i.at, i.count * 4)) return false;
    return true;
}

// fp32 backward: dT, T (each M x r) and the partial sums of the factor gradients, whose contraction over
// the batch is split over work-groups.  `limit`: in the static scratch array the split only takes what dT and T
// leave of it, so that every shape that fits without one is served; a workspace of the caller's has room for the
// split that fills the chip (whole backward, 256 x 256, r = 256, 32768 rows: 285 us; 783 without a split).  The partial sums of dT
// itself, where its contraction is split too, are added before the others come, in the same place.  T again is not split: its sums are the forward's.
struct BwdLayoutF32 { size_t dT, T, partials, total; int split_dT, split_A, split_B; };

GemmF32 grad_A_f32(const float* dY, const float* T, float* dA, int64_t M, int64_t m, int64_t r, int acc) {
    return gemm(dY, T, dA, m, r, M, m, r, r, 1, 0, acc);
}
GemmF32 grad_B_f32(const float* dT, const float* X, float* dB, int64_t M, int64_t n, int64_t r, int acc) {
    return gemm(dT, X, dB, r, n, M, r, n, n, 1, 0, acc);
}

BwdLayoutF32 bwd_layout_f32(int64_t M, int64_t m, int64_t n, int64_t r, size_t limit) {
    BwdLayoutF32 w{};
    const size_t each = align_up((size_t)M * r * 4, 256);
    w.dT = 0; w.T = each; w.partials = 2 * each;
    const GemmF32 a = grad_A_f32(nullptr, nullptr, nullptr, M, m, r, 0), b = grad_B_f32(nullptr, nullptr, nullptr, M, n, r, 0);
    w.split_A = gemm_f32_splits(a);
    w.split_B = gemm_f32_splits(b);
    const GemmF32 d = gemm(nullptr, nullptr, nullptr, M, r, m, m, r, r, 0, 0, 0);
    w.split_dT = gemm_f32_row_splits(d);
    // (a shape that the static array serves: no further than that has room for, so that dX has the same bits in either call)
    const size_t room = w.partials <= ABT_STATIC_SCRATCH_BYTES ? ABT_STATIC_SCRATCH_BYTES : limit;
    while (w.partials + gemm_f32_partial_bytes(d, w.split_dT) > room && w.split_dT > 1) w.split_dT /= 2;
    auto bytes = [&] { return gemm_f32_partial_bytes(a, w.split_A) + gemm_f32_partial_bytes(b, w.split_B); };
    while (w.partials + bytes() > limit && (w.split_A > 1 || w.split_B > 1)) {
        w.split_A = w.split_A > 1 ? w.split_A / 2 : 1;
        w.split_B = w.split_B > 1 ? w.split_B / 2 : 1;
    }
    const size_t first = gemm_f32_partial_bytes(d, w.split_dT), second = bytes();
    w.total = w.partials + (first > second ? first : second);
    return w;
}

struct BwdLayout {  // bf16 backward workspace
    size_t At, Bt, dT, T, partials, total;
};

BwdLayout bwd_layout_bf16(int64_t M, int64_t m, int64_t n, int64_t r) {
    BwdLayout w{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    w.At = take((size_t)r * m * 2);
    w.Bt = take((size_t)n * r * 2);
    w.dT = take((size_t)M * r * 2);
    w.T = take((size_t)M * r * 2);
    // the split count depends on which gradients are requested: size for the worst subset
    TnJob jobs[2] = {{nullptr, nullptr, nullptr, (int)m, 0}, {nullptr, nullptr, nullptr, (int)n, 1}};
    size_t part = tn_partials_bytes(M, jobs, 2, (int)r);
    const size_t only_a = tn_partials_bytes(M, jobs, 1, (int)r), only_b = tn_partials_bytes(M, jobs + 1, 1, (int)r);
    if (only_a > part) part = only_a;
    if (only_b > part) part = only_b;
    w.partials = take(part);
    w.total = off;
    return w;
}

// what a backward needs if it may use `limit` bytes at most (more than that: it does not fit)
size_t bwd_bytes(int64_t M, int64_t m, int64_t n, int64_t r, int dt, size_t limit) {
    return dt == ABT_F32 ? bwd_layout_f32(M, m, n, r, limit).total : bwd_layout_bf16(M, m, n, r).total;
}

int check_merge_layer(const abt_merge_desc& d) {
    if (!d.A_copies || !d.B_copies || !d.A_out || !d.B_out || !d.S_out || !d.k_out) return ABT_EINVAL;
    if (d.G < 1 || (d.mode != 0 && d.mode != 1)) return ABT_EINVAL;
    if (!(d.tau >= 0.0f && d.tau <= 1.0f) || d.k_fixed < 0) return ABT_EINVAL;
    if (d.m < 1 || d.n < 1 || d.k < 1 || d.k_cap < 1) return ABT_ESHAPE;
    if (d.k % 32) return ABT_ESHAPE;
    const int64_t K = d.mode == 0 ? d.k : d.k * d.G;
    if (K > 2048 || d.m > 0x7fffffff || d.n > 0x7fffffff || d.k_cap > 0x7fffffff) return ABT_ESHAPE;
    for (int g = 0; g < d.G; ++g) {
        if (!d.A_copies[g] || !d.B_copies[g]) return ABT_EINVAL;
        if (!aligned(d.A_copies[g], 16) || !aligned(d.B_copies[g], 16)) return ABT_EALIGN;
    }
    if (!aligned(d.A_out, 16) || !aligned(d.B_out, 16) || !aligned(d.S_out, 4) || !aligned(d.k_out, 4))
        return ABT_EALIGN;
    if (d.W_out && !aligned(d.W_out, 16)) return ABT_EALIGN;
    return ABT_OK;
}

// Backward of few rows: all gradients come from one launch, and a factor gradient over something that it reads (kOver) has to wait for its end.
enum SmallBwd { kNotSmall, kSmall, kOver };

// Runs `launch(dA, dB, accumulate)`; kOver: into `part` (room for both), from where the gradients then go to their places.
template <class F>
hipError_t few_gradients(SmallBwd few, float* dA, float* dB, int64_t m, int64_t n, int64_t r, int acc, float* part, hipStream_t s, F&& launch) {
    if (few == kSmall) return launch(dA, dB, acc);
    const hipError_t e = launch(dA ? part : nullptr, dB ? part + (dA ? m * r : 0) : nullptr, 0);
    if (e != hipSuccess) return e;
    TnJob done[2];
    int nd = 0;
    if (dA) done[nd++] = TnJob{nullptr, nullptr, dA, (int)m, 0};
    if (dB) done[nd++] = TnJob{nullptr, nullptr, dB, (int)n, 1};
    return launch_tn_finish(done, nd, (int)r, acc, part, s);
}

}  // namespace

extern "C" {

const char* abt_status_string(int status) {
    switch (status) {
        case ABT_OK: return "ABT_OK";
        case ABT_EINVAL: return "ABT_EINVAL: invalid argument";
        case ABT_ESHAPE: return "ABT_ESHAPE: unsupported shape";
        case ABT_EALIGN: return "ABT_EALIGN: misaligned pointer";
        case ABT_EWORKSPACE: return "ABT_EWORKSPACE: workspace missing or too small";
        case ABT_EDTYPE: return "ABT_EDTYPE: unknown dtype";
        case ABT_ENOCONV: return "ABT_ENOCONV: Jacobi sweep cap reached";
        case ABT_EHIP: return "ABT_EHIP: HIP runtime error";
        case ABT_ENOMEM: return "ABT_ENOMEM: host memory allocation failed";
        case ABT_ETOOLARGE: return "ABT_ETOOLARGE: shape needs more than the static scratch array";
        default: return "unknown abt_status";
    }
}

namespace {

// output grid of a convolution with zero padding kh/2, kw/2 and stride s: ceil(H / s) x ceil(W / s)
inline int64_t conv_out(int64_t extent, int stride) { return (extent + stride - 1) / stride; }
inline int64_t conv_rows(const abt_conv_geom& g) { return g.N * conv_out(g.H, g.stride) * conv_out(g.W, g.stride); }
// the three gathers of a factored convolution
PatchGeom conv_patches_geom(const abt_conv_geom& g) {        // rows = output pixels, image = act
    return PatchGeom{(int)g.H, (int)g.W, (int)g.C, g.kh, g.kw, +1,
                     (int)conv_out(g.H, g.stride), (int)conv_out(g.W, g.stride), g.stride, 0};
}
ConvShape conv_shape(const abt_conv_geom& g) {
    return ConvShape{(int)g.N, (int)g.H, (int)g.W, (int)conv_out(g.H, g.stride), (int)conv_out(g.W, g.stride), (int)g.C, g.kh, g.kw, g.stride};
}
PatchGeom conv_adjoint_geom(const abt_conv_geom& g, int r) {  // rows = input pixels, image = dT on the output grid
    return PatchGeom{(int)conv_out(g.H, g.stride), (int)conv_out(g.W, g.stride), r, g.kh, g.kw, -1,
                     (int)g.H, (int)g.W, 1, g.stride == 2 ? 1 : 0};
}

int check_conv(const abt_conv_geom* g, int64_t m, int64_t r, int dt) {
    if (!g) return ABT_EINVAL;
    if (dt != ABT_BF16) return ABT_EDTYPE;
    if (g->stride != 1 && g->stride != 2) return ABT_ESHAPE;
    if (g->N < 1 || g->H < 1 || g->W < 1 || g->C < 1 || m < 1 || r < 1 || g->kh < 1 || g->kw < 1) return ABT_ESHAPE;
    if (!(g->kh & 1) || !(g->kw & 1) || g->kh > 15 || g->kw > 15) return ABT_ESHAPE;
    if (g->C % 64 || m % 64 || r % 32 || r > 384 || r == 224 || r == 288 || r == 352) return ABT_ESHAPE;
    if (g->H > (1 << 20) || g->W > (1 << 20) || g->C > (1 << 20) || m > (1 << 20)) return ABT_ESHAPE;
    if ((int64_t)g->kh * g->kw * g->C > (1 << 20)) return ABT_ESHAPE;
    if (g->N > 0x7fffffff / (g->H * g->W)) return ABT_ESHAPE;     // pixel count fits an int
    // the window of the image that one 128-row block's patches touch is addressed with 32-bit offsets
    // (the launchers check their own windows again, with the exact geometry)
    if (((int64_t)g->stride * g->stride * (128 + 2 * g->W + 2) + 2 * g->stride * g->W +
         2 * ((g->kh / 2) * g->W + g->kw / 2)) * g->C * 2 >= kBufMaxBytes)
        return ABT_ESHAPE;
    return ABT_OK;
}

// A 1 x 1 window with stride 1: the patch matrix is the activation itself, and the layer a linear one on N H W rows.
inline bool is_linear(const abt_conv_geom& g) { return g.kh == 1 && g.kw == 1 && g.stride == 1; }

// T = patches(act) B^T, Y = T A^T (Y NULL: T alone).  A linear layer goes to its kernels, which read whole lines, but for the
// ranks whose gathered form has more work-groups per compute unit than the other at large batches (forward, us, as a matrix /
// gathered: 28 x 28 x 512, r = 192, batch 256 101 / 91, 128 55 / 51; 56 x 56 x 256, r = 128, batch 128 79 / 79, r = 192 117 / 106;
// below: 14 x 14 x 1024, batch 256, r = 128 32 / 33, r = 192 40 / 42; 7 x 7 x 2048, r = 64 18 / 25; 28 x 28 x 512, r = 256 110 / 179).
bool as_matrix(const abt_conv_geom& g, int64_t M, int64_t r) { return is_linear(g) && !(M > 65536 && r > 96 && r <= 192); }
hipError_t conv_chain(const void* act, const abt_conv_geom& g, const void* A, const void* B, void* Y, void* T, int64_t m, int64_t r,
                      hipStream_t s) {
    const int64_t M = conv_rows(g);
    if (as_matrix(g, M, r)) return chain(act, B, A, Y, T, M, (int)g.C, (int)m, (int)r, s);
    return chain_gather(act, conv_patches_geom(g), B, A, Y, T, (int)r, M, (int)m, (int)r, s);
}

// Where the two launches for few rows (lr_small.hip) are the faster backward.  us, the other kernels / these, m x n, r:
//   2304 x 768    r = 96, 1 row 27 / 13, 197 rows 29 / 15, 1000 rows 35 / 18
//   768 x 3072    r = 32, 197 rows 17 / 10, 4000 rows 34 / 25
//   64 x 64       r = 96, 197 rows 16 / 9, 2000 rows 22 / 15, 4000 rows 21 / 22: the smallest layers up to 2048 rows
// Their products take no operand through LDS, so with many of them the others win, the more so where those run as two products.
// dY is read twice, for dT and for dA, so m counts three halves of n; fewer gradients leave room for more rows:
//   3072 x 768    4096 rows r = 192 51 / 52, r = 256 56 / 61, r = 384 76 / 87;  2500 rows r = 320 55 / 59
//   1024 x 4096   4096 rows r = 192 55 / 57, r = 384 79 / 98
//   1920 x 1920   3000 rows r = 192 45 / 44, r = 256 50 / 54;  4096 rows r = 320 67 / 81
//   4096 x 4096   2048 rows r = 384 80 / 97, 4096 rows 114 / 170;  4096 rows r = 96 59 / 58
//   dX and dA     768 x 3072, 4055 rows, r = 352 and T again 83 / 76;  3072 x 768, r = 384 2491 rows 57 / 60, 4096 rows 71 / 83
//   dX and dB     2304 x 768, 3066 rows, r = 384 54 / 47;  768 x 3072, 4055 rows, r = 352 64 / 69
// Wide dX of a short contraction, stored in 4-byte pieces, where the rank makes it more than latency:
//   64 x 16384    1024 rows r = 96 34 / 37, r = 192 43 / 55;  64 x 8192, 2048 rows r = 192 37 / 29
// dT, one work-group per 32 rows and 64 columns, whose eight waves share out all of m:
//   8192 x 2048   197 rows r = 96 34 / 41, r = 384 46 / 56;  6464 x 1664, 161 rows r = 96 29 / 32
// but where dT would otherwise come from the fused kernel (few rows at r = 32 and 64), longer by one that waits for less:
//   8192 x 512    197 rows r = 64 40 / 32;  16384 x 64 r = 32 48 / 60;  8320 x 7232, 175 rows r = 32 64 / 34
bool few_rows(int64_t M, int64_t m, int64_t n, int64_t r, bool dA, bool dB) {
    if (M > (m + n >= 1024 ? 4096 : 2048)) return false;
    if (M * r * ((dA ? 30 : 24) * m + (!dB ? 10 : dA ? 20 : 19) * n) > 85000000000ll) return false;
    if (r >= 96 && n >= 16 * m && M * n * r > 2500000000ll) return false;
    if (m > 7168 && (r >= 96 || M >= 1024 || (m > (r == 32 ? 8192 : 12288) && 2 * n < m))) return false;
    return lr_small_supports(M, (int)m, (int)n, (int)r);
}
SmallBwd small_bwd(const void* dY, const void* X, const void* T, const void* B, const void* dX, const void* dA, const void* dB,
                   int64_t M, int64_t m, int64_t n, int64_t r) {
    if (g_chain_rows.load() != 0 || g_chain_parts.load() != 0) return kNotSmall;
    if (!few_rows(M, m, n, r, dA != nullptr, dB != nullptr)) return kNotSmall;
    auto over = [&](const void* out, int64_t bytes) {
        return (dA && (overlap(out, bytes, dY, M * m * 2) || overlap(out, bytes, T, M * r * 2))) || (dB && overlap(out, bytes, X, M * n * 2)) ||
               (dX && overlap(out, bytes, B, r * n * 2));
    };
    if (over(dX, M * n * 2)) return kNotSmall;
    return over(dA, m * r * 4) || over(dB, r * n * 4) ? kOver : kSmall;
}

// Where they are the faster backward of a convolution.  us, the other kernels / these; side x side x C, window, r:
//   14 x 14 x 256, 3 x 3            r = 64, 1 image 27 / 9, 980 rows 38 / 12, 3920 49 / 23, 8036 45 / 38, 12544 49 / 57;  r = 256, 980 rows 66 / 21
//   7 x 7 x 512, 3 x 3              r = 64, 8183 rows 54 / 47;  r = 128 67 / 72;  r = 256, 4067 rows 93 / 68, 5978 rows 91 / 93;  r = 384, 4067 rows 95 / 95
//   28 x 28 x 128, 3 x 3, stride 2  r = 256, 8036 rows 75 / 56
// Always up to 2048 rows.  Beyond, as many products, a patch matrix of many columns (read again for every 64 ranks) and an activation of
// many pixels (dAct in 4-byte pieces, less of the whole at wide ranks) go to the others:
//   31 x 31 x 2944, 3 x 3           r = 256, 3844 rows 231 / 342       53 x 53 x 1536, 3 x 3    r = 384, 2809 rows 160 / 205
//   60 x 60 x 1344, 3 x 3           r = 128, 3600 rows 71 / 83         11 x 11 x 1024, 3 x 3    r = 256, 1936 rows 88 / 67
//   14 x 14 x 1024, 1 x 1, stride 2 r = 32, 4067 rows 57 / 64, r = 192 73 / 73
//   7 x 7 x 2048, 1 x 1, stride 2   r = 64, 2992 rows 87 / 75, 4096 rows 88 / 98;  r = 256, 16 rows 87 / 10, 4096 rows 125 / 121, 6000 rows 142 / 169
// From 4096 rows on only few of each, and of the products with A (57 x 57 x 320, 3 x 3, m = 1728, r = 160, 6498 rows: 74 / 79).
bool few_pixels(const abt_conv_geom& g, int64_t M, int64_t m, int64_t r) {
    const int64_t n = (int64_t)g.kh * g.kw * g.C, pixels = (int64_t)g.N * g.H * g.W * g.C;
    if (M > 8192) return false;
    if (M > 4096) {
        if (pixels > (4 << 20) || M * n * r > 3500000000ll || M * m > 10000000) return false;
    } else if (M > 2048) {
        if (M * n * r > 7500000000ll || M * n > 40000000 || M * pixels > (r >= 256 ? 110000000000ll : 60000000000ll)) return false;
    }
    return lr_small_conv_supports(conv_shape(g), M, (int)m, (int)r);
}
SmallBwd small_conv_bwd(const abt_conv_geom& g, const void* dY, const void* act, const void* T, const void* B, const void* dAct, const void* dA,
                        const void* dB, int64_t M, int64_t m, int64_t r) {
    if (g_chain_rows.load() != 0 || g_chain_parts.load() != 0 || !few_pixels(g, M, m, r)) return kNotSmall;
    const int64_t n = (int64_t)g.kh * g.kw * g.C, image = (int64_t)g.N * g.H * g.W * g.C * 2;
    auto over = [&](const void* out, int64_t bytes) {
        return (dA && (overlap(out, bytes, dY, M * m * 2) || overlap(out, bytes, T, M * r * 2))) || (dB && overlap(out, bytes, act, image)) ||
               (dAct && overlap(out, bytes, B, r * n * 2));
    };
    if (over(dAct, image)) return kNotSmall;
    return over(dA, m * r * 4) || over(dB, r * n * 4) ? kOver : kSmall;
}

int linear_bwd(const void* dY, const void* X, const void* T, const void* A, const void* B,
               void* dX, float* dA, float* dB,
               int64_t M, int64_t m, int64_t n, int64_t r, int dt, int accumulate,
               void* workspace, size_t workspace_bytes, size_t limit, void* stream);

// column block of the activation gradient computed per launch: the widest supported tile that divides C
int conv_dact_chunk(int64_t C) {
    static const int sizes[] = {384, 320, 256, 192, 160, 128, 96, 64};
    for (int v : sizes) if (C % v == 0) return v;
    return 64;
}

struct ConvBwdLayout { size_t At, dT, T, Pst, partials, total; int r_pad; };

ConvBwdLayout conv_bwd_layout(const abt_conv_geom& g, int64_t m, int64_t r) {
    ConvBwdLayout w{};
    const int64_t M = conv_rows(g), taps = (int64_t)g.kh * g.kw;     // rows of Y, T, dY, dT
    if (is_linear(g)) {
        const BwdLayout l = bwd_layout_bf16(M, m, g.C, r);
        w.T = l.T;
        w.total = l.total;
        return w;
    }
    w.r_pad = (int)((r + 63) / 64 * 64);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    w.At = take((size_t)r * m * 2);
    w.dT = take((size_t)M * r * 2);
    w.T = take((size_t)M * r * 2);
    w.Pst = take((size_t)g.C * taps * w.r_pad * 2);
    const TnJob ja{nullptr, nullptr, nullptr, (int)m, 0}, jb{nullptr, nullptr, nullptr, (int)(taps * g.C), 1};
    const TnJob both[2] = {ja, jb};
    const size_t pa = tn_partials_bytes(M, &ja, 1, (int)r), pb = tn_partials_bytes(M, &jb, 1, (int)r, true);
    const size_t pab = tn_partials_bytes(M, both, 2, (int)r, true);
    w.partials = take(pa > pb ? (pa > pab ? pa : pab) : (pb > pab ? pb : pab));
    w.total = off;
    return w;
}

// Where the narrow-rank kernel computes the activation gradient (a product without a second stage, one launch for all
// parities and blocks of output channels; gradient of the activation alone, us, this kernel / the others): with stride
// 2, for its parities; where the others take a launch per block of channels (14 x 14 x 1024, 1 x 1, r = 64, batch 1 to
// 128: 17 / 42 to 41 / 86; 7 x 7 x 512, 3 x 3: 22 / 34); for a single slab (1 x 1, r <= 64: 17 / 18); and for large batches
// (28 x 28 x 128, r = 64: 32 images 26 / 28, 128 images 53 / 83). With few row blocks and one launch on both sides the
// others' deeper prefetch wins: 28 x 28 x 128, 16 images 24 / 23, r = 384 58 / 50; 27 x 27 x 192, 32 images, r = 192 45 / 43.
// Through a window in LDS always, with blocks of 64 channels while those find idle compute units (narrow_dact_chunk): 14 x 14 x 256,
// batch 1 to 32, r = 64 23 / 24, r = 128 24 / 29, r = 192 28 / 36; 28 x 28 x 128, batch 8 23 / 23, 24 / 27, 29 / 33.
bool narrow_dact(const abt_conv_geom& g, int p, bool window) {
    if (g_chain_rows.load() != 0 || g_chain_parts.load() != 0 || !chain4_supports(64, p, 64)) return false;
    return window || g.stride == 2 || g.C > conv_dact_chunk(g.C) || p == 64 || ceil_div(g.N * g.H * g.W, 128) > 192;
}

// Output channels per work-group there: 64 where all of those fit one launch and the compute units (a wider block: 14 x 14 x 256, batch 8, r = 128
// 29 us, 24 with 64; 7 x 7 x 512, batch 64, r = 192 42 / 36; not with more: 28 x 28 x 128, batch 32, r = 128 31 / 34).
int narrow_dact_chunk(const abt_conv_geom& g) {
    const int64_t parts = g.C / 64;
    if (parts * (g.stride == 2 ? 4 : 1) <= kChainMaxGroups && parts * ceil_div(g.N * g.H * g.W, 128) <= 256) return 64;
    for (int v : {192, 160, 128, 96}) if (g.C % v == 0) return v;
    return 64;
}

ChainGather dact_gather(const abt_conv_geom& g, int r) {
    return ChainGather{(int)conv_out(g.H, g.stride), (int)conv_out(g.W, g.stride), r, 0, g.kh, g.kw, -1, g.kh / 2, g.kw / 2,
                       (int)g.H, (int)g.W, 1, 1, 0, 0, (int)g.H, (int)g.W};
}

// dAct[q, c] = sum over taps and j of dT[(q - shift(tap)) / stride, j] B[j, tap, c] (only where the division
// is exact): the same gathered product as the forward, on the image dT [N, H', W', r] with mirrored
// shifts, against the re-laid-out factor Pst; rows are the input pixels.
// With stride 2 a tap reaches only the pixels of one parity, so the pixels are taken parity by
// parity, each with its own taps: 2.25 instead of 9 taps per pixel for a 3 x 3 window.  All parities and blocks
// of output channels go into one launch (whole backward, us, against the kernel for all taps, batch 64, r = 64:
// 28 x 28 x 128 stride 2 56 / 75, stride 1 75 / 91; 56 x 56 x 64 stride 2 79 / 179; 7 x 7 x 2048 1 x 1 48 / 101).
// Pst: B laid out for it, by parity if `narrow` and stride 2.
hipError_t conv_dact(const void* dT, const void* B, void* dAct, void* Pst, const abt_conv_geom& g, int r, int r_pad, bool narrow, hipStream_t s) {
    const int C = (int)g.C, taps = g.kh * g.kw;
    const int64_t M_in = g.N * g.H * g.W;
    hipError_t e;
    if (narrow) {
        const bool by_parity = g.stride == 2;
        const int chunk = narrow_dact_chunk(g);
        const ChainGather whole = dact_gather(g, r);
        GatherProblem pr[kChainMaxGroups];
        int n = 0;
        bool wide = false;                       // a window that 32-bit offsets do not cover: the kernels below check again
        for (int cls = by_parity ? 3 : 0; cls >= 0 && !wide; --cls) {      // most taps first
            const int py = cls >> 1, px = cls & 1;
            ChainGather cg = whole;
            int64_t before = 0;
            if (by_parity) {
                const int ny = parity_count(g.kh, py), nx = parity_count(g.kw, px), ny0 = parity_count(g.kh, 0), nx0 = parity_count(g.kw, 0);
                before = (py ? ny0 * g.kw : 0) + (px ? ny * nx0 : 0);
                cg.kh = ny; cg.kw = nx;
                cg.cy = (py - parity_first(g.kh, py) + g.kh / 2) / 2; cg.cx = (px - parity_first(g.kw, px) + g.kw / 2) / 2;
                cg.RH = ((int)g.H - py + 1) / 2; cg.RW = ((int)g.W - px + 1) / 2;
                cg.omul = 2; cg.oy = py; cg.ox = px;
                if (ny * nx == 0) { cg.H = 0; cg.kh = cg.kw = 1; cg.cy = cg.cx = 0; before = 0; }     // no tap: zeros
            }
            const int64_t pitch = (int64_t)cg.kh * cg.kw * r_pad, M = g.N * cg.RH * cg.RW;
            for (int c0 = 0; c0 < C && !wide; c0 += chunk) {
                pr[n++] = GatherProblem{dT, (const char*)Pst + ((before * C) * r_pad + (int64_t)c0 * pitch) * 2, nullptr, nullptr,
                                        (char*)dAct + (size_t)c0 * 2, M, cg};
                if (n == kChainMaxGroups || (cls == 0 && c0 + chunk >= C)) {
                    e = launch_chain4_gather_bf16(pr, n, 64, chunk, C, 128, 1, s);
                    if (e == hipErrorInvalidValue) { (void)hipGetLastError(); wide = true; break; }
                    if (e != hipSuccess) return e;
                    n = 0;
                }
            }
        }
        if (!wide) return hipSuccess;
    }
    if (narrow && g.stride == 2) {               // laid out by parity
        e = launch_conv_factors_bf16(nullptr, nullptr, 64, B, Pst, r, C, g.kh, g.kw, r_pad, false, s);
        if (e != hipSuccess) return e;
    }
    const PatchGeom adj = conv_adjoint_geom(g, r);
    const int chunk = conv_dact_chunk(C);        // one launch per block of output channels
    const int64_t pst_pitch = (int64_t)taps * r_pad;
    for (int64_t c0 = 0; c0 < C; c0 += chunk) {
        e = chain_gather(dT, adj, (const char*)Pst + (size_t)c0 * pst_pitch * 2, nullptr, nullptr, (char*)dAct + c0 * 2, C, M_in, 64, chunk, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

size_t lr_conv_bwd_workspace_bytes(const abt_conv_geom* geom, int64_t m, int64_t r, int dt) {
    if (check_conv(geom, m, r, dt) != ABT_OK) return 0;
    return conv_bwd_layout(*geom, m, r).total;
}

int lr_conv_fwd_wants_T(const abt_conv_geom* geom, int64_t m, int64_t r, int dt) {
    if (check_conv(geom, m, r, dt) != ABT_OK) return 0;
    const abt_conv_geom& g = *geom;
    const int64_t M = conv_rows(g);
    if (as_matrix(g, M, r)) return place_pays(M, M, (int)g.C, (int)m, (int)r);
    return two_products(M, g.kh * g.kw * (int)g.C, (int)m, (int)r, true) && lr_small_gather_supports(conv_patches_geom(g), M, (int)m, (int)r);
}

int lr_conv_fwd(const void* act, const void* A, const void* B, void* Y, void* T_save,
                const abt_conv_geom* geom, int64_t m, int64_t r, int dt, void* stream) {
    int st = check_conv(geom, m, r, dt);
    if (st != ABT_OK) return st;
    if (!act || !A || !B || !Y) return ABT_EINVAL;
    if (!aligned(act, 16) || !aligned(A, 16) || !aligned(B, 16) || !aligned(Y, 16) || !aligned(T_save, 16))
        return ABT_EALIGN;
    return conv_chain(act, *geom, A, B, Y, T_save, m, r, (hipStream_t)stream) == hipSuccess ? ABT_OK : ABT_EHIP;
}

int lr_conv_bwd(const void* dY, const void* act, const void* T, const void* A, const void* B,
                void* dAct, float* dA, float* dB,
                const abt_conv_geom* geom, int64_t m, int64_t r, int dt, int accumulate,
                void* workspace, size_t workspace_bytes, void* stream) {
    int st = check_conv(geom, m, r, dt);
    if (st != ABT_OK) return st;
    if (!dY || !act || !A || !B) return ABT_EINVAL;
    if (!aligned(dY, 16) || !aligned(act, 16) || !aligned(T, 16) || !aligned(A, 16) || !aligned(B, 16) ||
        !aligned(dAct, 16) || !aligned(dA, 16) || !aligned(dB, 16))
        return ABT_EALIGN;
    const abt_conv_geom& g = *geom;
    const ConvBwdLayout w = conv_bwd_layout(g, m, r);
    if (!workspace || workspace_bytes < w.total) return ABT_EWORKSPACE;
    if (!aligned(workspace, 256)) return ABT_EALIGN;
    if (!dAct && !dA && !dB) return ABT_OK;
    hipStream_t s = (hipStream_t)stream;
    char* ws = (char*)workspace;
    const int64_t M = conv_rows(g);     // output pixels (rows of dY, T, dT)
    const int taps = g.kh * g.kw;
    const int acc = accumulate ? 1 : 0;
    const PatchGeom fwd_geom = conv_patches_geom(g);
    void* dT = ws + w.dT;
    const void* Tp = T;
    if (!Tp && dA) {   // recompute T = patches(act) B^T (first stage of the chain only)
        if (conv_chain(act, g, nullptr, B, nullptr, ws + w.T, m, r, s) != hipSuccess) return ABT_EHIP;
        Tp = ws + w.T;
    }
    // as a linear layer (backward, us, gathered before / now: 7 x 7 x 2048, m = 512, r = 64, batch 256 69 / 48, batch 1 34 / 27; 14 x 14 x
    // 1024, m = 256, batch 128 60 / 46; 56 x 56 x 256, m = 128, batch 128 198 / 142, r = 256 406 / 271)
    if (is_linear(g)) return linear_bwd(dY, act, Tp, A, B, dAct, dA, dB, M, m, g.C, r, dt, accumulate, workspace, workspace_bytes, SIZE_MAX, stream);
    // few rows: two launches, as for the linear layer (the same bits as on an explicit patch matrix)
    const SmallBwd few = small_conv_bwd(g, dY, act, Tp, B, dAct, dA, dB, M, m, r);
    if (few != kNotSmall) {
        if ((dAct || dB) && launch_lr_small_dt(dY, A, dT, M, (int)m, (int)r, s) != hipSuccess) return ABT_EHIP;
        const int64_t n = (int64_t)taps * g.C;
        return few_gradients(few, dA, dB, m, n, r, acc, (float*)(ws + w.partials), s, [&](float* dA_to, float* dB_to, int add) {
                   return launch_lr_small_conv_grad(conv_shape(g), dY, act, Tp, B, dAct, dA_to, dB_to, dT, M, (int)m, (int)r, add, s);
               }) == hipSuccess ? ABT_OK : ABT_EHIP;
    }
    const bool narrow = dAct && narrow_dact(g, taps * w.r_pad, g.stride == 1 && chain4_window(dact_gather(g, (int)r), narrow_dact_chunk(g), 128));
    if (dAct || dB) {
        // dT = dY A = dY (A^T)^T: first stage of the plain chain on the transposed factor
        if (launch_conv_factors_bf16(A, ws + w.At, (int)m, dAct ? B : nullptr, ws + w.Pst, (int)r, (int)g.C, g.kh, g.kw, w.r_pad, narrow && g.stride == 2, s) !=
            hipSuccess)
            return ABT_EHIP;
        if (chain(dY, ws + w.At, nullptr, nullptr, dT, M, (int)m, 64, (int)r, s) != hipSuccess) return ABT_EHIP;
    }
    if (dAct) {
        const hipError_t e = conv_dact(dT, B, dAct, ws + w.Pst, g, (int)r, w.r_pad, narrow, s);
        if (e != hipSuccess) return ABT_EHIP;
    }
    // factor gradients: dA = dY^T T (plain) and dB = patches(act)^T dT (gathered), one launch
    TnJob jobs[2];
    int nj = 0;
    if (dA) jobs[nj++] = TnJob{dY, Tp, dA, (int)m, 0};
    if (dB) jobs[nj++] = TnJob{act, dT, dB, taps * (int)g.C, 1};
    if (dB) {
        if (launch_tn_gather_bf16(jobs, nj, fwd_geom, M, (int)r, acc, (float*)(ws + w.partials), s) != hipSuccess) return ABT_EHIP;
    } else if (nj) {
        if (launch_tn_bf16(jobs, 1, M, (int)r, acc, (float*)(ws + w.partials), s) != hipSuccess) return ABT_EHIP;
    }
    return ABT_OK;
}

int ab_adamw_step(const abt_adamw_tensor* tensors, int n, int64_t step,
                  double lr, double lr_scale, double beta1, double beta2, double eps,
                  double weight_decay, void* stream) {
    if (n < 0 || (n > 0 && !tensors) || step < 1) return ABT_EINVAL;
    if (!std::isfinite(lr) || !std::isfinite(lr_scale) || !std::isfinite(eps) || !std::isfinite(weight_decay) ||
        !(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || eps < 0.0)
        return ABT_EINVAL;
    return guarded([&]() -> int {
    std::vector<AdamwTensor> v;
    v.reserve((size_t)n);
    for (int i = 0; i < n; ++i) {
        const abt_adamw_tensor& t = tensors[i];
        if (t.count < 0) return ABT_ESHAPE;
        if (t.count == 0) continue;
        if (!t.param || !t.grad || !t.exp_avg || !t.exp_avg_sq) return ABT_EINVAL;
        if (!aligned(t.param, 16) || !aligned(t.grad, 16) || !aligned(t.exp_avg, 16) ||
            !aligned(t.exp_avg_sq, 16) || !aligned(t.param_bf16, 16))
            return ABT_EALIGN;
        v.push_back(AdamwTensor{t.param, t.grad, t.exp_avg, t.exp_avg_sq, (uint16_t*)t.param_bf16, t.count});
    }
    if (v.empty()) return ABT_OK;
    AdamwHyper h;
    const double b1 = beta1, b2 = beta2;
    h.beta1 = (float)beta1; h.beta2 = (float)beta2;
    h.one_minus_beta1 = (float)(1.0 - b1); h.one_minus_beta2 = (float)(1.0 - b2);
    // 1 - beta^step, without cancellation when beta^step is close to 1
    const double bc1 = b1 > 0.0 ? -std::expm1((double)step * std::log(b1)) : 1.0;
    const double bc2 = b2 > 0.0 ? -std::expm1((double)step * std::log(b2)) : 1.0;
    h.inv_bc1 = (float)(1.0 / bc1);
    h.inv_sqrt_bc2 = (float)(1.0 / std::sqrt(bc2));
    h.eps = (float)eps; h.eta = (float)(lr * lr_scale); h.weight_decay = (float)weight_decay;
    return launch_adamw(v.data(), (int)v.size(), h, (hipStream_t)stream) == hipSuccess ? ABT_OK : ABT_EHIP;
    });
}

double ab_lr_rebound_scale(int64_t i, int64_t rebound_steps) {
    if (rebound_steps <= 0) return 1.0;
    if (i < 0) i = 0;
    if (i + 1 >= rebound_steps) return 1.0;
    return (double)(i + 1) / (double)rebound_steps;
}

int ab_reconstruct(const float* A, const float* B, float* W,
                   int64_t m, int64_t n, int64_t k, void* stream) {
    if (!A || !B || !W) return ABT_EINVAL;
    if (m < 1 || n < 1 || k < 1 || m > INT32_MAX || n > INT32_MAX || k > INT32_MAX) return ABT_ESHAPE;
    if (!aligned(A, 16) || !aligned(B, 16) || !aligned(W, 16)) return ABT_EALIGN;
    return launch_gemm_f32_one(gemm(A, B, W, m, n, k, k, n, n, 0, 0, 0), (hipStream_t)stream) == hipSuccess
               ? ABT_OK : ABT_EHIP;
}

int abt_set_chain_rows(int rows) {
    if (rows == 0 || rows == 64 || rows == 128) return g_chain_rows.exchange(rows);
    return g_chain_rows.load();
}

int abt_set_chain_parts(int parts) {
    if (parts >= 0 && parts <= 8) return g_chain_parts.exchange(parts);
    return g_chain_parts.load();
}

int abt_set_jacobi_max_sweeps(int max_sweeps) {
    return g_max_sweeps.exchange(max_sweeps < 1 ? 1 : (max_sweeps > 64 ? 64 : max_sweeps));
}

int abt_set_merge_groups(int groups) { return merge_set_groups(groups); }

int abt_set_merge_stage_timing(int on) { return merge_set_stage_timing(on); }

int ab_merge_stage_ms(float* ms) {
    if (!ms) return ABT_EINVAL;
    return merge_stage_ms(ms) == hipSuccess ? ABT_OK : ABT_EHIP;
}

size_t lr_linear_fwd_workspace_bytes(int64_t M, int64_t m, int64_t n, int64_t r, int dt) {
    if (check_lr_shapes(M, m, n, r, dt) != ABT_OK) return 0;
    return dt == ABT_F32 ? align_up((size_t)M * r * 4, 256) : 0;
}

int lr_linear_fwd_wants_T(int G, int64_t M, int64_t m, int64_t n, int64_t r, int dt) {
    if (G < 1 || G > ABT_MAX_GROUPS || dt != ABT_BF16 || check_lr_shapes(M, m, n, r, dt) != ABT_OK) return 0;
    return place_pays(G * M, M, (int)n, (int)m, (int)r);
}

size_t lr_linear_bwd_workspace_bytes(int64_t M, int64_t m, int64_t n, int64_t r, int dt) {
    if (check_lr_shapes(M, m, n, r, dt) != ABT_OK) return 0;
    return bwd_bytes(M, m, n, r, dt, SIZE_MAX);
}

int lr_linear_fwd(const void* X, const void* A, const void* B, void* Y, void* T_save,
                  int64_t M, int64_t m, int64_t n, int64_t r, int dt,
                  void* workspace, size_t workspace_bytes, void* stream) {
    int st = check_lr_shapes(M, m, n, r, dt);
    if (st != ABT_OK) return st;
    if (!X || !A || !B || !Y) return ABT_EINVAL;
    if (!aligned(X, 16) || !aligned(A, 16) || !aligned(B, 16) || !aligned(Y, 16) || !aligned(T_save, 16))
        return ABT_EALIGN;
    hipStream_t s = (hipStream_t)stream;
    if (dt == ABT_BF16) {
        return chain(X, B, A, Y, T_save, M, (int)n, (int)m, (int)r, s) == hipSuccess ? ABT_OK : ABT_EHIP;
    }
    float* T = (float*)T_save;
    const bool tiny = tiny_f32(M, m, n, r, {{X, M * n}, {A, m * r}, {B, r * n}}, {{Y, M * m}, {T_save, M * r}});
    if (!T) {
        if (!workspace || workspace_bytes < lr_linear_fwd_workspace_bytes(M, m, n, r, dt)) return ABT_EWORKSPACE;
        if (!aligned(workspace, 256)) return ABT_EALIGN;
        T = (float*)workspace;
    }
    if (tiny)
        return launch_tiny_f32_fwd((const float*)X, (const float*)A, (const float*)B, (float*)Y, (float*)T_save, M, m, n, r, s) == hipSuccess ? ABT_OK : ABT_EHIP;
    // T = X B^T ; Y = T A^T
    if (launch_gemm_f32_one(gemm((const float*)X, (const float*)B, T, M, r, n, n, n, r, 0, 1, 0), s) != hipSuccess) return ABT_EHIP;
    if (launch_gemm_f32_one(gemm(T, (const float*)A, (float*)Y, M, m, r, r, r, m, 0, 1, 0), s) != hipSuccess) return ABT_EHIP;
    return ABT_OK;
}

namespace {
int linear_bwd(const void* dY, const void* X, const void* T, const void* A, const void* B,
               void* dX, float* dA, float* dB,
               int64_t M, int64_t m, int64_t n, int64_t r, int dt, int accumulate,
               void* workspace, size_t workspace_bytes, size_t limit, void* stream) {
    int st = check_lr_shapes(M, m, n, r, dt);
    if (st != ABT_OK) return st;
    if (!dY || !X || !A || !B) return ABT_EINVAL;
    if (!aligned(dY, 16) || !aligned(X, 16) || !aligned(T, 16) || !aligned(A, 16) || !aligned(B, 16) ||
        !aligned(dX, 16) || !aligned(dA, 16) || !aligned(dB, 16))
        return ABT_EALIGN;
    if (!workspace || workspace_bytes < bwd_bytes(M, m, n, r, dt, limit)) return ABT_EWORKSPACE;
    if (!aligned(workspace, 256)) return ABT_EALIGN;
    hipStream_t s = (hipStream_t)stream;
    char* ws = (char*)workspace;
    const int acc = accumulate ? 1 : 0;
    if (!dX && !dA && !dB) return ABT_OK;

    if (dt == ABT_F32) {
        // (dT of 32 rows once per work-group, of two blocks of rows in tiles of dB: no more than two chunks of 256 of the contraction in all)
        if ((T || !dA) && ceil_div(M, 32) * ceil_div(m, 256) <= 2 && tiny_f32(M, m, n, r, {{dY, M * m}, {X, M * n}, {T, M * r}, {A, m * r}, {B, r * n}}, {{dX, M * n}, {dA, m * r}, {dB, r * n}}))
            return launch_tiny_f32_bwd((const float*)dY, (const float*)X, (const float*)T, (const float*)A, (const float*)B, (float*)dX, dA, dB, M, m, n, r, acc, s) ==
                   hipSuccess ? ABT_OK : ABT_EHIP;
        // two launches (each with one that adds its split sums, if any): first what depends on the inputs alone, then the rest
        const BwdLayoutF32 w = bwd_layout_f32(M, m, n, r, limit);
        float* dT = (float*)(ws + w.dT);
        const float* Tp = (const float*)T;
        GemmF32 g[3];
        int split[3], k = 0;
        // T again: unsplit, and in tiles of the size that the forward takes, so that it has the bits of the forward's
        if (!Tp && dA) {
            float* Tw = (float*)(ws + w.T);
            split[k] = 1;
            g[k++] = gemm((const float*)X, (const float*)B, Tw, M, r, n, n, n, r, 0, 1, 0);
            Tp = Tw;
        }
        if (dX || dB) { split[k] = w.split_dT; g[k++] = gemm((const float*)dY, (const float*)A, dT, M, r, m, m, r, r, 0, 0, 0); }
        float* const partials = (float*)(ws + w.partials);
        if (k == 2 && !gemm_f32_first_as_alone(g, split, k)) {
            if (launch_gemm_f32_one(g[0], s) != hipSuccess) return ABT_EHIP;
            g[0] = g[1];
            split[0] = split[1];
            k = 1;
        }
        if (k && launch_gemm_f32(g, split, k, partials, s) != hipSuccess) return ABT_EHIP;
        // an output over an operand of the second launch is written after its readers: one product after the other
        const void* out[3] = {dX, dA, dB};
        const int64_t out_bytes[3] = {M * n * 4, m * r * 4, r * n * 4};
        bool in_turn = false;
        for (int i = 0; i < 3; ++i)
            in_turn |= overlap(out[i], out_bytes[i], dY, M * m * 4) || overlap(out[i], out_bytes[i], Tp, M * r * 4) ||
                       overlap(out[i], out_bytes[i], X, M * n * 4) || overlap(out[i], out_bytes[i], B, r * n * 4);
        k = 0;
        if (dX && in_turn) { split[k] = 1; g[k++] = gemm(dT, (const float*)B, (float*)dX, M, n, r, r, n, n, 0, 0, 0); }
        if (dA) { split[k] = w.split_A; g[k++] = grad_A_f32((const float*)dY, Tp, dA, M, m, r, acc); }
        if (dB) { split[k] = w.split_B; g[k++] = grad_B_f32(dT, (const float*)X, dB, M, n, r, acc); }
        if (dX && !in_turn) { split[k] = 1; g[k++] = gemm(dT, (const float*)B, (float*)dX, M, n, r, r, n, n, 0, 0, 0); }
        if (!in_turn) return launch_gemm_f32(g, split, k, partials, s) == hipSuccess ? ABT_OK : ABT_EHIP;
        for (int i = 0; i < k; ++i)
            if (launch_gemm_f32(g + i, split + i, 1, partials, s) != hipSuccess) return ABT_EHIP;
        return ABT_OK;
    }

    const BwdLayout w = bwd_layout_bf16(M, m, n, r);
    void* At = ws + w.At; void* Bt = ws + w.Bt; void* dT = ws + w.dT;
    const void* Tp = T;
    hipError_t e = hipSuccess;
    if (!Tp && dA) {  // recompute T = X B^T (first stage of the chain only)
        e = chain(X, B, nullptr, nullptr, ws + w.T, M, (int)n, (int)m, (int)r, s);
        if (e != hipSuccess) return ABT_EHIP;
        Tp = ws + w.T;
    }
    const SmallBwd few = small_bwd(dY, X, Tp, B, dX, dA, dB, M, m, n, r);
    if (few != kNotSmall) {
        if ((dX || dB) && launch_lr_small_dt(dY, A, dT, M, (int)m, (int)r, s) != hipSuccess) return ABT_EHIP;
        e = few_gradients(few, dA, dB, m, n, r, acc, (float*)(ws + w.partials), s, [&](float* dA_to, float* dB_to, int add) {
            return launch_lr_small_grad(dY, X, Tp, B, dX, dA_to, dB_to, dT, M, (int)m, (int)n, (int)r, add, s);
        });
        return e == hipSuccess ? ABT_OK : ABT_EHIP;
    }
    if (dX || dB) {
        // dT = dY A = dY (A^T)^T and dX = dT B = dT (B^T)^T: the forward chain on transposed factors
        const TransposeJob tj[2] = {{A, At, (int)m, (int)r}, {B, Bt, (int)r, (int)n}};
        e = launch_transpose_bf16(tj, dX ? 2 : 1, s);
        if (e != hipSuccess) return ABT_EHIP;
        e = chain(dY, At, dX ? Bt : nullptr, dX, dT, M, (int)m, (int)n, (int)r, s);
        if (e != hipSuccess) return ABT_EHIP;
    }
    TnJob jobs[2];
    int nj = 0;
    if (dA) jobs[nj++] = TnJob{dY, Tp, dA, (int)m, 0};
    if (dB) jobs[nj++] = TnJob{X, dT, dB, (int)n, 1};
    if (nj) {
        e = launch_tn_bf16(jobs, nj, M, (int)r, acc, (float*)(ws + w.partials), s);
        if (e != hipSuccess) return ABT_EHIP;
    }
    return ABT_OK;
}
}  // namespace

int lr_linear_bwd(const void* dY, const void* X, const void* T, const void* A, const void* B,
                  void* dX, float* dA, float* dB,
                  int64_t M, int64_t m, int64_t n, int64_t r, int dt, int accumulate,
                  void* workspace, size_t workspace_bytes, void* stream) {
    return linear_bwd(dY, X, T, A, B, dX, dA, dB, M, m, n, r, dt, accumulate, workspace, workspace_bytes, SIZE_MAX, stream);
}

// ------------------------------------------------------------------ G emulated groups per launch
namespace {
struct GroupedLayout { size_t At, Bt, dT, T, per_group, partials, total; };

GroupedLayout grouped_layout_bf16(int G, int64_t M, int64_t m, int64_t n, int64_t r) {
    GroupedLayout w{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    w.At = take((size_t)r * m * 2);
    w.Bt = take((size_t)n * r * 2);
    w.dT = take((size_t)M * r * 2);
    w.T = take((size_t)M * r * 2);
    w.per_group = off;
    w.partials = (size_t)G * w.per_group;
    // Partials of any subset of the 2 G jobs: elements x splits with splits <= max(1, 256 / tiles) and
    // elements <= tiles x 128 x r, hence at most max(all elements, 256 x 128 x r) floats.
    const size_t all = (size_t)G * (size_t)(m + n) * r, cap = (size_t)256 * 128 * r;
    w.total = w.partials + align_up((all > cap ? all : cap) * sizeof(float), 256);
    return w;
}

int chain_rows_for_groups(int G, int64_t M, int p, int q, int R) {
    const int forced = g_chain_rows.load();
    if (!chain2_tall_supports(R, p, q) || (forced == 64 && chain2_supports(R, p, q))) return 64;
    if (forced == 128 || !chain2_supports(R, p, q)) return 128;
    const double cost64 = (double)ceil_div(G * ceil_div(M, 64), 256);
    const double cost128 = 1.58 * (double)ceil_div(G * ceil_div(M, 128), 256);
    return cost128 < cost64 ? 128 : 64;
}

// One launch for the problems with a second stage and one for those without.  again: T for some of the groups, by the rules
// for all of them.
hipError_t chain_grouped(const ChainProblem* pr, int G, int64_t M, int p, int q, int R, bool again, hipStream_t s) {
    for (int second = 1; second >= 0; --second) {
        ChainProblem sel[kChainMaxGroups];
        int n = 0;
        for (int g = 0; g < G; ++g) {
            const bool has2 = pr[g].Yout != nullptr;
            if ((has2 && second) || (!has2 && !second && pr[g].Tout)) sel[n++] = pr[g];
        }
        if (n == 0) continue;
        hipError_t e;
        const int of = again ? G : n;
        // (the rule and the split of the rows are those of all groups: the order of the sums of T is the same for some of them)
        if (wide_products(G * M, p, q, R, G > 1) && pair_supports(M, p, q, R) && place_for_T(sel, n, M, p, R)) {
            e = launch_pair_bf16(sel, n, G, M, p, q, R, s);
        } else if (few_rows(sel, n, G, M, p, q, R)) {
            e = launch_few_fwd(sel, n, M, p, q, R, s);
        } else if (two_products(sel, n, of, M, p, q, R)) {
            e = launch_lr_small_fwd(sel, n, of, M, p, q, R, s);
        } else if (!narrow_chain(sel, n, of, M, p, q, R, s, &e)) {
            e = launch_chain2_grouped_bf16(sel, n, M, p, q, R, chain_rows_for_groups(of, M, p, q, R), 1, s);
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
}  // namespace

size_t lr_linear_bwd_grouped_workspace_bytes(int G, int64_t M, int64_t m, int64_t n, int64_t r, int dt) {
    if (G < 1 || G > ABT_MAX_GROUPS || check_lr_shapes(M, m, n, r, dt) != ABT_OK) return 0;
    if (dt == ABT_F32) return (size_t)G * lr_linear_bwd_workspace_bytes(M, m, n, r, dt);
    return grouped_layout_bf16(G, M, m, n, r).total;
}

int lr_linear_fwd_grouped(const abt_lr_group* groups, int G,
                          int64_t M, int64_t m, int64_t n, int64_t r, int dt,
                          void* workspace, size_t workspace_bytes, void* stream) {
    const int st = check_lr_shapes(M, m, n, r, dt);
    if (st != ABT_OK) return st;
    if (!groups || G < 1 || G > ABT_MAX_GROUPS) return ABT_EINVAL;
    for (int g = 0; g < G; ++g) {
        const abt_lr_group& q = groups[g];
        if (!q.X || !q.A || !q.B || !q.Y || ((q.T_save != nullptr) != (groups[0].T_save != nullptr))) return ABT_EINVAL;
        if (!aligned(q.X, 16) || !aligned(q.A, 16) || !aligned(q.B, 16) || !aligned(q.Y, 16) || !aligned(q.T_save, 16))
            return ABT_EALIGN;
    }
    if (dt == ABT_F32) {
        const size_t each = lr_linear_fwd_workspace_bytes(M, m, n, r, dt);
        if (!groups[0].T_save && (!workspace || workspace_bytes < each * G)) return ABT_EWORKSPACE;
        for (int g = 0; g < G; ++g) {
            const int e = lr_linear_fwd(groups[g].X, groups[g].A, groups[g].B, groups[g].Y, groups[g].T_save, M, m, n, r, dt,
                                        workspace ? (char*)workspace + each * g : nullptr, each, stream);
            if (e != ABT_OK) return e;
        }
        return ABT_OK;
    }
    ChainProblem pr[kChainMaxGroups];
    for (int g = 0; g < G; ++g) pr[g] = ChainProblem{groups[g].X, groups[g].B, groups[g].A, groups[g].Y, groups[g].T_save};
    return chain_grouped(pr, G, M, (int)n, (int)m, (int)r, false, (hipStream_t)stream) == hipSuccess ? ABT_OK : ABT_EHIP;
}

int lr_linear_bwd_grouped(const abt_lr_group* groups, int G,
                          int64_t M, int64_t m, int64_t n, int64_t r, int dt, int accumulate,
                          void* workspace, size_t workspace_bytes, void* stream) {
    const int st = check_lr_shapes(M, m, n, r, dt);
    if (st != ABT_OK) return st;
    if (!groups || G < 1 || G > ABT_MAX_GROUPS) return ABT_EINVAL;
    for (int g = 0; g < G; ++g) {
        const abt_lr_group& q = groups[g];
        if (!q.dY || !q.X || !q.A || !q.B) return ABT_EINVAL;
        if (!aligned(q.dY, 16) || !aligned(q.X, 16) || !aligned(q.T, 16) || !aligned(q.A, 16) || !aligned(q.B, 16) ||
            !aligned(q.dX, 16) || !aligned(q.dA, 16) || !aligned(q.dB, 16))
            return ABT_EALIGN;
    }
    if (!workspace || workspace_bytes < lr_linear_bwd_grouped_workspace_bytes(G, M, m, n, r, dt)) return ABT_EWORKSPACE;
    if (!aligned(workspace, 256)) return ABT_EALIGN;
    char* ws = (char*)workspace;
    if (dt == ABT_F32) {
        const size_t each = lr_linear_bwd_workspace_bytes(M, m, n, r, dt);
        for (int g = 0; g < G; ++g) {
            const abt_lr_group& q = groups[g];
            const int e = lr_linear_bwd(q.dY, q.X, q.T, q.A, q.B, q.dX, q.dA, q.dB, M, m, n, r, dt, accumulate,
                                        ws + each * g, each, stream);
            if (e != ABT_OK) return e;
        }
        return ABT_OK;
    }
    hipStream_t s = (hipStream_t)stream;
    const GroupedLayout w = grouped_layout_bf16(G, M, m, n, r);
    auto at = [&](int g, size_t off) { return ws + (size_t)g * w.per_group + off; };
    // T = X B^T again for the groups that did not keep it and need it for dA
    ChainProblem pr[kChainMaxGroups];
    const void* Tp[kChainMaxGroups];
    bool any = false;
    for (int g = 0; g < G; ++g) {
        const abt_lr_group& q = groups[g];
        Tp[g] = q.T;
        pr[g] = ChainProblem{};
        if (!q.T && q.dA) {
            pr[g] = ChainProblem{q.X, q.B, nullptr, nullptr, at(g, w.T)};
            Tp[g] = at(g, w.T);
            any = true;
        }
    }
    if (any && chain_grouped(pr, G, M, (int)n, (int)m, (int)r, true, s) != hipSuccess) return ABT_EHIP;
    // dT = dY (A^T)^T, dX = dT (B^T)^T: the forward chain on the transposed factors of every group
    TransposeJob tj[kTransposeMaxJobs];
    int ntj = 0;
    any = false;
    for (int g = 0; g < G; ++g) {
        const abt_lr_group& q = groups[g];
        pr[g] = ChainProblem{};
        if (!q.dX && !q.dB) continue;
        tj[ntj++] = TransposeJob{q.A, at(g, w.At), (int)m, (int)r};
        if (q.dX) tj[ntj++] = TransposeJob{q.B, at(g, w.Bt), (int)r, (int)n};
        pr[g] = ChainProblem{q.dY, at(g, w.At), q.dX ? at(g, w.Bt) : nullptr, q.dX, at(g, w.dT)};
        any = true;
    }
    if (any) {
        if (launch_transpose_bf16(tj, ntj, s) != hipSuccess) return ABT_EHIP;
        if (chain_grouped(pr, G, M, (int)m, (int)n, (int)r, false, s) != hipSuccess) return ABT_EHIP;
    }
    // factor gradients of all groups in one launch (and one split reduction)
    TnJob jobs[kTnMaxJobs];
    int nj = 0;
    for (int g = 0; g < G; ++g) {
        const abt_lr_group& q = groups[g];
        if (q.dA) jobs[nj++] = TnJob{q.dY, Tp[g], q.dA, (int)m, 0};
        if (q.dB) jobs[nj++] = TnJob{q.X, at(g, w.dT), q.dB, (int)n, 1};
    }
    if (nj && tn_partials_bytes(M, jobs, nj, (int)r) > w.total - w.partials) return ABT_EWORKSPACE;   // cannot happen: see the layout
    if (nj && launch_tn_bf16(jobs, nj, M, (int)r, accumulate ? 1 : 0, (float*)(ws + w.partials), s) != hipSuccess)
        return ABT_EHIP;
    return ABT_OK;
}

// ------------------------------------------------------------------ backward without allocation
// The scratch of lr_linear_bwd_static: one array per GPU, held from the moment the library's code is
// loaded on that GPU until the process ends.  In host code the name below is only a handle; the
// array's device address comes from hipGetSymbolAddress, once per device, and only that address is
// ever handed to a kernel.
static __device__ __align__(256) unsigned char scratch[ABT_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

int static_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ABT_EHIP;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ABT_EHIP;
        g_scratch_ptr[dev].store(p, std::memory_order_release);   // every thread gets the same address
    }
    *out = p;
    return ABT_OK;
}
}  // namespace

int lr_linear_bwd_static(const void* dY, const void* X, const void* T, const void* A, const void* B,
                         void* dX, float* dA, float* dB,
                         int64_t M, int64_t m, int64_t n, int64_t r, int dt, int accumulate, void* stream) {
    const int st = check_lr_shapes(M, m, n, r, dt);
    if (st != ABT_OK) return st;
    constexpr size_t limit = ABT_STATIC_SCRATCH_BYTES;
    if (bwd_bytes(M, m, n, r, dt, limit) > limit) return ABT_ETOOLARGE;
    void* ws = nullptr;
    const int sp = static_scratch(&ws);
    if (sp != ABT_OK) return sp;
    return linear_bwd(dY, X, T, A, B, dX, dA, dB, M, m, n, r, dt, accumulate, ws, limit, limit, stream);
}

size_t ab_merge_batched_workspace_bytes(const abt_merge_desc* layers, int L) {
    if (!layers || L < 1) return 0;
    for (int l = 0; l < L; ++l)
        if (layers[l].G < 1 || layers[l].m < 1 || layers[l].n < 1 || layers[l].k < 1 || layers[l].k_cap < 1 ||
            (layers[l].mode != 0 && layers[l].mode != 1))
            return 0;
    return guarded_size([&] { return merge_workspace_bytes(layers, L); });
}

int ab_merge_batched(const abt_merge_desc* layers, int L, void* workspace, size_t workspace_bytes, void* stream) {
    if (!layers || L < 1) return ABT_EINVAL;
    for (int l = 0; l < L; ++l) {
        const int st = check_merge_layer(layers[l]);
        if (st != ABT_OK) return st;
    }
    return guarded([&]() -> int {
        if (!workspace || workspace_bytes < merge_workspace_bytes(layers, L)) return ABT_EWORKSPACE;
        if (!aligned(workspace, 256)) return ABT_EALIGN;
        if (merge_stream_captures((hipStream_t)stream)) return ABT_EHIP;
        return merge_run(layers, nullptr, L, workspace, g_max_sweeps, (hipStream_t)stream) == hipSuccess ? ABT_OK : ABT_EHIP;
    });
}

size_t ab_merge_workspace_bytes(int G, int64_t m, int64_t n, int64_t k, int64_t k_cap, int mode) {
    abt_merge_desc d{};
    d.G = G; d.m = m; d.n = n; d.k = k; d.k_cap = k_cap; d.mode = mode;
    return ab_merge_batched_workspace_bytes(&d, 1);
}

int ab_merge(const float* const* A_copies, const float* const* B_copies, int G,
             int64_t m, int64_t n, int64_t k, float tau, int64_t k_fixed, int mode,
             float* A_out, float* B_out, float* S_out, int32_t* k_out, int64_t k_cap,
             float* W_out, void* workspace, size_t workspace_bytes, void* stream) {
    abt_merge_desc d{};
    d.A_copies = A_copies; d.B_copies = B_copies; d.G = G; d.mode = mode;
    d.m = m; d.n = n; d.k = k; d.tau = tau; d.k_fixed = k_fixed;
    d.A_out = A_out; d.B_out = B_out; d.S_out = S_out; d.k_out = k_out; d.k_cap = k_cap; d.W_out = W_out;
    return ab_merge_batched(&d, 1, workspace, workspace_bytes, stream);
}

// Dense W = W I (n <= m) or I W (n > m): the merge of one "copy" whose short-side factor is the
// identity.  Workspace: [merge workspace of the L layers][one K x K fp32 identity per distinct K].
}  // extern "C"

namespace {
int64_t factorize_K(int64_t m, int64_t n) { return m < n ? m : n; }

struct FactorizePlan {
    std::vector<abt_merge_desc> merge;      // A_copies / B_copies are filled in by the caller
    std::vector<int64_t> Ks;                // distinct K, in order of first use
    std::vector<size_t> eye_off;            // byte offset of each identity behind the merge workspace
    std::vector<int> eye_of_layer;
    size_t merge_bytes = 0, total = 0;
    int status = ABT_OK;
};

FactorizePlan plan_factorize(const abt_factorize_desc* layers, int L) {
    FactorizePlan p;
    if (!layers || L < 1) { p.status = ABT_EINVAL; return p; }
    p.merge.resize(L);
    p.eye_of_layer.resize(L);
    for (int l = 0; l < L; ++l) {
        const abt_factorize_desc& f = layers[l];
        if (f.m < 1 || f.n < 1 || f.k_cap < 1) { p.status = ABT_ESHAPE; return p; }
        const int64_t K = factorize_K(f.m, f.n);
        if (K % 32 || K > 2048) { p.status = ABT_ESHAPE; return p; }
        abt_merge_desc& d = p.merge[l];
        d = abt_merge_desc{};
        d.G = 1; d.mode = 0; d.m = f.m; d.n = f.n; d.k = K; d.tau = f.tau; d.k_fixed = f.k_fixed;
        d.A_out = f.A_out; d.B_out = f.B_out; d.S_out = f.S_out; d.k_out = f.k_out; d.k_cap = f.k_cap;
        int e = -1;
        for (size_t i = 0; i < p.Ks.size(); ++i) if (p.Ks[i] == K) e = (int)i;
        if (e < 0) { e = (int)p.Ks.size(); p.Ks.push_back(K); }
        p.eye_of_layer[l] = e;
    }
    p.merge_bytes = align_up(merge_workspace_bytes(p.merge.data(), L), 256);
    size_t off = p.merge_bytes;
    for (int64_t K : p.Ks) { p.eye_off.push_back(off); off += align_up(sizeof(float) * K * K, 256); }
    p.total = off;
    return p;
}
}  // namespace

extern "C" {

size_t ab_factorize_batched_workspace_bytes(const abt_factorize_desc* layers, int L) {
    return guarded_size([&]() -> size_t {
        const FactorizePlan p = plan_factorize(layers, L);
        return p.status == ABT_OK ? p.total : 0;
    });
}

int ab_factorize_batched(const abt_factorize_desc* layers, int L, void* workspace, size_t workspace_bytes,
                         void* stream) {
    return guarded([&]() -> int {
    FactorizePlan p = plan_factorize(layers, L);
    if (p.status != ABT_OK) return p.status;
    for (int l = 0; l < L; ++l) {
        if (!layers[l].W) return ABT_EINVAL;
        if (!aligned(layers[l].W, 16)) return ABT_EALIGN;
    }
    if (!workspace || workspace_bytes < p.total) return ABT_EWORKSPACE;
    if (!aligned(workspace, 256)) return ABT_EALIGN;
    // one pointer pair per layer: (W, I) or (I, W); the arrays are read before merge_run returns
    std::vector<const float*> a_ptr(L), b_ptr(L);
    std::vector<MergeSide> identity(L);
    for (int l = 0; l < L; ++l) {
        const float* eye = (const float*)((const char*)workspace + p.eye_off[p.eye_of_layer[l]]);
        const bool tall = layers[l].n <= layers[l].m;
        identity[l] = tall ? MergeSide::B : MergeSide::A;
        a_ptr[l] = tall ? layers[l].W : eye;
        b_ptr[l] = tall ? eye : layers[l].W;
        p.merge[l].A_copies = &a_ptr[l];
        p.merge[l].B_copies = &b_ptr[l];
        const int st = check_merge_layer(p.merge[l]);
        if (st != ABT_OK) return st;
    }
    if (merge_stream_captures((hipStream_t)stream)) return ABT_EHIP;
    for (size_t i = 0; i < p.Ks.size(); ++i)
        if (launch_identity_f32((float*)((char*)workspace + p.eye_off[i]), (int)p.Ks[i], (hipStream_t)stream) != hipSuccess)
            return ABT_EHIP;
    return merge_run(p.merge.data(), identity.data(), L, workspace, g_max_sweeps, (hipStream_t)stream) == hipSuccess ? ABT_OK : ABT_EHIP;
    });
}

size_t ab_factorize_workspace_bytes(int64_t m, int64_t n, int64_t k_cap) {
    abt_factorize_desc f{};
    f.m = m; f.n = n; f.k_cap = k_cap;
    return ab_factorize_batched_workspace_bytes(&f, 1);
}

int ab_factorize(const float* W, int64_t m, int64_t n, float tau, int64_t k_fixed,
                 float* A_out, float* B_out, float* S_out, int32_t* k_out, int64_t k_cap,
                 void* workspace, size_t workspace_bytes, void* stream) {
    abt_factorize_desc f{};
    f.W = W; f.m = m; f.n = n; f.tau = tau; f.k_fixed = k_fixed;
    f.A_out = A_out; f.B_out = B_out; f.S_out = S_out; f.k_out = k_out; f.k_cap = k_cap;
    return ab_factorize_batched(&f, 1, workspace, workspace_bytes, stream);
}

int ab_merge_info_batched(const void* workspace, int first, int count, int32_t* sweeps, int32_t* n_sigma, void* stream) {
    if (!workspace || first < 0 || count < 1) return ABT_EINVAL;
    return guarded([&]() -> int {
        std::vector<int32_t> info;                              // (not resized before the count has been checked)
        const hipError_t e = merge_read_info(workspace, first, count, info, (hipStream_t)stream);
        if (e == hipErrorInvalidValue) return ABT_EINVAL;       // not a merge workspace, or no such layers in it
        if (e != hipSuccess) return ABT_EHIP;
        bool converged = true;
        for (int i = 0; i < count; ++i) {
            if (sweeps) sweeps[i] = info[4 * i];
            if (n_sigma) n_sigma[i] = info[4 * i + 1];
            converged &= info[4 * i + 2] != 0;
        }
        return converged ? ABT_OK : ABT_ENOCONV;
    });
}

int ab_merge_info(const void* workspace, int layer, int32_t* sweeps, int32_t* n_sigma, void* stream) {
    return ab_merge_info_batched(workspace, layer, 1, sweeps, n_sigma, stream);
}

}  // extern "C"
