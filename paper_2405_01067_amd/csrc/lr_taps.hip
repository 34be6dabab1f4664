// Factor gradients of a factored convolution with a window three pixels wide, R <= 96: dB = patches(act)^T dT, and dA = dY^T T in the
// same launch (bf16 in, fp32 partial sums, which tn2_reduce_kernel adds).
//
// A work-group has 64 channels, one row of the window with its three taps, all R columns and one split of the pixels.  The kernel
// for any gathered operand (lr_tn2.hip) fetches, checks and transposes every tap by itself in registers, 128 columns at a time; that is what its time goes into.
// Here the pixels of a slab come straight to LDS once for the three taps (loads with the LDS flag, two or three slabs ahead), as they lie, and the
// transposing LDS loads make the matrix operands: an operand row is a pixel, so a tap is another address per lane, and one outside the image the address of a row of zeros.
//
// Eight waves: two blocks of 32 channels x four parts of a slab's pixels, whose sums are added through LDS at the end.  A wave reads 3 + R / 32
// operands for 3 R / 32 products and waits for them; only the wave beside it on the SIMD has products running then.  That, and the loads, is what bounds it: r = 64, 256 x 14 x 14,
// batch 256 (25 slabs): 30 us; 19 with the loads alone, 26 with the products alone, matrix units busy for 7.  A second work-group per compute unit does not fit the LDS,
// and one writes the fewer partial sums.  Tried: operands read one slab ahead (registers: spills from r = 96 on, no faster at 64), 64 channels and an eighth of the pixels per wave (spills).
// Factor gradients with dT and the sums, this kernel / the one for any window: 256 x 14 x 14, r = 64, batch 256 47 / 60 us; 128 x 28 x 28, stride 2, 43 / 50. The whole
// backward: 64 x 56 x 56, batch 160, r = 32 136 / 189, r = 64 165 / 219, r = 96 244 / 289; never slower at 80 shapes of r up to 96.  At r = 128 it spills and is slower everywhere (64 x 56 x 56, batch
// 160 398 / 325).
//
// Half a wave reads four rows of 64 bytes at a time.  In the LDS image of a pixel (128 bytes) and of a row of V (2 R bytes) the pieces of 64 bytes
// change places with the row so that the four lie in different banks; the loads fetch what belongs at the place they fill.
#include "tn_args.h"

namespace abt {

namespace {

// N transposing loads: lane l of 16 names row l / 4 of four and four 16-bit columns of it, and gets the four rows of column l.  With the builtin the
// compiler waits for all loads to LDS that are on their way before each group of them (factor gradients of 256 x 14 x 14, r = 64: 34 us); in assembly the
// waits are those below.  The loads are waited for where they are issued, so no register is written late.
template <int N>
__device__ __forceinline__ void load_transposed(const uint32_t (&a)[N], u32x2 (&v)[N]) {
#define ABT_TR(i, j) "ds_read_b64_tr_b16 %" #i ", %" #j "\n\t"
#define ABT_OUT(i) "=&v"(v[i])
#define ABT_IN(i) "v"(a[i])
    if constexpr (N == 6)
        asm volatile(ABT_TR(0, 6) ABT_TR(1, 7) ABT_TR(2, 8) ABT_TR(3, 9) ABT_TR(4, 10) ABT_TR(5, 11) "s_waitcnt lgkmcnt(0)"
                     : ABT_OUT(0), ABT_OUT(1), ABT_OUT(2), ABT_OUT(3), ABT_OUT(4), ABT_OUT(5)
                     : ABT_IN(0), ABT_IN(1), ABT_IN(2), ABT_IN(3), ABT_IN(4), ABT_IN(5) : "memory");
    else if constexpr (N == 8)
        asm volatile(ABT_TR(0, 8) ABT_TR(1, 9) ABT_TR(2, 10) ABT_TR(3, 11) ABT_TR(4, 12) ABT_TR(5, 13) ABT_TR(6, 14) ABT_TR(7, 15) "s_waitcnt lgkmcnt(0)"
                     : ABT_OUT(0), ABT_OUT(1), ABT_OUT(2), ABT_OUT(3), ABT_OUT(4), ABT_OUT(5), ABT_OUT(6), ABT_OUT(7)
                     : ABT_IN(0), ABT_IN(1), ABT_IN(2), ABT_IN(3), ABT_IN(4), ABT_IN(5), ABT_IN(6), ABT_IN(7) : "memory");
    else if constexpr (N == 10)
        asm volatile(ABT_TR(0, 10) ABT_TR(1, 11) ABT_TR(2, 12) ABT_TR(3, 13) ABT_TR(4, 14) ABT_TR(5, 15) ABT_TR(6, 16) ABT_TR(7, 17) ABT_TR(8, 18) ABT_TR(9, 19)
                     "s_waitcnt lgkmcnt(0)"
                     : ABT_OUT(0), ABT_OUT(1), ABT_OUT(2), ABT_OUT(3), ABT_OUT(4), ABT_OUT(5), ABT_OUT(6), ABT_OUT(7), ABT_OUT(8), ABT_OUT(9)
                     : ABT_IN(0), ABT_IN(1), ABT_IN(2), ABT_IN(3), ABT_IN(4), ABT_IN(5), ABT_IN(6), ABT_IN(7), ABT_IN(8), ABT_IN(9) : "memory");
    else {
        static_assert(N == 12, "");
        asm volatile(ABT_TR(0, 12) ABT_TR(1, 13) ABT_TR(2, 14) ABT_TR(3, 15) ABT_TR(4, 16) ABT_TR(5, 17) ABT_TR(6, 18) ABT_TR(7, 19) ABT_TR(8, 20) ABT_TR(9, 21)
                     ABT_TR(10, 22) ABT_TR(11, 23) "s_waitcnt lgkmcnt(0)"
                     : ABT_OUT(0), ABT_OUT(1), ABT_OUT(2), ABT_OUT(3), ABT_OUT(4), ABT_OUT(5), ABT_OUT(6), ABT_OUT(7), ABT_OUT(8), ABT_OUT(9), ABT_OUT(10), ABT_OUT(11)
                     : ABT_IN(0), ABT_IN(1), ABT_IN(2), ABT_IN(3), ABT_IN(4), ABT_IN(5), ABT_IN(6), ABT_IN(7), ABT_IN(8), ABT_IN(9), ABT_IN(10), ABT_IN(11) : "memory");
    }
#undef ABT_TR
#undef ABT_OUT
#undef ABT_IN
}

template <int R, int MUL>
struct Taps {
    static constexpr int RB = R / 32;
    static constexpr int BP = R <= 64 ? 128 : 64;          // pixels of a slab
    static constexpr int NS = R <= 64 ? 3 : 4;             // slabs in LDS
    static constexpr int STEPS = BP / 64;                  // steps of 16 pixels per wave and slab
    static constexpr int HALF = BP + 8;                    // (strided)
    static constexpr int UROWS = MUL == 1 ? BP + 8 : HALF + BP;                    // pixels that the taps of a slab touch
    static constexpr int ROWS = UROWS > 2 * BP ? UROWS : 2 * BP;                   // a plain job has 128 columns: two rows of 128 bytes per row
    static constexpr int VP = 2 * R;
    static constexpr int ubytes = ROWS * 128, slot = ubytes + BP * VP;
    static constexpr int zeros = NS * slot, lds = zeros + 256;
    static constexpr int NV = BP * VP / 1024;
    static_assert(lds <= 160 * 1024 && 1024 * R <= zeros, "LDS");
    __device__ static int u_turn(int row) { return (row & 2) << 1; }
    __device__ static int v_turn(int row) { return R == 64 ? (row & 2) << 1 : 0; }
};

// GATHER: a job over the image (T = 3 taps of window row `ky`, channels from c0 on); otherwise a plain one (T = 2 blocks of 64 columns from c0 on)
template <int R, int MUL, bool GATHER>
__device__ __forceinline__ void taps_tile(const Tn2Args& args, const Tn2Job& job, unsigned char* lds, int c0, int ky, int split) {
    using C = Taps<R, MUL>;
    constexpr int T = GATHER ? 3 : 2, RB = C::RB, BP = C::BP, NS = C::NS;
    constexpr int NU = GATHER ? C::UROWS / 8 : 2 * BP / 8, NE = (NU + C::NV + 7) / 8;
    static_assert(NE * (NS - 2) < 64, "loads under way");
    const Tn2Gather& g = args.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t k_begin = (int64_t)split * args.rows_per_split;
    int64_t k_end = k_begin + args.rows_per_split;
    if (k_end > args.M) k_end = args.M;
    const int rows = k_end > k_begin ? (int)(k_end - k_begin) : 0;
    const int nslab = (rows + BP - 1) / BP;
    const int dy = GATHER ? ky - g.kh / 2 : 0;

    // ---- descriptors: the split's rows of V and of a plain U; of the image the pixels that the split's patches can touch
    const rsrc_t rv = make_rsrc(job.V + k_begin * R, (int64_t)rows * C::VP);
    int64_t sp0 = 0;
    rsrc_t ru;
    if (GATHER) {
        const int64_t pixels = args.M / ((int64_t)g.RH * g.RW) * g.H * g.W, reach = (int64_t)(g.kh / 2) * g.W + 1;
        auto centre = [&](int64_t i) -> int64_t {          // centre pixel of row i (monotone in i)
            if (MUL == 1) return i;
            const uint32_t line = (uint32_t)i / (uint32_t)g.RW, img = line / (uint32_t)g.RH;
            return ((int64_t)img * g.H + MUL * (line - img * g.RH)) * g.W + MUL * ((uint32_t)i - line * g.RW);
        };
        int64_t sp1 = rows ? centre(k_end - 1) + reach + 1 : 0;
        sp0 = rows ? centre(k_begin) - reach : 0;
        if (sp0 < 0) sp0 = 0;
        if (sp1 > pixels) sp1 = pixels;
        ru = make_rsrc(job.U + sp0 * g.C, (sp1 - sp0) * g.C * 2);
    } else {
        ru = make_rsrc(job.U + k_begin * job.P, (int64_t)rows * job.P * 2);
    }

    // row i of the virtual operand (there are fewer than 2^31) -> grid position, image
    auto place = [&](uint32_t row, int& px, int& py, int& img) {
        const uint32_t line = row / (uint32_t)g.RW;
        px = (int)(row - line * g.RW);
        img = (int)(line / (uint32_t)g.RH);
        py = (int)(line - img * g.RH);
    };
    // ---- this wave's loads of a slab: pieces of 1 KB wave, wave + 8, ..; first those of U, then those of V; NE of them, or one less
    const bool full = wave + 8 * (NE - 1) < NU + C::NV;
    int off[NE], step[NE], px[NE], py[NE], pi[NE];         // px, py, pi: grid position and image of a strided piece's pixel
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int piece = wave + 8 * e;
        off[e] = kBufNowhere; step[e] = 0; px[e] = py[e] = pi[e] = 0;
        if (piece < NU) {
            const int row = 8 * piece + (lane >> 3), chunk = (lane & 7) ^ C::u_turn(row);
            if (!GATHER) {
                const int col = c0 + (row >= BP ? 64 : 0);
                if (col < job.P) { off[e] = ((row >= BP ? row - BP : row) * job.P + col) * 2 + 16 * chunk; step[e] = BP * job.P * 2; }
            } else if (MUL == 1) {
                off[e] = ((int)(k_begin - sp0) - 1 + dy * g.W + row) * (g.C * 2) + 2 * c0 + 16 * chunk;     // below zero: outside every descriptor
                step[e] = BP * g.C * 2;
            } else {
                // row HALF + j is the centre of pixel j, row j + 1 its right neighbour (and where it counts the left one of pixel j + 1), row 0 the left one of
                // pixel 0: the rows of an operand lie one behind the other here, too
                const int j = row >= C::HALF ? row - C::HALF : row - 1;
                place((uint32_t)k_begin + (j < 0 ? 0 : j), px[e], py[e], pi[e]);
                // (the product may leave 32 bits, the offset that it ends in does not)
                off[e] = (int)(((uint32_t)((row >= C::HALF ? 0 : row ? 1 : -1) + dy * g.W) - (uint32_t)sp0) * (uint32_t)(g.C * 2)) + 2 * c0 + 16 * chunk;
            }
        } else if (piece < NU + C::NV) {
            const int at = 1024 * (piece - NU) + 16 * lane, row = at / C::VP, chunk = (at % C::VP / 16) ^ C::v_turn(row);
            off[e] = row * C::VP + 16 * chunk;
            step[e] = BP * C::VP;
        }
    }
    const int adv_x = GATHER ? BP % g.RW : 0, adv_y = GATHER ? BP / g.RW : 0;
    // (x, y, image) BP rows on; the grid has BP positions or more, so y wraps twice at most
    auto advance = [&](int& x, int& y, int& img) {
        x += adv_x;
        const int carry = x >= g.RW ? 1 : 0;
        x -= carry ? g.RW : 0;
        y += adv_y + carry;
#pragma unroll
        for (int i = 0; i < 2; ++i) { const bool wrap = y >= g.RH; y -= wrap ? g.RH : 0; img += wrap ? 1 : 0; }
    };
    auto next_slot = [](int at) { return at == (NS - 1) * C::slot ? 0 : at + C::slot; };
    int into = 0, from = 0;                                // the slot that is filled next, the one that is read
    auto request = [&]() {                                 // the slabs in turn
        unsigned char* base = lds + into;
        into = next_slot(into);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int piece = wave + 8 * e;
            const bool u = piece < NU;
            if (piece >= NU + C::NV) break;                // (the last one, in some waves)
            unsigned char* dst = u ? base + 1024 * piece : base + C::ubytes + 1024 * (piece - NU);
            int o = off[e];
            if (GATHER && MUL == 2 && u) {
                o = (int)((uint32_t)o + (uint32_t)((pi[e] * g.H + 2 * py[e]) * g.W + 2 * px[e]) * (uint32_t)(g.C * 2));
                advance(px[e], py[e], pi[e]);
            }
            load_lds16(u ? ru : rv, dst, o, 0);
            off[e] += step[e];
        }
    };

    // ---- this lane's places in the operands of a step: row 16 step + 8 (group / 2) + 4 t + i / 4 of the slab, four columns
    const int grp = lane >> 4, i = lane & 15, cw = wave & 1, ks = wave >> 1;
    const int uchunk = 4 * cw + 2 * (grp & 1) + ((i >> 1) & 1), vchunk = 2 * (grp & 1) + ((i >> 1) & 1), half = 8 * (i & 1);
    int ua[C::STEPS][2][T], va[C::STEPS][2][RB], x[C::STEPS][2], y[C::STEPS][2];
#pragma unroll
    for (int u = 0; u < C::STEPS; ++u)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int r = 16 * (ks * C::STEPS + u) + 8 * (grp >> 1) + 4 * t + (i >> 2);
#pragma unroll
            for (int d = 0; d < T; ++d) {
                const int row = !GATHER ? d * BP + r : MUL == 1 ? r + d : d == 1 ? C::HALF + r : r + d / 2;
                ua[u][t][d] = 128 * row + 16 * (uchunk ^ C::u_turn(row)) + half;
            }
#pragma unroll
            for (int b = 0; b < RB; ++b) va[u][t][b] = C::ubytes + C::VP * r + 16 * ((vchunk + 4 * b) ^ C::v_turn(r)) + half;
            x[u][t] = y[u][t] = 0;
            if (GATHER) { int img; place((uint32_t)k_begin + r, x[u][t], y[u][t], img); }
        }
    if (threadIdx.x < 64) *reinterpret_cast<uint32_t*>(lds + C::zeros + 4 * threadIdx.x) = 0;

    f32x16 acc[T][RB];
#pragma unroll
    for (int d = 0; d < T; ++d)
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[d][b][v] = 0.0f;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;      // address within the LDS
    const uint32_t none = lds0 + C::zeros + half;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) request();
    for (int s = 0; s < nslab; ++s) {
        if (full) wait_newest<NE * (NS - 2)>();            // slab s is there (this wave's part of it)
        else wait_newest<(NE - 1) * (NS - 2)>();
        lds_barrier();                                     // all of it; and slab s - 1 is read
        request();
        const uint32_t base = lds0 + from;
        from = next_slot(from);
        const int left = rows - s * BP;
#pragma unroll
        for (int u = 0; u < C::STEPS; ++u) {
            constexpr int N = T + RB;                      // operands, a load each for t = 0 and 1
            uint32_t at[2 * N];
            u32x2 o[2 * N];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                bool in[3] = {true, true, true};
                if (GATHER) {
                    const int r = 16 * (ks * C::STEPS + u) + 8 * (grp >> 1) + 4 * t + (i >> 2), cx = MUL * x[u][t];
                    in[1] = r < left && (unsigned)(MUL * y[u][t] + dy) < (unsigned)g.H;
                    in[0] = in[1] && cx >= 1;
                    in[2] = in[1] && cx + 1 < g.W;
                    int img = 0;
                    advance(x[u][t], y[u][t], img);
                }
#pragma unroll
                for (int d = 0; d < T; ++d) at[N * t + d] = in[d] ? base + ua[u][t][d] : none;
#pragma unroll
                for (int b = 0; b < RB; ++b) at[N * t + T + b] = base + va[u][t][b];
            }
            load_transposed<2 * N>(at, o);
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int d = 0; d < T; ++d)
                    acc[d][b] = mfma_bf16(u32x4{o[d][0], o[d][1], o[N + d][0], o[N + d][1]}, u32x4{o[T + b][0], o[T + b][1], o[N + T + b][0], o[N + T + b][1]}, acc[d][b]);
        }
    }
    wait_newest<0>();                                      // nothing is on its way to LDS any more

    // ---- sums of the four parts, one tap at a time; accumulator v of block b: channel 8 (v / 4) + 4 (lane / 32) + v % 4, column 32 b + lane % 32
    float* part = job.part + (int64_t)split * job.P * R;
    f32x4* sums = reinterpret_cast<f32x4*>(lds);           // [channel block][part of the pixels][b][v / 4][lane]
#pragma unroll
    for (int d = 0; d < T; ++d) {
        lds_barrier();
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                sums[(((cw * 4 + ks) * RB + b) * 4 + q) * 64 + lane] = f32x4{acc[d][b][4 * q], acc[d][b][4 * q + 1], acc[d][b][4 * q + 2], acc[d][b][4 * q + 3]};
        lds_barrier();
#pragma unroll
        for (int n = 0; n < RB; ++n) {                     // 2 RB 256 values of four, 512 threads
            const int at = 512 * n + (int)threadIdx.x, ln = at & 63, q = (at >> 6) & 3, b = (at >> 8) % RB, block = (at >> 8) / RB;
            f32x4 v = sums[((block * 4 * RB + b) * 4 + q) * 64 + ln];
#pragma unroll
            for (int k = 1; k < 4; ++k) v += sums[(((block * 4 + k) * RB + b) * 4 + q) * 64 + ln];
            const int ch = 32 * block + 8 * q + 4 * (ln >> 5), col = 32 * b + (ln & 31);
            if (GATHER) {                                  // laid out [R, P]
                gstore(reinterpret_cast<f32x4*>(part + (int64_t)col * job.P + (ky * 3 + d) * g.C + c0 + ch), v);
            } else if (c0 + 64 * d < job.P) {
#pragma unroll
                for (int k = 0; k < 4; ++k) gstore(part + (int64_t)(c0 + 64 * d + ch + k) * R + col, (float)v[k]);
            }
        }
    }
}

template <int R, int MUL>
__global__ __launch_bounds__(512, 1) void taps_kernel(Tn2Args args) {
    extern __shared__ __align__(1024) unsigned char lds[];
    // every XCD takes a contiguous eighth of the (split, tile) pairs, so the tiles of a split share its rows through one L2
    const int pair = ((int)blockIdx.x & 7) * ((int)gridDim.x >> 3) + ((int)blockIdx.x >> 3);
    if (pair >= args.tiles * args.splits) return;
    const int tile = pair % args.tiles, split = pair / args.tiles;
    const int jid = args.njobs > 1 && tile >= args.job[1].tile_begin ? 1 : 0;
    const Tn2Job job = args.job[jid];
    const int local = tile - job.tile_begin;
    if (job.gather) {
        const int blocks = args.g.C / 64;
        taps_tile<R, MUL, true>(args, job, lds, local % blocks * 64, local / blocks, split);
    } else {
        taps_tile<R, MUL, false>(args, job, lds, local * 128, 0, split);
    }
}

template <int R, int MUL>
hipError_t launch(const Tn2Args& a, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&taps_kernel<R, MUL>), hipFuncAttributeMaxDynamicSharedMemorySize, Taps<R, MUL>::lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((taps_kernel<R, MUL>), dim3(8 * ((a.tiles * a.splits + 7) / 8)), dim3(512), (Taps<R, MUL>::lds), s, a);
    return hipGetLastError();
}

}  // namespace

int taps_rows(int R) { return R <= 64 ? 128 : 64; }

int taps_tiles(const TnJob& job, const Tn2Gather* g) { return g ? g->C / 64 * g->kh : (job.P + 127) / 128; }

int taps_splits(const TnJob* jobs, int njobs, const Tn2Gather& g, int64_t M, int R) {
    int tiles = 0;
    for (int i = 0; i < njobs; ++i) tiles += taps_tiles(jobs[i], i == njobs - 1 ? &g : nullptr);
    int64_t want = 256 / tiles;                            // one work-group per compute unit
    const int64_t by_rows = M / 512;
    if (want > by_rows) want = by_rows;
    return want < 1 ? 1 : want > 64 ? 64 : (int)want;
}

bool taps_supports(const TnJob* jobs, int njobs, const Tn2Gather& g, int64_t M, int R, int splits) {
    if (g.kw != 3 || g.C % 64 || (R != 32 && R != 64 && R != 96) || (int64_t)g.RH * g.RW < taps_rows(R)) return false;
    if (njobs > 1 && jobs[0].P % 64) return false;
    // 32-bit offsets inside a split, the slabs that are requested past its end included
    const int64_t rps = ceil_div(ceil_div(M, splits), taps_rows(R)) * taps_rows(R) + 8 * taps_rows(R);
    const int64_t row = njobs > 1 && jobs[0].P > R ? jobs[0].P : R;
    const int64_t window = (int64_t)g.mul * g.mul * (rps + g.RW + 2) + 2 * (int64_t)g.mul * g.W + 2 * ((int64_t)g.kh * g.W + 2);
    return rps * row * 2 < kBufMaxBytes && window * g.C * 2 < kBufMaxBytes;
}

hipError_t launch_taps(const Tn2Args& a, int R, hipStream_t s) {
    const bool two = a.g.mul == 2;
    switch (R) {
#define ABT_CASE(RR) case RR: return two ? launch<RR, 2>(a, s) : launch<RR, 1>(a, s);
        ABT_CASE(32) ABT_CASE(64) ABT_CASE(96)
#undef ABT_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace abt
