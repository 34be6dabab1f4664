// Chain kernel for narrow ranks (R <= 192), several small work-groups per compute unit:
//     Tout[M,R] = Xin[M,p] . P[R,p]^T  then  Yout[M,q] = Tout . Q[q,R]^T        (bf16 in, fp32 accumulate)
//
// What bounds it: at these ranks the layer moves about as many bytes as it has matrix work for, so the
// activations have to stream at memory rate while the factors come out of L2.  One work-group of
// specialised waves per compute unit (lr_chain2.hip) waits a whole load latency at each of its barriers
// and has nobody else to run meanwhile; here a work-group is four waves with 26 to 67 KB of LDS, and two
// or three of them share a compute unit (39597 x 3072 -> 768 at r = 96: 98 -> 82 us; 100000 x 768 -> 768 at r = 160:
// 136 -> 93; a 3 x 3 forward on 256 x 28 x 28 x 128 at r = 64: 150 -> 85).
//
//   * A wave owns 32 rows through both stages, and each activation element is used by one wave only.
//     From a matrix the wave loads whole 128-byte lines (slabs of 64 columns, two slabs ahead in registers)
//     and turns them into operands through an LDS tile of its own, without a barrier.  From an image (a
//     convolution's patches) each lane has one pixel for the whole kernel and loads the 16-byte pieces of
//     its operand directly: a tap is one range check per lane, and neighbouring pixels keep the lines in
//     L1.  (The direct loads on a matrix: 14 % slower at 39597 x 3072, r = 64 to 192.  The tile on an
//     image: four pixels per lane, spills, the 3 x 3 layers 25 % slower.)  Where the window of the image that a row block's
//     patches touch is small (stride 1, up to 256 pixels), it goes to LDS once per 64 channels and all taps read it there.
//   * The factors are shared by the four waves: slabs of 64 columns of P, then 64 rows of Q, travel
//     through registers (two slabs ahead) into two LDS buffers, one barrier per slab.
//   * The first operand's rows are fed in the order pi() (two bits of the row number swapped), so that the
//     accumulator registers of a lane hold eight consecutive columns of the result: T is packed in
//     place into the operand of stage 2, without LDS or lane exchange.
//   * Results leave through a 32 x 64 staging tile per wave (no barrier) as whole 128-byte lines.
//
// MFMA 32x32x16 bf16 layout (lane l, h = l / 32): A operand = 8 values A[l % 32][8h .. 8h+7], B operand
// = B[8h .. 8h+7][l % 32], accumulator v = C[8 (v / 4) + 4h + v % 4][l % 32].
#include <atomic>

#include "common.h"
#include "grid_window.h"

namespace abt {

namespace {

__device__ __forceinline__ f32x16 mfma16(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// this wave's LDS traffic has completed, then s_barrier; global loads in flight stay in flight
__device__ __forceinline__ void wg_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// order of a wave's own LDS accesses (they execute in order; this pins the compiler)
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kMaxRows = 128, NT = 256;
constexpr int kWinPieces = 8;                        // image window in LDS: 16-byte pieces per thread
static_assert(kMaxWindow == 32 * kWinPieces, "pixels of 64 channels");
// Where the first operand comes from: a matrix; an image, per lane; an image through a window in LDS (one block of 64 channels;
// several, with nine taps).
enum Source { kMatrix, kGather, kWindow, kWindows };
constexpr int kStagePitch = 64 * 2 + 16;             // staging tile: 32 rows x 64 columns, rows 36 words apart
constexpr int kStage = 32 * kStagePitch;

template <int R>
struct C4 {
    static constexpr int CB = R / 32, KB = R / 16;
    static constexpr int slab = R * 128;                 // R rows x 64 columns of P, or 64 rows x R columns of Q
    static constexpr int lds_bytes = 2 * slab + 4 * kStage;
    static constexpr int NCH = R / 32;                   // 16-byte chunks per thread and slab
    static constexpr int CPR2 = R / 8;                   // chunks per row of Q
    // the swizzle XORs the low XB bits of a Q row's chunk index with row bits (16 consecutive rows, one chunk:
    // 16 different bank groups)
    static constexpr int XB = CPR2 % 16 == 0 ? 4 : (CPR2 % 8 == 0 ? 3 : 2);
    static constexpr int PER = (1 << XB) / 2;
    // Slabs in flight per wave beside the one in use (3 and 4 measured the same, and spilled at R >= 96), and
    // work-groups per compute unit by registers (512 per lane and SIMD) and LDS (160 KB).
    static constexpr int D = 2;
    template <Source S> static constexpr int occupancy() { return R <= 96 || ((S == kGather || S == kWindow) && R == 128) ? 3 : 2; }
    static constexpr int U = D % 2 ? 2 * D : D;          // unrolled slabs: whole turns of the ring and of the two LDS buffers
};
template <int XB>
__device__ __forceinline__ int row_key(int row) {
    if constexpr (XB == 4) return row & 15;
    else if constexpr (XB == 3) return (row >> 1) & 7;
    else return (row >> 2) & 3;
}

struct C4Entry {
    const uint16_t* X; const uint16_t* P; const uint16_t* Q;
    uint16_t* Y; uint16_t* T;
    int64_t M;
    int p;
    ChainGather g;
};
struct C4Args {
    C4Entry e[kChainMaxGroups];
    int q, t_pitch, parts, stream_out;
    int rows;                                            // per work-group: four waves of rows / 4 <= 32
    int win_slots;                                       // pixels that the window in LDS holds, a multiple of 8
};

template <int R, Source SRC>
__global__ __launch_bounds__(NT, (C4<R>::template occupancy<SRC>())) void chain4_bf16_kernel(C4Args args) {
    extern __shared__ __align__(1024) unsigned char lds[];
    using C = C4<R>;
    constexpr bool GATHER = SRC != kMatrix, WINDOW = SRC == kWindow || SRC == kWindows;
    constexpr int CB = C::CB, KB = C::KB, NCH = C::NCH, D = C::D, U = C::U;
    const C4Entry en = args.e[blockIdx.y];
    const int64_t M = en.M;
    const int p = en.p, q = args.q, t_pitch = args.t_pitch;
    uint16_t* const Yout = en.Y;
    uint16_t* const Tout = en.T;
    // `parts` work-groups share a row block: each repeats stage 1 and does its share of the output tiles
    const int rb = (int)blockIdx.x / args.parts, part = (int)blockIdx.x - rb * args.parts;
    const int rows = args.rows, wrows = rows >> 2;
    const int64_t row0 = (int64_t)rb * rows;
    if (row0 >= M || (Yout == nullptr && Tout == nullptr)) return;       // uniform over the work-group
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lj = lane & 31, lh = lane >> 5;
    const int pj = (lj & 16) | ((lj & 4) << 1) | ((lj & 8) >> 1) | (lj & 3);       // pi(lj)
    const int rows_valid = M - row0 < rows ? (int)(M - row0) : rows;
    // row i of this wave is row wave wrows + i of the work-group; nowhere if it is another wave's or past M
    auto row_of = [&](int i) { const int r = (tid >> 6) * wrows + i; return i < wrows && r < rows_valid ? r : -1; };

    // ------------------------------------------------------------------ stage 1
    const int ns1 = p / 64;
    const int rot1 = (int)((unsigned)rb % (unsigned)ns1);    // work-groups start at different slabs
    f32x16 acc[CB];
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.0f;

    // activation, from a matrix: this lane fetches chunk sch of rows 8 e + srow of the wave's 32;
    // from an image: the pieces of row lj that its operand holds (columns 16 j + 8 h .. + 7 in step j)
    const int srow = lane >> 3, sch = lane & 7;
    int xoff[4], gy = 0, gx = 0, xslab = rot1, xcb = 0, xky = 0, xkx = 0;
    const ChainGather g = en.g;
    rsrc_t xres;
    if constexpr (GATHER) {
        // pixels that the work-group's patches can touch: the centres of its first and last grid row and the reach
        const int per = g.RH * g.RW;
        auto centre = [&](int64_t i, int end) -> int64_t {
            const int64_t img = i / per;
            const int rem = (int)(i - img * per), y = rem / g.RW, x = end ? g.RW - 1 : 0;
            return (img * g.H + (int64_t)g.mul * y) * g.W + (int64_t)g.mul * x;
        };
        const int ry = g.cy > g.kh - 1 - g.cy ? g.cy : g.kh - 1 - g.cy, rx = g.cx > g.kw - 1 - g.cx ? g.cx : g.kw - 1 - g.cx;
        const int64_t reach = (int64_t)ry * g.W + rx, pixels = (M / per) * g.H * g.W;
        auto pixel_of = [&](int64_t i) -> int64_t {      // mul = 1
            const int64_t img = i / per;
            const int rem = (int)(i - img * per), y = rem / g.RW;
            return (img * g.H + y) * g.W + (rem - y * g.RW);
        };
        const int64_t c0 = WINDOW ? pixel_of(row0) : centre(row0, 0), c1 = WINDOW ? pixel_of(row0 + rows_valid - 1) : centre(row0 + rows_valid - 1, 1);
        const int64_t p0 = c0 > reach ? c0 - reach : 0, p1 = c1 + reach + 1 < pixels ? c1 + reach + 1 : pixels;
        xres = make_rsrc(en.X + p0 * g.Cin, (p1 - p0) * g.Cin * 2);
        const int row = row_of(lj);
        const int i = (int)row0 + (row < 0 ? 0 : row), img = i / per;    // M fits an int (checked by the launcher)
        const int rem = i - img * per, y = rem / g.RW, x = rem - y * g.RW;
        gx = g.mul * x;
        gy = row >= 0 ? g.mul * y : -(1 << 24);                  // no row: never inside the image
        const int64_t own = ((int64_t)img * g.H + (int64_t)g.mul * y) * g.W + gx - p0;
        xoff[0] = WINDOW ? (int)own : (int)(own * g.Cin + 8 * lh) * 2;       // (window: the slot of the centre)
        const int tap = WINDOW ? (int)((unsigned)rb % (unsigned)(g.kh * g.kw)) : rot1 / g.cpb;
        if (!WINDOW) xcb = rot1 - tap * g.cpb;
        xky = tap / g.kw;
        xkx = tap - xky * g.kw;
    } else {
        xres = make_rsrc(en.X + row0 * p, (int64_t)rows_valid * p * 2);
#pragma unroll
        for (int e = 0; e < 4; ++e) xoff[e] = row_of(8 * e + srow) < 0 ? kBufNowhere : (row_of(8 * e + srow) * p + 8 * sch) * 2;
    }
    auto load_x = [&](u32x4 (&d)[4]) {                   // the next slab, in order, wrapping around
        if constexpr (GATHER) {
            const int dy = g.sign * (xky - g.cy), dx = g.sign * (xkx - g.cx);
            const int shift = ((dy * g.W + dx) * g.Cin + xcb * 64) * 2;
            const bool ok = (unsigned)(gy + dy) < (unsigned)g.H && (unsigned)(gx + dx) < (unsigned)g.W;
            const int left = ok ? g.Cin - xcb * 64 - 8 * lh : 0;         // channels beyond Cin read zeros
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = buf_load16(xres, 16 * j < left ? xoff[0] + shift + 32 * j : kBufNowhere, 0);
            if (++xcb == g.cpb) { xcb = 0; if (++xkx == g.kw) { xkx = 0; if (++xky == g.kh) xky = 0; } }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) d[e] = buf_load16(xres, xoff[e], xslab * 128);
            if (++xslab == ns1) xslab = 0;
        }
    };
    // the wave's own tile: 32 rows of 128 bytes, chunks XOR-swizzled by the row; later its output staging tile
    unsigned char* const stage = lds + 2 * C::slab + wave * kStage;
    const int xdst = srow * 128 + ((sch ^ ((srow >> 1) & 7)) << 4);      // row 8 e + srow: key differs by 4 for odd e
    auto store_x = [&](const u32x4 (&v)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) *reinterpret_cast<u32x4*>(stage + (xdst ^ ((e & 1) << 6)) + e * 1024) = v[e];
    };
    const int xread = lj * 128 + ((lh ^ ((lj >> 1) & 7)) << 4);
    // factor slab: thread t fetches chunk t % 8 of rows t / 8 + 32 e
    const rsrc_t pres = make_rsrc(en.P, (int64_t)R * p * 2);
    const int pr = tid >> 3, pc = tid & 7;
    const int psrc = (pr * p + pc * 8) * 2;
    const int pdst = pr * 128 + ((pc ^ ((pr >> 1) & 7)) << 4);
    int pslab = rot1;
    // window: taps in turn from the first on, then the next block of channels
    const int taps = WINDOW ? g.kh * g.kw : 1;
    int ptap = WINDOW ? xky * g.kw + xkx : 0, pleft = taps, pcb = 0;
    if constexpr (WINDOW) pslab = ptap * g.cpb;
    auto load_p = [&](u32x4 (&d)[NCH]) {
#pragma unroll
        for (int e = 0; e < NCH; ++e) d[e] = buf_load16(pres, psrc, pslab * 128 + e * 64 * p);
        if constexpr (WINDOW) {
            if (++ptap == taps) ptap = 0;
            if (--pleft == 0) { pleft = taps; if (++pcb == g.cpb) pcb = 0; }
            pslab = ptap * g.cpb + pcb;
        } else if (++pslab == ns1) pslab = 0;
    };
    auto store_p = [&](const u32x4 (&v)[NCH], int buf) {
#pragma unroll
        for (int e = 0; e < NCH; ++e) *reinterpret_cast<u32x4*>(lds + buf * C::slab + pdst + e * 4096) = v[e];
    };
    const int pread = pj * 128 + ((lh ^ ((pj >> 1) & 7)) << 4);
    u32x4 fr[D][NCH];
    if constexpr (WINDOW) {
        // The image window of the row block, a block of 64 channels at a time: pixels of 128 bytes, chunks XOR-swizzled by the
        // pixel, a row of zeros behind them.  It is loaded once, as whole lines, and every tap reads its operands there: pixel
        // shift and range check are an address (outside the image: the zeros).  Loading each tap's pieces from memory
        // instead, 32 lines per instruction and 9 instructions for each 16 bytes, is bound by those requests: forward,
        // batch 256, 14 x 14 x 256, r = 64 41 -> 30 us, r = 32 37 -> 23; 28 x 28 x 128, r = 64 74 -> 50, r = 192 125 -> 118; activation gradient
        // of 56 x 56 x 64, batch 100, r = 128 153 -> 94, r = 256 283 -> 154.  Now the LDS reads are the most of a slab (48 KB at R = 64 for
        // 256 cycles of matrix instructions, each wave reading all of P).
        static_assert(D == 2, "ring parity");
        unsigned char* const win = lds + 2 * C::slab;
        const int slots = args.win_slots;
        const int wch = tid & 7;
        const int wsrc = ((tid >> 3) * g.Cin + 8 * wch) * 2, wstep = 32 * g.Cin * 2;
        unsigned char* const wdst = win + (tid >> 3) * 128 + ((wch ^ ((tid >> 4) & 7)) << 4);
        u32x4 wr[kWinPieces];
        auto load_w = [&](u32x4& d, int e, int cb) {     // past the window, the channels or the last block: zeros
            d = buf_load16(xres, cb * 64 + 8 * wch < g.Cin && cb < g.cpb ? wsrc + e * wstep : kBufNowhere, cb * 128);
        };
        auto store_w = [&]() {
#pragma unroll
            for (int e = 0; e < kWinPieces; ++e)
                if (32 * e + (tid >> 3) < slots) *reinterpret_cast<u32x4*>(wdst + e * 4096) = wr[e];
        };
#pragma unroll
        for (int e = 0; e < kWinPieces; ++e) load_w(wr[e], e, 0);
        load_p(fr[0]);
        load_p(fr[1]);
        if (tid < 8) *reinterpret_cast<u32x4*>(win + slots * 128 + tid * 16) = u32x4{0, 0, 0, 0};
        store_w();
        store_p(fr[0], 0);
        load_p(fr[0]);
        wg_barrier();
        int cb = 0;
        auto slab1 = [&](const int u, const int e) __attribute__((always_inline)) {     // u: parity of the slab; e: piece of the next window
            store_p(fr[(u + 1) & 1], (u & 1) ^ 1);
            load_p(fr[(u + 1) & 1]);
            if constexpr (SRC == kWindows) { if (e < kWinPieces) load_w(wr[e], e, cb + 1); }
            __builtin_amdgcn_sched_barrier(0);
            const int dy = g.sign * (xky - g.cy), dx = g.sign * (xkx - g.cx), w = xoff[0] + dy * g.W + dx;
            const bool ok = (unsigned)(gy + dy) < (unsigned)g.H && (unsigned)(gx + dx) < (unsigned)g.W;
            const int xa = ok ? w * 128 + ((lh ^ ((w >> 1) & 7)) << 4) : slots * 128;
            if (++xkx == g.kw) { xkx = 0; if (++xky == g.kh) xky = 0; }
            const unsigned char* base = lds + (u & 1) * C::slab;
            u32x4 xf[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) xf[j] = *reinterpret_cast<const u32x4*>(win + (xa ^ (j << 5)));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int b = 0; b < CB; ++b)
                    acc[b] = mfma16(*reinterpret_cast<const u32x4*>(base + (pread ^ (j << 5)) + b * 4096), xf[j], acc[b]);
            }
            wg_barrier();
        };
        if constexpr (SRC == kWindow) {
            int s1 = 0;
            for (; s1 + 2 <= taps; s1 += 2) { slab1(0, 0); slab1(1, 0); }
            if (s1 < taps) slab1(0, 0);
        } else {
            auto block = [&](const int u) __attribute__((always_inline)) {       // nine taps, the first of parity u
#pragma unroll
                for (int i = 0; i < 9; ++i) slab1(u + i, i);
                store_w();
                wg_barrier();
                ++cb;
            };
            while (cb + 2 <= g.cpb) { block(0); block(1); }
            if (cb < g.cpb) block(0);
        }
    } else {
        u32x4 xr[D][4];
#pragma unroll
        for (int d = 0; d < D; ++d) { load_p(fr[d]); load_x(xr[d]); }
        store_p(fr[0], 0);
        load_p(fr[0]);
        wg_barrier();                                        // slab 0 is in buffer 0
        auto slab1 = [&](const int u) __attribute__((always_inline)) {     // u: the slab's place in the unrolled loop
            const int d = u % D, d1 = (u + 1) % D;
            if constexpr (!GATHER) store_x(xr[d]);
            store_p(fr[d1], (u & 1) ^ 1);
            load_p(fr[d1]);
            if constexpr (!GATHER) { load_x(xr[d]); wave_lds_order(); }
            __builtin_amdgcn_sched_barrier(0);
            const unsigned char* base = lds + (u & 1) * C::slab;
            u32x4 xf[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) xf[j] = GATHER ? xr[d][j] : *reinterpret_cast<const u32x4*>(stage + (xread ^ (j << 5)));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int b = 0; b < CB; ++b)
                    acc[b] = mfma16(*reinterpret_cast<const u32x4*>(base + (pread ^ (j << 5)) + b * 4096), xf[j], acc[b]);
            }
            if constexpr (GATHER) load_x(xr[d]); else wave_lds_order();
            wg_barrier();                                    // this slab's buffer may be overwritten, the other one is filled
        };
        // whole turns without a branch inside (a path that skips slabs would make the compiler wait for the
        // youngest loads at the top of every turn), then the rest
        int s1 = 0;
        for (; s1 + U <= ns1; s1 += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) slab1(u);
        }
#pragma unroll
        for (int u = 0; u + 1 < U; ++u)
            if (s1 + u < ns1) slab1(u);
    }

    // ------------------------------------------------------------------ stage 2's first factor slabs, and T
    const int ntile_all = q >> 6;
    const int tile0 = (int)((int64_t)part * ntile_all / args.parts), ntile = (int)((int64_t)(part + 1) * ntile_all / args.parts) - tile0;
    int qtile = tile0 + (ntile > 0 ? (int)((unsigned)rb % (unsigned)ntile) : 0);
    const int first_tile = qtile;
    auto load_q = [&](u32x4 (&d)[NCH]) {
        const rsrc_t qres = make_rsrc(en.Q + (int64_t)qtile * 64 * R, 64 * R * 2);
#pragma unroll
        for (int e = 0; e < NCH; ++e) d[e] = buf_load16(qres, tid * 16, e * (NT * 16));
        if (++qtile == tile0 + ntile) qtile = tile0;
    };
    int qdst[NCH];                                       // chunk ci = e NT + t of a slab: row ci / CPR2, chunk ci % CPR2
#pragma unroll
    for (int e = 0; e < NCH; ++e) {
        const int ci = e * NT + tid, row = ci / C::CPR2, ch = ci % C::CPR2;
        qdst[e] = row * (R * 2) + ((ch ^ row_key<C::XB>(row)) << 4);
    }
    auto store_q = [&](const u32x4 (&v)[NCH], int buf) {
#pragma unroll
        for (int e = 0; e < NCH; ++e) *reinterpret_cast<u32x4*>(lds + buf * C::slab + qdst[e]) = v[e];
    };
    if (Yout != nullptr) {
#pragma unroll
        for (int d = 0; d < D; ++d) load_q(fr[d]);
    }

    // T rounded to bf16: registers 8 k .. 8 k + 7 of block b are columns 32 b + 16 k + 8 h .. + 7 of row lj
    u32x4 tf[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            tf[kb][i] = pack2_bf16(acc[kb >> 1][8 * (kb & 1) + 2 * i], acc[kb >> 1][8 * (kb & 1) + 2 * i + 1]);

    // (what a lane moves out: chunk sch of rows 8 i + srow)
    if (Tout != nullptr && part == 0) {
        int trow[4];
        rsrc_t tres;
        if constexpr (GATHER) {
            // result rows are pixels of a grid OH x OW, omul apart
            const int per = g.RH * g.RW;
            auto pixel = [&](int64_t i) -> int64_t {
                const int64_t img = i / per;
                const int rem = (int)(i - img * per), y = rem / g.RW, x = rem - y * g.RW;
                return (img * g.OH + g.omul * y + g.oy) * g.OW + g.omul * x + g.ox;
            };
            const int64_t first = pixel(row0), last = pixel(row0 + rows_valid - 1);
            tres = make_rsrc(Tout + first * t_pitch, ((last - first) * t_pitch + R) * 2);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = row_of(8 * i + srow);
                trow[i] = r >= 0 ? (int)(pixel(row0 + r) - first) * t_pitch * 2 : kBufNowhere;
            }
        } else {
            tres = make_rsrc(Tout + row0 * t_pitch, ((int64_t)(rows_valid - 1) * t_pitch + R) * 2);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = row_of(8 * i + srow);
                trow[i] = r >= 0 ? r * t_pitch * 2 : kBufNowhere;
            }
        }
#pragma unroll
        for (int c0 = 0; c0 < KB; c0 += 4) {             // 64 columns at a time
            wave_lds_order();
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (c0 + k < KB) *reinterpret_cast<u32x4*>(stage + lj * kStagePitch + (16 * k + 8 * lh) * 2) = tf[c0 + k];
            wave_lds_order();
            if (c0 * 2 + sch < C::CPR2) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(stage + (8 * i + srow) * kStagePitch + sch * 16);
                    const int off = trow[i] == kBufNowhere ? kBufNowhere : trow[i] + c0 * 32 + sch * 16;
                    buf_store16_maybe_stream(args.stream_out != 0, v, tres, off, 0);
                }
            }
        }
    }
    if (Yout == nullptr || ntile == 0) return;

    // ------------------------------------------------------------------ stage 2
    const rsrc_t yres = make_rsrc(Yout + row0 * q, (int64_t)rows_valid * q * 2);
    int yrow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) yrow[i] = row_of(8 * i + srow) < 0 ? kBufNowhere : (row_of(8 * i + srow) * q + sch * 8) * 2;
    const int qkey = row_key<C::XB>(pj);
    const int qread = pj * (R * 2) + ((lh ^ qkey) << 4);
    store_q(fr[0], 0);
    load_q(fr[0]);
    wg_barrier();
    int out_tile = first_tile;
    auto tile2 = [&](const int u) __attribute__((always_inline)) {
        store_q(fr[(u + 1) % D], (u & 1) ^ 1);
        load_q(fr[(u + 1) % D]);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned char* base = lds + (u & 1) * C::slab;
        f32x16 o[2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[b][v] = 0.0f;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                o[b] = mfma16(*reinterpret_cast<const u32x4*>(base + (qread ^ ((kb % C::PER) << 5)) + (kb / C::PER) * (16 << C::XB) +
                                                              b * 32 * (R * 2)), tf[kb], o[b]);
        wave_lds_order();
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const u32x4 v = {pack2_bf16(o[b][8 * k], o[b][8 * k + 1]), pack2_bf16(o[b][8 * k + 2], o[b][8 * k + 3]),
                                 pack2_bf16(o[b][8 * k + 4], o[b][8 * k + 5]), pack2_bf16(o[b][8 * k + 6], o[b][8 * k + 7])};
                *reinterpret_cast<u32x4*>(stage + lj * kStagePitch + (32 * b + 16 * k + 8 * lh) * 2) = v;
            }
        wave_lds_order();
        u32x4 out[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) out[r] = *reinterpret_cast<const u32x4*>(stage + (8 * r + srow) * kStagePitch + sch * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            buf_store16_maybe_stream(args.stream_out != 0, out[r], yres, yrow[r], out_tile * 128);
        if (++out_tile == tile0 + ntile) out_tile = tile0;
        wg_barrier();
    };
    int t1 = 0;
    for (; t1 + U <= ntile; t1 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) tile2(u);
    }
#pragma unroll
    for (int u = 0; u + 1 < U; ++u)
        if (t1 + u < ntile) tile2(u);
}

// pixels from a row block's first patch to its last (mul = 1)
int64_t window_pixels(const ChainGather& g, int rows) {
    const int64_t ry = g.cy > g.kh - 1 - g.cy ? g.cy : g.kh - 1 - g.cy, rx = g.cx > g.kw - 1 - g.cx ? g.cx : g.kw - 1 - g.cx;
    return (g.RH == g.H && g.RW == g.W ? rows : grid_window(rows, g.RH, g.RW, 1, g.H, g.W)) + 2 * (ry * g.W + rx);
}

template <int R, Source SRC>
hipError_t launch_r(const C4Args& args, int G, int64_t blocks, hipStream_t s) {
    static_assert(2 * C4<R>::slab + (kMaxWindow + 1) * 128 <= 160 * 1024 && C4<R>::lds_bytes <= 160 * 1024, "LDS budget");
    constexpr bool window = SRC == kWindow || SRC == kWindows;
    constexpr int largest = window ? 2 * C4<R>::slab + (kMaxWindow + 1) * 128 : C4<R>::lds_bytes;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&chain4_bf16_kernel<R, SRC>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, largest);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    int bytes = C4<R>::lds_bytes;                        // (the staging tiles lie over the window)
    if (window && 2 * C4<R>::slab + (args.win_slots + 1) * 128 > bytes) bytes = 2 * C4<R>::slab + (args.win_slots + 1) * 128;
    hipLaunchKernelGGL((chain4_bf16_kernel<R, SRC>), dim3((unsigned)(blocks * args.parts), (unsigned)G), dim3(NT), bytes, s, args);
    return hipGetLastError();
}

template <Source SRC>
hipError_t launch_any(int R, const C4Args& args, int G, int64_t blocks, hipStream_t s) {
    switch (R) {
#define ABT_CASE(RR) case RR: return launch_r<RR, SRC>(args, G, blocks, s);
        ABT_CASE(32) ABT_CASE(64) ABT_CASE(96) ABT_CASE(128) ABT_CASE(160) ABT_CASE(192)
#undef ABT_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool chain4_window(const ChainGather& g, int R, int rows) {
    const int taps = g.kh * g.kw, cpb = (g.Cin + 63) / 64;
    if (g.mul != 1 || taps < 2 || (cpb > 1 && taps != 9)) return false;
    const int64_t w = window_pixels(g, rows);
    return window_fits(R, w) && !(R == 128 && cpb == 1 && w > 192) && !(R >= 128 && g.Cin <= 32);
}

bool chain4_supports(int R, int p, int q) {
    return R >= 32 && R <= 192 && R % 32 == 0 && p >= 64 && p % 64 == 0 && q % 64 == 0 && p <= (1 << 20) && q <= (1 << 20);
}

hipError_t launch_chain4_bf16(const ChainProblem* problems, int G, int64_t M, int p, int q, int R, int t_pitch, int rows, int parts, hipStream_t s) {
    if (rows < 4 || rows > kMaxRows || rows % 4) return hipErrorInvalidValue;
    if (!problems || G < 1 || G > kChainMaxGroups || parts < 1 || !chain4_supports(R, p, q) || M < 1 || t_pitch < R) return hipErrorInvalidValue;
    C4Args a{};
    for (int g = 0; g < G; ++g) {
        const ChainProblem& c = problems[g];
        a.e[g] = C4Entry{(const uint16_t*)c.Xin, (const uint16_t*)c.P, (const uint16_t*)c.Q, (uint16_t*)c.Yout, (uint16_t*)c.Tout, M, p, ChainGather{}};
        if (c.Yout == nullptr && parts != 1) return hipErrorInvalidValue;
    }
    if (parts > q / 64) return hipErrorInvalidValue;
    const int64_t out_bytes = M * ((problems[0].Yout ? q : 0) + R) * 2;
    a.q = q; a.t_pitch = t_pitch; a.rows = rows; a.parts = parts; a.stream_out = out_bytes >= kStreamOutBytes;
    return launch_any<kMatrix>(R, a, G, ceil_div(M, rows), s);
}

hipError_t launch_chain4_gather_bf16(const GatherProblem* problems, int n, int q, int R, int t_pitch, int rows, int parts, hipStream_t s) {
    if (rows < 4 || rows > kMaxRows || rows % 4) return hipErrorInvalidValue;
    if (!problems || n < 1 || n > kChainMaxGroups || t_pitch < R || parts < 1 || parts > 64) return hipErrorInvalidValue;
    C4Args a{};
    int64_t blocks = 0, out_bytes = 0, window = 0;
    bool second = false, single = true, windowed = true;
    const bool single_tap_ok = problems[0].g.kh * problems[0].g.kw > 1;         // the parities of a small window
    for (int i = 0; i < n; ++i) {
        const GatherProblem& c = problems[i];
        ChainGather g = c.g;
        g.cpb = (g.Cin + 63) / 64;
        const int64_t p = (int64_t)g.kh * g.kw * g.cpb * 64, per = (int64_t)g.RH * g.RW;
        if (p < 64 || p > (1 << 20) || !chain4_supports(R, (int)p, q) || g.H < 0 || g.W < 1 || g.Cin < 8 || g.Cin % 8 || g.kh < 1 || g.kw < 1 ||
            g.cy < 0 || g.cy >= g.kh || g.cx < 0 || g.cx >= g.kw || (g.sign != 1 && g.sign != -1) || g.RH < 0 || g.RW < 0 ||
            (g.mul != 1 && g.mul != 2) || (g.omul != 1 && g.omul != 2) || c.M > 0x7fffffff || (per ? c.M % per != 0 : c.M != 0) ||
            (g.omul == 2 && c.Yout))
            return hipErrorInvalidValue;
        // 32-bit offsets inside a row block's window of the image and of the result
        const int64_t reach = (int64_t)g.kh * g.W + g.kw;
        const int64_t span = grid_window(rows, g.RH, g.RW, g.mul, g.H, g.W) + 2 * reach;
        const int64_t ospan = grid_window(rows, g.RH, g.RW, g.omul, g.OH, g.OW);
        if (span * g.Cin * 2 >= kBufMaxBytes || ospan * t_pitch * 2 >= kBufMaxBytes || (int64_t)R * p * 2 >= kBufMaxBytes) return hipErrorInvalidValue;
        if (per && (c.M / per) * g.H * g.W > 0x7fffffff) return hipErrorInvalidValue;
        a.e[i] = C4Entry{(const uint16_t*)c.image, (const uint16_t*)c.P, (const uint16_t*)c.Q, (uint16_t*)c.Yout, (uint16_t*)c.Tout, c.M, (int)p, g};
        if (ceil_div(c.M, rows) > blocks) blocks = ceil_div(c.M, rows);
        if (g.mul == 1 && window_pixels(g, rows) > window) window = window_pixels(g, rows);
        windowed = windowed && (chain4_window(g, R, rows) || (single_tap_ok && g.kh * g.kw == 1 && g.mul == 1 && g.cpb == 1 && window_fits(R, window)));
        single = single && g.cpb == 1;
        out_bytes += c.M * ((c.Yout ? q : 0) + (c.Tout ? R : 0)) * 2;
        second |= c.Yout != nullptr;
    }
    if (parts > 1 && (!second || parts > q / 64)) return hipErrorInvalidValue;
    if (blocks == 0) return hipSuccess;
    a.q = q; a.t_pitch = t_pitch; a.rows = rows; a.parts = parts; a.stream_out = out_bytes >= kStreamOutBytes;
    a.win_slots = (int)(ceil_div(window, 8) * 8);
    if (windowed) return single ? launch_any<kWindow>(R, a, n, blocks, s) : launch_any<kWindows>(R, a, n, blocks, s);
    return launch_any<kGather>(R, a, n, blocks, s);
}

}  // namespace abt
