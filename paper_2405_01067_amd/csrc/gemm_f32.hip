// fp32 GEMM on the fp32 matrix cores of gfx950 (v_mfma_f32_32x32x2_f32), grouped over a list of
// independent problems.  Serves the fp32 flavour of the factored layer (all six products of the
// forward and backward), W = A B, and the merge's back-projections A' = Abar P_A, B' = P_B Bbar, Wbar = Abar Bbar.
//
// What bounds it: the matrix instruction takes 64 cycles for 4096 operations, so LDS bandwidth is never
// short; what has to be hidden is the latency of the global loads, and the chip has to be filled although
// the problems are small (outputs of 64 x 32 up to 3152 x 3072, contractions of 32 up to the batch size).
// Hence
//   * loads of 16 bytes per lane, two slabs ahead in registers beside two LDS buffers, and the traffic
//     of a slab dealt out between its matrix instructions,
//   * small tiles (64 x 64; 32 x 32 with the four waves sharing out the contraction for launches that
//     would not give every compute unit a tile), four work-groups per compute unit,
//   * a contraction over the batch (factor gradients) or, in a backward pass, over a long width (dT) is split over work-groups; the partial sums are
//     added in a fixed order by a second launch.
// Measured: 4096 x 4096 x 1024 279 to 302 us = 114 to 123 TFLOP/s by the card, a large library product of this size 139;
// 768 x 3072 x 384 (W = A B of a ViT-B/16 MLP layer) 26 us, 79 us in an earlier form with 128 x 128 tiles
// and 4-byte loads one slab ahead; the products of a factored layer at M = 3152, m = 3072, n = 768,
// r = 192: T 18 us, Y 46, dT 44 and 6, and dX, dA and dB in one launch 63 and 7; forward and backward together 161 us, 171 without work-groups
// that stay (gemm_stream).
//
// LDS: both operands lie [row][k], 16-byte chunks of four k XOR-swizzled by the row; an operand read is
// one 16-byte read for four matrix instructions: instruction i of a group of eight k takes k = 4 h + i
// from the lanes of half h, the same permutation of the contraction on both sides.  Operands stored
// with k slow are transposed on the way (four 4-byte stores per 16-byte load).
//
// MFMA 32x32x2 f32 register layout (lane l of 64): A operand = A[l % 32][l / 32],
// B operand = B[l / 32][l % 32], accumulator register v holds C[8*(v/4) + 4*(l/32) + v%4][l % 32].
#include <type_traits>

#include "common.h"

namespace abt {

namespace {

constexpr int NT = 256;

struct GemmF32Dev {
    GemmF32 d;
    int begin;           // problems in the kernel arguments: the XCD that its shares begin with; in a table: first tile
    int tiles_q, tiles;  // tiles per row of tiles, tiles of one split
    int splits, k_split; // splits of the contraction, columns of each (a multiple of 64)
    float* part;         // splits > 1: partial sums [split][P][Q]
};

// WR x WC x KS = 4 waves: row groups, column groups, contraction groups of a TM x TN tile
template <int TM_, int TN_, int WR_, int WC_, int KS_, int BK_>
struct GemmCfg {
    static constexpr int TM = TM_, TN = TN_, WR = WR_, WC = WC_, KS = KS_, BK = BK_;
    static constexpr int RA = TM / 32 / WR, CB = TN / 32 / WC;        // 32 x 32 blocks per wave
    static constexpr int GPW = BK / 8 / KS;                           // groups of eight k per wave and slab
    static constexpr int NVA = TM * BK / 4 / NT, NVB = TN * BK / 4 / NT;   // 16-byte loads per thread and slab
    static constexpr int slab = (TM + TN) * BK;                       // floats
    static constexpr int red = (KS - 1) * WR * WC * RA * CB * 16 * 64;    // floats: partial sums of the other contraction groups
    static constexpr int lds_floats = 2 * slab > red ? 2 * slab : red;
    static_assert(WR * WC * KS == 4 && NVA >= 1 && NVB >= 1 && GPW >= 1 && (BK == 32 || BK == 64), "tile shape");
};

// float index of chunk c (four k) of row r.  16 consecutive rows, same chunk, fall on 16 different
// 16-byte bank groups; the 4-byte stores of the transposing path (rows 4 apart) meet at most in pairs.
template <int BK>
__device__ __forceinline__ int lds_at(int r, int c) {
    if constexpr (BK == 64) return r * 64 + ((c ^ (r & 15) ^ ((r >> 4) & 1)) << 2);
    else return r * 32 + ((c ^ ((r >> 1) & 7) ^ ((r >> 4) & 1)) << 2);
}

// One operand of a tile: TR rows.  kc: k is the fast index in memory, else the row is.  Load e of a thread
// covers four k of row row0 + 1024 / BK e (kc), or four rows of k kfirst + 1024 / TR e.
template <int TR, int BK, bool VEC, bool KC>
struct Loader {
    static constexpr int NV = TR * BK / 4 / NT;
    static constexpr int ER = 1024 / BK, EK = 1024 / TR;      // distance of consecutive loads in rows (KC) / in k
    const float* base; const float* ptr[NV];
    int64_t step;
    int row0, kfirst, at, kend, first, rows, ld, klast;

    __device__ __forceinline__ void init(const float* m, int ld_, int tile_row, int rows_, int k0, int kend_, int K) {
        base = m; ld = ld_; first = tile_row; rows = rows_; kend = kend_; klast = K - 1;
        step = KC ? (int64_t)BK : (int64_t)BK * ld;
        const int t = (int)threadIdx.x;
        row0 = KC ? t / (BK / 4) : (t % (TR / 4)) * 4;
        const int kk = KC ? (t % (BK / 4)) * 4 : t / (TR / 4);
        kfirst = k0 + kk;
        at = lds_at<BK>(row0, kk >> 2) + (kk & 3);
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            // rows past the matrix repeat its last ones: they only feed outputs that are not stored
            int r = tile_row + row0 + (KC ? ER * e : 0);
            const int rmax = KC ? rows - 1 : rows - 4;
            r = r < rmax ? r : rmax;
            const int k = kfirst + (KC ? 0 : EK * e);
            if (VEC) ptr[e] = m + (KC ? (int64_t)r * ld + k : (int64_t)k * ld + r);
        }
    }
    // Load e of a slab.  Unpredicated (addresses clamped into the matrix), so that no load is waited for
    // before the next; what lies past the contraction's end becomes zero on the way to LDS.  WHOLE
    // slabs (all but the last of a contraction) need neither.
    template <bool WHOLE>
    __device__ __forceinline__ void load(f32x4& v, int e, int slab) {
        const int k = kfirst + slab * BK + (KC ? 0 : EK * e);
        if constexpr (VEC) {
            v = gload(reinterpret_cast<const f32x4*>(WHOLE || k < kend ? ptr[e] : base));
            ptr[e] += step;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int r = first + row0 + (KC ? ER * e : j), q = k + (KC ? j : 0);
                r = r < rows ? r : rows - 1;
                q = q < klast ? q : klast;
                v[j] = gload(base + (KC ? (int64_t)r * ld + q : (int64_t)q * ld + r));
            }
        }
    }
    template <bool WHOLE>
    __device__ __forceinline__ void store(f32x4 v, int e, float* lds, int slab) {
        if constexpr (!WHOLE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = kfirst + slab * BK + (KC ? j : EK * e) < kend ? v[j] : 0.0f;
        }
        if constexpr (KC) {      // rows ER apart: the swizzle of a 32-column slab repeats, that of a 64-column slab flips its lowest bit
            *reinterpret_cast<f32x4*>(lds + (BK == 64 ? at ^ ((e & 1) << 2) : at) + e * ER * BK) = v;
        } else {                 // row j of the four moves the swizzle by j / 2 (32 columns) or j (64); k EK apart is chunk EK / 4 apart
#pragma unroll
            for (int j = 0; j < 4; ++j)
                lds[(at ^ ((BK == 64 ? j : j >> 1) << 2) ^ (e * EK)) + j * BK] = v[j];
        }
    }
};

__device__ __forceinline__ void gemm_barrier() {   // keeps the global loads in flight
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr int kGemmArgs = 4;         // problems that travel in the kernel arguments
struct GemmF32Args { GemmF32Dev g[kGemmArgs]; };

// The values of a wave's blocks to the output (or to the split's partial sums): rows from r0, columns from c0 on.  What decides is the same for the
// whole work-group and looked at once; what is added to is read before anything is written (with a predicate, a branch and, where
// something is added to, a load and a wait per value, layers of 200 to 1400 rows took 1.05 to 1.16 times as long).
template <class C>
__device__ __forceinline__ void put_values(const GemmF32Dev& g, const f32x16 (&acc)[C::RA][C::CB], int split, int r0, int c0, int rows_left, int cols_left) {
    const GemmF32& d = g.d;
    const bool partial = g.splits > 1;
    float* const out = partial ? g.part + (int64_t)split * d.P * d.Q : d.C;
    const int64_t ldo = partial ? d.Q : d.ldc;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const float alpha = partial ? 1.0f : d.alpha;
    const bool add = !partial && d.accumulate;
    const bool inside = rows_left >= 32 * C::RA && cols_left >= 32 * C::CB;      // (of the wave)
#pragma unroll
    for (int a = 0; a < C::RA; ++a)
#pragma unroll
        for (int b = 0; b < C::CB; ++b) {
            float* const c = out + (int64_t)(r0 + 32 * a + 4 * lh) * ldo + c0 + 32 * b + li;
            auto row = [](int v) { return 8 * (v >> 2) + (v & 3); };
            float old[16];
            const bool col_in = 32 * b + li < cols_left;
            if (add) {
#pragma unroll
                for (int v = 0; v < 16; ++v) old[v] = inside || (col_in && 32 * a + 4 * lh + row(v) < rows_left) ? gload(c + row(v) * ldo) : 0.0f;
            }
            if (inside) {
#pragma unroll
                for (int v = 0; v < 16; ++v) gstore(c + row(v) * ldo, add ? alpha * acc[a][b][v] + old[v] : alpha * acc[a][b][v]);
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (col_in && 32 * a + 4 * lh + row(v) < rows_left) gstore(c + row(v) * ldo, add ? alpha * acc[a][b][v] + old[v] : alpha * acc[a][b][v]);
            }
        }
}

// The work of one tile; KCA, KCB: k is the fast index of A / B in memory.
template <class C, bool VEC, bool KCA, bool KCB>
__device__ __forceinline__ void gemm_tile(const GemmF32Dev& g, int local, float* lds) {
    const GemmF32& d = g.d;
    const int split = local / g.tiles;
    local -= split * g.tiles;
    const int i0 = (local / g.tiles_q) * C::TM;
    const int j0 = (local % g.tiles_q) * C::TN;
    const int k0 = split * g.k_split;
    const int kend = k0 + g.k_split < d.K ? k0 + g.k_split : d.K;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ks = wave / (C::WR * C::WC), wrc = wave % (C::WR * C::WC);
    const int wi = (wrc / C::WC) * (32 * C::RA), wj = (wrc % C::WC) * (32 * C::CB);
    const int li = lane & 31, lh = lane >> 5;

    // Output columns (or rows) at or beyond *limit are defined to be zero: skip the arithmetic.
    const int lim = d.limit ? *d.limit : (d.limit_rows ? d.P : d.Q);
    const bool dead = d.limit && (d.limit_rows ? (i0 >= lim) : (j0 >= lim));

    f32x16 acc[C::RA][C::CB];
#pragma unroll
    for (int a = 0; a < C::RA; ++a)
#pragma unroll
        for (int b = 0; b < C::CB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

    if (!dead) {
        Loader<C::TM, C::BK, VEC, KCA> la;
        Loader<C::TN, C::BK, VEC, KCB> lb;
        la.init(d.A, d.lda, i0, d.P, k0, kend, d.K);
        lb.init(d.B, d.ldb, j0, d.Q, k0, kend, d.K);
        f32x4 ra[2][C::NVA], rb[2][C::NVB];
        const int nslab = (kend - k0 + C::BK - 1) / C::BK;
        const int nwhole = (kend - k0) / C::BK;
        // piece i of a slab's traffic: first the 16-byte pieces of slab s on their way to LDS, then the
        // requests for slab s + 2 into the same registers
        constexpr int NPIECE = 2 * (C::NVA + C::NVB);
        auto piece = [&](auto whole, int i, int s, int r) {
            constexpr bool W = decltype(whole)::value;
            float* buf = lds + (s & 1) * C::slab;
            if (i < C::NVA) { if (W || s < nslab) la.template store<W>(ra[r][i], i, buf, s); }
            else if (i < C::NVA + C::NVB) { if (W || s < nslab) lb.template store<W>(rb[r][i - C::NVA], i - C::NVA, buf + C::TM * C::BK, s); }
            else if (i < 2 * C::NVA + C::NVB) { if (W || s + 2 < nslab) la.template load<W>(ra[r][i - C::NVA - C::NVB], i - C::NVA - C::NVB, s + 2); }
            else { if (W || s + 2 < nslab) lb.template load<W>(rb[r][i - 2 * C::NVA - C::NVB], i - 2 * C::NVA - C::NVB, s + 2); }
        };
        struct Ops { f32x4 a[C::RA], b[C::CB]; } ops[2];
        auto read = [&](Ops& o, int s, int gq) {
            const float* As = lds + (s & 1) * C::slab;
            const float* Bs = As + C::TM * C::BK;
            const int c = 2 * (ks * C::GPW + gq) + lh;           // chunk of this lane's four k
#pragma unroll
            for (int x = 0; x < C::RA; ++x) o.a[x] = *reinterpret_cast<const f32x4*>(As + lds_at<C::BK>(wi + 32 * x + li, c));
#pragma unroll
            for (int x = 0; x < C::CB; ++x) o.b[x] = *reinterpret_cast<const f32x4*>(Bs + lds_at<C::BK>(wj + 32 * x + li, c));
        };
        // Slab s is multiplied out of buffer s % 2 while slab s + 1 goes to the other buffer (everybody left
        // it before the last barrier) and slab s + 3 is requested.  A matrix instruction waits for the one
        // before it on the same accumulators, so the pieces of that traffic are dealt out between them.
        auto step = [&](auto whole, int s, int u) {
            read(ops[0], s, 0);
#pragma unroll
            for (int gq = 0; gq < C::GPW; ++gq) {
                if (gq + 1 < C::GPW) read(ops[(gq + 1) & 1], s, gq + 1);
                __builtin_amdgcn_sched_barrier(0);
                const Ops& o = ops[gq & 1];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int x = 0; x < C::RA; ++x)
#pragma unroll
                        for (int y = 0; y < C::CB; ++y)
                            acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.a[x][i], o.b[y][i], acc[x][y], 0, 0, 0);
                    constexpr int NSLOT = 4 * C::GPW;
                    const int slot = gq * 4 + i;
#pragma unroll
                    for (int q = slot * NPIECE / NSLOT; q < (slot + 1) * NPIECE / NSLOT; ++q) piece(whole, q, s + 1, u ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            gemm_barrier();
        };
        using Yes = std::integral_constant<bool, true>;
        using No = std::integral_constant<bool, false>;
#pragma unroll
        for (int i = NPIECE / 2; i < NPIECE; ++i) piece(No{}, i, -2, 0);      // request slab 0
#pragma unroll
        for (int i = NPIECE / 2; i < NPIECE; ++i) piece(No{}, i, -1, 1);      // request slab 1
#pragma unroll
        for (int i = 0; i < NPIECE; ++i) piece(No{}, i, 0, 0);                // slab 0 to LDS, request slab 2
        gemm_barrier();
        int s = 0;
        for (; s + 4 < nwhole; s += 2) { step(Yes{}, s, 0); step(Yes{}, s + 1, 1); }
        for (; s < nslab; s += 2) {
            step(No{}, s, 0);
            if (s + 1 < nslab) step(No{}, s + 1, 1);
        }
        if constexpr (C::KS > 1) {
            // contraction groups 1 .. KS-1 hand their sums to group 0, which adds them in order
            constexpr int per = C::WR * C::WC * C::RA * C::CB * 16;
            if (ks > 0) {
#pragma unroll
                for (int x = 0; x < C::RA; ++x)
#pragma unroll
                    for (int y = 0; y < C::CB; ++y)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            lds[((ks - 1) * per + (wrc * C::RA * C::CB + x * C::CB + y) * 16 + v) * 64 + lane] = acc[x][y][v];
            }
            gemm_barrier();
            if (ks > 0) return;
#pragma unroll
            for (int o = 0; o < C::KS - 1; ++o)
#pragma unroll
                for (int x = 0; x < C::RA; ++x)
#pragma unroll
                    for (int y = 0; y < C::CB; ++y)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            acc[x][y][v] += lds[(o * per + (wrc * C::RA * C::CB + x * C::CB + y) * 16 + v) * 64 + lane];
        }
    } else if (C::KS > 1 && ks > 0) {
        return;
    }

    if (d.limit == nullptr) {
        put_values<C>(g, acc, split, i0 + wi, j0 + wj, d.P - i0 - wi, d.Q - j0 - wj);
        return;
    }
#pragma unroll
    for (int a = 0; a < C::RA; ++a)
#pragma unroll
        for (int b = 0; b < C::CB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = i0 + wi + a * 32 + 8 * (v >> 2) + 4 * lh + (v & 3);
                const int col = j0 + wj + b * 32 + li;
                if (row < d.P && col < d.Q)              // (never split, never added to)
                    gstore(d.C + (int64_t)row * d.ldc + col, (d.limit_rows ? (row >= lim) : (col >= lim)) ? 0.0f : d.alpha * acc[a][b][v]);
            }
}

template <class C, bool VEC>
__global__ __launch_bounds__(NT, 3) void gemm_f32_kernel(const GemmF32Dev* __restrict__ table, GemmF32Args args, int ndesc) {
    __shared__ __align__(16) float lds[C::lds_floats];
    // Block b runs on XCD b % 8.  A few problems: every XCD gets a contiguous eighth of the tiles of each, which share their operand panels through
    // one L2; problems of unlike contractions weigh the same on every XCD then (an eighth of the whole list instead left two thirds
    // of the work of the joint launch of dA, dB and dX to three of them: 124 us against 64, 3152 x 3072 x 768, r = 192).  The tiles that eighths leave over
    // go to the XCDs in turn, on from one problem to the next (rounded up for each, dA and dB of 5675 x 28 x 770, r = 30, were 33 work-groups for
    // the 32 compute units of an XCD: 21.5 us, 16.0 so).  A table of
    // many: an eighth of the list, whole problems for the most part (96 back-projections of a merge 294 us, 380 the other way).
    const int slot = (int)(blockIdx.x >> 3), xcd = (int)(blockIdx.x & 7);
    GemmF32Dev g;
    int tile;
    if (table == nullptr) {
        int i = 0, at = slot;
        for (;; ++i) {
            if (i == ndesc) return;
            const int all = args.g[i].tiles * args.g[i].splits, x = (xcd - args.g[i].begin) & 7, over = all & 7;
            const int share = (all >> 3) + (x < over ? 1 : 0);
            tile = x * (all >> 3) + (x < over ? x : over) + at;
            if (at < share) break;
            at -= share;
        }
        g = args.g[i];
    } else {
        const int at = xcd * (int)(gridDim.x >> 3) + slot;
        int lo = 0, hi = ndesc - 1;
        while (lo < hi) {  // last descriptor whose first tile is not beyond
            int mid = (lo + hi + 1) >> 1;
            if (table[mid].begin <= at) lo = mid; else hi = mid - 1;
        }
        g = table[lo];
        tile = at - g.begin;
        if (tile >= g.tiles) return;
    }
    if (g.d.transA) {
        if (g.d.transB) gemm_tile<C, VEC, false, true>(g, tile, lds);
        else gemm_tile<C, VEC, false, false>(g, tile, lds);
    } else {
        if (g.d.transB) gemm_tile<C, VEC, true, true>(g, tile, lds);
        else gemm_tile<C, VEC, true, false>(g, tile, lds);
    }
}

// The same tiles by work-groups that stay: each takes tiles first, first + stride, .. below `share` of a problem, and the slabs of all of them are one
// stream, so a tile's first loads are on their way while the one before is multiplied out, and its values leave meanwhile.  Whole slabs
// and 16-byte loads only.  Short contractions gain: 3072 x 3072 x 192 46.0 -> 38.8 us, the forward at M = 3152, m = 3072, n = 768, r = 192 72 -> 64,
// 3072 x 768 x 384 27.2 -> 25.5; long ones are equal.  (Two to a compute unit: 42, 69, 26.8, and 4096 x 4096 x 1024 324 of 310; four spill.)
template <class C, bool KCA, bool KCB>
__device__ __forceinline__ void gemm_stream(const GemmF32Dev& g, int origin, int first, int share, int stride, float* lds) {
    const GemmF32& d = g.d;
    struct Tile { int split, i0, j0, k0, kend; };
    auto tile_at = [&](int at) {
        int local = origin + at;
        Tile t;
        t.split = local / g.tiles;
        local -= t.split * g.tiles;
        t.i0 = (local / g.tiles_q) * C::TM;
        t.j0 = (local % g.tiles_q) * C::TN;
        t.k0 = t.split * g.k_split;
        t.kend = t.k0 + g.k_split < d.K ? t.k0 + g.k_split : d.K;
        return t;
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi = (wave / C::WC) * (32 * C::RA), wj = (wave % C::WC) * (32 * C::CB);
    const int li = lane & 31, lh = lane >> 5;
    f32x16 acc[C::RA][C::CB];
    auto clear = [&] {
#pragma unroll
        for (int a = 0; a < C::RA; ++a)
#pragma unroll
            for (int b = 0; b < C::CB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;
    };
    clear();

    // the loaders run ahead through the tiles; past the last one they read the last slab's neighbours of the first rows again
    Loader<C::TM, C::BK, true, KCA> la;
    Loader<C::TN, C::BK, true, KCB> lb;
    int next = first, left = 0;                            // slabs of the loaders' tile that are still to be asked for
    auto turn = [&] {
        if (left > 0) return;
        if (next < share) {
            const Tile t = tile_at(next);
            la.init(d.A, d.lda, t.i0, d.P, t.k0, t.kend, d.K);
            lb.init(d.B, d.ldb, t.j0, d.Q, t.k0, t.kend, d.K);
            left = (t.kend - t.k0) / C::BK;
            next += stride;
        } else {
#pragma unroll
            for (int e = 0; e < C::NVA; ++e) la.ptr[e] = d.A;
#pragma unroll
            for (int e = 0; e < C::NVB; ++e) lb.ptr[e] = d.B;
            la.step = lb.step = 0;
            left = 1 << 30;
        }
    };
    f32x4 ra[2][C::NVA], rb[2][C::NVB];
    constexpr int NPIECE = 2 * (C::NVA + C::NVB);
    auto piece = [&](int i, int buffer, int r) {
        float* buf = lds + buffer * C::slab;
        if (i < C::NVA) la.template store<true>(ra[r][i], i, buf, 0);
        else if (i < C::NVA + C::NVB) lb.template store<true>(rb[r][i - C::NVA], i - C::NVA, buf + C::TM * C::BK, 0);
        else if (i < 2 * C::NVA + C::NVB) la.template load<true>(ra[r][i - C::NVA - C::NVB], i - C::NVA - C::NVB, 0);
        else lb.template load<true>(rb[r][i - 2 * C::NVA - C::NVB], i - 2 * C::NVA - C::NVB, 0);
    };
    struct Ops { f32x4 a[C::RA], b[C::CB]; } ops[2];
    auto read = [&](Ops& o, int buffer, int gq) {
        const float* As = lds + buffer * C::slab;
        const float* Bs = As + C::TM * C::BK;
        const int c = 2 * gq + lh;
#pragma unroll
        for (int x = 0; x < C::RA; ++x) o.a[x] = *reinterpret_cast<const f32x4*>(As + lds_at<C::BK>(wi + 32 * x + li, c));
#pragma unroll
        for (int x = 0; x < C::CB; ++x) o.b[x] = *reinterpret_cast<const f32x4*>(Bs + lds_at<C::BK>(wj + 32 * x + li, c));
    };
    auto request = [&](int r) {
        turn();
#pragma unroll
        for (int i = NPIECE / 2; i < NPIECE; ++i) piece(i, 0, r);
        --left;
    };
    gemm_barrier();                                        // (the problem before has left the LDS)
    request(0);
    request(1);
#pragma unroll
    for (int i = 0; i < NPIECE / 2; ++i) piece(i, 0, 0);
    request(0);
    gemm_barrier();

    Tile cur = tile_at(first);
    int at = first, slabs = (cur.kend - cur.k0) / C::BK;
    while (at < share) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (at >= share) break;
            turn();
            read(ops[0], u, 0);
#pragma unroll
            for (int gq = 0; gq < C::GPW; ++gq) {
                if (gq + 1 < C::GPW) read(ops[(gq + 1) & 1], u, gq + 1);
                __builtin_amdgcn_sched_barrier(0);
                const Ops& o = ops[gq & 1];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int x = 0; x < C::RA; ++x)
#pragma unroll
                        for (int y = 0; y < C::CB; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(o.a[x][i], o.b[y][i], acc[x][y], 0, 0, 0);
                    constexpr int NSLOT = 4 * C::GPW;
                    const int slot = gq * 4 + i;
#pragma unroll
                    for (int q = slot * NPIECE / NSLOT; q < (slot + 1) * NPIECE / NSLOT; ++q) piece(q, u ^ 1, u ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            --left;
            gemm_barrier();
            if (--slabs > 0) continue;
            put_values<C>(g, acc, cur.split, cur.i0 + wi, cur.j0 + wj, d.P - cur.i0 - wi, d.Q - cur.j0 - wj);
            clear();
            at += stride;
            if (at < share) { cur = tile_at(at); slabs = (cur.kend - cur.k0) / C::BK; }
        }
    }
}

template <class C>
__global__ __launch_bounds__(NT, 3) void gemm_f32_stream_kernel(GemmF32Args args, int ndesc) {
    __shared__ __align__(16) float lds[C::lds_floats];
    const int slot = (int)(blockIdx.x >> 3), xcd = (int)(blockIdx.x & 7), slots = (int)(gridDim.x >> 3);      // shares as in gemm_f32_kernel
    int before = 0;
    for (int i = 0; i < ndesc; ++i) {
        const GemmF32Dev& g = args.g[i];
        const int all = g.tiles * g.splits, x = (xcd - g.begin) & 7, over = all & 7;
        const int share = (all >> 3) + (x < over ? 1 : 0), origin = x * (all >> 3) + (x < over ? x : over);
        const int first = ((slot - before) % slots + slots) % slots;
        before += share;
        if (first >= share) continue;
        if (g.d.transA) {
            if (g.d.transB) gemm_stream<C, false, true>(g, origin, first, share, slots, lds);
            else gemm_stream<C, false, false>(g, origin, first, share, slots, lds);
        } else {
            if (g.d.transB) gemm_stream<C, true, true>(g, origin, first, share, slots, lds);
            else gemm_stream<C, true, false>(g, origin, first, share, slots, lds);
        }
    }
}

// C (+)= alpha * (sum over the splits of the partial sums, in order), for the split problems of a launch
__global__ __launch_bounds__(NT) void gemm_f32_reduce_kernel(GemmF32Args args, int ndesc) {
    const GemmF32Dev& g = args.g[blockIdx.y];
    if ((int)blockIdx.y >= ndesc || g.splits < 2) return;
    const int64_t total = (int64_t)g.d.P * g.d.Q;
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < total; i += (int64_t)gridDim.x * NT) {
        float s = gload(g.part + i);
        for (int q = 1; q < g.splits; ++q) s += gload(g.part + q * total + i);
        float* c = g.d.C + (g.d.ldc == g.d.Q ? i : (i / g.d.Q) * g.d.ldc + i % g.d.Q);
        s *= g.d.alpha;
        gstore(c, g.d.accumulate ? s + gload(c) : s);
    }
}

using Wide = GemmCfg<64, 64, 2, 2, 1, 32>;
using Small = GemmCfg<32, 32, 1, 1, 4, 64>;

int tiles_of(const GemmF32& d, int tm, int tn) { return (int)(ceil_div(d.P, tm) * ceil_div(d.Q, tn)); }

// 16-byte loads: rows start on 16 bytes and hold whole pieces of four
bool vec_ok(const GemmF32& d) {
    auto ok = [](const float* p, int ld, int fast) { return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 4 == 0 && fast % 4 == 0; };
    return ok(d.A, d.lda, d.transA ? d.P : d.K) && ok(d.B, d.ldb, d.transB ? d.K : d.Q);
}

GemmF32Dev describe(const GemmF32& d, int tm, int tn, int begin, int splits) {
    GemmF32Dev g{};
    g.d = d;
    g.begin = begin;
    g.tiles_q = (int)ceil_div(d.Q, tn);
    g.tiles = tiles_of(d, tm, tn);
    g.k_split = (int)ceil_div(ceil_div(d.K, splits), 64) * 64;
    g.splits = (int)ceil_div(d.K, g.k_split);
    return g;
}

void launch_form(bool small, bool vec, int slots, const GemmF32Dev* table, const GemmF32Args& a, int n, hipStream_t s) {
    const dim3 grid(8 * slots), block(NT);
    if (small && vec) hipLaunchKernelGGL((gemm_f32_kernel<Small, true>), grid, block, 0, s, table, a, n);
    else if (small) hipLaunchKernelGGL((gemm_f32_kernel<Small, false>), grid, block, 0, s, table, a, n);
    else if (vec) hipLaunchKernelGGL((gemm_f32_kernel<Wide, true>), grid, block, 0, s, table, a, n);
    else hipLaunchKernelGGL((gemm_f32_kernel<Wide, false>), grid, block, 0, s, table, a, n);
}

// 64 x 64 tiles once they give every compute unit one; below that the 32 x 32 form (measured: 150 tiles of
// 64 x 64, K = 768: 19.1 us against 17.1; K = 3072: 62.8 against 47.2; 432 tiles, K = 384: 19.5 against 24.2)
bool use_small(int64_t wide_tiles) { return wide_tiles < 256; }

int64_t wide_tiles_of(const GemmF32* p, const int* splits, int n) {
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (int64_t)tiles_of(p[i], Wide::TM, Wide::TN) * (splits ? splits[i] : 1);
    return tiles;
}

}  // namespace

int gemm_f32_splits(const GemmF32& d) {
    // A contraction much longer than the output is wide (the factor gradients: K = batch rows) is split
    // until the launch has about two work-groups per compute unit, at least 256 columns per split
    // (measured, the reduction included, K = 3152: 3072 x 192 65.9 us whole, 52.3 in four; 192 x 768 65.2
    // whole, 22.9 in four, 25.5 in eight).
    const int64_t tiles = tiles_of(d, Wide::TM, Wide::TN);
    int64_t s = 512 / (tiles > 0 ? tiles : 1);
    const int64_t by_k = d.K / 256;
    if (s > by_k) s = by_k;
    if (s > 64) s = 64;
    return s < 1 ? 1 : (int)s;
}

// The time of a product and of the sum of its partial ones, us, fitted to backward passes of 100 to 3152 rows, r = 32 to 384, K = 1024 to 3072, in up
// to 12 splits (120 shapes: 2.97 ms in all with the splits of this estimate, 2.93 with the best, 3.34 unsplit; none slower by more than
// 4 %): 32 x 32 tiles cost 11 us per 3072 of the contraction and 0.05 per tile (traffic from L2), 64 x 64 tiles 54 for each round of the compute
// units.  dT and a dX of 768 columns: 3152 x 3072, r = 192 63.6 -> 59.5 us (594 tiles of 32 x 32; 750 of 64 x 64), 3152 x 2304, r = 384 103 -> 85,
// 800 x 3072, r = 64 27.7 -> 20.
int gemm_f32_row_splits(const GemmF32& d) {
    const int64_t wide = (int64_t)tiles_of(d, Wide::TM, Wide::TN), narrow = (int64_t)tiles_of(d, Small::TM, Small::TN);
    auto time = [&](int s) {
        const double k = (double)(ceil_div(ceil_div(d.K, s), 64) * 64) / 3072.0;
        const double t = use_small(wide * s) ? k * (11.0 + 0.05 * (double)(narrow * s)) : k * 54.0 * (double)ceil_div(wide * s, 256);
        return s == 1 ? t : t + 3.5 + (s + 1) * 0.7e-6 * (double)d.P * (double)d.Q;
    };
    int best = 1;
    for (int s = 2; s <= 8 && (int64_t)s * 512 <= d.K; ++s)
        if (time(s) < time(best)) best = s;
    return best;
}

size_t gemm_f32_partial_bytes(const GemmF32& d, int splits) {
    return splits > 1 ? align_up((size_t)splits * d.P * d.Q * sizeof(float), 256) : 0;
}

bool gemm_f32_first_as_alone(const GemmF32* p, const int* splits, int n) { return use_small(wide_tiles_of(p, splits, n)) == use_small(wide_tiles_of(p, nullptr, 1)); }

hipError_t launch_gemm_f32(const GemmF32* p, const int* splits, int n, float* partials, hipStream_t s) {
    if (n < 1 || n > kGemmArgs) return hipErrorInvalidValue;
    bool any_split = false, vec = true;
    for (int i = 0; i < n; ++i) {
        if (splits && splits[i] > 1) any_split = true;
        vec = vec && vec_ok(p[i]);
    }
    const bool small = use_small(wide_tiles_of(p, splits, n));
    const int tm = small ? Small::TM : Wide::TM, tn = small ? Small::TN : Wide::TN;
    GemmF32Args a{};
    int tiles = 0;
    int64_t largest = 0;
    char* part = (char*)partials;
    for (int i = 0; i < n; ++i) {
        a.g[i] = describe(p[i], tm, tn, tiles & 7, splits ? splits[i] : 1);
        if (a.g[i].splits > 1) {
            if (!partials) return hipErrorInvalidValue;
            a.g[i].part = (float*)part;
            part += gemm_f32_partial_bytes(p[i], a.g[i].splits);
            if ((int64_t)p[i].P * p[i].Q > largest) largest = (int64_t)p[i].P * p[i].Q;
        }
        tiles += a.g[i].tiles * a.g[i].splits;
    }
    if (tiles <= 0) return hipSuccess;
    // whole slabs: work-groups that stay, three to a compute unit
    bool stream = !small && vec;
    for (int i = 0; i < n; ++i) stream = stream && p[i].limit == nullptr && p[i].K % Wide::BK == 0;
    if (stream) {
        const int share = (tiles + 7) / 8;
        hipLaunchKernelGGL((gemm_f32_stream_kernel<Wide>), dim3(8 * (share < 96 ? share : 96)), dim3(NT), 0, s, a, n);
    } else {
        launch_form(small, vec, (tiles + 7) / 8, nullptr, a, n, s);
    }
    if (any_split && largest > 0) {
        const int64_t blocks = ceil_div(largest, NT);
        hipLaunchKernelGGL(gemm_f32_reduce_kernel, dim3((unsigned)(blocks < 2048 ? blocks : 2048), n), dim3(NT), 0, s, a, n);
    }
    return hipGetLastError();
}

hipError_t launch_gemm_f32_one(const GemmF32& d, hipStream_t s) { return launch_gemm_f32(&d, nullptr, 1, nullptr, s); }

// Grouped launch in two steps so the caller can batch the upload with its other tables:
// gemm_f32_build_table fills `host_image` (n * gemm_f32_desc_bytes() bytes) and says which form of the
// kernel takes it; after the caller has copied the image to device memory, launch_gemm_f32_table runs it.
size_t gemm_f32_desc_bytes() { return sizeof(GemmF32Dev); }

GemmF32Table gemm_f32_build_table(const GemmF32* descs_host, int n, void* host_image) {
    GemmF32Dev* tmp = static_cast<GemmF32Dev*>(host_image);
    GemmF32Table t{n, 0, true, true};
    int64_t wide_tiles = 0;
    for (int i = 0; i < n; ++i) {
        wide_tiles += tiles_of(descs_host[i], Wide::TM, Wide::TN);
        t.vec = t.vec && vec_ok(descs_host[i]);
    }
    t.small = use_small(wide_tiles);
    for (int i = 0; i < n; ++i) {
        tmp[i] = describe(descs_host[i], t.small ? Small::TM : Wide::TM, t.small ? Small::TN : Wide::TN, t.tiles, 1);
        t.tiles += tmp[i].tiles;
    }
    return t;
}

hipError_t launch_gemm_f32_table(const void* dev_image, const GemmF32Table& t, hipStream_t s) {
    if (t.n <= 0 || t.tiles <= 0) return hipSuccess;
    launch_form(t.small, t.vec, (t.tiles + 7) / 8, (const GemmF32Dev*)dev_image, GemmF32Args{}, t.n, s);
    return hipGetLastError();
}

}  // namespace abt
