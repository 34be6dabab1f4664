// The bf16 factored layer for few rows, two launches each way:
//     T[M,r] = X[M,n] . B[r,n]^T,  Y[M,m] = T . A[m,r]^T                (small_nt_kernel, twice)
//     dT[M,r] = dY[M,m] . A[m,r]                                       (small_dt_kernel)
//     dX[M,n] = dT . B[r,n],  dA[m,r] = dY^T . T,  dB[r,n] = dT^T . X   (small_grad_kernel, all of them at once; small_conv_grad_kernel)
//
// What bounds it: latency.  The kernels for many rows walk a contraction of thousands of columns in one work-group per
// 64 rows, a barrier per slab of 64, behind a launch that transposes the factors, and the factor gradients
// come in two more launches.  Here the backward stages nothing: operands come straight from memory (L2) into registers, a work-group's waves
// share out the contraction and add their sums once through LDS, and tiles are small, so that a layer of 200 rows is some
// hundred work-groups.  A factor (or a batch) whose contraction index is its slow dimension is read as it lies: a lane
// loads, for each of the eight k of its operand, the 4 bytes of two neighbouring columns, and the two columns go to
// two 32-wide blocks of the tile (byte permutes); column c of a 64-wide tile is lane c / 2 of block c % 2, and results leave in
// pairs of columns.
//
// MFMA 32x32x16 bf16 layout (lane l, j = l % 32, h = l / 32): A operand = 8 values A[j][8h .. 8h+7], B operand
// = B[8h .. 8h+7][j], accumulator v = C[8 (v / 4) + 4h + v % 4][j].
#include <atomic>

#include "common.h"

namespace abt {

namespace {

__device__ __forceinline__ f32x16 mfma16(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t load4(rsrc_t r, int lane_off, int wave_off) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, lane_off, wave_off, 0);
}
__device__ __forceinline__ void zero(f32x16& a) {
#pragma unroll
    for (int v = 0; v < 16; ++v) a[v] = 0.0f;
}
// row of accumulator v
__device__ __forceinline__ int acc_row(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }
// the pairs of columns of eight consecutive k -> the operands of the two blocks
__device__ __forceinline__ void unpair(const uint32_t (&d)[8], u32x4 (&op)[2]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        op[0][i] = __builtin_amdgcn_perm(d[2 * i + 1], d[2 * i], 0x05040100u);
        op[1][i] = __builtin_amdgcn_perm(d[2 * i + 1], d[2 * i], 0x07060302u);
    }
}

// ------------------------------------------------------------------ forward
// C = U V^T (bf16, both operands contraction-fast), T = X B^T and then Y = T A^T: two launches of tiles where the fused kernels have one
// work-group per row block, which reads all of B before it has a row of T (197 x 768 -> 2304: r = 96 12 us, 7.3 here; r = 384 38, 9.1).
// Bound by the latency of the loads, so short chains and many of them:
//   * A work-group of RM CN SK waves has a tile of 32 RM rows and 32 CN columns, a wave 32 x 32 of it and every SK-th unit of 64 of the
//     contraction (sums through LDS).  Where tiles are few, SK = 8 waves share one (T of 197 x 3072, r = 32: 11 us for both launches; 23 with
//     a tile of 64 x 64 and SK = 1); where they are many, larger tiles read less (T of 4000 x 3072, r = 384: 32 x 32 58 us, 64 x 128 35).
//   * Whole 128-byte lines travel through registers (two stages of SK units ahead) into two LDS buffers, one barrier per stage.  (Each
//     lane loading the pieces of its operand: 32 lines per instruction instead of 8, 197 x 3072, r = 192 16.2 us, 11.1.)
//   * A wave's tile with 64 x 64 values instead of 32 x 32: no gain below 16000 rows.
// The order of the sums depends on SK, which launch_t picks by the rows of all groups of the call, the rank and the tile: T is the same bits
// kept or computed again (for all groups of a call or some).
struct SmallNtEntry { const uint16_t* U; const uint16_t* V; uint16_t* C; };
struct SmallNt {
    SmallNtEntry e[kChainMaxGroups];                     // problems of one shape
    int M, N, K, tiles_n;
    int64_t u_bytes;
    int H, W, Cin, kh, kw, RH, RW, mul;                  // image: rows are the pixels of a grid RH x RW, centred on pixel (mul y, mul x)
};

// this wave's LDS traffic has completed, then s_barrier; global loads in flight stay in flight
__device__ __forceinline__ void nt_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int RM, int CN, int SK>
struct Nt {
    static constexpr int threads = 64 * RM * CN * SK, rows = 32 * RM, cols = 32 * CN;
    static constexpr int unit = (rows + cols) * 128, stage = SK * unit, lds_bytes = 2 * stage;
    static constexpr int NU = 4 / CN, NV = 4 / RM;       // 16-byte pieces per thread and stage
};

template <int RM, int CN, int SK, bool GATHER>
__global__ __launch_bounds__((Nt<RM, CN, SK>::threads)) void small_nt_kernel(SmallNt p) {
    using G = Nt<RM, CN, SK>;
    constexpr int NU = G::NU, NV = G::NV, NT = G::threads;
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, j = lane & 31, h = lane >> 5, ch = tid & 7;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = (int)blockIdx.x / p.tiles_n, tn = (int)blockIdx.x - rb * p.tiles_n, row0 = G::rows * rb, col0 = G::cols * tn;
    const SmallNtEntry en = p.e[blockIdx.y];
    const rsrc_t ures = make_rsrc(en.U, p.u_bytes), vres = make_rsrc(en.V, (int64_t)p.N * p.K * 2);

    // Piece i of U is chunk ch of row (i NT + tid) / 8 % rows, in unit (i NT + tid) / (8 rows) of the stage; V alike.  In LDS the chunks of a row
    // are swizzled, so that 16 lanes reading one chunk of 16 rows, and 8 lanes writing a row, meet no bank twice.
    int uoff[NU], gy[NU], gx[NU], uc[NU], uky[NU], ukx[NU], voff[NV], uslot[NU], vslot[NV];
    auto unit_u = [&](int i) { return (i * NT + 64 * wave) / (8 * G::rows); };
    auto unit_v = [&](int i) { return (i * NT + 64 * wave) / (8 * G::cols); };
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const int row = ((i * NT + tid) / 8) % G::rows, at = row0 + row;
        uslot[i] = unit_u(i) * G::unit + row * 128 + 16 * (ch ^ ((row >> 1) & 7));
        if constexpr (GATHER) {
            const int q = at < p.M ? at : 0, per = p.RH * p.RW, img = q / per, rem = q - img * per, y = rem / p.RW;
            gx[i] = p.mul * (rem - y * p.RW);
            uoff[i] = (((img * p.H + p.mul * y) * p.W + gx[i]) * p.Cin + 8 * ch) * 2;
            gy[i] = at < p.M ? p.mul * y : -(1 << 24);   // no row: never inside the image
            uc[i] = 64 * unit_u(i); uky[i] = ukx[i] = 0; // channel and tap of the next piece
        } else {
            uoff[i] = (at * p.K + 8 * ch) * 2;           // rows past M: outside the descriptor, zeros
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int row = ((i * NT + tid) / 8) % G::cols;
        vslot[i] = unit_v(i) * G::unit + (G::rows + row) * 128 + 16 * (ch ^ ((row >> 1) & 7));
        voff[i] = ((col0 + row) * p.K + 8 * ch) * 2;     // columns past N: outside the descriptor
    }
    struct Stage { u32x4 u[NU], v[NV]; } ring[2];
    const int stages = (p.K + 64 * SK - 1) / (64 * SK);  // the last one may reach past the contraction: zeros there
    auto load = [&](Stage& d, int t) {                   // stages are loaded in order
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            const int k = 64 * (t * SK + unit_u(i));
            if constexpr (GATHER) {
                while (uc[i] >= p.Cin) { uc[i] -= p.Cin; if (++ukx[i] == p.kw) { ukx[i] = 0; ++uky[i]; } }
                const int dy = uky[i] - p.kh / 2, dx = ukx[i] - p.kw / 2;
                const bool ok = k < p.K && (unsigned)(gy[i] + dy) < (unsigned)p.H && (unsigned)(gx[i] + dx) < (unsigned)p.W;
                d.u[i] = buf_load16(ures, ok ? uoff[i] + ((dy * p.W + dx) * p.Cin + uc[i]) * 2 : kBufNowhere, 0);
                uc[i] += 64 * SK;
            } else {
                d.u[i] = buf_load16(ures, k + 8 * ch < p.K ? uoff[i] : kBufNowhere, 2 * k);
            }
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int k = 64 * (t * SK + unit_v(i));
            d.v[i] = buf_load16(vres, k + 8 * ch < p.K ? voff[i] : kBufNowhere, 2 * k);
        }
    };
    auto to_lds = [&](const Stage& d, int b) {
        unsigned char* const at = lds + b * G::stage;
#pragma unroll
        for (int i = 0; i < NU; ++i) *reinterpret_cast<u32x4*>(at + uslot[i]) = d.u[i];
#pragma unroll
        for (int i = 0; i < NV; ++i) *reinterpret_cast<u32x4*>(at + vslot[i]) = d.v[i];
    };
    // This wave: unit s of the stage, rows 32 wr and columns 32 wc of the tile.  The columns are fed in an order (two bits of their number swapped)
    // that leaves eight neighbouring ones in accumulators 0 .. 7 and 8 .. 15 of a lane, whose row is j.
    const int s = wave / (RM * CN), wt = wave % (RM * CN), wr = wt / CN, wc = wt % CN;
    const int pj = (j & 16) | ((j & 4) << 1) | ((j & 8) >> 1) | (j & 3);
    f32x16 acc;
    zero(acc);
    auto multiply = [&](int b) {
        const unsigned char* const u = lds + b * G::stage + s * G::unit + (32 * wr + j) * 128;
        const unsigned char* const v = lds + b * G::stage + s * G::unit + (G::rows + 32 * wc + pj) * 128;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc = mfma16(*reinterpret_cast<const u32x4*>(v + 16 * ((2 * q + h) ^ ((pj >> 1) & 7))),
                         *reinterpret_cast<const u32x4*>(u + 16 * ((2 * q + h) ^ ((j >> 1) & 7))), acc);
    };
    load(ring[0], 0);
    if (1 < stages) load(ring[1], 1);
    for (int t = 0; t < stages; t += 2) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (t + e >= stages) break;
            to_lds(ring[e], e);                          // read last two stages ago, before the barrier of the stage between
            if (t + e + 2 < stages) load(ring[e], t + e + 2);
            nt_barrier();
            multiply(e);
        }
    }
    const rsrc_t cres = make_rsrc(en.C, (int64_t)p.M * p.N * 2);
    const bool live = col0 + 32 * wc < p.N;              // N is a multiple of 32
    const int out = ((row0 + 32 * wr + j) * p.N + col0 + 32 * wc + 8 * h) * 2;          // rows past M are dropped
    if constexpr (SK == 1) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            u32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = pack2_bf16(acc[8 * g + 2 * e], acc[8 * g + 2 * e + 1]);
            buf_store16(o, cres, live ? out + 32 * g : kBufNowhere, 0);
        }
    } else {
        float (*red)[RM * CN][16][64] = reinterpret_cast<float (*)[RM * CN][16][64]>(lds);
        static_assert(sizeof(float) * NT * 16 <= G::lds_bytes);
        nt_barrier();
#pragma unroll
        for (int v = 0; v < 16; ++v) red[s][wt][v][lane] = acc[v];
        nt_barrier();
#pragma unroll
        for (int e = 0; e < 8 / SK; ++e) {
            const int v = (16 / SK) * s + 2 * e;
            float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
            for (int w = 0; w < SK; ++w) { t0 += red[w][wt][v][lane]; t1 += red[w][wt][v + 1][lane]; }
            __builtin_amdgcn_raw_buffer_store_b32(pack2_bf16(t0, t1), cres, live ? out + 32 * (v / 8) + 2 * (v % 8) : kBufNowhere, 0, 0);
        }
    }
}

// ------------------------------------------------------------------ dT
constexpr int kDtWaves = 8;

struct SmallDt { const uint16_t* dY; const uint16_t* A; uint16_t* dT; int M, m, r; };

// 32 rows x COLS columns of dT; wave w takes the slabs of 64 columns of dY w, w + 8, ..  Of 64 columns a lane loads two neighbours for all eight k of
// its operands, of 32 for four of them, and lanes j and j + 16 exchange halves.
// Bound by the loads a wave may have on the way (63) and their latency: 36 loads per slab of 64 columns, 20 of 32.  The wave's number has to be
// known to be uniform (readfirstlane), or every load whose offset depends on it sits in a loop over the distinct values of its lanes
// (108 such loops; 197 x 768 -> 2304, r = 96: 11.0 us, 9.0 without them, 8.0 with tiles of 32 columns and three slabs ahead).
template <int COLS>
__global__ __launch_bounds__(64 * kDtWaves, 2) void small_dt_kernel(SmallDt p) {
    constexpr int CB = COLS / 32, KI = 4 * CB, NB = COLS == 64 ? 2 : 4;      // blocks, loads per operand, slabs in flight
    __shared__ float red[kDtWaves][CB][16][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, h = lane >> 5;
    const int row0 = 32 * (int)blockIdx.x, col = COLS * (int)blockIdx.y + 2 * (j & (COLS / 2 - 1)), kq = 8 * h + (COLS == 32 ? 4 * (j >> 4) : 0);
    const rsrc_t xres = make_rsrc(p.dY, (int64_t)p.M * p.m * 2), ares = make_rsrc(p.A, (int64_t)p.m * p.r * 2);
    const int xoff = ((row0 + j) * p.m + 8 * h) * 2;                 // rows past M: outside the descriptor, zeros
    const int aoff = col < p.r ? (kq * p.r + col) * 2 : kBufNowhere;
    f32x16 acc[CB];
#pragma unroll
    for (int b = 0; b < CB; ++b) zero(acc[b]);
    struct Slab { u32x4 x[4]; uint32_t a[4][KI]; } buf[NB];
    auto load = [&](Slab& s, int slab) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            s.x[q] = buf_load16(xres, xoff, (64 * slab + 16 * q) * 2);
#pragma unroll
            for (int i = 0; i < KI; ++i) s.a[q][i] = load4(ares, aoff, (64 * slab + 16 * q + i) * p.r * 2);
        }
    };
    auto multiply = [&](const Slab& s) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (CB == 2) {
                u32x4 op[2];
                unpair(s.a[q], op);
                acc[0] = mfma16(s.x[q], op[0], acc[0]);
                acc[1] = mfma16(s.x[q], op[1], acc[1]);
            } else {
                u32x4 op;                                    // lane j: column 2 (j % 16) + j / 16 of the tile
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint32_t even = __builtin_amdgcn_perm(s.a[q][2 * i + 1], s.a[q][2 * i], 0x05040100u);
                    const uint32_t odd = __builtin_amdgcn_perm(s.a[q][2 * i + 1], s.a[q][2 * i], 0x07060302u);
                    const auto both = __builtin_amdgcn_permlane16_swap(even, odd, false, false);
                    op[i] = both[0];
                    op[2 + i] = both[1];
                }
                acc[0] = mfma16(s.x[q], op, acc[0]);
            }
        }
    };
    const int slabs = p.m / 64;
#pragma unroll
    for (int b = 0; b < NB - 1; ++b)
        if (wave + b * kDtWaves < slabs) load(buf[b], wave + b * kDtWaves);
    for (int s = wave; s < slabs; s += NB * kDtWaves)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int at = s + b * kDtWaves;
            if (at + (NB - 1) * kDtWaves < slabs) load(buf[(b + NB - 1) % NB], at + (NB - 1) * kDtWaves);
            if (at < slabs) multiply(buf[b]);
        }
#pragma unroll
    for (int b = 0; b < CB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[wave][b][v][lane] = acc[b][v];
    __syncthreads();
    const rsrc_t tres = make_rsrc(p.dT, (int64_t)p.M * p.r * 2);     // rows past M are dropped
#pragma unroll
    for (int e = 0; e < CB; ++e) {
        // a pair of columns: two blocks of one lane, or one block of the lanes c and c + 16
        const int v = CB == 2 ? wave + kDtWaves * e : 2 * wave + h, c = CB == 2 ? lane : (lane & 15) + 2 * (lane & 16);
        const int hh = CB == 2 ? h : (lane >> 4) & 1, oc = COLS * (int)blockIdx.y + 2 * (lane & (COLS / 2 - 1));
        float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
        for (int w = 0; w < kDtWaves; ++w) { t0 += red[w][0][v][c]; t1 += CB == 2 ? red[w][CB - 1][v][c] : red[w][0][v][c + 16]; }
        const int off = oc < p.r ? ((row0 + acc_row(v, hh)) * p.r + oc) * 2 : kBufNowhere;
        __builtin_amdgcn_raw_buffer_store_b32(pack2_bf16(t0, t1), tres, off, 0, 0);
    }
}

// ------------------------------------------------------------------ dX, dA, dB
constexpr int kGradWaves = 8;

// C[P,Q] (+)= R[M,P]^T . S[M,Q], fp32
struct SmallTn { const uint16_t* R; const uint16_t* S; float* C; int P, Q, tiles_q; };
struct SmallGrad {
    const uint16_t* dT; const uint16_t* B; uint16_t* dX;
    int M, n, r, rows_blocks, dx_shared, accumulate, njobs;
    SmallTn job[2];
};

// 32 rows x 64 columns of dX, contraction over r: by one wave, or (SHARED) by all of the work-group, wave w taking the
// steps of 16 columns of dT w, w + 8, ..
template <bool SHARED>
__device__ __forceinline__ void dx_tile(const SmallGrad& p, int rb, int tile, float (*red)[2][16][64]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int j = lane & 31, h = lane >> 5, row0 = 32 * rb, col = 64 * tile + 2 * j;
    const rsrc_t tres = make_rsrc(p.dT, (int64_t)p.M * p.r * 2), bres = make_rsrc(p.B, (int64_t)p.r * p.n * 2);
    const int toff = ((row0 + j) * p.r + 8 * h) * 2, boff = (8 * h * p.n + col) * 2;
    f32x16 acc[2];
    zero(acc[0]); zero(acc[1]);
    struct Step { u32x4 t; uint32_t b[8]; } buf[2];
    auto load = [&](Step& s, int k) {
        s.t = buf_load16(tres, toff, 32 * k);
#pragma unroll
        for (int i = 0; i < 8; ++i) s.b[i] = load4(bres, boff, (16 * k + i) * p.n * 2);
    };
    auto multiply = [&](const Step& s) {
        u32x4 op[2];
        unpair(s.b, op);
        acc[0] = mfma16(s.t, op[0], acc[0]);
        acc[1] = mfma16(s.t, op[1], acc[1]);
    };
    const int steps = p.r / 16, stride = SHARED ? kGradWaves : 1;
    int k = SHARED ? wave : 0;
    if (k < steps) load(buf[0], k);
    for (; k < steps; k += 2 * stride) {
        if (k + stride < steps) load(buf[1], k + stride);
        multiply(buf[0]);
        if (k + stride < steps) {
            if (k + 2 * stride < steps) load(buf[0], k + 2 * stride);
            multiply(buf[1]);
        }
    }
    const rsrc_t xres = make_rsrc(p.dX, (int64_t)p.M * p.n * 2);         // rows past M are dropped
    auto store = [&](int v, float t0, float t1) {
        __builtin_amdgcn_raw_buffer_store_b32(pack2_bf16(t0, t1), xres, ((row0 + acc_row(v, h)) * p.n + col) * 2, 0, 0);
    };
    if constexpr (!SHARED) {
#pragma unroll
        for (int v = 0; v < 16; ++v) store(v, acc[0][v], acc[1][v]);
    } else {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) red[wave][b][v][lane] = acc[b][v];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 16 / kGradWaves; ++e) {
            const int v = wave + kGradWaves * e;
            float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
            for (int w = 0; w < kGradWaves; ++w) { t0 += red[w][0][v][lane]; t1 += red[w][1][v][lane]; }
            store(v, t0, t1);
        }
    }
}

// A factored convolution: image [N, H, W, C], rows of dY, T and dT on the grid Ho x Wo
struct SmallConv { int N, H, W, Ho, Wo, C, kh, kw, stride; };

// 64 x 64 of C; wave w takes the steps of 16 rows w, w + 8, ..  GATHER: S is the patch matrix of an image; a tile's 64 columns lie in one tap, so the
// work-group looks up the pixel of every row once (offsets in `red`, which is free until the sums).
template <bool GATHER>
__device__ __forceinline__ void tn_tile(const SmallTn& g, int M, int accumulate, int tile, float (*red)[4][16][64], const SmallConv& cv) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, h = lane >> 5;
    const int i0 = 64 * (tile / g.tiles_q), j0 = 64 * (tile % g.tiles_q);
    const rsrc_t rres = make_rsrc(g.R, (int64_t)M * g.P * 2);
    const rsrc_t sres = make_rsrc(g.S, GATHER ? (int64_t)cv.N * cv.H * cv.W * cv.C * 2 : (int64_t)M * g.Q * 2);
    const int steps = (M + 15) / 16;
    int* const pixel = reinterpret_cast<int*>(red);
    if constexpr (GATHER) {
        const int tap = j0 / cv.C, ky = tap / cv.kw - cv.kh / 2, kx = tap % cv.kw - cv.kw / 2, per = cv.Ho * cv.Wo;
        for (int i = tid; i < 16 * steps; i += 64 * kGradWaves) {
            const int img = i / per, rem = i - img * per, yo = rem / cv.Wo;
            const int y = cv.stride * yo + ky, x = cv.stride * (rem - yo * cv.Wo) + kx;
            const bool ok = i < M && (unsigned)y < (unsigned)cv.H && (unsigned)x < (unsigned)cv.W;
            pixel[i] = ok ? (((img * cv.H + y) * cv.W + x) * cv.C + (j0 - tap * cv.C)) * 2 : kBufNowhere;
        }
        __syncthreads();
    }
    const bool rin = i0 + 2 * j < g.P, sin = j0 + 2 * j < g.Q;
    f32x16 acc[2][2];
    zero(acc[0][0]); zero(acc[0][1]); zero(acc[1][0]); zero(acc[1][1]);
    struct Step { uint32_t r[8], s[8]; } buf[2];
    auto load = [&](Step& d, int k) {
        // rows past M lie outside the descriptors: the row is part of the lane's offset, the only part that is checked
        const int ro = rin ? ((16 * k + 8 * h) * g.P + i0 + 2 * j) * 2 : kBufNowhere;
        const int so = sin ? ((16 * k + 8 * h) * g.Q + j0 + 2 * j) * 2 : kBufNowhere;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            d.r[i] = load4(rres, rin ? ro + i * g.P * 2 : kBufNowhere, 0);
            if constexpr (GATHER) d.s[i] = load4(sres, (int)((unsigned)pixel[16 * k + 8 * h + i] + 4u * j), 0);      // nowhere stays past any image
            else d.s[i] = load4(sres, sin ? so + i * g.Q * 2 : kBufNowhere, 0);
        }
    };
    auto multiply = [&](const Step& d) {
        u32x4 a[2], b[2];
        unpair(d.r, a);
        unpair(d.s, b);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[x][y] = mfma16(a[x], b[y], acc[x][y]);
    };
    int k = wave;
    if (k < steps) load(buf[0], k);
    for (; k < steps; k += 2 * kGradWaves) {
        if (k + kGradWaves < steps) load(buf[1], k + kGradWaves);
        multiply(buf[0]);
        if (k + kGradWaves < steps) {
            if (k + 2 * kGradWaves < steps) load(buf[0], k + 2 * kGradWaves);
            multiply(buf[1]);
        }
    }
    if constexpr (GATHER) __syncthreads();
    // wave w takes over the sums of wave w + 4, then all add up those of the first four, in order
    constexpr int half = kGradWaves / 2;
    if (wave >= half) {
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int v = 0; v < 16; ++v) red[wave - half][x][v][lane] = acc[x >> 1][x & 1][v];
    }
    __syncthreads();
    if (wave < half) {
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int v = 0; v < 16; ++v) red[wave][x][v][lane] += acc[x >> 1][x & 1][v];
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int e = 0; e < 16 / kGradWaves; ++e) {
            const int v = wave + kGradWaves * e;
            float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
            for (int w = 0; w < half; ++w) { t0 += red[w][2 * x][v][lane]; t1 += red[w][2 * x + 1][v][lane]; }
            const int row = i0 + 2 * acc_row(v, h) + x;
            if (row < g.P && sin) {
                f32x2* c = reinterpret_cast<f32x2*>(g.C + (int64_t)row * g.Q + j0 + 2 * j);
                f32x2 val = {t0, t1};
                if (accumulate) val += gload(c);
                gstore(c, val);
            }
        }
}

__global__ __launch_bounds__(64 * kGradWaves, 2) void small_grad_kernel(SmallGrad p) {
    __shared__ float red[kGradWaves / 2][4][16][64];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int b = (int)blockIdx.x;
    // the factor gradients first: their contraction is the longer chain
    for (int i = 0; i < p.njobs; ++i) {
        const int tiles = ((p.job[i].P + 63) / 64) * p.job[i].tiles_q;
        if (b < tiles) { tn_tile<false>(p.job[i], p.M, p.accumulate, b, red, SmallConv{}); return; }
        b -= tiles;
    }
    if (p.dX == nullptr) return;
    const int rb = b % p.rows_blocks, c = b / p.rows_blocks;
    if (p.dx_shared) dx_tile<true>(p, rb, c, reinterpret_cast<float (*)[2][16][64]>(red));
    else if (64 * (kGradWaves * c + wave) < p.n) dx_tile<false>(p, rb, kGradWaves * c + wave, nullptr);
}

// The gradients of a convolution: dAct [N, H, W, C] = the sum over taps of dT (shifted) . B, without a re-laid-out copy of B; dA and dB as
// above.  One launch for what are four or five elsewhere (copy of B, dAct, dA, dB and the sums of its parts).  Bound by latency as above: 14 x 14 x
// 256, 3 x 3, r = 64, 4 images, whole backward 38 us in the other kernels, 12 here.  M up to 16384 rows, whose offsets fit the LDS.
struct SmallConvGrad {
    const uint16_t* dT; const uint16_t* B; uint16_t* dAct;
    SmallConv cv;
    int M, n, r, accumulate, blocks_A, blocks_B;
    SmallTn A_job, B_job;
};

// 32 pixels x 64 channels of dAct; wave w takes the steps of 16 columns of dT, tap by tap, w, w + 8, ..  With stride 2 a tap reaches only the pixels
// of one parity, so the pixels are taken parity by parity.
__device__ __forceinline__ void dact_tile(const SmallConvGrad& p, int b, float (*red)[2][16][64]) {
    const SmallConv& cv = p.cv;
    const int lane = threadIdx.x & 63, j = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int tiles = cv.C / 64;
    int rb = b / tiles, py = 0, px = 0, RH = cv.H, RW = cv.W;
    const int col = 64 * (b - rb * tiles) + 2 * j, st = cv.stride;
    if (st == 2)
        for (int cls = 3; cls >= 0; --cls) {
            py = cls >> 1; px = cls & 1;
            RH = (cv.H - py + 1) / 2; RW = (cv.W - px + 1) / 2;
            const int blocks = (cv.N * RH * RW + 31) / 32;
            if (rb < blocks) break;
            rb -= blocks;
        }
    const int per = RH * RW, i = 32 * rb + j, img = i / per, rem = i - img * per, ry = rem / RW;
    const int y = st * ry + py, x = st * (rem - ry * RW) + px;
    const bool live = img < cv.N;
    const int at = live ? (img * cv.H + y) * cv.W + x : -1;
    const int gy = live ? y + cv.kh / 2 : -(1 << 24), gx = x + cv.kw / 2;        // no pixel: never on the grid of dT
    const int ky0 = (st - 1) & (py + cv.kh / 2), kx0 = (st - 1) & (px + cv.kw / 2);
    const int rs = p.r / 16, steps = ((cv.kh - ky0 + st - 1) / st) * ((cv.kw - kx0 + st - 1) / st) * rs;
    const rsrc_t tres = make_rsrc(p.dT, (int64_t)p.M * p.r * 2), bres = make_rsrc(p.B, (int64_t)p.r * p.n * 2);
    const int boff = (8 * h * p.n + col) * 2;
    f32x16 acc[2];
    zero(acc[0]); zero(acc[1]);
    struct Step { u32x4 t; uint32_t b[8]; } buf[2];
    int c = wave, ky = ky0, kx = kx0;                    // of the next step
    auto load = [&](Step& s) {
        while (c >= rs) { c -= rs; kx += st; if (kx >= cv.kw) { kx = kx0; ky += st; } }
        const int ty = (gy - ky) >> (st - 1), tx = (gx - kx) >> (st - 1);
        const bool ok = (unsigned)ty < (unsigned)cv.Ho && (unsigned)tx < (unsigned)cv.Wo;
        s.t = buf_load16(tres, ok ? (((img * cv.Ho + ty) * cv.Wo + tx) * p.r + 16 * c + 8 * h) * 2 : kBufNowhere, 0);
#pragma unroll
        for (int e = 0; e < 8; ++e) s.b[e] = load4(bres, boff, ((16 * c + e) * p.n + (ky * cv.kw + kx) * cv.C) * 2);
        c += kGradWaves;
    };
    auto multiply = [&](const Step& s) {
        u32x4 op[2];
        unpair(s.b, op);
        acc[0] = mfma16(s.t, op[0], acc[0]);
        acc[1] = mfma16(s.t, op[1], acc[1]);
    };
    int k = wave;
    if (k < steps) load(buf[0]);
    for (; k < steps; k += 2 * kGradWaves) {
        if (k + kGradWaves < steps) load(buf[1]);
        multiply(buf[0]);
        if (k + kGradWaves < steps) {
            if (k + 2 * kGradWaves < steps) load(buf[0]);
            multiply(buf[1]);
        }
    }
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[wave][b2][v][lane] = acc[b2][v];
    __syncthreads();
    const rsrc_t xres = make_rsrc(p.dAct, (int64_t)cv.N * cv.H * cv.W * cv.C * 2);
#pragma unroll
    for (int e = 0; e < 16 / kGradWaves; ++e) {
        const int v = wave + kGradWaves * e;
        float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
        for (int w = 0; w < kGradWaves; ++w) { t0 += red[w][0][v][lane]; t1 += red[w][1][v][lane]; }
        const int to = __shfl(at, acc_row(v, h));
        __builtin_amdgcn_raw_buffer_store_b32(pack2_bf16(t0, t1), xres, to >= 0 ? (to * cv.C + col) * 2 : kBufNowhere, 0, 0);
    }
}

__global__ __launch_bounds__(64 * kGradWaves, 2) void small_conv_grad_kernel(SmallConvGrad p) {
    __shared__ float red[kGradWaves / 2][4][16][64];
    const int b = (int)blockIdx.x;
    if (b < p.blocks_B) tn_tile<true>(p.B_job, p.M, p.accumulate, b, red, p.cv);
    else if (b - p.blocks_B < p.blocks_A) tn_tile<false>(p.A_job, p.M, p.accumulate, b - p.blocks_B, red, p.cv);
    else dact_tile(p, b - p.blocks_B - p.blocks_A, reinterpret_cast<float (*)[2][16][64]>(red));
}

}  // namespace

bool lr_small_supports(int64_t M, int m, int n, int r) {
    const int64_t widest = m > n ? (m > r ? m : r) : (n > r ? n : r);
    return M >= 1 && (M + 127) * widest * 2 < kBufMaxBytes && (int64_t)widest * r * 2 < kBufMaxBytes && m % 64 == 0 && n % 64 == 0 && r % 32 == 0;
}

namespace {
template <int RM, int CN, int SK, bool GATHER>
hipError_t launch_nt(SmallNt p, int problems, hipStream_t s) {
    using G = Nt<RM, CN, SK>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&small_nt_kernel<RM, CN, SK, GATHER>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, G::lds_bytes);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    p.tiles_n = (int)ceil_div(p.N, G::cols);
    hipLaunchKernelGGL((small_nt_kernel<RM, CN, SK, GATHER>), dim3((unsigned)(ceil_div(p.M, G::rows) * p.tiles_n), (unsigned)problems), dim3(G::threads),
                       G::lds_bytes, s, p);
    return hipGetLastError();
}

// T: a long contraction and few columns.  The smallest tile whose work-groups, one per compute unit, still run all at once.  us for both launches with a
// tile of 32 x 32 by eight waves / 32 x 64 by eight / 64 x 64 by eight / 64 x 128:
//   768 -> 2304, r = 384: 197 rows 10.6 / 10.1 / 11.6 / 12.1, 1000 18.3 / 16.2 / 17.3 / 18.3, 2000 27.7 / 26.1 / 23.7 / 24.4, 4000 48 / 40 / 38 / 35;
//   3072 -> 768, r = 384: 13.2 / 15.4 / 18.6 / 25.6, 22.9 / 17.5 / 21.0 / 28.5, 32.6 / 29.8 / 24.5 / 30.7, 58 / 45 / 41 / 35.
template <bool GATHER>
hipError_t launch_t(const SmallNt& p, int problems, int of, hipStream_t s) {
    auto groups = [&](int rows, int cols) { return of * ceil_div(p.M, rows) * ceil_div(p.N, cols); };
    if (groups(32, 32) <= 256) return launch_nt<1, 1, 8, GATHER>(p, problems, s);
    if (groups(32, 64) <= 256) return launch_nt<1, 2, 4, GATHER>(p, problems, s);
    if (groups(64, 64) <= 256) return launch_nt<2, 2, 2, GATHER>(p, problems, s);
    return launch_nt<2, 4, 1, GATHER>(p, problems, s);
}
// Y: the contraction is the rank, which four waves read whole (64 x 64 / 64 x 128: 197 x 2304 9.2 / 9.4 at r = 384, 1000 x 2304 15.1 / 15.9,
// 4000 x 2304 38.8 / 38.1; 32 x 64 shared by eight waves 78)
hipError_t launch_y(const SmallNt& p, int problems, hipStream_t s) {
    if (problems * ceil_div(p.M, 64) * ceil_div(p.N, 64) <= 1024) return launch_nt<2, 2, 1, false>(p, problems, s);
    return launch_nt<2, 4, 1, false>(p, problems, s);
}
}  // namespace

hipError_t launch_lr_small_fwd(const ChainProblem* problems, int G, int of, int64_t M, int p, int q, int R, hipStream_t s) {
    if (G < 1 || G > kChainMaxGroups || of < G || !lr_small_supports(M, q, p, R)) return hipErrorInvalidValue;
    SmallNt t{}, y{};
    t.M = y.M = (int)M;
    t.N = R; t.K = p; t.u_bytes = M * p * 2;
    y.N = q; y.K = R; y.u_bytes = M * R * 2;
    for (int g = 0; g < G; ++g) {
        const ChainProblem& c = problems[g];
        if (!c.Tout || (c.Yout != nullptr) != (problems[0].Yout != nullptr)) return hipErrorInvalidValue;
        t.e[g] = SmallNtEntry{(const uint16_t*)c.Xin, (const uint16_t*)c.P, (uint16_t*)c.Tout};
        y.e[g] = SmallNtEntry{(const uint16_t*)c.Tout, (const uint16_t*)c.Q, (uint16_t*)c.Yout};
    }
    const hipError_t e = launch_t<false>(t, G, of, s);
    return e != hipSuccess || !problems[0].Yout ? e : launch_y(y, G, s);
}

bool lr_small_gather_supports(const PatchGeom& g, int64_t M, int q, int R) {
    const int64_t p = (int64_t)g.kh * g.kw * g.Cin, per = (int64_t)g.RH * g.RW;
    if (g.sign != 1 || g.shift != 0 || g.Cin % 64 || p > (1 << 20) || per < 1 || M % per != 0) return false;
    return (M / per) * g.H * g.W * g.Cin * 2 < kBufMaxBytes && (p + 127) * R * 2 < kBufMaxBytes && lr_small_supports(M, q, q, R);
}

hipError_t launch_lr_small_fwd_gather(const void* image, const PatchGeom& g, const void* P, const void* Q, void* Yout, void* Tout, int64_t M, int q, int R,
                                      hipStream_t s) {
    if (!Tout || !lr_small_gather_supports(g, M, q, R)) return hipErrorInvalidValue;
    SmallNt t{}, y{};
    t.M = y.M = (int)M;
    t.e[0] = SmallNtEntry{(const uint16_t*)image, (const uint16_t*)P, (uint16_t*)Tout};
    t.N = R; t.K = g.kh * g.kw * g.Cin; t.u_bytes = (M / ((int64_t)g.RH * g.RW)) * g.H * g.W * g.Cin * 2;
    t.H = g.H; t.W = g.W; t.Cin = g.Cin; t.kh = g.kh; t.kw = g.kw; t.RH = g.RH; t.RW = g.RW; t.mul = g.mul;
    y.e[0] = SmallNtEntry{(const uint16_t*)Tout, (const uint16_t*)Q, (uint16_t*)Yout};
    y.N = q; y.K = R; y.u_bytes = M * R * 2;
    const hipError_t e = launch_t<true>(t, 1, 1, s);
    return e != hipSuccess || !Yout ? e : launch_y(y, 1, s);
}

hipError_t launch_lr_small_dt(const void* dY, const void* A, void* dT, int64_t M, int m, int r, hipStream_t s) {
    if (!lr_small_supports(M, m, m, r)) return hipErrorInvalidValue;
    const SmallDt d{(const uint16_t*)dY, (const uint16_t*)A, (uint16_t*)dT, (int)M, m, r};
    // (tiles of 32 columns / 64, backward, us: 197 x 768 -> 2304, r = 96 12.2 / 13.2, 1600 rows 20.2 / 21.3; 94 row blocks x 2 even; past one tile
    // for each compute unit 64 columns read dY less often: 800 rows, r = 384, 300 tiles 31 / 25, 3000 rows, r = 96, 282 tiles 34 / 27)
    const int64_t blocks = ceil_div(M, 32);
    if (blocks * (r / 32) <= 256) hipLaunchKernelGGL(small_dt_kernel<32>, dim3((unsigned)blocks, (unsigned)(r / 32)), dim3(64 * kDtWaves), 0, s, d);
    else hipLaunchKernelGGL(small_dt_kernel<64>, dim3((unsigned)blocks, (unsigned)ceil_div(r, 64)), dim3(64 * kDtWaves), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_lr_small_grad(const void* dY, const void* X, const void* T, const void* B, void* dX, float* dA, float* dB, const void* dT,
                                int64_t M, int m, int n, int r, int accumulate, hipStream_t s) {
    if (!lr_small_supports(M, m, n, r)) return hipErrorInvalidValue;
    if (!dX && !dA && !dB) return hipSuccess;
    const int blocks = (int)ceil_div(M, 32);
    SmallGrad g{};
    g.dT = (const uint16_t*)dT; g.B = (const uint16_t*)B; g.dX = (uint16_t*)dX;
    g.M = (int)M; g.n = n; g.r = r; g.rows_blocks = blocks; g.accumulate = accumulate;
    int64_t grid = 0;
    auto job = [&](const void* R, const void* S, float* C, int P, int Q) {
        const int tq = (int)ceil_div(Q, 64);
        g.job[g.njobs++] = SmallTn{(const uint16_t*)R, (const uint16_t*)S, C, P, Q, tq};
        grid += ceil_div(P, 64) * tq;
    };
    if (dA) job(dY, T, dA, m, r);
    if (dB) job(dT, X, dB, r, n);
    const int64_t tiles = grid;
    // A work-group per tile of dX for few tiles and wide ranks, else a wave per tile (backward, us, n = 768: r = 384, 84 tiles
    // 18.8 / 24.9, 384 tiles 28.9 / 30.7; r = 192, 84 tiles 14.9 / 17.0, 384 tiles 22.3 / 19.8; r = 96 the same for few, n = 3072, 336
    // tiles 12.8 / 10.4).
    g.dx_shared = r >= 160 && (int64_t)blocks * (n / 64) <= 256;
    if (dX) grid += (int64_t)blocks * (g.dx_shared ? n / 64 : ceil_div(n, 64 * kGradWaves));
    // Two work-groups share a compute unit.  Only one does (LDS that nobody uses keeps the other away) where the few tiles of dA and dB are the longest chains,
    // in rows, and would wait for those of dX, in ranks, beside them.  Backward, us, two / one: 4063 rows, 1280 -> 256, r = 288 (120 tiles) 34.7 / 29.7;
    // 2494 rows, 1792 -> 128, r = 160 (90) 22.0 / 19.1;  2051 rows, 1344 -> 704, r = 320 (160) 40.8 / 42.3.  Of 4500 shapes of 300 to 4096 rows two are more than
    // 3 % slower for 190 than the kernel was with one, one for 860 than with two; by this rule some 25 each.
    const size_t alone = tiles <= 120 && grid <= 640 && M > 1400 && M > 10 * (int64_t)r ? 24 * 1024 : 0;
    hipLaunchKernelGGL(small_grad_kernel, dim3((unsigned)grid), dim3(64 * kGradWaves), alone, s, g);
    return hipGetLastError();
}

bool lr_small_conv_supports(const ConvShape& g, int64_t M, int m, int r) {
    const int64_t n = (int64_t)g.kh * g.kw * g.C;
    return M <= 16384 && g.C % 64 == 0 && n <= (1 << 20) && (int64_t)g.N * g.H * g.W * g.C * 2 < kBufMaxBytes && n * r * 2 < kBufMaxBytes &&
           lr_small_supports(M, m, m, r);
}

hipError_t launch_lr_small_conv_grad(const ConvShape& g, const void* dY, const void* act, const void* T, const void* B, void* dAct, float* dA, float* dB,
                                     const void* dT, int64_t M, int m, int r, int accumulate, hipStream_t s) {
    if (!lr_small_conv_supports(g, M, m, r) || (dA && !T) || ((dAct || dB) && !dT)) return hipErrorInvalidValue;
    const int64_t n = (int64_t)g.kh * g.kw * g.C;
    SmallConvGrad p{};
    p.dT = (const uint16_t*)dT; p.B = (const uint16_t*)B; p.dAct = (uint16_t*)dAct;
    p.cv = SmallConv{g.N, g.H, g.W, g.Ho, g.Wo, g.C, g.kh, g.kw, g.stride};
    p.M = (int)M; p.n = (int)n; p.r = r; p.accumulate = accumulate;
    const int tiles_r = (int)ceil_div(r, 64);
    if (dA) { p.A_job = SmallTn{(const uint16_t*)dY, (const uint16_t*)T, dA, m, r, tiles_r}; p.blocks_A = m / 64 * tiles_r; }
    if (dB) { p.B_job = SmallTn{(const uint16_t*)dT, (const uint16_t*)act, dB, r, (int)n, (int)(n / 64)}; p.blocks_B = (int)(n / 64) * tiles_r; }
    int64_t grid = (int64_t)p.blocks_A + p.blocks_B, rows = 0;
    for (int cls = 0; cls < (g.stride == 2 ? 4 : 1); ++cls) {
        const int64_t RH = g.stride == 2 ? (g.H - (cls >> 1) + 1) / 2 : g.H, RW = g.stride == 2 ? (g.W - (cls & 1) + 1) / 2 : g.W;
        rows += ceil_div(g.N * RH * RW, 32);
    }
    if (dAct) grid += rows * (g.C / 64);
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL(small_conv_grad_kernel, dim3((unsigned)grid), dim3(64 * kGradWaves), 0, s, p);
    return hipGetLastError();
}

}  // namespace abt
