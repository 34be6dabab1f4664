// Backward of the bf16 factored layer for few rows, in two launches:
//     dT[M,r] = dY[M,m] . A[m,r]                                       (small_dt_kernel)
//     dX[M,n] = dT . B[r,n],  dA[m,r] = dY^T . T,  dB[r,n] = dT^T . X   (small_grad_kernel, all of them at once)
//
// What bounds it: latency.  The kernels for many rows walk a contraction of thousands of columns in one work-group per
// 64 rows, a barrier per slab of 64, behind a launch that transposes the factors, and the factor gradients
// come in two more launches.  Here nothing is staged: operands come straight from memory (L2) into registers, a work-group's waves
// share out the contraction and add their sums once through LDS, and tiles are small, so that a layer of 200 rows is some
// hundred work-groups.  A factor (or a batch) whose contraction index is its slow dimension is read as it lies: a lane
// loads, for each of the eight k of its operand, the 4 bytes of two neighbouring columns, and the two columns go to
// two 32-wide blocks of the tile (byte permutes); column c of a 64-wide tile is lane c / 2 of block c % 2, and results leave in
// pairs of columns.
//
// MFMA 32x32x16 bf16 layout (lane l, j = l % 32, h = l / 32): A operand = 8 values A[j][8h .. 8h+7], B operand
// = B[8h .. 8h+7][j], accumulator v = C[8 (v / 4) + 4h + v % 4][j].
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

// ------------------------------------------------------------------ dT
constexpr int kDtWaves = 8;

struct SmallDt { const uint16_t* dY; const uint16_t* A; uint16_t* dT; int M, m, r; };

// 32 rows x 64 columns of dT; wave w takes the slabs of 64 columns of dY w, w + 8, ..
__global__ __launch_bounds__(64 * kDtWaves, 2) void small_dt_kernel(SmallDt p) {
    __shared__ float red[kDtWaves][2][16][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 31, h = lane >> 5;
    const int row0 = 32 * (int)blockIdx.x, col = 64 * (int)blockIdx.y + 2 * j;
    const rsrc_t xres = make_rsrc(p.dY, (int64_t)p.M * p.m * 2), ares = make_rsrc(p.A, (int64_t)p.m * p.r * 2);
    const int xoff = ((row0 + j) * p.m + 8 * h) * 2;                 // rows past M: outside the descriptor, zeros
    const int aoff = col < p.r ? (8 * h * p.r + col) * 2 : kBufNowhere;
    f32x16 acc[2];
    zero(acc[0]); zero(acc[1]);
    struct Slab { u32x4 x[4]; uint32_t a[4][8]; } buf[2];
    auto load = [&](Slab& s, int slab) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            s.x[q] = buf_load16(xres, xoff, (64 * slab + 16 * q) * 2);
#pragma unroll
            for (int i = 0; i < 8; ++i) s.a[q][i] = load4(ares, aoff, (64 * slab + 16 * q + i) * p.r * 2);
        }
    };
    auto multiply = [&](const Slab& s) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32x4 op[2];
            unpair(s.a[q], op);
            acc[0] = mfma16(s.x[q], op[0], acc[0]);
            acc[1] = mfma16(s.x[q], op[1], acc[1]);
        }
    };
    const int slabs = p.m / 64;
    int s = wave;
    if (s < slabs) load(buf[0], s);
    for (; s < slabs; s += 2 * kDtWaves) {
        if (s + kDtWaves < slabs) load(buf[1], s + kDtWaves);
        multiply(buf[0]);
        if (s + kDtWaves < slabs) {
            if (s + 2 * kDtWaves < slabs) load(buf[0], s + 2 * kDtWaves);
            multiply(buf[1]);
        }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[wave][b][v][lane] = acc[b][v];
    __syncthreads();
    const rsrc_t tres = make_rsrc(p.dT, (int64_t)p.M * p.r * 2);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int v = wave + kDtWaves * e;
        float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
        for (int w = 0; w < kDtWaves; ++w) { t0 += red[w][0][v][lane]; t1 += red[w][1][v][lane]; }
        const int off = col < p.r ? ((row0 + acc_row(v, h)) * p.r + col) * 2 : kBufNowhere;      // rows past M are dropped
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
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
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

// 64 x 64 of C; wave w takes the steps of 16 rows w, w + 8, ..
__device__ __forceinline__ void tn_tile(const SmallTn& g, int M, int accumulate, int tile, float (*red)[4][16][64]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 31, h = lane >> 5;
    const int i0 = 64 * (tile / g.tiles_q), j0 = 64 * (tile % g.tiles_q);
    const rsrc_t rres = make_rsrc(g.R, (int64_t)M * g.P * 2), sres = make_rsrc(g.S, (int64_t)M * g.Q * 2);
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
            d.s[i] = load4(sres, sin ? so + i * g.Q * 2 : kBufNowhere, 0);
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
    const int steps = (M + 15) / 16;
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
    const int wave = threadIdx.x >> 6;
    int b = (int)blockIdx.x;
    // the factor gradients first: their contraction is the longer chain
    for (int i = 0; i < p.njobs; ++i) {
        const int tiles = ((p.job[i].P + 63) / 64) * p.job[i].tiles_q;
        if (b < tiles) { tn_tile(p.job[i], p.M, p.accumulate, b, red); return; }
        b -= tiles;
    }
    if (p.dX == nullptr) return;
    const int rb = b % p.rows_blocks, c = b / p.rows_blocks;
    if (p.dx_shared) dx_tile<true>(p, rb, c, reinterpret_cast<float (*)[2][16][64]>(red));
    else if (64 * (kGradWaves * c + wave) < p.n) dx_tile<false>(p, rb, kGradWaves * c + wave, nullptr);
}

}  // namespace

bool lr_small_supports(int64_t M, int m, int n, int r) {
    const int64_t widest = m > n ? (m > r ? m : r) : (n > r ? n : r);
    return M >= 1 && (M + 31) * widest * 2 < kBufMaxBytes && (int64_t)widest * r * 2 < kBufMaxBytes && m % 64 == 0 && n % 64 == 0 && r % 32 == 0;
}

hipError_t launch_lr_small_dt(const void* dY, const void* A, void* dT, int64_t M, int m, int r, hipStream_t s) {
    if (!lr_small_supports(M, m, m, r)) return hipErrorInvalidValue;
    const SmallDt d{(const uint16_t*)dY, (const uint16_t*)A, (uint16_t*)dT, (int)M, m, r};
    hipLaunchKernelGGL(small_dt_kernel, dim3((unsigned)ceil_div(M, 32), (unsigned)ceil_div(r, 64)), dim3(64 * kDtWaves), 0, s, d);
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
    // A work-group per tile of dX for few tiles and wide ranks, else a wave per tile (backward, us, n = 768: r = 384, 84 tiles
    // 18.8 / 24.9, 384 tiles 28.9 / 30.7; r = 192, 84 tiles 14.9 / 17.0, 384 tiles 22.3 / 19.8; r = 96 the same for few, n = 3072, 336
    // tiles 12.8 / 10.4).
    g.dx_shared = r >= 160 && (int64_t)blocks * (n / 64) <= 256;
    if (dX) grid += (int64_t)blocks * (g.dx_shared ? n / 64 : ceil_div(n, 64 * kGradWaves));
    hipLaunchKernelGGL(small_grad_kernel, dim3((unsigned)grid), dim3(64 * kGradWaves), 0, s, g);
    return hipGetLastError();
}

}  // namespace abt
