// The fp32 layer at its smallest (up to 64 rows, ranks up to 32, both widths up to 512): forward and backward in one launch each.
//
// Nothing but latency: as products of their own T, Y, dT and {dX, dA, dB} take 6 to 8 us each (first loads, a few slabs, a launch on the host)
// for 0.5 to 2 us of matrix instructions.  Here every work-group makes the rows of T (dT) that it needs itself, in LDS: 32 rows for a tile of Y or
// dX, all of them for a tile of dB.  64 x 256 x 256, r = 32, us of the GPU: forward 12.0 -> 7.7, backward 12.3 -> 9.7; the step, which the host's
// two launches instead of four bound then, 28 -> 22, with the calls in native code and two teams of waves in the backward 17.4.  The limits are where making T again costs what a launch does: at r = 64 the forward of 64 x 512 x 512
// 13.3 -> 15.8, the backward 13.6 -> 28.9; at r = 32 two blocks of rows by two chunks of the contraction, backward 13.6 -> 17.2.
//
// v_mfma_f32_32x32x2: A operand lane l = A[l % 32][l / 32], B operand = B[l / 32][l % 32], accumulator register v = C[8 (v / 4) + 4 (l / 32) + v % 4][l % 32].
// Instruction i of a group of eight k takes k = 4 h + i from the lanes of half h, the same permutation on both sides: one 16-byte LDS read
// per operand and group.  All sums are in the order of the 32 x 32 tiles of gemm_f32.hip (four parts, two groups of each 64 k; their sum), which
// serve the calls that do not come here: whether one does (its T kept or not, an output over an input) changes no bit.
#include "common.h"

namespace abt {

namespace {

constexpr int CH = 256;              // contraction indices in LDS at a time
constexpr int PITCH = CH + 4;        // floats per row: 16 rows of the same chunk in 16 bank groups
constexpr int TP = 32 + 4;           // of T [32 rows][column]
constexpr int RP = 64 + 4;           // of T [column][64 rows]

// A work-group is one or two teams of four waves; the second has the rows from 32 on.
template <int TEAMS>
struct TinyLds {
    float P[TEAMS][32 * PITCH];      // 32 rows of X or dY
    float F[32 * PITCH];             // the factor, [column of T][k]
    float red[TEAMS][4][16 * 64];    // sums of the four waves
    float T[32 * RP];                // 32 rows of T or all of them
    float T2[TEAMS == 2 ? 32 * TP : 4];      // as [row][column], the second team's 32 rows
};

// 32 rows from r0 on of a matrix [rows][K], CH indices from k0 on, to LDS; what lies outside is zero.
template <bool VEC>
struct RowLoader {
    f32x4 v[8];
    __device__ __forceinline__ void load(const float* m, int r0, int rows, int k0, int K) {
        const int t = threadIdx.x & 255, k = k0 + 4 * (t & 63);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int r = r0 + (t >> 6) + 4 * e;
            const float* p = m + (int64_t)(r < rows ? r : 0) * K;
            if constexpr (VEC) v[e] = gload(reinterpret_cast<const f32x4*>(p + (k < K ? k : 0)));
            else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[e][i] = gload(p + (k + i < K ? k + i : 0));
            }
        }
    }
    __device__ __forceinline__ void store(float* lds, int r0, int rows, int k0, int K) {
        const int t = threadIdx.x & 255, k = k0 + 4 * (t & 63);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int row = (t >> 6) + 4 * e;
            f32x4 x = v[e];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = r0 + row < rows && k + i < K ? x[i] : 0.0f;
            *reinterpret_cast<f32x4*>(lds + row * PITCH + 4 * (t & 63)) = x;
        }
    }
};
// The factor [k][column] (column fast in memory): all r columns of CH indices, transposed on the way to LDS.
template <int TEAMS>
struct ColumnLoader {
    float v[32 / TEAMS];
    __device__ __forceinline__ void load(const float* m, int r, int k0, int K) {
        const int j = threadIdx.x & 31;
#pragma unroll
        for (int e = 0; e < 32 / TEAMS; ++e) {
            const int k = k0 + (threadIdx.x >> 5) + 8 * TEAMS * e;
            v[e] = gload(m + (int64_t)(k < K ? k : 0) * r + (j < r ? j : 0));
        }
    }
    __device__ __forceinline__ void store(float* lds, int r, int k0, int K) {
        const int j = threadIdx.x & 31;
#pragma unroll
        for (int e = 0; e < 32 / TEAMS; ++e) {
            const int kk = (threadIdx.x >> 5) + 8 * TEAMS * e;
            lds[j * PITCH + kk] = j < r && k0 + kk < K ? v[e] : 0.0f;
        }
    }
};

// Rows r0 .. r0 + 31 (each team's own) of T = P . F' (KSLOW: F is [K][r], else [r][K]) to Tl, as [row][column] of pitch TP, or (TR) as [column][row] of pitch RP.
template <bool KSLOW, bool VEC, bool TR, int TEAMS>
__device__ __forceinline__ void rows_of_T(TinyLds<TEAMS>& sh, const float* P, const float* F, int r0, int M, int K, int r, float* Tl) {
    const int t = threadIdx.x, lane = t & 63, wave = (t >> 6) & 3, li = lane & 31, lh = lane >> 5, team = t >> 8;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    for (int k0 = 0; k0 < K; k0 += CH) {
        RowLoader<VEC> p;
        p.load(P, r0, M, k0, K);
        if constexpr (KSLOW) {
            ColumnLoader<TEAMS> f;
            f.load(F, r, k0, K);
            __syncthreads();                              // LDS of the chunk before is read
            p.store(sh.P[team], r0, M, k0, K);
            f.store(sh.F, r, k0, K);
        } else {
            RowLoader<VEC> f;
            f.load(F, 0, r, k0, K);
            __syncthreads();
            p.store(sh.P[team], r0, M, k0, K);
            f.store(sh.F, 0, r, k0, K);
        }
        __syncthreads();
        const int groups = K - k0 < CH ? (K - k0 + 7) / 8 : CH / 8;
        for (int g0 = 2 * wave; g0 < groups; g0 += 8)     // the waves share out the contraction, two groups of each 64 columns
#pragma unroll
            for (int g = g0; g < g0 + 2; ++g) {
                const f32x4 a = *reinterpret_cast<const f32x4*>(sh.P[team] + li * PITCH + 8 * g + 4 * lh);
                const f32x4 b = *reinterpret_cast<const f32x4*>(sh.F + li * PITCH + 8 * g + 4 * lh);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], acc, 0, 0, 0);
            }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) sh.red[team][wave][v * 64 + lane] = acc[v];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int v = wave + 4 * e, at = v * 64 + lane;
        const float s = ((sh.red[team][0][at] + sh.red[team][1][at]) + sh.red[team][2][at]) + sh.red[team][3][at];
        const int row = 8 * (v >> 2) + 4 * lh + (v & 3);
        Tl[TR ? li * RP + row : row * TP + li] = s;
    }
    __syncthreads();
}

// Operands of N groups of eight k for this lane's column: rows k of a matrix [rows][ld] (clamped; tile_product drops what is outside)
template <int N>
__device__ __forceinline__ void column_operands(float (&f)[N][4], const float* m, int rows, int64_t ld, int col, int cols) {
    const int lh = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int g = 0; g < N; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 8 * g + 4 * lh + i;
            f[g][i] = gload(m + (int64_t)(k < rows ? k : 0) * ld + (col < cols ? col : 0));
        }
}
// C[32 x 32] of a wave over `rows` k: a(g) gives the first operand's four values of group g.  A sum for each two groups, added in order.
template <int N, class A>
__device__ __forceinline__ f32x16 tile_product(A&& a, const float (&f)[N][4], int rows) {
    const int lh = (threadIdx.x >> 5) & 1;
    f32x16 acc[N / 2];
#pragma unroll
    for (int w = 0; w < N / 2; ++w)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[w][v] = 0.0f;
#pragma unroll
    for (int g = 0; g < N; ++g) {
        if (8 * g >= rows) break;
        const f32x4 x = a(g);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = 8 * g + 4 * lh + i < rows;    // past the contraction both sides are zero
            acc[g / 2] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? x[i] : 0.0f, in ? f[g][i] : 0.0f, acc[g / 2], 0, 0, 0);
        }
    }
#pragma unroll
    for (int w = 1; w < N / 2; ++w) acc[0] += acc[w];
    return acc[0];
}
template <class F>
__device__ __forceinline__ void each_value(const f32x16& acc, F&& f) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 16; ++v) f(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), lane & 31, acc[v]);
}

// Work-group: 32 rows and 128 columns of Y, a wave 32 of them.
template <bool VEC>
__global__ __launch_bounds__(256) void tiny_fwd_kernel(const float* X, const float* A, const float* B, float* Y, float* T, int M, int m, int n, int r) {
    __shared__ __align__(16) TinyLds<1> sh;
    const int r0 = (int)blockIdx.y * 32, li = threadIdx.x & 31, lh = (threadIdx.x >> 5) & 1;
    const int col = (int)blockIdx.x * 128 + 32 * (threadIdx.x >> 6) + li;
    // this wave's operands of the second product (four consecutive k of a row of A), asked for before the first
    float f[4][4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 8 * g + 4 * lh + i;
            f[g][i] = gload(A + (int64_t)(col < m ? col : 0) * r + (k < r ? k : 0));
        }
    rows_of_T<false, VEC, false>(sh, X, B, r0, M, n, r, sh.T);
    if (T != nullptr && blockIdx.x == 0)
        for (int i = threadIdx.x; i < 32 * r; i += 256) {
            const int row = i / r, j = i - row * r;
            if (r0 + row < M) gstore(T + (int64_t)(r0 + row) * r + j, sh.T[row * TP + j]);
        }
    const f32x16 acc = tile_product([&](int g) { return *reinterpret_cast<const f32x4*>(sh.T + li * TP + 8 * g + 4 * lh); }, f, r);
    each_value(acc, [&](int row, int, float v) {
        if (r0 + row < M && col < m) gstore(Y + (int64_t)(r0 + row) * m + col, v);
    });
}

// Work-groups: tiles of dB (128 columns of X per team), of dX (32 rows per team, 128 columns) and of dA (128 columns of dY per team), in this order.  Two teams
// for more than 32 rows: a tile of dB needs all rows of dT, which one team made one block after the other (64 x 256 x 256, r = 32: 11.0 us, two teams 9.7).
struct TinyBwd { const float* dY; const float* X; const float* T; const float* A; const float* B; float* dX; float* dA; float* dB; int M, m, n, r, accumulate; };

template <bool VEC, int TEAMS>
__global__ __launch_bounds__(256 * TEAMS) void tiny_bwd_kernel(TinyBwd p) {
    __shared__ __align__(16) TinyLds<TEAMS> sh;
    const int wave = (threadIdx.x >> 6) & 3, team = threadIdx.x >> 8, li = threadIdx.x & 31, lh = (threadIdx.x >> 5) & 1, M = p.M, m = p.m, n = p.n, r = p.r;
    const int wide = 128 * TEAMS, nb = (n + wide - 1) / wide, nx = (n + 127) / 128;
    int job = (int)blockIdx.x;
    auto put = [&](float* out, int64_t at, float v) { gstore(out + at, p.accumulate ? v + gload(out + at) : v); };
    if (p.dB != nullptr) {
        if (job < nb) {                                   // dB = dT^T X
            const int c0 = job * wide + 128 * team + 32 * wave;
            float f[8][4];
            column_operands(f, p.X, M, n, c0 + li, n);
            rows_of_T<true, VEC, true>(sh, p.dY, p.A, 32 * team, M, m, r, sh.T + 32 * team);
            const f32x16 acc = tile_product([&](int g) { return *reinterpret_cast<const f32x4*>(sh.T + li * RP + 8 * g + 4 * lh); }, f, M);
            each_value(acc, [&](int j, int c, float v) {
                if (j < r && c0 + c < n) put(p.dB, (int64_t)j * n + c0 + c, v);
            });
            return;
        }
        job -= nb;
    }
    if (p.dX != nullptr) {
        if (job < nx) {                                   // dX = dT B
            const int r0 = 32 * team, c0 = job * 128 + 32 * wave;
            float* const Tl = TEAMS == 2 && team == 1 ? sh.T2 : sh.T;
            float f[4][4];
            column_operands(f, p.B, r, n, c0 + li, n);
            rows_of_T<true, VEC, false>(sh, p.dY, p.A, r0, M, m, r, Tl);
            const f32x16 acc = tile_product([&](int g) { return *reinterpret_cast<const f32x4*>(Tl + li * TP + 8 * g + 4 * lh); }, f, r);
            each_value(acc, [&](int row, int c, float v) {
                if (r0 + row < M && c0 + c < n) gstore(p.dX + (int64_t)(r0 + row) * n + c0 + c, v);
            });
            return;
        }
        job -= nx;
    }
    // dA = dY^T T: both operands from memory, k = row
    const int c0 = job * wide + 128 * team + 32 * wave;
    float f[8][4], q[8][4];
    column_operands(f, p.dY, M, m, c0 + li, m);
    column_operands(q, p.T, M, r, li, r);
    const f32x16 acc = tile_product([&](int g) { return f32x4{f[g][0], f[g][1], f[g][2], f[g][3]}; }, q, M);
    each_value(acc, [&](int row, int j, float v) {
        if (c0 + row < m && j < r) put(p.dA, (int64_t)(c0 + row) * r + j, v);
    });
}

bool rows16(const float* p, int64_t ld) { return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 4 == 0; }

}  // namespace

bool tiny_f32_supports(int64_t M, int64_t m, int64_t n, int64_t r) { return M <= 64 && r <= 32 && m <= 512 && n <= 512; }

hipError_t launch_tiny_f32_fwd(const float* X, const float* A, const float* B, float* Y, float* T, int64_t M, int64_t m, int64_t n, int64_t r, hipStream_t s) {
    if (!tiny_f32_supports(M, m, n, r)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)ceil_div(m, 128), (unsigned)ceil_div(M, 32));
    auto go = [&](auto* k) { hipLaunchKernelGGL(k, grid, dim3(256), 0, s, X, A, B, Y, T, (int)M, (int)m, (int)n, (int)r); };
    if (rows16(X, n) && rows16(B, n)) go(&tiny_fwd_kernel<true>);
    else go(&tiny_fwd_kernel<false>);
    return hipGetLastError();
}

hipError_t launch_tiny_f32_bwd(const float* dY, const float* X, const float* T, const float* A, const float* B, float* dX, float* dA, float* dB,
                               int64_t M, int64_t m, int64_t n, int64_t r, int accumulate, hipStream_t s) {
    if (!tiny_f32_supports(M, m, n, r) || (dA && !T)) return hipErrorInvalidValue;
    const TinyBwd p{dY, X, T, A, B, dX, dA, dB, (int)M, (int)m, (int)n, (int)r, accumulate};
    const int teams = M > 32 ? 2 : 1, wide = 128 * teams;
    const int grid = (int)((dB ? ceil_div(n, wide) : 0) + (dX ? ceil_div(n, 128) : 0) + (dA ? ceil_div(m, wide) : 0));
    if (grid == 0) return hipSuccess;
    auto go = [&](auto* k) { hipLaunchKernelGGL(k, dim3(grid), dim3(256 * teams), 0, s, p); };
    if (rows16(dY, m)) teams == 2 ? go(&tiny_bwd_kernel<true, 2>) : go(&tiny_bwd_kernel<true, 1>);
    else teams == 2 ? go(&tiny_bwd_kernel<false, 2>) : go(&tiny_bwd_kernel<false, 1>);
    return hipGetLastError();
}

}  // namespace abt
