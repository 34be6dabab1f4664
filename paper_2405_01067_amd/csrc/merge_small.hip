// The stages of the merge around the Jacobi iteration for layers with a core of 32 (K = 32), three launches in the place of eight: the work of each
// is next to nothing and a launch with its first loads takes 4 to 13 us (one 256 x 256 layer, G = 2: 103 us of Gram matrix, Cholesky,
// core, norm, sort and projectors; now 27).  Results as in the stages for all sizes, but for the order of the fp64 sums.
//   gram32_kernel    average of the copies and their Gram matrix, the contraction shared among up to 16 work-groups per side (one walked
//                    through 256 rows in 35 us, a memory latency per 32 of them)
//   core32_kernel    one work-group per layer: sum of those parts, both Cholesky factors, C^T = L_B^T L_A, ||C||_F^2
//   finish32_kernel  one work-group per layer: singular values, rank, both projection matrices
#include "merge_internal.h"

namespace abt {

namespace {

// contraction indices per work-group of a side of `len`: the part of each of at most kGramParts, in whole steps of 64
__device__ __forceinline__ int gram_part(int len) { return ((len + kGramParts - 1) / kGramParts + 63) / 64 * 64; }

// Work-group (part, side, layer).
__global__ __launch_bounds__(256) void gram32_kernel(const LayerDev* __restrict__ layers) {
    constexpr int PA = 48, PB = 65;                       // LDS pitch, A side [index][column] / B side [row][index]
    __shared__ float X[64 * PA];
    __shared__ double red[4][3][256];
    const LayerDev& L = layers[blockIdx.z];
    const bool bside = blockIdx.y != 0;
    const int len = bside ? L.n : L.m, G = L.G, per = gram_part(len);
    const int c0 = (int)blockIdx.x * per, c1 = c0 + per < len ? c0 + per : len;
    if (c0 >= c1) return;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, n = lane & 15, kq = lane >> 4;
    const float* const* src = bside ? L.B_ptrs : L.A_ptrs;
    const float scale = 1.0f / (float)G;
    f64x4 acc[3];                                         // tiles (0, 0), (1, 0), (1, 1)
#pragma unroll
    for (int i = 0; i < 3; ++i) acc[i] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int base = c0; base < c1; base += 64) {
        if (!bside) {
            const int row = t >> 3, col = 4 * (t & 7);    // and row + 32
            f32x4 sum[2] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}, f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll 4
            for (int g = 0; g < G; ++g) {
                const float* p = gload(src + g);
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int r = base + row + 32 * e;
                    sum[e] += gload(reinterpret_cast<const f32x4*>(p + (int64_t)(r < c1 ? r : c0) * 32 + col));
                }
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int r = base + row + 32 * e;
                const f32x4 v = r < c1 ? sum[e] * scale : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                *reinterpret_cast<f32x4*>(X + (row + 32 * e) * PA + col) = v;
                if (r < c1) gstore(reinterpret_cast<f32x4*>(L.Abar + (int64_t)r * 32 + col), v);
            }
        } else {
            const int c = base + lane;
            float sum[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[e] = 0.0f;
#pragma unroll 4
            for (int g = 0; g < G; ++g) {
                const float* p = gload(src + g) + (c < c1 ? c : c0);
#pragma unroll
                for (int e = 0; e < 8; ++e) sum[e] += gload(p + (int64_t)(wave + 4 * e) * len);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = c < c1 ? sum[e] * scale : 0.0f;
                X[(wave + 4 * e) * PB + lane] = v;
                if (c < c1) gstore(L.Bbar + (int64_t)(wave + 4 * e) * len + c, v);
            }
        }
        __syncthreads();
        // each wave takes 16 of the 64 indices; operand lane l = X[index l / 16][column l % 16]
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int cc = 16 * wave + 4 * q + kq;
            const double x0 = bside ? X[n * PB + cc] : X[cc * PA + n], x1 = bside ? X[(16 + n) * PB + cc] : X[cc * PA + 16 + n];
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x0, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, x0, acc[1], 0, 0, 0);
            acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, x1, acc[2], 0, 0, 0);
        }
        __syncthreads();
    }
    // element (i, j) of a tile sits in lane (j, i % 4), register i / 4
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][i][(kq + 4 * v) * 16 + n] = acc[i][v];
    __syncthreads();
    double* out = L.gparts + ((int64_t)(bside ? kGramParts : 0) + blockIdx.x) * 1024;
    const int i = t >> 4, j = t & 15;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double s = ((red[0][k][t] + red[1][k][t]) + red[2][k][t]) + red[3][k][t];
        const int row = (k > 0 ? 16 : 0) + i, col = (k == 2 ? 16 : 0) + j;
        gstore(out + row * 32 + col, s);
        if (k == 1) gstore(out + col * 32 + row, s);
    }
}

__global__ __launch_bounds__(256) void core32_kernel(const LayerDev* __restrict__ layers) {
    __shared__ double F[2][32][33];                       // Gram matrices, then their Cholesky factors
    __shared__ double red[4];
    const LayerDev& L = layers[blockIdx.x];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int len = side ? L.n : L.m, per = gram_part(len), parts = (len + per - 1) / per;
        const double* p = L.gparts + (int64_t)side * kGramParts * 1024 + 4 * t;
        f64x2 s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
#pragma unroll 4
        for (int k = 0; k < parts; ++k) {
            s0 += gload(reinterpret_cast<const f64x2*>(p + k * 1024));
            s1 += gload(reinterpret_cast<const f64x2*>(p + k * 1024 + 2));
        }
        double* row = &F[side][t >> 3][4 * (t & 7)];
        row[0] = s0[0]; row[1] = s0[1]; row[2] = s1[0]; row[3] = s1[1];
        if (side) {
            gstore(reinterpret_cast<f64x2*>(L.GB + 4 * t), s0);
            gstore(reinterpret_cast<f64x2*>(L.GB + 4 * t + 2), s1);
        }
    }
    __syncthreads();
    if (wave < 2) {
        const int r = lane & 31;
        double mx = F[wave][r][r];
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
        double row[32];
#pragma unroll
        for (int c = 0; c < 32; ++c) row[c] = F[wave][r][c];
        factor_diagonal_block(row, r, mx * 1e-14, [](int, double) {});
        if (lane < 32) {
#pragma unroll
            for (int c = 0; c < 32; ++c) F[wave][r][c] = row[c];
        }
    }
    __syncthreads();
    const int i = t & 31;
    double ss = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = (t >> 5) + 8 * e;
        double c = 0.0;
#pragma unroll 8
        for (int k = 0; k < 32; ++k) c = fma(F[1][k][j], F[0][k][i], c);
        gstore(L.Ct + j * 32 + i, c);
        gstore(L.LA + j * 32 + i, F[0][j][i]);
        ss = fma(c, c, ss);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
    if (lane == 0) red[wave] = ss;
    __syncthreads();
    if (t < 8) gstore(L.trace + 2 + t, t == 0 ? ((red[0] + red[1]) + red[2]) + red[3] : 0.0);
}

__global__ __launch_bounds__(256) void finish32_kernel(const LayerDev* __restrict__ layers, int max_sweeps) {
    __shared__ double C[32][33], A[32][33], B[32][33], Y[32][33];
    __shared__ double key[32], s3[32], s5[32];
    __shared__ int perm[32];
    const LayerDev& L = layers[blockIdx.x];
    const int t = threadIdx.x, lane = t & 63, i = t & 31;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = (t >> 5) + 8 * e;
        C[j][i] = gload(L.Ct + j * 32 + i);
        A[j][i] = gload(L.LA + j * 32 + i);
        B[j][i] = gload(L.GB + j * 32 + i);
    }
    __syncthreads();
    if (t < 64) {                                         // one wave: lanes l and l + 32 do the same
        double ss = 0.0;
#pragma unroll 8
        for (int k = 0; k < 32; ++k) ss = fma(C[i][k], C[i][k], ss);
        // Bitonic sort, descending (ties: lower index first), by the comparisons of the sort for all sizes: it only exchanges entries, so that values
        // which compare false against any other (NaN) come out too, each once and in the same places as there.
        double mine = sqrt(ss);
        int from = i;
#pragma unroll
        for (int size = 2; size <= 32; size <<= 1)
#pragma unroll
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                const double other = __shfl_xor(mine, stride, 64);
                const int other_from = __shfl_xor(from, stride, 64);
                const bool low = (i & stride) == 0;       // the pair's lower place is this lane's
                const double klo = low ? mine : other, khi = low ? other : mine;
                const int ilo = low ? from : other_from, ihi = low ? other_from : from;
                const bool lo_first = klo > khi || (klo == khi && ilo < ihi);
                if (lo_first != ((i & size) == 0)) { mine = other; from = other_from; }
            }
        if (lane < 32) { key[i] = mine; perm[i] = from; }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // rank rule in fp32: keep sigma_i iff (float)sigma_i >= tau * (float)sigma_1
        const double top = key[0], sg = key[i];
        const float cut = L.tau * (float)top;
        const int count = __popcll(__ballot(lane < 32 && (float)sg >= cut));
        int kp = L.k_fixed > 0 ? L.k_fixed : (count < 1 ? 1 : count);
        if (kp > 32) kp = 32;
        if (kp > L.k_cap) kp = L.k_cap;
        const bool live = i < kp && sg > top * kSigmaFloor && sg > 0.0;
        const double rs = live ? 1.0 / sqrt(sg) : 0.0;    // sigma^(-1/2)
        if (lane < 32) { s3[i] = live ? rs / sg : 0.0; s5[i] = live ? rs / (sg * sg) : 0.0; }
        for (int k = lane; k < L.k_cap; k += 64) gstore(L.S_out + k, k < 32 ? (float)key[k] : 0.0f);
        if (lane == 0) {
            gstore(L.k_out, (int32_t)kp);
            int sweeps = max_sweeps, conv = 0;
            for (int s = 0; s < max_sweeps; ++s)
                if (gload(L.rotated + s) == 0) { sweeps = s + 1; conv = 1; break; }
            L.info[0] = sweeps; L.info[1] = 32; L.info[2] = conv; L.info[3] = kp;
        }
    }
    __syncthreads();
    const int kc = L.k_cap < 32 ? L.k_cap : 32;
    // Y[j] = L_A c_perm(j), PB = diag(s3) Y
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = (t >> 5) + 8 * e, from = perm[j];
        double y = 0.0;
#pragma unroll 8
        for (int k = 0; k < 32; ++k) y = fma(C[from][k], A[i][k], y);
        Y[j][i] = y;
        if (j < kc) gstore(L.PB + j * 32 + i, (float)(y * s3[j]));
    }
    __syncthreads();
    // PA = G_B Y^T diag(s5)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int r = (t >> 5) + 8 * e;
        double s = 0.0;
#pragma unroll 8
        for (int k = 0; k < 32; ++k) s = fma(B[r][k], Y[i][k], s);
        if (i < kc) gstore(L.PA + (int64_t)r * L.k_cap + i, (float)(s * s5[i]));
    }
}

}  // namespace

hipError_t launch_gram32(const LayerDev* layers, int L, hipStream_t s) {
    hipLaunchKernelGGL(gram32_kernel, dim3(kGramParts, 2, L), dim3(256), 0, s, layers);
    return hipGetLastError();
}
hipError_t launch_core32(const LayerDev* layers, int L, hipStream_t s) {
    hipLaunchKernelGGL(core32_kernel, dim3(L), dim3(256), 0, s, layers);
    return hipGetLastError();
}
hipError_t launch_finish32(const LayerDev* layers, int L, int max_sweeps, hipStream_t s) {
    hipLaunchKernelGGL(finish32_kernel, dim3(L), dim3(256), 0, s, layers, max_sweeps);
    return hipGetLastError();
}

}  // namespace abt
