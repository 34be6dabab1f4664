// Layout helpers of the bf16 factored layer: transposed factors (backward of many rows: dT = dY A and dX = dT B are the forward chain on
// them) and the re-laid-out factor of a convolution's activation gradient.
#include "common.h"

namespace abt {

namespace {

// =====================================================================================
// bf16 transpose (for A^T and B^T, which turn dT = dY A and dX = dT B into the same
// "rows times rows" shape the chain kernel consumes).
// =====================================================================================
// One launch serves up to kTransposeMaxJobs matrices (rows and cols multiples of 8).  A work-group moves one
// 64 x 64 tile: 16-byte loads of row pieces into LDS, 16-byte stores of column pieces out of it.
struct TrJob { const uint16_t* src; uint16_t* dst; int rows, cols, tiles_x, tile_begin; };
struct TrArgs { TrJob job[kTransposeMaxJobs]; int njobs; };

__device__ __forceinline__ void transpose_tile(const TrJob& j, int t) {
    __shared__ uint16_t tile[64][72];                  // pitch 144 B: 16-byte aligned rows
    const int r0 = (t / j.tiles_x) * 64, c0 = (t % j.tiles_x) * 64;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int ci = e * 256 + threadIdx.x;          // 64 rows x 8 chunks of 8 elements
        const int row = ci >> 3, ch = ci & 7;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (r0 + row < j.rows && c0 + ch * 8 < j.cols)
            v = *reinterpret_cast<const u32x4*>(j.src + (int64_t)(r0 + row) * j.cols + c0 + ch * 8);
        *reinterpret_cast<u32x4*>(&tile[row][ch * 8]) = v;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int ci = e * 256 + threadIdx.x;          // 64 output rows (source columns) x 8 chunks
        const int orow = ci >> 3, ch = ci & 7;
        if (c0 + orow < j.cols && r0 + ch * 8 < j.rows) {
            uint16_t v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = tile[ch * 8 + i][orow];
            u32x4 o = {(uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16),
                       (uint32_t)v[4] | ((uint32_t)v[5] << 16), (uint32_t)v[6] | ((uint32_t)v[7] << 16)};
            *reinterpret_cast<u32x4*>(j.dst + (int64_t)(c0 + orow) * j.rows + r0 + ch * 8) = o;
        }
    }
}

__global__ __launch_bounds__(256) void transpose_bf16_kernel(TrArgs args) {
    int jid = 0;
    for (int i = 1; i < args.njobs; ++i)
        if ((int)blockIdx.x >= args.job[i].tile_begin) jid = i;
    transpose_tile(args.job[jid], (int)blockIdx.x - args.job[jid].tile_begin);
}

// Re-layout of the factor B [r, taps C] of a factored convolution for the activation gradient:
// Pst [C, taps r_pad] with Pst[c, tap r_pad + j] = B[j, tap C + c] for j < r and 0 for r <= j < r_pad
// (every tap padded to a multiple of 64 columns, the slab width of the chain kernel).  One thread
// writes eight consecutive j (16 bytes).
struct BstackArgs { const uint16_t* B; uint16_t* Pst; int r, C, kh, kw, r_pad, by_parity; };
__device__ __forceinline__ void bstack_piece(const BstackArgs& a, int block) {
    const uint16_t* __restrict__ const B = a.B;
    uint16_t* __restrict__ const Pst = a.Pst;
    const int r = a.r, C = a.C, kh = a.kh, kw = a.kw, r_pad = a.r_pad, by_parity = a.by_parity;
    const int taps = kh * kw;
    const int per_row = taps * (r_pad / 8);
    const int64_t idx = (int64_t)block * 256 + threadIdx.x;
    if (idx >= (int64_t)C * per_row) return;
    const int c = (int)(idx / per_row), rest = (int)(idx % per_row);
    const int tap = rest / (r_pad / 8), j0 = (rest % (r_pad / 8)) * 8;
    uint16_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = j0 + i < r ? B[(int64_t)(j0 + i) * taps * C + (int64_t)tap * C + c] : (uint16_t)0;
    u32x4 o = {(uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16),
               (uint32_t)v[4] | ((uint32_t)v[5] << 16), (uint32_t)v[6] | ((uint32_t)v[7] << 16)};
    int64_t dst = (int64_t)c * taps * r_pad + (int64_t)tap * r_pad;
    if (by_parity) {
        // the parity this tap belongs to, the taps of the parities before it, its place among its own
        const int ky = tap / kw, kx = tap - ky * kw, py = (ky + kh / 2) & 1, px = (kx + kw / 2) & 1;
        const int ny0 = parity_count(kh, 0), nx0 = parity_count(kw, 0), ny = py ? kh - ny0 : ny0, nx = px ? kw - nx0 : nx0;
        const int before = (py ? ny0 * kw : 0) + (px ? ny * nx0 : 0);
        const int place = ((ky - parity_first(kh, py)) >> 1) * nx + ((kx - parity_first(kw, px)) >> 1);
        dst = ((int64_t)before * C + (int64_t)c * ny * nx + place) * r_pad;
    }
    *reinterpret_cast<u32x4*>(Pst + dst + j0) = o;
}

// A^T and the re-laid-out B of a convolution's backward together: a launch costs more than either (3.6 us each)
__global__ __launch_bounds__(256) void conv_factors_kernel(TrJob j, int tiles, BstackArgs a) {
    if ((int)blockIdx.x < tiles) transpose_tile(j, (int)blockIdx.x);
    else bstack_piece(a, (int)blockIdx.x - tiles);
}

}  // namespace

hipError_t launch_conv_factors_bf16(const void* A, void* At, int m, const void* B, void* Pst, int r, int C, int kh, int kw, int r_pad, bool by_parity,
                                    hipStream_t s) {
    if (r < 1 || C < 1 || kh < 1 || kw < 1 || r_pad % 64 || r_pad < r || m % 8 || r % 8) return hipErrorInvalidValue;
    const TrJob j{(const uint16_t*)A, (uint16_t*)At, m, r, (r + 63) / 64, 0};
    const int tiles = A ? j.tiles_x * ((m + 63) / 64) : 0;
    const BstackArgs a{(const uint16_t*)B, (uint16_t*)Pst, r, C, kh, kw, r_pad, by_parity ? 1 : 0};
    const int64_t pieces = B ? ceil_div((int64_t)C * kh * kw * (r_pad / 8), 256) : 0;
    if (tiles + pieces == 0) return hipSuccess;
    hipLaunchKernelGGL(conv_factors_kernel, dim3((unsigned)(tiles + pieces)), dim3(256), 0, s, j, tiles, a);
    return hipGetLastError();
}

hipError_t launch_transpose_bf16(const TransposeJob* jobs, int njobs, hipStream_t s) {
    if (njobs < 1 || njobs > kTransposeMaxJobs) return hipErrorInvalidValue;
    TrArgs args{};
    args.njobs = njobs;
    int tiles = 0;
    for (int i = 0; i < njobs; ++i) {
        if (jobs[i].rows % 8 || jobs[i].cols % 8) return hipErrorInvalidValue;
        const int tx = (jobs[i].cols + 63) / 64, ty = (jobs[i].rows + 63) / 64;
        args.job[i] = TrJob{(const uint16_t*)jobs[i].src, (uint16_t*)jobs[i].dst, jobs[i].rows, jobs[i].cols, tx, tiles};
        tiles += tx * ty;
    }
    hipLaunchKernelGGL(transpose_bf16_kernel, dim3(tiles), dim3(256), 0, s, args);
    return hipGetLastError();
}

}  // namespace abt
