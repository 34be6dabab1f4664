// The forward of a few rows at ranks up to 192 in one launch:  T[M,R] = X[M,p] . P[R,p]^T,  Y[M,q] = T[M,R] . Q[q,R]^T  (bf16, fp32 accumulators).
//
// Nothing but latency: a chain of a launch, the loads of the first product, its sum, the second product.  A work-group has 32 rows and 256 columns of Y
// (128 above r = 96, where LDS has room for four waves instead of eight) and makes the rows of T itself.  Its waves share the contraction, 32 columns
// at a time, each through two buffers of its own in LDS (whole 64-byte pieces, no barrier, the loads of two pieces on their way); their sums are
// added in the order of the waves, and each wave then makes 32 columns of Y, whose rows of Q have come meanwhile to where its buffers were.  The fused
// kernels walk through the contraction with a barrier per 64 columns, the two products add a launch.  197 rows, 768 -> 2304, us: r = 32 8.0 -> 4.1,
// r = 96 11.7 -> 5.9, r = 128 14.5 -> 6.6.  With the parts of a row block on eight XCDs,
// as they come, 3072 -> 768, r = 96, 788 rows took 13.6 instead of 10.1.
#include <atomic>
#include <type_traits>

#include "common.h"

namespace abt {

namespace {

__device__ __forceinline__ void lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int R>
struct FewCfg {
    static constexpr int RB = R / 32;
    static constexpr int NW = R <= 96 ? 8 : 4;            // waves, what LDS has room for
    static constexpr int NC = 32 * NW;                    // columns of Y
    static constexpr int NL = 2 + 2 * RB;                 // load instructions of a piece: 16 rows of 64 bytes each, X first
    static constexpr int piece = NL * 1024;
    static constexpr int qrows = 32 * R * 2;              // a wave's rows of Q
    static constexpr int sums = RB * 4096;                // a wave's part of the sums of T
    static constexpr int own = 2 * piece > qrows + sums ? 2 * piece : qrows + sums;
    static constexpr int pitch = R * 2 + 16;              // of T
    static constexpr int lds = NW * own + 32 * pitch;
    static_assert(lds <= 160 * 1024, "");
};

// GATHER: X is the patch matrix of a channels-last image of `bytes` bytes: column tap C + c of row (y, x) of the grid is channel c of the pixel
// (mul y + ky - kh / 2, mul x + kx - kw / 2), zero outside the image; a piece of 32 columns lies in one tap (C is a multiple of 64).
struct FewImage { int H, W, C, kh, kw, RH, RW, mul, bytes; };

struct FewPtrs { const uint16_t* X[kChainMaxGroups]; const uint16_t* P[kChainMaxGroups]; const uint16_t* Q[kChainMaxGroups]; uint16_t* Y[kChainMaxGroups]; uint16_t* T[kChainMaxGroups]; };

template <int R, bool GATHER>
__global__ __launch_bounds__(FewCfg<R>::NW * 64) void few_fwd_kernel(FewPtrs ptrs, int M, int p, int q, int parts,
                                                                     FewImage im) {
    using L = FewCfg<R>;
    constexpr int RB = L::RB, NL = L::NL, NW = L::NW;
    extern __shared__ __align__(1024) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lj = lane & 31, lh = lane >> 5;
    const uint16_t* const X = ptrs.X[blockIdx.y];
    const uint16_t* const P = ptrs.P[blockIdx.y];
    const uint16_t* const Q = ptrs.Q[blockIdx.y];
    uint16_t* const Y = ptrs.Y[blockIdx.y];
    uint16_t* const T = ptrs.T[blockIdx.y];
    // block b runs on XCD b % 8: each takes a contiguous eighth of the (rows, columns), so that the parts of a row block share X through one L2
    int part = blockIdx.x;
    {
        const int nb = gridDim.x, xcd = part & 7, i = part >> 3, per = nb >> 3, rem = nb & 7;
        part = xcd * per + (xcd < rem ? xcd : rem) + i;
    }
    const int64_t row0 = (int64_t)(part / parts) * 32;
    part %= parts;
    const int rows = M - row0 < 32 ? (int)(M - row0) : 32;
    // only the per-lane offset of an access is range-checked: rows past M arrive as zeros and are not stored
    const rsrc_t xr = GATHER ? make_rsrc(X, im.bytes) : make_rsrc(X + row0 * p, (int64_t)rows * p * 2), pr = make_rsrc(P, (int64_t)R * p * 2);
    unsigned char* const own = lds + wave * L::own;
    unsigned char* const tl = lds + NW * L::own;

    // ---- T, 32 columns of the contraction per piece.  Chunk c of row i of a piece lies at position c ^ ((i >> 2) & 3): sixteen
    // neighbouring rows, same chunk, in all of the 256 bytes of banks.
    const int lrow = lane >> 2, loff = (lrow * p + ((lane & 3) ^ ((lrow >> 2) & 3)) * 8) * 2, lstep = 16 * p * 2;
    const int np = p / 32, mine = wave < np ? (np - wave + NW - 1) / NW : 0;    // pieces wave, wave + NW, ..
    int cy[2], cx[2], pixel[2];                           // of the two rows of X this lane loads: the window's first pixel
#pragma unroll
    for (int j = 0; j < 2 && GATHER; ++j) {
        const int per = im.RH * im.RW, g = (int)row0 + lrow + 16 * j, img = g / per, rem = g - img * per, y = rem / im.RW;
        cy[j] = lrow + 16 * j < rows ? im.mul * y - im.kh / 2 : -0x10000000;     // rows past M: never inside
        cx[j] = im.mul * (rem - y * im.RW) - im.kw / 2;
        pixel[j] = (img * im.H + im.mul * y - im.kh / 2) * im.W + cx[j];
    }
    auto issue = [&](int i) {
        unsigned char* dst = own + (i & 1) * L::piece;
        const int at = (wave + NW * i) * 64;
        if constexpr (GATHER) {
            const int tap = at / (2 * im.C), ky = tap / im.kw, kx = tap - ky * im.kw;
            const int chan = at / 2 - tap * im.C + ((lane & 3) ^ ((lrow >> 2) & 3)) * 8;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const bool in = (unsigned)(cy[j] + ky) < (unsigned)im.H && (unsigned)(cx[j] + kx) < (unsigned)im.W;
                load_lds16(xr, dst + j * 1024, in ? ((pixel[j] + ky * im.W + kx) * im.C + chan) * 2 : kBufNowhere, 0);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) load_lds16(xr, dst + j * 1024, loff + j * lstep + at, 0);
        }
#pragma unroll
        for (int j = 0; j < 2 * RB; ++j) load_lds16(pr, dst + (2 + j) * 1024, loff + j * lstep + at, 0);
    };
    f32x16 acc[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.0f;
    if (mine > 0) issue(0);
    if (mine > 1) issue(1);
    const int prow = out_row(lj);
    for (int i = 0; i < mine; ++i) {
        if (i + 1 < mine) wait_newest<NL>();              // piece i + 1 may still be on its way
        else wait_newest<0>();
        const unsigned char* const b = own + (i & 1) * L::piece;
        u32x4 x[2], f[2][RB];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int c = 2 * j + lh;
            x[j] = *reinterpret_cast<const u32x4*>(b + lj * 64 + ((c ^ ((lj >> 2) & 3)) * 16));
#pragma unroll
            for (int k = 0; k < RB; ++k) f[j][k] = *reinterpret_cast<const u32x4*>(b + 2048 + (32 * k + prow) * 64 + ((c ^ ((prow >> 2) & 3)) * 16));
        }
        lds_done();                                       // read: the buffer may be filled again
        __builtin_amdgcn_sched_barrier(0);
        if (i + 2 < mine) issue(i + 2);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int k = 0; k < RB; ++k) acc[k] = mfma_bf16(f[j][k], x[j], acc[k]);
    }
    // ---- this wave's rows of Q on their way, its sums to LDS behind them (its buffers are read)
    const int col0 = part * L::NC + 32 * wave;
    const bool have = Y != nullptr && col0 < q;
    if (have) {
        const rsrc_t qr = make_rsrc(Q + (int64_t)col0 * R, L::qrows);
#pragma unroll
        for (int j = 0; j < 2 * RB; ++j) load_lds16(qr, own + j * 1024, j * 1024 + lane * 16, 0);
    }
    float* const sums = reinterpret_cast<float*>(own + L::qrows);
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            *reinterpret_cast<f32x4*>(sums + ((b * 4 + v) * 64 + lane) * 4) = f32x4{acc[b][4 * v], acc[b][4 * v + 1], acc[b][4 * v + 2], acc[b][4 * v + 3]};
    lds_barrier();
    for (int i = threadIdx.x; i < RB * 256; i += 64 * NW) {   // four columns of a row of T: lane's row, columns 16 (lane / 32) + 4 v of block b
        f32x4 s = *reinterpret_cast<const f32x4*>(lds + L::qrows + i * 16);
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *reinterpret_cast<const f32x4*>(lds + w * L::own + L::qrows + i * 16);
        const int l = i & 63, v = (i >> 6) & 3, b = i >> 8;
        uint32_t* d = reinterpret_cast<uint32_t*>(tl + (l & 31) * L::pitch + (32 * b + 16 * (l >> 5) + 4 * v) * 2);
        d[0] = pack2_bf16(s[0], s[1]);
        d[1] = pack2_bf16(s[2], s[3]);
    }
    lds_barrier();
    if (have) {                                           // ---- 32 columns of Y
        wait_newest<0>();
        f32x16 y;
#pragma unroll
        for (int v = 0; v < 16; ++v) y[v] = 0.0f;
#pragma unroll
        for (int k = 0; k < R / 16; ++k) {
            const u32x4 a = *reinterpret_cast<const u32x4*>(own + prow * (R * 2) + (2 * k + lh) * 16);
            const u32x4 t = *reinterpret_cast<const u32x4*>(tl + lj * L::pitch + (2 * k + lh) * 16);
            y = mfma_bf16(a, t, y);
        }
        const rsrc_t yr = make_rsrc(Y + row0 * q + col0, ((int64_t)(rows - 1) * q + 32) * 2);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = pack2_bf16(y[8 * h + 2 * i], y[8 * h + 2 * i + 1]);
            buf_store16(v, yr, lj < rows ? (lj * q + 16 * lh + 8 * h) * 2 : kBufNowhere, 0);
        }
    }
    if (T != nullptr && part == 0) {
        constexpr int CPR = R / 8;
        const rsrc_t tr = make_rsrc(T + row0 * R, (int64_t)rows * R * 2);
        for (int i = threadIdx.x; i < 32 * CPR; i += 64 * NW) {
            const int row = i / CPR, c = i - row * CPR;
            buf_store16(*reinterpret_cast<const u32x4*>(tl + row * L::pitch + c * 16), tr, (row * R + c * 8) * 2, 0);
        }
    }
}

template <int R, bool GATHER>
hipError_t launch_few_r(const FewPtrs& c, int G, int M, int p, int q, const FewImage& im, hipStream_t s) {
    using L = FewCfg<R>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&few_fwd_kernel<R, GATHER>), hipFuncAttributeMaxDynamicSharedMemorySize, L::lds);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const int parts = c.Y[0] ? (q + L::NC - 1) / L::NC : 1;
    hipLaunchKernelGGL((few_fwd_kernel<R, GATHER>), dim3((unsigned)(parts * ((M + 31) / 32)), (unsigned)G), dim3(64 * L::NW), L::lds, s, c, M, p, q, parts, im);
    return hipGetLastError();
}

template <bool GATHER>
hipError_t launch_few(const ChainProblem* problems, int G, int M, int p, int q, int R, const FewImage& im, hipStream_t s) {
    if (G < 1 || G > kChainMaxGroups) return hipErrorInvalidValue;
    FewPtrs c{};
    for (int g = 0; g < G; ++g) {
        const ChainProblem& f = problems[g];
        if ((!f.Yout && !f.Tout) || (f.Yout != nullptr) != (problems[0].Yout != nullptr)) return hipErrorInvalidValue;
        c.X[g] = (const uint16_t*)f.Xin; c.P[g] = (const uint16_t*)f.P; c.Q[g] = (const uint16_t*)f.Q;
        c.Y[g] = (uint16_t*)f.Yout; c.T[g] = (uint16_t*)f.Tout;
    }
    switch (R / 32) {
        case 1: return launch_few_r<32, GATHER>(c, G, M, p, q, im, s);
        case 2: return launch_few_r<64, GATHER>(c, G, M, p, q, im, s);
        case 3: return launch_few_r<96, GATHER>(c, G, M, p, q, im, s);
        case 4: return launch_few_r<128, GATHER>(c, G, M, p, q, im, s);
        case 5: return launch_few_r<160, GATHER>(c, G, M, p, q, im, s);
        case 6: return launch_few_r<192, GATHER>(c, G, M, p, q, im, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool few_supports(int64_t M, int p, int q, int R) {
    return M >= 1 && M <= 8192 && p % 64 == 0 && q % 64 == 0 && p >= 64 && q >= 64 && p <= (1 << 20) && q <= (1 << 20) && R % 32 == 0 && R >= 32 && R <= 192;
}

hipError_t launch_few_fwd(const ChainProblem* problems, int G, int64_t M, int p, int q, int R, hipStream_t s) {
    if (!few_supports(M, p, q, R)) return hipErrorInvalidValue;
    return launch_few<false>(problems, G, (int)M, p, q, R, FewImage{}, s);
}

bool few_gather_supports(const PatchGeom& g, int64_t M, int q, int R) {
    const int64_t per = (int64_t)g.RH * g.RW;
    if (g.sign != 1 || g.shift != 0 || g.Cin % 64 || per < 1 || M % per != 0 || (int64_t)g.kh * g.kw * g.Cin > (1 << 20)) return false;
    return (M / per) * g.H * g.W * g.Cin * 2 < kBufMaxBytes && few_supports(M, g.kh * g.kw * g.Cin, q, R);
}

hipError_t launch_few_fwd_gather(const ChainProblem& c, const PatchGeom& g, int64_t M, int q, int R, hipStream_t s) {
    if (!few_gather_supports(g, M, q, R)) return hipErrorInvalidValue;
    const FewImage im{g.H, g.W, g.Cin, g.kh, g.kw, g.RH, g.RW, g.mul, (int)((M / ((int64_t)g.RH * g.RW)) * g.H * g.W * g.Cin * 2)};
    return launch_few<true>(&c, 1, (int)M, g.kh * g.kw * g.Cin, q, R, im, s);
}

}  // namespace abt
