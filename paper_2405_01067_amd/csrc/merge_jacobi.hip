// Block form of the one-sided Jacobi iteration on the K x K core of the merge (the truncated SVD
// of Eq. 3 on the merged matrix), for K <= 768, on the fp64 matrix cores.
//
// The columns of C (rows of Ct) are grouped in blocks of 16; a round pairs every block with one
// partner (round-robin tournament over the blocks), one work-group per block pair.  For its 32
// columns P (K x 32) a work-group
//   1. forms the Gram matrix S = P^T P (32 x 32) with v_mfma_f64_16x16x4: the 16 x 16 tile between the blocks; the
//      tiles inside them are what the last round's rotations left of S, and formed anew in round 0 of a sweep only,
//   2. runs the cyclic Jacobi eigenvalue iteration on S: 16 steps of 16 disjoint rotations, every rotation applied to S
//      from both sides and accumulated in Q (32 x 32).  These are the plane rotations the column form of the
//      method would apply to the 256 column pairs of the two blocks, in the same order; they are
//      worked out on the 32 x 32 Gram matrix instead of on K-long columns,
//   3. applies them at once: P <- P Q, again on the matrix cores.
// Round 0 of a sweep first rotates the pairs inside each of the two blocks the same way (15 steps).
//
// The panel lives in registers from load to store, in the operand layout of step 3: a lane holds
// the rows r = l % 16 of its wave's row tiles and the columns l / 16 + 4 s (s = 0..7); with the
// product taken as (Q^T P^T) the result tile comes out of the matrix core in that same layout, so
// the update is in place.  Step 1 needs the transposed operand order (contraction over rows); each
// wave passes its row tiles through a private 4 KB LDS tile for that.
//
// What bounds it: a round is one dependent chain.  K = 384, cycles of a work-group: panel load 3400 alone, 7000 to 10000 with 576
// of them (nothing survives in L2 from the round before), Gram matrix 3000 (6500 with the tiles inside the blocks), rotations 14000 of which Q
// 2000, update 6400 (fp64 matrix instructions), store 2000, and some 10000 between the end of a round and the start of
// the next.  Sweeps of config 5 (48 cores of 384, 8 sweeps): 6.07 ms before the rotations moved to registers, 4.97 after,
// 4.60 with the kept diagonal tiles; 16 cores of 768, 9 sweeps: 17.5, 16.7, 16.2 ms (one work-group per compute unit, 384 of them).
#include <type_traits>

#include "merge_internal.h"

namespace abt {

namespace {

// swizzled address (in doubles) of element (row n, column c) of a 16 x 32 staging tile: stores of one
// column by 16 rows and loads of 16 consecutive columns of one row both spread over all banks
__device__ __forceinline__ int stage_addr(int n, int c) {
    return 32 * n + ((c + 16 * (n & 1) + 2 * (n >> 1)) & 31);
}

struct __align__(16) JacobiShared {
    double stage[4][16 * 32];       // per wave: transposition tile; afterwards the waves' partial Gram tiles
    double Q[32][48];
    float S[32][33];                // the Gram matrix times a power of two
    int flags;                      // of a round: 1 rotated anything, 2 anything significant
    float tan[2][31][16];           // tangents of the rotations of all steps (second half: what other lanes than the pairs' own come to)
};

// ---- The rotations of a block pair.  Columns 0..31 (the two blocks) are paired by exclusive or: step m pairs every i with
// i ^ m, so 31 steps meet all pairs once, m = 16..31 those between the blocks, m < 16 those inside them.  The
// steps whose m has p as its highest bit form level p: with L(u), R(u) = the 4-bit u with a 0 or a 1 put in at bit p, step t pairs L(u)
// with R(u ^ t), t below 2^p.
__device__ __forceinline__ int left_of(int u, int p) { return ((u >> p) << (p + 1)) | (u & ((1 << p) - 1)); }
__device__ __forceinline__ int right_of(int u, int p) { return left_of(u, p) | (1 << p); }

__device__ __forceinline__ void lds_barrier() {    // leaves stores to memory on their way
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// cosine and sine of a tangent to fp64 rounding (hardware reciprocal square root, two Newton steps)
__device__ __forceinline__ f64x2 cosine_sine(float tangent) {
    const double t = (double)tangent, w = fma(t, t, 1.0);
    double y = __builtin_amdgcn_rsq(w);
    y = y * fma(-0.5 * w, y * y, 1.5);
    y = y * fma(-0.5 * w, y * y, 1.5);
    return f64x2{y, y * t};
}

template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); static_for<N, F, I + 1>(static_cast<F&&>(f)); }
}

template <int CTRL>
__device__ __forceinline__ int dpp(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_rows(int old, int v) { return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false); }
// the value of lane ^ B (B = 1, 2, 3, 4, 8) by data-parallel moves: quad permutations, mirrored half rows, rotated rows
template <int B>
__device__ __forceinline__ int lane_xor(int v) {
    if constexpr (B == 1) return dpp<0xB1>(v);
    else if constexpr (B == 2) return dpp<0x4E>(v);
    else if constexpr (B == 3) return dpp<0x1B>(v);
    else if constexpr (B == 4) return dpp<0x1B>(dpp<0x141>(v));
    else return dpp<0x128>(v);
}
template <int B>
__device__ __forceinline__ float lane_xor(float v) { return __int_as_float(lane_xor<B>(__float_as_int(v))); }
template <int B>
__device__ __forceinline__ double lane_xor(double v) {
    return __hiloint2double(lane_xor<B>(__double2hiint(v)), lane_xor<B>(__double2loint(v)));
}
// the value of lane ^ 16 or ^ 32: whole rows of 16 lanes change places
template <int B>
__device__ __forceinline__ float row_xor(float v) {
    const unsigned x = __float_as_uint(v);
    if constexpr (B == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);      // r[0]: even rows twice, r[1]: odd rows twice
        return __uint_as_float((threadIdx.x & 16) ? r[0] : r[1]);
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
    }
}
// lanes 0..15 to all four rows
__device__ __forceinline__ float first_row(float v) {
    const unsigned x = __float_as_uint(v);
    const unsigned lo = __builtin_amdgcn_permlane32_swap(x, x, false, false)[0];
    return __uint_as_float(__builtin_amdgcn_permlane16_swap(lo, lo, false, false)[0]);
}
// of a value that all rows hold alike: lane u ^ 4 q of it for lane (u, q)
__device__ __forceinline__ float xor_by_row(float v) {
    int x = __float_as_int(v);
    x = dpp_rows<0x128, 0xc>(x, x);                           // rows 2, 3: lanes 8 apart
    const int w = dpp_rows<0x141, 0xa>(x, x);                 // rows 1, 3: lanes 4 apart, in two moves
    return __int_as_float(dpp_rows<0x1B, 0xa>(w, w));
}

// Level p on S by one wave, S in registers in fp32: lane (u = l % 16, q = l / 16) owns, for x = 4 q + e, the 2 x 2 cell rows
// L(u), R(u ^ t) x columns L(v), R(v ^ t) with v = u ^ x.  t runs through a Gray code; when bit b of it changes, a cell finds its new
// off-diagonal entries in the cell x ^ b (another register of the lane for b = 1, 2) and its new last
// entry, like the one below the diagonal, in lane ^ b: register names and data-parallel moves, no LDS and no barrier
// in a step.  The pairs' own cells are x = 0, in the first 16 lanes, which work the tangents out; these go to the other lanes by row
// swaps and row-masked moves.
// The tangent is that of jacobi_rotation(), without branches.  Any tangent gives a rotation that is orthogonal to fp64 rounding, as
// the work-group forms cosine and sine from it in fp64 afterwards; one good to 1e-7 leaves the pair with 1e-7 of its cosine.  S is
// scaled by a power of two near 1 / ||C||_F^2: squared norms lie between kZeroColumn2 and 1, inner products of a pair that is
// rotated above 1e-9 of that, inside the fp32 range (their squares are not: the cosine is formed from two reciprocal square roots).
// fp32 is enough for S: the columns themselves, the rotations and their product Q stay in fp64, and what 1e-7 of a cosine leaves is seen
// by the next sweep, which forms S anew; the sweeps are as many (simulated for cores of 128 to 768, measured on those of the case table).
// The steps are serial, so the chain through the pairs' own cells sets the pace, and the issue of the other cells' updates comes next: a
// step updates the cells that the next tangent needs first and the others between the links of its formula.
// A cell is multiplied by (1, -t; t, 1) from both sides and by the product of the cosines.
// A step took 790 cycles in fp64 with lane permutes, 720 in fp32 with all cells ahead of the formula.
template <int P>
__device__ __forceinline__ void rotate_level(float (*S)[33], float* tangents, float floor2, bool& any, bool& any_signif, int* flags = nullptr,
                                             double unscale = 1.0, double* diagI = nullptr, double* diagJ = nullptr) {
    const int lane = threadIdx.x & 63, u = lane & 15, q = lane >> 4;
    float* const mine = tangents + u + (q ? 31 * 16 : 0);
    float m00[4], m01[4], m10[4], m11[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int v = u ^ (4 * q + e);
        m00[e] = S[left_of(u, P)][left_of(v, P)]; m01[e] = S[left_of(u, P)][right_of(v, P)];
        m10[e] = S[right_of(u, P)][left_of(v, P)]; m11[e] = S[right_of(u, P)][right_of(v, P)];
    }
    // the tangent of the pair with squared norms alpha, beta and inner product gamma, in three links
    float zeta, w, ra, rb, rg, own;
    auto link1 = [&](float alpha, float beta, float gamma) {
        rg = __builtin_amdgcn_rcpf(gamma + gamma);
        ra = __builtin_amdgcn_rsqf(alpha); rb = __builtin_amdgcn_rsqf(beta);
        zeta = beta - alpha;
    };
    auto link2 = [&]() {
        zeta *= rg;                                      // an overflow of its square ends in t = 0 (|t| < 1e-19)
        w = __builtin_amdgcn_sqrtf(fmaf(zeta, zeta, 1.0f));
    };
    auto link3 = [&](float alpha, float beta, float gamma) {
        const float cosine = fabsf(gamma) * ra * rb;
        const bool live = alpha > floor2 && beta > floor2;
        any_signif |= live && cosine > (float)kSignifTol;                  // (this and the next count in the first 16 lanes)
        any |= live && cosine > (float)kRotateTol;
        const float ta = __builtin_amdgcn_rcpf(fabsf(zeta) + w);
        own = live && cosine > (float)kRotateTol ? copysignf(ta, zeta) : 0.0f;
    };
    link1(m00[0], m11[0], m01[0]); link2(); link3(m00[0], m11[0], m01[0]);
    // one step; B: the bit of t that changes after it (0: the last step)
    auto step = [&](auto bit, int k) {
        constexpr int B = decltype(bit)::value;
        constexpr int E1 = B == 2 ? 2 : 1, E2 = B == 2 ? 1 : 2;            // the second cell to be updated, the third
        mine[16 * k] = own;
        const float t = first_row(own);
        float t2[4], c12[4];
        t2[0] = xor_by_row(t);
        const float c1 = __builtin_amdgcn_rsqf(fmaf(t, t, 1.0f));
        const float c2 = xor_by_row(c1);
        t2[1] = lane_xor<1>(t2[0]); t2[2] = lane_xor<2>(t2[0]); t2[3] = lane_xor<3>(t2[0]);
        c12[0] = c1 * c2; c12[1] = c1 * lane_xor<1>(c2); c12[2] = c1 * lane_xor<2>(c2); c12[3] = c1 * lane_xor<3>(c2);
        float n01[4], n10[4], n11[4];
        auto update = [&](auto which) {
            constexpr int e = decltype(which)::value;
            const float a = fmaf(-t, m10[e], m00[e]), b = fmaf(-t, m11[e], m01[e]), c = fmaf(t, m00[e], m10[e]), d = fmaf(t, m01[e], m11[e]);
            m00[e] = fmaf(-t2[e], b, a) * c12[e]; n01[e] = fmaf(t2[e], a, b) * c12[e];
            n10[e] = fmaf(-t2[e], d, c) * c12[e]; n11[e] = fmaf(t2[e], c, d) * c12[e];
        };
        update(std::integral_constant<int, 0>{});
        if constexpr (B == 1 || B == 2) update(std::integral_constant<int, E1>{});
        float beta = 0.0f, gamma = 0.0f;
        if constexpr (B != 0) {
            beta = lane_xor<B>(n11[0]);
            if constexpr (B < 4) gamma = n01[E1];
            else gamma = row_xor<4 * B>(n01[0]);
            link1(m00[0], beta, gamma);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (B != 1 && B != 2) update(std::integral_constant<int, E1>{});
        update(std::integral_constant<int, E2>{});
        if constexpr (B != 0) link2();
        __builtin_amdgcn_sched_barrier(0);
        update(std::integral_constant<int, 3>{});
        if constexpr (B != 0) link3(m00[0], beta, gamma);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (B == 0) { m01[e] = n01[e]; m10[e] = n10[e]; m11[e] = n11[e]; }
            else if constexpr (B < 4) { m01[e] = n01[e ^ B]; m10[e] = lane_xor<B>(n10[e ^ B]); m11[e] = lane_xor<B>(n11[e]); }
            else { m01[e] = row_xor<4 * B>(n01[e]); m10[e] = row_xor<4 * B>(lane_xor<B>(n10[e])); m11[e] = lane_xor<B>(n11[e]); }
        }
    };
    static_for<(1 << P)>([&](auto i) {
        constexpr int k = decltype(i)::value;
        if constexpr (P == 4 && k == 8) lds_barrier();   // the first eight tangents: the other waves begin with Q
        step(std::integral_constant<int, (k + 1 < (1 << P) ? (k + 1) & -(k + 1) : 0)>{}, k);
    });
    constexpr int t = ((1 << P) - 1) ^ (((1 << P) - 1) >> 1);
    if constexpr (P == 4) {                              // the last level: the two diagonal blocks, for the next round
        const bool r = __builtin_amdgcn_ballot_w64(any && lane < 16) != 0, sg = __builtin_amdgcn_ballot_w64(any_signif && lane < 16) != 0;
        if (lane == 0) *flags = (r ? 1 : 0) | (sg ? 2 : 0);
        lds_barrier();
        if (diagI == nullptr) return;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int v = u ^ (4 * q + e);
            gstore(diagI + 16 * u + v, (double)m00[e] * unscale);
            gstore(diagJ + 16 * (u ^ t) + (v ^ t), (double)m11[e] * unscale);
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int v = u ^ (4 * q + e);
        S[left_of(u, P)][left_of(v, P)] = m00[e]; S[left_of(u, P)][right_of(v ^ t, P)] = m01[e];
        S[right_of(u ^ t, P)][left_of(v, P)] = m10[e]; S[right_of(u ^ t, P)][right_of(v ^ t, P)] = m11[e];
    }
    wave_lds_fence();
}

// The rotations on the columns of Q, by the three waves that do not work them out (w = 0..2): rows 12 w .. 12 w + 11, lane (u, q) owning
// rows q, q + 4 and q + 8 of them (up to row 31).
// A level inside the blocks: columns L(u), R(u ^ t).
template <int P>
__device__ __forceinline__ void accumulate_level(double (*Q)[48], const f64x2* table, int w) {
    const int lane = threadIdx.x & 63, u = lane & 15, r = 12 * w + (lane >> 4);
    double a[3], b[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) { a[i] = Q[(r + 4 * i) & 31][left_of(u, P)]; b[i] = Q[(r + 4 * i) & 31][right_of(u, P)]; }
    static_for<(1 << P)>([&](auto which) {
        constexpr int k = decltype(which)::value, B = k + 1 < (1 << P) ? (k + 1) & -(k + 1) : 0;
        const f64x2 rot = table[16 * k + u];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double x = rot[0] * a[j] - rot[1] * b[j], y = rot[1] * a[j] + rot[0] * b[j];
            a[j] = x;
            if constexpr (B == 0) b[j] = y;
            else b[j] = lane_xor<B>(y);
        }
    });
    constexpr int t = ((1 << P) - 1) ^ (((1 << P) - 1) >> 1);
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (r + 4 * i < 32) { Q[r + 4 * i][left_of(u, P)] = a[i]; Q[r + 4 * i][right_of(u ^ t, P)] = b[i]; }
    wave_lds_fence();
}
// All levels inside the blocks, on the identity, once their tangents are there
__device__ __forceinline__ void accumulate_inside(double (*Q)[48], const float (*tangents)[16], f64x2* table, int w) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int row = 12 * w + 2 * i + (lane >> 5), col = lane & 31;
        if (row < 32) Q[row][col] = row == col ? 1.0 : 0.0;
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 4 * i + (lane >> 4);
        if (k < 15) table[64 * i + lane] = cosine_sine(tangents[16 + k][lane & 15]);
    }
    wave_lds_fence();
    accumulate_level<3>(Q, table, w);
    accumulate_level<2>(Q, table + 16 * 8, w);
    accumulate_level<1>(Q, table + 16 * 12, w);
    accumulate_level<0>(Q, table + 16 * 14, w);
}

// The rotations between the blocks: columns u and 16 + (u ^ t).  The tangents come in two halves; each wave makes a table of its own of
// their cosines and sines.  FRESH: Q is the identity so far.
template <bool FRESH>
__device__ __forceinline__ void accumulate_cross(double (*Q)[48], const float (*tangents)[16], f64x2* table, int w) {
    const int lane = threadIdx.x & 63, u = lane & 15, r = 12 * w + (lane >> 4);
    double a[3], b[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int row = r + 4 * i;
        if (FRESH) { a[i] = row == u ? 1.0 : 0.0; b[i] = row == u + 16 ? 1.0 : 0.0; }
        else { a[i] = Q[row & 31][u]; b[i] = Q[row & 31][u + 16]; }
    }
    static_for<2>([&](auto half) {
        constexpr int H = decltype(half)::value;
        lds_barrier();
        table[lane] = cosine_sine(tangents[8 * H + (lane >> 4)][u]);
        table[64 + lane] = cosine_sine(tangents[8 * H + 4 + (lane >> 4)][u]);
        wave_lds_fence();
        static_for<8>([&](auto i) {
            constexpr int k = 8 * H + decltype(i)::value, B = k + 1 < 16 ? (k + 1) & -(k + 1) : 0;
            const f64x2 rot = table[16 * (k & 7) + u];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double x = rot[0] * a[j] - rot[1] * b[j], y = rot[1] * a[j] + rot[0] * b[j];
                a[j] = x;
                if constexpr (B == 0) b[j] = y;
                else b[j] = lane_xor<B>(y);
            }
        });
        wave_lds_fence();
    });
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (r + 4 * i < 32) { Q[r + 4 * i][u] = a[i]; Q[r + 4 * i][16 + (u ^ 8)] = b[i]; }
}

// NT: 16-row tiles per wave (two per 32-row chunk: its even and its odd rows), K <= 64 NT.
// (Three work-groups per compute unit at K = 384 spill and take 7.0 ms in place of 4.6 over a merge; two at K = 768, 24.7 of 16.2.)
// WHOLE (K = 32: two blocks, one pair): the work-group holds the whole core, so it runs all sweeps in one launch, the
// panel in registers throughout; `round` is the sweep cap.  A launch and a poll of the convergence flags per
// sweep took 129 us for one core of 32, this 54.
template <int NT, bool WHOLE>
__global__ __launch_bounds__(256, (WHOLE ? 1 : NT <= 2 ? 3 : NT <= 6 ? 2 : 1))
void jacobi_block_kernel(double* cores, int* rotated, int K, int sweep, int round, const LayerDev* __restrict__ layers, const int2* __restrict__ wg_map) {
    __shared__ JacobiShared sh;
    // Layers of one size: everything follows from the arguments.  Looked up in the tables, work-group -> layer -> flag
    // and pointers -> panel, four loads that wait for each other and miss every cache at the start of a launch took 8000 of the 40000
    // cycles of a round of 12 cores of 384.
    double *Ct, *diag;
    const double* trace;
    int slot;
    if (cores != nullptr) {
        Ct = cores + (int64_t)blockIdx.y * core_doubles(K);
        diag = Ct + core_diag(K);
        trace = Ct + core_trace(K);
        rotated += (int)blockIdx.y * (kMaxSweepsCap + 1);
        slot = (int)blockIdx.x;
    } else {
        const int2 wm = wg_map[blockIdx.x];               // (layer, pair slot)
        const LayerDev& L = layers[wm.x];
        Ct = L.Ct; diag = L.diag; trace = L.trace; rotated = L.rotated; K = L.K;
        slot = wm.y;
    }
    if (sweep > 0 && rotated[sweep - 1] == 0) return;     // the previous sweep found no significant pair: the iteration has converged
    const int nb = K >> 4;
    const int max_sweeps = WHOLE ? round : 0;
    if (WHOLE) round = 0;
    if (round >= nb - 1 || K > 64 * NT || (WHOLE && nb != 2)) return;
    // circle method: slot 0 pairs block nb-1 with `round`; slot j pairs (round + j) with (round - j)
    int bI = round + slot, bJ = round - slot;
    if (slot == 0) bI = nb - 1;
    else { if (bI >= nb - 1) bI -= nb - 1; if (bJ < 0) bJ += nb - 1; }
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 15, kq = lane >> 4;

    // Gram matrices of the two blocks as the last round left them, a value of each per thread; ||C||_F^2
    const int gi = (tid >> 6) + 4 * (tid & 3), gj = (tid >> 2) & 15;      // this thread's element of a 16 x 16 tile
    double* const diagI = diag + bI * 256;
    double* const diagJ = diag + bJ * 256;
    const bool fresh = WHOLE || round == 0;               // formed again from the columns once per sweep
    double ownII = fresh ? 0.0 : gload(diagI + 16 * gi + gj), ownJJ = fresh ? 0.0 : gload(diagJ + 16 * gi + gj);
    const double frob = frob2(trace);
    // ---- load the panel: D[t][s] = P[row(t, n)][column kq + 4 s], columns 0..15 = block I, 16..31 = block J (rows past K
    // repeat row 0 and are cleared behind the last load: a predicate on a load would be waited for with it)
    double D[NT][8];
#pragma unroll
    for (int tt = 0; tt < NT / 2; ++tt) {
        const int row0 = 32 * (wave + 4 * tt) + 2 * n;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int col = (s < 4 ? bI * 16 + kq + 4 * s : bJ * 16 + kq + 4 * (s - 4));
            const f64x2 v = gload(reinterpret_cast<const f64x2*>(Ct + (int64_t)col * K + (row0 < K ? row0 : 0)));
            D[2 * tt][s] = v[0];
            D[2 * tt + 1][s] = v[1];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int tt = 0; tt < NT / 2; ++tt) {
        const bool in = 32 * (wave + 4 * tt) + 2 * n < K;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            D[2 * tt][s] = in ? D[2 * tt][s] : 0.0;
            D[2 * tt + 1][s] = in ? D[2 * tt + 1][s] : 0.0;
        }
    }

    for (;; ++sweep) {                                   // one turn; WHOLE: until a sweep rotates nothing of weight
    // ---- S = P^T P: the tile between the blocks, and those inside them (II, JJ) if there are none of the last round
    f64x4 gII = {0.0, 0.0, 0.0, 0.0}, gIJ = gII, gJJ = gII;
    double* stage = sh.stage[wave];
    auto gram = [&](auto all) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int s = 0; s < 8; ++s) stage[stage_addr(n, kq + 4 * s)] = D[t][s];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            double a0[4], a1[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a0[q] = stage[stage_addr(4 * q + kq, n)];
                a1[q] = stage[stage_addr(4 * q + kq, 16 + n)];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (decltype(all)::value) gII = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[q], a0[q], gII, 0, 0, 0);
                gIJ = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[q], a1[q], gIJ, 0, 0, 0);
                if (decltype(all)::value) gJJ = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[q], a1[q], gJJ, 0, 0, 0);
            }
        }
    };
    if (fresh) gram(std::true_type{});
    else gram(std::false_type{});
    // partial tiles of the four waves, added in wave order; result element (i, j) of a tile sits in
    // lane (j, i % 4), register i / 4
    auto total = [&](int at) { return ((sh.stage[0][at] + sh.stage[1][at]) + sh.stage[2][at]) + sh.stage[3][at]; };
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        stage[1 * 256 + lane * 4 + v] = gIJ[v];
        if (fresh) stage[0 * 256 + lane * 4 + v] = gII[v];
    }
    __syncthreads();
    const double scale = ldexp(1.0, -__builtin_amdgcn_frexp_exp(frob));
    {
        const float sIJ = (float)(total(256 + tid) * scale);
        sh.S[gi][16 + gj] = sIJ;
        sh.S[16 + gj][gi] = sIJ;
        if (fresh) ownII = total(tid);
    }
    if (fresh) {
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) stage[lane * 4 + v] = gJJ[v];
        __syncthreads();
        ownJJ = total(tid);
    }
    sh.S[gi][gj] = (float)(ownII * scale);
    sh.S[16 + gi][16 + gj] = (float)(ownJJ * scale);
    const bool intra = round == 0;
    __syncthreads();

    // ---- cyclic Jacobi on S by one wave (which one differs among the work-groups that share a compute unit), the same
    // rotations on Q by the others, eight steps behind
    const float floor2 = (float)(kZeroColumn2 * frob * scale);
    const int other = (wave - (int)((blockIdx.x + blockIdx.y) & 3) - 1) & 3;         // 3: this wave works the rotations out
    bool any = false, any_signif = false;
    if (other == 3) {
        if (intra) {
            rotate_level<3>(sh.S, sh.tan[0][16], floor2, any, any_signif);
            rotate_level<2>(sh.S, sh.tan[0][24], floor2, any, any_signif);
            rotate_level<1>(sh.S, sh.tan[0][28], floor2, any, any_signif);
            rotate_level<0>(sh.S, sh.tan[0][30], floor2, any, any_signif);
            lds_barrier();
        }
        rotate_level<4>(sh.S, sh.tan[0][0], floor2, any, any_signif, &sh.flags, 1.0 / scale, WHOLE ? nullptr : diagI, WHOLE ? nullptr : diagJ);
    } else if (intra) {
        accumulate_inside(sh.Q, sh.tan[0], reinterpret_cast<f64x2*>(stage), other);
        accumulate_cross<false>(sh.Q, sh.tan[0], reinterpret_cast<f64x2*>(stage), other);
    } else {
        accumulate_cross<true>(sh.Q, sh.tan[0], reinterpret_cast<f64x2*>(stage), other);
    }
    lds_barrier();
    const int flags = sh.flags;
    const bool again = WHOLE && (flags & 2);
    if (tid == 0 && (flags & 2)) gstore(rotated + sweep, 1);
    if (!(flags & 1)) {
        if (WHOLE) break;
        return;                              // the columns are untouched: nothing else to store
    }

    // ---- P <- P Q as (Q^T P^T): A operand = Q^T tile, B operand = the panel registers
    double qa[2][8];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int s = 0; s < 8; ++s) qa[ct][s] = sh.Q[kq + 4 * s][16 * ct + n];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        f64x4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = acc0;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[0][s], D[t][s], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[1][s], D[t][s], acc1, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) { D[t][v] = acc0[v]; D[t][4 + v] = acc1[v]; }
    }
    if (!again || sweep + 1 >= max_sweeps) break;
    __syncthreads();                                     // Q is read, the next sweep's stages may overwrite
    }

    // ---- store
#pragma unroll
    for (int tt = 0; tt < NT / 2; ++tt) {
        const int row0 = 32 * (wave + 4 * tt) + 2 * n;
        if (row0 < K) {
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int col = (s < 4 ? bI * 16 + kq + 4 * s : bJ * 16 + kq + 4 * (s - 4));
                gstore(reinterpret_cast<f64x2*>(Ct + (int64_t)col * K + row0), f64x2{D[2 * tt][s], D[2 * tt + 1][s]});
            }
        }
    }
}

}  // namespace

hipError_t launch_jacobi_block_round(const LayerDev* layers, const int2* wg_map, int n_wg, int K_max,
                                     int sweep, int round, double* cores, int* rotated, hipStream_t s) {
    if (n_wg <= 0) return hipSuccess;
    const int slots = K_max / 32;
    const dim3 grid(cores ? slots : n_wg, cores ? n_wg / slots : 1), block(256);
    if (K_max <= 128) hipLaunchKernelGGL((jacobi_block_kernel<2, false>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else if (K_max <= 256) hipLaunchKernelGGL((jacobi_block_kernel<4, false>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else if (K_max <= 384) hipLaunchKernelGGL((jacobi_block_kernel<6, false>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else if (K_max <= 512) hipLaunchKernelGGL((jacobi_block_kernel<8, false>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else if (K_max <= 768) hipLaunchKernelGGL((jacobi_block_kernel<12, false>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_jacobi_single_pair(double* cores, int* rotated, int n, int max_sweeps, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((jacobi_block_kernel<2, true>), dim3(1, n), dim3(256), 0, s, cores, rotated, 32, 0, max_sweeps, (const LayerDev*)nullptr, (const int2*)nullptr);
    return hipGetLastError();
}

}  // namespace abt
