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
    double S[32][48];
    double Q[32][48];
    f64x2 cs[31][16];               // (cosine, sine) of the rotations of all steps
};

// ---- The rotations of a block pair.  Columns 0..31 (the two blocks) are paired by exclusive or: step m pairs every i with
// i ^ m, so 31 steps meet all pairs once, m = 16..31 those between the blocks, m < 16 those inside them.  The
// steps whose m has p as its highest bit form level p: with L(u), R(u) = the 4-bit u with a 0 or a 1 put in at bit p, step t pairs L(u)
// with R(u ^ t), t below 2^p.
__device__ __forceinline__ int left_of(int u, int p) { return ((u >> p) << (p + 1)) | (u & ((1 << p) - 1)); }
__device__ __forceinline__ int right_of(int u, int p) { return left_of(u, p) | (1 << p); }

template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); static_for<N, F, I + 1>(static_cast<F&&>(f)); }
}

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true));
}
// the value of lane ^ B (B = 1, 2, 3, 4, 8) by data-parallel moves: quad permutations, mirrored half rows, rotated rows
template <int B>
__device__ __forceinline__ double lane_xor(double v) {
    if constexpr (B == 1) return dpp<0xB1>(v);
    else if constexpr (B == 2) return dpp<0x4E>(v);
    else if constexpr (B == 3) return dpp<0x1B>(v);
    else if constexpr (B == 4) return dpp<0x1B>(dpp<0x141>(v));
    else return dpp<0x128>(v);
}

// The rotation of jacobi_rotation(), arranged for a short dependency chain (the 16 steps of a block
// pair are serial, and this is the longest link of a step): no branches, the tangent in fp32, the
// cosine from an fp32 reciprocal square root corrected by two terms of its series.  Any tangent
// gives a rotation that is orthogonal to fp64 rounding (c = (1 + t^2)^(-1/2), s = c t); a tangent
// good to 1e-7 leaves the pair with 1e-7 of its cosine.  `scale` is a power of two near
// 1 / ||C||_F^2: squared norms lie between kZeroColumn2 and 1 times ||C||_F^2, so scaled inputs of a
// pair that is rotated stay inside the fp32 range (|gamma| scale >= 1e-9 sqrt(1e-18 1e-18)).
__device__ __forceinline__ void fast_rotation(double alpha, double beta, double gamma, double floor2, double scale,
                                              double& c, double& s, bool& significant) {
    const double lim = alpha * beta;
    const double g2 = gamma * gamma;
    const bool live = alpha > floor2 && beta > floor2;
    significant = live && g2 > (kSignifTol * kSignifTol) * lim;
    const bool rot = live && g2 > (kRotateTol * kRotateTol) * lim;
    const float d = (float)((beta - alpha) * scale);
    const float g2x = (float)((gamma + gamma) * scale);
    const float zeta = d * __builtin_amdgcn_rcpf(g2x);
    const float az = fabsf(zeta);                        // an overflow of az^2 ends in t = 0 (|t| < 1e-19)
    const float ta = __builtin_amdgcn_rcpf(az + __builtin_amdgcn_sqrtf(fmaf(az, az, 1.0f)));
    const float tf = zeta >= 0.0f ? ta : -ta;
    const double c0 = (double)__builtin_amdgcn_rsqf(fmaf(tf, tf, 1.0f));
    const double tn = (double)tf;
    const double w = fma(tn, tn, 1.0);
    const double e = fma(-(c0 * c0), w, 1.0);            // c = c0 (1 - e)^(-1/2) = c0 (1 + e/2 + 3 e^2/8 + ...)
    const double cc = fma(c0, e * fma(0.375, e, 0.5), c0);
    c = rot ? cc : 1.0;
    s = rot ? cc * tn : 0.0;
}

// Level p on S by one wave, S in registers: lane (u = l % 16, q = l / 16) owns, for x = 4 q + e, the 2 x 2 cell rows
// L(u), R(u ^ t) x columns L(v), R(v ^ t) with v = u ^ x.  t runs through a Gray code; when bit b of it changes, a cell finds its new
// off-diagonal entries in the cell x ^ b (another register of the lane for b = 1, 2) and its new last
// entry, like the one below the diagonal, in lane ^ b: register names and data-parallel moves, no LDS and no barrier
// in a step.  The pairs' own cells are x = 0, in the first 16 lanes, which work the rotations out; the lanes that need
// them fetch them with a lane permute.  A step takes 790 cycles, most of it the chain of the rotation formula, the permute
// and the update of the pairs' cells.  With S in LDS, cells dealt to four waves and a barrier a step it took 1150; in a loop of four
// steps a turn, with half the code, 920.
template <int P>
__device__ __forceinline__ void rotate_level(double (*S)[48], f64x2 (*cs)[16], double floor2, double scale, bool& any_signif,
                                             double* diagI = nullptr, double* diagJ = nullptr) {
    const int lane = threadIdx.x & 63, u = lane & 15, q = lane >> 4;
    double m00[4], m01[4], m10[4], m11[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int v = u ^ (4 * q + e);
        m00[e] = S[left_of(u, P)][left_of(v, P)]; m01[e] = S[left_of(u, P)][right_of(v, P)];
        m10[e] = S[right_of(u, P)][left_of(v, P)]; m11[e] = S[right_of(u, P)][right_of(v, P)];
    }
    // one step; B: the bit of t that changes after it (0: the last step)
    auto step = [&](auto bit, int k) {
        constexpr int B = decltype(bit)::value;
        double c, s; bool signif;
        fast_rotation(m00[0], m11[0], m01[0], floor2, scale, c, s, signif);
        if (lane < 16) { any_signif |= signif; cs[k][u] = f64x2{c, s}; }
        const double c1 = __shfl(c, u, 64), s1 = __shfl(s, u, 64);
        double c2[4], s2[4];
        c2[0] = __shfl(c, u ^ (4 * q), 64); s2[0] = __shfl(s, u ^ (4 * q), 64);
        c2[1] = lane_xor<1>(c2[0]); s2[1] = lane_xor<1>(s2[0]);
        c2[2] = lane_xor<2>(c2[0]); s2[2] = lane_xor<2>(s2[0]);
        c2[3] = lane_xor<3>(c2[0]); s2[3] = lane_xor<3>(s2[0]);
        double n01[4], n10[4], n11[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double t00 = c1 * m00[e] - s1 * m10[e], t01 = c1 * m01[e] - s1 * m11[e];
            const double t10 = s1 * m00[e] + c1 * m10[e], t11 = s1 * m01[e] + c1 * m11[e];
            m00[e] = c2[e] * t00 - s2[e] * t01; n01[e] = s2[e] * t00 + c2[e] * t01;
            n10[e] = c2[e] * t10 - s2[e] * t11; n11[e] = s2[e] * t10 + c2[e] * t11;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (B == 0) { m01[e] = n01[e]; m10[e] = n10[e]; m11[e] = n11[e]; }
            else if constexpr (B < 4) { m01[e] = n01[e ^ B]; m10[e] = lane_xor<B>(n10[e ^ B]); m11[e] = lane_xor<B>(n11[e]); }
            else {
                m01[e] = __shfl_xor(n01[e], 4 * B, 64); m10[e] = __shfl_xor(n10[e], 5 * B, 64); m11[e] = lane_xor<B>(n11[e]);
            }
        }
    };
    static_for<(1 << P)>([&](auto i) {
        constexpr int k = decltype(i)::value;
        step(std::integral_constant<int, (k + 1 < (1 << P) ? (k + 1) & -(k + 1) : 0)>{}, k);
    });
    constexpr int t = ((1 << P) - 1) ^ (((1 << P) - 1) >> 1);
    if (P == 4) {                                        // the last level: the two diagonal blocks, for the next round
        if (diagI == nullptr) return;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int v = u ^ (4 * q + e);
            gstore(diagI + 16 * u + v, m00[e]);
            gstore(diagJ + 16 * (u ^ t) + (v ^ t), m11[e]);
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int v = u ^ (4 * q + e);
        S[left_of(u, P)][left_of(v, P)] = m00[e]; S[left_of(u, P)][right_of(v ^ t, P)] = m01[e];
        S[right_of(u ^ t, P)][left_of(v, P)] = m10[e]; S[right_of(u ^ t, P)][right_of(v ^ t, P)] = m11[e];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same rotations on the columns of Q, rows 8 wave .. 8 wave + 7 by this wave: lane (u, q) owns columns L(u), R(u ^ t) of
// rows q and q + 4 of them.
template <int P>
__device__ __forceinline__ void accumulate_level(double (*Q)[48], const f64x2 (*cs)[16]) {
    const int lane = threadIdx.x & 63, u = lane & 15, r = 8 * (threadIdx.x >> 6) + (lane >> 4);
    double a0 = Q[r][left_of(u, P)], b0 = Q[r][right_of(u, P)], a1 = Q[r + 4][left_of(u, P)], b1 = Q[r + 4][right_of(u, P)];
    auto step = [&](auto bit, int k) {
        constexpr int B = decltype(bit)::value;
        const f64x2 rot = cs[k][u];
        const double c = rot[0], s = rot[1];
        const double x0 = c * a0 - s * b0, y0 = s * a0 + c * b0, x1 = c * a1 - s * b1, y1 = s * a1 + c * b1;
        a0 = x0; a1 = x1;
        if constexpr (B == 0) { b0 = y0; b1 = y1; }
        else { b0 = lane_xor<B>(y0); b1 = lane_xor<B>(y1); }
    };
    static_for<(1 << P)>([&](auto i) {
        constexpr int k = decltype(i)::value;
        step(std::integral_constant<int, (k + 1 < (1 << P) ? (k + 1) & -(k + 1) : 0)>{}, k);
    });
    constexpr int t = ((1 << P) - 1) ^ (((1 << P) - 1) >> 1);
    Q[r][left_of(u, P)] = a0; Q[r][right_of(u ^ t, P)] = b0; Q[r + 4][left_of(u, P)] = a1; Q[r + 4][right_of(u ^ t, P)] = b1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// NT: 16-row tiles per wave (two per 32-row chunk: its even and its odd rows), K <= 64 NT.
// (Three work-groups per compute unit at K = 384 spill and take 7.0 ms in place of 4.6 over a merge; two at K = 768, 24.7 of 16.2.)
// WHOLE (K = 32: two blocks, one pair): the work-group holds the whole core, so it runs all sweeps in one launch, the
// panel in registers throughout; `round` is the sweep cap.  A launch and a poll of the convergence flags per
// sweep took 129 us for one core of 32, this 54.
template <int NT, bool WHOLE>
__global__ __launch_bounds__(256, (WHOLE ? 1 : NT <= 2 ? 3 : NT <= 6 ? 2 : 1))
void jacobi_block_kernel(const LayerDev* __restrict__ layers, const int2* __restrict__ wg_map, int sweep, int round) {
    __shared__ JacobiShared sh;
    const int2 wm = wg_map[blockIdx.x];                   // (layer, pair slot)
    const LayerDev& L = layers[wm.x];
    if (sweep_finished(L, sweep)) return;
    const int K = L.K, nb = K >> 4;
    const int max_sweeps = WHOLE ? round : 0;
    if (WHOLE) round = 0;
    if (round >= nb - 1 || K > 64 * NT || (WHOLE && nb != 2)) return;
    // circle method: slot 0 pairs block nb-1 with `round`; slot j pairs (round + j) with (round - j)
    int bI, bJ;
    if (wm.y == 0) { bI = nb - 1; bJ = round; }
    else { bI = (round + wm.y) % (nb - 1); bJ = (round - wm.y + (nb - 1)) % (nb - 1); }
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 15, kq = lane >> 4;

    // Gram matrices of the two blocks as the last round left them, a value of each per thread; ||C||_F^2
    const int gi = (tid >> 6) + 4 * (tid & 3), gj = (tid >> 2) & 15;      // this thread's element of a 16 x 16 tile
    double* const diagI = L.diag + bI * 256;
    double* const diagJ = L.diag + bJ * 256;
    const bool fresh = WHOLE || round == 0;               // formed again from the columns once per sweep
    double ownII = fresh ? 0.0 : gload(diagI + 16 * gi + gj), ownJJ = fresh ? 0.0 : gload(diagJ + 16 * gi + gj);
    const double frob = frob2(L);
    // ---- load the panel: D[t][s] = P[row(t, n)][column kq + 4 s], columns 0..15 = block I, 16..31 = block J (rows past K
    // repeat row 0 and are cleared behind the last load: a predicate on a load would be waited for with it)
    double D[NT][8];
#pragma unroll
    for (int tt = 0; tt < NT / 2; ++tt) {
        const int row0 = 32 * (wave + 4 * tt) + 2 * n;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int col = (s < 4 ? bI * 16 + kq + 4 * s : bJ * 16 + kq + 4 * (s - 4));
            const f64x2 v = gload(reinterpret_cast<const f64x2*>(L.Ct + (int64_t)col * K + (row0 < K ? row0 : 0)));
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
    {
        const double sIJ = total(256 + tid);
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
    sh.S[gi][gj] = ownII;
    sh.S[16 + gi][16 + gj] = ownJJ;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int idx = tid + 256 * e;
        sh.Q[idx >> 5][idx & 31] = (idx >> 5) == (idx & 31) ? 1.0 : 0.0;
    }
    __syncthreads();

    // ---- anything to rotate?  (pairs inside the blocks count in round 0 only)
    const double floor2 = kZeroColumn2 * frob;
    const double scale = ldexp(1.0, -__builtin_amdgcn_frexp_exp(frob));
    const bool intra = round == 0;
    int need = 0;
    {
        const int i = tid >> 4, j = tid & 15;
        auto test = [&](int p, int q) {
            const double a = sh.S[p][p], b = sh.S[q][q], g = sh.S[p][q];
            if (a > floor2 && b > floor2 && g * g > (kRotateTol * kRotateTol) * (a * b)) need = 1;
        };
        test(i, 16 + j);
        if (intra && i < j) { test(i, j); test(16 + i, 16 + j); }
    }
    if (!__syncthreads_or(need)) {
        if (WHOLE) break;
        if (fresh) { gstore(diagI + 16 * gi + gj, ownII); gstore(diagJ + 16 * gi + gj, ownJJ); }
        return;                              // the columns are untouched: nothing else to store
    }

    // ---- cyclic Jacobi on S by one wave (which one differs among the work-groups that share a compute unit), then the
    // same rotations on Q by all
    bool any_signif = false;
    if (wave == (int)(blockIdx.x & 3)) {
        if (intra) {
            rotate_level<3>(sh.S, sh.cs + 16, floor2, scale, any_signif);
            rotate_level<2>(sh.S, sh.cs + 24, floor2, scale, any_signif);
            rotate_level<1>(sh.S, sh.cs + 28, floor2, scale, any_signif);
            rotate_level<0>(sh.S, sh.cs + 30, floor2, scale, any_signif);
        }
        rotate_level<4>(sh.S, sh.cs, floor2, scale, any_signif, WHOLE ? nullptr : diagI, WHOLE ? nullptr : diagJ);
    }
    __syncthreads();
    if (intra) {
        accumulate_level<3>(sh.Q, sh.cs + 16);
        accumulate_level<2>(sh.Q, sh.cs + 24);
        accumulate_level<1>(sh.Q, sh.cs + 28);
        accumulate_level<0>(sh.Q, sh.cs + 30);
    }
    accumulate_level<4>(sh.Q, sh.cs);
    __syncthreads();
    const bool again = WHOLE && __syncthreads_or(any_signif);
    if (any_signif) L.rotated[sweep] = 1;

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
                gstore(reinterpret_cast<f64x2*>(L.Ct + (int64_t)col * K + row0), f64x2{D[2 * tt][s], D[2 * tt + 1][s]});
            }
        }
    }
}

}  // namespace

hipError_t launch_jacobi_block_round(const LayerDev* layers, const int2* wg_map, int n_wg, int K_max,
                                     int sweep, int round, hipStream_t s) {
    if (n_wg <= 0) return hipSuccess;
    const dim3 grid(n_wg), block(256);
    if (K_max <= 128) hipLaunchKernelGGL((jacobi_block_kernel<2, false>), grid, block, 0, s, layers, wg_map, sweep, round);
    else if (K_max <= 256) hipLaunchKernelGGL((jacobi_block_kernel<4, false>), grid, block, 0, s, layers, wg_map, sweep, round);
    else if (K_max <= 384) hipLaunchKernelGGL((jacobi_block_kernel<6, false>), grid, block, 0, s, layers, wg_map, sweep, round);
    else if (K_max <= 512) hipLaunchKernelGGL((jacobi_block_kernel<8, false>), grid, block, 0, s, layers, wg_map, sweep, round);
    else if (K_max <= 768) hipLaunchKernelGGL((jacobi_block_kernel<12, false>), grid, block, 0, s, layers, wg_map, sweep, round);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_jacobi_single_pair(const LayerDev* layers, const int2* wg_map, int n_wg, int max_sweeps, hipStream_t s) {
    if (n_wg <= 0) return hipSuccess;
    hipLaunchKernelGGL((jacobi_block_kernel<2, true>), dim3(n_wg), dim3(256), 0, s, layers, wg_map, 0, max_sweeps);
    return hipGetLastError();
}

}  // namespace abt
