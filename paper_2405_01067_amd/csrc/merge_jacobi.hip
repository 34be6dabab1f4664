// Block form of the one-sided Jacobi iteration on the K x K core of the merge (the truncated SVD
// of Eq. 3 on the merged matrix), for K <= 768, on the fp64 matrix cores.
//
// The columns of C (rows of Ct) are grouped in blocks of 16; a round pairs every block with one
// partner (round-robin tournament over the blocks), one work-group per block pair.  For its 32
// columns P (K x 32) a work-group
//   1. forms the Gram matrix S = P^T P (32 x 32) with v_mfma_f64_16x16x4: the 16 x 16 tile between the blocks; the
//      tiles inside them are what the last round's rotations left of S, and formed anew in round 0 of a sweep only,
//   2. runs the cyclic Jacobi eigenvalue iteration on S, by one wave: 16 steps of 16 disjoint rotations, every rotation applied to S
//      from both sides; three other waves accumulate them in Q (32 x 32).  These are the plane rotations the column form of the
//      method would apply to the 256 column pairs of the two blocks, in the same order; they are
//      worked out on the 32 x 32 Gram matrix instead of on K-long columns,
//   3. applies them at once: P <- P Q, again on the matrix cores, all waves.
// Round 0 of a sweep first rotates the pairs inside each of the two blocks the same way (15 steps).
//
// With many work-groups (the rule is where the batch is planned) a work-group has four blocks instead, a, b | c, d: double blocks meet in
// the tournament, and a round rotates the pairs (a, c) and (b, d), then (a, d) and (b, c), two at a time; round 0 begins with (a, b) and (c, d).
//
// The panel lives in registers from load to store, in the operand layout of step 3: a lane holds
// the rows r = l % 16 of its wave's row tiles and the columns l / 16 + 4 s of a block (s = 0..3); with the
// product taken as (Q^T P^T) the result tile comes out of the matrix core in that same layout, so
// the update is in place.  Step 1 needs the transposed operand order (contraction over rows); each
// wave passes its row tiles through a private LDS tile for that.
//
// What bounds it: nothing survives in L2 from one round to the next, so a round reads and writes all cores beyond it: 64 GB for 16 cores
// of 768 in 9 sweeps, 4.8 TB/s in 13.3 ms, near what a large copy reaches (one work-group per compute unit, one thing after the other, 16.2).  48 cores
// of 384, 8 sweeps: 4.6 ms that way, 4.0 with four blocks, which is half the traffic.  With few cores a work-group's chain counts: cycles at K = 384 (two blocks): arguments and flag 1500, first
// columns 3000, Gram matrix 5600, rotations 12000, the last of Q 1100, update 6400 (fp64 matrix instructions); four blocks some 80000 a round of three times
// those links.  Launches follow each other in 1.3 us.
#include <type_traits>

#include "merge_internal.h"

namespace abt {

namespace {

// swizzled address (in doubles) of element (row n, column c) of a 16 x 32 staging tile: stores of one
// column by 16 rows and loads of 16 consecutive columns of one row both spread over all banks
__device__ __forceinline__ int stage_addr(int n, int c) {
    return 32 * n + ((c + 16 * (n & 1) + 2 * (n >> 1)) & 31);
}

// What the rotations of a block pair need in LDS
struct __align__(16) PairShared {
    double Q[32][48];
    double S[32][33];               // the Gram matrix times a power of two
    int did;                        // 0: rotated nothing, 1: nothing significant, 2: something
    float tan[31][16];              // tangents of the rotations of all steps
};

// ---- The rotations of a block pair.  Columns 0..31 (the two blocks) are paired by exclusive or: step m pairs every i with
// i ^ m, so 31 steps meet all pairs once, m = 16..31 those between the blocks, m < 16 those inside them.  The
// steps whose m has p as its highest bit form level p: with L(u), R(u) = the 4-bit u with a 0 or a 1 put in at bit p, step t pairs L(u)
// with R(u ^ t), t below 2^p.
__device__ __forceinline__ int left_of(int u, int p) { return ((u >> p) << (p + 1)) | (u & ((1 << p) - 1)); }
__device__ __forceinline__ int right_of(int u, int p) { return left_of(u, p) | (1 << p); }

// threadIdx.x, anew: what is computed from it in a loop is not carried through the loop in registers (150 of them otherwise, and as many spilled)
__device__ __forceinline__ int thread_anew() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}
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
__device__ __forceinline__ int row_xor(int x) {
    if constexpr (B == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);      // r[0]: even rows twice, r[1]: odd rows twice
        return (threadIdx.x & 16) ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (threadIdx.x & 32) ? r[0] : r[1];
    }
}
template <int B>
__device__ __forceinline__ double row_xor(double v) { return __hiloint2double(row_xor<B>(__double2hiint(v)), row_xor<B>(__double2loint(v))); }
// lanes 0..15 to all four rows
__device__ __forceinline__ float first_row(float v) {
    const unsigned x = __float_as_uint(v);
    const unsigned lo = __builtin_amdgcn_permlane32_swap(x, x, false, false)[0];
    return __uint_as_float(__builtin_amdgcn_permlane16_swap(lo, lo, false, false)[0]);
}
// of a value that all rows hold alike: lane u ^ 4 q of it for lane (u, q)
__device__ __forceinline__ int xor_by_row(int x) {
    x = dpp_rows<0x128, 0xc>(x, x);                           // rows 2, 3: lanes 8 apart
    const int w = dpp_rows<0x141, 0xa>(x, x);                 // rows 1, 3: lanes 4 apart, in two moves
    return dpp_rows<0x1B, 0xa>(w, w);
}
__device__ __forceinline__ float xor_by_row(float v) { return __int_as_float(xor_by_row(__float_as_int(v))); }
__device__ __forceinline__ double xor_by_row(double v) { return __hiloint2double(xor_by_row(__double2hiint(v)), xor_by_row(__double2loint(v))); }

// Level p on S by one wave, S in registers: lane (u = l % 16, q = l / 16) owns, for x = 4 q + e, the 2 x 2 cell rows
// L(u), R(u ^ t) x columns L(v), R(v ^ t) with v = u ^ x.  t runs through a Gray code; when bit b of it changes, a cell finds its new
// off-diagonal entries in the cell x ^ b (another register of the lane for b = 1, 2) and its new last
// entry, like the one below the diagonal, in lane ^ b: register names and data-parallel moves, no LDS and no barrier
// in a step.  The pairs' own cells are x = 0, in the first 16 lanes, which work the tangents out; these go to the other lanes by row
// swaps and row-masked moves.
// The tangent is that of jacobi_rotation(), without branches, in fp32 from a difference taken in fp64.  Any tangent gives a rotation
// that is orthogonal to fp64 rounding, as cosine and sine are formed from it in fp64; one good to 1e-7 leaves the pair with 1e-7 of its cosine.  S is
// scaled by a power of two near 1 / ||C||_F^2: squared norms lie between kZeroColumn2 and 1, inner products of a pair that is
// rotated above 1e-9 of that, inside the fp32 range.
// S itself is fp64 throughout.  In fp32 the difference of the norms of nearly equal columns is rounding, and what is left of a small
// column's norm beside a large one's too: two clusters of values 1e-3 apart took 18 to 20 sweeps of 768 columns instead of 14 or 15 and were
// left twice as far off.  (A step is 750 cycles, 540 in fp32: one core of 32 41 us / 33, 48 cores of 384 4.0 ms / 3.7, 16 of 768 13.3 / 12.7.)
// The steps are serial, so the chain through the pairs' own cells sets the pace, and the issue of the other cells' updates comes next: a
// step updates the cells that the next tangent needs first and the others between the links of its formula.
// A cell is multiplied by (1, -t; t, 1) from both sides and by the product of the cosines.
// `spare`: where other lanes than the pairs' own put what they come to for a tangent.
// keep(block, row, column, value): what is left of the two blocks' own Gram matrices (level 4).
template <int P, class Keep>
__device__ __forceinline__ void rotate_level(double (*S)[33], float* tangents, float* spare, double floor2, bool& any, bool& any_signif, int* did, Keep&& keep) {
    const int lane = thread_anew() & 63, u = lane & 15, q = lane >> 4;
    float* const mine = (q ? spare : tangents) + u;
    double m00[4], m01[4], m10[4], m11[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int v = u ^ (4 * q + e);
        m00[e] = S[left_of(u, P)][left_of(v, P)]; m01[e] = S[left_of(u, P)][right_of(v, P)];
        m10[e] = S[right_of(u, P)][left_of(v, P)]; m11[e] = S[right_of(u, P)][right_of(v, P)];
    }
    // the tangent of the pair with squared norms alpha, beta and inner product gamma, in three links
    float zeta, w, own;
    bool turn;
    auto link1 = [&](double alpha, double beta, double gamma) {
        const float g = (float)gamma;
        zeta = (float)(beta - alpha) * __builtin_amdgcn_rcpf(g + g);
        const double lim = alpha * beta, g2 = gamma * gamma;
        const bool live = alpha > floor2 && beta > floor2;
        any_signif |= live && g2 > (kSignifTol * kSignifTol) * lim;        // (this and the next count in the first 16 lanes)
        turn = live && g2 > (kRotateTol * kRotateTol) * lim;
        any |= turn;
    };
    auto link2 = [&]() {
        w = __builtin_amdgcn_sqrtf(fmaf(zeta, zeta, 1.0f));                // an overflow of the square ends in t = 0 (|t| < 1e-19)
    };
    auto link3 = [&]() {
        const float ta = __builtin_amdgcn_rcpf(fabsf(zeta) + w);
        own = turn ? copysignf(ta, zeta) : 0.0f;
    };
    link1(m00[0], m11[0], m01[0]); link2(); link3();
    // one step; B: the bit of t that changes after it (0: the last step)
    auto step = [&](auto bit, int k) {
        constexpr int B = decltype(bit)::value;
        constexpr int E1 = B == 2 ? 2 : 1, E2 = B == 2 ? 1 : 2;            // the second cell to be updated, the third
        mine[16 * k] = own;
        const float t = first_row(own);
        const float f2 = xor_by_row(t);
        const double t1 = (double)t;
        // c = c0 (1 - e)^(-1/2) = c0 (1 + e/2 + 3 e^2/8 + ..) with c0 in fp32
        const double c0 = (double)__builtin_amdgcn_rsqf(fmaf(t, t, 1.0f));
        const double err = fma(-(c0 * c0), fma(t1, t1, 1.0), 1.0), c1 = fma(c0, err * fma(0.375, err, 0.5), c0), c2 = xor_by_row(c1);
        double n01[4], n10[4], n11[4];
        auto update = [&](auto which) {
            constexpr int e = decltype(which)::value;
            double t2, c12;
            if constexpr (e == 0) { t2 = (double)f2; c12 = c1 * c2; }
            else { t2 = (double)lane_xor<e>(f2); c12 = c1 * lane_xor<e>(c2); }
            const double a = fma(-t1, m10[e], m00[e]), b = fma(-t1, m11[e], m01[e]), c = fma(t1, m00[e], m10[e]), d = fma(t1, m01[e], m11[e]);
            m00[e] = fma(-t2, b, a) * c12; n01[e] = fma(t2, a, b) * c12;
            n10[e] = fma(-t2, d, c) * c12; n11[e] = fma(t2, c, d) * c12;
        };
        update(std::integral_constant<int, 0>{});
        if constexpr (B == 1 || B == 2) update(std::integral_constant<int, E1>{});
        if constexpr (B != 0) {
            const double beta = lane_xor<B>(n11[0]);
            double gamma;
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
        if constexpr (B != 0) link3();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (B == 0) { m01[e] = n01[e]; m10[e] = n10[e]; m11[e] = n11[e]; }
            else if constexpr (B < 4) { m01[e] = n01[e ^ B]; m10[e] = lane_xor<B>(n10[e ^ B]); m11[e] = lane_xor<B>(n11[e]); }
            else { m01[e] = row_xor<4 * B>(n01[e]); m10[e] = row_xor<4 * B>(lane_xor<B>(n10[e])); m11[e] = lane_xor<B>(n11[e]); }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    static_for<(1 << P)>([&](auto i) {
        constexpr int k = decltype(i)::value;
        if constexpr (P == 4 && k == 8) lds_barrier();   // the first eight tangents: the other waves begin with Q
        step(std::integral_constant<int, (k + 1 < (1 << P) ? (k + 1) & -(k + 1) : 0)>{}, k);
    });
    constexpr int t = ((1 << P) - 1) ^ (((1 << P) - 1) >> 1);
    if constexpr (P == 4) {                              // the last level: the two diagonal blocks, for the next round
        const bool r = __builtin_amdgcn_ballot_w64(any && lane < 16) != 0, sg = __builtin_amdgcn_ballot_w64(any_signif && lane < 16) != 0;
        if (lane == 0) *did = sg ? 2 : r ? 1 : 0;
        lds_barrier();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int v = u ^ (4 * q + e);
            keep(0, u, v, m00[e]);
            keep(1, u ^ t, v ^ t, m11[e]);
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
    const int lane = thread_anew() & 63, u = lane & 15, r = 12 * w + (lane >> 4);
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
    const int lane = thread_anew() & 63;
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
    const int lane = thread_anew() & 63, u = lane & 15, r = 12 * w + (lane >> 4);
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

// The sixteen steps of a block pair, after those inside its blocks if `inside`, by the waves that share it: `role` 3 works the rotations out,
// 0 to 2 accumulate them.  `table`: 4 KB of LDS of the wave's own.  Four barriers with `inside`, three without; Q and `did` are
// there after the last.  after(): at the end, by the wave that works the rotations out.
template <class Keep, class After>
__device__ __forceinline__ void rotate_pair(PairShared& sh, bool inside, int role, f64x2* table, double floor2, Keep&& keep, After&& after) {
    if (role == 3) {
        bool any = false, any_signif = false;
        float* const spare = reinterpret_cast<float*>(table);
        if (inside) {
            rotate_level<3>(sh.S, sh.tan[16], spare, floor2, any, any_signif, nullptr, keep);
            rotate_level<2>(sh.S, sh.tan[24], spare, floor2, any, any_signif, nullptr, keep);
            rotate_level<1>(sh.S, sh.tan[28], spare, floor2, any, any_signif, nullptr, keep);
            rotate_level<0>(sh.S, sh.tan[30], spare, floor2, any, any_signif, nullptr, keep);
            lds_barrier();
        }
        rotate_level<4>(sh.S, sh.tan[0], spare, floor2, any, any_signif, &sh.did, keep);
        lds_barrier();
        after();
        return;
    } else if (inside) {
        accumulate_inside(sh.Q, sh.tan, table, role);
        accumulate_cross<false>(sh.Q, sh.tan, table, role);
    } else {
        accumulate_cross<true>(sh.Q, sh.tan, table, role);
    }
    lds_barrier();
}

struct Core { double *Ct, *diag; const double* trace; int* rotated; int K, slot; };
// Layers of one size: everything follows from the arguments.  Looked up in the tables, work-group -> layer -> flag
// and pointers -> columns, four loads that wait for each other and miss every cache at the start of a launch took 8000
// cycles of a round of 12 cores of 384, now 1500.
__device__ __forceinline__ Core find_core(double* cores, int* rotated, int K, const LayerDev* layers, const int2* wg_map) {
    if (cores != nullptr) {
        double* const Ct = cores + (int64_t)blockIdx.y * core_doubles(K);
        return Core{Ct, Ct + core_diag(K), Ct + core_trace(K), rotated + (int)blockIdx.y * (kMaxSweepsCap + 1), K, (int)blockIdx.x};
    }
    const int2 wm = wg_map[blockIdx.x];                   // (layer, pair slot)
    const LayerDev& L = layers[wm.x];
    return Core{L.Ct, L.diag, L.trace, L.rotated, L.K, wm.y};
}

// NT: 16-row tiles per wave (two per 32-row chunk: its even and its odd rows), K <= 128 NT.  Eight waves, one work-group per compute
// unit; waves 0 to 3 work on the first block pair of the two, 4 to 7 on the second, and all of them on both where rows count.
// max_sweeps > 0 (cores of 64, one pair of double blocks): the work-group holds the whole core and runs all sweeps in one launch.
template <int NT>
__global__ __launch_bounds__(512, 1)
void jacobi_quad_kernel(double* cores, int* rotated, int K, int sweep, int round, int max_sweeps, const LayerDev* __restrict__ layers, const int2* __restrict__ wg_map) {
    __shared__ struct __align__(16) {
        double stage[8][2][16 * 32];    // per wave: transposition tiles; afterwards the waves' partial Gram tiles, then tables of rotations
        PairShared pair[2];
        double diag[4][16 * 17];        // Gram matrices of the blocks, scaled
    } sh;
    const Core c = find_core(cores, rotated, K, layers, wg_map);
    double* const Ct = c.Ct;
    double* const diag = c.diag;
    K = c.K;
    rotated = c.rotated;
    const int slot = c.slot;
    if (sweep > 0 && rotated[sweep - 1] == 0) return;     // the previous sweep found no significant pair: the iteration has converged
    const int nd = K >> 5;                                // double blocks, an even number
    const bool whole = max_sweeps > 0;
    if (round >= nd - 1 || K > 128 * NT) return;
    // circle method: slot 0 pairs double block nd - 1 with `round`; slot j pairs (round + j) with (round - j)
    int dI = round + slot, dJ = round - slot;
    if (slot == 0) dI = nd - 1;
    else { if (dI >= nd - 1) dI -= nd - 1; if (dJ < 0) dJ += nd - 1; }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, kq = lane >> 4;
    const int half = wave >> 2, t8 = tid & 255;            // block pair of this wave, thread within it
    const int gi = (t8 >> 6) + 4 * (t8 & 3), gj = (t8 >> 2) & 15;         // this thread's element of a 16 x 16 tile
    PairShared& mine = sh.pair[half];

    // Position i holds block blk[i], whose Gram matrix is tile id[i]; the pairs are positions (0, 2) and (1, 3).  Round 0 begins
    // with positions 1 and 2 exchanged, so that its first pairs are (a, b) and (c, d).
    int blk[4], id[4] = {0, 1, 2, 3};
    {
        const int b0 = 2 * dI, b1 = 2 * dI + 1, b2 = 2 * dJ, b3 = 2 * dJ + 1;
        blk[0] = b0; blk[1] = round == 0 ? b2 : b1; blk[2] = round == 0 ? b1 : b2; blk[3] = b3;
        if (round == 0) { id[1] = 2; id[2] = 1; }
    }
    // Gram matrices of the blocks as the last round left them, two values of each thread; ||C||_F^2
    double kept[2] = {0.0, 0.0};
    if (round != 0) {
        kept[0] = gload(diag + (half ? blk[1] : blk[0]) * 256 + 16 * gi + gj);
        kept[1] = gload(diag + (half ? blk[3] : blk[2]) * 256 + 16 * gi + gj);
    }
    const double frob = frob2(c.trace);
    // ---- load the columns: D[t][4 i + s] = C[row(t, n)][16 blk[i] + kq + 4 s].  Chunks past K are zero,
    // the same for the whole wave, so nothing is done to a value that has just been asked for and the Gram matrix begins with the first chunk.
    double D[NT][16];
#pragma unroll
    for (int tt = 0; tt < NT / 2; ++tt) {
        const int row0 = 32 * (wave + 8 * tt) + 2 * n;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (32 * (wave + 8 * tt) < K) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const f64x2 v = gload(reinterpret_cast<const f64x2*>(Ct + (int64_t)(16 * blk[i] + kq + 4 * s) * K + row0));
                    D[2 * tt][4 * i + s] = v[0];
                    D[2 * tt + 1][4 * i + s] = v[1];
                }
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) D[2 * tt][4 * i + s] = D[2 * tt + 1][4 * i + s] = 0.0;
            }
        }
    }
    const double scale = ldexp(1.0, -__builtin_amdgcn_frexp_exp(frob));
    const double floor2 = kZeroColumn2 * frob * scale;
    if (round != 0) {
        sh.diag[half][17 * gi + gj] = kept[0] * scale;           // (id[i] = i)
        sh.diag[2 + half][17 * gi + gj] = kept[1] * scale;
    }
    // exchange positions A and B
    auto exchange = [&](auto a, auto b) {
        constexpr int A = decltype(a)::value, B = decltype(b)::value;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int s = 0; s < 4; ++s) { const double v = D[t][4 * A + s]; D[t][4 * A + s] = D[t][4 * B + s]; D[t][4 * B + s] = v; }
        int v = blk[A]; blk[A] = blk[B]; blk[B] = v;
        v = id[A]; id[A] = id[B]; id[B] = v;
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Three = std::integral_constant<int, 3>;

    auto store_chunk = [&](int tt, int n, int kq) {
        const int row0 = 32 * (wave + 8 * tt) + 2 * n;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                gstore(reinterpret_cast<f64x2*>(Ct + (int64_t)(16 * blk[i] + kq + 4 * s) * K + row0), f64x2{D[2 * tt][4 * i + s], D[2 * tt + 1][4 * i + s]});
        }
    };
    int touched = 0, seen = 0;                            // the most that was done, ever and in this sweep
    for (;; ++sweep) {                                    // one turn; a whole core: until a sweep rotates nothing of weight
#pragma unroll 1
    for (int inner = round == 0 ? 0 : 1; inner < 3; ++inner) {
        const bool inside = inner == 0;
        const int tid = thread_anew(), lane = tid & 63, n = lane & 15, kq = lane >> 4;
        const int gi = ((tid >> 6) & 3) + 4 * (tid & 3), gj = (tid >> 2) & 15;
        // ---- S = P^T P of both pairs: the tile between the blocks, and those inside them if there are none yet
        f64x4 gIJ[2] = {}, gII[2] = {}, gJJ[2] = {};
        auto gram = [&](auto all) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if (t % 2 == 0 && 32 * (wave + 4 * t) >= K) break;        // no rows of this core
                double a0[2][4], a1[2][4];
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        sh.stage[wave][p][stage_addr(n, kq + 4 * s)] = D[t][4 * p + s];
                        sh.stage[wave][p][stage_addr(n, 16 + kq + 4 * s)] = D[t][8 + 4 * p + s];
                    }
                wave_lds_fence();
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        a0[p][q] = sh.stage[wave][p][stage_addr(4 * q + kq, n)];
                        a1[p][q] = sh.stage[wave][p][stage_addr(4 * q + kq, 16 + n)];
                    }
                wave_lds_fence();
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        gIJ[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[p][q], a1[p][q], gIJ[p], 0, 0, 0);
                        if constexpr (decltype(all)::value) {
                            gII[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[p][q], a0[p][q], gII[p], 0, 0, 0);
                            gJJ[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[p][q], a1[p][q], gJJ[p], 0, 0, 0);
                        }
                    }
            }
        };
        if (inside) gram(std::true_type{});
        else gram(std::false_type{});
        // partial tiles of the eight waves, added in wave order; result element (i, j) of a tile sits in
        // lane (j, i % 4), register i / 4.  Each pair's by the threads of its half.
        auto total = [&](const f64x4 (&g)[2]) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) sh.stage[wave][0][256 * p + 4 * lane + v] = g[p][v];
            __syncthreads();
            double sum = sh.stage[0][0][tid];
#pragma unroll
            for (int w = 1; w < 8; ++w) sum += sh.stage[w][0][tid];
            return sum * scale;
        };
        const double sIJ = total(gIJ);
        mine.S[gi][16 + gj] = sIJ;
        mine.S[16 + gj][gi] = sIJ;
        if (inside) {
            __syncthreads();
            mine.S[gi][gj] = total(gII);
            __syncthreads();
            mine.S[16 + gi][16 + gj] = total(gJJ);
        } else {
            mine.S[gi][gj] = sh.diag[half ? id[1] : id[0]][17 * gi + gj];
            mine.S[16 + gi][16 + gj] = sh.diag[half ? id[3] : id[2]][17 * gi + gj];
        }
        __syncthreads();

        // ---- the rotations of the two pairs; the waves that work them out sit on two SIMDs
        rotate_pair(mine, inside, ((wave & 3) - 2 * half - 1) & 3, reinterpret_cast<f64x2*>(sh.stage[wave][0]), floor2,
                    [&](int block, int i, int j, double v) { sh.diag[block ? (half ? id[3] : id[2]) : (half ? id[1] : id[0])][17 * i + j] = v; }, [] {});
        // (the larger is what was done to the two together, see PairShared::did)
        const int did[2] = {__builtin_amdgcn_readfirstlane(sh.pair[0].did), __builtin_amdgcn_readfirstlane(sh.pair[1].did)};
        const int more = did[0] > did[1] ? did[0] : did[1];
        if (more > touched) touched = more;
        if (more > seen) seen = more;

        // ---- P <- P Q as (Q^T P^T): A operand = Q^T tile, B operand = the columns in registers.  The last time (not of a core that is
        // here for all sweeps) a chunk leaves as soon as it is done.
        const bool leave = inner == 2 && !whole && touched > 0;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (did[p] == 0 && !(p == 1 && leave)) continue;
            double qa[2][8];
#pragma unroll
            for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                for (int s = 0; s < 8; ++s) qa[ct][s] = sh.pair[p].Q[kq + 4 * s][16 * ct + n];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if (t % 2 == 0 && 32 * (wave + 4 * t) >= K) break;        // no rows of this core
                if (did[p] != 0) {
                    f64x4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = acc0;
#pragma unroll
                    for (int s = 0; s < 8; ++s) {
                        const double d = s < 4 ? D[t][4 * p + s] : D[t][8 + 4 * p + s - 4];
                        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[0][s], d, acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[1][s], d, acc1, 0, 0, 0);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) { D[t][4 * p + v] = acc0[v]; D[t][8 + 4 * p + v] = acc1[v]; }
                }
                if (p == 1 && t % 2 == 1 && leave) store_chunk(t / 2, n, kq);
            }
        }
        if (inner == 0) exchange(One{}, Two{});
        else exchange(Two{}, Three{});                    // the second time back to a, b, c, d
    }
    if (tid == 0 && seen == 2) gstore(rotated + sweep, 1);
    if (!whole || seen != 2 || sweep + 1 >= max_sweeps) break;
    seen = 0;
    exchange(One{}, Two{});
    }

    if (!whole) {                                        // (a, b, c, d again; scaled by a power of two)
        const double unscale = 1.0 / scale;
        gstore(diag + (half ? blk[1] : blk[0]) * 256 + 16 * gi + gj, sh.diag[half][17 * gi + gj] * unscale);
        gstore(diag + (half ? blk[3] : blk[2]) * 256 + 16 * gi + gj, sh.diag[2 + half][17 * gi + gj] * unscale);
    }
    if (whole && touched > 0) {
#pragma unroll
        for (int tt = 0; tt < NT / 2; ++tt)
            if (32 * (wave + 8 * tt) < K) store_chunk(tt, n, kq);
    }
}

// Two blocks per work-group, four waves of up to NT row tiles, K <= 64 NT.  Work-groups per compute unit: as many as the registers allow, three or
// two (K = 768: 13.3 ms over 16 decompositions; four blocks, one work-group per compute unit and some registers in memory, 15.0 where two blocks took 12.7).
template <int NT>
__global__ __launch_bounds__(256, (NT <= 6 ? 3 : 2))
void jacobi_pair_kernel(double* cores, int* rotated, int K, int sweep, int round, const LayerDev* __restrict__ layers, const int2* __restrict__ wg_map) {
    // the wave that works the rotations out has no registers for its whole panel meanwhile: its last rows wait in LDS (16 cores of 768 13.3 ms, 15.3
    // with 60 registers spilled to memory)
    constexpr int PARK = NT == 12 ? 32 : NT == 6 ? 16 : 0;
    __shared__ struct __align__(16) { double stage[4][16 * 32]; PairShared pair; double parked[PARK ? PARK : 1][64]; } sh;
    const Core c = find_core(cores, rotated, K, layers, wg_map);
    if (sweep > 0 && c.rotated[sweep - 1] == 0) return;   // the previous sweep found no significant pair: the iteration has converged
    K = c.K;
    const int nb = K >> 4;
    if (round >= nb - 1 || K > 64 * NT) return;
    // circle method: slot 0 pairs block nb - 1 with `round`; slot j pairs (round + j) with (round - j)
    int bI = round + c.slot, bJ = round - c.slot;
    if (c.slot == 0) bI = nb - 1;
    else { if (bI >= nb - 1) bI -= nb - 1; if (bJ < 0) bJ += nb - 1; }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 15, kq = lane >> 4;
    const int gi = wave + 4 * (tid & 3), gj = (tid >> 2) & 15;            // this thread's element of a 16 x 16 tile
    const bool inside = round == 0;
    double* const diagI = c.diag + bI * 256;
    double* const diagJ = c.diag + bJ * 256;
    const double keptI = inside ? 0.0 : gload(diagI + 16 * gi + gj), keptJ = inside ? 0.0 : gload(diagJ + 16 * gi + gj);
    const double frob = frob2(c.trace);
    // columns 4 s + kq of block I in D[t][s], of block J in D[t][4 + s]
    double D[NT][8];
#pragma unroll
    for (int tt = 0; tt < NT / 2; ++tt) {
        if (32 * (wave + 4 * tt) < K) {
            const int row0 = 32 * (wave + 4 * tt) + 2 * n;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int col = 16 * (s < 4 ? bI : bJ) + kq + 4 * (s & 3);
                const f64x2 v = gload(reinterpret_cast<const f64x2*>(c.Ct + (int64_t)col * K + row0));
                D[2 * tt][s] = v[0];
                D[2 * tt + 1][s] = v[1];
            }
        } else {
#pragma unroll
            for (int s = 0; s < 8; ++s) D[2 * tt][s] = D[2 * tt + 1][s] = 0.0;
        }
    }
    const double scale = ldexp(1.0, -__builtin_amdgcn_frexp_exp(frob));
    const double floor2 = kZeroColumn2 * frob * scale;
    double* const stage = sh.stage[wave];
    f64x4 g[3] = {};                                      // IJ, II, JJ
    auto gram = [&](auto all) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t % 2 == 0 && 32 * (wave + 2 * t) >= K) break;
#pragma unroll
            for (int s = 0; s < 8; ++s) stage[stage_addr(n, kq + 4 * s)] = D[t][s];
            wave_lds_fence();
            double a0[4], a1[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a0[q] = stage[stage_addr(4 * q + kq, n)];
                a1[q] = stage[stage_addr(4 * q + kq, 16 + n)];
            }
            wave_lds_fence();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                g[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[q], a1[q], g[0], 0, 0, 0);
                if constexpr (decltype(all)::value) {
                    g[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[q], a0[q], g[1], 0, 0, 0);
                    g[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[q], a1[q], g[2], 0, 0, 0);
                }
            }
        }
    };
    if (inside) gram(std::true_type{});
    else gram(std::false_type{});
    const int role = (wave - (int)((blockIdx.x + blockIdx.y) & 3) - 1) & 3;
    if (PARK && role == 3) {
        const int lane = thread_anew() & 63;
#pragma unroll
        for (int i = 0; i < PARK; ++i) sh.parked[i][lane] = D[NT - 1 - i / 8][i % 8];
    }
    // partial tiles of the four waves, added in wave order (see jacobi_quad_kernel)
    auto total = [&](const f64x4& part) {
#pragma unroll
        for (int v = 0; v < 4; ++v) stage[4 * lane + v] = part[v];
        __syncthreads();
        return (((sh.stage[0][tid] + sh.stage[1][tid]) + sh.stage[2][tid]) + sh.stage[3][tid]) * scale;
    };
    const double sIJ = total(g[0]);
    sh.pair.S[gi][16 + gj] = sIJ;
    sh.pair.S[16 + gj][gi] = sIJ;
    if (inside) {
        __syncthreads();
        sh.pair.S[gi][gj] = total(g[1]);
        __syncthreads();
        sh.pair.S[16 + gi][16 + gj] = total(g[2]);
    } else {
        sh.pair.S[gi][gj] = keptI * scale;
        sh.pair.S[16 + gi][16 + gj] = keptJ * scale;
    }
    __syncthreads();
    rotate_pair(sh.pair, inside, role, reinterpret_cast<f64x2*>(stage), floor2,
                [&](int block, int i, int j, double v) { gstore((block ? diagJ : diagI) + 16 * i + j, v * (1.0 / scale)); },
                [&] {
                    const int lane = thread_anew() & 63;
#pragma unroll
                    for (int i = 0; i < PARK; ++i) D[NT - 1 - i / 8][i % 8] = sh.parked[i][lane];
                });
    {
    const int tid = thread_anew(), lane = tid & 63, n = lane & 15, kq = lane >> 4;
    const int did = __builtin_amdgcn_readfirstlane(sh.pair.did);
    if (did == 0) return;                                 // the columns are what they were
    if (tid == 0 && did == 2) gstore(c.rotated + sweep, 1);

    // ---- P <- P Q as (Q^T P^T); a chunk leaves as soon as it is done
    double qa[2][8];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int s = 0; s < 8; ++s) qa[ct][s] = sh.pair.Q[kq + 4 * s][16 * ct + n];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (t % 2 == 0 && 32 * (wave + 2 * t) >= K) break;
        f64x4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = acc0;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[0][s], D[t][s], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[1][s], D[t][s], acc1, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) { D[t][v] = acc0[v]; D[t][4 + v] = acc1[v]; }
        if (t % 2 == 1) {
            const int row0 = 32 * (wave + 2 * (t - 1)) + 2 * n;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int col = 16 * (s < 4 ? bI : bJ) + kq + 4 * (s & 3);
                gstore(reinterpret_cast<f64x2*>(c.Ct + (int64_t)col * K + row0), f64x2{D[t - 1][s], D[t][s]});
            }
        }
    }
    }
}

// Cores of 32: two blocks, one pair.  The work-group (four waves, of which the first has all rows) holds the whole core and runs all
// sweeps in one launch, the columns in registers throughout.  A launch and a poll of the convergence flags per
// sweep took 129 us for one core of 32, this 41.
__global__ __launch_bounds__(256, 1)
void jacobi_single_pair_kernel(double* cores, int* rotated, int max_sweeps) {
    __shared__ struct __align__(16) { double stage[4][16 * 32]; PairShared pair; } sh;
    constexpr int K = 32;
    double* const Ct = cores + (int64_t)blockIdx.x * core_doubles(K);
    rotated += (int)blockIdx.x * (kMaxSweepsCap + 1);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 15, kq = lane >> 4;
    const double frob = frob2(Ct + core_trace(K));
    // D[t][s] = C[2 n + t][kq + 4 s], in the first wave
    double D[2][8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const f64x2 v = gload(reinterpret_cast<const f64x2*>(Ct + (kq + 4 * s) * K + 2 * n));
        D[0][s] = v[0];
        D[1][s] = v[1];
    }
    const double scale = ldexp(1.0, -__builtin_amdgcn_frexp_exp(frob));
    const double floor2 = kZeroColumn2 * frob * scale;
    for (int sweep = 0;; ++sweep) {
        const int lane = thread_anew() & 63, n = lane & 15, kq = lane >> 4;
        if (wave == 0) {
            f64x4 g[3] = {};
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int s = 0; s < 8; ++s) sh.stage[t][stage_addr(n, kq + 4 * s)] = D[t][s];
            }
            wave_lds_fence();
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double a0 = sh.stage[t][stage_addr(4 * q + kq, n)], a1 = sh.stage[t][stage_addr(4 * q + kq, 16 + n)];
                    g[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, a0, g[0], 0, 0, 0);
                    g[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, a1, g[1], 0, 0, 0);
                    g[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, a1, g[2], 0, 0, 0);
                }
            // result element (i, j) of a tile sits in lane (j, i % 4), register i / 4
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = kq + 4 * v, j = n;
                sh.pair.S[i][j] = g[0][v] * scale;
                const double cross = g[1][v] * scale;
                sh.pair.S[i][16 + j] = cross;
                sh.pair.S[16 + j][i] = cross;
                sh.pair.S[16 + i][16 + j] = g[2][v] * scale;
            }
        }
        __syncthreads();
        rotate_pair(sh.pair, true, (wave - 1) & 3, reinterpret_cast<f64x2*>(sh.stage[wave]), floor2, [](int, int, int, double) {}, [] {});
        const int did = __builtin_amdgcn_readfirstlane(sh.pair.did);
        if (did == 0) break;
        if (wave == 0) {
            double qa[2][8];
#pragma unroll
            for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                for (int s = 0; s < 8; ++s) qa[ct][s] = sh.pair.Q[kq + 4 * s][16 * ct + n];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                f64x4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = acc0;
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[0][s], D[t][s], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[1][s], D[t][s], acc1, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) { D[t][v] = acc0[v]; D[t][4 + v] = acc1[v]; }
            }
        }
        if (tid == 0 && did == 2) gstore(rotated + sweep, 1);
        if (did != 2 || sweep + 1 >= max_sweeps) break;
        __syncthreads();                                 // Q is read, the next sweep's tiles may overwrite
    }
    if (wave == 0) {
#pragma unroll
        for (int s = 0; s < 8; ++s) gstore(reinterpret_cast<f64x2*>(Ct + (kq + 4 * s) * K + 2 * n), f64x2{D[0][s], D[1][s]});
    }
}

}  // namespace

hipError_t launch_jacobi_block_round(const LayerDev* layers, const int2* wg_map, int n_wg, int K_max, bool quad,
                                     int sweep, int round, int max_sweeps, double* cores, int* rotated, hipStream_t s) {
    if (n_wg <= 0) return hipSuccess;
    if (K_max > (quad ? 512 : 768) || (quad && K_max % 64)) return hipErrorInvalidValue;
    const int slots = jacobi_slots(K_max, quad);
    const dim3 grid(cores ? slots : n_wg, cores ? n_wg / slots : 1), block(quad ? 512 : 256);
    if (quad) {
        if (K_max <= 256) hipLaunchKernelGGL((jacobi_quad_kernel<2>), grid, block, 0, s, cores, rotated, K_max, sweep, round, max_sweeps, layers, wg_map);
        else hipLaunchKernelGGL((jacobi_quad_kernel<4>), grid, block, 0, s, cores, rotated, K_max, sweep, round, max_sweeps, layers, wg_map);
    }
    else if (K_max <= 128) hipLaunchKernelGGL((jacobi_pair_kernel<2>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else if (K_max <= 256) hipLaunchKernelGGL((jacobi_pair_kernel<4>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else if (K_max <= 384) hipLaunchKernelGGL((jacobi_pair_kernel<6>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else if (K_max <= 512) hipLaunchKernelGGL((jacobi_pair_kernel<8>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    else hipLaunchKernelGGL((jacobi_pair_kernel<12>), grid, block, 0, s, cores, rotated, K_max, sweep, round, layers, wg_map);
    return hipGetLastError();
}

hipError_t launch_jacobi_single_pair(double* cores, int* rotated, int n, int max_sweeps, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(jacobi_single_pair_kernel, dim3(n), dim3(256), 0, s, cores, rotated, max_sweeps);
    return hipGetLastError();
}

}  // namespace abt
