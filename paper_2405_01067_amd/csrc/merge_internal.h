// Declarations shared by the merge sources: the per-layer device record, the constants of the
// Jacobi iteration and the rotation formula.
#pragma once

#include "common.h"

namespace abt {

constexpr int kInfoInts = 4;      // per layer: sweeps, n_sigma, converged, k'
constexpr int kMaxSweepsCap = 64;
constexpr double kRotateTol = 1e-9;    // |cos| above which a column pair is rotated
// A sweep in which no visited pair had |cos| above kSignifTol ends the iteration.  Every pair above
// kRotateTol was still rotated to orthogonality when visited, and the later rotations of that sweep
// disturb it only in second order: measured on cores of 384 with a falling spectrum a sweep that starts at 1.2e-4 leaves
// 9e-8 behind (about 6 cos^2), so the cosines left at the end are below 1e-6, two orders under the
// 1e-4 the results are held to.  Where values are equal or nearly so their columns turn by any angle in that sweep,
// and what is left can come near kSignifTol itself (eight clusters with relative gaps of 1e-6 to 1e-3: 1e-7 to 2e-4).
constexpr double kSignifTol = 3e-4;
constexpr double kSigmaFloor = 1e-7;   // sigma_i <= floor * sigma_1: singular vectors returned as zero
// A column of C with |c|^2 below kZeroColumn2 ||C||_F^2 (|c| < 1e-9 ||C||_F) is numerically zero
// and is left alone: what it holds is the rounding noise (about 1e-16 ||C||) of the large columns
// it was rotated with, so its angles are noise at the level the convergence test looks at and
// would keep the iteration from ending.  It belongs to a singular value far below
// kSigmaFloor sigma_1 (||C||_F <= sqrt(K) sigma_1).
constexpr double kZeroColumn2 = 1e-18;

constexpr int kGramParts = 16;    // work-groups that share a side's contraction where K = 32

struct LayerDev {
    const float* const* A_ptrs;
    const float* const* B_ptrs;
    int G, mode, m, n, k, K, k_cap, k_fixed;
    float tau;
    int jb, nb;            // Jacobi: columns per block, number of blocks
    float* Abar; float* Bbar;
    double* LA; double* GB; double* LB; double* Ct; double* Yt;
    double* sigma; double* s3; double* s5;
    double* trace;         // [10]: the last eight are partial sums of ||C||_F^2
    double* diag;          // [K / 16][16][16]: Gram matrices of the column blocks between two rounds of a sweep
    double* nrm;           // [K]: squared column norms of the rotated core (colnorm_kernel -> finalize_kernel)
    int* perm;
    double* gparts;        // K = 32: parts of the Gram matrices [A, B][kGramParts][32][32]
    float* PA; float* PB;
    int* rotated;          // [kMaxSweepsCap + 1]
    int* info;             // [kInfoInts]
    float* S_out; int32_t* k_out;
};


typedef __attribute__((ext_vector_type(2))) double f64x2;

__device__ __forceinline__ bool sweep_finished(const LayerDev& L, int sweep) {
    // the previous sweep found no significant pair: the iteration has converged
    return sweep > 0 && L.rotated[sweep - 1] == 0;
}

__device__ __forceinline__ double frob2(const double* trace) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) s += gload(trace + 2 + j);
    return s;
}
__device__ __forceinline__ double frob2(const LayerDev& L) { return frob2(L.trace); }

// Ct, diag and trace of a layer lie behind each other, those of the layers too: where all cores are of one size, the kernels of the
// iteration find theirs without the table.
__host__ __device__ inline int64_t core_diag(int K) { return (int64_t)K * K; }
__host__ __device__ inline int64_t core_trace(int K) { return (int64_t)K * K + 16 * K; }
__host__ __device__ inline int64_t core_doubles(int K) { return (int64_t)K * K + 16 * K + 32; }

// Rotation for a pair with squared norms alpha, beta and inner product gamma; returns false when
// the pair counts as orthogonal.  x' = c x - s y, y' = s x + c y.
// A column whose squared norm is below `floor2` (kZeroColumn2 ||C||_F^2) is numerically zero and
// is left alone (rank-deficient cores).
__device__ __forceinline__ bool jacobi_rotation(double alpha, double beta, double gamma, double floor2,
                                                double& c, double& s, bool& significant, double* tangent = nullptr) {
    const double lim = alpha * beta;
    const double g2 = gamma * gamma;
    significant = false;
    if (!(alpha > floor2) || !(beta > floor2)) return false;
    significant = g2 > (kSignifTol * kSignifTol) * lim;
    if (!(g2 > (kRotateTol * kRotateTol) * lim)) return false;
    // tangent of the rotation angle, the smaller root of t^2 + 2 zeta t - 1 = 0 with
    // zeta = (beta - alpha) / (2 gamma), written so that it costs one square root and one division:
    // t = 2 gamma sign(d) / (|d| + sqrt(d^2 + 4 gamma^2)), d = beta - alpha
    const double d = beta - alpha;
    const double g2x = 2.0 * gamma;
    const double tn = (d >= 0.0 ? g2x : -g2x) / (fabs(d) + sqrt(fma(d, d, g2x * g2x)));
    // c = (1 + t^2)^(-1/2): hardware reciprocal square root refined by two Newton steps (the
    // rotation stays orthogonal to rounding: c^2 + s^2 = c^2 (1 + t^2))
    const double w = fma(tn, tn, 1.0);
    double y = __builtin_amdgcn_rsq(w);
    y = y * fma(-0.5 * w, y * y, 1.5);
    y = y * fma(-0.5 * w, y * y, 1.5);
    c = y;
    s = c * tn;
    if (tangent) *tangent = tn;
    return true;
}

__device__ __forceinline__ double lane_value(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}

// Factor a 32 x 32 block in one wave: lane r (and r + 32) holds row r; step c takes the pivot and the
// finished column c from the other lanes with lane reads (no LDS, no waits).  keep(c, 1 / pivot or 0).
template <class F>
__device__ __forceinline__ void factor_diagonal_block(double (&row)[32], int r, double floor_piv, F&& keep) {
#pragma unroll
    for (int c = 0; c < 32; ++c) {
        const double d = lane_value(row[c], c);
        const bool ok = d > floor_piv;
        // 1 / sqrt(d): hardware estimate and two Newton steps (a square root and a division in
        // fp64 would be several times the rest of the step); the pivot itself is d / sqrt(d)
        const double dd = ok ? d : 1.0;
        double y = __builtin_amdgcn_rsq(dd);
        y = y * fma(-0.5 * dd, y * y, 1.5);
        y = y * fma(-0.5 * dd, y * y, 1.5);
        const double ip = ok ? y : 0.0;
        const double piv = ok ? dd * y : 0.0;
        const double v = (r == c) ? piv : (r > c ? row[c] * ip : 0.0);
        row[c] = v;
        keep(c, ip);
#pragma unroll
        for (int cc = c + 1; cc < 32; ++cc) row[cc] = fma(-v, lane_value(v, cc), row[cc]);
    }
}

// Average of the copies + Gram matrices (merge_gram.hip): one work-group per job; layer < 0 marks
// an empty slot; (ti, tj), ti >= tj, is a 128 x 128 tile of the lower triangle; which = 0: G_A
// (stored into LA), 1: G_B (stored into GB and LB).  The diagonal tiles also write Abar / Bbar.
struct GramJob { int layer, which, ti, tj; };
// `jobs` holds njobs entries for the kernel with 16-byte loads, then njobs_unaligned entries (B sides
// whose row length n is not a multiple of four) for the element-wise one.
hipError_t launch_mean_gram(const LayerDev* layers, const GramJob* jobs, int njobs, int njobs_unaligned, hipStream_t s);

// One round of the block Jacobi iteration for cores with K <= 768 (every layer of the batch): `n_wg` work-groups,
// wg_map[i] = (layer, slot), jacobi_slots() slots a layer, jacobi_rounds() rounds a sweep: `quad` pairs double blocks of 32 columns
// (K_max up to 512, every K a multiple of 64), otherwise blocks of 16.  Round 0 of a sweep also orthogonalises the columns inside every (double) block.  `cores`: the first core's record where the launch has whole layers one behind the other, all of size K_max, whose
// convergence flags begin at `rotated` (otherwise null, and the work-groups look everything up in the tables).  max_sweeps: 0, or, with `quad` where all
// cores are 64 wide (and `cores` is given), the number of sweeps that the launch may make.
inline int jacobi_slots(int K, bool quad) { return quad ? K / 64 : K / 32; }
inline int jacobi_rounds(int K, bool quad) { return 2 * jacobi_slots(K, quad) - 1; }
hipError_t launch_jacobi_block_round(const LayerDev* layers, const int2* wg_map, int n_wg, int K_max, bool quad,
                                     int sweep, int round, int max_sweeps, double* cores, int* rotated, hipStream_t s);

// All sweeps of `n` layers with K = 32 (every layer of the batch): one work-group per layer, one launch.
hipError_t launch_jacobi_single_pair(double* cores, int* rotated, int n, int max_sweeps, hipStream_t s);

// The stages around it where every core is 32 wide and no layer a dense weight (merge_small.hip): averages and parts of the Gram matrices;
// Cholesky factors and core; values, rank and projections.
hipError_t launch_gram32(const LayerDev* layers, int L, hipStream_t s);
hipError_t launch_core32(const LayerDev* layers, int L, hipStream_t s);
hipError_t launch_finish32(const LayerDev* layers, int L, int max_sweeps, hipStream_t s);

}  // namespace abt
