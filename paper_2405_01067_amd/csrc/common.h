// Shared declarations of the HIP side: vector types for the gfx950 MFMA builtins, bf16
// conversion, and the launcher prototypes that api.hip calls.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "abtrain.h"

namespace abt {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) double f64x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int kWave = 64;

// Loads and stores through a pointer known to point into device memory.  A pointer read from a table
// is generic to the compiler, which then emits FLAT instructions; those count in the LDS counter as
// well as in the memory counter, so every wait for an LDS read would also wait for all global loads
// in flight (prefetches included).  These helpers emit GLOBAL instructions.
template <typename T>
__device__ __forceinline__ T gload(const T* p) {
    return *(const __attribute__((address_space(1))) T*)(p);
}
template <typename T>
__device__ __forceinline__ void gstore(T* p, const T& v) {
    *(__attribute__((address_space(1))) T*)(p) = v;
}

// Two fp32 -> packed bf16 (low half = lo), round-to-nearest-even: one v_cvt_pk_bf16_f32 on gfx950.
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Buffer addressing: a wave-uniform 128-bit descriptor (base, byte count) + wave-uniform byte
// offset + one 32-bit byte offset per lane.  Accesses past the byte count read zeros / are dropped.
// Only the per-lane offset is range-checked, not the wave-uniform one.  A byte count beyond
// kBufMaxBytes is clamped to it: per-lane offsets must stay below that (callers check sizes on the
// host), and kBufNowhere is a per-lane offset that no descriptor covers.
using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr int kBufMaxBytes = 0x7ffffff0;
constexpr int kBufNowhere = 0x7ffffff0;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, int64_t bytes) {
    const int n = bytes > kBufMaxBytes ? kBufMaxBytes : (bytes < 0 ? 0 : (int)bytes);
    // last word: raw buffer, 32-bit data format field as the gfx9 family expects for untyped access
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, n, 0x00020000);
}
__device__ __forceinline__ u32x4 buf_load16(rsrc_t r, int lane_off, int wave_off) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, wave_off, 0);
}
// A 16-byte store reads its data registers for a few cycles after it has issued, and the compiler
// does not keep the next instructions away from them when the wave-uniform offset is a register
// (seen: the address of the next store, written into the first data register one instruction after
// the store, went to memory in place of the data).  Nothing may follow for eight wait states: 64 lanes
// of 16 bytes leave the register file at 64 bytes per cycle.
__device__ __forceinline__ void store_data_guard() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void buf_store16(u32x4 v, rsrc_t r, int lane_off, int wave_off) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, lane_off, wave_off, 0);
    store_data_guard();
}

// A store with the non-temporal hint, for results that a launch writes once and that are too large
// to be found in the last-level cache by whoever reads them next: such lines should not push the
// factors, which every work-group re-reads, out of L2.  (The hint on the loads of the activations
// measured slower than plain loads; on the stores it is worth 6 % of a config-3 step.)
__device__ __forceinline__ void buf_store16_stream(u32x4 v, rsrc_t r, int lane_off, int wave_off) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, lane_off, wave_off, 2);
    store_data_guard();
}
// `stream` is uniform over the launch
__device__ __forceinline__ void buf_store16_maybe_stream(bool stream, u32x4 v, rsrc_t r, int lane_off, int wave_off) {
    if (stream) buf_store16_stream(v, r, lane_off, wave_off);
    else buf_store16(v, r, lane_off, wave_off);
}
// Outputs (Yout and Tout of the chain kernels) of this many bytes or more are stored with the hint: a quarter of
// the 256 MB last-level cache.  Counted per problem of a grouped launch; the parities and channel blocks of one image
// are one output.
constexpr int64_t kStreamOutBytes = 64ll << 20;

// ---- what the kernels share that load straight to LDS without a barrier per load (lr_few.hip, lr_pair.hip)
__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// All but the newest N global accesses of this wave (loads, loads to LDS, stores) have completed: they are counted off in the order of issue, on which
// the compiler relies too (a load with two stores behind it is waited for with two left).
template <int N>
__device__ __forceinline__ void wait_newest() {
    static_assert(N >= 0 && N < 64, "six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
    asm volatile("" ::: "memory");
}
// this wave's LDS traffic has completed, then s_barrier (global accesses stay in flight)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// 1 KB: lane l's 16 bytes go to LDS address dst + 16 l
__device__ __forceinline__ void load_lds16(rsrc_t r, unsigned char* dst, int lane_off, int wave_off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, lane_off, wave_off, 0, 0);
}
// Row i of a block of 32 of the first MFMA operand is matrix row out_row(i): the 16 accumulators of a lane are then
// 16 consecutive columns of the result, 16 (lane / 32) .. + 15.
__device__ __forceinline__ int out_row(int i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
// Do two byte ranges share memory?  (A caller may hand in an output that lies over an input, as far as everything
// that reads the input is done before the output is written.)
inline bool overlap(const void* a, int64_t na, const void* b, int64_t nb) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return a && b && x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
}

// ------------------------------------------------------------------ bf16 factored layer
// Fused chain  Tout[M,R] = Xin[M,p] . P[R,p]^T ;  Yout[M,q] = Tout . Q[q,R]^T  (bf16, fp32 acc).
// Yout or Tout may be NULL.  p, q multiples of 64; R in {32..384 step 32}.
// With 64-row work-groups: four MFMA waves fed by four loader waves; covers
// R in {32, 64, 96, 128, 160, 192, 256, 320, 384} with p a multiple of 64 and p, q <= 2^20
// (32-bit byte offsets inside a work-group's rows and inside the factors) (chain2_supports).
bool chain2_supports(int R, int p, int q);
hipError_t launch_chain2_bf16(const void* Xin, const void* P, const void* Q, void* Yout, void* Tout,
                              int64_t M, int p, int q, int R, hipStream_t s);
// The same chain with 128-row work-groups (eight MFMA waves in two row groups fed by four loader
// waves): every slab of a factor serves twice the rows.  R in {32, 64, 96, 128, 192}.  With
// parts > 1 the grid gets that many work-groups per row block, each doing its share of the output
// tiles of stage 2 after repeating stage 1 (for batches too small to fill the chip otherwise).
bool chain2_tall_supports(int R, int p, int q);
hipError_t launch_chain2_tall_bf16(const void* Xin, const void* P, const void* Q, void* Yout, void* Tout,
                              int64_t M, int p, int q, int R, int parts, hipStream_t s);
// (From R = 192 on the plain 128-row launches go to the kernel of eight equal waves below; the
// gathered form has 128-row work-groups for R in {32, 64, 96, 128, 192, 384}.)
// Up to kChainMaxGroups problems of one shape in one launch (the emulated groups of a training step).
// rows = 64 or 128 (work-group height; the caller has checked chain2_supports / chain2_tall_supports);
// Yout must be NULL for all problems or for none; a problem with Yout == Tout == NULL is skipped.
constexpr int kChainMaxGroups = 8;
struct ChainProblem { const void* Xin; const void* P; const void* Q; void* Yout; void* Tout; };
hipError_t launch_chain2_grouped_bf16(const ChainProblem* problems, int G, int64_t M, int p, int q, int R,
                                      int rows, int parts, hipStream_t s);
// The same chain for R = 192 .. 384 with 128-row work-groups of eight equal waves, slabs loaded
// straight into LDS; p, q multiples of 64, at most 2^20; `parts` as above; groups as above.
bool chain3_supports(int R, int p, int q);
hipError_t launch_chain3_bf16(const ChainProblem* problems, int G, int64_t M, int p, int q, int R, int parts, hipStream_t s);
// The same chain with the first operand gathered from a channels-last image [images, H, W, Cin]
// instead of read from a matrix: row i of the virtual operand is the kh x kw patch around a pixel
// (zero outside the image), columns ordered (tap, channel) with every tap padded to a multiple of
// 64 channels: p = kh kw ceil(Cin / 64) 64 columns, which is the row length of P [R, p].
// Rows are the pixels of a grid RH x RW per image (M = images RH RW); row (y, x) is centred on image
// pixel (mul y, mul x) and tap (ky, kx) reads the position sign (ky - kh/2, kx - kw/2) away from it,
// which with shift = 1 exists only where both coordinates are even, as pixel (ty / 2, tx / 2):
//   patches, stride 1:        RH x RW = H x W, mul = 1, shift = 0, sign = +1
//   patches, stride 2:        RH x RW = output grid, mul = 2, shift = 0, sign = +1
//   adjoint gather, stride 1: the same with sign = -1
//   adjoint gather, stride 2: image = gradient on the output grid, RH x RW = input grid, mul = 1,
//                             shift = 1, sign = -1 (only where a work-group height is forced, which the tests of the form
//                             by parity compare it with, and where a parity's window is beyond 32-bit offsets).
// Tout rows are t_pitch elements apart (>= R).
struct PatchGeom { int H, W, Cin, kh, kw, sign, RH, RW, mul, shift; };
hipError_t launch_chain2_gather_bf16(const void* image, const PatchGeom& g, const void* P, const void* Q,
                                     void* Yout, void* Tout, int t_pitch, int64_t M, int q, int R, hipStream_t s);
hipError_t launch_chain2_tall_gather_bf16(const void* image, const PatchGeom& g, const void* P, const void* Q,
                                     void* Yout, void* Tout, int t_pitch, int64_t M, int q, int R, hipStream_t s);
// The same chain for R <= 192 with work-groups of four waves and `rows` rows (a multiple of four, at most 128),
// two or three per compute unit; p, q multiples of 64, at most 2^20.  With parts > 1 a row block is shared by that many work-groups, each
// repeating stage 1 and doing its share of the 64-column output tiles (parts <= q / 64, second stage only).  Rows of Tout
// are t_pitch elements apart (>= R).
bool chain4_supports(int R, int p, int q);
hipError_t launch_chain4_bf16(const ChainProblem* problems, int G, int64_t M, int p, int q, int R, int t_pitch, int rows, int parts, hipStream_t s);
// Its gathered form, up to kChainMaxGroups problems of one R and q in a launch.  As PatchGeom, but the
// window may have any size and centre: tap (ky, kx) reads the image pixel sign (ky - cy, kx - cx) away from the
// centre (mul y, mul x) of grid row (y, x); an image of height 0 reads as zeros everywhere.  Row (y, x) of
// the result is pixel (omul y + oy, omul x + ox) of a grid OH x OW (omul = 2 without a second stage only).
struct ChainGather { int H, W, Cin, cpb, kh, kw, sign, cy, cx, RH, RW, mul, omul, oy, ox, OH, OW; };   // cpb: set by the launcher
struct GatherProblem { const void* image; const void* P; const void* Q; void* Yout; void* Tout; int64_t M; ChainGather g; };
// Does it read this image through a window in LDS?  Two taps or more, stride 1; one block of 64 channels, or several with nine taps;
// no more pixels touched by a row block's patches than window_fits allows, and at R = 128 with one block no more than 192 (three
// work-groups share a compute unit up to 168, two beyond; the gathered form has three; forward, us, window / gathered:
// 31 x 31 x 64, 64387 rows, 192 pixels 19.1 / 22.7, 56 x 56 x 64, batch 64, 242 pixels 57 / 55); not wide results of 32
// channels, the other half of whose slabs is zeros (activation gradient of 28 x 28 x 128, r = 32, batch 256 61 / 58).
bool chain4_window(const ChainGather& g, int R, int rows);
hipError_t launch_chain4_gather_bf16(const GatherProblem* problems, int n, int q, int R, int t_pitch, int rows, int parts, hipStream_t s);
// dst[c, r] = src[r, c] for a bf16 matrix of `rows` x `cols`.
struct TransposeJob { const void* src; void* dst; int rows, cols; };   // dst[cols, rows] = src[rows, cols]^T
constexpr int kTransposeMaxJobs = 16;   // per launch
hipError_t launch_transpose_bf16(const TransposeJob* jobs, int njobs, hipStream_t s);
// part[split][P,Q] = U[rows of split, P]^T . V[rows of split, Q]  (bf16 in, fp32 partials)
// followed by out[P,Q] (+)= sum over splits, in fixed order.  One of P, Q equals R.
// job: out[P,R] = U[M,P]^T . V[M,R]; with transposed != 0 the result is stored as out[R,P].
struct TnJob {
    const void* U; const void* V; float* out; int P; int transposed;
};
constexpr int kTnMaxJobs = 16;   // per launch (all with the same M and R)
size_t tn_partials_bytes(int64_t M, const TnJob* jobs, int njobs, int R, bool gather = false);
hipError_t launch_tn_bf16(const TnJob* jobs, int njobs, int64_t M, int R, int accumulate,
                          float* partials, hipStream_t s);
// out (+)= sums, which lie end to end in the order of the jobs (their operands are not looked at)
hipError_t launch_tn_finish(const TnJob* jobs, int njobs, int R, int accumulate, const float* sums, hipStream_t s);

// The chain of many rows as two products (lr_pair.hip), T and Y or T alone (Yout NULL, for all problems or none); Tout must have a place that lies
// over no input.  The rows per work-group are those of a launch of `of` problems (at least G).
bool pair_supports(int64_t M, int p, int q, int R);
hipError_t launch_pair_bf16(const ChainProblem* problems, int G, int of, int64_t M, int p, int q, int R, hipStream_t s);

// The chain of a few rows in one launch, R <= 192 (lr_few.hip): T, Y or both (Yout NULL for all problems or none); neither may lie over an input.
bool few_supports(int64_t M, int p, int q, int R);
hipError_t launch_few_fwd(const ChainProblem* problems, int G, int64_t M, int p, int q, int R, hipStream_t s);
bool few_gather_supports(const PatchGeom& g, int64_t M, int q, int R);      // the rows of an image's patch matrix
hipError_t launch_few_fwd_gather(const ChainProblem& c, const PatchGeom& g, int64_t M, int q, int R, hipStream_t s);

// 32-bit offsets: M, m, n and r against each other
bool lr_small_supports(int64_t M, int m, int n, int r);
// The chain for few rows as two products, T and Y or T alone (Yout NULL, for all problems or none); Tout must have a place that lies over no input.
// The tile and the split of the contraction are those of a launch of `of` problems (at least G).
hipError_t launch_lr_small_fwd(const ChainProblem* problems, int G, int of, int64_t M, int p, int q, int R, hipStream_t s);
// first operand gathered from an image: sign = +1, shift = 0
bool lr_small_gather_supports(const PatchGeom& g, int64_t M, int q, int R);
hipError_t launch_lr_small_fwd_gather(const void* image, const PatchGeom& g, const void* P, const void* Q, void* Yout, void* Tout, int64_t M, int q, int R,
                                      hipStream_t s);

// Backward for few rows in two launches: dT = dY A, then dX = dT B, dA = dY^T T and dB = dT^T X together (NULL: not wanted; none
// may lie over what another reads).
hipError_t launch_lr_small_dt(const void* dY, const void* A, void* dT, int64_t M, int m, int r, hipStream_t s);
hipError_t launch_lr_small_grad(const void* dY, const void* X, const void* T, const void* B, void* dX, float* dA, float* dB, const void* dT,
                                int64_t M, int m, int n, int r, int accumulate, hipStream_t s);
// The same for a convolution (dAct [N, H, W, C] in the place of dX; image and factor as they lie), M = N Ho Wo rows, at most 16384.
struct ConvShape { int N, H, W, Ho, Wo, C, kh, kw, stride; };
bool lr_small_conv_supports(const ConvShape& g, int64_t M, int m, int r);
hipError_t launch_lr_small_conv_grad(const ConvShape& g, const void* dY, const void* act, const void* T, const void* B, void* dAct, float* dA, float* dB,
                                     const void* dT, int64_t M, int m, int r, int accumulate, hipStream_t s);

// Pst [C, taps r_pad] (bf16) from B [r, taps C]: Pst[c, tap r_pad + j] = B[j, tap C + c], zero for j >= r.
// by_parity: four matrices end to end instead, one per parity (py, px) of the pixel in the order (0,0), (0,1),
// (1,0), (1,1), each [C, taps of that parity r_pad] with the taps ky = py + kh/2 (mod 2), kx = px + kw/2 (mod 2).
// Together with At [r, m] = A^T; A or B may be NULL (not wanted).
hipError_t launch_conv_factors_bf16(const void* A, void* At, int m, const void* B, void* Pst, int r, int C, int kh, int kw, int r_pad, bool by_parity,
                                    hipStream_t s);
// taps of one parity along one axis of a window of k taps (centre k / 2): first, first + 2, ..; count may be 0
inline __host__ __device__ int parity_first(int k, int parity) { return (parity + k / 2) & 1; }
inline __host__ __device__ int parity_count(int k, int parity) { const int f = parity_first(k, parity); return f < k ? (k - f + 1) / 2 : 0; }
// One or two jobs; the U of the LAST one is the patch matrix of a channels-last image (g.sign is
// ignored: always +1): column tap Cin + c of row i is channel c of pixel (y + ky - kh/2, x + kx - kw/2),
// and its P = kh kw Cin.  A job before it is a plain one.  Partials as for launch_tn_bf16.
hipError_t launch_tn_gather_bf16(const TnJob* jobs, int njobs, const PatchGeom& g, int64_t M, int R, int accumulate,
                                 float* partials, hipStream_t s);

// ------------------------------------------------------------------ fp32 GEMM (MFMA)
// C[P,Q] = alpha * op(A) . op(B) (+ C if accumulate).  op(A) is P x K: transA == 0 reads
// A[P,K] (lda = row length), else A[K,P].  op(B) is K x Q: transB == 0 reads B[K,Q], else B[Q,K].
// col_limit: optional device int; output columns >= *col_limit are written as zero without
// being computed (rows when limit_rows != 0).
struct GemmF32 {
    const float* A; const float* B; float* C;
    int P, Q, K;
    int lda, ldb, ldc;
    int transA, transB;
    int accumulate;
    float alpha;
    const int32_t* limit;   // may be NULL
    int limit_rows;
};
// Up to four problems in one launch, descriptors in the kernel arguments.  splits[i] > 1 (NULL = 1
// everywhere) splits problem i's contraction over work-groups; its partial sums
// (gemm_f32_partial_bytes each, laid end to end in `partials`) are added in a fixed order by a second
// launch.  gemm_f32_splits is the split that fills the chip.
int gemm_f32_splits(const GemmF32& d);
// The split of dT: few columns, a contraction over a width of the layer.
int gemm_f32_row_splits(const GemmF32& d);
size_t gemm_f32_partial_bytes(const GemmF32& d, int splits);
hipError_t launch_gemm_f32(const GemmF32* problems, const int* splits, int n, float* partials, hipStream_t s);
hipError_t launch_gemm_f32_one(const GemmF32& d, hipStream_t s);
// Are the sums of the first problem in the order of launch_gemm_f32_one, if it is not split?
bool gemm_f32_first_as_alone(const GemmF32* problems, const int* splits, int n);
// n problems in one launch: build the table on the host (n * gemm_f32_desc_bytes() bytes), copy it to the
// device, then launch from the device copy.
struct GemmF32Table { int n, tiles; bool small, vec; };
size_t gemm_f32_desc_bytes();
GemmF32Table gemm_f32_build_table(const GemmF32* descs_host, int n, void* host_image);
hipError_t launch_gemm_f32_table(const void* dev_image, const GemmF32Table& t, hipStream_t s);

// The smallest fp32 layers in one launch each way (layer_f32_small.hip).  No output may lie over an input; T (or NULL) as in the other calls, but
// dA needs it.
bool tiny_f32_supports(int64_t M, int64_t m, int64_t n, int64_t r);
hipError_t launch_tiny_f32_fwd(const float* X, const float* A, const float* B, float* Y, float* T, int64_t M, int64_t m, int64_t n, int64_t r, hipStream_t s);
hipError_t launch_tiny_f32_bwd(const float* dY, const float* X, const float* T, const float* A, const float* B, float* dX, float* dA, float* dB,
                               int64_t M, int64_t m, int64_t n, int64_t r, int accumulate, hipStream_t s);

// ------------------------------------------------------------------ merge
// Host-side plan of a batched merge: validates nothing (api.hip does), lays out the workspace
// and enqueues every stage.
size_t merge_workspace_bytes(const abt_merge_desc* layers, int L);
// identity: per layer the side whose (only) copy is the K x K identity, i.e. the layer is a dense weight; NULL: none
enum class MergeSide : uint8_t { none, A, B };
// A merge cannot be captured in a graph: the host decides between sweeps.  (The smallest ones do not come to a call that a capture would refuse.)
bool merge_stream_captures(hipStream_t s);
hipError_t merge_run(const abt_merge_desc* layers, const MergeSide* identity, int L, void* workspace, int max_sweeps, hipStream_t s);
// (sweeps, values, converged, rank) of `count` layers of the last merge on this workspace (waits for the stream); hipErrorInvalidValue: not a
// merge workspace, or no such layers in it.
hipError_t merge_read_info(const void* workspace, int first, int count, std::vector<int32_t>& out, hipStream_t s);
hipError_t launch_identity_f32(float* dst, int K, hipStream_t s);   // dst[K, K] = I
// Stage timers of the batched merge: with the switch on, merge_run records events on the caller's
// stream at its stage boundaries and merge_stage_ms waits for the last and returns the elapsed
// milliseconds of the ABT_MERGE_STAGES stages (hipErrorNotReady if no timed merge has run).
int merge_set_stage_timing(int on);
hipError_t merge_stage_ms(float out[ABT_MERGE_STAGES]);
int merge_set_groups(int n);   // upper bound on the layer groups (streams) of the Jacobi stage; returns the previous one

// ------------------------------------------------------------------ optimiser step
// Adam with decoupled weight decay on up to any number of tensors (kAdamwMaxTensors per launch).
constexpr int kAdamwMaxTensors = 48;
struct AdamwTensor {
    float* param; const float* grad; float* exp_avg; float* exp_avg_sq; uint16_t* param_bf16; int64_t count;
};
struct AdamwHyper {   // everything the kernel needs, prepared on the host in double precision
    float beta1, beta2, one_minus_beta1, one_minus_beta2;
    float inv_bc1;        // 1 / (1 - beta1^step)
    float inv_sqrt_bc2;   // 1 / sqrt(1 - beta2^step)
    float eps, eta, weight_decay;   // eta = lr * lr_scale
};
hipError_t launch_adamw(const AdamwTensor* tensors, int n, const AdamwHyper& h, hipStream_t s);

}  // namespace abt
