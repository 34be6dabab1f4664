// The chain of many rows as two products, each a kernel of its own:
//   contract   T[M,R] = X[M,p] . P[R,p]^T     the whole width of T stays in accumulators, X streams through LDS once
//   expand     Y[M,q] = T[M,R] . Q[q,R]^T     a wave keeps 64 rows of Q in registers, T streams past them
// (bf16 in and out, fp32 accumulators).  A fused work-group has to stream both factors past its 64 or 128 rows, and its rows come in whole
// blocks: 50432 rows are 394 work-groups of 128 on 256 compute units.  Here Q is read once per work-group whatever its rows, and contract shares
// out the rows of the batch evenly, 8 at a time; what it costs is the second launch and T read again, from the cache.
// Alone, M = 50432, buffers in turn, in brackets the share of the bytes' time at the 5.9 and 6.8 TB/s of launches that only read or only write, as these
// nearly do (a copy, half of each, moves 4.8 TB/s):
//                          r = 96           r = 192          r = 384
//   contract, p = 3072     63 us (0.85)     83 us (0.67)     134 us: 890 TFLOP/s
//   expand, q = 3072       57 us (0.83)     66 us (0.75)     119 us: 1000 TFLOP/s
// Products of random values alone, operands in registers, run at 1200 to 1500 TFLOP/s on this card (the clock falls).
#include <atomic>
#include <type_traits>

#include "common.h"

namespace abt {

namespace {

// f(0), .., f(N - 1) with constants: at wide ranks the loops below are beyond what the compiler unrolls, and an array of registers with
// an index that is not a constant goes to memory
template <int I, int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<I + 1, N>(f);
    }
}

struct PairPtrs {
    const uint16_t* in[kChainMaxGroups];     // X or T
    const uint16_t* f[kChainMaxGroups];      // P or Q
    uint16_t* out[kChainMaxGroups];          // T or Y
};

// ------------------------------------------------------------------------------------------ expand
// A wave owns 64 columns of Y and keeps their rows of Q as MFMA operands (R / 2 registers a lane), four waves side by side a work-group's 256 columns; up to
// r = 192 two such groups share a work-group and its slots of T, beyond a wave needs the registers of two.  One work-group per compute unit walks over its rows:
// slots of 64 or 128 rows of T come straight to LDS one or two ahead, one barrier per slot, and the finished block of 32 rows leaves piece by piece between
// the MFMA steps of the next: through 4 KB of LDS of the wave's own, as whole 128-byte lines.
// Bound by the stores up to r = 128 or so, beyond by the matrix units, neither quite beside the other (r = 192, 50432 x 3072: 67 us, 54 without the products,
// 50 without the stores).  Tried: Q straight from memory as operands (32 rows per load instruction: 7 us more per launch), two work-groups of four waves per
// compute unit (the same time, Q read twice), six or eight T operands in flight (slower).
template <int R>
struct ExCfg {
    static constexpr int RG = R <= 192 ? 2 : 1;           // row groups of four waves: 256 or 512 registers a lane
    static constexpr int NW = 4 * RG, NT = 64 * NW;
    static constexpr int KB = R / 16;                     // MFMA steps of a block of 32 rows
    static constexpr int NB = 4;                          // T operands in flight
    static constexpr int CH = 64 * RG;                    // rows of T per slot
    static constexpr int slot = CH * R * 2;
    static constexpr int NL = slot / (1024 * NW);         // load instructions per wave and slot
    static constexpr int stage = NW * 4096;               // 32 x 64 values per wave on their way out
    static constexpr int NS = R == 192 ? 2 : 3;
    static constexpr int PH = slot + 512 * R <= 160 * 1024 ? 1 : 2;            // Q comes through LDS behind the first slot, in two halves if too large
    static constexpr int qbytes = 512 * R / PH, NQ = qbytes / (1024 * NW);
    static constexpr int lds = NS * slot + stage > slot + qbytes ? NS * slot + stage : slot + qbytes;
    static constexpr int CPR = R / 8;                     // 16-byte chunks per row of T
    static constexpr int NV = R % 128 == 0 ? 8 : R % 64 == 0 ? 4 : 2;          // steps after which the swizzle repeats
    static_assert(lds <= 160 * 1024 && NL * 1024 * NW == slot && NQ * 1024 * NW == qbytes && (2 * KB) % NB == 0, "");
    // chunk c of row i lies at position c ^ swz(i): the same chunk of sixteen neighbouring rows in all of the 256 bytes of banks
    static __device__ __forceinline__ int swz(int i) { return R % 128 == 0 ? i & 15 : R % 64 == 0 ? (i >> 1) & 7 : (i >> 2) & 3; }
};

template <int R, bool STREAM>
__global__ __launch_bounds__(ExCfg<R>::NT) void expand_kernel(PairPtrs ptrs, int M, int q, int ncol, int nrow, int each) {
    using L = ExCfg<R>;
    constexpr int KB = L::KB, NB = L::NB, NS = L::NS, NL = L::NL, CPR = L::CPR, NW = L::NW;
    extern __shared__ __align__(1024) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rg = wave >> 2;
    const int lj = lane & 31, lh = lane >> 5;
    // each XCD takes a contiguous eighth of the (group, rows, columns): the column groups of a row range share its rows of T in one L2
    int w = blockIdx.x;
    {
        const int nb = gridDim.x, xcd = w & 7, i = w >> 3, per = nb >> 3, rem = nb & 7;
        w = xcd * per + (xcd < rem ? xcd : rem) + i;
    }
    const int g = w / (ncol * nrow);
    w -= g * (ncol * nrow);
    const int rs = w / ncol, cg = w - rs * ncol;
    const uint16_t* const T = ptrs.in[g];
    const uint16_t* const Q = ptrs.f[g];
    uint16_t* const Y = ptrs.out[g];
    const int nch = (M + L::CH - 1) / L::CH;
    const int ch0 = rs * each, ch1 = ch0 + each < nch ? ch0 + each : nch;
    const int col0 = (cg * 4 + (wave & 3)) * 64;
    const bool have = col0 < q;

    int voff[NL];
#pragma unroll
    for (int j = 0; j < NL; ++j) {
        const int pos = 64 * (wave + NW * j) + lane, row = pos / CPR, c = (pos - row * CPR) ^ L::swz(row);
        voff[j] = (row * CPR + c) * 16;
    }
    auto issue = [&](int ch, int at) {
        const int rows = M - ch * L::CH < L::CH ? M - ch * L::CH : L::CH;
        const rsrc_t tr = make_rsrc(T + (int64_t)ch * (L::CH * R), rows * (R * 2));
        unsigned char* dst = lds + at * L::slot + wave * 1024;
#pragma unroll
        for (int j = 0; j < NL; ++j) load_lds16(tr, dst + j * (NW * 1024), voff[j], 0);
    };
    issue(ch0, 0);
    // this wave's 64 rows of Q as MFMA operands; whole rows come to LDS
    u32x4 qf[2][KB];
    {
        const int rows = q - cg * 256 < 256 ? q - cg * 256 : 256;
        const rsrc_t qr = make_rsrc(Q + (int64_t)cg * (256 * R), rows * (R * 2));
        unsigned char* const qs = lds + L::slot;
#pragma unroll
        for (int ph = 0; ph < L::PH; ++ph) {
#pragma unroll
            for (int j = 0; j < L::NQ; ++j) {
                const int pos = 64 * (wave + NW * j) + lane, row = pos / CPR, c = (pos - row * CPR) ^ L::swz(row);
                const int from = L::PH == 1 ? row : (row >> 5) * 64 + 32 * ph + (row & 31);
                load_lds16(qr, qs + (wave + NW * j) * 1024, (from * CPR + c) * 16, 0);
            }
            wait_newest<0>();
            lds_barrier();
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                if (L::PH == 2 && b != ph) continue;
                const int row = (wave & 3) * (64 / L::PH) + (L::PH == 1 ? 32 * b : 0) + out_row(lj);
#pragma unroll
                for (int kk = 0; kk < KB; ++kk) qf[b][kk] = *reinterpret_cast<const u32x4*>(qs + row * (R * 2) + (((2 * kk + lh) ^ L::swz(row)) * 16));
            }
            lds_barrier();                                // read: the next half or the next slots may come
        }
    }
    if (NS > 2 && ch0 + 1 < ch1) issue(ch0 + 1, 1);
    // operand kk of the rows 32 blk ..: chunk 2 kk + lh of row lj
    int tbase[L::NV];
#pragma unroll
    for (int j = 0; j < L::NV; ++j) tbase[j] = (64 * rg + lj) * (R * 2) + (((2 * j + lh) ^ L::swz(lj)) * 16);
    unsigned char* const stg = lds + NS * L::slot + wave * 4096;
    const int sw = (lj >> 1) & 7;
    // a piece leaves as 8 rows of 128 bytes
    const int out_off = ((lane >> 3) * q + (lane & 7) * 8) * 2;
    unsigned char* const rd = stg + (lane >> 3) * 128;   // chunk c of row i at position c ^ ((i >> 1) & 7)

    u32x4 ring[NB], piece[4];
    f32x16 acc[2][2];
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NB; ++i) ring[i] = u32x4{0, 0, 0, 0};
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[x][b] = zero;
    auto yres = [&](int ch, int blk) {                    // rows 32 blk .. of a chunk; nothing for a chunk before the first
        const int64_t row = (int64_t)ch * L::CH + 64 * rg + 32 * blk;
        const int rows = M - row < 32 ? (int)(M - row) : 32;
        const bool ok = have && ch >= ch0 && rows > 0;
        return make_rsrc(Y + (ok ? row * q + col0 : 0), ok ? ((int64_t)(rows - 1) * q + 64) * 2 : 0);
    };
    // twelve pieces of the way out of acc[x]: to LDS (16 columns of a lane's row in halves), from there as rows, to memory
    auto out_piece = [&](int x, int e, rsrc_t yr) {
        if (e < 4) {
            const int b = e >> 1, h = e & 1;
            u32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = pack2_bf16(acc[x][b][8 * h + 2 * i], acc[x][b][8 * h + 2 * i + 1]);
            *reinterpret_cast<u32x4*>(stg + lj * 128 + (((4 * b + 2 * lh + h) ^ sw) * 16)) = v;
        } else if (e < 8) {
            piece[e - 4] = *reinterpret_cast<const u32x4*>(rd + (e - 4) * 1024 + (((lane & 7) ^ ((lane >> 4) + 4 * (e & 1))) * 16));
        } else {
            if constexpr (STREAM) buf_store16_stream(piece[e - 8], yr, out_off + (e - 8) * 16 * q, 0);
            else buf_store16(piece[e - 8], yr, out_off + (e - 8) * 16 * q, 0);
        }
    };
    auto out_pieces = [&](int x, int step, rsrc_t yr) {   // those of one of KB steps
#pragma unroll
        for (int e = 12 * step / KB; e < 12 * (step + 1) / KB; ++e) out_piece(x, e, yr);
    };
    auto mma = [&](int x, int kk, u32x4 t) {
        acc[x][0] = mfma_bf16(qf[0][kk], t, kk == 0 ? zero : acc[x][0]);
        acc[x][1] = mfma_bf16(qf[1][kk], t, kk == 0 ? zero : acc[x][1]);
    };
    rsrc_t y0 = yres(ch0 - 1, 0), y1 = y0;                // where the blocks of the chunk before go
    int at = 0;                                           // slot of the chunk
    for (int ch = ch0; ch < ch1; ++ch) {
        // The loads of this chunk have landed (the first did with Q): behind them this wave has issued the eight stores of each chunk since
        // and the loads of the chunk after.  Accesses of one wave are counted off in the order of issue.
        if (ch > ch0) {
            if constexpr (NS == 2) wait_newest<8>();
            else if (ch == ch0 + 1) {
                if (ch + 1 < ch1) wait_newest<8 + NL>();
                else wait_newest<8>();
            }
            else if (ch + 1 < ch1) wait_newest<16 + NL>();
            else wait_newest<16>();
        }
        lds_barrier();
        if (ch + NS - 1 < ch1) issue(ch + NS - 1, at == 0 ? NS - 1 : at - 1);
        const unsigned char* const tb = lds + at * L::slot;
        at = at == NS - 1 ? 0 : at + 1;
        const rsrc_t n0 = yres(ch, 0), n1 = yres(ch, 1);
        unrolled<0, 2 * KB>([&](auto step) {
            // the operand read now is used NB steps on, across the barrier too
            constexpr int s = decltype(step)::value, t = s - NB;
            if (t < 0) mma(1, KB + t, ring[s % NB]);
            else if (t < KB) mma(0, t, ring[s % NB]);
            else mma(1, t - KB, ring[s % NB]);
            __builtin_amdgcn_sched_barrier(0);
            const int blk = s / KB, kk = s % KB;
            ring[s % NB] = *reinterpret_cast<const u32x4*>(tb + tbase[kk % L::NV] + (kk / L::NV) * (L::NV * 32) + blk * (32 * R * 2));
            if (t < 0) out_pieces(0, KB + t, y0);
            else if (t < KB) out_pieces(1, t, y1);
            else out_pieces(0, t - KB, n0);
            __builtin_amdgcn_sched_barrier(0);
        });
        y0 = n0;
        y1 = n1;
    }
#pragma unroll
    for (int t = KB - NB; t < KB; ++t) {
        mma(1, t, ring[(KB + t) % NB]);
        out_pieces(0, t, y0);
    }
#pragma unroll
    for (int e = 0; e < 12; ++e) out_piece(1, e, y1);
}

template <int R>
hipError_t launch_expand_r(const PairPtrs& ptrs, int G, int M, int q, hipStream_t s) {
    using L = ExCfg<R>;
    const bool stream = (int64_t)M * q * 2 >= kStreamOutBytes;
    const void* fn = stream ? reinterpret_cast<const void*>(&expand_kernel<R, true>) : reinterpret_cast<const void*>(&expand_kernel<R, false>);
    static std::atomic<bool> attr_set[2] = {};
    if (!attr_set[stream].load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, L::lds);
        if (e != hipSuccess) return e;
        attr_set[stream].store(true, std::memory_order_release);
    }
    const int ncol = (q + 255) / 256, nch = (M + L::CH - 1) / L::CH;
    // one work-group per compute unit, each with the same number of chunks but for the last of a column group
    int nrow = 256 / (ncol * G);
    if (nrow < 1) nrow = 1;
    const int each = (nch + nrow - 1) / nrow;
    nrow = (nch + each - 1) / each;
    const dim3 grid((unsigned)(ncol * nrow * G));
    if (stream) hipLaunchKernelGGL((expand_kernel<R, true>), grid, dim3(L::NT), L::lds, s, ptrs, M, q, ncol, nrow, each);
    else hipLaunchKernelGGL((expand_kernel<R, false>), grid, dim3(L::NT), L::lds, s, ptrs, M, q, ncol, nrow, each);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ contract
// Bound by what a compute unit can have on its way: loads come back in the order of issue, so P, which hits in L2, waits behind X, which does not, and both
// take room (p = 3072, r = 192: 82 us, 72 without the products, 61 without P, 47 without any load).  Hence as many rows per work-group as there are, against the
// share of P, and slabs two ahead where LDS allows (one ahead 90 us; three of X 80).  Few rows share out the steps of a slab instead of the rows: every
// operand is read from LDS once (12608 rows, p = 3072, r = 192: 26 us; as 128 rows per work-group 35).
// Tried: slabs of 32 columns (half lines: 95 against 87 us), 128 columns (equal), a start of its own per work-group (equal), the non-temporal hint on X
// (4 % at r = 192, but 25.3 -> 33.9 for 12608 rows), four waves of 128 x 96 values (87 against 82), T stored from the accumulators (equal).
// RP: the rank or, with one more block of 32, the next multiple of 64.  Eight waves: two column groups of RP / 2, RW row groups, and KW = 4 / RW
// waves that share the steps of a slab of 64 contraction columns (their sums are added at the end, in order).  A work-group has xr rows, a
// multiple of 8 up to 64 RW: row group i has the blocks of 32 rows i and i + RW.  Slabs of X are requested LX ahead, of P one ahead.
template <int RP, int RW>
struct CoCfg {
    static constexpr int KW = 4 / RW, CB = RP / 64;
    static constexpr int ppart = RP * 128, NPI = RP / 64; // P's part of a slab, its load instructions per wave
    static constexpr int SPW = 4 / KW;                    // steps of a wave per slab
    static constexpr bool TWO = RP <= 256;                // operands of two steps in registers
    static constexpr int red = (KW - 1) * RW * 2 * CB * 4096, tile = 32 * RW * (RP * 2 + 16);
    static __host__ __device__ constexpr int lds(int xr, int LX, int LP) {
        const int slabs = (LX + 1) * xr * 128 + (LP + 1) * ppart, over = LX * xr * 128 + RW * 64 * 128;       // blocks past xr are read, not used
        const int need = slabs > over ? slabs : over, end = red > tile ? red : tile;
        return need > end ? need : end;
    }
    static __device__ __forceinline__ int swz(int i) { return (i >> 1) & 7; }
};

template <int RP, int RW, int LX, int LP>
__global__ __launch_bounds__(512) void contract_kernel(PairPtrs ptrs, int M, int p, int r, int xr) {
    using L = CoCfg<RP, RW>;
    constexpr int CB = L::CB, KW = L::KW, SPW = L::SPW;
    extern __shared__ __align__(1024) unsigned char lds[];
    const uint16_t* const X = ptrs.in[blockIdx.y];
    const uint16_t* const P = ptrs.f[blockIdx.y];
    uint16_t* const T = ptrs.out[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lj = lane & 31, lh = lane >> 5;
    const int kw = wave / (2 * RW), rw = wave / 2 % RW, cw = wave & 1;
    const int64_t row0 = (int64_t)blockIdx.x * xr;
    const int rows = M - row0 < xr ? (int)(M - row0) : xr;
    const int ns = p / 64;
    const rsrc_t xres = make_rsrc(X + row0 * p, (int64_t)rows * p * 2), pres = make_rsrc(P, (int64_t)r * p * 2);
    // A load instruction covers eight rows; instructions wave, wave + 8, .. of X and of P.  Rows past M and past the rank arrive as zeros.
    const int nx = (xr / 8 - wave + 7) / 8;               // at most RW
    const int lrow = 8 * wave + (lane >> 3);
    const int off = (lrow * p + ((lane & 7) ^ L::swz(lrow)) * 8) * 2, step = 64 * p * 2;
    const int xpart = xr * 128, pbase = (LX + 1) * xpart;
    int pslot = pbase;                                    // of the next slab of P and of X to be requested
    auto issue_p = [&](int s) {
        unsigned char* dst = lds + pslot + wave * 1024;
        pslot = pslot == pbase + LP * L::ppart ? pbase : pslot + L::ppart;
        const int so = s * 128;
#pragma unroll
        for (int j = 0; j < L::NPI; ++j) load_lds16(pres, dst + j * 8192, off + j * step, so);
    };
    int xslot = 0;
    auto issue_x = [&](int s) {
        unsigned char* dst = lds + xslot + wave * 1024;
        xslot = xslot == LX * xpart ? 0 : xslot + xpart;
        const int so = s * 128;
#pragma unroll
        for (int j = 0; j < RW; ++j)
            if (j < nx) load_lds16(xres, dst + j * 8192, off + j * step, so);
    };
    f32x16 acc[2][CB];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;
    struct Ops { u32x4 x[2], f[CB]; };
    constexpr int NOB = L::TWO ? 2 : 1;
    Ops ob[NOB];
#pragma unroll
    for (int i = 0; i < NOB; ++i) {
#pragma unroll
        for (int a = 0; a < 2; ++a) ob[i].x[a] = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < CB; ++b) ob[i].f[b] = u32x4{0, 0, 0, 0};
    }
    const int prow = out_row(lj);
    int xat[SPW], pat[SPW];                               // chunk 2 (kw SPW + j) + lh of this lane's row
#pragma unroll
    for (int j = 0; j < SPW; ++j) {
        const int c = 2 * (kw * SPW + j) + lh;
        xat[j] = (32 * rw + lj) * 128 + ((c ^ L::swz(lj)) * 16);
        pat[j] = (cw * (RP / 2) + prow) * 128 + ((c ^ L::swz(prow)) * 16);
    }
    const int xlive = xr > 32 * (rw + RW) ? 2 : 1;        // blocks of rows of this wave
    auto read = [&](Ops& o, const unsigned char* xs, const unsigned char* ps, int j) {
#pragma unroll
        for (int b = 0; b < CB; ++b) o.f[b] = *reinterpret_cast<const u32x4*>(ps + pat[j] + b * 4096);
#pragma unroll
        for (int a = 0; a < 2; ++a) o.x[a] = *reinterpret_cast<const u32x4*>(xs + xat[j] + a * (RW * 4096));
    };
    auto mma = [&](const Ops& o) {
#pragma unroll
        for (int b = 0; b < CB; ++b) acc[0][b] = mfma_bf16(o.f[b], o.x[0], acc[0][b]);
        if (xlive > 1) {
#pragma unroll
            for (int b = 0; b < CB; ++b) acc[1][b] = mfma_bf16(o.f[b], o.x[1], acc[1][b]);
        }
    };
#pragma unroll
    for (int d = 0; d < LX; ++d) {                        // in the order of the loop below
        if (d >= LX - LP && d - LX + LP < ns) issue_p(d - LX + LP);
        if (d < ns) issue_x(d);
    }
    int xs_at = 0, ps_at = pbase;
    // Slab s has landed.  Loads come back in the order of issue; those issued after the last one of slab s may still be on their way.
    auto landed = [&](int s) {
        constexpr int A = LP == LX ? LP - 1 : LP, B = (LP - 1) * L::NPI;
        if (s + LX > ns) wait_newest<0>();
        else if (nx == RW) wait_newest<RW * A + B>();
        else if (nx == RW - 1) wait_newest<(RW - 1) * A + B>();
        else if (RW > 2 && nx == RW - 2) wait_newest<(RW > 2 ? RW - 2 : 0) * A + B>();
        else wait_newest<B>();
    };
    static_assert(LP >= 1 && LP <= LX && RW * LP + (LP - 1) * L::NPI < 64, "");
    auto slab = [&](int s, auto parity) {
        constexpr int par = decltype(parity)::value;
        landed(s);
        lds_barrier();
        // into the slots whose reads ended before this barrier
        if (s + LP < ns) issue_p(s + LP);
        if (s + LX < ns) issue_x(s + LX);
        const unsigned char* const xs = lds + xs_at;
        const unsigned char* const ps = lds + ps_at;
        xs_at = xs_at == LX * xpart ? 0 : xs_at + xpart;
        ps_at = ps_at == pbase + LP * L::ppart ? pbase : ps_at + L::ppart;
        if constexpr (L::TWO) {
#pragma unroll
            for (int j = 0; j < SPW; ++j) {
                read(ob[(par + j) & 1], xs, ps, j);
                __builtin_amdgcn_sched_barrier(0);
                mma(ob[(par + j + 1) & 1]);               // the step before, of the slab before at j = 0
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int j = 0; j < SPW; ++j) {
                read(ob[0], xs, ps, j);
                mma(ob[0]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    int s = 0;
    for (; s + 1 < ns; s += 2) {
        slab(s, std::integral_constant<int, 0>{});
        slab(s + 1, std::integral_constant<int, SPW & 1>{});
    }
    if (s < ns) slab(s, std::integral_constant<int, 0>{});
    if constexpr (L::TWO) {                               // the last step
        if ((SPW & 1) && s == ns) mma(ob[1]);
        else mma(ob[(SPW - 1) & 1]);
    }
    // T leaves through LDS as whole rows, 32 RW rows at a time
    const rsrc_t tres = make_rsrc(T + row0 * r, (int64_t)rows * r * 2);
    const int tpitch = r * 2 + 16, cpr = r / 8;
    const int tile = rw * 2 + cw;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        if (a && xr <= 32 * RW) break;
        lds_barrier();
        if constexpr (KW > 1) {
            // column block b is finished by wave b % KW of those that share it, the others hand theirs over through LDS
#pragma unroll
            for (int b = 0; b < CB; ++b)
                if (kw != b % KW) {
                    const int from = kw > b % KW ? kw - 1 : kw;
                    unsigned char* d = lds + ((tile * (KW - 1) + from) * CB + b) * 4096 + lane * 16;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        *reinterpret_cast<f32x4*>(d + v * 1024) = f32x4{acc[a][b][4 * v], acc[a][b][4 * v + 1], acc[a][b][4 * v + 2], acc[a][b][4 * v + 3]};
                }
            lds_barrier();
#pragma unroll
            for (int b = 0; b < CB; ++b)
                if (kw == b % KW) {
#pragma unroll
                    for (int from = 0; from < KW - 1; ++from) {
                        const unsigned char* d = lds + ((tile * (KW - 1) + from) * CB + b) * 4096 + lane * 16;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const f32x4 x = *reinterpret_cast<const f32x4*>(d + v * 1024);
#pragma unroll
                            for (int i = 0; i < 4; ++i) acc[a][b][4 * v + i] += x[i];
                        }
                    }
                }
            lds_barrier();
        }
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            const int col = cw * (RP / 2) + 32 * b + 16 * lh;
            if ((KW > 1 && kw != b % KW) || col >= r) continue;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = pack2_bf16(acc[a][b][8 * h + 2 * i], acc[a][b][8 * h + 2 * i + 1]);
                *reinterpret_cast<u32x4*>(lds + (32 * rw + lj) * tpitch + (col + 8 * h) * 2) = v;
            }
        }
        lds_barrier();
        const int here = xr - 32 * RW * a < 32 * RW ? xr - 32 * RW * a : 32 * RW;
        for (int i = threadIdx.x; i < here * cpr; i += 512) {
            const int row = i / cpr, ch = i - row * cpr;
            buf_store16(*reinterpret_cast<const u32x4*>(lds + row * tpitch + ch * 16), tres, ((32 * RW * a + row) * r + ch * 8) * 2, 0);
        }
    }
}

template <int RP, int RW, int LX, int LP>
hipError_t launch_contract_c(const PairPtrs& ptrs, int G, int M, int p, int r, int xr, hipStream_t s) {
    using L = CoCfg<RP, RW>;
    static_assert(L::lds(64 * RW, LX, LP) <= 160 * 1024, "");
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&contract_kernel<RP, RW, LX, LP>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 L::lds(64 * RW, LX, LP));
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const dim3 grid((unsigned)((M + xr - 1) / xr), (unsigned)G);
    hipLaunchKernelGGL((contract_kernel<RP, RW, LX, LP>), grid, dim3(512), L::lds(xr, LX, LP), s, ptrs, M, p, r, xr);
    return hipGetLastError();
}

// Rows per work-group: the smallest whole number of work-groups per compute unit with at most 256 rows each, and the rows of all `of`
// problems shared out evenly among them; at least 32.
int contract_rows(int of, int64_t M) {
    for (int64_t per_cu = 1;; ++per_cu) {
        const int64_t blocks = 256 * per_cu / of;         // of one problem
        const int64_t rows = blocks ? ceil_div(M, blocks) : M;
        if (rows <= 256) return rows <= 32 ? 32 : (int)ceil_div(rows, 8) * 8;
    }
}

template <int RP>
hipError_t launch_contract_r(const PairPtrs& ptrs, int G, int M, int p, int r, int xr, hipStream_t s) {
    if constexpr (RP != 256)                              // (no batch that small goes here at r = 224 and 256)
        if (xr <= 64) return launch_contract_c<RP, 1, 2, RP <= 320 ? 2 : 1>(ptrs, G, M, p, r, xr, s);
    if (xr <= 128) return launch_contract_c<RP, 2, 2, RP <= 256 ? 2 : 1>(ptrs, G, M, p, r, xr, s);
    return launch_contract_c<RP, 4, RP <= 256 ? 2 : 1, RP <= 128 ? 2 : 1>(ptrs, G, M, p, r, xr, s);
}

}  // namespace

bool pair_supports(int64_t M, int p, int q, int R) {
    return M >= 1 && M <= (1 << 30) && p % 64 == 0 && q % 64 == 0 && p >= 64 && q >= 64 && p <= (1 << 20) && q <= (1 << 20) && R % 32 == 0 && R >= 64 && R <= 384;
}

hipError_t launch_pair_bf16(const ChainProblem* problems, int G, int of, int64_t M, int p, int q, int R, hipStream_t s) {
    if (G < 1 || of < G || of > kChainMaxGroups || !problems || !pair_supports(M, p, q, R)) return hipErrorInvalidValue;
    PairPtrs a{}, b{};
    for (int g = 0; g < G; ++g) {
        if (!problems[g].Tout || (problems[g].Yout != nullptr) != (problems[0].Yout != nullptr)) return hipErrorInvalidValue;
        a.in[g] = (const uint16_t*)problems[g].Xin; a.f[g] = (const uint16_t*)problems[g].P; a.out[g] = (uint16_t*)problems[g].Tout;
        b.in[g] = (const uint16_t*)problems[g].Tout; b.f[g] = (const uint16_t*)problems[g].Q; b.out[g] = (uint16_t*)problems[g].Yout;
    }
    const int xr = contract_rows(of, M);
    hipError_t e = hipErrorInvalidValue;
    switch ((R + 63) / 64) {
        case 1: e = launch_contract_r<64>(a, G, (int)M, p, R, xr, s); break;
        case 2: e = launch_contract_r<128>(a, G, (int)M, p, R, xr, s); break;
        case 3: e = launch_contract_r<192>(a, G, (int)M, p, R, xr, s); break;
        case 4: e = launch_contract_r<256>(a, G, (int)M, p, R, xr, s); break;
        case 5: e = launch_contract_r<320>(a, G, (int)M, p, R, xr, s); break;
        case 6: e = launch_contract_r<384>(a, G, (int)M, p, R, xr, s); break;
    }
    if (e != hipSuccess || !problems[0].Yout) return e;
    switch (R / 32) {
        case 2: return launch_expand_r<64>(b, G, (int)M, q, s);
        case 3: return launch_expand_r<96>(b, G, (int)M, q, s);
        case 4: return launch_expand_r<128>(b, G, (int)M, q, s);
        case 5: return launch_expand_r<160>(b, G, (int)M, q, s);
        case 6: return launch_expand_r<192>(b, G, (int)M, q, s);
        case 7: return launch_expand_r<224>(b, G, (int)M, q, s);
        case 8: return launch_expand_r<256>(b, G, (int)M, q, s);
        case 9: return launch_expand_r<288>(b, G, (int)M, q, s);
        case 10: return launch_expand_r<320>(b, G, (int)M, q, s);
        case 11: return launch_expand_r<352>(b, G, (int)M, q, s);
        case 12: return launch_expand_r<384>(b, G, (int)M, q, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace abt
