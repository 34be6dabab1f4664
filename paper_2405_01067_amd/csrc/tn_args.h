// Arguments of a launch that forms partial factor gradients (lr_tn2.hip, lr_taps.hip).
#pragma once

#include "common.h"

namespace abt {

struct Tn2Job { const uint16_t* U; const uint16_t* V; float* part; int P; int tile_begin; int transposed; int gather; };
// Gather form of U (jobs with gather != 0): U is a channels-last image [M / (H W), H, W, C] and column
// tap C + c of row i of the virtual U is channel c of pixel (y + ky - kh/2, x + kx - kw/2) of the
// same image (tap = ky kw + kx), zero outside it.  job.P = kh kw C.
// Rows are the pixels of a grid RH x RW per image; row (y, x) is centred on image pixel (mul y, mul x)
// (mul = 1 with RH x RW = H x W: every pixel; mul = 2: the patches of a stride-2 convolution).
struct Tn2Gather { int H, W, C, kh, kw, RH, RW, mul; };
struct Tn2Args { Tn2Job job[kTnMaxJobs]; int njobs; int tiles; int splits; int64_t M; int64_t rows_per_split; Tn2Gather g; };

// lr_taps.hip
bool taps_supports(const TnJob* jobs, int njobs, const Tn2Gather& g, int64_t M, int R, int splits);
int taps_tiles(const TnJob& job, const Tn2Gather* g);           // g: of the gathered job
int taps_splits(const TnJob* jobs, int njobs, const Tn2Gather& g, int64_t M, int R);
int taps_rows(int R);                                          // rows of a slab: rows_per_split is a multiple
hipError_t launch_taps(const Tn2Args& a, int R, hipStream_t s);

}  // namespace abt
