// Declarations shared by the training step's translation units (train.hip: layout, small products, weight
// gradients, host side; train_back.hip: the kernels of the backward pass).  gfx950 only, fp32.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels_common.h"
#include "tig_internal.h"

namespace tig {

constexpr int kSumCopies = 8;

// Device arrays of a training step besides the model's own.  Rows "per query" are rows of the step's query
// set (distinct source / destination queries from 0, the negative of event b at 2 * count + b).
struct TrainArrays {
    // per query: what the forward pass keeps (S is [state row | has neighbours]) and the gradients
    float *S, *QT, *KVB, *H1;           // [R x (M + 1)], [R x N1], [R x N1], [R x E]
    float *DA, *DB;                     // [R x E] gradients of the decoder halves' pre-activations
    float *DEMB, *DZ1, *DQT;            // [R x E], [R x E], [R x N1]: embedding, merge layer 1's pre-activation, q~
    float *LOSS;                        // [2B] loss terms
    // per applied winner r, and per entry of the applied batch
    float *MSG, *GATES, *DGI, *DGH, *D_STAG;
    // sums over rows, added up with atomics and cleared by the update that reads them
    // (every XCD's workgroups add to a copy of their own: additions of hundreds of workgroups to one address wait for each other)
    double *TACC;                       // [copies][2T] time-encoding gradients [frequencies | phases]
    float *WACC;                        // [copies][E + 1] gradients of w_d2, b_d2
    // transposed weights, prepared like the forward kernels' (lane-ordered, padded with zeros)
    float *Wd1T;                        // [Ep x 2Ek]   W_d1[k][n], W_d1[k][E + n]
    float *Wm2T;                        // [Ep x Ek]
    float *PRT;                         // [K2 x Ek]    folded merge layer 1 | its state part
    float *A1T;                         // [Mq x N1]    folded query
    float *WiT;                         // [Tp x 3Mp]   message columns of the time encoding, all gates
};

struct BackParams {
    int M, T, F, E, K;
    int dkv, dkvp, Mq, N1, K2, Ep, Ek;
    int row_bytes;            // LDS bytes per row: [DA | DB | d emb], then [d kvbar / d q~ (N1) | d s_u (Mq)]
    int ldz;                  // LDS bytes per row of d z1
    int off_z, off_meta, off_tab;
    int rpt;                  // rows a workgroup takes, 4 .. ROWS (the rest of its tile's rows stay empty)
    int slots;                // rows of the LDS table that collects the staged rows' gradients (0: none)
};

hipError_t launch_train_decode(const Dims &d, const StepArgs &a, const PackedWeights &pw, const TrainArrays &t, hipStream_t s);
hipError_t launch_train_back(const Dims &d, const LaunchPlan &plan, const StepArgs &a, const PackedWeights &pw,
                             const TrainArrays &t, hipStream_t s);
hipError_t launch_train_gru_back(const Dims &d, const LaunchPlan &plan, const StepArgs &a, const PackedWeights &pw,
                                 const TrainArrays &t, hipStream_t s);
hipError_t prepare_train_back(const Dims &d);
bool train_back_fits(const Dims &d);  // the kernels' LDS and registers hold a row of this shape

// sin of the time-encoding phase (see time_enc): the derivative of Phi needs it
__device__ inline float time_enc_sin(double w_rev, double b_rev, double x)
{
    const double phase = fma(w_rev, x, b_rev);
    return __builtin_amdgcn_sinf((float)__builtin_amdgcn_fract(phase));
}

}  // namespace tig
