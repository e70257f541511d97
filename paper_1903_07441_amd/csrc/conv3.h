// The network's 3x3 convolutions (conv3.hip): forward layers and input
// gradients.
#pragma once

#include "twg_internal.h"

namespace twg {

// Where a convolution's input comes from: one tensor [B][H][W][CIN], or the
// concatenation of a half-resolution tensor (nearest upsampling, channels
// < CA) with a full-resolution one.
constexpr int kPlain = 0, kUpCat = 1;

// What becomes of its output: bf16(relu(acc + bias)); the same and its 2x2
// mean (the next level's input); the network's head on the same, not stored;
// the FP32 accumulators (input gradients); the gradient of a low activation
// behind an upsampling: 2x2 sums, where `act` is positive, as bf16; or the
// gradient of an activation used by a skip connection and by a pooling:
// bf16((acc + dp / 4) [act > 0]), dp the FP32 gradient of the pooled one.
constexpr int kOutAct = 0, kOutPool = 1, kOutHead = 2, kOutF32 = 3, kOutUpGrad = 4, kOutSkipGrad = 5;

struct ConvArgs {
    const uint16_t *A, *Bs;  // input (Bs: the full-resolution half of kUpCat)
    const uint16_t *wt;      // weights [COUT][9][CIN]
    const float *bias;
    void *out;               // [B][H][W][COUT] bf16 (kOutF32: FP32); unused by kOutHead and kOutUpGrad
    uint16_t *pool;          // kOutPool, kOutUpGrad: [B][H/2][W/2][COUT]
    const float *hw, *hb;    // kOutHead: the head's weights and bias
    float *y;                // kOutHead: [B][H][W]
    int nb, H, W;
    const uint16_t *act = nullptr;  // kOutUpGrad: [B][H/2][W/2][COUT]; kOutSkipGrad: [B][H][W][COUT]
    const float *dp = nullptr;      // kOutSkipGrad: [B][H/2][W/2][COUT]
};

template <int CIN, int COUT, int MODE, int CA, int OUT>
int launch_conv3(const ConvArgs &a, int num_cu, hipStream_t st);

}  // namespace twg
