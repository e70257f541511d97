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
// the FP32 accumulators (input gradients); or, of the input gradient of a
// concatenation, the upsampled half summed over 2x2 pixels, where the low
// activation `act` is positive, as bf16 (its gradient), and the other half as
// FP32 accumulators.
constexpr int kOutAct = 0, kOutPool = 1, kOutHead = 2, kOutF32 = 3, kOutCatGrad = 4;

struct ConvArgs {
    const uint16_t *A, *Bs;  // input (Bs: the full-resolution half of kUpCat)
    const uint16_t *wt;      // weights [COUT][9][CIN]
    const float *bias;
    void *out;               // [B][H][W][COUT] bf16 (kOutF32: FP32; kOutCatGrad: the upper
                             // COUT/2 channels, FP32); unused by kOutHead
    uint16_t *pool;          // kOutPool: [B][H/2][W/2][COUT]; kOutCatGrad: [..][COUT/2]
    const float *hw, *hb;    // kOutHead: the head's weights and bias
    float *y;                // kOutHead: [B][H][W]
    int nb, H, W;
    const uint16_t *act = nullptr;  // kOutCatGrad: [B][H/2][W/2][COUT/2]
};

template <int CIN, int COUT, int MODE, int CA, int OUT>
int launch_conv3(const ConvArgs &a, int num_cu, hipStream_t st);

}  // namespace twg
