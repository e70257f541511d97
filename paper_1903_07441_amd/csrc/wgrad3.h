// Weight and bias gradients of the network's 3x3 convolutions (wgrad3.hip).
#pragma once

#include "conv3.h"

namespace twg {

// scratch for the splits' partial sums (floats)
constexpr size_t kPartFloats = (size_t)16384 * 9 * 128;

// g receives [COUT][9][CIN] then [COUT] (a layer's place in the gradient
// vector); the input as launch_conv3 takes it
template <int CIN, int COUT, int MODE, int CA>
int launch_wgrad3(const uint16_t *A, const uint16_t *Bs, const uint16_t *dout, float *part, float *g, int nb, int H,
                  int W, int num_cu, hipStream_t st);
// the first layer: x4 [B][H][W][4], g [32][9][32] (channels 0 to 2) then [32]
int launch_wgrad_in(const uint16_t *x4, const uint16_t *dout, float *part, float *g, int nb, int H, int W, int num_cu,
                    hipStream_t st);

}  // namespace twg
