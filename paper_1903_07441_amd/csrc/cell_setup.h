// Set-up of a relaxation's cells for gfx950: the field's boundary and initial
// values and the sweeps' free mask from the class map, in one pass over it.
#pragma once

#include "twg_internal.h"

namespace twg {

// What a set-up writes; psi or mask may be null.
struct CellSetup {
    const uint8_t *cls;
    float *psi;      // field values by `mode` (below)
    uint8_t *mask;   // 0xFF on FREE cells, 0 on the others
    int nx, ny, pitch, mode, gx, gy;
};

// The value the cell (x, y) of class `code` gets; false: it keeps its own.
// OBST and WALL 0, GOAL 1, FIXED unchanged; FREE cells by mode: HALF 0.5,
// ZERO 0, LINEAR the ramp 1 - d / (max(nx, ny) sqrt 2) of the Euclidean
// distance d to the goal cell (gx, gy), evaluated in FP64 and rounded once;
// KEEP leaves them.
__device__ __forceinline__ bool init_value(const CellSetup &s, uint32_t code, int x, int y, float *v)
{
    *v = 0.0f;
    switch (code) {
    case TWG_CELL_OBST:
    case TWG_CELL_WALL: return true;
    case TWG_CELL_GOAL: *v = 1.0f; return true;
    case TWG_CELL_FREE:
        if (s.mode == HPF_INIT_HALF) {
            *v = 0.5f;
        } else if (s.mode == HPF_INIT_LINEAR) {
            const double dx = (double)(x - s.gx), dy = (double)(y - s.gy);
            const double d = sqrt(dx * dx + dy * dy);
            *v = (float)(1.0 - d / ((double)max(s.nx, s.ny) * sqrt(2.0)));
        } else {
            return s.mode == HPF_INIT_ZERO;
        }
        return true;
    default: return false;
    }
}

// Bound by memory: 1 byte read and 5 written a cell.  A lane takes one column of
// K rows, dy apart, read before any is written.  2048 x 2048, one launch for field
// and mask: 8.7 us (9.2 at an odd pitch); with four neighbouring cells a lane,
// written as words where rows are aligned, 10.1 (13.5 where they are not), and
// cell by cell in two launches 9 + 6.  Beyond the caches the wide words were
// faster (8192 x 8192, the field alone: 84 us, 110 here, 157 a row a wave).
template <int K>
__device__ __forceinline__ void setup_rows(const CellSetup &s, int x, int y0, int dy, int yend)
{
    if (x >= s.nx) return;
    uint8_t c[K];
#pragma unroll
    for (int k = 0; k < K; ++k) c[k] = s.cls[(size_t)min(y0 + k * dy, yend - 1) * s.pitch + x];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int y = y0 + k * dy;
        if (y >= yend) return;
        const size_t i = (size_t)y * s.pitch + x;
        float v;
        if (init_value(s, c[k], x, y, &v) && s.psi) s.psi[i] = v;
        if (s.mask) s.mask[i] = c[k] == TWG_CELL_FREE ? 0xff : 0;
    }
}

// One grid: a wave takes 64 columns of kSetupRows rows, of narrow grids several
// rows at once (1 << lane_bits lanes a row; 8 x 32767 cells: 5.5 us a call, 9.4
// with two lanes of 64 at work).
constexpr int kSetupRows = 4;
inline int setup_lane_bits(int nx)
{
    int b = 0;
    while (b < 6 && (1 << b) < nx) ++b;
    return b;
}
inline dim3 setup_blocks(int nx, int ny)
{
    const int b = setup_lane_bits(nx), rows = kSetupRows * (256 >> b);
    return dim3((nx + (1 << b) - 1) >> b, (ny + rows - 1) / rows);
}
__device__ __forceinline__ void setup_grid(const CellSetup &s, int lane_bits)
{
    const int at_once = 256 >> lane_bits;  // rows a block takes at once
    setup_rows<kSetupRows>(s, (blockIdx.x << lane_bits) + (threadIdx.x & ((1 << lane_bits) - 1)),
                           blockIdx.y * kSetupRows * at_once + (threadIdx.x >> lane_bits), at_once, s.ny);
}

}  // namespace twg
