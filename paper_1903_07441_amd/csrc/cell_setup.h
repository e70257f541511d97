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

// Bound by memory: 1 byte read and 5 written a cell.  A lane takes four
// neighbouring cells, read as one word and written as one mask word and one
// 16-byte store, where rows are aligned for that (`quads`: wave-uniform);
// else, at a row's end and where a cell keeps its value, cell by cell.  K
// rows, dy apart, are read before any is written.  2048 x 2048: field 9 and
// mask 6 us cell by cell in two launches, 9 us here.
template <int K>
__device__ __forceinline__ void setup_rows(const CellSetup &s, int x, int y0, int dy, int yend, bool quads)
{
    if (x >= s.nx) return;
    const bool wide = quads && x + 4 <= s.nx;
    uint32_t c[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (wide) c[k] = *reinterpret_cast<const uint32_t *>(s.cls + (size_t)min(y0 + k * dy, yend - 1) * s.pitch + x);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int y = y0 + k * dy;
        if (y >= yend) return;
        const size_t i = (size_t)y * s.pitch + x;
        if (wide) {
            float v[4];
            bool all = true, set[4];
            uint32_t m = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t code = c[k] >> 8 * j & 0xffu;
                set[j] = init_value(s, code, x + j, y, &v[j]);
                all = all && set[j];
                m |= code == TWG_CELL_FREE ? 0xffu << 8 * j : 0u;
            }
            if (s.mask) *reinterpret_cast<uint32_t *>(s.mask + i) = m;
            if (!s.psi) continue;
            if (all) {
                *reinterpret_cast<float4 *>(s.psi + i) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (set[j]) s.psi[i + j] = v[j];
            }
            continue;
        }
        for (int j = 0; j < 4 && x + j < s.nx; ++j) {
            const uint32_t code = s.cls[i + j];
            float v;
            if (init_value(s, code, x + j, y, &v) && s.psi) s.psi[i + j] = v;
            if (s.mask) s.mask[i + j] = code == TWG_CELL_FREE ? 0xff : 0;
        }
    }
}

__device__ __forceinline__ bool setup_quads(const CellSetup &s)
{
    return !((uintptr_t)s.cls & 3) && !((uintptr_t)s.psi & 15) && !((uintptr_t)s.mask & 3) && !(s.pitch & 3);
}

// one grid: a wave takes runs of 256 columns of kSetupRows rows (a block: of
// four times as many)
constexpr int kSetupRows = 4;
inline int setup_blocks(int nx, int ny)
{
    return (int)(((long long)ny + 4 * kSetupRows - 1) / (4 * kSetupRows) * ((nx + 255) / 256));
}
__device__ __forceinline__ void setup_grid(const CellSetup &s)
{
    const int runs = (s.nx + 255) / 256, band = blockIdx.x / runs;
    setup_rows<kSetupRows>(s, (blockIdx.x - band * runs) * 256 + 4 * (threadIdx.x & 63),
                           band * 4 * kSetupRows + (threadIdx.x >> 6), 4, s.ny, setup_quads(s));
}

}  // namespace twg
