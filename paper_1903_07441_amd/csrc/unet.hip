// Learned warm start for the relaxation: a small encoder-decoder network that
// maps occupancy, goal-distance and ring-time channels to an initial field
// psi0.  Inference and training run in the kernels below on gfx950 matrix
// cores (bf16 operands, FP32 accumulation).
//
// Network (4 levels, 32 base channels, 443,745 parameters):
//   e0 = relu(conv3(x, 3 -> 32))                H
//   e1 = relu(conv3(pool(e0), 32 -> 64))        H/2
//   e2 = relu(conv3(pool(e1), 64 -> 128))       H/4
//   e3 = relu(conv3(pool(e2), 128 -> 128))      H/8
//   d2 = relu(conv3(cat(up(e3), e2), 256 -> 64)) H/4
//   d1 = relu(conv3(cat(up(d2), e1), 128 -> 32)) H/2
//   d0 = relu(conv3(cat(up(d1), e0), 64 -> 32))  H
//   y  = conv1(d0, 32 -> 1)
// conv3: 3x3 cross-correlation, zero padding 1, bias; pool: 2x2 mean; up: 2x
// nearest; cat: channel concatenation.  Every stored activation is bf16
// (round to nearest even); products accumulate in FP32.
//
// Layout: activations NHWC (channels contiguous), [B][H][W][C] bf16.  The
// network input is padded from 3 to 32 channels (zeros) so that every conv
// has a channel count that is a multiple of 32.  Weights [Cout][9][Cin] bf16
// (K = tap * Cin + c contiguous: the operand order of the matrix
// instruction), tap = ky * 3 + kx; the FP32 masters and Adam moments share
// that layout.  The input-gradient pass uses a second copy with the taps
// flipped and the channel roles swapped, [Cin][9][Cout].
//
// The 3x3 convolutions (forward and input gradients) are in conv3.hip; the
// first layer, with its three input channels, is here.  The layers that are
// pooled write their 2x2 means next to their output.
//
// Weight gradients are in wgrad3.hip.
#include "twg_internal.h"
#include "conv3.h"
#include "unet.h"
#include "unet_dev.h"
#include "wgrad3.h"

#include <cmath>
#include <cstring>
#include <vector>

namespace twg {

namespace {

using namespace ndev;

int last_status() { return hipGetLastError() == hipSuccess ? TWG_OK : TWG_EDEVICE; }

constexpr int kTS = 16;       // tile side of the first layer
constexpr int kHS = 18;       // halo side

// ---- first layer ---------------------------------------------------------
// The input has 3 real channels, so one K = 32 slice of the implicit GEMM
// covers all nine taps (k = 3 tap + c; k >= 27 is zero) and a 16-pixel row
// of 16 output channels takes one MFMA instead of nine.  x4 is
// [B][H][W][4] bf16 (channel 3 zero); the weights keep the layers' internal
// layout [32][9][32] (input channels padded to 32, only 0..2 used).  256
// threads; a workgroup builds its weight fragments once and then loops over
// 16 x 16 pixel tiles (t = blockIdx.x, + gridDim.x, ... < B tx ty), four
// rows per wave: every workgroup reading the same few weight lines for
// every tile would queue on the cache channels that hold them.
// out = bf16(relu(acc + bias)), [B][H][W][32].
__global__ __launch_bounds__(256) void k_conv3_in(const uint16_t *__restrict__ x4, const uint16_t *__restrict__ wt,
                                                  const float *__restrict__ bias, uint16_t *__restrict__ out,
                                                  uint16_t *__restrict__ pool, int nb, int H, int W)
{
    constexpr int COUT = 32, RT = 2, ZERO = kHS * kHS * 4;  // lds[ZERO..ZERO + 3] stay zero
    __shared__ __align__(16) uint16_t lds[kHS * kHS * 4 + 4];
    __shared__ __align__(16) uint16_t stg[4 * 64 * (COUT + 8)];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, g = lane >> 4;
    const int tx = (W + kTS - 1) / kTS, ty = (H + kTS - 1) / kTS, ntile = nb * tx * ty;
    // this lane's k = 8 g + i: A element (output channel rt * 16 + j) and the
    // LDS offset of its B element from the pixel's own halo position.  Every
    // load is unconditional (k >= 27 reads a valid element and is zeroed, or
    // reads the zero slot), so no load waits inside a divergent branch.
    uint32_t a[RT][4];
    int off[8];
    bool live[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int k = 8 * g + i, tap = k / 3, c = k - 3 * tap;
        live[i] = k < 27;
        off[i] = live[i] ? ((tap / 3) * kHS + (tap % 3)) * 4 + c : 0;
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            uint32_t w2[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int k = 8 * g + 2 * h + e, tap = live[2 * h + e] ? k / 3 : 0, c = live[2 * h + e] ? k - 3 * tap : 0;
                const uint32_t w = wt[((size_t)(rt * 16 + j) * 9 + tap) * 32 + c];
                w2[e] = live[2 * h + e] ? w : 0u;
            }
            a[rt][h] = w2[0] | (w2[1] << 16);
        }
    if (tid == 0) *reinterpret_cast<uint2 *>(&lds[ZERO]) = make_uint2(0, 0);
    float bs[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) bs[rt][v] = bias[rt * 16 + g * 4 + v];

    for (int t = blockIdx.x; t < ntile; t += gridDim.x) {
        const int b = t / (tx * ty), r = t - b * (tx * ty);
        const int x0 = (r % tx) * kTS, y0 = (r / tx) * kTS;
        for (int v = tid; v < kHS * kHS; v += 256) {
            const int hy = v / kHS, hx = v - hy * kHS;
            const int yy = y0 + hy - 1, xx = x0 + hx - 1;
            const bool in = yy >= 0 && yy < H && xx >= 0 && xx < W;
            const uint2 ld = *reinterpret_cast<const uint2 *>(
                x4 + (((size_t)b * H + min(max(yy, 0), H - 1)) * W + min(max(xx, 0), W - 1)) * 4);
            *reinterpret_cast<uint2 *>(&lds[v * 4]) = in ? ld : make_uint2(0, 0);
        }
        __syncthreads();

        f32x4 acc[4][RT];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const int base = ((wave * 4 + ct) * kHS + j) * 4;
            uint32_t bw[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const uint32_t lo = lds[live[2 * h] ? base + off[2 * h] : ZERO];
                const uint32_t hi = lds[live[2 * h + 1] ? base + off[2 * h + 1] : ZERO];
                bw[h] = lo | (hi << 16);
            }
            const uint4 bv = make_uint4(bw[0], bw[1], bw[2], bw[3]);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                acc[ct][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    as_bf8(make_uint4(a[rt][0], a[rt][1], a[rt][2], a[rt][3])), as_bf8(bv),
                    f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
        // A lane's accumulators hold 4 consecutive channels of one pixel:
        // each wave puts its 4 rows of bf16(relu(acc + bias)) into its part
        // of LDS and writes 16-byte runs of channels, and the 2x2 means
        // (two rows of eight pixels, one 16-byte run a lane)
        uint16_t *sw = stg + wave * 64 * (COUT + 8);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) {
                const f32x4 v = acc[ct][rt];
                *reinterpret_cast<uint2 *>(sw + (ct * 16 + j) * (COUT + 8) + rt * 16 + g * 4) =
                    make_uint2(pack2(relu(v[0] + bs[rt][0]), relu(v[1] + bs[rt][1])),
                               pack2(relu(v[2] + bs[rt][2]), relu(v[3] + bs[rt][3])));
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = i * 16 + (lane >> 2), c8 = lane & 3;
            const int y = y0 + wave * 4 + (p >> 4), x = x0 + (p & 15);
            const uint4 v = *reinterpret_cast<const uint4 *>(sw + p * (COUT + 8) + c8 * 8);
            if (y < H && x < W) *reinterpret_cast<uint4 *>(out + (((size_t)b * H + y) * W + x) * COUT + c8 * 8) = v;
        }
        {
            const int p = lane >> 2, c8 = lane & 3, y = y0 / 2 + wave * 2 + (p >> 3), x = x0 / 2 + (p & 7);
            const uint16_t *q = sw + ((p >> 3) * 32 + (p & 7) * 2) * (COUT + 8) + c8 * 8;
            const uint4 v = mean4(*reinterpret_cast<const uint4 *>(q), *reinterpret_cast<const uint4 *>(q + COUT + 8),
                                  *reinterpret_cast<const uint4 *>(q + 16 * (COUT + 8)),
                                  *reinterpret_cast<const uint4 *>(q + 17 * (COUT + 8)));
            if (y < H / 2 && x < W / 2)
                *reinterpret_cast<uint4 *>(pool + (((size_t)b * (H / 2) + y) * (W / 2) + x) * COUT + c8 * 8) = v;
        }
        // the next tile's halo overwrites what every wave has read above
        // (its products precede the barrier), and its staging follows the
        // next barrier
    }
}

// ---- head, loss, routing ---------------------------------------------------
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// v summed over the 16 lanes of a row, by halves (every lane gets the sum)
__device__ __forceinline__ float row_sum(float v)
{
    auto ror = [](float f, auto n) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(f), 0x120 + decltype(n)::value, 0xf, 0xf, true));
    };
    v += ror(v, std::integral_constant<int, 8>{});
    v += ror(v, std::integral_constant<int, 4>{});
    v += ror(v, std::integral_constant<int, 2>{});
    v += ror(v, std::integral_constant<int, 1>{});
    return v;
}
// lanes of the first half: a summed over both halves of the wave; of the
// second: b (the halves change places between two registers)
__device__ __forceinline__ float half_sums(float a, float b)
{
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    const uint32_t x = r[0], y = r[1];
    return __uint_as_float(x) + __uint_as_float(y);
}
// the same for the rows of a pair: a in even rows of 16 lanes, b in odd ones
__device__ __forceinline__ float pair_sums(float a, float b)
{
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    const uint32_t x = r[0], y = r[1];
    return __uint_as_float(x) + __uint_as_float(y);
}

// bytes of w that are zero
__device__ __forceinline__ int zero_bytes(uint32_t w)
{
    return __popc(~(((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u);
}

// Rows a thread takes, four apart (a block: 64 columns, 4 kRows rows), in the
// kernels that go over a map's cells: their loads are in flight together.
constexpr int kRows = 4;
dim3 rows_grid(int nx, int ny) { return dim3((nx + 63) / 64, (ny + 4 * kRows - 1) / (4 * kRows)); }

// Training head: masked MSE over FREE cells.  Per pixel: y, diff = y - t
// (0 outside the mask), loss += diff^2 / (n_b B), dy = 2 diff / (n_b B),
// dd0 = bf16(dy * hw * [d0 > 0]); block partial sums of the head gradients
// (hw: 32, hb: 1) and of the loss go to part[block][34].  Bound by memory
// (130 bytes a pixel) once the sums over a wave take few steps: 34 sums by
// shuffles were 204 trips through LDS, and 52 us for 16 x 256 x 256; here
// registers change halves, so that after two steps a lane sums 8 of them over
// its row (the same pairs in the same order).
__global__ __launch_bounds__(256) void k_head_loss(const uint16_t *__restrict__ d0, const float *__restrict__ hw,
                                                   const float *__restrict__ hb, const float *__restrict__ target,
                                                   const uint8_t *__restrict__ cls,
                                                   const unsigned int *__restrict__ cnt, int hw_pixels, int nb,
                                                   uint16_t *__restrict__ dd0, float *__restrict__ y_out,
                                                   float *__restrict__ part)
{
    __shared__ float red[4][34];
    const int p = blockIdx.x * 256 + threadIdx.x;
    const int total = hw_pixels * nb;
    float gw[32], gb = 0.f, lp = 0.f;
#pragma unroll
    for (int c = 0; c < 32; ++c) gw[c] = 0.f;
    if (p < total) {
        const int b = p / hw_pixels;
        float d[32];
        uint4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = reinterpret_cast<const uint4 *>(d0 + (size_t)p * 32)[q];
        const float y = head_value(v, hw, hb[0], d);
        if (y_out) y_out[p] = y;
        const float diff = cls[p] == TWG_CELL_FREE ? y - target[p] : 0.f;
        const unsigned int nf = cnt[b];
        const float sc = (1.f / (float)(nf > 1u ? nf : 1u)) / (float)nb;
        lp = diff * diff * sc;
        const float dy = 2.f * diff * sc;
        gb = dy;
        float dd[32];
#pragma unroll
        for (int c = 0; c < 32; ++c) {
            gw[c] = dy * d[c];
            dd[c] = d[c] > 0.f ? dy * hw[c] : 0.f;
        }
        uint4 *o = reinterpret_cast<uint4 *>(dd0 + (size_t)p * 32);
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = pack8(dd + 8 * q);
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // channel c + 8 r ends in row r of 16 lanes
    float s16[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) s16[c] = half_sums(gw[c], gw[c + 16]);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float s = row_sum(pair_sums(s16[c], s16[c + 8]));
        if ((lane & 15) == 0) red[wave][c + 8 * (lane >> 4)] = s;
    }
    {
        const float h = half_sums(gb, lp);  // gb in the first half, lp in the second
        const float s = row_sum(pair_sums(h, h));
        if ((lane & 31) == 0) red[wave][32 + (lane >> 5)] = s;
    }
    __syncthreads();
    if (threadIdx.x < 34) {
        const int c = threadIdx.x;
        part[(size_t)blockIdx.x * 34 + c] = ((red[0][c] + red[1][c]) + (red[2][c] + red[3][c]));
    }
}

// a network value into a cell of class c
__device__ __forceinline__ void put_psi(uint8_t c, float v, float *psi, unsigned int *bad)
{
    if (c == TWG_CELL_FREE) {
        if (!isfinite(v)) atomicOr(bad, 1u);
        *psi = fminf(fmaxf(v, 0.f), 1.f);
    } else if (c == TWG_CELL_OBST || c == TWG_CELL_WALL) {
        *psi = 0.f;
    } else if (c == TWG_CELL_GOAL) {
        *psi = 1.f;
    }
}

// Inference head into a field: FREE cells get clamp(y, 0, 1); OBST/WALL 0,
// GOAL 1; FIXED cells keep their value.  The network runs on a padded
// Hp x Wp frame; only the grid's nx x ny cells are written.
// A non-finite output at a FREE cell sets *bad (the whole field then falls
// back to the plain start, k_net_fallback).
__global__ __launch_bounds__(256) void k_head_psi(const float *__restrict__ yv, const uint8_t *__restrict__ cls,
                                                  float *__restrict__ psi, int nx, int ny, int pitch, int Wp,
                                                  unsigned int *bad)
{
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y0 = blockIdx.y * 4 * kRows + (threadIdx.x >> 6);
    if (x >= nx) return;
    uint8_t c[kRows];
    float v[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int y = min(y0 + 4 * k, ny - 1);
        c[k] = cls[(size_t)y * pitch + x];
        v[k] = yv[(size_t)y * Wp + x];
    }
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int y = y0 + 4 * k;
        if (y < ny) put_psi(c[k], v[k], psi + (size_t)y * pitch + x, bad);
    }
}

// Fallback of a warm start whose network produced a non-finite value: every
// FREE cell gets the plain start 0.5 (the fixed cells are already set);
// *status (if given) receives TWG_OK or TWG_NET_FALLBACK.
__global__ __launch_bounds__(256) void k_net_fallback(const uint8_t *__restrict__ cls, float *__restrict__ psi,
                                                      int nx, int ny, int pitch, const unsigned int *bad,
                                                      int32_t *status)
{
    const bool fall = *bad != 0u;
    if (status && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        *status = fall ? TWG_NET_FALLBACK : TWG_OK;
    if (!fall) return;
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (x >= nx || y >= ny) return;
    const size_t i = (size_t)y * pitch + x;
    if (cls[i] == TWG_CELL_FREE) psi[i] = 0.5f;
}

// Zero n device words (a kernel, so that the call can be captured into a
// graph without memset nodes).
__global__ void k_zero_words(unsigned int *w, int n)
{
    if (blockIdx.x == 0 && (int)threadIdx.x < n) w[threadIdx.x] = 0u;
}

// ---- input packing and features ------------------------------------------
// x [P][3] FP32 -> xp [P][4] bf16 (channel 3 zero)
__global__ __launch_bounds__(256) void k_pack_input(const float *__restrict__ x, uint16_t *__restrict__ xp,
                                                    long long total)
{
    const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
    if (p >= total) return;
    *reinterpret_cast<uint2 *>(xp + (size_t)p * 4) = make_uint2(pack2(x[3 * p], x[3 * p + 1]), pack2(x[3 * p + 2], 0.f));
}

// Network input channels of a grid on an Hp x Wp frame (frame cells outside
// the grid read as walls): occupancy (1 on OBST and WALL), Euclidean goal
// distance / (max(nx, ny) sqrt 2), ring / max ring (0 without a ring map).
// Writes FP32 [Hp][Wp][3] to xf and/or bf16 [Hp][Wp][4] (channel 3 zero) to xp.
__global__ __launch_bounds__(256) void k_features(const uint8_t *__restrict__ cls, const uint16_t *__restrict__ ring,
                                                  int nx, int ny, int pitch, int Hp, int Wp, int gx, int gy,
                                                  float inv_diag, const unsigned int *__restrict__ jmax,
                                                  float *__restrict__ xf, uint16_t *__restrict__ xp)
{
    const unsigned int jm = ring ? *jmax : 0u;
    const float inv_jmax = jm > 0u ? 1.f / (float)jm : 0.f;
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y0 = blockIdx.y * 4 * kRows + (threadIdx.x >> 6);
    if (x >= Wp) return;
    uint8_t c[kRows];
    uint16_t j[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const size_t i = (size_t)min(y0 + 4 * k, ny - 1) * pitch + min(x, nx - 1);
        c[k] = cls[i];
        j[k] = ring ? ring[i] : (uint16_t)0;
    }
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int y = y0 + 4 * k;
        if (y >= Hp) break;
        float occ = 1.f, rt = 0.f;
        if (x < nx && y < ny) {
            occ = (c[k] == TWG_CELL_OBST || c[k] == TWG_CELL_WALL) ? 1.f : 0.f;
            rt = (float)j[k] * inv_jmax;
        }
        const float ddx = (float)(x - gx), ddy = (float)(y - gy);
        const float gd = sqrtf(ddx * ddx + ddy * ddy) * inv_diag;
        const size_t p = (size_t)y * Wp + x;
        if (xf) {
            xf[3 * p] = occ;
            xf[3 * p + 1] = gd;
            xf[3 * p + 2] = rt;
        }
        if (xp) *reinterpret_cast<uint2 *>(xp + p * 4) = make_uint2(pack2(occ, gd), pack2(rt, 0.f));
    }
}

// ---- coarse-scale warm start ------------------------------------------------
// Input channels of a grid seen at 1/f of its resolution on an Hc x Wc frame:
// coarse cell (X, Y) covers the fine cells [fX, fX + f) x [fY, fY + f),
// cells outside the grid reading as walls.  Occupancy = share of OBST, WALL
// and outside cells in the block; goal distance of the block's centre
// (fX + (f - 1) / 2, fY + (f - 1) / 2) / (max(nx, ny) sqrt 2), the fine
// scale's normalisation; ring of the fine cell at the block's centre
// (fX + f / 2, fY + f / 2), clamped into the grid, / max ring (0 without a
// ring map).  ccls (optional): FREE where the block holds a FREE cell, else
// OBST (the training loss's mask at the coarse scale).
__global__ __launch_bounds__(256) void k_features_coarse(const uint8_t *__restrict__ cls,
                                                         const uint16_t *__restrict__ ring, int nx, int ny,
                                                         int pitch, int f, int Hc, int Wc, int gx, int gy,
                                                         float inv_diag, const unsigned int *__restrict__ jmax,
                                                         float *__restrict__ xf, uint16_t *__restrict__ xp,
                                                         uint8_t *__restrict__ ccls)
{
    const unsigned int jm = ring ? *jmax : 0u;
    const float inv_jmax = jm > 0u ? 1.f / (float)jm : 0.f;
    const int X = blockIdx.x * 64 + (threadIdx.x & 63);
    const int Y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (X >= Wc || Y >= Hc) return;
    // blocks inside the grid are read four cells at a time where rows are
    // aligned for that; a wave with a block at the edge goes cell by cell whole
    // (both ways one after the other took 45 us for f = 16 on 1001 columns, this 25)
    const bool words = !(f & 3) && !(pitch & 3) && !((uintptr_t)cls & 3);
    const int lf = __builtin_ctz(f);  // f is a power of two
    int blocked = 0, nfree = 0;
    if (words && __all((X + 1) * f <= nx && (Y + 1) * f <= ny)) {
        const uint8_t *p = cls + (size_t)Y * f * pitch + X * f;
        const int lw = lf - 2;  // words of a row
#pragma unroll 8
        for (int q = 0; q < f << lw; ++q) {
            const uint32_t w = *reinterpret_cast<const uint32_t *>(p + (size_t)(q >> lw) * pitch + 4 * (q & ((1 << lw) - 1)));
            blocked += zero_bytes(w ^ 0x01010101u * TWG_CELL_OBST) + zero_bytes(w ^ 0x01010101u * TWG_CELL_WALL);
            nfree += zero_bytes(w);
        }
    } else {
        // (every load unconditional: cells outside the grid read one inside)
#pragma unroll 8
        for (int q = 0; q < f * f; ++q) {
            const int y = Y * f + (q >> lf), x = X * f + (q & (f - 1));
            const uint8_t c = cls[(size_t)min(y, ny - 1) * pitch + min(x, nx - 1)];
            const bool in = x < nx && y < ny;
            blocked += !in || c == TWG_CELL_OBST || c == TWG_CELL_WALL ? 1 : 0;
            nfree += in && c == TWG_CELL_FREE ? 1 : 0;
        }
    }
    const float occ = (float)blocked / (float)(f * f);
    const float half = 0.5f * (float)(f - 1);
    const float ddx = ((float)(X * f) + half) - (float)gx, ddy = ((float)(Y * f) + half) - (float)gy;
    const float gd = sqrtf(ddx * ddx + ddy * ddy) * inv_diag;
    float rt = 0.f;
    if (ring && X * f < nx && Y * f < ny) {
        const int xc = min(X * f + f / 2, nx - 1), yc = min(Y * f + f / 2, ny - 1);
        rt = (float)ring[(size_t)yc * pitch + xc] * inv_jmax;
    }
    const size_t p = (size_t)Y * Wc + X;
    if (xf) {
        xf[3 * p] = occ;
        xf[3 * p + 1] = gd;
        xf[3 * p + 2] = rt;
    }
    if (xp) *reinterpret_cast<uint2 *>(xp + p * 4) = make_uint2(pack2(occ, gd), pack2(rt, 0.f));
    if (ccls) ccls[p] = nfree > 0 ? TWG_CELL_FREE : TWG_CELL_OBST;
}

// Coarse training target: out[Y][X] = mean of psi over the FREE fine cells of
// block (X, Y), summed in row order in FP32 (0 when the block has none).
__global__ __launch_bounds__(256) void k_coarse_target(const float *__restrict__ psi, const uint8_t *__restrict__ cls,
                                                       int nx, int ny, int pitch, int f, int Hc, int Wc,
                                                       float *__restrict__ out)
{
    const int X = blockIdx.x * 64 + (threadIdx.x & 63);
    const int Y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (X >= Wc || Y >= Hc) return;
    float sum = 0.f;
    int cnt = 0;
    for (int dy = 0; dy < f; ++dy) {
        const int y = Y * f + dy;
        if (y >= ny) break;
        for (int dx = 0; dx < f; ++dx) {
            const int x = X * f + dx;
            if (x >= nx) break;
            const size_t i = (size_t)y * pitch + x;
            if (cls[i] == TWG_CELL_FREE) {
                sum = sum + psi[i];
                ++cnt;
            }
        }
    }
    out[(size_t)Y * Wc + X] = cnt > 0 ? sum / (float)cnt : 0.f;
}

// Warm-start field from a coarse output yc [Hc][Wc]: a FREE cell (x, y) takes
// the bilinear interpolation of yc at coarse coordinates
// ((x + 1/2) / f - 1/2, (y + 1/2) / f - 1/2), clamped to the frame, then to
// [0, 1]; OBST and WALL 0, GOAL 1, FIXED unchanged.  A non-finite value at a
// FREE cell sets *bad.
__global__ __launch_bounds__(256) void k_up_psi(const float *__restrict__ yc, int Hc, int Wc, int f,
                                                const uint8_t *__restrict__ cls, float *__restrict__ psi, int nx,
                                                int ny, int pitch, unsigned int *bad)
{
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int row = blockIdx.y * 4 * kRows + (threadIdx.x >> 6);
    if (x >= nx) return;
    const float inv_f = 1.f / (float)f;  // f is a power of two: exact
    const float u = fminf(fmaxf(((float)x + 0.5f) * inv_f - 0.5f, 0.f), (float)(Wc - 1));
    const int x0 = (int)u, x1 = min(x0 + 1, Wc - 1);
    const float a = u - (float)x0;
    uint8_t c[kRows];
    float t[kRows][4], b[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int y = min(row + 4 * k, ny - 1);
        const float v = fminf(fmaxf(((float)y + 0.5f) * inv_f - 0.5f, 0.f), (float)(Hc - 1));
        const int y0 = (int)v, y1 = min(y0 + 1, Hc - 1);
        b[k] = v - (float)y0;
        c[k] = cls[(size_t)y * pitch + x];
        t[k][0] = yc[(size_t)y0 * Wc + x0];
        t[k][1] = yc[(size_t)y0 * Wc + x1];
        t[k][2] = yc[(size_t)y1 * Wc + x0];
        t[k][3] = yc[(size_t)y1 * Wc + x1];
    }
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int y = row + 4 * k;
        const float top = (1.f - a) * t[k][0] + a * t[k][1];
        const float bot = (1.f - a) * t[k][2] + a * t[k][3];
        const float val = (1.f - b[k]) * top + b[k] * bot;
        if (y < ny) put_psi(c[k], val, psi + (size_t)y * pitch + x, bad);
    }
}

// Largest ring number of a grid; *out must be zero beforehand.  A wave takes
// runs of 512 cells of a row, eight a lane, in one load where rows are aligned
// for that, else 64 apart; one atomic per block, of which there are few (they meet on one
// address, 10 ns each: 512 blocks of single-cell loads took 16 us at
// 2048 x 2048).
constexpr int kRingThreads = 512, kRingBlocks = 128;
__global__ __launch_bounds__(kRingThreads) void k_ring_max(const uint16_t *__restrict__ ring, int nx, int ny, int pitch,
                                                           unsigned int *out)
{
    constexpr int NW = kRingThreads / 64;
    __shared__ unsigned int red[NW];
    const int lane = threadIdx.x & 63;
    const int runs = (nx + 511) / 512, items = ny * runs;
    const bool quads = !((uintptr_t)ring & 15) && !(pitch & 7);
    unsigned int r = 0;
#pragma unroll 4
    for (int it = blockIdx.x * NW + (threadIdx.x >> 6); it < items; it += gridDim.x * NW) {
        const int y = it / runs, x0 = (it - y * runs) * 512, x = x0 + 8 * lane;
        const uint16_t *p = ring + (size_t)y * pitch;
        if (!quads) {
            // (a row's end reads its last cell again)
#pragma unroll
            for (int k = 0; k < 8; ++k) r = max(r, (unsigned int)p[min(x0 + 64 * k + lane, nx - 1)]);
        } else if (x + 8 <= nx) {
            const uint4 v = *reinterpret_cast<const uint4 *>(p + x);
            r = max(r, max(max(v.x & 0xffffu, v.x >> 16), max(v.y & 0xffffu, v.y >> 16)));
            r = max(r, max(max(v.z & 0xffffu, v.z >> 16), max(v.w & 0xffffu, v.w >> 16)));
        } else {
            for (int k = 0; k < 8 && x + k < nx; ++k) r = max(r, (unsigned int)p[x + k]);
        }
    }
    for (int o = 32; o > 0; o >>= 1) r = max(r, (unsigned int)__shfl_xor((int)r, o));
    if (lane == 0) red[threadIdx.x >> 6] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < NW; ++k) r = max(r, red[k]);
        if (r) atomicMax(out, r);
    }
}

// ---- parameters ------------------------------------------------------------
// Element i of the internal parameter vector: layer, and for a conv weight
// its (o, tap, c).  Returns the layer or -1; *kind = 0 weight, 1 bias.
struct ParamPos {
    int layer, kind, o, tap, c;
};
__device__ __forceinline__ ParamPos locate(const NetLayout &L, int i)
{
    ParamPos r{-1, 0, 0, 0, 0};
#pragma unroll
    for (int l = 0; l < kNetLayers; ++l) {
        const int kk = L.k[l] * L.k[l];
        const int nw = L.cout[l] * kk * L.cinp[l];
        if (i >= L.offw[l] && i < L.offw[l] + nw) {
            const int q = i - L.offw[l];
            r.layer = l;
            r.kind = 0;
            r.c = q % L.cinp[l];
            r.tap = (q / L.cinp[l]) % kk;
            r.o = q / (L.cinp[l] * kk);
        } else if (i >= L.offb[l] && i < L.offb[l] + L.cout[l]) {
            r.layer = l;
            r.kind = 1;
            r.o = i - L.offb[l];
        }
    }
    return r;
}

// write the bf16 copies of weight element (o, tap, c) of a 3x3 layer
__device__ __forceinline__ void store_copies(const NetLayout &L, const ParamPos &pp, float v,
                                             uint16_t *__restrict__ wt, uint16_t *__restrict__ wf, int i)
{
    const uint16_t h = (uint16_t)(pack2(v, 0.f) & 0xffffu);
    wt[i] = h;
    if (L.k[pp.layer] == 3)
        wf[L.offw[pp.layer] + ((size_t)pp.c * 9 + (8 - pp.tap)) * L.cout[pp.layer] + pp.o] = h;
}

// external (oracle order: per layer w[cout][cin][ky][kx], then b[cout]) ->
// internal masters + bf16 copies
__global__ void k_params_in(NetLayout L, const float *__restrict__ ext, float *__restrict__ master,
                            uint16_t *__restrict__ wt, uint16_t *__restrict__ wf)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= L.total_int) return;
    const ParamPos pp = locate(L, i);
    if (pp.layer < 0) return;
    const int l = pp.layer;
    float v;
    if (pp.kind == 1) {
        v = ext[L.extb[l] + pp.o];
    } else {
        const int k = L.k[l];
        v = pp.c < L.cin[l] ? ext[L.extw[l] + ((pp.o * L.cin[l] + pp.c) * k + pp.tap / k) * k + pp.tap % k] : 0.f;
    }
    master[i] = v;
    if (pp.kind == 0) store_copies(L, pp, v, wt, wf, i);
}

// internal -> external order
__global__ void k_params_out(NetLayout L, const float *__restrict__ master, float *__restrict__ ext)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= L.total_int) return;
    const ParamPos pp = locate(L, i);
    if (pp.layer < 0) return;
    const int l = pp.layer;
    if (pp.kind == 1) {
        ext[L.extb[l] + pp.o] = master[i];
    } else if (pp.c < L.cin[l]) {
        const int k = L.k[l];
        ext[L.extw[l] + ((pp.o * L.cin[l] + pp.c) * k + pp.tap / k) * k + pp.tap % k] = master[i];
    }
}

// Adam (Kingma & Ba) on the FP32 masters; bias corrections c1 = 1 / (1 -
// b1^t), c2 = 1 / (1 - b2^t) come from the host.  Padded input channels of
// the first layer stay zero.
__global__ void k_adam(NetLayout L, float *__restrict__ master, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ grad, uint16_t *__restrict__ wt, uint16_t *__restrict__ wf,
                       float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= L.total_int) return;
    const ParamPos pp = locate(L, i);
    if (pp.layer < 0) return;
    if (pp.kind == 0 && pp.c >= L.cin[pp.layer]) return;
    const float gi = grad[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi * c1, vh = vi * c2;
    const float p = master[i] - lr * mh / (sqrtf(vh) + eps);
    master[i] = p;
    if (pp.kind == 0) store_copies(L, pp, p, wt, wf, i);
}

__global__ void k_zero_u32n(unsigned int *__restrict__ w, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) w[i] = 0u;
}

// Per-image count of FREE cells; grid (blocks per image, images).  One block
// an image stores its count, several add theirs (integer additions are exact
// in any order).  Sixteen cells a load where `cls` is aligned for that.
__global__ __launch_bounds__(256) void k_count_free(const uint8_t *__restrict__ cls, int hw_pixels,
                                                    unsigned int *__restrict__ cnt)
{
    static_assert(TWG_CELL_FREE == 0, "FREE cells are counted as zero bytes");
    __shared__ unsigned int red[4];
    const uint8_t *c = cls + (size_t)blockIdx.y * hw_pixels;
    unsigned int n = 0;
    const int first = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
    if (!((uintptr_t)c & 15)) {  // images are multiples of 64 cells
#pragma unroll 8
        for (int p = first; p < hw_pixels / 16; p += step) {
            const uint4 v = reinterpret_cast<const uint4 *>(c)[p];
            n += (zero_bytes(v.x) + zero_bytes(v.y)) + (zero_bytes(v.z) + zero_bytes(v.w));
        }
    } else {
        for (int p = first; p < hw_pixels; p += step) n += c[p] == TWG_CELL_FREE;
    }
    for (int o = 32; o > 0; o >>= 1) n += (unsigned int)__shfl_xor((int)n, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x != 0) return;
    n = (red[0] + red[1]) + (red[2] + red[3]);
    if (gridDim.x == 1) cnt[blockIdx.y] = n;
    else if (n) atomicAdd(cnt + blockIdx.y, n);
}

// column c < 34 of part[nblk][34] summed by block c: thread t adds rows t,
// t + 256, ... in order, then a fixed tree over the 256 thread sums.
__global__ __launch_bounds__(256) void k_sum_loss(const float *__restrict__ part, int nblk, float *__restrict__ loss,
                                                  float *__restrict__ head_grad)
{
    __shared__ float red[256];
    const int c = blockIdx.x;
    float s = 0.f;
    for (int k = threadIdx.x; k < nblk; k += 256) s += part[(size_t)k * 34 + c];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (c < 33) head_grad[c] = red[0];
        else if (loss) loss[0] = red[0];
    }
}

}  // namespace

// ---- host side ----------------------------------------------------------------

NetLayout net_layout()
{
    static const int spec[kNetLayers][3] = {{3, 32, 3},   {32, 64, 3},  {64, 128, 3}, {128, 128, 3},
                                            {256, 64, 3}, {128, 32, 3}, {64, 32, 3},  {32, 1, 1}};
    NetLayout L{};
    int oi = 0, oe = 0;
    for (int l = 0; l < kNetLayers; ++l) {
        L.cin[l] = spec[l][0];
        L.cinp[l] = spec[l][0] < 32 ? 32 : spec[l][0];
        L.cout[l] = spec[l][1];
        L.k[l] = spec[l][2];
        const int kk = L.k[l] * L.k[l];
        L.offw[l] = oi;
        oi += L.cout[l] * kk * L.cinp[l];
        L.offb[l] = oi;
        oi += L.cout[l];
        L.extw[l] = oe;
        oe += L.cout[l] * kk * L.cin[l];
        L.extb[l] = oe;
        oe += L.cout[l];
    }
    L.total_int = oi;
    L.total_ext = oe;
    return L;
}

int net_forward(twg_unet *n, int nb, int H, int W, float *y, hipStream_t st)
{
    const NetLayout &L = n->L;
    const int cu = n->ctx->num_cu;
    const int H1 = H / 2, W1 = W / 2, H2 = H / 4, W2 = W / 4, H3 = H / 8, W3 = W / 8;
    auto args = [&](int l, const uint16_t *A, const uint16_t *Bs, uint16_t *out, uint16_t *pool, int h, int w) {
        return ConvArgs{A, Bs, n->wt + L.offw[l], n->master + L.offb[l], out, pool, n->master + L.offw[7],
                        n->master + L.offb[7], y, nb, h, w};
    };
    {
        const long long ntile = (long long)nb * ((W + kTS - 1) / kTS) * ((H + kTS - 1) / kTS);
        const int grid = (int)std::max<long long>(1, std::min<long long>(ntile, 2048));
        hipLaunchKernelGGL(k_conv3_in, dim3(grid), dim3(256), 0, st, n->xp, n->wt + L.offw[0], n->master + L.offb[0],
                           n->e0, n->p0, nb, H, W);
    }
    int rc = last_status();
    if (!rc) rc = launch_conv3<32, 64, kPlain, 0, kOutPool>(args(1, n->p0, nullptr, n->e1, n->p1, H1, W1), cu, st);
    if (!rc) rc = launch_conv3<64, 128, kPlain, 0, kOutPool>(args(2, n->p1, nullptr, n->e2, n->p2, H2, W2), cu, st);
    if (!rc) rc = launch_conv3<128, 128, kPlain, 0, kOutAct>(args(3, n->p2, nullptr, n->e3, nullptr, H3, W3), cu, st);
    if (!rc) rc = launch_conv3<256, 64, kUpCat, 128, kOutAct>(args(4, n->e3, n->e2, n->d2, nullptr, H2, W2), cu, st);
    if (!rc) rc = launch_conv3<128, 32, kUpCat, 64, kOutAct>(args(5, n->d2, n->e1, n->d1, nullptr, H1, W1), cu, st);
    const ConvArgs last = args(6, n->d1, n->e0, n->d0, nullptr, H, W);
    if (!rc) rc = y ? launch_conv3<64, 32, kUpCat, 32, kOutHead>(last, cu, st)
                    : launch_conv3<64, 32, kUpCat, 32, kOutAct>(last, cu, st);
    return rc;
}

int net_backward(twg_unet *n, int nb, int H, int W, const float *target, const uint8_t *cls, float *loss,
                 hipStream_t st)
{
    const NetLayout &L = n->L;
    const uint16_t *wf = n->wf;
    auto grad_args = [&](const uint16_t *g, int l, float *out, int h, int w) {
        return ConvArgs{g, nullptr, wf + L.offw[l], nullptr, out, nullptr, nullptr, nullptr, nullptr, nb, h, w};
    };
    // of a concatenation: the low activation's gradient (the first cin channels
    // of layer l's input), then, of the others, that of the skip connection
    auto up_args = [&](const uint16_t *g, int l, const uint16_t *low, uint16_t *dlow, int h, int w) {
        ConvArgs c = grad_args(g, l, nullptr, h, w);
        c.pool = dlow;
        c.act = low;
        return c;
    };
    auto skip_args = [&](const uint16_t *g, int l, const float *dp, const uint16_t *e, uint16_t *de, int h, int w) {
        ConvArgs c = grad_args(g, l, nullptr, h, w);
        c.wt += (size_t)(L.cin[l] / 2) * 9 * L.cout[l];
        c.out = de;
        c.act = e;
        c.dp = dp;
        return c;
    };
    auto GW = [&](int l) { return n->grad + L.offw[l]; };
    const int cu = n->ctx->num_cu;
    const int H1 = H / 2, W1 = W / 2, H2 = H / 4, W2 = W / 4, H3 = H / 8, W3 = W / 8;
    const int hwp = H * W, total = nb * hwp;
    // head and loss
    unsigned int *cnt = n->counts;
    // one block counts an image of up to 65536 cells (16 loads a thread: 4 us,
    // where zeroing and adding up 16 blocks' counts took 24)
    const int count_blocks = std::min(64, (hwp + 65535) / 65536);
    if (count_blocks > 1) hipLaunchKernelGGL(k_zero_u32n, dim3((nb + 255) / 256), dim3(256), 0, st, cnt, nb);
    hipLaunchKernelGGL(k_count_free, dim3(count_blocks, nb), dim3(256), 0, st, cls, hwp, cnt);
    const int nblk = (total + 255) / 256;
    hipLaunchKernelGGL(k_head_loss, dim3(nblk), dim3(256), 0, st, n->d0, n->master + L.offw[7],
                       n->master + L.offb[7], target, cls, cnt, hwp, nb, n->g_d0, nullptr, n->part);
    hipLaunchKernelGGL(k_sum_loss, dim3(34), dim3(256), 0, st, n->part, nblk, loss, n->grad + L.offw[7]);
    int rc = last_status();
    // d0: input cat(up(d1), e0) at H
    if (!rc) rc = launch_wgrad3<64, 32, kUpCat, 32>(n->d1, n->e0, n->g_d0, n->part, GW(6), nb, H, W, cu, st);
    if (!rc) rc = launch_conv3<32, 32, kPlain, 0, kOutUpGrad>(up_args(n->g_d0, 6, n->d1, n->g_d1, H, W), cu, st);
    // d1: input cat(up(d2), e1) at H/2
    if (!rc) rc = launch_wgrad3<128, 32, kUpCat, 64>(n->d2, n->e1, n->g_d1, n->part, GW(5), nb, H1, W1, cu, st);
    if (!rc) rc = launch_conv3<32, 64, kPlain, 0, kOutUpGrad>(up_args(n->g_d1, 5, n->d2, n->g_d2, H1, W1), cu, st);
    // d2: input cat(up(e3), e2) at H/4
    if (!rc) rc = launch_wgrad3<256, 64, kUpCat, 128>(n->e3, n->e2, n->g_d2, n->part, GW(4), nb, H2, W2, cu, st);
    if (!rc) rc = launch_conv3<64, 128, kPlain, 0, kOutUpGrad>(up_args(n->g_d2, 4, n->e3, n->g_e3, H2, W2), cu, st);
    // e3: input pool(e2) at H/8
    if (!rc) rc = launch_wgrad3<128, 128, kPlain, 0>(n->p2, nullptr, n->g_e3, n->part, GW(3), nb, H3, W3, cu, st);
    if (!rc) rc = launch_conv3<128, 128, kPlain, 0, kOutF32>(grad_args(n->g_e3, 3, n->f_p2, H3, W3), cu, st);
    if (!rc)
        rc = launch_conv3<64, 128, kPlain, 0, kOutSkipGrad>(skip_args(n->g_d2, 4, n->f_p2, n->e2, n->g_e2, H2, W2), cu, st);
    // e2: input pool(e1) at H/4
    if (!rc) rc = launch_wgrad3<64, 128, kPlain, 0>(n->p1, nullptr, n->g_e2, n->part, GW(2), nb, H2, W2, cu, st);
    if (!rc) rc = launch_conv3<128, 64, kPlain, 0, kOutF32>(grad_args(n->g_e2, 2, n->f_p1, H2, W2), cu, st);
    if (!rc)
        rc = launch_conv3<32, 64, kPlain, 0, kOutSkipGrad>(skip_args(n->g_d1, 5, n->f_p1, n->e1, n->g_e1, H1, W1), cu, st);
    // e1: input pool(e0) at H/2
    if (!rc) rc = launch_wgrad3<32, 64, kPlain, 0>(n->p0, nullptr, n->g_e1, n->part, GW(1), nb, H1, W1, cu, st);
    if (!rc) rc = launch_conv3<64, 32, kPlain, 0, kOutF32>(grad_args(n->g_e1, 1, n->f_p0, H1, W1), cu, st);
    if (!rc)
        rc = launch_conv3<32, 32, kPlain, 0, kOutSkipGrad>(skip_args(n->g_d0, 6, n->f_p0, n->e0, n->g_e0, H, W), cu, st);
    // e0: input x (padded to 32 channels)
    if (!rc) rc = launch_wgrad_in(n->xp, n->g_e0, n->part, GW(0), nb, H, W, cu, st);
    return rc;
}

int net_adam(twg_unet *n, float lr, hipStream_t st)
{
    const double b1 = 0.9, b2 = 0.999;
    n->adam_t += 1;
    const float c1 = (float)(1.0 / (1.0 - std::pow(b1, n->adam_t)));
    const float c2 = (float)(1.0 / (1.0 - std::pow(b2, n->adam_t)));
    hipLaunchKernelGGL(k_adam, dim3((n->L.total_int + 255) / 256), dim3(256), 0, st, n->L, n->master, n->m, n->v,
                       n->grad, n->wt, n->wf, lr, (float)b1, (float)b2, 1e-8f, c1, c2);
    return last_status();
}

int net_params_in(twg_unet *n, const float *ext, hipStream_t st)
{
    hipLaunchKernelGGL(k_params_in, dim3((n->L.total_int + 255) / 256), dim3(256), 0, st, n->L, ext, n->master,
                       n->wt, n->wf);
    return last_status();
}

int net_params_out(twg_unet *n, float *ext, hipStream_t st)
{
    hipLaunchKernelGGL(k_params_out, dim3((n->L.total_int + 255) / 256), dim3(256), 0, st, n->L, n->master, ext);
    return last_status();
}

int net_grads_out(twg_unet *n, float *ext, hipStream_t st)
{
    hipLaunchKernelGGL(k_params_out, dim3((n->L.total_int + 255) / 256), dim3(256), 0, st, n->L, n->grad, ext);
    return last_status();
}

int net_pack_input(twg_unet *n, const float *x, long long total, hipStream_t st)
{
    hipLaunchKernelGGL(k_pack_input, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, x, n->xp, total);
    return last_status();
}

int net_head_psi(twg_unet *n, const uint8_t *cls, float *psi, int nx, int ny, int pitch, int Wp, int32_t *status,
                 hipStream_t st)
{
    const dim3 grid((nx + 63) / 64, (ny + 3) / 4);
    hipLaunchKernelGGL(k_head_psi, rows_grid(nx, ny), dim3(256), 0, st, n->y, cls, psi, nx, ny, pitch, Wp, n->words + 1);
    hipLaunchKernelGGL(k_net_fallback, grid, dim3(256), 0, st, cls, psi, nx, ny, pitch, n->words + 1, status);
    return last_status();
}

int net_features_coarse(const uint8_t *cls, const uint16_t *ring, int nx, int ny, int pitch, int f, int Hc, int Wc,
                        int gx, int gy, const unsigned int *jmax, float *xf, uint16_t *xp, uint8_t *ccls,
                        hipStream_t st)
{
    const float inv_diag = (float)(1.0 / ((double)std::max(nx, ny) * std::sqrt(2.0)));
    hipLaunchKernelGGL(k_features_coarse, dim3((Wc + 63) / 64, (Hc + 3) / 4), dim3(256), 0, st, cls, ring, nx, ny,
                       pitch, f, Hc, Wc, gx, gy, inv_diag, jmax, xf, xp, ccls);
    return last_status();
}

int net_coarse_target(const float *psi, const uint8_t *cls, int nx, int ny, int pitch, int f, int Hc, int Wc,
                      float *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_coarse_target, dim3((Wc + 63) / 64, (Hc + 3) / 4), dim3(256), 0, st, psi, cls, nx, ny,
                       pitch, f, Hc, Wc, out);
    return last_status();
}

int net_up_psi(twg_unet *n, const float *yc, int Hc, int Wc, int f, const uint8_t *cls, float *psi, int nx, int ny,
               int pitch, int32_t *status, hipStream_t st)
{
    const dim3 grid((nx + 63) / 64, (ny + 3) / 4);
    hipLaunchKernelGGL(k_up_psi, rows_grid(nx, ny), dim3(256), 0, st, yc, Hc, Wc, f, cls, psi, nx, ny, pitch, n->words + 1);
    hipLaunchKernelGGL(k_net_fallback, grid, dim3(256), 0, st, cls, psi, nx, ny, pitch, n->words + 1, status);
    return last_status();
}

int net_zero_words(twg_unet *n, int count, hipStream_t st)
{
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, st, n->words, count);
    return last_status();
}

int net_features(const uint8_t *cls, const uint16_t *ring, int nx, int ny, int pitch, int Hp, int Wp, int gx,
                 int gy, const unsigned int *jmax, float *xf, uint16_t *xp, hipStream_t st)
{
    const float inv_diag = (float)(1.0 / ((double)std::max(nx, ny) * std::sqrt(2.0)));
    hipLaunchKernelGGL(k_features, rows_grid(Wp, Hp), dim3(256), 0, st, cls, ring, nx, ny, pitch,
                       Hp, Wp, gx, gy, inv_diag, jmax, xf, xp);
    return last_status();
}

int net_ring_max(const uint16_t *ring, int nx, int ny, int pitch, unsigned int *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_ring_max, dim3(kRingBlocks), dim3(kRingThreads), 0, st, ring, nx, ny, pitch, out);
    return last_status();
}


}  // namespace twg
