// Weight and bias gradients of the network's 3x3 convolutions on gfx950
// matrix cores: dW[cout][tap][c] = sum_pixels dOut[p][cout] In[p + tap][c],
// the reduction over pixels as the K dimension of
// v_mfma_f32_16x16x32_bf16 (32 pixels of one row per product).
//
// A workgroup takes one 32-channel chunk of the input and every split-th tile
// of 32 x TH pixels.  The tile's output gradient and input halo go to LDS as
// they lie in memory (pixel by pixel, channels contiguous; the memory system
// copies them and fills what lies outside the image with zeros), and the
// fragments, which need eight pixels of one channel per lane, are read with
// the transposing LDS load: no transposed copy is ever written (writing the
// halo as three shifted, transposed copies, two bytes at a time, took most of
// the previous kernel).  A wave keeps the accumulators of 16 input channels,
// nine taps and up to 64 output channels, and walks its rows with the last
// three rows' fragments in registers: a row costs three new input fragments
// and COUT / 16 gradient fragments for 9 COUT / 16 products.
//
// The splits' partial sums are added in a fixed order by k_sum_parts, so the
// gradients do not depend on scheduling.
#include "tile_map.h"
#include "unet_dev.h"
#include "wgrad3.h"

#include <algorithm>

namespace twg {

namespace {

using namespace ndev;

constexpr int kTW = 32;       // tile width: the pixels of one product
constexpr int kHW = kTW + 2;  // halo width
constexpr int kCK = 32;       // input channels per workgroup
constexpr uint32_t kOutside = 0x80000000u;  // a byte offset no resource reaches

typedef short s16x4 __attribute__((__vector_size__(8)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void copy16(__amdgpu_buffer_rsrc_t r, uint16_t *to, uint32_t vo)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)to, 16, (int)vo, 0, 0, 0);
}
// lane (j, g) receives element j of the 16-element rows that lanes 16 g + 4 e
// .. 16 g + 4 e + 3 address, for e = 0 .. 3 (each lane addresses four
// elements)
__device__ __forceinline__ uint2 read_tr(const uint16_t *p)
{
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p));
}

// Swizzle of a pixel's 16-byte channel groups in LDS (P of them), by the
// pixel's column: the four pixels a transposing load touches lie in
// different banks.
template <int P> __device__ __forceinline__ int swz(int col)
{
    return P == 4 ? (col >> 2) & 3 : P == 8 ? ((col >> 1) & 3) * 2 : (col & 7) * 2;
}

// output channels per wave, rows per wave and tile height
template <int COUT> struct Shape {
    static constexpr int WO = COUT / 16;
    // waves split rows (32 output channels), else output channels: at most
    // 64 a wave, whose 144 accumulator registers leave two waves a SIMD
    static constexpr bool kByRows = WO == 2;
    static constexpr int NOT = kByRows ? WO : WO / 2, TH = WO <= 4 ? 8 : 4, NR = kByRows ? TH / 2 : TH;
};

template <int CIN, int COUT, int MODE, int CA>
__global__ __launch_bounds__(256, 2) void k_wgrad3(const uint16_t *__restrict__ A, const uint16_t *__restrict__ Bs,
                                                   const uint16_t *__restrict__ dout, float *__restrict__ part,
                                                   int nb, int H, int W, int nsplit)
{
    using S = Shape<COUT>;
    constexpr int NOT = S::NOT, TH = S::TH, NR = S::NR, NCH = CIN / kCK, CB = CIN - CA;
    constexpr int PO = COUT / 8;                                  // 16-byte groups of an output pixel
    constexpr int NPX = (TH + 2) * kHW, HG = (NPX * 4 + 63) / 64;  // halo copies of 64 x 16 bytes
    constexpr int OG = TH * kTW * PO / 64;
    constexpr int HALO = HG * 512, RED = S::kByRows ? 2 * NOT * 9 * 256 * 2 : 0;  // bf16 units
    __shared__ __align__(16) uint16_t lds[std::max(HALO + OG * 512, RED)];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int ch = id % NCH, split = id / NCH;
    const int cti = wave & 1, ot0 = S::kByRows ? 0 : (wave >> 1) * NOT, r0 = S::kByRows ? (wave >> 1) * NR : 0;
    const int tx = (W + kTW - 1) / kTW, ty = (H + TH - 1) / TH, per = tx * ty, ntile = nb * per;
    const bool low = MODE == kPlain || ch < CA / kCK;

    f32x4 acc[NOT][9];
    float bsum[NOT];
#pragma unroll
    for (int q = 0; q < NOT; ++q) {
        bsum[q] = 0.f;
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    uint16_t *ldo = lds + HALO;
    // a lane's place in a transposing load: pixel i / 4 of four, channels
    // 4 (i % 4) .. + 3 of sixteen
    const int li = lane & 15, lp = li >> 2, lg = (li & 3) >> 1, lh = (li & 1) * 4;
    auto frag = [&](const uint16_t *row, int P, int col, int c16, auto sw) __attribute__((always_inline)) -> uint4 {
        uint2 v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = col + g * 8 + h * 4 + lp;
            v[h] = read_tr(row + (c * P + ((c16 * 2 + lg) ^ sw(c))) * 8 + lh);
        }
        return make_uint4(v[0].x, v[0].y, v[1].x, v[1].y);
    };
    auto in_frag = [&](int row, int dx) __attribute__((always_inline)) {
        return frag(lds + row * kHW * 32, 4, dx, cti, [](int c) { return swz<4>(c); });
    };
    auto out_frag = [&](int row, int ot) __attribute__((always_inline)) {
        return frag(ldo + row * kTW * COUT, PO, 0, ot, [](int c) { return swz<PO>(c); });
    };

    for (int t = split; t < ntile; t += nsplit) {
        const int b = t / per, r = t - b * per;
        const int y0 = (r / tx) * TH, x0 = (r % tx) * kTW;
        const int ylo = max(y0 - 1, 0), yhi = min(y0 + TH + 1, H);
        const __amdgpu_buffer_rsrc_t ro = rsrc(dout + ((size_t)b * H + y0) * W * COUT,
                                               (uint32_t)(min(y0 + TH, H) - y0) * W * COUT * 2);
        __amdgpu_buffer_rsrc_t ri;
        if (MODE != kPlain && low)
            ri = rsrc(A + ((size_t)b * (H / 2) + ylo / 2) * (W / 2) * CA,
                      (uint32_t)((yhi - 1) / 2 - ylo / 2 + 1) * (W / 2) * CA * 2);
        else if (MODE != kPlain)
            ri = rsrc(Bs + ((size_t)b * H + ylo) * W * CB, (uint32_t)(yhi - ylo) * W * CB * 2);
        else
            ri = rsrc(A + ((size_t)b * H + ylo) * W * CIN, (uint32_t)(yhi - ylo) * W * CIN * 2);
        __syncthreads();  // the previous tile has been read
#pragma unroll
        for (int i = 0; i < (HG + 3) / 4; ++i) {
            const int q = i * 4 + wave;
            if (q >= HG) continue;
            const int slot = q * 64 + lane, p = slot >> 2, hy = p / kHW, hx = p - hy * kHW;
            const int c8 = (slot & 3) ^ swz<4>(hx), yy = y0 + hy - 1, xx = x0 + hx - 1;
            const bool in = p < NPX && yy >= 0 && yy < H && xx >= 0 && xx < W;
            uint32_t o;
            if (MODE != kPlain && low)
                o = (uint32_t)((yy / 2 - ylo / 2) * (W / 2) + xx / 2) * (CA * 2) + ch * (kCK * 2);
            else if (MODE != kPlain)
                o = (uint32_t)((yy - ylo) * W + xx) * (CB * 2) + (ch - CA / kCK) * (kCK * 2);
            else
                o = (uint32_t)((yy - ylo) * W + xx) * (CIN * 2) + ch * (kCK * 2);
            copy16(ri, lds + q * 512, in ? o + c8 * 16 : kOutside);
        }
#pragma unroll
        for (int i = 0; i < OG / 4; ++i) {
            const int q = i * 4 + wave, slot = q * 64 + lane, p = slot / PO, oy = p / kTW, ox = p % kTW;
            const int c8 = (slot % PO) ^ swz<PO>(ox);
            const bool in = y0 + oy < H && x0 + ox < W;
            copy16(ro, ldo + q * 512, in ? (uint32_t)(oy * W + x0 + ox) * (COUT * 2) + c8 * 16 : kOutside);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        uint4 in[NR + 2][3];
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) in[y][dx] = in_frag(r0 + y, dx);
#pragma unroll
        for (int y = 0; y < NR; ++y) {
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) in[y + 2][dx] = in_frag(r0 + y + 2, dx);
#pragma unroll
            for (int q = 0; q < NOT; ++q) {
                const uint4 ov = out_frag(r0 + y, ot0 + q);
                if (ch == 0 && cti == 0) {
                    float v[8];
                    unpack8(ov, v);
                    bsum[q] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
                }
#pragma unroll
                for (int tap = 0; tap < 9; ++tap)
                    acc[q][tap] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(ov), as_bf8(in[y + tap / 3][tap % 3]),
                                                                         acc[q][tap], 0, 0, 0);
            }
        }
    }

    // a lane holds dW[ot * 16 + 4 g + v][tap][ch * 32 + cti * 16 + j]; where
    // the waves split rows, the second half's sums are added to the first's
    float *out = part + (size_t)split * (COUT * 9 * CIN + COUT);
    const int c = ch * kCK + cti * 16 + j;
    float *red = reinterpret_cast<float *>(lds) + cti * (2 * 9 * 256);
#pragma unroll
    for (int q = 0; q < NOT; ++q) {
        if (S::kByRows) {
            if ((q & 1) == 0) {  // two output channel blocks at a time
                __syncthreads();
                if (wave >= 2)
#pragma unroll
                    for (int e = 0; e < 2; ++e)
#pragma unroll
                        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
                            for (int v = 0; v < 4; ++v) red[((e * 9 + tap) * 4 + v) * 64 + lane] = acc[q + e][tap][v];
                __syncthreads();
            }
            if (wave >= 2) continue;
        }
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = (ot0 + q) * 16 + g * 4 + v;
                const float s = S::kByRows ? acc[q][tap][v] + red[(((q & 1) * 9 + tap) * 4 + v) * 64 + lane]
                                           : acc[q][tap][v];
                out[(o * 9 + tap) * CIN + c] = s;
            }
    }
    if (ch == 0) {
        __syncthreads();
        float *rb = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int q = 0; q < NOT; ++q) {
            float s = bsum[q] + __shfl_xor(bsum[q], 16);
            s = s + __shfl_xor(s, 32);
            if (cti == 0 && g == 0) rb[(wave >> 1) * COUT + (ot0 + q) * 16 + j] = s;
        }
        __syncthreads();
        if (tid < COUT)
            out[COUT * 9 * CIN + tid] = S::kByRows ? rb[tid] + rb[COUT + tid] : rb[(tid / (NOT * 16)) * COUT + tid];
    }
}

// First layer: its three input channels make the nine taps' 27 (tap, channel)
// pairs one 32-column product.  x4 [B][H][W][4] bf16; a lane's column is
// pair n = tap * 3 + c, its eight pixels two bytes each in LDS.  part[split]
// holds [32][32] (cout, n), then the bias sums.
__global__ __launch_bounds__(256) void k_wgrad_in(const uint16_t *__restrict__ x4, const uint16_t *__restrict__ dout,
                                                  float *__restrict__ part, int nb, int H, int W, int nsplit)
{
    constexpr int COUT = 32, TH = 8, NPX = (TH + 2) * kHW, OG = TH * kTW * 4 / 64, RED = 4 * 4 * 256;
    __shared__ __align__(16) uint16_t ldo[std::max(OG * 512, RED * 2)];
    __shared__ __align__(16) uint16_t ldx[NPX * 4];
    __shared__ float rb[4][32];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int split = xcd_remap(blockIdx.x, gridDim.x);
    const int tx = (W + kTW - 1) / kTW, ty = (H + TH - 1) / TH, per = tx * ty, ntile = nb * per;
    f32x4 acc[2][2];
    float bsum[2] = {0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[q][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    int at[2];
    uint32_t live[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int k = n * 16 + j, tap = k < 27 ? k / 3 : 0, c = k < 27 ? k - 3 * tap : 0;
        at[n] = ((tap / 3) * kHW + tap % 3 + g * 8) * 4 + c;
        live[n] = k < 27 ? 0xffffffffu : 0u;
    }
    const int lp = (lane & 15) >> 2, lg = (lane & 3) >> 1, lh = (lane & 1) * 4;
    for (int t = split; t < ntile; t += nsplit) {
        const int b = t / per, r = t - b * per;
        const int y0 = (r / tx) * TH, x0 = (r % tx) * kTW;
        const __amdgpu_buffer_rsrc_t ro = rsrc(dout + ((size_t)b * H + y0) * W * COUT,
                                               (uint32_t)(min(y0 + TH, H) - y0) * W * COUT * 2);
        __syncthreads();  // the previous tile has been read
#pragma unroll
        for (int i = 0; i < OG / 4; ++i) {
            const int q = i * 4 + wave, slot = q * 64 + lane, p = slot >> 2, oy = p / kTW, ox = p % kTW;
            const int c8 = (slot & 3) ^ swz<4>(ox);
            const bool in = y0 + oy < H && x0 + ox < W;
            copy16(ro, ldo + q * 512, in ? (uint32_t)(oy * W + x0 + ox) * (COUT * 2) + c8 * 16 : kOutside);
        }
        for (int p = tid; p < NPX; p += 256) {
            const int hy = p / kHW, hx = p - hy * kHW, yy = y0 + hy - 1, xx = x0 + hx - 1;
            const bool in = yy >= 0 && yy < H && xx >= 0 && xx < W;
            const uint2 v = *reinterpret_cast<const uint2 *>(
                x4 + (((size_t)b * H + min(max(yy, 0), H - 1)) * W + min(max(xx, 0), W - 1)) * 4);
            *reinterpret_cast<uint2 *>(ldx + p * 4) = in ? v : make_uint2(0, 0);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int row = wave * 2 + y;
            uint4 xv[2];
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const uint16_t *p = ldx + row * kHW * 4 + at[n];
                uint32_t w[4];
#pragma unroll
                for (int h = 0; h < 4; ++h) w[h] = ((uint32_t)p[8 * h] | ((uint32_t)p[8 * h + 4] << 16)) & live[n];
                xv[n] = make_uint4(w[0], w[1], w[2], w[3]);
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                uint2 h[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int c = g * 8 + e * 4 + lp;
                    h[e] = read_tr(ldo + ((row * kTW + c) * 4 + ((q * 2 + lg) ^ swz<4>(c))) * 8 + lh);
                }
                const uint4 ov = make_uint4(h[0].x, h[0].y, h[1].x, h[1].y);
                float v[8];
                unpack8(ov, v);
                bsum[q] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
#pragma unroll
                for (int n = 0; n < 2; ++n)
                    acc[q][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(ov), as_bf8(xv[n]), acc[q][n], 0, 0, 0);
            }
        }
    }
    // the four waves' sums, in order
    float *red = reinterpret_cast<float *>(ldo);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[((wave * 2 + q) * 2 + n) * 256 + (g * 4 + v) * 16 + j] = acc[q][n][v];
        float s = bsum[q] + __shfl_xor(bsum[q], 16);
        s = s + __shfl_xor(s, 32);
        if (g == 0) rb[wave][q * 16 + j] = s;
    }
    __syncthreads();
    float *out = part + (size_t)split * (32 * 32 + 32);
    for (int i = tid; i < 1024; i += 256) {
        const int o = i >> 5, n = i & 31;
        const float *p = red + ((o >> 4) * 2 + (n >> 4)) * 256 + (o & 15) * 16 + (n & 15);
        out[i] = ((p[0] + p[1024]) + p[2048]) + p[3072];
    }
    if (tid < 32) out[1024 + tid] = ((rb[0][tid] + rb[1][tid]) + rb[2][tid]) + rb[3][tid];
}

// out[i] = sum over s < n of part[s * count + i].  A block covers 256 / Q
// consecutive i with Q lanes each; lane q adds s = q, q + Q, ... in order and
// the lane sums are added in lane order, so the result does not depend on
// scheduling.  IN: the first layer's [32][32] + 32 layout into [32][9][32]
// (channels from 3 on are not parameters) + 32.
template <int Q, bool IN>
__global__ __launch_bounds__(256) void k_sum_parts(const float *__restrict__ part, float *__restrict__ out, int count,
                                                   int n)
{
    constexpr int NI = 256 / Q;
    __shared__ float red[Q][NI];
    const int q = threadIdx.x / NI, l = threadIdx.x % NI;
    const int i = blockIdx.x * NI + l;
    float s = 0.f;
    if (i < count) {
#pragma unroll 8
        for (int k = q; k < n; k += Q) s += part[(size_t)k * count + i];
    }
    red[q][l] = s;
    __syncthreads();
    if (q != 0 || i >= count) return;
#pragma unroll
    for (int k = 1; k < Q; ++k) s += red[k][l];
    if (!IN) {
        out[i] = s;
    } else if (i >= 1024) {
        out[32 * 9 * 32 + (i - 1024)] = s;
    } else if ((i & 31) < 27) {
        const int tap = (i & 31) / 3, c = (i & 31) - 3 * tap;
        out[((i >> 5) * 9 + tap) * 32 + c] = s;
    }
}

int last_status() { return hipGetLastError() == hipSuccess ? TWG_OK : TWG_EDEVICE; }

// Splits of the pixel reduction: per_cu workgroups per CU (two; with 128 output
// channels, whose products fill a CU by themselves, one: its partial sums are
// half the bytes, 18 + 13 to 16 + 8 us at 32 x 32 x 16), at most one per tile,
// and partial sums within the scratch.
int choose_split(int nchunk, int ntile, int count, int per_cu, int num_cu)
{
    const int s = std::min(std::max(1, per_cu * std::max(1, num_cu) / nchunk), (int)(kPartFloats / count));
    return std::max(1, std::min(s, ntile));
}

template <bool IN>
int sum_parts(const float *part, float *g, int count, int ns, hipStream_t st)
{
    if (count >= 32768)
        hipLaunchKernelGGL((k_sum_parts<4, IN>), dim3((count + 63) / 64), dim3(256), 0, st, part, g, count, ns);
    else
        hipLaunchKernelGGL((k_sum_parts<16, IN>), dim3((count + 15) / 16), dim3(256), 0, st, part, g, count, ns);
    return last_status();
}

int tiles(int nb, int H, int W, int TH) { return nb * ((H + TH - 1) / TH) * ((W + kTW - 1) / kTW); }

}  // namespace

template <int CIN, int COUT, int MODE, int CA>
int launch_wgrad3(const uint16_t *A, const uint16_t *Bs, const uint16_t *dout, float *part, float *g, int nb, int H,
                  int W, int num_cu, hipStream_t st)
{
    constexpr int NCH = CIN / kCK, count = COUT * 9 * CIN + COUT;
    const int ns = choose_split(NCH, tiles(nb, H, W, Shape<COUT>::TH), count, COUT > 64 ? 1 : 2, num_cu);
    hipLaunchKernelGGL((k_wgrad3<CIN, COUT, MODE, CA>), dim3(NCH * ns), dim3(256), 0, st, A, Bs, dout, part, nb, H, W,
                       ns);
    return sum_parts<false>(part, g, count, ns, st);
}

int launch_wgrad_in(const uint16_t *x4, const uint16_t *dout, float *part, float *g, int nb, int H, int W, int num_cu,
                    hipStream_t st)
{
    constexpr int count = 32 * 32 + 32;
    const int ns = choose_split(1, tiles(nb, H, W, 8), count, 2, num_cu);
    hipLaunchKernelGGL(k_wgrad_in, dim3(ns), dim3(256), 0, st, x4, dout, part, nb, H, W, ns);
    return sum_parts<true>(part, g, count, ns, st);
}

template int launch_wgrad3<64, 32, kUpCat, 32>(const uint16_t *, const uint16_t *, const uint16_t *, float *, float *,
                                               int, int, int, int, hipStream_t);
template int launch_wgrad3<128, 32, kUpCat, 64>(const uint16_t *, const uint16_t *, const uint16_t *, float *, float *,
                                                int, int, int, int, hipStream_t);
template int launch_wgrad3<256, 64, kUpCat, 128>(const uint16_t *, const uint16_t *, const uint16_t *, float *,
                                                 float *, int, int, int, int, hipStream_t);
template int launch_wgrad3<128, 128, kPlain, 0>(const uint16_t *, const uint16_t *, const uint16_t *, float *, float *,
                                                int, int, int, int, hipStream_t);
template int launch_wgrad3<64, 128, kPlain, 0>(const uint16_t *, const uint16_t *, const uint16_t *, float *, float *,
                                               int, int, int, int, hipStream_t);
template int launch_wgrad3<32, 64, kPlain, 0>(const uint16_t *, const uint16_t *, const uint16_t *, float *, float *,
                                              int, int, int, int, hipStream_t);

}  // namespace twg
