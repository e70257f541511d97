// The network's 3x3 convolutions on gfx950 matrix cores, as an implicit GEMM
// on v_mfma_f32_16x16x32_bf16: D[cout][pixel] = sum_k W[cout][k] In[k][pixel].
//
// A workgroup (4 waves) computes 32 output channels of a tile 16 pixels wide
// and 4 R high (R rows a wave).  Per 32-channel chunk of the input, the
// tile's halo and the chunk's weights are copied to LDS by the memory system
// itself (buffer loads with LDS as the destination: no staging registers, and
// the range check fills the pixels outside the image with zeros), then every
// wave keeps the chunk's 18 weight fragments in registers and walks its rows:
// R + 2 halo rows are read once per column shift for 9 R products of each
// fragment.  LDS holds the weights in fragment order and the halo with its
// 16-byte groups swizzled by the pixel's column, so every LDS read is free of
// bank conflicts.  A pixel's products are added in the order chunk, tap,
// whatever the tile, so every tiling gives the same bits.
//
// The tile height is chosen for the number of workgroups: R = 8 (a wave reads
// 67 KB of LDS per chunk for 144 products of 16 x 16 x 32; with R = 4, 43 KB for
// 72) as long as that leaves two workgroups per CU, else lower tiles (a 32 x 32
// layer has four 16 x 16 tiles, on a device of 256 CUs).  At 2048 x 2048 the
// layers of R = 8 reach 19 to 43 % of the matrix cores' rate: the rest is
// waiting for the halos at two workgroups a CU.
//
// The epilogue goes through LDS: stores are 16-byte runs of channels, the
// layers that the encoder pools write the 2x2 means as well (their consumers
// then read a quarter of the bytes, once, instead of pooling while staging),
// and the last layer's head is evaluated from LDS instead of from a stored
// activation.  The input gradient of a concatenation is never stored: the
// upsampled half leaves as 2x2 sums in bf16, and the skip half is computed
// when the pooled tensor's gradient, which adds to it, is there (its input is
// read once more; stored in FP32 in between, it was written and read twice).
// Loss and gradients of 16 x 256 x 256: 841 -> 661 us.
//
// Measured (whole calls, against 16 x 16 tiles that staged through registers,
// pooled while staging and loaded every wave's weights from global memory one
// tap ahead of their use): warm start at 2048 x 2048 1231 -> 583 us, at 1/8
// of it 214 -> 72 us.
#include "conv3.h"
#include "tile_map.h"
#include "unet_dev.h"

#include <algorithm>

namespace twg {

namespace {

using namespace ndev;

constexpr int kTW = 16;         // tile width
constexpr int kHW = kTW + 2;    // halo width
constexpr int kCK = 32;         // input channels per chunk
constexpr int kCO = 32;         // output channels per workgroup
constexpr int kSS = kCO + 8;    // LDS stride of an output pixel (bf16)
constexpr uint32_t kOutside = 0x80000000u;  // a byte offset no resource reaches

typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

// Large layers of at most two chunks keep all their weights in LDS, and two
// workgroups per CU go over the tiles (2048 x 2048: 88 -> 80 us for 32 -> 64
// channels at half resolution, 56 -> 53 for 64 -> 128 at a quarter, 200 -> 184
// for the last layer); deeper ones would leave one workgroup per CU, and the
// epilogues that read ahead have no registers left for the loop.
constexpr bool keeps_weights(int cin, int out, int R)
{
    return R == 8 && cin <= 2 * kCK && out != kOutSkipGrad && out != kOutF32;
}

// the value of the lane at the right of an even one
__device__ __forceinline__ float lane_right(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xb1, 0xf, 0xf, true));
}

// eight bf16 values, zero where e's are not positive
__device__ __forceinline__ uint4 where_positive(uint4 v, uint4 e)
{
    auto two = [](uint32_t a, uint32_t q) {
        return (bf_pos(q & 0xffffu) ? a & 0xffffu : 0u) | (bf_pos(q >> 16) ? a & 0xffff0000u : 0u);
    };
    return make_uint4(two(v.x, e.x), two(v.y, e.y), two(v.z, e.z), two(v.w, e.w));
}

template <int CIN, int COUT, int MODE, int CA, int OUT, int R>
__global__ __launch_bounds__(256, 2) void k_conv3(ConvArgs a, int tx, int ty)
{
    constexpr int NCO = COUT / kCO, NCH = CIN / kCK, CB = CIN - CA;
    constexpr int TH = 4 * R, NPX = (TH + 2) * kHW;
    constexpr int HG = (NPX * 4 + 63) / 64;  // halo copies of 64 x 16 bytes
    constexpr int HPW = (HG + 3) / 4, WPW = (18 + 3) / 4;  // per wave
    constexpr bool KEEP = keeps_weights(CIN, OUT, R);
    constexpr int STAGE = TH * kTW * kSS;
    constexpr int HALO = KEEP ? std::max(HG * 512, STAGE) : HG * 512;
    constexpr int LDS = KEEP ? HALO + NCH * 18 * 512 : std::max(HALO + 18 * 512, STAGE);  // bf16
    __shared__ __align__(16) uint16_t lds[LDS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int H = a.H, W = a.W;
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int co0 = (id % NCO) * kCO;
    auto tile = [&](const int t, const bool weights) __attribute__((always_inline)) {
        const int b = t / (tx * ty), r = t - b * (tx * ty);
        const int x0 = (r % tx) * kTW, y0 = (r / tx) * TH;

        // resources of the image rows the halo touches, and each lane's offsets
        // in them: slot 4 p + s of LDS takes channel group s ^ (column / 4) of
        // halo pixel p
        const int ylo = max(y0 - 1, 0), yhi = min(y0 + TH + 1, H);
        const size_t row = (size_t)b * H + ylo;
        __amdgpu_buffer_rsrc_t ra, rb;
        if constexpr (MODE == kPlain) {
            ra = rsrc(a.A + row * W * CIN, (uint32_t)(yhi - ylo) * W * CIN * 2);
            rb = ra;
        } else {
            const int W2 = W / 2;
            ra = rsrc(a.A + ((size_t)b * (H / 2) + ylo / 2) * W2 * CA,
                      (uint32_t)((yhi - 1) / 2 - ylo / 2 + 1) * W2 * CA * 2);
            rb = rsrc(a.Bs + row * W * CB, (uint32_t)(yhi - ylo) * W * CB * 2);
        }
        uint32_t oa[HPW], ob[HPW];
#pragma unroll
        for (int i = 0; i < HPW; ++i) {
            const int slot = (i * 4 + wave) * 64 + lane, p = slot >> 2;
            const int hy = p / kHW, hx = p - hy * kHW;
            const int cg = (slot & 3) ^ ((hx >> 2) & 3);
            const int yy = y0 + hy - 1, xx = x0 + hx - 1;
            const bool in = p < NPX && yy >= 0 && yy < H && xx >= 0 && xx < W;
            if constexpr (MODE == kPlain) {
                oa[i] = in ? (uint32_t)((yy - ylo) * W + xx) * (CIN * 2) + cg * 16 : kOutside;
            } else {
                oa[i] = in ? (uint32_t)((yy / 2 - ylo / 2) * (W / 2) + xx / 2) * (CA * 2) + cg * 16 : kOutside;
                ob[i] = in ? (uint32_t)((yy - ylo) * W + xx) * (CB * 2) + cg * 16 : kOutside;
            }
        }
        const __amdgpu_buffer_rsrc_t rw = rsrc(a.wt + (size_t)co0 * 9 * CIN, kCO * 9 * CIN * 2);
        const uint32_t ow = (uint32_t)(j * 9 * CIN + g * 8) * 2;
        auto copy16 = [&](__amdgpu_buffer_rsrc_t rs, int at, uint32_t vo, uint32_t so) __attribute__((always_inline)) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(lds + at), 16, (int)vo, (int)so, 0, 0);
        };
        auto load = [&](int ch) __attribute__((always_inline)) {
            const bool low = MODE == kPlain || ch < CA / kCK;
            const uint32_t so = (uint32_t)(low ? ch : ch - CA / kCK) * (kCK * 2);
#pragma unroll
            for (int i = 0; i < HPW; ++i) {
                const int q = i * 4 + wave;
                if (q >= HG) continue;
                if (low) copy16(ra, q * 512, oa[i], so);
                else copy16(rb, q * 512, MODE == kPlain ? oa[i] : ob[i], so);
            }
#pragma unroll
            for (int i = 0; i < WPW; ++i) {
                const int q = i * 4 + wave;  // tap * 2 + row block
                if (q >= 18 || !weights) continue;
                copy16(rw, HALO + (KEEP ? ch * 18 * 512 : 0) + q * 512, ow, (uint32_t)((q & 1) * 16 * 9 * CIN + (q >> 1) * CIN + ch * kCK) * 2);
            }
        };

        f32x4 acc[R][2];
#pragma unroll
        for (int ct = 0; ct < R; ++ct)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) acc[ct][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
        // this lane's halo fragment of row 0 of its wave at the three shifts
        const uint16_t *hp[3];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
            hp[dx] = lds + (((wave * R) * kHW + j + dx) * 4 + (g ^ (((j + dx) >> 2) & 3))) * 8;
        const uint16_t *wp = lds + HALO + lane * 8;

        load(0);
        // What the epilogue of an activation's gradient adds and masks by is read
        // ahead of the products, one memory latency less per tile (56 instead of
        // 69 us for 32 channels of 16 x 256 x 256); dp: a row of the pooled grid
        // serves two rows, with R = 1 every row its own.
        constexpr int ND = OUT == kOutSkipGrad || OUT == kOutUpGrad ? (R + 1) / 2 : 1, NE = OUT == kOutSkipGrad ? R : 1;
        float4 dp[ND][2];
        uint4 ev[NE];
        uint2 lv[ND][2];  // kOutUpGrad
        if constexpr (OUT == kOutUpGrad) {
            const int x = min(x0 + j, W - 1);
#pragma unroll
            for (int q = 0; q < R / 2; ++q) {
                const int y = min(y0 + wave * R + 2 * q, H - 1);
                const uint16_t *l = a.act + (((size_t)b * (H / 2) + y / 2) * (W / 2) + x / 2) * COUT + co0 + g * 4;
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) lv[q][rt] = *reinterpret_cast<const uint2 *>(l + rt * 16);
            }
        }
        auto read_mask = [&] {
#pragma unroll
            for (int q = 0; q < NE; ++q) {
                const int p = (tid + 256 * q) >> 2;
                const int y = min(y0 + p / kTW, H - 1), xe = min(x0 + p % kTW, W - 1);
                ev[q] = *reinterpret_cast<const uint4 *>(a.act + (((size_t)b * H + y) * W + xe) * COUT + co0 + (tid & 3) * 8);
            }
        };
        if constexpr (OUT == kOutSkipGrad) {
            const int x = min(x0 + j, W - 1);
            const float *d = a.dp + ((size_t)b * (H / 2) * (W / 2) + x / 2) * COUT + co0 + g * 4;
#pragma unroll
            for (int q = 0; q < ND; ++q) {
                const int y = min(y0 + wave * R + 2 * q, H - 1);
#pragma unroll
                for (int rt = 0; rt < 2; ++rt)
                    dp[q][rt] = *reinterpret_cast<const float4 *>(d + (size_t)(y / 2) * (W / 2) * COUT + rt * 16);
            }
            if (NCH == 1) read_mask();  // with more chunks the registers do not reach
        }
        for (int ch = 0; ch < NCH; ++ch) {
            // the copies of every wave have landed
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            uint4 w[18];
#pragma unroll
            for (int q = 0; q < 18; ++q) w[q] = *reinterpret_cast<const uint4 *>(wp + ((KEEP ? ch * 18 : 0) + q) * 512);
            // two rows at a time: four independent chains of products
            constexpr int RB = R > 1 ? 2 : 1;
#pragma unroll
            for (int c0 = 0; c0 < R; c0 += RB) {
                uint4 h[RB + 2][3];
#pragma unroll
                for (int q = 0; q < RB + 2; ++q)
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
                        h[q][dx] = *reinterpret_cast<const uint4 *>(hp[dx] + (c0 + q) * kHW * 32);
#pragma unroll
                for (int tap = 0; tap < 9; ++tap)
#pragma unroll
                    for (int c = 0; c < RB; ++c)
#pragma unroll
                        for (int rt = 0; rt < 2; ++rt)
                            acc[c0 + c][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                as_bf8(w[tap * 2 + rt]), as_bf8(h[c + tap / 3][tap % 3]), acc[c0 + c][rt], 0, 0, 0);
            }
            __syncthreads();
            if (ch + 1 < NCH) load(ch + 1);
        }
        if constexpr (OUT == kOutSkipGrad && NCH > 1) read_mask();

        if constexpr (OUT == kOutUpGrad) {
            // 2x2 sums, left to right and top to bottom: rows in this lane's
            // registers, the column at its right in the next lane; H and W are
            // even, so a pair lies inside whole
            const int W2 = W / 2, H2 = H / 2, x = x0 + j;
#pragma unroll
            for (int ct = 0; ct + 1 < R; ct += 2) {
                const int y = y0 + wave * R + ct;
                const bool in = !(j & 1) && y < H && x < W;
                const size_t at = (((size_t)b * H2 + y / 2) * W2 + x / 2) * COUT + co0 + g * 4;
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    float s[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        s[i] = (((0.f + acc[ct][rt][i]) + lane_right(acc[ct][rt][i])) + acc[ct + 1][rt][i]) +
                               lane_right(acc[ct + 1][rt][i]);
                    if (!in) continue;
                    const uint2 av = lv[ct / 2][rt];
                    *reinterpret_cast<uint2 *>(a.pool + at + rt * 16) =
                        make_uint2(pack2(bf_pos(av.x & 0xffffu) ? s[0] : 0.f, bf_pos(av.x >> 16) ? s[1] : 0.f),
                                   pack2(bf_pos(av.y & 0xffffu) ? s[2] : 0.f, bf_pos(av.y >> 16) ? s[3] : 0.f));
                }
            }
        } else if constexpr (OUT == kOutF32) {
            const int x = x0 + j;
#pragma unroll
            for (int ct = 0; ct < R; ++ct) {
                const int y = y0 + wave * R + ct;
                if (y >= H || x >= W) continue;
                float *o = static_cast<float *>(a.out) + (((size_t)b * H + y) * W + x) * COUT + co0 + g * 4;
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    const f32x4 v = acc[ct][rt];
                    *reinterpret_cast<float4 *>(o + rt * 16) = make_float4(v[0], v[1], v[2], v[3]);
                }
            }
        } else {
            // the tile as bf16(relu(acc + bias)), or bf16(acc + dp / 4), in LDS,
            // pixel by pixel
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                if constexpr (OUT == kOutSkipGrad) {
#pragma unroll
                    for (int ct = 0; ct < R; ++ct) {
                        const float4 d = dp[ct / 2][rt];
                        const f32x4 v = acc[ct][rt];
                        *reinterpret_cast<uint2 *>(lds + ((wave * R + ct) * kTW + j) * kSS + rt * 16 + g * 4) =
                            make_uint2(pack2(v[0] + d.x * 0.25f, v[1] + d.y * 0.25f),
                                       pack2(v[2] + d.z * 0.25f, v[3] + d.w * 0.25f));
                    }
                    continue;
                }
                const float *bp = a.bias + co0 + rt * 16 + g * 4;
                const float b0 = bp[0], b1 = bp[1], b2 = bp[2], b3 = bp[3];
#pragma unroll
                for (int ct = 0; ct < R; ++ct) {
                    const f32x4 v = acc[ct][rt];
                    *reinterpret_cast<uint2 *>(lds + ((wave * R + ct) * kTW + j) * kSS + rt * 16 + g * 4) =
                        make_uint2(pack2(relu(v[0] + b0), relu(v[1] + b1)), pack2(relu(v[2] + b2), relu(v[3] + b3)));
                }
            }
            __syncthreads();
            if constexpr (OUT == kOutHead) {
                for (int p = tid; p < TH * kTW; p += 256) {
                    const int y = y0 + p / kTW, x = x0 + p % kTW;
                    uint4 v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const uint4 *>(lds + p * kSS + q * 8);
                    float d[32];
                    const float yv = head_value(v, a.hw, a.hb[0], d);
                    if (y < H && x < W) a.y[((size_t)b * H + y) * W + x] = yv;
                }
            } else {
                uint16_t *out = static_cast<uint16_t *>(a.out);
#pragma unroll
                for (int k = 0; k < R; ++k) {  // TH * kTW pixels, 4 groups each
                    const int q = tid + 256 * k, p = q >> 2, c8 = q & 3;
                    const int y = y0 + p / kTW, x = x0 + p % kTW;
                    uint4 v = *reinterpret_cast<const uint4 *>(lds + p * kSS + c8 * 8);
                    if (y >= H || x >= W) continue;
                    const size_t at = (((size_t)b * H + y) * W + x) * COUT + co0 + c8 * 8;
                    if constexpr (OUT == kOutSkipGrad) v = where_positive(v, ev[k]);
                    *reinterpret_cast<uint4 *>(out + at) = v;
                }
                if constexpr (OUT == kOutPool) {
                    const int H2 = H / 2, W2 = W / 2;
                    for (int q = tid; q < TH * kTW; q += 256) {  // TH / 2 x kTW / 2 pixels, 4 groups each
                        const int p = q >> 2, c8 = q & 3, py = p / (kTW / 2), px = p % (kTW / 2);
                        const int y = y0 / 2 + py, x = x0 / 2 + px;
                        const uint16_t *s = lds + ((2 * py) * kTW + 2 * px) * kSS + c8 * 8;
                        const uint4 v = mean4(*reinterpret_cast<const uint4 *>(s), *reinterpret_cast<const uint4 *>(s + kSS),
                                              *reinterpret_cast<const uint4 *>(s + kTW * kSS),
                                              *reinterpret_cast<const uint4 *>(s + kTW * kSS + kSS));
                        if (y < H2 && x < W2)
                            *reinterpret_cast<uint4 *>(a.pool + (((size_t)b * H2 + y) * W2 + x) * COUT + co0 + c8 * 8) = v;
                    }
                }
            }
        }
    };
    if constexpr (KEEP) {
        bool first = true;
        for (int t = id / NCO; t < a.nb * tx * ty; t += (int)gridDim.x / NCO) {
            if (!first) __syncthreads();  // the last tile's LDS is read
            tile(t, first);
            first = false;
        }
    } else {
        tile(id / NCO, true);
    }
}

template <int CIN, int COUT, int MODE, int CA, int OUT, int R>
int launch_r(const ConvArgs &a, int wgs, hipStream_t st)
{
    const int tx = (a.W + kTW - 1) / kTW, ty = (a.H + 4 * R - 1) / (4 * R);
    unsigned blocks = (unsigned)(a.nb * tx * ty * (COUT / kCO));
    if (keeps_weights(CIN, OUT, R)) blocks = std::min(blocks, (unsigned)(wgs / (COUT / kCO) * (COUT / kCO)));
    hipLaunchKernelGGL((k_conv3<CIN, COUT, MODE, CA, OUT, R>), dim3(blocks), dim3(256), 0, st, a, tx, ty);
    return hipGetLastError() == hipSuccess ? TWG_OK : TWG_EDEVICE;
}

}  // namespace

template <int CIN, int COUT, int MODE, int CA, int OUT>
int launch_conv3(const ConvArgs &a, int num_cu, hipStream_t st)
{
    // workgroups at R rows per wave
    auto groups = [&](int R) {
        return (long long)a.nb * ((a.W + kTW - 1) / kTW) * ((a.H + 4 * R - 1) / (4 * R)) * (COUT / kCO);
    };
    const long long want = 2LL * std::max(1, num_cu);
    if (groups(8) >= want) return launch_r<CIN, COUT, MODE, CA, OUT, 8>(a, (int)want, st);
    if (groups(4) >= want) return launch_r<CIN, COUT, MODE, CA, OUT, 4>(a, (int)want, st);
    // (2x2 sums take a wave's rows in pairs)
    if (OUT == kOutUpGrad || groups(2) >= want) return launch_r<CIN, COUT, MODE, CA, OUT, 2>(a, (int)want, st);
    if constexpr (OUT != kOutUpGrad) return launch_r<CIN, COUT, MODE, CA, OUT, 1>(a, (int)want, st);
}

// forward
template int launch_conv3<32, 64, kPlain, 0, kOutPool>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<64, 128, kPlain, 0, kOutPool>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<128, 128, kPlain, 0, kOutAct>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<256, 64, kUpCat, 128, kOutAct>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<128, 32, kUpCat, 64, kOutAct>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<64, 32, kUpCat, 32, kOutAct>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<64, 32, kUpCat, 32, kOutHead>(const ConvArgs &, int, hipStream_t);
// input gradients
template int launch_conv3<32, 32, kPlain, 0, kOutUpGrad>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<32, 64, kPlain, 0, kOutUpGrad>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<64, 128, kPlain, 0, kOutUpGrad>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<32, 32, kPlain, 0, kOutSkipGrad>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<32, 64, kPlain, 0, kOutSkipGrad>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<64, 128, kPlain, 0, kOutSkipGrad>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<128, 128, kPlain, 0, kOutF32>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<128, 64, kPlain, 0, kOutF32>(const ConvArgs &, int, hipStream_t);
template int launch_conv3<64, 32, kPlain, 0, kOutF32>(const ConvArgs &, int, hipStream_t);

}  // namespace twg
