// Map update on the time-warped grid (Algorithm 1, "Map Update"; sections
// "Time-Warped Grid" and "Integration of Kalman Filter with Time-Warps").
//
//   k_map    ring number and the WALL / GOAL / static-OBST / FREE class, eight
//            cells a thread.
//   k_discs  per (obstacle, ring), one lane makes the constant-velocity
//            Kalman prediction of Eq. (9) to the ring's horizon, its Q.8 disc (optionally grown by the
//            predicted position covariance), and a conservative test of
//            whether the disc can touch the ring and the grid; the survivors
//            are marked by the whole wave: an exact integer test of every
//            cell of the disc's bounding box (ring match + inside the disc).
//            A marked cell that is not a border wall or the goal becomes
//            OBST: nothing is read back, and every writer stores the same
//            byte, so the result does not depend on the order.  With the
//            per-object horizon of Algorithm 1 the obstacle has one disc, at
//            the horizon of its own ring.
//
// Bound by launches and latency (500 discs on 2048 x 2048: 12.6 MB, 2.5 us at
// the copy rate): two launches instead of four (a counter cleared, cells, a
// list of (obstacle, ring) pairs built with atomics, and its scatter), squares
// and ring numbers in 32 bits instead of FP64 square roots and 64-bit
// divisions.
//
// Exactness: the horizon, the product and the sum of the prediction are each
// rounded once (contraction is off for this file), 256*mu is exact, and the
// Q.8 rounding is round-half-to-even; the inside test is in 64-bit integers.
#include "twg_internal.h"

#include <algorithm>

namespace twg {

namespace {

struct Disc {
    long long cx, cy, R;  // Q.8 centre and radius
    int j;                // ring, or -1: all its cells
};

__device__ __forceinline__ int dev_isqrt(long long n)
{
    long long s = (long long)sqrt((double)n);
    while (s * s > n) --s;
    while ((s + 1) * (s + 1) <= n) ++s;
    return (int)s;
}

__device__ __forceinline__ int ring_of(long long dx, long long dy, int W)
{
    return dev_isqrt(dx * dx + dy * dy) / W;
}

// Elliptical warp metric (Eqs. 14-15): relative to the robot, with heading
// (hc, hs), u = hc dx + hs dy and v = hs dx - hc dy; the ellipse through the
// cell has its centre 0.9 r_x ahead and r_x = 4 r_y, so
// r_x = (-1.8 u + sqrt(4 u^2 + 12.16 v^2)) / 0.38.  Ring j = floor(r_x / W)
// is settled by the exact, monotone test r_x >= j W  <=>  0.38 j W + 1.8 u
// <= 0 or 4 u^2 + 12.16 v^2 >= (0.38 j W + 1.8 u)^2 (each term one rounded
// IEEE operation, so host and device agree bit for bit).
__host__ __device__ inline bool ellipse_reaches(double u, double v, int j, int W)
{
    const double q = 4.0 * (u * u) + 12.16 * (v * v);
    const double rhs = 0.38 * ((double)j * (double)W) + 1.8 * u;
    return rhs <= 0.0 || q >= rhs * rhs;
}

__host__ __device__ inline int ring_ellipse(long long dx, long long dy, double hc, double hs, int W)
{
    const double u = hc * (double)dx + hs * (double)dy;
    const double v = hs * (double)dx - hc * (double)dy;
    const double r = (-1.8 * u + sqrt(4.0 * (u * u) + 12.16 * (v * v))) / 0.38;  // estimate only
    int j = (r > 0.0 && r < 1e9) ? (int)(r / (double)W) : 0;
    while (j > 0 && !ellipse_reaches(u, v, j, W)) --j;
    while (ellipse_reaches(u, v, j + 1, W)) ++j;
    return j;
}

struct WarpMode {
    int ring_mode;  // 0 circular, 1 elliptical
    double hc, hs;  // heading
};

// floor(floor(sqrt(n)) / W) for a squared distance of two cells: the largest j
// with (j W)^2 <= n.  n < 2^31, so the root is below 46341: the hardware root
// is within 0.02 of it and the product with 1 / W within 0.01 of its quotient,
// so one step up or down makes j exact.  Every product has 24-bit factors (a
// 32-bit multiply takes four times as long): W counts up to 65536, where every
// j is 0, and the next ring's edge up to 65535, beyond any root.
__device__ __forceinline__ int ring_of_square(uint32_t n, uint32_t W, float inv_w)
{
    uint32_t j = (uint32_t)(__builtin_amdgcn_sqrtf((float)n) * inv_w);
    const uint32_t t = __umul24(j, W), u = min(t + W, 65535u);
    j -= __umul24(t, t) > n ? 1u : 0u;
    return (int)(j + (__umul24(u, u) <= n ? 1u : 0u));
}
__device__ __forceinline__ int ring_of_cells(int dx, int dy, int W, float inv_w)
{
    return ring_of_square((uint32_t)(__mul24(dx, dx) + __mul24(dy, dy)), (uint32_t)min(W, 65536), inv_w);
}

// Disc radius with covariance inflation: r + min(W, kappa sqrt(lambda_max)),
// lambda_max the larger eigenvalue of the position covariance after horizon
// t, P_pos(t) = P_pp + t (P_pv + P_vp) + t^2 P_vv (P row-major 4x4, state
// [x, y, vx, vy]).  kappa = 0 or no covariance: r.
__device__ __forceinline__ double inflated_radius(double r, const double *P, double t, double kappa, int W)
{
    if (!(kappa > 0.0) || !P) return r;
    const double tt = t * t;
    const double a = (P[0] + t * (P[2] + P[8])) + tt * P[10];
    const double b = (P[1] + t * (P[3] + P[9])) + tt * P[11];
    const double d = (P[5] + t * (P[7] + P[13])) + tt * P[15];
    const double h = (a - d) * 0.5;
    const double lam = (a + d) * 0.5 + sqrt(h * h + b * b);
    double g = kappa * sqrt(lam > 0.0 ? lam : 0.0);
    if (!(g <= (double)W)) g = (double)W;
    return r + g;
}

__device__ __forceinline__ long long floor_div256(long long a)
{
    return a >= 0 ? a / 256 : -((-a + 255) / 256);
}

// The obstacle's disc at ring j's horizon, to be marked on the cells of ring
// j; with the per-object horizon (Algorithm 1), its disc at the horizon of
// the ring of the cell nearest its current centre, to be marked whole (j is
// then -1).  False if it cannot touch a cell.
template <bool ELL>
__device__ __forceinline__ bool disc_at(int j, bool per_object, double px, double py, double vx, double vy, double r,
                                        const double *cov, double kappa, const WarpMode &wm, int W, double vr, int nx,
                                        int ny, int xr, int yr, Disc *out)
{
    if (!(r >= 0.0 && r <= 1e6)) return false;
    if (per_object) {
        const double cx = rint(px), cy = rint(py);
        if (!(fabs(cx) < 1e9) || !(fabs(cy) < 1e9)) return false;
        const long long ox = (long long)cx - xr, oy = (long long)cy - yr;
        j = ELL ? ring_ellipse(ox, oy, wm.hc, wm.hs, W) : ring_of(ox, oy, W);
    }
    // Eq. (9) with A(t): position p + t v, each operation rounded once
    const double t = ((double)j * (double)W) / vr;
    const double tvx = t * vx, tvy = t * vy;
    const double mx = px + tvx, my = py + tvy;
    const double sx = 256.0 * mx, sy = 256.0 * my;
    if (!(fabs(sx) < 1099511627776.0) || !(fabs(sy) < 1099511627776.0)) return false;
    const long long cx = (long long)rint(sx), cy = (long long)rint(sy);
    const double re = inflated_radius(r, cov, t, kappa, W);
    const long long R = (long long)rint(256.0 * re);
    // disc must reach the grid
    if (cx + R < 0 || cx - R > 256LL * (nx - 1) || cy + R < 0 || cy - R > 256LL * (ny - 1)) return false;
    if (!per_object) {
        // ...and ring j: cells of the disc lie within R of its centre; ring j
        // holds Euclidean distances [jW, (j+1)W) (circular) or, since the
        // elliptical r_x lies between d / 1.9 and 10 d, [jW / 10, 1.9 (j+1) W)
        // (elliptical); two cells of margin absorb rounding
        const double dx = (double)cx / 256.0 - xr, dy = (double)cy / 256.0 - yr;
        const double D = sqrt(dx * dx + dy * dy), Rc = (double)R / 256.0;
        const double lo = ELL ? (double)j * W / 10.0 : (double)j * W;
        const double hi = ELL ? 1.9 * (double)(j + 1) * W : (double)(j + 1) * W;
        if (D - Rc - 2.0 >= hi) return false;
        if (D + Rc + 2.0 < lo) return false;
    }
    *out = Disc{cx, cy, R, per_object ? -1 : j};
    return true;
}

// arguments of a map update's kernels (pairs: (obstacle, ring); waves: those
// that share them)
struct MapArgs {
    int nx, ny, pitch, xr, yr, xg, yg, W, border, J, per_object, vec;
    float inv_w;
    WarpMode wm;
    const uint8_t *static_occ;
    uint8_t *cls;
    uint16_t *ring;
    const double *pos, *vel, *rad, *cov;
    double kappa, vr;
    long long pairs, waves;
};

// Eight cells from x0 on.  VEC: pitch and bases allow 8-byte class and 16-byte
// ring stores.  ELL: the elliptical metric (its FP64 code is kept out of the
// other kernels).
template <bool ELL>
__device__ __forceinline__ void map_cells(const MapArgs &a, bool VEC, int x0, int y)
{
    const int nx = a.nx, ny = a.ny, pitch = a.pitch, xr = a.xr, yr = a.yr, xg = a.xg, yg = a.yg, W = a.W;
    const int border = a.border;
    const float inv_w = a.inv_w;
    const WarpMode wm = a.wm;
    const uint8_t *__restrict__ static_occ = a.static_occ;
    uint8_t *__restrict__ cls = a.cls;
    uint16_t *__restrict__ ring = a.ring;
    if (x0 >= nx || y >= ny) return;
    const size_t i = (size_t)y * pitch + x0;
    const bool whole = VEC && x0 + 8 <= nx;
    // classes, a byte each: static occupancy, then the goal, then the walls
    const uint64_t kOnes = 0x0101010101010101ull;
    uint64_t c = 0ull;
    if (static_occ) {
        if (whole) {
            const uint64_t v = *reinterpret_cast<const uint64_t *>(static_occ + i);
            c = ((((v & 0x7f * kOnes) + 0x7f * kOnes) | v) >> 7 & kOnes) * TWG_CELL_OBST;
        } else {
            for (int k = 0; k < 8; ++k)
                if (x0 + k < nx && static_occ[i + k]) c |= (uint64_t)TWG_CELL_OBST << 8 * k;
        }
    }
    auto set = [&](int k, uint64_t v) { c = (c & ~(0xffull << 8 * k)) | v << 8 * k; };
    if (y == yg && xg >= x0 && xg < x0 + 8) set(xg - x0, TWG_CELL_GOAL);
    if (border) {
        if (y == 0 || y == ny - 1) c = TWG_CELL_WALL * kOnes;
        if (x0 == 0) set(0, TWG_CELL_WALL);
        if (nx - 1 - x0 < 8) set(nx - 1 - x0, TWG_CELL_WALL);
    }
    uint32_t r[8];
    if (ring) {
        const int dx = x0 - xr, dy = y - yr;
        const uint32_t Wc = (uint32_t)min(W, 65536);
        uint32_t n = (uint32_t)(__mul24(dx, dx) + __mul24(dy, dy));
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            r[k] = (uint32_t)(ELL ? ring_ellipse(dx + k, dy, wm.hc, wm.hs, W) : ring_of_square(n, Wc, inv_w));
            n += (uint32_t)(2 * (dx + k) + 1);
        }
    }
    if (whole) {
        *reinterpret_cast<uint64_t *>(cls + i) = c;
        if (ring)
            *reinterpret_cast<uint4 *>(ring + i) = make_uint4(r[0] | r[1] << 16, r[2] | r[3] << 16, r[4] | r[5] << 16,
                                                              r[6] | r[7] << 16);
    } else {
        for (int k = 0; k < 8; ++k)
            if (x0 + k < nx) {
                cls[i + k] = (uint8_t)(c >> 8 * k);
                if (ring) ring[i + k] = (uint16_t)r[k];
            }
    }
}

// 32 x 8 threads of 8 cells
template <bool VEC, bool ELL>
__global__ __launch_bounds__(256) void k_map(MapArgs a)
{
    map_cells<ELL>(a, VEC, (blockIdx.x * 32 + (threadIdx.x & 31)) * 8, blockIdx.y * 8 + (threadIdx.x >> 5));
}

// Wave w of n_waves takes the (obstacle, ring) pairs w, w + n_waves, ..., one
// a lane, so that the rings of one obstacle (a disc that moves with the rings
// meets a hundred of them) go to different waves, then marks the discs that
// survive one after another.
template <bool ELL>
__device__ __forceinline__ void mark_discs(const MapArgs &a, long long w)
{
    const int lane = threadIdx.x & 63;
    const int nx = a.nx, ny = a.ny, pitch = a.pitch, xr = a.xr, yr = a.yr, xg = a.xg, yg = a.yg, W = a.W, J = a.J;
    const int border = a.border, per_object = a.per_object;
    const float inv_w = a.inv_w;
    const double kappa = a.kappa, vr = a.vr;
    const WarpMode wm = a.wm;
    const long long n_pairs = a.pairs, n_waves = a.waves;
    const double *__restrict__ pos = a.pos, *__restrict__ vel = a.vel, *__restrict__ rad = a.rad;
    const double *__restrict__ cov = a.cov;
    uint8_t *cls = a.cls;
    if (w >= n_waves) return;
    // cells a disc may mark: not the border walls
    const int xa = border ? 1 : 0, xb = border ? nx - 2 : nx - 1, ya = border ? 1 : 0, yb = border ? ny - 2 : ny - 1;
    const long long id = w + lane * n_waves;
    Disc d{};
    bool hit = false;
    if (id < n_pairs) {
        const long long i = per_object ? id : id >> 32 ? id / J : (long long)((uint32_t)id / (uint32_t)J);
        const int j = per_object ? 0 : (int)(id - i * J);
        hit = disc_at<ELL>(j, per_object, pos[2 * i], pos[2 * i + 1], vel[2 * i], vel[2 * i + 1], rad[i],
                      cov ? cov + 16 * i : nullptr, kappa, wm, W, vr, nx, ny, xr, yr, &d);
    }
    {
        for (unsigned long long todo = __ballot(hit); todo; todo &= todo - 1) {
            const int l = __builtin_ctzll(todo);
            const Disc p{__shfl(d.cx, l), __shfl(d.cy, l), __shfl(d.R, l), __shfl(d.j, l)};
            const int x0 = (int)max(-floor_div256(-(p.cx - p.R)), (long long)xa);
            const int x1 = (int)min(floor_div256(p.cx + p.R), (long long)xb);
            const int y0 = (int)max(-floor_div256(-(p.cy - p.R)), (long long)ya);
            const int y1 = (int)min(floor_div256(p.cy + p.R), (long long)yb);
            auto mark = [&](int x, int y) {
                if (p.j >= 0 && (ELL ? ring_ellipse(x - xr, y - yr, wm.hc, wm.hs, W)
                                     : ring_of_cells(x - xr, y - yr, W, inv_w)) != p.j)
                    return;
                if (x != xg || y != yg) cls[(size_t)y * pitch + x] = TWG_CELL_OBST;
            };
            // 8 x 8 cells at a time
            if (p.R < 65000) {  // squares within the box fit 32 bits
                const uint32_t R2 = (uint32_t)p.R * (uint32_t)p.R;
                for (int y = y0 + (lane >> 3); y <= y1; y += 8) {
                    const int dy = (int)(256LL * y - p.cy);
                    const uint32_t dy2 = (uint32_t)dy * (uint32_t)dy;
                    if (dy2 > R2) continue;
                    for (int x = x0 + (lane & 7); x <= x1; x += 8) {
                        const int dx = (int)(256LL * x - p.cx);
                        if ((uint32_t)dx * (uint32_t)dx <= R2 - dy2) mark(x, y);
                    }
                }
            } else {
                const long long R2 = p.R * p.R;
                for (int y = y0 + (lane >> 3); y <= y1; y += 8) {
                    const long long dy = 256LL * y - p.cy, in2 = R2 - dy * dy;
                    if (in2 < 0) continue;
                    for (int x = x0 + (lane & 7); x <= x1; x += 8) {
                        const long long dx = 256LL * x - p.cx;
                        if (dx * dx <= in2) mark(x, y);
                    }
                }
            }
        }
    }
}

template <bool ELL>
__global__ __launch_bounds__(256) void k_discs(MapArgs a)
{
    mark_discs<ELL>(a, (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// A small map whole in one workgroup: the cells, then the discs.  Each launch
// costs a call 3 us on the host, which bounds small maps (64 x 64 with 10
// discs: 10.5 us a call in two launches, 7.5 in one).
constexpr int kSmallCells = 16384, kSmallWaves = 16, kSmallPairs = 12 * kSmallWaves;
template <bool ELL>
__global__ __launch_bounds__(64 * kSmallWaves) void k_map_small(MapArgs a)
{
    const int groups = (a.nx + 7) / 8;
    for (int u = threadIdx.x; u < groups * a.ny; u += 64 * kSmallWaves) map_cells<ELL>(a, a.vec, u % groups * 8, u / groups);
    __syncthreads();
    mark_discs<ELL>(a, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

int host_ring(long long dx, long long dy, int W)
{
    unsigned long long d2 = (unsigned long long)(dx * dx + dy * dy);
    unsigned long long s = (unsigned long long)std::sqrt((double)d2);
    while (s * s > d2) --s;
    while ((s + 1) * (s + 1) <= d2) ++s;
    return (int)(s / (unsigned long long)W);
}

}  // namespace

int launch_rasterize(twg_ctx *ctx, const twg_grid &g, int n_obs, const double *pos,
                     const double *vel, const double *rad, const uint8_t *static_occ,
                     const twg_raster_params &p, uint8_t *cls, uint16_t *ring, hipStream_t st)
{
    const int nx = g.nx, ny = g.ny, pitch = g.pitch;
    const WarpMode wm{p.ring_mode, p.heading_x, p.heading_y};
    // rings touching the grid: the metric is convex in the offset (a norm
    // plus a linear term), so the largest ring is reached at a corner
    int J = 0;
    const int cxs[2] = {0, nx - 1}, cys[2] = {0, ny - 1};
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) {
            const long long dx = cxs[a] - p.robot_x, dy = cys[b] - p.robot_y;
            const int j = p.ring_mode == 1 ? ring_ellipse(dx, dy, wm.hc, wm.hs, p.ring_width)
                                           : host_ring(dx, dy, p.ring_width);
            if (j > J) J = j;
        }
    if (J > 65535) return set_err(ctx, TWG_EUNSUPPORTED, "more than 65536 rings: increase ring_width");
    J += 1;
    const float inv_w = 1.0f / (float)p.ring_width;
    const auto al = [](const void *q, uintptr_t a) { return (reinterpret_cast<uintptr_t>(q) & (a - 1)) == 0; };
    const bool vec = pitch % 8 == 0 && al(cls, 8) && al(ring, 16) && al(static_occ, 8);
    const bool ell = p.ring_mode == 1;
    // a full wave's worth of pairs each, but at least 4096 waves (or one pair
    // each): a wave marks its discs one after another (500 discs on 2048 x 2048:
    // 9.6 us with 2048 waves, 8.4, and 9.4 with 8192)
    const long long pairs = (long long)n_obs * (p.per_object ? 1 : J);
    MapArgs a{nx, ny, pitch, p.robot_x, p.robot_y, p.goal_x, p.goal_y, p.ring_width, p.border_walls, J, p.per_object,
              vec, inv_w, wm, static_occ, cls, ring, pos, vel, rad, p.cov, p.kappa, p.robot_speed, pairs,
              std::max((pairs + 63) / 64, std::min(pairs, 4096LL))};
    auto launch = [&](auto kernel, dim3 grid, int threads) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, st, a);
        return hipGetLastError() == hipSuccess;
    };
    // one launch where 16 waves soon have every cell and disc: up to 12 discs a
    // wave (7.5 to 9.3 us a call against 10.5 in two launches; with 20 discs a
    // wave it is 11)
    if ((long long)nx * ny <= kSmallCells && pairs > 0 && pairs <= kSmallPairs) {
        a.waves = std::min<long long>(pairs, kSmallWaves);
        const bool ok = ell ? launch(k_map_small<true>, dim3(1), 64 * kSmallWaves)
                            : launch(k_map_small<false>, dim3(1), 64 * kSmallWaves);
        return ok ? TWG_OK : set_err(ctx, TWG_EDEVICE, "map launch failed");
    }
    const dim3 grid((nx + 255) / 256, (ny + 7) / 8);
    const bool ok = vec ? (ell ? launch(k_map<true, true>, grid, 256) : launch(k_map<true, false>, grid, 256))
                        : (ell ? launch(k_map<false, true>, grid, 256) : launch(k_map<false, false>, grid, 256));
    if (!ok) return set_err(ctx, TWG_EDEVICE, "map launch failed");
    if (n_obs == 0) return TWG_OK;
    const dim3 blocks((unsigned)((a.waves + 3) / 4));
    if (!(ell ? launch(k_discs<true>, blocks, 256) : launch(k_discs<false>, blocks, 256)))
        return set_err(ctx, TWG_EDEVICE, "rasterize launch failed");
    return TWG_OK;
}

}  // namespace twg
