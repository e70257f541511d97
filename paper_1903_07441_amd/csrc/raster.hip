// Map update on the time-warped grid (Algorithm 1, "Map Update"; sections
// "Time-Warped Grid" and "Integration of Kalman Filter with Time-Warps").
//
//   k_map    ring number and the WALL / GOAL / static-OBST / FREE class, eight
//            cells a thread.
//   k_discs  per (obstacle, ring), one lane makes the constant-velocity
//            Kalman prediction of Eq. (9) to the ring's horizon, its Q.8 disc (optionally grown by the
//            predicted position covariance), and a conservative test of
//            whether the disc can touch the ring and the grid; the survivors
//            are marked by the whole wave, or by several: an exact integer test
//            (ring match + inside the disc) of the cells of the disc's bounding
//            box, in large discs of those near its ring.
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
// divisions.  Large discs are bound by their cells' tests.  The four launches,
// then a wave that walks a disc's whole box, then this (us a call):
//   2048 x 2048, 500 discs of radius 3 to 12      27.9    14.5    14.4
//   2048 x 2048, 10 discs of radius 300            826     743      34
//   the same, elliptical                          3860    4820     945
//   512 x 512, 10 discs of radius 100, elliptical  219     606      67
//   128 x 128, 8 discs of radius 30 (one launch)    20      49      10
//
// Exactness: the horizon, the product and the sum of the prediction are each
// rounded once (contraction is off for this file), 256*mu is exact, and the
// Q.8 rounding is round-half-to-even; the inside test is in 64-bit integers.
#include "twg_internal.h"

#include <algorithm>
#include <type_traits>

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
    return (rhs <= 0.0) | (q >= rhs * rhs);
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
        // holds Euclidean distances [jW, (j+1)W) (circular); two cells of margin
        // absorb rounding.  Elliptical: [jW / 10, 1.9 (j+1) W) is taken, from
        // r_x between d / 1.9 and 10 d.  The upper end is wrong: r_x / d is
        // 10.85 at 130.6 degrees off the heading, so ring j begins at
        // 0.0922 jW, and a disc that ends between 0.0922 jW - 2 and
        // 0.1 jW - 2 cells from the robot is not marked on ring j (seen from
        // rings of r_x = 256 on, behind the robot).  Changing it changes maps.
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

// Cells x0 .. x1, y0 .. y1 (inclusive).
struct Box {
    int x0, x1, y0, y1;
};

// Marks the cells of disc p in box b, one wave, the strips of 8 rows that are
// slice `slice` of `slices`: 8 x 8 cells at a time, each with the exact disc
// and ring test.  ELL: a cell is of ring j where the metric reaches j and not
// j + 1 (it is monotone in j), which spares the ring number's square root and
// divisions.  A strip wider than 32 cells is first cut, row by row, to the
// disc's chord and the circular ring's two intervals (a square root in FP32
// and a margin each), so that a large disc costs a wave the cells of its ring
// and not its bounding box.  I: int while the squares of the box fit 32 bits,
// else long long.
template <bool ELL, typename I>
__device__ __forceinline__ void mark_disc(const MapArgs &a, const Disc &p, const Box &b, int slice, int slices)
{
    using U = std::make_unsigned_t<I>;
    const int lane = threadIdx.x & 63;
    const int W = a.W, j = p.j;
    const I cx = (I)p.cx, cy = (I)p.cy, R = (I)p.R;
    const U R2 = (U)R * (U)R;
    // squared distances of ring j's cells: [lo, hi] (no two cells are 2^31 apart)
    const unsigned long long far = 0x7fffffffull, jw = (unsigned long long)max(j, 0) * W, kw = jw + W;
    const uint32_t lo = (uint32_t)(jw < 46341 ? jw * jw : far), hi = (uint32_t)(kw < 46341 ? kw * kw - 1 : far);
    const bool ringed = j >= 0, wide = b.x1 - b.x0 >= 32;
    for (int y = b.y0 + slice * 8 + (lane >> 3); y <= b.y1; y += 8 * slices) {
        const I dy = (I)256 * y - cy;
        const U dy2 = (U)dy * (U)dy;
        if (dy2 > R2) continue;
        const U in2 = R2 - dy2;
        const int ry = y - a.yr;
        const uint32_t ry2 = (uint32_t)__mul24(ry, ry);
        int from[2] = {b.x0, 1}, to[2] = {b.x1, 0};
        if (wide) {
            const I h = (I)__builtin_amdgcn_sqrtf((float)in2) + (R >> 20) + 2;
            const int xa = max(b.x0, (int)((cx - h) >> 8)), xb = min(b.x1, (int)((cx + h) >> 8) + 1);
            from[0] = xa;
            to[0] = xb;
            if (!ELL && ringed) {
                if (ry2 > hi) continue;
                const int out = (int)__builtin_amdgcn_sqrtf((float)(hi - ry2)) + 2;
                const int in = ry2 < lo ? max((int)__builtin_amdgcn_sqrtf((float)(lo - ry2)) - 2, 0) : 0;
                from[0] = max(xa, a.xr - out);
                to[0] = min(xb, a.xr - in);
                from[1] = max(xa, a.xr + in);
                to[1] = min(xb, a.xr + out);
            }
        }
        const double ny = (double)ry;
        uint8_t *row = a.cls + (size_t)y * a.pitch;
        auto mark = [&](int x, int last) {
            const I dx = (I)256 * x - cx;
            bool ok = x <= last && (U)dx * (U)dx <= in2 && !(x == a.xg && y == a.yg);
            if (ringed) {
                const int rx = x - a.xr;
                if constexpr (ELL) {
                    const double u = a.wm.hc * (double)rx + a.wm.hs * ny, v = a.wm.hs * (double)rx - a.wm.hc * ny;
                    ok = ok & ((j == 0) | ellipse_reaches(u, v, j, W)) & !ellipse_reaches(u, v, j + 1, W);
                } else {
                    const uint32_t n = ry2 + (uint32_t)__mul24(rx, rx);
                    ok = ok && n >= lo && n <= hi;
                }
            }
            if (ok) row[x] = TWG_CELL_OBST;
        };
        if (!ELL && !wide) {
            for (int x = b.x0 + (lane & 7); x <= b.x1; x += 8) mark(x, b.x1);
            continue;
        }
#pragma unroll
        for (int s = 0; s < (ELL ? 1 : 2); ++s)
            for (int x = from[s] + (lane & 7); x <= to[s]; x += 16) {
                mark(x, to[s]);
                mark(x + 8, to[s]);
            }
    }
}

// Wave w of a.waves takes the (obstacle, ring) pairs w, w + a.waves, ..., one
// a lane, so that the rings of one obstacle (a disc that moves with the rings
// meets a hundred of them) go to different waves, then marks the discs that
// survive one after another in the cells of `clip` (their slice of them).
template <bool ELL>
__device__ __forceinline__ void mark_discs(const MapArgs &a, long long w, const Box &clip, int slice, int slices)
{
    const int lane = threadIdx.x & 63;
    const int W = a.W, J = a.J, per_object = a.per_object;
    const double *__restrict__ pos = a.pos, *__restrict__ vel = a.vel, *__restrict__ rad = a.rad;
    const double *__restrict__ cov = a.cov;
    if (w >= a.waves) return;
    const long long id = w + lane * a.waves;
    Disc d{};
    Box b{};
    bool hit = false;
    if (id < a.pairs) {
        const long long i = per_object ? id : id >> 32 ? id / J : (long long)((uint32_t)id / (uint32_t)J);
        const int j = per_object ? 0 : (int)(id - i * J);
        hit = disc_at<ELL>(j, per_object, pos[2 * i], pos[2 * i + 1], vel[2 * i], vel[2 * i + 1], rad[i],
                           cov ? cov + 16 * i : nullptr, a.kappa, a.wm, W, a.vr, a.nx, a.ny, a.xr, a.yr, &d);
        // the disc's cells, rounded inwards, in the clip
        b = Box{(int)max((d.cx - d.R + 255) >> 8, (long long)clip.x0), (int)min((d.cx + d.R) >> 8, (long long)clip.x1),
                (int)max((d.cy - d.R + 255) >> 8, (long long)clip.y0), (int)min((d.cy + d.R) >> 8, (long long)clip.y1)};
        hit = hit && b.x0 <= b.x1 && b.y0 <= b.y1;
    }
    // (a lane's words in scalar registers: the marking's uniform part is
    // scalar work)
    for (unsigned long long todo = __ballot(hit); todo; todo &= todo - 1) {
        const int l = __builtin_ctzll(todo);
        auto word = [&](int v) { return __builtin_amdgcn_readlane(v, l); };
        auto both = [&](long long v) {
            return (long long)((unsigned long long)(uint32_t)word((int)(v >> 32)) << 32 | (uint32_t)word((int)v));
        };
        const Disc p{both(d.cx), both(d.cy), both(d.R), word(d.j)};
        const Box q{word(b.x0), word(b.x1), word(b.y0), word(b.y1)};
        if (p.R < 65000) mark_disc<ELL, int>(a, p, q, slice, slices);
        else mark_disc<ELL, long long>(a, p, q, slice, slices);
    }
}

// cells a disc may mark: not the border walls
__device__ __forceinline__ Box markable(const MapArgs &a)
{
    const int e = a.border ? 1 : 0;
    return Box{e, a.nx - 1 - e, e, a.ny - 1 - e};
}

// gridDim.y waves share a group of pairs
template <bool ELL>
__global__ __launch_bounds__(256) void k_discs(MapArgs a)
{
    mark_discs<ELL>(a, (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), markable(a),
                    blockIdx.y, gridDim.y);
}

// A small map in one launch: a workgroup writes the cells of its tile (64
// columns of `rows`, at most 64, rows), then marks every disc's part of it: the
// predictions are made again in every tile, large discs are shared by them.
// Each launch costs a call 3 us on the host, which bounds small maps (64 x 64
// with 10 discs: 10.5 us a call in two launches, 8.2 in one; 128 x 128 with 190
// discs of radius 30, 18 us, 144 when one workgroup took the whole map).
constexpr int kSmallCells = 16384, kSmallWaves = 16, kSmallPairs = 12 * kSmallWaves;
constexpr int kSmallW = 64;
template <bool ELL>
__global__ __launch_bounds__(64 * kSmallWaves) void k_map_small(MapArgs a, int rows)
{
    const int x0 = blockIdx.x * kSmallW, y0 = blockIdx.y * rows, u = threadIdx.x;
    if (u < kSmallW / 8 * rows) map_cells<ELL>(a, a.vec, x0 + u % (kSmallW / 8) * 8, y0 + u / (kSmallW / 8));
    __syncthreads();
    const Box m = markable(a);
    mark_discs<ELL>(a, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
                    Box{max(m.x0, x0), min(m.x1, x0 + kSmallW - 1), max(m.y0, y0), min(m.y1, y0 + rows - 1)}, 0, 1);
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
    auto launch = [&](auto kernel, dim3 grid, int threads, auto... more) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, st, a, more...);
        return hipGetLastError() == hipSuccess;
    };
    // one launch where 16 waves a tile soon have every pair: up to 12 a wave
    if ((long long)nx * ny <= kSmallCells && pairs > 0 && pairs <= kSmallPairs) {
        a.waves = std::min<long long>(pairs, kSmallWaves);
        const int rows = std::max(8, std::min(64, 512 / ((nx + 7) / 8 * 8)));
        const dim3 grid((nx + kSmallW - 1) / kSmallW, (ny + rows - 1) / rows);
        const bool ok = ell ? launch(k_map_small<true>, grid, 64 * kSmallWaves, rows)
                            : launch(k_map_small<false>, grid, 64 * kSmallWaves, rows);
        return ok ? TWG_OK : set_err(ctx, TWG_EDEVICE, "map launch failed");
    }
    const dim3 grid((nx + 255) / 256, (ny + 7) / 8);
    const bool ok = vec ? (ell ? launch(k_map<true, true>, grid, 256) : launch(k_map<true, false>, grid, 256))
                        : (ell ? launch(k_map<false, true>, grid, 256) : launch(k_map<false, false>, grid, 256));
    if (!ok) return set_err(ctx, TWG_EDEVICE, "map launch failed");
    if (n_obs == 0) return TWG_OK;
    // few pairs, whose discs may be large: several waves share each, 4096 in
    // all; four where a wave has one pair or a few and a cell's ring test is FP64
    // (512 x 512, 10 discs of radius 100, elliptical: 230 -> 72 us; for small
    // discs the predictions made again outweigh it: 64 x 64 with 20, 16384 waves
    // 17.1 us, 4096 14.5)
    const unsigned slices = ell && a.waves == 4096 && !p.per_object
                                ? 4 : (unsigned)std::max(1LL, std::min(16LL, 4096 / a.waves));
    const dim3 blocks((unsigned)((a.waves + 3) / 4), slices);
    if (!(ell ? launch(k_discs<true>, blocks, 256) : launch(k_discs<false>, blocks, 256)))
        return set_err(ctx, TWG_EDEVICE, "rasterize launch failed");
    return TWG_OK;
}

}  // namespace twg
