// Index matrix (Eq. 3) and steepest-descent path extraction (Algorithm 1,
// "Path Planning": index matrix, then the path from the robot's position).
//
//   k_tiles  one workgroup per 32 x 32 tile computes the index matrix from
//            LDS: direction (E 0, W 1, S 2, N 3) of the walkable neighbour
//            with the highest psi (lowest phi), first one on ties; 4 when none
//            is strictly higher than the cell itself.  For descents it then
//            follows the directions inside the tile by pointer jumping in
//            LDS, so that every cell knows the cell where its descent ends or
//            leaves the tile and the moves to it.  A descent enters a tile
//            only through the tile's perimeter, so the perimeter cells'
//            exits (a node each: the perimeter cell of the next tile, and the
//            moves to it) are the whole grid's descents on an eighth of its
//            cells.
//   k_hops, k_emit
//            the path of one cell: one lane follows the nodes (one dependent
//            read per tile crossed, not per cell) and lists the tiles with
//            the path index at which each is entered; then the tiles' parts
//            are walked and written by a workgroup each.
//   k_chase, k_lengths
//            the descent length of every cell: every node follows the nodes
//            to its end, reading what the others have already covered (in
//            place: a node is one 64-bit word that is always a valid part of
//            its descent, so any mixture of old and new ones is); then each
//            cell adds its exit's node to its own moves.
//
// Descent strictly raises psi, so no chain has a cycle and every loop ends.
//
//   k_rubber one workgroup relaxes a path as a rubber band (Eqs. 4-6): per
//            iteration the interior points of odd index, then those of even
//            index, each move to the best of nine candidate cells given the
//            positions of their two neighbours (see hpf_rubber_band).
#include "twg_internal.h"

namespace twg {

namespace {

__device__ __forceinline__ bool walkable(uint8_t c)
{
    return c == TWG_CELL_FREE || c == TWG_CELL_GOAL;
}

constexpr int kTile = 32;             // tile side
constexpr int kTH = kTile + 2;        // with a halo of one cell
constexpr int kThreads = 256;
constexpr int kCells = kTile * kTile / kThreads;  // cells per thread
constexpr uint32_t kGoalCode = 5;     // on GOAL cells, else the index code
constexpr int kNodes = 4 * kTile;     // node numbers of a tile

// Node number of a tile's perimeter cell: the top and the bottom row, then
// the left and the right column.  Cells of a ragged tile keep their place in
// the full one.
__device__ __forceinline__ int node_of(int lx, int ly)
{
    return ly == 0 ? lx : ly == kTile - 1 ? kTile + lx : lx == 0 ? 2 * kTile + ly : 3 * kTile + ly;
}
__device__ __forceinline__ int2 cell_of_node(int n)
{
    const int side = n / kTile, i = n % kTile;
    return side == 0 ? make_int2(i, 0) : side == 1 ? make_int2(i, kTile - 1) : side == 2 ? make_int2(0, i)
                                                                                        : make_int2(kTile - 1, i);
}
__device__ __forceinline__ bool on_perimeter(int lx, int ly)
{
    return lx == 0 || ly == 0 || lx == kTile - 1 || ly == kTile - 1;
}

// A node: where a descent goes on (a node, or how it ends) and the moves to
// there.
constexpr int kAtGoal = -1, kStuck = -2;
struct Node {
    int next, moves;
};
__device__ __forceinline__ unsigned long long pack(Node n)
{
    return (unsigned long long)(uint32_t)n.next << 32 | (uint32_t)n.moves;
}
__device__ __forceinline__ Node unpack(unsigned long long v) { return {(int)(v >> 32), (int)(uint32_t)v}; }

// A cell's descent inside its tile, packed: the tile cell where it ends or
// leaves, the moves to it, and (k_tiles' output) that cell's code.
__device__ __forceinline__ uint32_t pack_local(int cell, int moves) { return (uint32_t)cell | (uint32_t)moves << 12; }
__device__ __forceinline__ int local_cell(uint32_t v) { return (int)(v & 4095u); }
__device__ __forceinline__ int local_moves(uint32_t v) { return (int)(v >> 12 & 4095u); }

__device__ __forceinline__ int dir_x(int d) { return d == 0 ? 1 : d == 1 ? -1 : 0; }
__device__ __forceinline__ int dir_y(int d) { return d == 2 ? 1 : d == 3 ? -1 : 0; }

// the node through which a descent that leaves tile (tx, ty) at tile cell
// (lx, ly) in direction d goes on
__device__ __forceinline__ int next_node(int tx, int ty, int lx, int ly, int d, int tiles_x)
{
    const int gx = tx * kTile + lx + dir_x(d), gy = ty * kTile + ly + dir_y(d);
    return ((gy / kTile) * tiles_x + gx / kTile) * kNodes + node_of(gx % kTile, gy % kTile);
}

// MODE kIndex: idx receives the index matrix; kPath: the codes, and the nodes
// (with the start cell (sx, sy)'s in the word after the last tile's); kAll:
// local receives every cell's packed descent inside its tile (with its last
// cell's code in bits 24 to 26), and the nodes.
constexpr int kIndex = 0, kPath = 1, kAll = 2;

template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) void k_tiles(const uint8_t *__restrict__ cls, const T *__restrict__ u,
                                                    uint8_t *__restrict__ idx, uint32_t *__restrict__ local,
                                                    unsigned long long *__restrict__ nodes, int nx, int ny, int pitch,
                                                    int sx, int sy)
{
    __shared__ T tu[kTH * kTH];
    __shared__ uint8_t tc[kTH * kTH];
    __shared__ uint32_t ptr[MODE == kIndex ? 1 : kTile * kTile];
    __shared__ uint8_t code[MODE == kIndex ? 1 : kTile * kTile];
    const int tid = threadIdx.x, tx = blockIdx.x, ty = blockIdx.y;
    const int x0 = tx * kTile, y0 = ty * kTile;
    // cells outside the grid read as walls; every load of a thread is issued
    // before its first LDS store
    {
        constexpr int PER = (kTH * kTH + kThreads - 1) / kThreads;
        T v[PER];
        uint8_t c[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int q = k * kThreads + tid, y = y0 + q / kTH - 1, x = x0 + q % kTH - 1;
            const size_t i = (size_t)min(max(y, 0), ny - 1) * pitch + min(max(x, 0), nx - 1);
            const uint8_t cl = cls[i];
            v[k] = u[i];
            c[k] = x >= 0 && y >= 0 && x < nx && y < ny ? cl : (uint8_t)TWG_CELL_WALL;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int q = k * kThreads + tid;
            if (q < kTH * kTH) {
                tu[q] = v[k];
                tc[q] = c[k];
            }
        }
    }
    __syncthreads();
    uint32_t mine[kCells];
#pragma unroll
    for (int k = 0; k < kCells; ++k) {
        const int c = k * kThreads + tid, lx = c % kTile, ly = c / kTile;
        const int q = (ly + 1) * kTH + lx + 1;
        constexpr int off[4] = {1, -1, kTH, -kTH};
        uint32_t best = 4;
        T bv = T(0);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const T v = tu[q + off[d]];
            const bool ok = walkable(tc[q + off[d]]) && (best == 4 || v > bv);
            best = ok ? d : best;
            bv = ok ? v : bv;
        }
        if (best != 4 && !(bv > tu[q])) best = 4;
        const bool in = x0 + lx < nx && y0 + ly < ny;
        const uint8_t cl = tc[q];
        if constexpr (MODE != kIndex) {
            if (cl == TWG_CELL_GOAL) best = kGoalCode;
            else if (MODE == kAll && !walkable(cl)) best = 4;
        }
        if constexpr (MODE != kAll) {
            if (in) idx[(size_t)(y0 + ly) * pitch + x0 + lx] = (uint8_t)best;
        }
        if constexpr (MODE != kIndex) {
            const int ex = lx + dir_x((int)best), ey = ly + dir_y((int)best);
            const bool stays = best < 4 && ex >= 0 && ey >= 0 && ex < kTile && ey < kTile;
            code[c] = (uint8_t)best;
            mine[k] = stays ? pack_local(ey * kTile + ex, 1) : pack_local(c, 0);
            ptr[c] = mine[k];
        }
    }
    if constexpr (MODE == kIndex) return;
    // pointer jumping in place, every wave at its own pace: a word is always
    // a valid part of its cell's descent, whenever the words read through it
    // were written; a cell is done when the word it points to makes no move
    __syncthreads();
    {
        volatile uint32_t *words = ptr;
        uint32_t todo = (1u << kCells) - 1u;
        while (todo) {
            uint32_t w[kCells];
#pragma unroll
            for (int k = 0; k < kCells; ++k) w[k] = words[local_cell(mine[k])];
#pragma unroll
            for (int k = 0; k < kCells; ++k) {
                if (local_moves(w[k]) != 0) {
                    mine[k] = pack_local(local_cell(w[k]), local_moves(mine[k]) + local_moves(w[k]));
                    words[k * kThreads + tid] = mine[k];
                } else {
                    todo &= ~(1u << k);
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kCells; ++k) {
        const int c = k * kThreads + tid, lx = c % kTile, ly = c / kTile;
        const int x = x0 + lx, y = y0 + ly;
        if (x >= nx || y >= ny) continue;
        const int r = local_cell(mine[k]), m = local_moves(mine[k]), d = code[r];
        if constexpr (MODE == kAll) local[(size_t)y * nx + x] = mine[k] | (uint32_t)d << 24;
        const bool start = MODE == kPath && x == sx && y == sy;
        if (!start && !on_perimeter(lx, ly)) continue;
        const Node n = d < 4 ? Node{next_node(tx, ty, r % kTile, r / kTile, d, gridDim.x), m + 1}
                             : Node{d == (int)kGoalCode ? kAtGoal : kStuck, m};
        if (on_perimeter(lx, ly)) nodes[((size_t)ty * gridDim.x + tx) * kNodes + node_of(lx, ly)] = pack(n);
        if (start) nodes[(size_t)gridDim.x * gridDim.y * kNodes] = pack(n);
    }
}

// The parts of the start cell's descent, tile by tile: segs[k] = (node
// entered, path index of its cell) with the start as node `start`, then
// count[0] = their number; info = [length, status] of the path in cap cells.
__global__ void k_hops(const uint8_t *__restrict__ cls, const unsigned long long *__restrict__ nodes, int start, int sx,
                       int sy, int pitch, int cap, int2 *__restrict__ segs, int *__restrict__ count,
                       int32_t *__restrict__ info)
{
    if (threadIdx.x != 0) return;
    if (!walkable(cls[(size_t)sy * pitch + sx])) {
        count[0] = 0;
        info[0] = 0;
        info[1] = TWG_START_BLOCKED;
        return;
    }
    int k = 0, at = start, n = 0;
    for (;;) {
        segs[k++] = make_int2(at, n);
        const Node v = unpack(nodes[at]);
        n += v.moves;
        at = v.next;
        // parts past the buffer's end are not written: stop there
        if (at < 0 || n >= cap) break;
    }
    count[0] = k;
    // the descent's last cell has path index n when it has ended (a part
    // that goes on has its next cell there)
    const bool ended = at < 0 && n < cap;
    info[0] = ended ? n + 1 : cap;
    info[1] = !ended ? TWG_PATH_TRUNCATED : at == kAtGoal ? TWG_OK : TWG_NO_PATH;
}

// One wave per part of the path (parts blockIdx.x, + gridDim.x, ...): the
// tile's moves in LDS (the byte offset of the next cell in the tile, 0 where
// the descent ends or leaves it), followed from the entered cell, one LDS
// read a step; lane k keeps the k-th cell of the current group of 64, stored
// in one coalesced write per group.
__global__ __launch_bounds__(64) void k_emit(const uint8_t *__restrict__ code, int nx, int ny, int pitch, int tiles_x,
                                             int start, int sx, int sy, int cap, const int2 *__restrict__ segs,
                                             const int *__restrict__ count, int32_t *__restrict__ path)
{
    __shared__ int16_t move[kTile * kTile];
    const int lane = threadIdx.x, n = *count;
    for (int k = blockIdx.x; k < n; k += gridDim.x) {
        const int2 s = segs[k];
        int x = sx, y = sy;
        if (s.x != start) {
            const int t = s.x / kNodes;
            const int2 c = cell_of_node(s.x % kNodes);
            x = (t % tiles_x) * kTile + c.x;
            y = (t / tiles_x) * kTile + c.y;
        }
        const int x0 = x / kTile * kTile, y0 = y / kTile * kTile;
        constexpr int PER = kTile * kTile / 64;
        uint8_t d[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = i * 64 + lane;
            d[i] = code[(size_t)min(y0 + q / kTile, ny - 1) * pitch + min(x0 + q % kTile, nx - 1)];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = i * 64 + lane, lx = q % kTile, ly = q / kTile;
            int m = d[i] == 0 ? 2 : d[i] == 1 ? -2 : d[i] == 2 ? 2 * kTile : d[i] == 3 ? -2 * kTile : 0;
            if ((d[i] == 0 && lx == kTile - 1) || (d[i] == 1 && lx == 0)) m = 0;
            if ((d[i] == 2 && ly == kTile - 1) || (d[i] == 3 && ly == 0)) m = 0;
            move[q] = (int16_t)m;
        }
        __syncthreads();
        int a = __builtin_amdgcn_readfirstlane(2 * ((y - y0) * kTile + x - x0)), at = s.y;
        const char *moves = reinterpret_cast<const char *>(move);
        int m = *reinterpret_cast<const int16_t *>(moves + a);
        for (bool on = true; on && at < cap;) {
            const int lim = min(64, cap - at);
            int rec = a, q = 1;
            while (m != 0 && q < lim) {
                a += m;
                rec = lane == q ? a : rec;
                ++q;
                m = *reinterpret_cast<const int16_t *>(moves + a);
            }
            if (lane < q) {
                path[2 * (size_t)(at + lane)] = x0 + (rec >> 1) % kTile;
                path[2 * (size_t)(at + lane) + 1] = y0 + (rec >> 1) / kTile;
            }
            at += q;
            // the next group opens with the cell after this one's last
            on = m != 0;
            a += m;
            if (on) m = *reinterpret_cast<const int16_t *>(moves + a);
        }
    }
}

// Every node follows the nodes to its descent's end, in place.
__global__ __launch_bounds__(256) void k_chase(unsigned long long *__restrict__ nodes, int nx, int ny, int tiles_x)
{
    const int t = blockIdx.x, i = threadIdx.x;
    const int2 c = cell_of_node(i);
    if (node_of(c.x, c.y) != i) return;  // a corner's second number
    if ((t % tiles_x) * kTile + c.x >= nx || (t / tiles_x) * kTile + c.y >= ny) return;
    unsigned long long *own = nodes + (size_t)t * kNodes + i;
    Node v = unpack(__hip_atomic_load(own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    while (v.next >= 0) {
        const Node w = unpack(__hip_atomic_load(nodes + v.next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        v = {w.next, v.moves + w.moves};
        __hip_atomic_store(own, pack(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// steps[c] = descent length to a GOAL cell, or -1 (not walkable, or the
// descent ends elsewhere)
__global__ __launch_bounds__(256) void k_lengths(const uint32_t *__restrict__ local,
                                                 const unsigned long long *__restrict__ nodes, int nx, int ny,
                                                 int tiles_x, int32_t *__restrict__ steps, int pitch_out)
{
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (x >= nx || y >= ny) return;
    const uint32_t v = local[(size_t)y * nx + x];
    const int d = (int)(v >> 24 & 7u), r = local_cell(v), m = local_moves(v);
    int out = d == (int)kGoalCode ? m : -1;
    if (d < 4) {
        const Node n = unpack(nodes[next_node(x / kTile, y / kTile, r % kTile, r / kTile, d, tiles_x)]);
        out = n.next == kAtGoal ? m + 1 + n.moves : -1;
    }
    steps[(size_t)y * pitch_out + x] = out;
}

// Candidate offsets: stay, E, W, S, N, then the diagonals.
__constant__ int kRbDx[9] = {0, 1, -1, 0, 0, 1, -1, 1, -1};
__constant__ int kRbDy[9] = {0, 0, 0, 1, -1, 1, 1, -1, -1};

template <typename T>
__global__ __launch_bounds__(1024) void k_rubber(const uint8_t *__restrict__ cls, const T *__restrict__ u,
                                                 int32_t *__restrict__ path, const int32_t *__restrict__ len,
                                                 int cap, int nx, int ny, int pitch, double k, int iters)
{
    const int n = min(*len, cap);
    const double inv_sqrt2 = 0.70710678118654752440;
    for (int it = 0; it < iters; ++it) {
        for (int color = 1; color >= 0; --color) {
            // points of this colour read only points of the other colour
            for (int i = 1 + (color ^ 1) + 2 * (int)threadIdx.x; i + 1 < n; i += 2 * (int)blockDim.x) {
                const int px = path[2 * i], py = path[2 * i + 1];
                const int ax = path[2 * i - 2], ay = path[2 * i - 1];
                const int bx = path[2 * i + 2], by = path[2 * i + 3];
                const double p0 = (double)u[(size_t)py * pitch + px];
                if (!(p0 > 0.0)) continue;
                const double g0 = 1.0 / p0;
                int best = -1;
                double bestv = 0.0;
                for (int d = 0; d < 9; ++d) {
                    const int cx = px + kRbDx[d], cy = py + kRbDy[d];
                    if (cx < 0 || cy < 0 || cx >= nx || cy >= ny) continue;
                    const size_t c = (size_t)cy * pitch + cx;
                    const double pc = (double)u[c];
                    if (!walkable(cls[c]) || !(pc > 0.0)) continue;
                    if (abs(cx - ax) > 1 || abs(cy - ay) > 1 || abs(cx - bx) > 1 || abs(cy - by) > 1) continue;
                    const double tx = k * (double)((ax - cx) + (bx - cx));
                    const double ty = k * (double)((ay - cy) + (by - cy));
                    double fx = 0.0, fy = 0.0;
                    if (d > 0) {
                        const double m = -(1.0 / pc - g0);
                        const double w = (kRbDx[d] != 0 && kRbDy[d] != 0) ? inv_sqrt2 : 1.0;
                        fx = m * ((double)kRbDx[d] * w);
                        fy = m * ((double)kRbDy[d] * w);
                    }
                    const double rx = fx + tx, ry = fy + ty;
                    const double v = rx * rx + ry * ry;
                    if (best < 0 || v < bestv) {
                        best = d;
                        bestv = v;
                    }
                }
                if (best > 0) {
                    path[2 * i] = px + kRbDx[best];
                    path[2 * i + 1] = py + kRbDy[best];
                }
            }
            __syncthreads();
        }
    }
}

}  // namespace

int launch_rubber(const uint8_t *cls, const float *psi, const double *psi64, int32_t *path, const int32_t *len,
                  int cap, int nx, int ny, int pitch, double k, int iters, hipStream_t st)
{
    if (psi64)
        hipLaunchKernelGGL(k_rubber<double>, dim3(1), dim3(1024), 0, st, cls, psi64, path, len, cap, nx, ny, pitch, k,
                           iters);
    else
        hipLaunchKernelGGL(k_rubber<float>, dim3(1), dim3(1024), 0, st, cls, psi, path, len, cap, nx, ny, pitch, k,
                           iters);
    return hipGetLastError() == hipSuccess ? TWG_OK : TWG_EDEVICE;
}

namespace {

dim3 tile_grid(int nx, int ny) { return dim3((nx + kTile - 1) / kTile, (ny + kTile - 1) / kTile); }

template <int MODE>
void tiles(const uint8_t *cls, const float *psi, const double *psi64, uint8_t *idx, uint32_t *local,
           unsigned long long *nodes, int nx, int ny, int pitch, int sx, int sy, hipStream_t st)
{
    if (psi64)
        hipLaunchKernelGGL((k_tiles<double, MODE>), tile_grid(nx, ny), dim3(kThreads), 0, st, cls, psi64, idx, local,
                           nodes, nx, ny, pitch, sx, sy);
    else
        hipLaunchKernelGGL((k_tiles<float, MODE>), tile_grid(nx, ny), dim3(kThreads), 0, st, cls, psi, idx, local,
                           nodes, nx, ny, pitch, sx, sy);
}

int last_status() { return hipGetLastError() == hipSuccess ? TWG_OK : TWG_EDEVICE; }

size_t node_words(int nx, int ny)
{
    const dim3 g = tile_grid(nx, ny);
    return (size_t)g.x * g.y * kNodes + 1;
}

}  // namespace

int launch_index(const uint8_t *cls, const float *psi, const double *psi64, uint8_t *idx, int nx, int ny, int pitch,
                 hipStream_t st)
{
    tiles<kIndex>(cls, psi, psi64, idx, nullptr, nullptr, nx, ny, pitch, 0, 0, st);
    return last_status();
}

// scratch: the nodes, the parts (one per node at most) and their number
size_t descend_bytes(int nx, int ny) { return node_words(nx, ny) * 16 + 16; }

int launch_descend(const uint8_t *cls, const float *psi, const double *psi64, uint8_t *code, void *scratch, int nx,
                   int ny, int pitch, int sx, int sy, int cap, int32_t *path, int32_t *info, hipStream_t st)
{
    const size_t n = node_words(nx, ny);
    unsigned long long *nodes = static_cast<unsigned long long *>(scratch);
    int2 *segs = reinterpret_cast<int2 *>(nodes + n);
    int *count = reinterpret_cast<int *>(segs + n);
    const int start = (int)(n - 1), tiles_x = (int)tile_grid(nx, ny).x;
    tiles<kPath>(cls, psi, psi64, code, nullptr, nodes, nx, ny, pitch, sx, sy, st);
    hipLaunchKernelGGL(k_hops, dim3(1), dim3(64), 0, st, cls, nodes, start, sx, sy, pitch, cap, segs, count, info);
    hipLaunchKernelGGL(k_emit, dim3(256), dim3(64), 0, st, code, nx, ny, pitch, tiles_x, start, sx, sy, cap, segs, count,
                       path);
    return last_status();
}

// scratch: the nodes, then 4 bytes a cell
size_t descent_all_bytes(int nx, int ny) { return node_words(nx, ny) * 8 + (size_t)nx * ny * 4; }

int launch_descent_all(const uint8_t *cls, const float *psi, const double *psi64, void *scratch, int nx, int ny,
                       int pitch, int32_t *steps, int pitch_out, hipStream_t st)
{
    unsigned long long *nodes = static_cast<unsigned long long *>(scratch);
    uint32_t *local = reinterpret_cast<uint32_t *>(nodes + node_words(nx, ny));
    const dim3 g = tile_grid(nx, ny);
    tiles<kAll>(cls, psi, psi64, nullptr, local, nodes, nx, ny, pitch, 0, 0, st);
    hipLaunchKernelGGL(k_chase, dim3(g.x * g.y), dim3(kNodes), 0, st, nodes, nx, ny, (int)g.x);
    hipLaunchKernelGGL(k_lengths, dim3((nx + 63) / 64, (ny + 3) / 4), dim3(256), 0, st, local, nodes, nx, ny, (int)g.x,
                       steps, pitch_out);
    return last_status();
}

}  // namespace twg
