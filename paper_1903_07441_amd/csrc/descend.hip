// Index matrix (Eq. 3) and steepest-descent path extraction (Algorithm 1,
// "Path Planning": index matrix, then the path from the robot's position).
//
//   k_tiles  32 x 32 tiles, a workgroup each, compute the index matrix from
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
//   k_path   the path of one cell: every wave follows the nodes (one dependent
//            read per tile crossed, not per cell) and writes the cells of the
//            tiles that fall to it.
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
#include "tile_map.h"
#include "twg_internal.h"

#include <algorithm>

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

// where a tile cell's word lies during the jumping
__device__ __forceinline__ int slot(int cell) { return (cell & 3) * (kTile * kTile / 4) + (cell >> 2); }
__device__ __forceinline__ int cell_of_slot(int s)
{
    return (s & (kTile * kTile / 4 - 1)) * 4 + s / (kTile * kTile / 4);
}
// row stride of the packed descents and of a path's codes
__host__ __device__ inline int local_pitch(int nx) { return (nx + 3) & ~3; }

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

// four neighbouring elements
__device__ __forceinline__ void load4(const float *p, float (&v)[4])
{
    const float4 q = *reinterpret_cast<const float4 *>(p);
    v[0] = q.x, v[1] = q.y, v[2] = q.z, v[3] = q.w;
}
__device__ __forceinline__ void load4(const double *p, double (&v)[4])
{
    const double2 q = reinterpret_cast<const double2 *>(p)[0], r = reinterpret_cast<const double2 *>(p)[1];
    v[0] = q.x, v[1] = q.y, v[2] = r.x, v[3] = r.y;
}
__device__ __forceinline__ uint8_t byte_of(uint32_t w, int k) { return (uint8_t)(w >> 8 * k); }

// A thread takes four neighbouring cells of a row, read as one word of classes
// and one or two 16-byte values where rows are aligned for that, else cell by
// cell.  Bound by memory, the jumping by LDS latency.  2048 x 2048 in FP64, with
// a cell a load, all its words in volatile LDS accesses (each waits for the one
// before), then now: index matrix 17.0 -> 14.6 us, codes and nodes 31.9 -> 19.4,
// packed descents and nodes 31.3 -> 22.4; 64 x 64, codes and nodes 8.6 -> 5.0.
template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) void k_tiles(const uint8_t *__restrict__ cls, const T *__restrict__ u,
                                                    uint8_t *__restrict__ idx, uint32_t *__restrict__ local,
                                                    unsigned long long *__restrict__ nodes, int nx, int ny, int pitch,
                                                    int idx_pitch, int sx, int sy)
{
    constexpr int kStride = kTile + 8;  // of a row in LDS: 4 columns (one in use) left of the tile
    __shared__ __align__(16) T tu[kTH * kStride];
    __shared__ __align__(16) uint8_t tc[kTH * kStride];
    // a cell's word lies at slot(cell), so that a thread's four are 256 apart
    __shared__ uint32_t ptr[MODE == kIndex ? 1 : kTile * kTile];
    __shared__ __align__(4) uint8_t code[MODE == kIndex ? 4 : kTile * kTile];
    static_assert(kCells == 4 && kTile == 32, "a thread's four cells, eight threads a row");
    const int tid = threadIdx.x, r = tid >> 3, g = tid & 7;
    const int own = (r + 1) * kStride + 4 + 4 * g;  // this thread's cells in LDS
    // the halo's sides: above, below, left, right
    const int side = tid >> 5, hi = tid & 31;
    const int hx = side < 2 ? hi : side == 2 ? -1 : kTile, hy = side == 0 ? -1 : side == 1 ? kTile : hi;
    const int halo = (hy + 1) * kStride + 4 + hx;
    const bool rows4 = !(pitch & 3), cls4 = rows4 && !((uintptr_t)cls & 3), u4 = rows4 && !((uintptr_t)u & 15);
    const int tiles_x = (nx + kTile - 1) / kTile, n_tiles = tiles_x * ((ny + kTile - 1) / kTile);
    // An XCD's workgroups share a run of the tiles: a tile's halo columns lie in
    // its neighbours' cache lines.  The index matrix alone goes over several
    // tiles a workgroup, whose loads overlap the last one's work; the jumping
    // is faster with all tiles in flight (2048 x 2048: 21.6 against 22.8 us).
    int t, t_end = n_tiles, step = n_tiles;
    if constexpr (MODE == kIndex) {
        const int X = min(8, (int)gridDim.x), xcd = blockIdx.x % X;
        step = ((int)gridDim.x - xcd + X - 1) / X;
        t = (int)((long long)n_tiles * xcd / X) + blockIdx.x / X;
        t_end = (int)((long long)n_tiles * (xcd + 1) / X);
    } else {
        t = xcd_remap(blockIdx.x, gridDim.x);
    }
    T v[4], hv;
    uint32_t c;
    uint8_t hc;
    // a tile's cells as they lie in memory (columns and rows outside the grid
    // read others inside)
    auto load = [&](int tile) __attribute__((always_inline)) {
        const int x0 = tile % tiles_x * kTile, y0 = tile / tiles_x * kTile, x = x0 + 4 * g;
        const size_t row = (size_t)min(y0 + r, ny - 1) * pitch;
        const bool whole = x + 4 <= nx;
        if (cls4 && whole) {
            c = *reinterpret_cast<const uint32_t *>(cls + row + x);
        } else {
            c = 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) c |= (uint32_t)cls[row + min(x + k, nx - 1)] << 8 * k;
        }
        if (u4 && whole) {
            load4(u + row + x, v);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = u[row + min(x + k, nx - 1)];
        }
        if (side < 4) {
            const size_t at = (size_t)min(max(y0 + hy, 0), ny - 1) * pitch + min(max(x0 + hx, 0), nx - 1);
            hv = u[at];
            hc = cls[at];
        }
    };
    if (t < t_end) load(t);
    for (; t < t_end; t += step) {
        const int tx = t % tiles_x, ty = t / tiles_x, x0 = tx * kTile, y0 = ty * kTile, x = x0 + 4 * g, y = y0 + r;
        const bool whole = x + 4 <= nx;
        // cells outside the grid read as walls
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (x + k >= nx || y >= ny) c = (c & ~(0xffu << 8 * k)) | (uint32_t)TWG_CELL_WALL << 8 * k;
#pragma unroll
        for (int k = 0; k < 4; ++k) tu[own + k] = v[k];
        *reinterpret_cast<uint32_t *>(tc + own) = c;
        if (side < 4) {
            const int gx = x0 + hx, gy = y0 + hy;
            tu[halo] = hv;
            tc[halo] = gx >= 0 && gy >= 0 && gx < nx && gy < ny ? hc : (uint8_t)TWG_CELL_WALL;
        }
        __syncthreads();
        const uint32_t cc = c;
        const T vv[4] = {v[0], v[1], v[2], v[3]};
        // the next tile's cells arrive while this one is worked on
        if (t + step < t_end) load(t + step);
        const uint32_t cn = *reinterpret_cast<const uint32_t *>(tc + own - kStride);
        const uint32_t cs = *reinterpret_cast<const uint32_t *>(tc + own + kStride);
        const uint8_t cw = tc[own - 1], ce = tc[own + 4];
        const T w = tu[own - 1], e = tu[own + 4];
        uint32_t codes = 0u, mine[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const T nb[4] = {k < 3 ? vv[k < 3 ? k + 1 : 3] : e, k > 0 ? vv[k > 0 ? k - 1 : 0] : w,
                             tu[own + kStride + k], tu[own - kStride + k]};
            const uint8_t nc[4] = {k < 3 ? byte_of(cc, k + 1) : ce, k > 0 ? byte_of(cc, k - 1) : cw, byte_of(cs, k),
                                   byte_of(cn, k)};
            uint32_t best = 4;
            T bv = T(0);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const bool ok = walkable(nc[d]) && (best == 4 || nb[d] > bv);
                best = ok ? d : best;
                bv = ok ? nb[d] : bv;
            }
            if (best != 4 && !(bv > vv[k])) best = 4;
            if constexpr (MODE != kIndex) {
                const uint8_t cl = byte_of(cc, k);
                if (cl == TWG_CELL_GOAL) best = kGoalCode;
                else if (MODE == kAll && !walkable(cl)) best = 4;
                const int lx = 4 * g + k, ex = lx + dir_x((int)best), ey = r + dir_y((int)best);
                const bool stays = best < 4 && ex >= 0 && ey >= 0 && ex < kTile && ey < kTile;
                mine[k] = stays ? pack_local(slot(ey * kTile + ex), 1) : pack_local(slot(4 * tid + k), 0);
                ptr[slot(4 * tid + k)] = mine[k];
            }
            codes |= best << 8 * k;
        }
        if constexpr (MODE != kAll) {
            if (y < ny) {
                uint8_t *o = idx + (size_t)y * idx_pitch + x;
                if (!(idx_pitch & 3) && !((uintptr_t)idx & 3) && whole) {
                    *reinterpret_cast<uint32_t *>(o) = codes;
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (x + k < nx) o[k] = byte_of(codes, k);
                }
            }
        }
        if constexpr (MODE != kIndex) *reinterpret_cast<uint32_t *>(code + 4 * tid) = codes;
        // (also: what the next tile overwrites has been read)
        __syncthreads();
        if constexpr (MODE != kIndex) {
            // pointer jumping in place, every wave at its own pace: a word is
            // always a valid part of its cell's descent, whenever the words read
            // through it were written; a cell is done when the word it points to
            // makes no move (relaxed atomics: a volatile word's access would wait
            // for the one before)
            // (a path: five rounds, which cover 32 moves at least; its perimeter
            // cells go on from there below)
            int rounds = 0;
            for (bool todo = true; MODE == kPath ? rounds < 5 : todo; ++rounds) {
                uint32_t q[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    q[k] = __hip_atomic_load(ptr + local_cell(mine[k]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                todo = false;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    // a word that makes no move adds nothing
                    todo = todo || local_moves(q[k]) != 0;
                    mine[k] = pack_local(local_cell(q[k]), local_moves(mine[k]) + local_moves(q[k]));
                    __hip_atomic_store(ptr + slot(4 * tid + k), mine[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            __syncthreads();
            if constexpr (MODE == kAll) {
                uint32_t out[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int end = cell_of_slot(local_cell(mine[k]));
                    out[k] = pack_local(end, local_moves(mine[k])) | (uint32_t)code[end] << 24;
                }
                if (x < nx && y < ny)
                    *reinterpret_cast<uint4 *>(local + (size_t)y * local_pitch(nx) + x) =
                        make_uint4(out[0], out[1], out[2], out[3]);
            }
            // a thread a perimeter cell, and one for the start
            const int2 p = tid < kNodes ? cell_of_node(tid) : make_int2(sx - x0, sy - y0);
            const bool has = tid < kNodes ? node_of(p.x, p.y) == tid  // (not a corner's second number)
                                          : MODE == kPath && tid == kNodes && p.x >= 0 && p.y >= 0 && p.x < kTile &&
                                                p.y < kTile;
            if (has && x0 + p.x < nx && y0 + p.y < ny) {
                uint32_t q = ptr[slot(p.y * kTile + p.x)];
                if constexpr (MODE == kPath)
                    for (uint32_t w = ptr[local_cell(q)]; local_moves(w) != 0; w = ptr[local_cell(q)])
                        q = pack_local(local_cell(w), local_moves(q) + local_moves(w));
                const int end = cell_of_slot(local_cell(q)), m = local_moves(q), d = code[end];
                nodes[tid < kNodes ? (size_t)t * kNodes + tid : (size_t)n_tiles * kNodes] =
                    pack(d < 4 ? Node{next_node(tx, ty, end % kTile, end / kTile, d, tiles_x), m + 1}
                               : Node{d == (int)kGoalCode ? kAtGoal : kStuck, m});
            }
        }
    }
}

// The start cell's descent, tile by tile: every wave (a workgroup each) follows
// the nodes from the start (node `start`), notes the parts that are its own
// (parts blockIdx.x, + gridDim.x, ...: the node entered and the path index of
// its cell), and writes them; info = [length, status] of the path in cap cells.
// Following the nodes in every wave costs the time of following them once and
// spares the launch that would list the parts (a call on 200 x 200 cells, start
// in a corner: 17.9 us with it, 14.3 without; in the next tile, 14.0 and 11.1).
// A part: the tile's moves in LDS (the byte offset of the next cell in the
// tile, 0 where the descent ends or leaves it), followed from the entered cell,
// one LDS read a step; lane k keeps the k-th cell of the current group of 64,
// stored in one coalesced write per group.
__global__ __launch_bounds__(64) void k_path(const uint8_t *__restrict__ cls, const uint8_t *__restrict__ code,
                                             const unsigned long long *__restrict__ nodes, int nx, int ny, int pitch,
                                             int tiles_x, int start, int sx, int sy, int cap,
                                             int32_t *__restrict__ path, int32_t *__restrict__ info)
{
    __shared__ __align__(8) int16_t move[kTile * kTile];
    const int lane = threadIdx.x, code_pitch = local_pitch(nx);
    if (!walkable(cls[(size_t)sy * pitch + sx])) {
        if (blockIdx.x == 0 && lane == 0) {
            info[0] = 0;
            info[1] = TWG_START_BLOCKED;
        }
        return;
    }
    // parts past the buffer's end are not written: the walk stops there
    int at = start, n = 0, turn = blockIdx.x;  // turn: parts until this wave's next one
    while (at >= 0 && n < cap) {
        // up to 64 parts at a time: lane k keeps the k-th
        int own = 0, part_at = 0, part_n = 0;
        while (at >= 0 && n < cap && own < 64) {
            const Node v = unpack(nodes[at]);
            if (turn == 0) {
                part_at = lane == own ? at : part_at;
                part_n = lane == own ? n : part_n;
                ++own;
                turn = gridDim.x;
            }
            --turn;
            n += v.moves;
            at = v.next;
        }
        for (int k = 0; k < own; ++k) {
            const int2 s = make_int2(__builtin_amdgcn_readlane(part_at, k), __builtin_amdgcn_readlane(part_n, k));
            int x = sx, y = sy;
            if (s.x != start) {
                const int t = s.x / kNodes;
                const int2 c = cell_of_node(s.x % kNodes);
                x = (t % tiles_x) * kTile + c.x;
                y = (t / tiles_x) * kTile + c.y;
            }
            const int x0 = x / kTile * kTile, y0 = y / kTile * kTile;
            // (words past a row's or the grid's end read others inside: no
            // descent comes to their cells)
            constexpr int PER = kTile * kTile / 4 / 64;
            uint32_t d[PER];
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int q = i * 64 + lane, cy = min(y0 + q / 8, ny - 1), cx = min(x0 + q % 8 * 4, code_pitch - 4);
                d[i] = *reinterpret_cast<const uint32_t *>(code + (size_t)cy * code_pitch + cx);
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int q = i * 64 + lane, ly = q / 8;
                uint32_t m[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int lx = q % 8 * 4 + k, c = byte_of(d[i], k);
                    const bool out = (c == 0 && lx == kTile - 1) || (c == 1 && lx == 0) || (c == 2 && ly == kTile - 1) ||
                                     (c == 3 && ly == 0);
                    m[k] = (uint16_t)(out ? 0 : c == 0 ? 2 : c == 1 ? -2 : c == 2 ? 2 * kTile : c == 3 ? -2 * kTile : 0);
                }
                *reinterpret_cast<uint2 *>(move + 4 * q) = make_uint2(m[0] | m[1] << 16, m[2] | m[3] << 16);
            }
            __syncthreads();
            int a = __builtin_amdgcn_readfirstlane(2 * ((y - y0) * kTile + x - x0)), p = s.y;
            const char *moves = reinterpret_cast<const char *>(move);
            int m = *reinterpret_cast<const int16_t *>(moves + a);
            for (bool on = true; on && p < cap;) {
                const int lim = min(64, cap - p);
                int rec = a, q = 1;
                while (m != 0 && q < lim) {
                    a += m;
                    rec = lane == q ? a : rec;
                    ++q;
                    m = *reinterpret_cast<const int16_t *>(moves + a);
                }
                if (lane < q) {
                    path[2 * (size_t)(p + lane)] = x0 + (rec >> 1) % kTile;
                    path[2 * (size_t)(p + lane) + 1] = y0 + (rec >> 1) / kTile;
                }
                p += q;
                // the next group opens with the cell after this one's last
                on = m != 0;
                a += m;
                if (on) m = *reinterpret_cast<const int16_t *>(moves + a);
            }
        }
    }
    // the descent's last cell has path index n when it has ended (a part
    // that goes on has its next cell there)
    if (blockIdx.x == 0 && lane == 0) {
        const bool ended = at < 0 && n < cap;
        info[0] = ended ? n + 1 : cap;
        info[1] = !ended ? TWG_PATH_TRUNCATED : at == kAtGoal ? TWG_OK : TWG_NO_PATH;
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
    const uint32_t v = local[(size_t)y * local_pitch(nx) + x];
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

constexpr int kTileGroups = 8 * 256;  // workgroups of k_tiles at most

template <int MODE>
void tiles(const uint8_t *cls, const float *psi, const double *psi64, uint8_t *idx, uint32_t *local,
           unsigned long long *nodes, int nx, int ny, int pitch, int idx_pitch, int sx, int sy, hipStream_t st)
{
    const dim3 g = tile_grid(nx, ny), blocks(MODE == kIndex ? std::min((int)(g.x * g.y), kTileGroups) : (int)(g.x * g.y));
    if (psi64)
        hipLaunchKernelGGL((k_tiles<double, MODE>), blocks, dim3(kThreads), 0, st, cls, psi64, idx, local, nodes, nx, ny,
                           pitch, idx_pitch, sx, sy);
    else
        hipLaunchKernelGGL((k_tiles<float, MODE>), blocks, dim3(kThreads), 0, st, cls, psi, idx, local, nodes, nx, ny,
                           pitch, idx_pitch, sx, sy);
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
    tiles<kIndex>(cls, psi, psi64, idx, nullptr, nullptr, nx, ny, pitch, pitch, 0, 0, st);
    return last_status();
}

size_t descend_code_bytes(int nx, int ny) { return (size_t)local_pitch(nx) * ny; }
// scratch: the nodes
size_t descend_bytes(int nx, int ny) { return node_words(nx, ny) * 8; }

int launch_descend(const uint8_t *cls, const float *psi, const double *psi64, uint8_t *code, void *scratch, int nx,
                   int ny, int pitch, int sx, int sy, int cap, int32_t *path, int32_t *info, hipStream_t st)
{
    unsigned long long *nodes = static_cast<unsigned long long *>(scratch);
    tiles<kPath>(cls, psi, psi64, code, nullptr, nodes, nx, ny, pitch, local_pitch(nx), sx, sy, st);
    hipLaunchKernelGGL(k_path, dim3(256), dim3(64), 0, st, cls, code, nodes, nx, ny, pitch, (int)tile_grid(nx, ny).x,
                       (int)(node_words(nx, ny) - 1), sx, sy, cap, path, info);
    return last_status();
}

// scratch: 4 bytes a cell, then the nodes
size_t descent_all_bytes(int nx, int ny) { return (size_t)local_pitch(nx) * ny * 4 + node_words(nx, ny) * 8; }

int launch_descent_all(const uint8_t *cls, const float *psi, const double *psi64, void *scratch, int nx, int ny,
                       int pitch, int32_t *steps, int pitch_out, hipStream_t st)
{
    uint32_t *local = static_cast<uint32_t *>(scratch);
    unsigned long long *nodes = reinterpret_cast<unsigned long long *>(local + (size_t)local_pitch(nx) * ny);
    const dim3 g = tile_grid(nx, ny);
    tiles<kAll>(cls, psi, psi64, nullptr, local, nodes, nx, ny, pitch, 0, 0, 0, st);
    hipLaunchKernelGGL(k_chase, dim3(g.x * g.y), dim3(kNodes), 0, st, nodes, nx, ny, (int)g.x);
    hipLaunchKernelGGL(k_lengths, dim3((nx + 63) / 64, (ny + 3) / 4), dim3(256), 0, st, local, nodes, nx, ny, (int)g.x,
                       steps, pitch_out);
    return last_status();
}

}  // namespace twg
