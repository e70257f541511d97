// Streamed, temporally blocked red-black SOR tile for gfx950, shared by the
// kernels of sor_stream.hip (fixed sweep counts, FP64 sweeps, batches) and
// solve.hip (the device-driven relaxation).  See sor_stream.hip for the
// scheme.
#pragma once

#include <type_traits>
#include <utility>

#include "tile_map.h"
#include "twg_internal.h"
#include "update.h"

namespace twg {
namespace sdev {

constexpr int kWave = 64;

// ---- wave-wide DPP shifts (gfx9 wave_shr:1 / wave_shl:1) ----------------
// shr: lane i receives lane i-1 (lane 0 receives 0); shl: lane i receives
// lane i+1 (lane 63 receives 0).
__device__ __forceinline__ float shr1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float shl1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ double shr1(double v)
{
    int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double shl1(double v)
{
    int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// ---- buffer addressing ---------------------------------------------------
// A tile reads its rows through buffer resources based at its first row and
// writes through one based at its first output row, so every access is a
// scalar row offset plus a per-lane column offset.  The hardware checks the
// sum of the two against the resource's size and turns an access outside it
// into a zero read or a dropped store; the row loop relies on that instead
// of clamping: rows above or below the tile read zeros, rows that are not
// output rows (and halo lanes, whose column offset is kNoStore) are not
// stored.  A tile spans less than 2^30 bytes, so no offset sum wraps.
constexpr uint32_t kNoStore = 0x80000000u;
constexpr int64_t kMaxTileBytes = 1LL << 30;

// The base (wave-uniform) passes through an empty asm, so that the compiler
// knows nothing of what it points to: a load it took for invariant (the mask
// is never written) would sink to its use, and the row step would wait a
// whole memory latency for it.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *base, uint32_t bytes)
{
    asm volatile("" : "+s"(base));
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
// Store cache policy of the field rows.  kStoreThrough (sc1): the L2 writes
// them through at agent scope, so its lines are clean when the kernel ends
// and the release between two passes has nothing to write back.  Measured
// on one 2048 x 2048 grid (one wave per SIMD): the gap from one pass's last
// wave to the next pass's first falls from 2.2 to 0.9 us, while a wave's own
// time grows by 0.15 us.  A batch pass (several waves per SIMD, long passes)
// is faster with the default write-back policy (kStoreBack): 44.8 against
// 47.4 ms for 256 grids.
constexpr int kStoreThrough = 16, kStoreBack = 0;

// the 64- and 128-bit buffer builtins take and return these (GCC-style)
// vector types; they are only ever bit-cast or subscripted
typedef uint32_t bv2 __attribute__((__vector_size__(8)));
typedef uint32_t bv4 __attribute__((__vector_size__(16)));
template <int AUX>
__device__ __forceinline__ void bstore(float v, __amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, (int)vo, (int)so, AUX);
}
template <int AUX>
__device__ __forceinline__ void bstore(double v, __amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(bv2, v), r, (int)vo, (int)so, AUX);
}

// Two adjacent elements in one access.  Rows need no alignment beyond the
// element's (buffer accesses of several dwords are dword aligned), and the
// range check of such an access is made dword by dword.
template <typename T> struct Pair { T a, b; };
__device__ __forceinline__ Pair<float> bload2(float *, __amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so)
{
    // elements are copied out before the bit cast: clang bit-casts a vector
    // element lvalue from the vector's first element
    const bv2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, 0);
    const uint32_t a = v[0], b = v[1];
    return {__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
__device__ __forceinline__ Pair<double> bload2(double *, __amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so)
{
    struct D2 { double a, b; };
    const D2 v = __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(r, (int)vo, (int)so, 0));
    return {v.a, v.b};
}
template <int AUX>
__device__ __forceinline__ void bstore2(float a, float b, __amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so)
{
    bv2 v;
    v[0] = __builtin_bit_cast(uint32_t, a);
    v[1] = __builtin_bit_cast(uint32_t, b);
    __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)vo, (int)so, AUX);
}
template <int AUX>
__device__ __forceinline__ void bstore2(double a, double b, __amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so)
{
    struct D2 { double a, b; };
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(bv4, D2{a, b}), r, (int)vo, (int)so, AUX);
}

// v where the sign-extended mask byte m is all ones (a FREE cell), +0 where it
// is zero: one AND (the compiler folds the byte's sign extension into it)
__device__ __forceinline__ float keep(float v, int32_t m) { return __int_as_float(__float_as_int(v) & m); }
__device__ __forceinline__ double keep(double v, int32_t m)
{
    return __hiloint2double(__double2hiint(v) & m, __double2loint(v) & m);
}

// Source term of a tile: none; f (the constants of update.h are formed from
// f as the rows arrive); or c = omega f already formed (0 on fixed cells),
// from which a row needs only a and b.  kSrcC gives the bits of kSrcF with
// c = fl(omega f): a = w / 4 and b = 1 - w = fma(a, -4, 1) are exact.
constexpr int kSrcNone = 0, kSrcF = 1, kSrcC = 2;

// ---- streamed temporal-blocked red-black SOR ----------------------------
// One wave relaxes one tile: output columns [x0 + 2S, x0 + 128 - 2S) and
// rows [ybeg, yend) of a grid; x0 and ybeg are even, all tile values are
// wave-uniform.  wsrc is the one-byte free mask (0xFF on FREE cells, else
// 0): a FREE cell takes the factor omega, any other cell 0 (it is rewritten
// unchanged).  f is the source term of mode RHS.  Each lane moves its two
// columns in one access (three memory operations per row), which keeps a whole window
// of prefetches within the hardware's count of outstanding vector memory
// operations.  EVEN: nx is even, so a lane's two columns lie on the same side
// of the grid's edge; else the lane at the edge has its second column masked
// off as its row enters the pipeline and stores its first one alone (1001 x
// 743, S = 4: 6.3 us a pass with two accesses per lane for odd widths and
// pitches, before).
//
// Registers.  The pipeline needs NW = 2S + 2 rows at a time (the rows its
// stages touch and the row the last stage finishes), and each row is fetched
// NW row steps before it enters the pipeline.  Rows therefore live in a ring
// of 2 NW register slots: row t sits in slot t mod 2NW from its fetch to its
// last use, and the fetch of row t + NW refills the slot row t - NW has just
// left.  The loop body covers one turn of the ring, so every slot is a fixed
// register across iterations: no value is copied at the back edge, and no
// row step waits for a load younger than NW row steps.  Cells outside the
// grid read as zeros with factor 0, straight from the out-of-range loads.
//
// Measured at 2048 x 2048 (S = 6, 46 rows: 900 waves on 1024 SIMDs, bound by
// VALU issue): the trimmed first turn, tiles that end at their own last row and
// their heights took a replanning step from 6.16 to 5.65 ms and 256 FP64 sweeps
// from 1.13 to 0.92 ms at S = 4 (0.63 at the S = 6 of an untuned context).
// 1001 x 743 to residual 1e-6, with the mask bytes loaded at their use before:
// 5.5 to 2.96 ms, and 1.69 with two columns in one access at any width and
// passes fused between the checks.
//
// CHECK: the pass also measures the residual of its INPUT field, in FP64:
// r = ((E + W) + (S + N)) / 4 (+ f) - c over the FREE cells of its output
// rows and columns, the expression of the standalone residual kernels.  Row
// y's residual needs rows y - 1 and y + 1 as they were loaded; the pipeline's
// first stage rewrites row y - 1's red cells one row step before row y + 1
// arrives, so the loaded values of the previous row are kept in two extra
// registers.  rmax receives max |r| and rrel max |r| / |c| (|c| >= 1e-30,
// evaluated with the hardware reciprocal: a diagnostic), both per lane; a
// NaN residual propagates.  A check is VALU work next to the pass's own (at
// S = 8 a checking row costs 43 instructions on top of 80, a third of them
// FP64), so it takes the fewest: the maxima of all lanes, the halo's dropped
// once at the end, and NaN seen by the integer maxima of the converted
// residuals instead of a test per cell (64 before; with fewer control
// launches a batch of 64 grids went from 8.47 to 8.00 ms).
__device__ __forceinline__ double nan_max(double a, double b) { return (b > a || b != b) ? b : a; }

// f(integral_constant<int, U>) for U = 0, 1, ..., one inlined copy each: the
// row loop's body is one of these, so it is unrolled whatever its size (a
// rolled body would index the register ring at run time, i.e. in scratch)
template <class F, int... U>
__device__ __forceinline__ void static_for(std::integer_sequence<int, U...>, F &&f)
{
    (f(std::integral_constant<int, U>{}), ...);
}
// the same, up to the first U whose f returns false
template <class F, int... U>
__device__ __forceinline__ void static_while(std::integer_sequence<int, U...>, F &&f)
{
    (void)(f(std::integral_constant<int, U>{}) && ...);
}
__device__ __forceinline__ float nan_maxf(float a, float b) { return (b > a || b != b) ? b : a; }

template <typename T, int S, int RHS, bool EVEN, bool CHECK = false, int STORE = kStoreThrough, bool SLOT_OFS = true>
__device__ __forceinline__ void stream_tile(const T *__restrict__ src, T *__restrict__ dst,
                                            const uint8_t *__restrict__ wsrc, T omega,
                                            const T *__restrict__ f, int nx, int ny, int pitch,
                                            int x0, int ybeg, int yend, double *rmax = nullptr,
                                            float *rrel = nullptr)
{
    static_assert(RHS == kSrcNone || RHS == kSrcF || RHS == kSrcC, "source mode");
    static_assert(!(CHECK && RHS == kSrcC), "the residual check needs f");
    constexpr int NW = 2 * S + 2;      // rows the pipeline holds (even)
    constexpr int NR = 2 * NW;         // ring slots
    const T quarter = omega * T(0.25);  // exact
    const int lane = threadIdx.x & (kWave - 1);
    const int r0 = ybeg - 2 * S;                   // first row streamed (even)
    const int T_rows = (yend - ybeg) + 4 * S;
    // rows that can reach a stored row: [lo, hi)
    const int lo = max(r0, 0), hi = min(yend + 2 * S, ny);
    // read resources end at the last cell of row hi - 1 and the write
    // resource at the last cell of row yend - 1, so no access reaches past
    // the caller's last row even when its allocation ends there
    const uint32_t rowb = (uint32_t)pitch * sizeof(T);
    const uint32_t cells = (uint32_t)(hi - lo - 1) * (uint32_t)pitch + (uint32_t)nx;
    const uint32_t outc = (uint32_t)(yend - ybeg - 1) * (uint32_t)pitch + (uint32_t)nx;
    const size_t base = (size_t)lo * pitch;
    const __amdgpu_buffer_rsrc_t rs = rsrc(src + base, cells * sizeof(T));
    // the mask's two bytes are read in one access, whole or not at all: its
    // resource ends one byte later (the mask buffer has that byte)
    const __amdgpu_buffer_rsrc_t rw = rsrc(wsrc + base, cells + 1);
    const __amdgpu_buffer_rsrc_t rf = rsrc(RHS ? f + base : src + base, cells * sizeof(T));
    const __amdgpu_buffer_rsrc_t rd = rsrc(dst + (size_t)ybeg * pitch, outc * sizeof(T));
    // per-lane constants: a column outside the grid gets an out-of-range
    // offset, so its value and factor read as zero; rows outside the grid
    // are out of range as well.  The row step thus uses the loads as they are.
    const int xa = x0 + 2 * lane;
    const bool in0 = xa >= 0 && xa < nx, in1 = xa + 1 >= 0 && xa + 1 < nx;
    const bool writer = lane >= S && lane < kWave - S;
    const uint32_t xb = in0 ? (uint32_t)xa * sizeof(T) : kNoStore;
    const uint32_t xm = in0 ? (uint32_t)xa : kNoStore;
    const uint32_t so2 = writer && (EVEN || in1) ? xb : kNoStore;  // both columns
    const uint32_t so1 = writer && !in1 ? xb : kNoStore;           // the first alone
    const int32_t in1m = in1 ? -1 : 0;
    // row offsets (bytes) of streamed row t and of output row t - 4S;
    // negative ones are far out of range as unsigned sums
    const int vrow0 = (r0 - lo) * (int)rowb, mrow0 = (r0 - lo) * pitch;
    const int orow0 = (r0 - 2 * S - ybeg) * (int)rowb;

    // ring: the two columns of a row (P0 = column 2 lane, P1 = 2 lane + 1),
    // its raw mask bytes and, with a source term, its f (or c) values
    T P0[NR], P1[NR], F0[NR], F1[NR];
    uint32_t M[NR];
    // factors of the rows in the pipeline, by row mod NW (red, black), and
    // with a source term the update constants of update.h
    T wR[NW], wB[NW];
    SrcConst<T> kR[NW], kB[NW];
    // loads of a row into ring slot `slot`: lane offsets (of the field, then
    // of the mask) and scalar row offsets.  The field is loaded before the
    // mask: the row step that takes the row in needs both, and loads complete
    // in order, so one wait (for the mask) covers the two.
    auto fetch_at = [&](int slot, uint32_t b, uint32_t m, uint32_t vo, uint32_t mo) {
        const Pair<T> v = bload2((T *)nullptr, rs, b, vo);
        P0[slot] = v.a;
        P1[slot] = v.b;
        M[slot] = __builtin_amdgcn_raw_buffer_load_b16(rw, (int)m, (int)mo, 0);
        if (RHS) {
            const Pair<T> h = bload2((T *)nullptr, rf, b, vo);
            F0[slot] = h.a;
            F1[slot] = h.b;
        }
    };
    // The first window (stream rows 0 .. NW - 1, some of them above the
    // grid) puts the whole row offset, negative for rows above the grid, in
    // the scalar part.  The loop fetches stream rows from NW on, which lie
    // at or below the tile's first in-grid row lo (r0 + NW > ybeg >= lo), so
    // there the row offset of stream row tb + NW + u (tb: the turn's first
    // step) splits into u rows, added to the lane offsets once per tile,
    // and tb + NW rows in one scalar offset per turn.  Both parts are
    // non-negative and the sums are the same as in one piece, so the range
    // check sees the same offsets and no sum wraps; the row steps spend no
    // scalar instruction on load offsets.  That costs 2 NR registers;
    // SLOT_OFS = false (kernels that run several waves per SIMD)
    // forms every fetch's offsets in the scalar part instead.
    uint32_t lb[NR], lm[NR];
#pragma unroll
    for (int u = 0; u < NR && SLOT_OFS; ++u) {
        lb[u] = xb + (uint32_t)u * rowb;
        lm[u] = xm + (uint32_t)u * (uint32_t)pitch;
        // kept as registers (not re-formed in the loop, where they would
        // cost an instruction each)
        asm volatile("" : "+v"(lb[u]), "+v"(lm[u]));
    }
    auto fetch = [&](int slot, int t) {
        fetch_at(slot, xb, xm, (uint32_t)(vrow0 + t * (int)rowb), (uint32_t)(mrow0 + t * pitch));
    };
    auto fetch_loop = [&](int slot, int u, int tb) {
        if constexpr (SLOT_OFS)
            fetch_at(slot, lb[u], lm[u], (uint32_t)(vrow0 + (tb + NW) * (int)rowb),
                     (uint32_t)(mrow0 + (tb + NW) * pitch));
        else
            fetch(slot, tb + u + NW);
    };
    // red and black cells of the row in ring slot s (red is the first
    // column on even rows; r0 is even, so a row's parity is its slot's)
    auto red = [&](int s) -> T & { return (s & 1) == 0 ? P0[s] : P1[s]; };
    auto blk = [&](int s) -> T & { return (s & 1) == 0 ? P1[s] : P0[s]; };

    // CHECK: loaded values of the row above the checked one (columns 2 lane
    // and 2 lane + 1), and the running maxima
    // (of every lane; the halo lanes' are dropped at the end).  The floats'
    // are kept as bit patterns, which order like non-negative floats with NaN
    // above infinity; cmax takes no NaN, cnan does.
    double upa = 0.0, upb = 0.0, cmax = 0.0;
    uint32_t crel = 0u, cnan = 0u;
    // rows t - 1 checked at row step t: t - 1 in [ybeg - r0, yend - r0)
    const int tchk0 = ybeg - r0 + 1, tchk1 = yend - r0 + 1;
    // rows before the first streamed one are zeros with factor 0; the first
    // window is fetched in slot order, so that slot 0's loads are the oldest
    // in flight when the loop starts
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        P0[i] = P1[i] = F0[i] = F1[i] = T(0);
        M[i] = 0u;
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) wR[i] = wB[i] = T(0);
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        fetch(i, i);
        __builtin_amdgcn_sched_barrier(0);
    }

    // One row step: row t (ring slot u, pipeline index u mod NW) enters the
    // pipeline, row t + NW is fetched, the first `stages` stages advance and
    // row t - 2S is stored (`out`).  u, stages and the flags are constants
    // wherever the step is inlined.
    auto step = [&](const int u, const int t, const bool prefetch, const int stages,
                    const bool out) __attribute__((always_inline)) {
        const int uw = u % NW;
        {
            // the mask bytes sign-extended (all ones on a FREE cell); the
            // factor is omega or +0, bit for bit omega x (0 or 1)
            const int32_t e0 = (int32_t)(M[u] << 24) >> 24;
            int32_t e1 = (int32_t)(M[u] << 16) >> 24;
            if constexpr (!EVEN) {
                // a second column outside the grid reads as zero and fixed
                e1 &= in1m;
                P1[u] = keep(P1[u], in1m);
                if (RHS) F1[u] = keep(F1[u], in1m);
            }
            const bool ev = (u & 1) == 0;
            if constexpr (RHS != kSrcC) {
                const T w0 = keep(omega, e0), w1 = keep(omega, e1);
                wR[uw] = ev ? w0 : w1;
                wB[uw] = ev ? w1 : w0;
                if constexpr (RHS == kSrcF) {
                    const SrcConst<T> k0 = src_const(w0, F0[u]), k1 = src_const(w1, F1[u]);
                    kR[uw] = ev ? k0 : k1;
                    kB[uw] = ev ? k1 : k0;
                }
            } else {
                const T a0 = keep(quarter, e0), a1 = keep(quarter, e1);
                const SrcConst<T> k0{a0, fused(a0, T(-4), T(1)), F0[u]}, k1{a1, fused(a1, T(-4), T(1)), F1[u]};
                kR[uw] = ev ? k0 : k1;
                kB[uw] = ev ? k1 : k0;
            }
        }
        if constexpr (CHECK) {
            // residual of row t - 1 (slot um, not yet touched by any
            // stage) from the kept row t - 2 and the new row t (slot u).
            // The sum of four is scaled by 1/4 and the centre subtracted (or
            // f added) in one fma: a scaled sum is exact, so the bits are
            // those of the separate operations.
            const int um = (u + NR - 1) % NR, uwm = (uw + NW - 1) % NW;
            const T ca = P0[um], cb = P1[um];
            const double dca = (double)ca, dcb = (double)cb;
            // only the tile's own rows (a uniform branch: the halo and
            // pipeline rows, two fifths of the steps, skip the FP64 work)
            if (t >= tchk0 && t < tchk1) {
                const bool ev = (um & 1) == 0;
                const T wa = ev ? wR[uwm] : wB[uwm], wb = ev ? wB[uwm] : wR[uwm];
                const double sa = (dcb + (double)shr1(cb)) + ((double)P0[u] + upa);
                const double sb = ((double)shl1(ca) + dca) + ((double)P1[u] + upb);
                double ra, rb;
                if constexpr (RHS == kSrcF) {
                    ra = __builtin_fma(sa, 0.25, (double)F0[um]) - dca;
                    rb = __builtin_fma(sb, 0.25, (double)F1[um]) - dcb;
                } else {
                    ra = __builtin_fma(sa, 0.25, -dca);
                    rb = __builtin_fma(sb, 0.25, -dcb);
                }
                ra = wa != T(0) ? ra : 0.0;
                rb = wb != T(0) ? rb : 0.0;
                cmax = fmax(cmax, fmax(fabs(ra), fabs(rb)));
                const float fa = fabsf((float)ra), fb = fabsf((float)rb);
                cnan = max(cnan, max(__float_as_uint(fa), __float_as_uint(fb)));
                const float aa = fabsf((float)ca), ab = fabsf((float)cb);
                const float qa = aa >= 1e-30f ? fa * __builtin_amdgcn_rcpf(aa) : 0.0f;
                const float qb = ab >= 1e-30f ? fb * __builtin_amdgcn_rcpf(ab) : 0.0f;
                crel = max(crel, max(__float_as_uint(fabsf(qa)), __float_as_uint(fabsf(qb))));
            }
            upa = dca;
            upb = dcb;
        }
        // row t + NW goes to the slot row t - NW left at the last step
        __builtin_amdgcn_sched_barrier(0);
        if (prefetch) fetch_loop((u + NW) % NR, u, t - u);
        // stage k: half-sweep k of the pass (red for even k) at row
        // t - 1 - k (slot s).  Its E, W and N (row above, slot sm)
        // neighbours were finished in earlier row steps; S (row below, slot
        // sp) is the value stage k - 1 produces in this row step and is
        // added last, so the chain through the stages is three operations
        // deep per stage.
        // E + W + N of stage k (red cells for even k, black for odd)
        auto ewn = [&](const int k) __attribute__((always_inline)) -> T {
            const int s = (u - 1 - k + 2 * NR) % NR;
            const int sm = (s + NR - 1) % NR;
            if ((k & 1) == 0) {
                const T b = blk(s);
                return ((s & 1) == 0 ? shr1(b) + b : shl1(b) + b) + blk(sm);
            }
            const T r = red(s);
            return ((s & 1) == 0 ? shl1(r) + r : shr1(r) + r) + red(sm);
        };
        // each stage's sum is formed one stage ahead of its update, which
        // gives the scheduler two independent chains to interleave
        T e_next = T(0);
        if (stages > 0) e_next = ewn(0);
#pragma unroll
        for (int k = 0; k < 2 * S; ++k) {
            if (k >= stages) continue;
            const int s = (u - 1 - k + 2 * NR) % NR;
            const int sp = (s + 1) % NR;
            const int sw = (uw - 1 - k + 2 * NW) % NW;
            const T e = e_next;
            if (k + 1 < stages) e_next = ewn(k + 1);
            if constexpr (RHS != kSrcNone) {
                if ((k & 1) == 0)
                    red(s) = upd_src(red(s), e, blk(sp), kR[sw]);
                else
                    blk(s) = upd_src(blk(s), e, red(sp), kB[sw]);
            } else {
                if ((k & 1) == 0)
                    red(s) = upd(red(s), e, blk(sp), wR[sw]);
                else
                    blk(s) = upd(blk(s), e, red(sp), wB[sw]);
            }
        }
        // the row finished by this step (row t - 2S) is stored; rows
        // outside [ybeg, yend) fall outside the write resource
        if (out) {
            const int s = (u - 2 * S + 2 * NR) % NR;
            const uint32_t ro = (uint32_t)(orow0 + t * (int)rowb);
            bstore2<STORE>(P0[s], P1[s], rd, so2, ro);
            if constexpr (!EVEN) bstore<STORE>(P0[s], rd, so1, ro);
        }
        // keep this row's prefetch in this row step: without the fence
        // the scheduler sinks every prefetch of the window to its end
        __builtin_amdgcn_sched_barrier(0);
    };

    // The first turn fills the pipeline: a stored row depends on the rows
    // within 2S - 1 - k of it after stage k, so stage k first matters at row
    // k + 1, which it meets at step 2k + 2, and the first stored row leaves
    // at step 4S.  Step u of that turn therefore runs u / 2 stages and stores
    // from u = 4S on: 2S(2S + 1) of a tile's 2S(RH + 4S) stage steps drop out
    // (19 % at S = 6 and 46 rows).  A tile of two rows or fewer ends inside
    // that turn (rows past its last one are computed but never stored).
    static_for(std::make_integer_sequence<int, NR>{}, [&](auto U) __attribute__((always_inline)) {
        constexpr int u = decltype(U)::value;
        step(u, u, true, u / 2 < 2 * S ? u / 2 : 2 * S, u >= 4 * S);
    });
    // Whole turns have no per-row branches: fetches are unconditional (rows
    // past the grid read zeros).
    const int T_end = SLOT_OFS ? T_rows : (T_rows + NW - 1) / NW * NW;
    int tb = NR;
    for (; tb + NR <= T_end; tb += NR)
        static_for(std::make_integer_sequence<int, NR>{}, [&](auto U) __attribute__((always_inline)) {
            step(decltype(U)::value, tb + U, true, 2 * S, true);
        });
    // The rest, fewer than NR steps: a whole window without branches if there
    // is one (fetching if more follows it), then single steps that leave at
    // the tile's last row, so any height costs only its own row steps.  The
    // kernels held to fewer registers (SLOT_OFS = false) pad the rest to
    // whole windows instead: their single steps spill (a batch of 64 grids
    // at S = 8 took 8.25 against 7.87 ms).
    auto window = [&](auto more) __attribute__((always_inline)) {
        static_for(std::make_integer_sequence<int, NW>{}, [&](auto U) __attribute__((always_inline)) {
            step(decltype(U)::value, tb + U, decltype(more)::value, 2 * S, true);
        });
    };
    auto last_steps = [&](auto from) __attribute__((always_inline)) {
        static_while(std::make_integer_sequence<int, NW - 1>{}, [&](auto U) __attribute__((always_inline)) {
            constexpr int u = decltype(from)::value + decltype(U)::value;
            if (tb + u >= T_rows) return false;
            step(u, tb + u, false, 2 * S, true);
            return true;
        });
    };
    if (T_end - tb == NW) {
        window(std::false_type{});
    } else if constexpr (SLOT_OFS) {
        if (T_end - tb > NW) {
            window(std::true_type{});
            last_steps(std::integral_constant<int, NW>{});
        } else {
            last_steps(std::integral_constant<int, 0>{});
        }
    }
    if constexpr (CHECK) {
        if (cnan > 0x7f800000u) cmax = __longlong_as_double(0x7ff8000000000000ll);
        *rmax = nan_max(*rmax, writer ? cmax : 0.0);
        *rrel = nan_maxf(*rrel, writer ? __uint_as_float(crel) : 0.0f);
    }
}

}  // namespace sdev
}  // namespace twg
