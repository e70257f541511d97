// Device-driven relaxation for gfx950: the convergence control of hpf_relax
// (Eqs. 1-2 relaxed to a residual tolerance; the FP64 defect-correction
// polish that certifies the field by the discrete maximum principle) runs on
// the GPU, so a solve needs no host round trip and can be captured into a
// graph.
//
// A solve is a sequence of launches of ONE kernel, k_relax_slot, each a
// "slot" whose work the device decides from a control block (RelaxCtl) in
// device memory:
//   PLAIN     one streamed pass of S red-black sweeps of the FP32 field
//             (ping-pong between the caller's psi and the context's alt);
//   DEFECT32  the first FP64 defect: psi64 = psi widened, r32 = the FP64
//             residual avg4(psi64) - psi64 rounded to FP32, e = 0;
//   CORR      one streamed pass of the FP32 correction solve
//             (I - J) e = r32 (ping-pong e / alt);
//   UPDATE    psi64 += e on FREE cells, psi = psi64 rounded, e = 0;
//   DEFECT64  the FP64 defect of psi64;
//   FINISH    the FP32 result into psi if it ended in alt, stats written;
//   DONE      nothing: surplus slots return at once.
// A pass measures the FP64 residual of its input field when the control
// block schedules a check there (stream_tile's CHECK path: no extra launch).
// Every workgroup of a slot adds its maxima to the block with atomics and
// then takes a ticket; the workgroup that takes the last ticket runs the
// controller (one thread):
// it reads the maxima, applies the stop rules (tolerance, sweep budget,
// rounding-floor stall), predicts the next check from the measured
// contraction, and moves the phase.  A decision is also published to a
// host-mapped word, which lets a blocking caller keep just enough slots
// queued; an asynchronous caller enqueues a fixed number of slots and one
// final slot that finishes whatever is left.
#include "cell_setup.h"
#include "stream_tile.h"

#include <algorithm>
#include <cmath>

namespace twg {

namespace {

using namespace sdev;

enum : int { PH_PLAIN = 0, PH_DEFECT32, PH_CORR, PH_UPDATE, PH_DEFECT64, PH_FINISH, PH_DONE };

// a solve stops at the FP32 rounding floor after three checks without a 10 %
// gain on its best residual that together span at least this many sweeps
constexpr int64_t kStallSweeps = 256;

// The words every slot reads when it starts, loaded together (one scalar
// load): a run of passes of the current solve began at slot run_slot with
// pass number `pass` and the field (or correction) in buffer parity
// `parity` (`cparity`); slot k of the run starts at the pass run_passes
// gives, on parity ^ ((k - run_slot) & 1), so a pass that does not check
// writes nothing to the control block.
struct alignas(32) RelaxHot {
    int32_t phase;
    int32_t parity;        // FP32 field at run_slot: 0 in psi, 1 in alt
    int32_t cparity;       // correction at run_slot: 0 in e, 1 in alt
    int32_t pass;          // pass number of slot run_slot
    int32_t run_slot;
    int32_t next_check;    // pass of the next residual check
    int32_t fresh;         // psi holds the rounded polished field
    int32_t wide;          // psi64 holds the (widened or polished) field
};

constexpr int kParts = 128;

struct RelaxCtl {
    RelaxHot h;
    RelaxConfig c;
    int32_t last_check;    // pass of the last check
    int32_t lead_check;    // the next check ends a correction start phase
    int32_t solve_checks;  // checks of the current solve
    int32_t stalls;
    int32_t checks;        // residual evaluations of the whole call
    int32_t rounds;        // defect-correction updates
    int32_t status;
    int32_t pad;
    uint32_t ticket;       // workgroups of the current slot that have finished
    uint32_t pad2;
    int64_t last_chunk, since, sweeps, polish_sweeps;
    double tol_cur, r_prev, best, rate, rate_dc;
    double residual32, residual_rel, residual;
    // bit patterns of the slot's maxima, spread over kParts words so that
    // the workgroups' atomics seldom meet on one address (workgroup b uses
    // part[b % kParts]); the slot's last workgroup combines and clears them
    unsigned long long part[kParts][2];
};

// A run of n passes before a check, fused `fuse` (a power of two) at a time:
// passes done before slot k of the run, and (*level) the log2 of the passes
// slot k does.  From the slot of the check on, one pass a slot.
__device__ __forceinline__ int run_passes(int n, int fuse, int k, int *level)
{
    int done = 0;
    for (int l = fuse >= 4 ? 2 : fuse >= 2 ? 1 : 0; l > 0; --l) {
        const int q = max(n - done, 0) >> l;  // slots at this level
        if (k < q) {
            *level = l;
            return done + (k << l);
        }
        done += q << l;
        k -= q;
    }
    *level = 0;
    return done + k;
}
// slots such a run takes
__device__ __forceinline__ int run_slots(int n, int fuse)
{
    int slots = 0;
    for (int l = fuse >= 4 ? 2 : fuse >= 2 ? 1 : 0; l > 0; --l) {
        slots += n >> l;
        n &= (1 << l) - 1;
    }
    return slots + n;
}

__device__ __forceinline__ unsigned long long dbits(double d) { return (unsigned long long)__double_as_longlong(d); }
__device__ __forceinline__ double bitsd(unsigned long long b) { return __longlong_as_double((long long)b); }

__device__ __forceinline__ double wave_max(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = nan_max(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_maxf(float v)
{
    for (int o = 32; o > 0; o >>= 1) v = nan_maxf(v, __shfl_xor(v, o));
    return v;
}

// ---- controller (one thread of the last workgroup of a slot) --------------

// predicted passes to the next check of an FP32 solve at residual r
__device__ int32_t next_passes(RelaxCtl *c, double r)
{
    const int S = c->c.S;
    int64_t chunk;
    if (c->c.check_passes > 0) {
        chunk = (int64_t)c->c.check_passes * S;
    } else {
        // sweeps the measured contraction predicts, at most twice the last
        // chunk (a rate near 1 near the rounding floor must not turn into
        // one huge chunk); the prediction after the FP32 solve's initial
        // check (the first of a call, the rate still a guess) aims short
        const double want = log(c->tol_cur / r) / log(c->rate);
        const double k = c->h.phase == PH_PLAIN && c->solve_checks <= 1 ? 0.8 : 1.05;
        chunk = (int64_t)fmin(ceil(want * k), 1e12) + S;
        chunk = chunk > 8 * S ? chunk : 8 * S;
        if (c->last_chunk > 0) {
            const int64_t cap = 2 * c->last_chunk > 64 * S ? 2 * c->last_chunk : 64 * S;
            chunk = chunk < cap ? chunk : cap;
        }
    }
    int64_t passes = (chunk + S - 1) / S;
    const int64_t pmax = c->c.max_sweeps / S;
    if (c->h.pass + passes > pmax) passes = pmax - c->h.pass;
    if (passes < 1) passes = 1;
    c->last_chunk = passes * S;
    return (int32_t)passes;
}

// start the correction solve of one defect-correction round from residual r64
__device__ void start_correction(RelaxCtl *c, double r64, int32_t first_slot)
{
    c->h.phase = PH_CORR;
    c->h.pass = 0;
    c->h.cparity = 0;
    c->h.run_slot = first_slot;
    c->solve_checks = 0;
    // at most four decades per round (the FP32 correction keeps about that
    // much relative accuracy), and no further than the target with a 25 %
    // margin: after the FP64 update the field's residual is the correction
    // solve's own residual plus the rounding of the defect to FP32 (a
    // relative 6e-8) and of the update (about 1e-16)
    c->tol_cur = fmax(r64 * 1e-4, c->c.need / 1.25);
    c->r_prev = r64;
    c->best = r64;
    c->stalls = 0;
    c->since = 0;
    c->last_chunk = 0;
    c->last_check = 0;
    c->rate = (c->rate_dc > 0.0 && c->rate_dc < 1.0) ? c->rate_dc : fmax((double)c->c.omega_dc - 1.0, 0.5);
    if (c->c.lead_passes > 0 && c->c.max_sweeps >= c->c.S) {
        // the start phase runs at the smaller factor, then a check
        int32_t lp = c->c.lead_passes;
        const int32_t pmax = (int32_t)(c->c.max_sweeps / c->c.S);
        c->h.next_check = lp < pmax ? lp : pmax;
        c->lead_check = 1;
    } else {
        // the defect is the solve's initial residual (e = 0)
        c->solve_checks = 1;
        c->h.next_check = next_passes(c, r64);
        c->lead_check = 0;
    }
}

// end of the FP32 solve at pass p (the result is this pass's input)
__device__ void end_solve(RelaxCtl *c, bool conv, double r, double rel)
{
    if (c->h.phase == PH_PLAIN) {
        c->sweeps = (int64_t)c->h.pass * c->c.S;
        c->residual32 = r;
        c->residual_rel = rel;
        c->residual = r;
        c->status = conv ? TWG_OK : TWG_NOT_CONVERGED;
        c->h.phase = c->c.polish ? PH_DEFECT32 : PH_FINISH;
    } else {
        c->polish_sweeps += (int64_t)c->h.pass * c->c.S;
        c->rate_dc = c->rate;
        c->h.phase = PH_UPDATE;
    }
}

// a residual check of an FP32 solve at pass c->h.pass
__device__ void on_check(RelaxCtl *c, double r, double rel)
{
    ++c->checks;
    const bool initial = c->solve_checks == 0 || c->lead_check;
    ++c->solve_checks;
    if (r != r) {
        c->status = TWG_EINVAL;
        c->h.phase = PH_FINISH;
        return;
    }
    if (initial) {
        c->best = r;
        c->stalls = 0;
        c->since = 0;
        c->lead_check = 0;
    } else {
        const int64_t chunk = (int64_t)(c->h.pass - c->last_check) * c->c.S;
        double q = 1.0;
        if (r < c->r_prev && chunk > 0) {
            q = pow(r / c->r_prev, 1.0 / (double)chunk);
            if (q > 0.0 && q < 1.0) c->rate = q;
        }
        // A correction solve that contracts at less than half the speed its
        // factor gives every mode once the factor is at or above a domain's
        // optimum (omega - 1 per sweep) has met the FP32 rounding floor of
        // its correction: a correction with a large smooth part leaves FP32
        // residual noise of ~1e-7 times its own size, which can lie above
        // the solve's target.  The round ends there; the FP64 update and
        // the next round's exact defect carry on from it.  Judged over at
        // least 128 sweeps.
        if (c->h.phase == PH_CORR && chunk >= 128) {
            const double w = (double)c->c.omega_dc;
            if (q > 1.0 - 0.5 * (2.0 - w)) {
                // the next round's first prediction starts from the nominal
                // rate, not from the floor's
                c->rate = fmax(w - 1.0, 0.5);
                end_solve(c, false, r, rel);
                return;
            }
        }
        // the max-norm residual is not monotone, so progress is judged
        // against the best residual, over a span of sweeps
        if (r < 0.9 * c->best) {
            c->best = r;
            c->stalls = 0;
            c->since = 0;
        } else {
            c->since += chunk;
            ++c->stalls;
        }
    }
    c->r_prev = r;
    c->last_check = c->h.pass;
    if (r <= c->tol_cur) {
        end_solve(c, true, r, rel);
        return;
    }
    if ((int64_t)c->h.pass * c->c.S >= c->c.max_sweeps || (c->stalls >= 3 && c->since >= kStallSweeps)) {
        end_solve(c, false, r, rel);
        return;
    }
    c->h.next_check = c->h.pass + next_passes(c, r);
}

// a defect: polish done, or the next correction round.  The first defect
// of a kept field's polish (no check has run yet) also stands in for the
// FP32 stage's initial check: it evaluates the same FP64 expression over
// the same FREE cells of the same field, so when that residual meets tol the
// FP32 stage ends as it would at that check, with no sweep; else the FP32
// solve runs from its own initial check and the first defect comes again.
__device__ void on_defect(RelaxCtl *c, double r64, double rel, int32_t slot_now)
{
    if (c->h.phase == PH_DEFECT32 && c->checks == 0 && r64 == r64 && !(r64 <= c->tol_cur)) {
        ++c->checks;
        c->h.phase = PH_PLAIN;
        c->h.pass = 0;
        c->h.run_slot = slot_now + 1;
        c->h.next_check = 0;
        return;
    }
    if (c->h.phase == PH_DEFECT32 && c->checks == 0 && r64 == r64) {
        c->sweeps = 0;
        c->residual32 = r64;
        c->residual_rel = rel;
        c->status = TWG_OK;
    }
    ++c->checks;
    c->residual = r64;
    c->h.wide = 1;
    if (r64 != r64) {
        c->status = TWG_EINVAL;
        c->h.phase = PH_FINISH;
    } else if (r64 <= c->c.need) {
        c->status = TWG_OK;
        c->h.phase = PH_FINISH;
    } else if (c->rounds >= c->c.max_rounds) {
        c->status = TWG_NOT_CONVERGED;
        c->h.phase = PH_FINISH;
    } else {
        start_correction(c, r64, slot_now + 1);
    }
}

__device__ void write_stats(const RelaxCtl *c, hpf_stats *s)
{
    s->sweeps = c->sweeps;
    s->polish_sweeps = c->polish_sweeps;
    s->residual = c->residual;
    s->residual32 = c->residual32;
    s->cert_bound = c->residual * c->c.wbound;
    s->wbound = c->c.wbound;
    s->omega = c->c.omega;
    s->status = c->status;
    s->polish_rounds = c->rounds;
    s->checks = c->checks;
    s->residual_rel = c->residual_rel;
}

// decision published for a blocking caller: the slot of the next decision
// (+1) in the low word, bit 63 when the solve is done
__device__ void publish(const RelaxCtl *c, unsigned long long *mirror, int32_t slot_now)
{
    if (!mirror) return;
    unsigned long long w;
    if (c->h.phase == PH_DONE) {
        w = 1ull << 63;
    } else {
        int64_t next = slot_now + 1;  // DEFECT, UPDATE and FINISH decide in their own slot
        if (c->h.phase == PH_PLAIN || c->h.phase == PH_CORR) next = slot_now + run_slots(c->h.next_check - c->h.pass, c->c.fuse) + 1;
        w = (unsigned long long)(next + 1);
    }
    *reinterpret_cast<volatile unsigned long long *>(mirror) = w;
    __threadfence_system();
}

// The controller of a slot that decides: a checking pass (at pass p, on
// buffer parity par), a defect, an update, or the finish (`forced`: the
// final slot ends a solve whose phase was `was`, at pass p on parity par
// if that phase was a solve).
__device__ void controller_on(RelaxCtl *c, const SlotArgs &a, int32_t slot_now, unsigned long long *mirror, int phase,
                              int was, bool forced, int32_t p, int32_t par, double r, double rel)
{
    switch (phase) {
    case PH_PLAIN:
    case PH_CORR: {
        // the run's state at this pass, then the check
        c->h.pass = p;
        c->h.run_slot = slot_now;
        if (phase == PH_PLAIN) c->h.parity = par;
        else c->h.cparity = par;
        on_check(c, r, rel);
        // the pass's output is the field from here on, unless the solve
        // ended at this check (its input is the result)
        if (c->h.phase == phase && c->h.pass == p) {
            if (phase == PH_PLAIN) c->h.parity = par ^ 1;
            else c->h.cparity = par ^ 1;
            c->h.pass = p + 1;
            c->h.run_slot = slot_now + 1;
        }
        break;
    }
    case PH_DEFECT32:
    case PH_DEFECT64: on_defect(c, r, rel, slot_now); break;
    case PH_UPDATE:
        ++c->rounds;
        c->h.fresh = 1;
        c->h.phase = PH_DEFECT64;
        break;
    case PH_FINISH:
        if (forced) {
            c->status = TWG_NOT_CONVERGED;
            // a solve cut short between checks: its passes so far count,
            // and the FP32 field is where its last pass wrote it
            if (was == PH_PLAIN) {
                c->h.parity = par;
                c->sweeps = (int64_t)p * c->c.S;
            } else if (was == PH_CORR) {
                c->polish_sweeps += (int64_t)p * c->c.S;
            }
        }
        write_stats(c, a.stats);
        c->h.phase = PH_DONE;
        break;
    }
    publish(c, mirror, slot_now);
}

// The controller works on a copy of the control block in registers: read in
// one batch of independent loads and written back once, instead of a chain
// of dependent global accesses (each a memory latency).  The words other
// workgroups update atomically (ticket, maxima) are read and reset here with
// atomics and not written back.
__device__ void controller(RelaxCtl *cg, const SlotArgs &a, int phase, int was, bool forced, int32_t p, int32_t par,
                           double r, double rel)
{
    RelaxCtl c = *cg;
    controller_on(&c, a, a.slot, a.mirror, phase, was, forced, p, par, r, rel);
    cg->h = c.h;
    cg->last_check = c.last_check;
    cg->lead_check = c.lead_check;
    cg->solve_checks = c.solve_checks;
    cg->stalls = c.stalls;
    cg->checks = c.checks;
    cg->rounds = c.rounds;
    cg->status = c.status;
    cg->last_chunk = c.last_chunk;
    cg->since = c.since;
    cg->sweeps = c.sweeps;
    cg->polish_sweeps = c.polish_sweeps;
    cg->tol_cur = c.tol_cur;
    cg->r_prev = c.r_prev;
    cg->best = c.best;
    cg->rate = c.rate;
    cg->rate_dc = c.rate_dc;
    cg->residual32 = c.residual32;
    cg->residual_rel = c.residual_rel;
    cg->residual = c.residual;
}

// ---- element-wise and stencil phases ----------------------------------------

// The cells of a slot's elementwise phases: work items are (row, run of 256
// columns), spread over all waves of the launch; each lane takes four
// columns 64 apart.  K work items at a time, each cell split into `load`
// (reads and arithmetic, returning a value) and `store` (writes): every load
// of the 4K cells is issued before the first store, so a wave has that many
// cells' loads in flight instead of one cell's (the stores could alias the
// loads, so the compiler keeps them in program order).  A cell outside the
// grid loads cell (0, 0) and stores nothing.
template <int K, typename L, typename St>
__device__ __forceinline__ void for_cells_batched(const SlotArgs &a, int gw, int nwaves, L load, St store)
{
    using V = decltype(load(0, 0));
    const int lane = threadIdx.x & 63;
    const int runs = (a.nx + 255) / 256;
    const int items = a.ny * runs;
    for (int it0 = gw; it0 < items; it0 += K * nwaves) {
        V v[K][4];
        int ys[K], xs[K][4];
        bool ok[K][4];
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int it = it0 + q * nwaves;
            const bool in = it < items;
            const int y = in ? it / runs : 0;
            const int x0 = in ? (it - y * runs) * 256 + lane : 0;
            ys[q] = y;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                xs[q][j] = x0 + 64 * j;
                ok[q][j] = in && xs[q][j] < a.nx;
                v[q][j] = load(ok[q][j] ? xs[q][j] : 0, ok[q][j] ? y : 0);
            }
        }
#pragma unroll
        for (int q = 0; q < K; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (ok[q][j]) store(xs[q][j], ys[q], v[q][j]);
    }
}
// a store written through L2 at agent scope (sc1)
template <typename T>
__device__ __forceinline__ void st_through(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
struct DefectCell {
    double c, r;
    bool fr;
};
struct UpdateCell {
    double v;
    float e;
    bool fr;
};

// FP64 residual of u at (x, y) with the neighbours outside the grid at 0;
// every load unconditional (clamped, then zeroed), as in the standalone
// residual kernels
template <typename T>
__device__ __forceinline__ double defect_at(const T *u, int nx, int ny, int pitch, int x, int y, double *c_out)
{
    const size_t row = (size_t)y * pitch;
    const int xe = min(x + 1, nx - 1), xw = max(x - 1, 0);
    const double ue = (double)u[row + xe], uw = (double)u[row + xw];
    const double us = (double)u[(size_t)min(y + 1, ny - 1) * pitch + x];
    const double un = (double)u[(size_t)max(y - 1, 0) * pitch + x];
    const double c = (double)u[row + x];
    const double e = x + 1 < nx ? ue : 0.0;
    const double w = x > 0 ? uw : 0.0;
    const double s = y + 1 < ny ? us : 0.0;
    const double n = y > 0 ? un : 0.0;
    *c_out = c;
    return ((e + w) + (s + n)) * 0.25 - c;
}

// A phase that is no pass, on the cells that `cells` goes over (a callable
// taking `load` and `store`); fpar, cpar: the buffers of the FP32 field and
// of the correction.  The maxima of a defect go to m and mr.
template <typename Cells>
__device__ __forceinline__ void element_phase(const SlotArgs &a, int phase, int fpar, int cpar, int fresh, int wide,
                                              double &m, float &mr, Cells cells)
{
    if (phase == PH_DEFECT32 || phase == PH_DEFECT64) {
        const bool first = phase == PH_DEFECT32;
        const float *u32 = fpar ? a.alt : a.psi;
        // the defect's maxima, and its outputs written through L2 (as the
        // passes' field rows are, so the kernel's end has nothing to write
        // back): the widened field and a cleared correction the first time
        auto store = [&](int x, int y, const DefectCell &d) {
            const size_t i = (size_t)y * a.pitch + x;
            if (first) {
                st_through(a.psi64 + i, d.c);
                st_through(a.e + i, 0.0f);
            }
            // the correction solves' source, and its products with their
            // two factors, formed here once instead of in every pass
            const float f = d.fr ? (float)d.r : 0.0f;
            st_through(a.r32 + i, f);
            st_through(a.cdc + i, a.omega_dc * f);
            if (a.lead_passes > 0) st_through(a.clead + i, a.omega_lead * f);
            m = nan_max(m, d.fr ? fabs(d.r) : 0.0);
            const float ac = fabsf((float)d.c);
            mr = nan_maxf(mr, d.fr && ac >= 1e-30f ? fabsf((float)d.r) * __builtin_amdgcn_rcpf(ac) : 0.0f);
        };
        auto load = [&](const auto *u, int x, int y) {
            DefectCell d;
            d.r = defect_at(u, a.nx, a.ny, a.pitch, x, y, &d.c);
            d.fr = a.mask[(size_t)y * a.pitch + x] != 0;
            return d;
        };
        if (first)
            cells([&](int x, int y) { return load(u32, x, y); }, store);
        else
            cells([&](int x, int y) { return load(a.psi64, x, y); }, store);
    } else if (phase == PH_UPDATE) {
        const float *ecur = cpar ? a.alt : a.e;
        // ecur may be e itself: every cell's correction is read before any
        // cell's is cleared
        cells(
            [&](int x, int y) {
                const size_t i = (size_t)y * a.pitch + x;
                return UpdateCell{a.psi64[i], ecur[i], a.mask[i] != 0};
            },
            [&](int x, int y, const UpdateCell &u) {
                const size_t i = (size_t)y * a.pitch + x;
                double v = u.v;
                if (u.fr) {
                    v = v + (double)u.e;
                    st_through(a.psi64 + i, v);
                }
                st_through(a.psi + i, (float)v);
                st_through(a.e + i, 0.0f);
            });
    } else {  // PH_FINISH
        const bool copy = !fresh && fpar;
        const bool widen = a.psi64 && a.polish && !wide;
        if (copy || widen) {
            const float *u = copy ? a.alt : a.psi;
            cells([&](int x, int y) { return u[(size_t)y * a.pitch + x]; },
                  [&](int x, int y, float v) {
                      const size_t i = (size_t)y * a.pitch + x;
                      if (copy) a.psi[i] = v;
                      if (widen) a.psi64[i] = (double)v;
                  });
        }
    }
}

// F: passes of S sweeps that one launch may do at once (1, 2 or 4)
//
// A pass of a small grid is mostly latency, so the kernel's scalar reads come
// in two batches: the control block's hot words (ctl and slot, the first
// arguments, arrive in registers with the wave) next to every other argument
// a pass uses, then nothing more before the first rows (read where they are
// used, they were four dependent batches; 0.3 us of a pass).
template <int S, int F, bool EVEN>
__global__ __launch_bounds__(256) void k_relax_slot(void *ctl, int slot, SlotArgs a)
{
    RelaxCtl *c = static_cast<RelaxCtl *>(ctl);
    // the hot words in one load; everything below is wave-uniform
    const RelaxHot h = *static_cast<const RelaxHot *>(ctl);
    asm volatile("" ::"s"(a.mask), "s"(a.psi), "s"(a.alt), "s"(a.e), "s"(a.r32), "s"(a.cdc), "s"(a.clead), "s"(a.nx),
                 "s"(a.ny), "s"(a.pitch), "s"(a.blocks), "s"(a.final_slot), "s"(a.tiling[0].strips),
                 "s"(a.tiling[0].RH), "s"(a.tiling[0].tiles), "s"(a.omega), "s"(a.omega_dc), "s"(a.lead_passes));
    const int was = __builtin_amdgcn_readfirstlane(h.phase);
    // position in the current run of passes (solve phases), derived before
    // any branch so that the words above arrive in one load
    const int k = __builtin_amdgcn_readfirstlane(slot - h.run_slot);
    // slot k of a run: passes fused F (then F / 2, ...) at a time while that
    // many are left before the next check, which starts a slot of its own
    const int next_check = __builtin_amdgcn_readfirstlane(h.next_check);
    int level = 0;
    const int pass = __builtin_amdgcn_readfirstlane(h.pass) +
                     run_passes(__builtin_amdgcn_readfirstlane(next_check - h.pass), F > 1 ? a.fuse : 1, k, &level);
    const int par = (__builtin_amdgcn_readfirstlane(was == PH_CORR ? h.cparity : h.parity) ^ k) & 1;
    const int hfresh = __builtin_amdgcn_readfirstlane(h.fresh), hwide = __builtin_amdgcn_readfirstlane(h.wide);
    const int hpar = __builtin_amdgcn_readfirstlane(h.parity), hcpar = __builtin_amdgcn_readfirstlane(h.cparity);
    if (was == PH_DONE) return;
    const bool forced = a.final_slot && was < PH_FINISH;
    const int phase = forced ? (int)PH_FINISH : was;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = a.blocks * 4;
    double m = 0.0;
    float mr = 0.0f;
    bool reduce = false;

    if (phase == PH_PLAIN || phase == PH_CORR) {
        const bool corr = phase == PH_CORR;
        const bool check = pass >= next_check;
        reduce = check;
        float *x0 = corr ? a.e : a.psi;
        float *src = par ? a.alt : x0, *dst = par ? x0 : a.alt;
        const float om = corr ? (pass < a.lead_passes ? a.omega_lead : a.omega_dc) : a.omega;
        const SlotTiling t = a.tiling[F > 1 ? level : 0];
        // this tiling's blocks, spread over all XCDs
        const int used = (t.tiles + 3) / 4;
        const int gw = ((int)blockIdx.x < used ? xcd_remap(blockIdx.x, used) : used) * 4 + wave;
        if (gw < t.tiles) {
            const int strip = gw % t.strips, seg = gw / t.strips;
            const int ybeg = seg * t.RH, yend = min(ybeg + t.RH, a.ny);
            const float *cs = pass < a.lead_passes ? a.clead : a.cdc;
            // a tile of D sweeps that does not check
            auto tile = [&](auto D) __attribute__((always_inline)) {
                constexpr int d = decltype(D)::value;
                const int xs = strip * (128 - 4 * d) - 2 * d;
                if (corr)
                    stream_tile<float, d, kSrcC, EVEN, false>(src, dst, a.mask, om, cs, a.nx, a.ny, a.pitch, xs, ybeg,
                                                              yend);
                else
                    stream_tile<float, d, kSrcNone, EVEN, false>(src, dst, a.mask, om, nullptr, a.nx, a.ny, a.pitch,
                                                                 xs, ybeg, yend);
            };
            if (check) {
                const int xs = strip * (128 - 4 * S) - 2 * S;
                if (corr)
                    stream_tile<float, S, kSrcF, EVEN, true>(src, dst, a.mask, om, a.r32, a.nx, a.ny, a.pitch,
                                                             xs, ybeg, yend, &m, &mr);
                else
                    stream_tile<float, S, kSrcNone, EVEN, true>(src, dst, a.mask, om, nullptr, a.nx, a.ny,
                                                                a.pitch, xs, ybeg, yend, &m, &mr);
            } else if (F >= 4 && level == 2) {
                tile(std::integral_constant<int, F >= 4 ? 4 * S : S>{});
            } else if (F >= 2 && level == 1) {
                tile(std::integral_constant<int, F >= 2 ? 2 * S : S>{});
            } else {
                tile(std::integral_constant<int, S>{});
            }
        }
        // a pass that does not check decides nothing: the next slot derives
        // its pass and buffers from its own slot number
        if (!check) return;
    } else {
        reduce = phase != PH_UPDATE && phase != PH_FINISH;
        // the FP32 field's buffer: a solve cut short between checks left it
        // where its last pass wrote
        const int fpar = phase == PH_FINISH && was == PH_PLAIN ? par : hpar;
        element_phase(a, phase, fpar, hcpar, hfresh, hwide, m, mr,
                      [&](auto load, auto store) {
                          const int gw = xcd_remap(blockIdx.x, a.blocks) * 4 + wave;
                          for_cells_batched<2>(a, gw, nwaves, load, store);
                      });
    }

    // maxima, then the ticket, one per workgroup: the block's maxima are
    // combined in LDS, its atomics are performed before it takes its ticket
    // (a wait on their results), so the block that takes the last ticket
    // reads the maxima of every block
    __shared__ double bm[4];
    __shared__ float br[4];
    __shared__ int last;
    if (reduce) {
        m = wave_max(m);
        mr = wave_maxf(mr);
        if (lane == 0) {
            bm[wave] = m;
            br[wave] = mr;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (reduce) {
            m = nan_max(nan_max(bm[0], bm[1]), nan_max(bm[2], bm[3]));
            mr = nan_maxf(nan_maxf(br[0], br[1]), nan_maxf(br[2], br[3]));
            unsigned long long *pp = c->part[blockIdx.x % kParts];
            __hip_atomic_fetch_max(pp, dbits(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_max(pp + 1, dbits((double)mr), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_s_waitcnt(0);
        }
        const unsigned int ticket =
            __hip_atomic_fetch_add(&c->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = ticket == (unsigned)a.blocks - 1u;
    }
    __syncthreads();
    if (!last) return;
    // the last workgroup: the slot's maxima from the kParts words (one
    // thread each, read and cleared), combined as bit patterns like the
    // atomics (non-negative doubles order like their patterns; a NaN's is
    // larger than +inf's)
    unsigned long long pr = 0ull, pq = 0ull;
    if (threadIdx.x < kParts) {
        pr = __hip_atomic_exchange(&c->part[threadIdx.x][0], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        pq = __hip_atomic_exchange(&c->part[threadIdx.x][1], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int o = 32; o > 0; o >>= 1) {
        pr = max(pr, (unsigned long long)__shfl_xor((long long)pr, o));
        pq = max(pq, (unsigned long long)__shfl_xor((long long)pq, o));
    }
    __shared__ unsigned long long wr[4], wq[4];
    if (lane == 0) {
        wr[wave] = pr;
        wq[wave] = pq;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    pr = max(max(wr[0], wr[1]), max(wr[2], wr[3]));
    pq = max(max(wq[0], wq[1]), max(wq[2], wq[3]));
    __hip_atomic_exchange(&c->ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    controller(c, a, phase, was, forced, pass, par, bitsd(pr), bitsd(pq));
}

#ifndef TWG_DEPTH
// ---- small grids: the whole solve in one workgroup's registers ---------------
// A grid of at most 128 x 96 (or 64 x 128) cells is too small for the passes:
// a launch of eight sweeps takes 6 us there, half of it the launch and the
// first load, and every sweep of it is redone in the tiles' halos.  Here one
// workgroup keeps the field in registers for a whole solve: a lane holds two
// columns of a block of R rows, 64 lanes a row of up to 128 cells (NARROW: 32
// lanes a row of up to 64, two blocks a wave), a half-sweep updates one of a
// lane's two cells in every row, and the blocks' first and last rows go
// through LDS, one barrier a half-sweep.  A half-sweep is bound by VALU issue
// of the four waves (5 operations a row, 6 where the shift must stop between
// two blocks: 84 of 140 ns at R = 8) and by what the inner rows do not hide
// of the rows' way through LDS and the barrier.  The updates, the checks, the
// control (on an LDS copy of the control block) and the elementwise phases
// are those of the slots, so a field after N sweeps has the same bits.  A
// launch ends after kResidentWork sweeps, so none runs long; the field is then
// in psi (or e) and the next launch goes on.  4000 sweeps of 64 x 64 cells:
// 3.32 to 1.12 ms; certified to 1e-9 (1068 sweeps, 64 x 32): 1.01 to 0.38 ms.
constexpr int kResidentWork = 4096;
constexpr int kCheckWork = 16;  // a check's share of that

template <bool NARROW, int R>
__global__ __launch_bounds__(256) void k_relax_resident(void *ctl, int slot, SlotArgs a)
{
    constexpr int LW = NARROW ? 32 : 64;  // lanes of a row
    constexpr int B = 4 * (64 / LW);      // blocks of rows
    RelaxCtl *cg = static_cast<RelaxCtl *>(ctl);
    __shared__ RelaxCtl sc;
    // boundary rows by colour (a checked field's two columns use both):
    // block b's first and last row at [.][b + 1]; zeros above and below all
    __shared__ float halo[2][B + 2][2][LW];
    __shared__ double bm[4];
    __shared__ float br[4];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (static_cast<const RelaxHot *>(ctl)->phase == PH_DONE) return;
    for (int i = tid; i < (int)(sizeof(RelaxCtl) / 4); i += 256)
        reinterpret_cast<uint32_t *>(&sc)[i] = reinterpret_cast<const uint32_t *>(cg)[i];
    for (int i = tid; i < (int)(sizeof(halo) / 4); i += 256) (&halo[0][0][0][0])[i] = 0.0f;

    const int li = lane & (LW - 1), blk = NARROW ? 2 * wave + (lane >> 5) : wave;
    const int x = 2 * li, y0 = blk * R;
    // a neighbour across the two blocks of a wave is outside the grid
    int32_t lm = li == 0 ? 0 : -1, rm = li == LW - 1 ? 0 : -1;
    asm volatile("" : "+v"(lm), "+v"(rm));  // masks, not conditions: the shift folds into the AND
    auto from_left = [&](float v) { return NARROW ? keep(shr1(v), lm) : shr1(v); };
    auto from_right = [&](float v) { return NARROW ? keep(shl1(v), rm) : shl1(v); };
    // A lane's cells in memory.  Each use forms its own (the empty asm): kept
    // across the solve, the addresses and conditions of every cell would
    // spill.
    struct Cells {
        int x, y, nx, ny, pitch;
        __device__ bool in(int r, int j) const { return x + j < nx && y + r < ny; }
        __device__ size_t at(int r, int j) const { return (size_t)(y + r) * pitch + x + j; }
    };
    auto cells_now = [&] {
        Cells q{x, y0, a.nx, a.ny, a.pitch};
        asm volatile("" : "+v"(q.x), "+v"(q.y));
        return q;
    };

    uint32_t free0 = 0u, free1 = 0u;  // bit r: row r's cell is FREE
    {
        const Cells q = cells_now();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (q.in(r, 0) && a.mask[q.at(r, 0)]) free0 |= 1u << r;
            if (q.in(r, 1) && a.mask[q.at(r, 1)]) free1 |= 1u << r;
        }
    }
    float P0[R], P1[R];
    auto load_cells = [&](const float *u, float (&v0)[R], float (&v1)[R]) {
        const Cells q = cells_now();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v0[r] = q.in(r, 0) ? u[q.at(r, 0)] : 0.0f;
            v1[r] = q.in(r, 1) ? u[q.at(r, 1)] : 0.0f;
        }
    };
    auto store_cells = [&](float *u) {
        const Cells q = cells_now();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (q.in(r, 0)) u[q.at(r, 0)] = P0[r];
            if (q.in(r, 1)) u[q.at(r, 1)] = P1[r];
        }
    };
    // n sweeps; upd_cell(r, j, ewn, s) updates the cell of column j in row r
    auto sweeps = [&](int n, auto upd_cell) {
        // the black cells of the boundary rows, then one barrier a half-sweep
        halo[1][blk + 1][0][li] = P1[0];
        halo[1][blk + 1][1][li] = P0[R - 1];
        __syncthreads();
        auto half = [&](auto C) __attribute__((always_inline)) {
            constexpr int c = decltype(C)::value;
            const float up = halo[1 - c][blk][1][li], dn = halo[1 - c][blk + 2][0][li];
            auto row = [&](auto Rr) __attribute__((always_inline)) {
                constexpr int r = decltype(Rr)::value;
                constexpr int rn = r > 0 ? r - 1 : 0, rs = r + 1 < R ? r + 1 : R - 1;
                if constexpr (((r + c) & 1) == 0) {
                    const float ewn = (from_left(P1[r]) + P1[r]) + (r > 0 ? P0[rn] : up);
                    upd_cell(std::integral_constant<int, r>{}, std::integral_constant<int, 0>{}, ewn,
                             r + 1 < R ? P0[rs] : dn);
                } else {
                    const float ewn = (from_right(P0[r]) + P0[r]) + (r > 0 ? P1[rn] : up);
                    upd_cell(std::integral_constant<int, r>{}, std::integral_constant<int, 1>{}, ewn,
                             r + 1 < R ? P1[rs] : dn);
                }
            };
            // half of the inner rows while the neighbours' rows arrive, the
            // boundary rows, and the rest while those go out
            static_for(std::make_integer_sequence<int, R / 2 - 1>{},
                       [&](auto U) { row(std::integral_constant<int, decltype(U)::value + 1>{}); });
            row(std::integral_constant<int, 0>{});
            row(std::integral_constant<int, R - 1>{});
            halo[c][blk + 1][0][li] = c == 0 ? P0[0] : P1[0];
            halo[c][blk + 1][1][li] = c == 0 ? P1[R - 1] : P0[R - 1];
            __builtin_amdgcn_sched_barrier(0);
            static_for(std::make_integer_sequence<int, R / 2 - 1>{},
                       [&](auto U) { row(std::integral_constant<int, decltype(U)::value + R / 2>{}); });
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
        };
        for (int k = 0; k < n; ++k) {
            half(std::integral_constant<int, 0>{});
            half(std::integral_constant<int, 1>{});
        }
    };
    // the workgroup's maxima to thread 0, which decides
    auto decide = [&](int phase, int pass, double m, float mr) {
        m = wave_max(m);
        mr = wave_maxf(mr);
        __syncthreads();
        if (lane == 0) {
            bm[wave] = m;
            br[wave] = mr;
        }
        __syncthreads();
        if (tid == 0) {
            m = nan_max(nan_max(bm[0], bm[1]), nan_max(bm[2], bm[3]));
            mr = nan_maxf(nan_maxf(br[0], br[1]), nan_maxf(br[2], br[3]));
            // decisions are not published: the host queues launches, not slots
            controller_on(&sc, a, slot, nullptr, phase, phase, false, pass, 0, m, (double)mr);
            // fields stay in psi and e, and the checked pass is still to run
            sc.h.parity = sc.h.cparity = 0;
            if (sc.h.phase == phase && (phase == PH_PLAIN || phase == PH_CORR)) sc.h.pass = pass;
        }
        __syncthreads();
    };
    const int S = __builtin_amdgcn_readfirstlane(cg->c.S);
    int left = kResidentWork;
    __syncthreads();
    for (;;) {
        const int phase = __builtin_amdgcn_readfirstlane(sc.h.phase);
        if (phase == PH_DONE || left <= 0) break;
        if (phase != PH_PLAIN && phase != PH_CORR) {
            double m = 0.0;
            float mr = 0.0f;
            element_phase(a, phase, 0, 0, __builtin_amdgcn_readfirstlane(sc.h.fresh),
                          __builtin_amdgcn_readfirstlane(sc.h.wide), m, mr, [&](auto load, auto store) {
                              using V = decltype(load(0, 0));
                              constexpr int K = 4;  // rows at a time
                              Cells c = cells_now();
#pragma unroll 1
                              for (int q = 0; q < R; q += K, c.y += K) {
                                  V v[K][2];
#pragma unroll
                                  for (int r = 0; r < K; ++r)
#pragma unroll
                                      for (int j = 0; j < 2; ++j)
                                          v[r][j] = load(c.in(r, j) ? c.x + j : 0, c.in(r, j) ? c.y + r : 0);
#pragma unroll
                                  for (int r = 0; r < K; ++r)
#pragma unroll
                                      for (int j = 0; j < 2; ++j)
                                          if (c.in(r, j)) store(c.x + j, c.y + r, v[r][j]);
                              }
                          });
            left -= kCheckWork;
            decide(phase, 0, m, mr);  // its barriers also order the phases' stores and loads
            continue;
        }
        const bool corr = phase == PH_CORR;
        float *field = corr ? a.e : a.psi;
        load_cells(field, P0, P1);
        for (;;) {
            const int pass = __builtin_amdgcn_readfirstlane(sc.h.pass);
            const int next_check = __builtin_amdgcn_readfirstlane(sc.h.next_check);
            // passes of one factor, within this launch's work
            const bool lead = corr && pass < a.lead_passes;
            int n = lead ? min(next_check, a.lead_passes) - pass : next_check - pass;
            n = min(max(n, 0), (max(left, 0) + S - 1) / S);
            if (n > 0) {
                if (corr) {
                    const float om = lead ? a.omega_lead : a.omega_dc, quarter = om * 0.25f;
                    SrcConst<float> k0[R], k1[R];
                    float c0[R], c1[R];
                    load_cells(lead ? a.clead : a.cdc, c0, c1);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const float a0 = free0 >> r & 1u ? quarter : 0.0f, a1 = free1 >> r & 1u ? quarter : 0.0f;
                        k0[r] = {a0, fused(a0, -4.0f, 1.0f), c0[r]};
                        k1[r] = {a1, fused(a1, -4.0f, 1.0f), c1[r]};
                    }
                    sweeps(n * S, [&](auto Rr, auto J, float ewn, float s) __attribute__((always_inline)) {
                        constexpr int r = decltype(Rr)::value;
                        float &p = decltype(J)::value ? P1[r] : P0[r];
                        p = upd_src(p, ewn, s, decltype(J)::value ? k1[r] : k0[r]);
                    });
                } else {
                    float w0[R], w1[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        w0[r] = free0 >> r & 1u ? a.omega : 0.0f;
                        w1[r] = free1 >> r & 1u ? a.omega : 0.0f;
                    }
                    sweeps(n * S, [&](auto Rr, auto J, float ewn, float s) __attribute__((always_inline)) {
                        constexpr int r = decltype(Rr)::value;
                        float &p = decltype(J)::value ? P1[r] : P0[r];
                        p = upd(p, ewn, s, decltype(J)::value ? w1[r] : w0[r]);
                    });
                }
                left -= n * S;
            }
            if (pass + n < next_check) {
                __syncthreads();
                if (tid == 0) sc.h.pass = pass + n;
                __syncthreads();
                if (left <= 0) break;
                continue;
            }
            // the residual of the field at this check, in FP64, the
            // expression of the passes' checks (its source: the FP32 defect)
            halo[0][blk + 1][0][li] = P0[0];
            halo[1][blk + 1][0][li] = P1[0];
            halo[0][blk + 1][1][li] = P0[R - 1];
            halo[1][blk + 1][1][li] = P1[R - 1];
            __syncthreads();
            double m = 0.0;
            float mr = 0.0f;
            {
                const float up0 = halo[0][blk][1][li], up1 = halo[1][blk][1][li];
                const float dn0 = halo[0][blk + 2][0][li], dn1 = halo[1][blk + 2][0][li];
                float f0[R], f1[R];
                if (corr) load_cells(a.r32, f0, f1);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float n0 = r > 0 ? P0[r > 0 ? r - 1 : 0] : up0, n1 = r > 0 ? P1[r > 0 ? r - 1 : 0] : up1;
                    const float s0 = r + 1 < R ? P0[r + 1 < R ? r + 1 : 0] : dn0;
                    const float s1 = r + 1 < R ? P1[r + 1 < R ? r + 1 : 0] : dn1;
                    auto cell = [&](bool fr, float c, float e, float w, float nn, float ss, float f) {
                        double g = (((double)e + (double)w) + ((double)ss + (double)nn)) * 0.25;
                        if (corr) g = g + (double)f;
                        const double d = g - (double)c;
                        const float ac = fabsf(c);
                        m = nan_max(m, fr ? fabs(d) : 0.0);
                        mr = nan_maxf(mr, fr && ac >= 1e-30f ? fabsf((float)d) * __builtin_amdgcn_rcpf(ac) : 0.0f);
                    };
                    const float w = from_left(P1[r]), e = from_right(P0[r]);
                    cell(free0 >> r & 1u, P0[r], P1[r], w, n0, s0, corr ? f0[r] : 0.0f);
                    cell(free1 >> r & 1u, P1[r], e, P0[r], n1, s1, corr ? f1[r] : 0.0f);
                }
            }
            left -= kCheckWork;
            decide(phase, next_check, m, mr);
            if (__builtin_amdgcn_readfirstlane(sc.h.phase) != phase) break;
        }
        store_cells(field);
        __syncthreads();
    }
    // the control block (its maxima and ticket are not in use here), then the
    // word a blocking caller waits for
    for (int i = tid; i < (int)(offsetof(RelaxCtl, part) / 4); i += 256)
        reinterpret_cast<uint32_t *>(cg)[i] = reinterpret_cast<const uint32_t *>(&sc)[i];
    if (tid == 0) {
        const bool done = sc.h.phase == PH_DONE;
        *reinterpret_cast<volatile unsigned long long *>(a.mirror) = done ? 1ull << 63 : (unsigned long long)(slot + 2);
        __threadfence_system();
    }
}
#endif

// Set-up of a solve: the cells (boundary and initial values, free mask), and
// in the first block the control block.
__global__ __launch_bounds__(256) void k_relax_begin(RelaxCtl *c, RelaxConfig cfg, CellSetup cells, int lane_bits)
{
    setup_grid(cells, lane_bits);
    if (blockIdx.x != 0 || blockIdx.y != 0) return;
    for (int i = threadIdx.x; i < kParts; i += blockDim.x) {
        __hip_atomic_store(&c->part[i][0], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&c->part[i][1], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x != 0) return;
    // member by member: a copy of the whole would be staged by every thread
    c->c.tol = cfg.tol;
    c->c.need = cfg.need;
    c->c.wbound = cfg.wbound;
    c->c.max_sweeps = cfg.max_sweeps;
    c->c.omega = cfg.omega;
    c->c.omega_dc = cfg.omega_dc;
    c->c.omega_lead = cfg.omega_lead;
    c->c.lead_passes = cfg.lead_passes;
    c->c.S = cfg.S;
    c->c.polish = cfg.polish;
    c->c.check_passes = cfg.check_passes;
    c->c.max_rounds = cfg.max_rounds;
    c->c.fuse = cfg.fuse;
    c->c.kept = cfg.kept;
    c->h.phase = cfg.kept ? PH_DEFECT32 : PH_PLAIN;
    c->h.parity = c->h.cparity = c->h.fresh = c->h.wide = 0;
    c->h.pass = 0;
    c->h.run_slot = 0;
    c->h.next_check = 0;  // the initial field's residual, fused into pass 0
    c->last_check = 0;
    c->lead_check = 0;
    c->solve_checks = 0;
    c->stalls = 0;
    c->checks = c->rounds = 0;
    c->status = TWG_NOT_CONVERGED;
    c->last_chunk = c->since = c->sweeps = c->polish_sweeps = 0;
    c->tol_cur = cfg.tol;
    c->r_prev = c->best = 0.0;
    c->rate = fmax((double)cfg.omega - 1.0, 0.5);
    c->rate_dc = 0.0;
    c->residual32 = c->residual_rel = c->residual = 0.0;
    __hip_atomic_exchange(&c->ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

int last_status() { return hipGetLastError() == hipSuccess ? TWG_OK : TWG_EDEVICE; }

}  // namespace

// Each depth's kernels are instantiated in a translation unit of their own
// (this file compiled with TWG_DEPTH set), so that they build in parallel.
template <int S>
int launch_relax_slot_depth(const SlotArgs &a, hipStream_t st)
{
    constexpr int F = slot_fuse_limit(S);
    const dim3 blocks(a.blocks);
    if (F > 1 && a.fuse > 1) {
        if (a.even)
            hipLaunchKernelGGL((k_relax_slot<S, F, true>), blocks, dim3(256), 0, st, a.ctl, a.slot, a);
        else
            hipLaunchKernelGGL((k_relax_slot<S, F, false>), blocks, dim3(256), 0, st, a.ctl, a.slot, a);
    } else {
        if (a.even)
            hipLaunchKernelGGL((k_relax_slot<S, 1, true>), blocks, dim3(256), 0, st, a.ctl, a.slot, a);
        else
            hipLaunchKernelGGL((k_relax_slot<S, 1, false>), blocks, dim3(256), 0, st, a.ctl, a.slot, a);
    }
    return last_status();
}

#ifdef TWG_DEPTH
template int launch_relax_slot_depth<TWG_DEPTH>(const SlotArgs &, hipStream_t);
#else
#define TWG_SLOT_DEPTH(SV) extern template int launch_relax_slot_depth<SV>(const SlotArgs &, hipStream_t);
TWG_SLOT_DEPTH(1) TWG_SLOT_DEPTH(2) TWG_SLOT_DEPTH(3) TWG_SLOT_DEPTH(4)
TWG_SLOT_DEPTH(5) TWG_SLOT_DEPTH(6) TWG_SLOT_DEPTH(7) TWG_SLOT_DEPTH(8)
#undef TWG_SLOT_DEPTH

size_t relax_ctl_bytes() { return (sizeof(RelaxCtl) + 255) & ~size_t(255); }

// Blocks of 8, 16 and 24 rows take 0.28 (0.26 with 64 lanes a row), 0.45
// (0.40) and 0.60 us a sweep where the passes take 0.82 to 0.85; at 32 rows a
// block (128 x 128) it is 0.76, and certified solves gain nothing.
bool relax_resident(int nx, int ny) { return (nx <= 128 && ny <= 96) || (nx <= 64 && ny <= 128); }

int launch_relax_resident(const SlotArgs &a, hipStream_t st)
{
    if (!relax_resident(a.nx, a.ny)) return TWG_EUNSUPPORTED;
    // the fewest rows a block that hold the grid
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(1), dim3(256), 0, st, a.ctl, a.slot, a); };
    if (a.nx <= 64) {
        if (a.ny <= 64) go(k_relax_resident<true, 8>);
        else go(k_relax_resident<true, 16>);
    } else if (a.ny <= 32) {
        go(k_relax_resident<false, 8>);
    } else if (a.ny <= 64) {
        go(k_relax_resident<false, 16>);
    } else {
        go(k_relax_resident<false, 24>);
    }
    return last_status();
}

int launch_relax_begin(void *ctl, const RelaxConfig &cfg, const CellSetup &cells, hipStream_t st)
{
    hipLaunchKernelGGL(k_relax_begin, setup_blocks(cells.nx, cells.ny), dim3(256), 0, st, static_cast<RelaxCtl *>(ctl),
                       cfg, cells, setup_lane_bits(cells.nx));
    return last_status();
}

int launch_relax_slot(const SlotArgs &a, int S, hipStream_t st)
{
    switch (S) {
    case 1: return launch_relax_slot_depth<1>(a, st);
    case 2: return launch_relax_slot_depth<2>(a, st);
    case 3: return launch_relax_slot_depth<3>(a, st);
    case 4: return launch_relax_slot_depth<4>(a, st);
    case 5: return launch_relax_slot_depth<5>(a, st);
    case 6: return launch_relax_slot_depth<6>(a, st);
    case 7: return launch_relax_slot_depth<7>(a, st);
    case 8: return launch_relax_slot_depth<8>(a, st);
    default: return TWG_EUNSUPPORTED;
    }
}
#endif

}  // namespace twg
