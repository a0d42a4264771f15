// Multigrid drivers (Sec. 6.2): the V(nu_pre, nu_post) cycle with damped
// Jacobi smoothing, the FP64 solver and the mixed-precision defect
// correction with single-precision inner cycles.  Cycles are captured once
// per hierarchy into HIP graphs and replayed, which removes the launch cost
// of the coarse levels (tens of tiny kernels per cycle).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <chrono>
#include <cmath>
#include <string>
#include <vector>

#include "fused_ops.h"
#include "solve.h"

struct GraphEntry {
    int kind;  // 0: FP64 cycle + residual norm; 1: FP32 inner cycle + residual norm;
               // 2, 3: preconditioned CG step with an FP64 / FP32 cycle;
               // 4: `reps` guarded FP32 inner cycles, each with its norm and control;
               // 5: a guarded FP64 cycle with its norm and control, `reps` its CHAIN_ flags
    int reps;
    int nu_pre, nu_post;
    double omega;
    bool x_zero;
    hipGraphExec_t exec;
    double bytes;
    uint64_t epoch;  // tile table epoch the fused passes were captured with
};

// One cycle of a chain (enqueue_chain): starts with its own pre pass, ends with
// a post pass, finds the pre-smoothed iterate in the second buffer.
constexpr int CHAIN_ENTER = 1, CHAIN_LEAVE = 2, CHAIN_ODD = 4, CHAIN_CYCLE = 8;

struct GraphCache {
    hipStream_t st = nullptr;  // internal non-blocking stream (capture needs one)
    hipEvent_t ev_in = nullptr, ev_out = nullptr;  // order st after / before the caller's stream
    bool capture_ok = true;
    std::vector<GraphEntry> entries;
};

namespace mg {

namespace {

template <typename T>
struct LV;
template <>
struct LV<double> {
    static double* x(Level& l) { return l.x64; }
    static double* b(Level& l) { return l.b64; }
    static double* t(Level& l) { return l.t64; }
    static const double* bands(const Level& l) { return l.bands64; }
};
template <>
struct LV<float> {
    static float* x(Level& l) { return l.x32; }
    static float* b(Level& l) { return l.b32; }
    static float* t(Level& l) { return l.t32; }
    static const float* bands(const Level& l) { return l.bands32; }
};

#define MG_TRY(call)                         \
    do {                                     \
        hipError_t e_ = (call);              \
        if (e_ != hipSuccess) return e_;     \
    } while (0)

}  // namespace

// Byte model (algorithmic HBM traffic, s = sizeof(T)) of one level of the
// cycle as separate kernels: band product family 9 bands + x (+ b) (+ output);
// Jacobi from zero: diagonal + b + output; restriction: fine defect + coarse
// rhs; prolongation: coarse x + fine x read and written; a copy of the iterate
// after an odd number of sweeps.
static double unfused_level_bytes(double s, double n, double nc, bool x_zero, int nu_pre,
                                  int nu_post) {
    double b = x_zero && nu_pre == 0 ? s * n : 0.0;
    b += nu_pre > 0 && x_zero ? 3 * s * n + 12 * s * n * (nu_pre - 1) : 12 * s * n * nu_pre;
    b += 12 * s * n + s * (n + nc) + s * (nc + 2 * n) + 12 * s * n * nu_post;
    return b + ((nu_pre + nu_post) % 2 ? 2 * s * n : 0.0);
}

// The V(nu_pre, nu_post) cycle as separate kernels.  Cycles other than
// V(2,2) -- which has its own fused form (enqueue_vcycle_fused) and stays
// unfused here, as its reference -- run the levels of the coarse tail in its
// one launch, and a level with a single pre- or post-smoothing sweep as block
// passes where those exist; the same bits.
template <typename T>
hipError_t enqueue_vcycle(mg_hierarchy* h, int l, T* x, const T* b, bool x_zero, int nu_pre,
                          int nu_post, double omega, Enq& q) {
    Level& lv = h->lv[l];
    const double s = sizeof(T), n = (double)lv.n;
    const T om = (T)omega;
    if (l == h->Lc) {
        MG_TRY(launch_coarse<T>(coarse_solver(h), lv.N, b, x, q.st));
        q.bytes += 2 * s * n;
        return hipSuccess;
    }
    const bool reference = nu_pre == 2 && nu_post == 2;
    const bool one = !reference && one_sweep_blocks(lv.N, sizeof(T));
    const T* bands = LV<T>::bands(lv);
    Level& lc = h->lv[l - 1];
    q.bytes += unfused_level_bytes(s, n, (double)lc.n, x_zero, nu_pre, nu_post);
    T* cur = x;
    T* oth = LV<T>::t(lv);
    if (one && nu_pre == 1) {
        MG_TRY(launch_pre1<T>(lv, bands, cur, x_zero, b, om, oth, LV<T>::b(lc), h->dmask, q.st));
        std::swap(cur, oth);
    } else {
        bool zero = x_zero;
        if (zero && nu_pre == 0) {
            MG_TRY(launch_fill<T>(cur, lv.n, T(0), q.st));
            zero = false;
        }
        for (int k = 0; k < nu_pre; ++k) {
            if (zero)
                MG_TRY(launch_jacobi_zero<T>(lv, bands, b, oth, om, q.st));
            else
                MG_TRY(launch_jacobi<T>(lv, bands, b, cur, oth, om, q.st));
            zero = false;
            std::swap(cur, oth);
        }
        MG_TRY(launch_defect<T>(lv, bands, b, cur, oth, nullptr, nullptr, 0, nullptr, q.st));
        MG_TRY(launch_restrict<T>(lv.N, oth, LV<T>::b(lc), h->dmask, q.st));
    }
    if (!reference && l - 1 <= tail_max_level()) {
        MG_TRY(launch_tail<T>(h->lv, l - 1, h->Lc, coarse_solver(h), nu_pre, nu_post, om, q.st));
        for (int k = h->Lc + 1; k < l; ++k)
            q.bytes += unfused_level_bytes(s, (double)h->lv[k].n, (double)h->lv[k - 1].n, true,
                                           nu_pre, nu_post);
        q.bytes += 2 * s * (double)h->lv[h->Lc].n;
    } else {
        MG_TRY(enqueue_vcycle<T>(h, l - 1, LV<T>::x(lc), LV<T>::b(lc), true, nu_pre, nu_post,
                                 omega, q));
    }
    if (one && nu_post == 1) {
        MG_TRY(launch_post1<T>(lv, bands, cur, LV<T>::x(lc), b, om, oth, q.st));
        std::swap(cur, oth);
    } else {
        MG_TRY(launch_prolong<T>(lv.N, LV<T>::x(lc), cur, q.st));
        for (int k = 0; k < nu_post; ++k) {
            MG_TRY(launch_jacobi<T>(lv, bands, b, cur, oth, om, q.st));
            std::swap(cur, oth);
        }
    }
    if (cur != x) MG_TRY(launch_copy<T>(cur, x, lv.n, q.st));
    return hipSuccess;
}

template hipError_t enqueue_vcycle<double>(mg_hierarchy*, int, double*, const double*, bool, int,
                                           int, double, Enq&);
template hipError_t enqueue_vcycle<float>(mg_hierarchy*, int, float*, const float*, bool, int,
                                          int, double, Enq&);

template <typename T>
static hipError_t enqueue_pre(mg_hierarchy* h, int l, const T* x, const T* b, bool x_zero, T om,
                              T* t, Enq& q) {
    Level &lv = h->lv[l], &lc = h->lv[l - 1];
    const double s = sizeof(T);
    q.bytes += (x_zero ? 11 : 12) * s * (double)lv.n + s * (double)lc.n;
    return launch_pre<T>(lv, LV<T>::bands(lv), x, x_zero, b, om, t, LV<T>::b(lc), h->dmask, q.st,
                         q.guard);
}

// The levels below l of a fused cycle, from b_c to x_c.
template <typename T>
static hipError_t enqueue_coarse_cycle(mg_hierarchy* h, int l, double omega, Enq& q) {
    Level& lc = h->lv[l - 1];
    if (l - 1 > tail_max_level())
        return enqueue_vcycle_fused<T>(h, l - 1, LV<T>::x(lc), LV<T>::b(lc), true, omega, q,
                                       nullptr, nullptr, 0, nullptr);
    // every coarser level in one workgroup; same bytes as the unfused cycle there
    for (int k = h->Lc + 1; k < l; ++k) q.bytes += 84.0 * sizeof(T) * (double)h->lv[k].n;
    const RedJob job = q.pending;
    q.pending = RedJob{};
    return launch_tail<T>(h->lv, l - 1, h->Lc, coarse_solver(h), 2, 2, (T)omega, q.st, q.guard,
                          job);
}

template <typename T>
static hipError_t enqueue_post(mg_hierarchy* h, int l, const T* t, const T* b, T om, T* x, Enq& q,
                               double* partials, double* scal, int slot, double* host) {
    Level &lv = h->lv[l], &lc = h->lv[l - 1];
    const double s = sizeof(T);
    q.bytes += 12 * s * (double)lv.n + s * (double)lc.n;
    return launch_post<T>(lv, LV<T>::bands(lv), t, LV<T>::x(lc), b, om, x, partials, scal, slot,
                          host, q.st, q.guard, partials ? q.ctl : RedCtl{});
}

// V(2,2) cycle from the fused passes: per level one pre pass (two sweeps,
// defect, restriction: x -> t, b_c) and one post pass (prolongation, two
// sweeps: t + P x_c -> x).  With partials the top-level post pass also
// reduces ||b - A x|| into scal[slot], scal[slot + 1] (and host[slot..]).  Byte model: bands
// (9 s), iterate in (s, not when from zero), b (s) and iterate out (s) per
// node and pass, plus the coarse vector (s per coarse node).
template <typename T>
hipError_t enqueue_vcycle_fused(mg_hierarchy* h, int l, T* x, const T* b, bool x_zero,
                                double omega, Enq& q, double* partials, double* scal, int slot,
                                double* host) {
    Level& lv = h->lv[l];
    const double s = sizeof(T), n = (double)lv.n;
    const T om = (T)omega;
    const T* bands = LV<T>::bands(lv);
    if (l == h->Lc) {
        if (q.guard) return hipErrorInvalidValue;  // guarded cycles need a level above the tail
        MG_TRY(launch_coarse<T>(coarse_solver(h), lv.N, b, x, q.st));
        q.bytes += 2 * s * n;
        if (partials) {
            MG_TRY(launch_defect<T>(lv, bands, b, x, nullptr, partials, scal, slot, host, q.st));
            q.bytes += 11 * s * n;
        }
        return hipSuccess;
    }
    T* t = LV<T>::t(lv);
    MG_TRY(enqueue_pre<T>(h, l, x, b, x_zero, om, t, q));
    MG_TRY(enqueue_coarse_cycle<T>(h, l, omega, q));
    return enqueue_post<T>(h, l, t, b, om, x, q, partials, scal, slot, host);
}

template hipError_t enqueue_vcycle_fused<double>(mg_hierarchy*, int, double*, const double*, bool,
                                                 double, Enq&, double*, double*, int, double*);
template hipError_t enqueue_vcycle_fused<float>(mg_hierarchy*, int, float*, const float*, bool,
                                                double, Enq&, double*, double*, int, double*);

// V(2,2) cycles in a row on the finest level, each with its residual norm.
// MERGED: a cycle's post pass and the next one's pre pass in one (launch_mid):
// x gets every cycle's result, the smoothed iterate the next cycle starts from
// alternates between t and alt.  CHAIN_ENTER: the first cycle starts from x;
// otherwise from the pre-smoothed iterate that a merged chain without
// CHAIN_LEAVE left in t (in alt after an odd number of cycles).
//
// Under a guard, the norm of every cycle but the last is reduced beside the
// next cycle's coarse tail (on a level with 33 k partials a reduction took 6 us
// and a launch gap, a twelfth of a cycle).  If it ends the loop, what ran
// since (the way down to the tail) has written coarse vectors and t only; all
// that follows is skipped.
template <typename T>
static hipError_t enqueue_chain(mg_hierarchy* h, T* x, const T* b, T* t, T* alt, int cycles,
                                bool merged, bool x_zero, int part, double omega, Enq& q,
                                int slot) {
    const int L = h->L;
    Level &lv = h->lv[L], &lc = h->lv[L - 1];
    const T om = (T)omega;
    const double s = sizeof(T);
    for (int i = 0; i < cycles; ++i) {
        const bool last = i == cycles - 1;
        if (i == 0 ? (part & CHAIN_ENTER) != 0 : !merged)
            MG_TRY(enqueue_pre<T>(h, L, x, b, x_zero && i == 0, om, t, q));
        MG_TRY(enqueue_coarse_cycle<T>(h, L, omega, q));
        double* scal = last ? h->scal : nullptr;
        if (!merged || ((part & CHAIN_LEAVE) && last)) {
            MG_TRY(enqueue_post<T>(h, L, t, b, om, x, q, h->partials, scal, slot, h->host_scal));
        } else {
            MG_TRY(launch_mid<T>(lv, LV<T>::bands(lv), t, LV<T>::x(lc), b, om, x, alt,
                                 LV<T>::b(lc), h->dmask, h->partials, scal, slot, h->host_scal,
                                 q.st, q.guard, q.ctl));
            q.bytes += 13 * s * (double)lv.n + 2 * s * (double)lc.n;
            std::swap(t, alt);
        }
        if (!last)
            q.pending = reduce_job(h->partials, dev::fused_norm_parts(lv.N), h->scal, slot,
                                   h->host_scal, q.ctl);
    }
    return hipSuccess;
}

// The second buffer of the pre-smoothed iterate is a finest-level FP64 vector
// the solver has no use for: d64 in the FP64 solve, t64 in the mixed one.
static bool chained(const mg_hierarchy* h, int elem_bytes) {
    return h->L > h->Lc && use_mid(h->lv[h->L].N, elem_bytes);
}

// One step of CG preconditioned by one V-cycle from zero (Sec. 4.1: a
// solver as another's preconditioner; the cycle of Sec. 6.2), on the finest
// level's vectors: x in x64, r in d64, p in b64 (the right-hand side copy is
// not needed once r0 is formed), and z / q sharing the FP32 pair x32|b32
// (never live together, nor with the FP32 cycle's own use of the pair):
//   z = M r (kind 2: FP64 cycle; kind 3: FP32 cycle on r / ||r||, z =
//   ||r|| c32); rz = r.z; p = z + (rz / rz_old) p; rz_old = rz; q = A p;
//   alpha = rz / p.q; x += alpha p; r -= alpha q; ||r|| to the host mirror.
// Before the first step scal[SC_RZ] is +inf; the reduction of r.z moves it to
// scal[SC_RZ_OLD] before it writes its own, so the first p is z.  p.q comes out
// of the product's own pass (a pass over two vectors and two launches a step
// less: L = 11 with FP32 cycles, a solve of 6 steps 1.83 -> 1.74 ms).
static hipError_t enqueue_pcg_step(mg_hierarchy* h, bool mixed, int nu_pre, int nu_post,
                                   double omega, Enq& q) {
    Level& F = h->lv[h->L];
    const int64_t n = F.n;
    const double dn = (double)n;
    double* r = h->d64;
    double* p = F.b64;
    double* zq = reinterpret_cast<double*>(F.x32);
    const bool fused = nu_pre == 2 && nu_post == 2;
    RedCtl shift;
    shift.mode = RED_SHIFT;
    if (!mixed) {
        if (fused)
            MG_TRY(enqueue_vcycle_fused<double>(h, h->L, zq, r, true, omega, q, nullptr, nullptr,
                                                0, nullptr));
        else
            MG_TRY(enqueue_vcycle<double>(h, h->L, zq, r, true, nu_pre, nu_post, omega, q));
        MG_TRY(launch_dot<double>(r, zq, n, h->scal, -1, h->partials, h->scal, SC_RZ, q.st,
                                  shift));
        MG_TRY(launch_pcg_dir<double>(p, zq, n, h->scal, -1, SC_RZ, SC_RZ_OLD, q.st));
        q.bytes += (16.0 + 24.0) * dn;
    } else {
        MG_TRY(launch_cast_scaled(r, F.b32, n, h->scal, SC_RR, q.st));
        if (fused)
            MG_TRY(enqueue_vcycle_fused<float>(h, h->L, F.x32, F.b32, true, omega, q, nullptr,
                                               nullptr, 0, nullptr));
        else
            MG_TRY(enqueue_vcycle<float>(h, h->L, F.x32, F.b32, true, nu_pre, nu_post, omega, q));
        MG_TRY(launch_dot<float>(r, F.x32, n, h->scal, SC_RR, h->partials, h->scal, SC_RZ, q.st,
                                 shift));
        MG_TRY(launch_pcg_dir<float>(p, F.x32, n, h->scal, SC_RR, SC_RZ, SC_RZ_OLD, q.st));
        q.bytes += (12.0 + 12.0 + 20.0) * dn;
    }
    MG_TRY(launch_spmv_dot(F, F.bands64, p, zq, h->partials, h->scal, SC_PQ, q.st));
    MG_TRY(launch_pcg_step(F.x64, r, p, zq, n, h->scal, SC_RZ, SC_PQ, h->partials, SC_RR,
                           h->host_scal, q.st));
    q.bytes += (88.0 + 48.0) * dn;
    return hipSuccess;
}

// The unit replayed per iteration: FP64 cycle + FP64 residual norm (kind 0)
// or FP32 inner cycle + FP32 residual norm (kind 1), on the finest level's
// own vectors, or a preconditioned CG step (kinds 2, 3), or `reps` fused
// FP32 inner cycles under device control (kind 4: each cycle's kernels
// return at once when scal[SC_STOP] is set, and the reduction of its
// residual norm decides whether the loop goes on: RED_STEP).
static hipError_t enqueue_unit(mg_hierarchy* h, int kind, int reps, int nu_pre, int nu_post,
                               double omega, bool x_zero, Enq& q) {
    Level& F = h->lv[h->L];
    const double n = (double)F.n;
    if (kind == 4) {
        Enq g{q.st, 0.0, h->scal + SC_STOP};
        g.ctl.mode = RED_STEP;
        MG_TRY(enqueue_chain<float>(h, F.x32, F.b32, F.t32, (float*)F.t64, reps, chained(h, 4),
                                    x_zero, CHAIN_ENTER | CHAIN_LEAVE, omega, g, SC_R32));
        q.bytes += g.bytes;
        return hipSuccess;
    }
    if (kind == 5) {
        Enq g{q.st, 0.0, h->scal + SC_STOP};
        g.ctl.mode = RED_CYCLE;
        double* t = reps & CHAIN_ODD ? h->d64 : F.t64;
        double* alt = reps & CHAIN_ODD ? F.t64 : h->d64;
        MG_TRY(enqueue_chain<double>(h, F.x64, F.b64, t, alt, reps / CHAIN_CYCLE, chained(h, 8),
                                     false, reps % CHAIN_CYCLE, omega, g, SC_R64));
        q.bytes += g.bytes;
        return hipSuccess;
    }
    if (kind >= 2) return enqueue_pcg_step(h, kind == 3, nu_pre, nu_post, omega, q);
    if (nu_pre == 2 && nu_post == 2) {
        if (kind == 0)
            return enqueue_vcycle_fused<double>(h, h->L, F.x64, F.b64, false, omega, q,
                                                h->partials, h->scal, SC_R64, h->host_scal);
        return enqueue_vcycle_fused<float>(h, h->L, F.x32, F.b32, x_zero, omega, q, h->partials,
                                           h->scal, SC_R32, h->host_scal);
    }
    if (kind == 0) {
        MG_TRY(enqueue_vcycle<double>(h, h->L, F.x64, F.b64, false, nu_pre, nu_post, omega, q));
        MG_TRY(launch_defect<double>(F, F.bands64, F.b64, F.x64, nullptr, h->partials, h->scal,
                                     SC_R64, h->host_scal, q.st));
        q.bytes += 11 * 8 * n;
    } else {
        MG_TRY(enqueue_vcycle<float>(h, h->L, F.x32, F.b32, x_zero, nu_pre, nu_post, omega, q));
        MG_TRY(launch_defect<float>(F, F.bands32, F.b32, F.x32, nullptr, h->partials, h->scal,
                                    SC_R32, h->host_scal, q.st));
        q.bytes += 11 * 4 * n;
    }
    return hipSuccess;
}

static GraphCache* cache(mg_hierarchy* h) {
    if (!h->graphs) h->graphs = new GraphCache();
    return h->graphs;
}

void destroy_graphs(mg_hierarchy* h) {
    if (!h->graphs) return;
    for (auto& e : h->graphs->entries) (void)hipGraphExecDestroy(e.exec);
    if (h->graphs->ev_in) (void)hipEventDestroy(h->graphs->ev_in);
    if (h->graphs->ev_out) (void)hipEventDestroy(h->graphs->ev_out);
    if (h->graphs->st) (void)hipStreamDestroy(h->graphs->st);
    delete h->graphs;
    h->graphs = nullptr;
}

// Run one unit, from a captured graph when allowed.
static hipError_t run_unit(mg_hierarchy* h, int kind, const mg_solve_opts& o, bool x_zero,
                           bool use_graph, Enq& q, int reps = 1) {
    GraphCache* gc = cache(h);
    if (use_graph && gc->capture_ok) {
        const uint64_t epoch = tile_table_epoch();
        for (size_t i = 0; i < gc->entries.size(); ++i) {
            GraphEntry& e = gc->entries[i];
            if (e.kind == kind && e.reps == reps && e.nu_pre == o.nu_pre &&
                e.nu_post == o.nu_post && e.omega == o.omega && e.x_zero == x_zero) {
                if (e.epoch == epoch) {
                    q.bytes += e.bytes;
                    return hipGraphLaunch(e.exec, q.st);
                }
                // tiles changed since the capture: wait for earlier replays,
                // then capture again below
                MG_TRY(hipStreamSynchronize(q.st));
                (void)hipGraphExecDestroy(e.exec);
                gc->entries.erase(gc->entries.begin() + i);
                break;
            }
        }
        Enq cq{q.st, 0.0};
        hipError_t e = hipStreamBeginCapture(q.st, hipStreamCaptureModeThreadLocal);
        if (e == hipSuccess) {
            hipError_t ee = enqueue_unit(h, kind, reps, o.nu_pre, o.nu_post, o.omega, x_zero, cq);
            hipGraph_t g = nullptr;
            e = hipStreamEndCapture(q.st, &g);
            if (ee != hipSuccess) e = ee;
            hipGraphExec_t ex = nullptr;
            if (e == hipSuccess) e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
            if (g) (void)hipGraphDestroy(g);
            if (e == hipSuccess) {
                gc->entries.push_back(
                    {kind, reps, o.nu_pre, o.nu_post, o.omega, x_zero, ex, cq.bytes, epoch});
                q.bytes += cq.bytes;
                return hipGraphLaunch(ex, q.st);
            }
        }
        (void)hipGetLastError();
        gc->capture_ok = false;  // fall back to direct launches for this hierarchy
    }
    return enqueue_unit(h, kind, reps, o.nu_pre, o.nu_post, o.omega, x_zero, q);
}

// Host read-back of reduced norms.  Every reduction the drivers read writes
// its result straight into the hierarchy's pinned mirror (no copy).  Before
// the producing work is enqueued the host arms the slot with a value no
// norm takes; it then spins on the mirror, which returns as soon as the
// final reduction kernel has stored the norm, without the wake-up latency
// of a blocking stream synchronisation.  After 50 ms of spinning it falls
// back to synchronising the stream (which also reports device errors).
constexpr double kArmed = -1.0;

static void arm_scalar(mg_hierarchy* h, int slot) {
    ((volatile double*)h->host_scal)[slot + 1] = kArmed;
}

static hipError_t read_scalar(mg_hierarchy* h, int slot, hipStream_t st, double* out) {
    const TraceRange trace("host waits for a norm");
    const volatile double* v = (const volatile double*)h->host_scal + slot + 1;
    const auto t0 = std::chrono::steady_clock::now();
    for (unsigned i = 1;; ++i) {
        const double x = *v;
        if (!(x == kArmed)) {
            *out = x;
            return hipSuccess;
        }
        if ((i & 4095u) == 0 &&
            std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(50))
            break;
    }
    MG_TRY(hipStreamSynchronize(st));
    *out = *v;
    return hipSuccess;
}

// The inner-loop state red_control mirrors (cycles run, plus ITER_DONE once
// the loop is over): wait until the loop is over or has run `want` cycles.
static void arm_iter(mg_hierarchy* h) { ((volatile double*)h->host_scal)[SC_ITER] = kArmed; }

static hipError_t read_iter(mg_hierarchy* h, int want, hipStream_t st, int* cycles, bool* done) {
    const TraceRange trace("host waits for the inner loop");
    const volatile double* v = (const volatile double*)h->host_scal + SC_ITER;
    const auto t0 = std::chrono::steady_clock::now();
    double x = kArmed;
    for (unsigned i = 1;; ++i) {
        x = *v;
        if (!(x == kArmed) && (x >= ITER_DONE || x == (double)want)) break;
        if ((i & 4095u) == 0 &&
            std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(50)) {
            MG_TRY(hipStreamSynchronize(st));
            x = *v;
            break;
        }
    }
    *done = x >= ITER_DONE;
    *cycles = (int)(*done ? x - ITER_DONE : x);
    return hipSuccess;
}

}  // namespace mg

using namespace mg;

#define MG_HIPS(call)                                                                         \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess) {                                                               \
            st.status = MG_ERR_DEVICE;                                                        \
            if (stats) *stats = st;                                                           \
            return fail(MG_ERR_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_));   \
        }                                                                                     \
    } while (0)

static mg_status validate_opts(const mg_solve_opts& o) {
    if (o.nu_pre < 0 || o.nu_post < 0 || o.nu_pre + o.nu_post == 0 || o.nu_pre > 16 ||
        o.nu_post > 16)
        return fail(MG_ERR_INVALID, "smoothing steps must be in [0,16] and not both 0");
    if (!(o.omega > 0.0 && o.omega < 2.0)) return fail(MG_ERR_INVALID, "omega must lie in (0,2)");
    if (!(o.rel_tol >= 0.0) || o.max_cycles < 1)
        return fail(MG_ERR_INVALID, "rel_tol must be >= 0 and max_cycles >= 1");
    if (o.precision != MG_PREC_FP64 && o.precision != MG_PREC_MIXED)
        return fail(MG_ERR_INVALID, "unknown precision");
    if (o.precision == MG_PREC_MIXED &&
        (!(o.inner_reduction >= 0.0 && o.inner_reduction < 1.0) || o.inner_max_cycles < 1))
        return fail(MG_ERR_INVALID, "inner_reduction in [0,1) and inner_max_cycles >= 1 required");
    if (o.fixed_cycles < 0) return fail(MG_ERR_INVALID, "fixed_cycles must be >= 0");
    if (o.krylov != 0 && o.krylov != 1) return fail(MG_ERR_INVALID, "krylov must be 0 or 1");
    if (o.zero_guess != 0 && o.zero_guess != 1)
        return fail(MG_ERR_INVALID, "zero_guess must be 0 or 1");
    return MG_OK;
}

extern "C" mg_status mg_vcycle(mg_hierarchy* h, int level, mg_dtype dtype, const void* b,
                               void* x, int nu_pre, int nu_post, double omega, int fused,
                               void* stream) {
    if (!h) return fail(MG_ERR_INVALID, "null hierarchy");
    if (level < h->Lc || level > h->L) return fail(MG_ERR_INVALID, "level out of range");
    if (!h->assembled) return fail(MG_ERR_INVALID, "hierarchy not assembled");
    if (!b || !x || ((uintptr_t)b & 15) || ((uintptr_t)x & 15) || b == x)
        return fail(MG_ERR_INVALID, "b, x must be distinct 16-byte aligned device pointers");
    if (nu_pre < 0 || nu_post < 0 || nu_pre > 16 || nu_post > 16)
        return fail(MG_ERR_INVALID, "smoothing steps out of range");
    MG_HIP(hipSetDevice(h->ctx->device));
    Enq q{(hipStream_t)stream, 0.0};
    if (fused && (nu_pre != 2 || nu_post != 2))
        return fail(MG_ERR_INVALID, "the fused cycle is V(2,2)");
    if (fused && dtype == MG_F64)
        MG_HIP(enqueue_vcycle_fused<double>(h, level, (double*)x, (const double*)b, false, omega, q,
                                            nullptr, nullptr, 0, nullptr));
    else if (fused)
        MG_HIP(enqueue_vcycle_fused<float>(h, level, (float*)x, (const float*)b, false, omega, q,
                                           nullptr, nullptr, 0, nullptr));
    else if (dtype == MG_F64)
        MG_HIP(enqueue_vcycle<double>(h, level, (double*)x, (const double*)b, false, nu_pre,
                                      nu_post, omega, q));
    else
        MG_HIP(enqueue_vcycle<float>(h, level, (float*)x, (const float*)b, false, nu_pre, nu_post,
                                     omega, q));
    return MG_OK;
}

extern "C" mg_status mg_solve(mg_hierarchy* h, const double* dev_b, double* dev_x,
                              const mg_solve_opts* opts, void* stream, mg_stats* stats) {
    const TraceRange trace("mg_solve");
    const auto t0 = std::chrono::steady_clock::now();
    mg_stats st{};
    if (stats) *stats = st;
    if (!h) return fail(MG_ERR_INVALID, "null hierarchy");
    if (!h->assembled) return fail(MG_ERR_INVALID, "hierarchy not assembled");
    if (!dev_b || !dev_x || dev_b == dev_x || ((uintptr_t)dev_b & 15) || ((uintptr_t)dev_x & 15))
        return fail(MG_ERR_INVALID, "b, x must be distinct 16-byte aligned device pointers");
    mg_solve_opts o;
    if (opts)
        o = *opts;
    else
        mg_default_opts(&o);
    if (mg_status s = validate_opts(o)) return s;
    MG_HIP(hipSetDevice(h->ctx->device));
    GraphCache* gc = cache(h);
    if (!gc->st) MG_HIP(hipStreamCreateWithFlags(&gc->st, hipStreamNonBlocking));
    if (!gc->ev_in) MG_HIP(hipEventCreateWithFlags(&gc->ev_in, hipEventDisableTiming));
    if (!gc->ev_out) MG_HIP(hipEventCreateWithFlags(&gc->ev_out, hipEventDisableTiming));
    // The internal stream waits (on the device) for the caller's producers
    // of b and x.
    MG_HIPS(hipEventRecord(gc->ev_in, (hipStream_t)stream));
    MG_HIPS(hipStreamWaitEvent(gc->st, gc->ev_in, 0));
    Enq q{gc->st, 0.0};
    Level& F = h->lv[h->L];
    const int64_t n = F.n;
    const bool graphs = o.use_graph != 0;
    // The mixed-precision loop touches the FP64 vectors only in directly
    // launched kernels (defect, update), so it reads the caller's b and
    // updates the caller's x in place; the other solvers' captured graphs
    // work on the hierarchy's own copies.
    const bool direct = !o.krylov && o.precision == MG_PREC_MIXED;
    // (The preconditioned CG reads b only there too: its own b64 holds p.)
    const double* B64 = direct || o.krylov ? dev_b : F.b64;
    double* X64 = direct ? dev_x : F.x64;
    // zero_guess: x0 = 0 whatever dev_x holds (not read; the mixed solve's
    // first update writes x without reading it)
    const bool zg = o.zero_guess != 0;
    if (!direct) {
        if (!o.krylov) MG_HIPS(launch_copy<double>(dev_b, F.b64, n, q.st));
        if (zg)
            MG_HIPS(launch_fill<double>(F.x64, n, 0.0, q.st));
        else
            MG_HIPS(launch_copy<double>(dev_x, F.x64, n, q.st));
        q.bytes += ((zg ? 8.0 : 16.0) + (o.krylov ? 0.0 : 16.0)) * n;
    }
    // the mixed solve under device control (see the last branch below)
    const bool devctl = !o.krylov && o.precision == MG_PREC_MIXED && o.nu_pre == 2 &&
                        o.nu_post == 2 && h->L > tail_max_level() &&
                        o.inner_max_cycles < (int)ITER_DONE;
    auto nslot = [](int k) { return (k & 1) ? SC_R64 : SC_R64B; };
    auto outer_ctl = [&](int k) {
        RedCtl c;
        c.mode = RED_OUTER;
        c.thr = o.fixed_cycles > 0 ? -1.0 : o.rel_tol;
        c.div = 1e3;
        c.cap = (o.fixed_cycles > 0 ? k > o.fixed_cycles : k > o.max_cycles) ? 1 : 0;
        c.reset = 1;  // a step that goes on starts its inner loop
        c.ithr = o.inner_reduction;
        c.icap = o.inner_max_cycles;
        return c;
    };
    const double* wait = h->scal + SC_WAIT;
    // the update of step k and the defect of step k + 1
    auto queue_update_defect = [&](int k) -> hipError_t {
        MG_TRY(launch_update(X64, F.x32, n, h->scal, q.st, wait, zg && k == 1));
        arm_scalar(h, nslot(k + 1));
        return launch_defect_cast(F, F.bands64, B64, X64, F.b32, h->partials, h->scal,
                                  nslot(k + 1), h->host_scal, q.st, wait, outer_ctl(k + 1));
    };
    int last = 0;      // cycles of the previous inner loop of this solve
    int pred = 0;      // cycles queued at once for the latest queued step
    double cycle_bytes = 0.0;
    // the predicted cycles, the update and the next defect of step k (the
    // defect of step k wrote the FP32 right-hand side and started the loop)
    auto queue_step = [&](int k) -> hipError_t {
        const int slot = std::min(k, 8) - 1;
        pred = h->inner_pred[slot] > 0 ? h->inner_pred[slot] : (last > 0 ? last : 2);
        pred = std::min(pred, o.inner_max_cycles);
        arm_iter(h);
        Enq cq{q.st, 0.0};
        MG_TRY(run_unit(h, 4, o, true, graphs, cq, pred));
        cycle_bytes = cq.bytes / pred;
        MG_TRY(queue_update_defect(k));
        return hipSuccess;
    };
    auto ahead = [&](int k) { return h->outer_prev <= 0 || k <= h->outer_prev; };
    bool queued = false;  // outer step k already queued
    arm_scalar(h, SC_B);
    MG_HIPS(launch_norm<double>(B64, n, h->partials, h->scal, SC_B, h->host_scal, q.st));
    q.bytes += 8.0 * n;
    // A zero initial iterate (the usual start) makes the first defect b
    // itself: its kernel then reads b alone (same bits, see
    // launch_defect_zero_x).
    if (!zg) {
        arm_scalar(h, SC_XNZ);
        RedCtl zflag;
        zflag.mode = devctl ? RED_ZFLAG : RED_NONE;
        MG_HIPS(launch_count_nonzero(X64, n, h->partials, h->scal, SC_XNZ, h->host_scal, q.st,
                                     zflag));
        q.bytes += 8.0 * n;
    }
    if (devctl) {
        // the first defect (of the zero or the given iterate: the other
        // kernel returns at once) and, with a zero guess, step 1, before ||b||
        // reaches the host; the device's tests read ||b|| from its own copy
        arm_scalar(h, nslot(1));
        MG_HIPS(launch_defect_zero_x_cast(F, B64, F.b32, h->partials, h->scal, nslot(1),
                                          h->host_scal, q.st,
                                          zg ? nullptr : h->scal + SC_XNZ, outer_ctl(1)));
        if (!zg)
            MG_HIPS(launch_defect_cast(F, F.bands64, B64, X64, F.b32, h->partials, h->scal,
                                       nslot(1), h->host_scal, q.st, h->scal + SC_XZ,
                                       outer_ctl(1)));
        queued = zg && ahead(1);
        if (queued) MG_HIPS(queue_step(1));
    }
    double bn = 0.0, xnz = 0.0;
    MG_HIPS(read_scalar(h, SC_B, q.st, &bn));
    if (!zg) MG_HIPS(read_scalar(h, SC_XNZ, q.st, &xnz));
    const bool x_zero = xnz == 0.0;
    // A given iterate may be the solution already, and the cycles of a step
    // that is not taken are launches all the same (such a call: L = 9 143 -> 105
    // us, L = 11 241 -> 148): step 1 waits for the first defect's norm unless the
    // iterate turns out zero, which the host knows while that defect runs.
    if (devctl && !zg && x_zero && std::isfinite(bn) && bn != 0.0) {
        queued = ahead(1);
        if (queued) MG_HIPS(queue_step(1));
    }
    st.bnorm = bn;
    mg_status result = MG_OK;
    if (!std::isfinite(bn)) {
        result = fail(MG_ERR_NUMERIC, "right-hand side contains NaN or Inf");
    } else if (bn == 0.0) {
        MG_HIPS(launch_fill<double>(X64, n, 0.0, q.st));
    } else if (o.krylov) {
        // r0 = b - A x0 and its norm; the first direction is z (beta = 0)
        double r = 0.0;
        arm_scalar(h, SC_RR);
        if (x_zero) {
            MG_HIPS(launch_defect_zero_x(F, B64, h->d64, h->partials, h->scal, SC_RR,
                                         h->host_scal, q.st));
            q.bytes += 16.0 * n;
        } else {
            MG_HIPS(launch_defect<double>(F, F.bands64, B64, F.x64, h->d64, h->partials,
                                          h->scal, SC_RR, h->host_scal, q.st));
            q.bytes += 12.0 * 8 * n;
        }
        MG_HIPS(launch_fill<double>(h->scal + SC_RZ, 1, INFINITY, q.st));
        MG_HIPS(read_scalar(h, SC_RR, q.st, &r));
        st.rel_res = r / bn;
        const int kind = o.precision == MG_PREC_FP64 ? 2 : 3;
        for (int k = 1;; ++k) {
            if (o.fixed_cycles > 0) {
                if (k > o.fixed_cycles) break;
            } else {
                if (r <= o.rel_tol * bn) break;
                if (k > o.max_cycles) {
                    result = fail(MG_ERR_NOCONV, "no convergence within max_cycles");
                    break;
                }
            }
            arm_scalar(h, SC_RR);
            MG_HIPS(run_unit(h, kind, o, false, graphs, q));
            MG_HIPS(read_scalar(h, SC_RR, q.st, &r));
            st.cycles = k;
            if (st.n_hist < MG_HIST) st.res_hist[st.n_hist++] = r / bn;
            if (!std::isfinite(r) || r > 1e3 * bn) {
                result = fail(MG_ERR_NUMERIC, "residual diverged or became NaN");
                break;
            }
        }
        // the true residual at exit, from the caller's b (the copy holds p)
        double rt = 0.0;
        arm_scalar(h, SC_R64);
        MG_HIPS(launch_defect<double>(F, F.bands64, dev_b, F.x64, nullptr, h->partials, h->scal,
                                      SC_R64, h->host_scal, q.st));
        q.bytes += 11.0 * 8 * n;
        MG_HIPS(read_scalar(h, SC_R64, q.st, &rt));
        st.rel_res = rt / bn;
    } else if (o.precision == MG_PREC_FP64) {
        // V(2,2) cycles run under device control: the reduction that yields a
        // cycle's norm takes the tests below (RED_CYCLE), and cycles queued
        // behind the last one return at once.  So several cycles go out in one
        // graph before the host has read a norm, in powers of two up to 8, so
        // that few graphs are captured.  A graph per cycle leaves some 4 us
        // between cycles, whether or not the host waits for the norm between
        // them (solves of 9 cycles: L = 6 331 -> 303 us, L = 8 475 -> 435, L = 10
        // 918 -> 885).  A cycle too many costs more, about eight launches that
        // do nothing (10 us at L = 6, 40 at L = 9, 60 at L = 12): as many go out
        // as the first residual needs at the rate of the faster of the last two
        // solves, rounded up (or fixed_cycles).  From a zero iterate that
        // residual is b; any other one is read first, as the iterate may be the
        // solution already (with as many cycles as earlier solves took queued
        // behind it, such a call took 452 us at L = 9, now 109).  The first solve of
        // a hierarchy, and cycles past the prediction, go out one by one.
        const bool guarded = o.nu_pre == 2 && o.nu_post == 2 && h->L > h->Lc;
        const bool chain = guarded && chained(h, 8);
        const int cap = o.fixed_cycles > 0 ? o.fixed_cycles : o.max_cycles;
        double r = 0.0, cycle_cost = 0.0;
        RedCtl first;
        if (guarded) {
            first.mode = RED_START;
            first.thr = o.fixed_cycles > 0 ? -1.0 : o.rel_tol;
            first.icap = cap;
        }
        // its own slot: a queued cycle's norm must not overtake it
        arm_scalar(h, SC_R64B);
        if (x_zero) {
            MG_HIPS(launch_defect_zero_x(F, F.b64, nullptr, h->partials, h->scal, SC_R64B,
                                         h->host_scal, q.st, nullptr, first));
            q.bytes += 8.0 * n;
        } else {
            MG_HIPS(launch_defect<double>(F, F.bands64, F.b64, F.x64, nullptr, h->partials,
                                          h->scal, SC_R64B, h->host_scal, q.st, nullptr, first));
            q.bytes += 11.0 * 8 * n;
        }
        auto ring = [](int k) { return SC_HIST + k % HIST_RING - 1; };
        const double rate = std::max(h->rate_prev[0], h->rate_prev[1]);
        auto cycles_for = [&](double r0) -> int {
            if (o.fixed_cycles > 0) return h->fp64_solved ? cap : 0;
            if (!(rate > 0.0)) return 0;
            const double need = std::log(r0 / (o.rel_tol * bn)) / rate;
            return need > 0.0 ? (int)std::min((double)cap, std::ceil(need)) : 0;
        };
        int sent = 0;  // cycles queued
        auto queue_to = [&](int k) -> hipError_t {
            while (sent < k) {
                int m = 8;
                while (m > k - sent) m /= 2;
                const int c = sent + 1;
                int part = CHAIN_ENTER | CHAIN_LEAVE;
                if (chain)
                    part = (c == 1 ? CHAIN_ENTER : 0) | (sent + m == cap ? CHAIN_LEAVE : 0) |
                           (c % 2 == 0 ? CHAIN_ODD : 0);
                for (int i = 0; i < m; ++i) arm_scalar(h, ring(c + i));
                Enq cq{q.st, 0.0};
                MG_TRY(run_unit(h, 5, o, false, graphs, cq, part + m * CHAIN_CYCLE));
                cycle_cost = cq.bytes / m;
                sent += m;
            }
            return hipSuccess;
        };
        // the cycles to have been queued before the norm of cycle k is read: the
        // norms in flight stay within half the mirror's ring
        const bool known = x_zero || o.fixed_cycles > 0;
        int ahead = guarded && known ? cycles_for(bn) : 0;
        auto horizon = [&](int k) {
            return sent >= k ? sent : std::max(k, std::min(ahead, k + HIST_RING / 2 - 1));
        };
        if (ahead > 0) MG_HIPS(queue_to(horizon(1)));
        MG_HIPS(read_scalar(h, SC_R64B, q.st, &r));
        st.rel_res = r / bn;
        const double r0 = r;
        if (guarded && !known) ahead = cycles_for(r0);
        for (int k = 1;; ++k) {
            if (o.fixed_cycles > 0) {
                if (k > o.fixed_cycles) break;
            } else {
                if (r <= o.rel_tol * bn) break;
                if (k > o.max_cycles) {
                    result = fail(MG_ERR_NOCONV, "no convergence within max_cycles");
                    break;
                }
            }
            if (guarded) {
                MG_HIPS(queue_to(horizon(k)));
                MG_HIPS(read_scalar(h, ring(k), q.st, &r));
                q.bytes += cycle_cost;
            } else {
                arm_scalar(h, SC_R64);
                MG_HIPS(run_unit(h, 0, o, false, graphs, q));
                MG_HIPS(read_scalar(h, SC_R64, q.st, &r));
            }
            st.cycles = k;
            st.rel_res = r / bn;
            if (st.n_hist < MG_HIST) st.res_hist[st.n_hist++] = r / bn;
            if (!std::isfinite(r) || r > 1e3 * bn) {
                result = fail(MG_ERR_NUMERIC, "residual diverged or became NaN");
                break;
            }
        }
        if (guarded && result == MG_OK && st.cycles > 0) {
            h->fp64_solved = true;
            const double rate_now = std::log(r0 / r) / st.cycles;
            if (o.fixed_cycles == 0 && std::isfinite(rate_now)) {
                h->rate_prev[1] = h->rate_prev[0];
                h->rate_prev[0] = rate_now;
            }
        }
    } else if (!devctl) {
        // host-driven loop: one host read per FP64 defect and per FP32 cycle
        for (int k = 1;; ++k) {
            const TraceRange step("mixed outer step");
            double s = 0.0;
            arm_scalar(h, SC_R64);
            if (k == 1 && x_zero) {
                MG_HIPS(launch_defect_zero_x_cast(F, B64, F.b32, h->partials, h->scal, SC_R64,
                                                  h->host_scal, q.st));
                q.bytes += 12.0 * n;
            } else {
                MG_HIPS(launch_defect_cast(F, F.bands64, B64, X64, F.b32, h->partials, h->scal,
                                           SC_R64, h->host_scal, q.st));
                q.bytes += 92.0 * n;
            }
            MG_HIPS(read_scalar(h, SC_R64, q.st, &s));
            st.rel_res = s / bn;
            if (k > 1 && st.n_hist < MG_HIST) st.res_hist[st.n_hist++] = s / bn;
            if (!std::isfinite(s) || s > 1e3 * bn) {
                result = fail(MG_ERR_NUMERIC, "residual diverged or became NaN");
                break;
            }
            if (o.fixed_cycles > 0) {
                if (k > o.fixed_cycles) break;
            } else {
                if (s <= o.rel_tol * bn) break;
                if (k > o.max_cycles) {
                    result = fail(MG_ERR_NOCONV, "no convergence within max_cycles");
                    break;
                }
            }
            if (s == 0.0) break;
            // the FP32 right-hand side is the defect scaled by a power of
            // two: its loop stops relative to the scaled defect's norm
            const double dn = dev::pow2_scale(bn) * s;
            for (int it = 1; it <= o.inner_max_cycles; ++it) {
                double r32 = 0.0;
                arm_scalar(h, SC_R32);
                MG_HIPS(run_unit(h, 1, o, it == 1, graphs, q));
                MG_HIPS(read_scalar(h, SC_R32, q.st, &r32));
                st.cycles++;
                if (!std::isfinite(r32)) break;
                if (r32 <= o.inner_reduction * dn) break;
            }
            MG_HIPS(launch_update(X64, F.x32, n, h->scal, q.st, nullptr, zg && k == 1));
            q.bytes += 20.0 * n;
            st.outer_steps = k;
        }
    } else {
        // Device control (fused V(2,2) cycle): the decisions of the loop
        // above, taken on the device by the reductions that produce the
        // norms they test (RedCtl), with everything that follows a decision
        // queued behind it under a guard.  The FP64 defect of outer step k
        // writes the FP32 right-hand side, and its norm's reduction starts
        // the inner loop unless the solve is over.  After it the host
        // queues the FP32 cycles step k took in
        // the previous solve (each returning at once after the loop is
        // over), the update and the defect of step k + 1, which wait on the
        // device for the loop's end -- before reading the defect's norm when
        // the previous solve also took step k (then the device does not wait
        // for the host between outer steps), after it otherwise (a converged
        // solve leaves no skipped cycles behind).  The host reads the
        // defect's norm (its tests are the device's), then the loop's state;
        // if the loop needs more cycles than were queued, it queues single
        // cycles and then the update and the next defect.  Same kernels,
        // same decisions, same bits as the loop above.  Outer steps
        // alternate between two norm slots, so queueing step k + 1 never
        // overwrites a norm the host has yet to read.
        q.bytes += x_zero ? 12.0 * n : 92.0 * n;  // the first defect
        for (int k = 1;; ++k) {
            const TraceRange step("mixed outer step");
            double s = 0.0;
            MG_HIPS(read_scalar(h, nslot(k), q.st, &s));
            st.rel_res = s / bn;
            if (k > 1 && st.n_hist < MG_HIST) st.res_hist[st.n_hist++] = s / bn;
            if (!std::isfinite(s) || s > 1e3 * bn) {
                result = fail(MG_ERR_NUMERIC, "residual diverged or became NaN");
                break;
            }
            if (o.fixed_cycles > 0) {
                if (k > o.fixed_cycles) break;
            } else {
                if (s <= o.rel_tol * bn) break;
                if (k > o.max_cycles) {
                    result = fail(MG_ERR_NOCONV, "no convergence within max_cycles");
                    break;
                }
            }
            if (s == 0.0) break;
            if (!queued) MG_HIPS(queue_step(k));
            const int slot = std::min(k, 8) - 1;
            int cycles = 0;
            bool done = false;
            MG_HIPS(read_iter(h, pred, q.st, &cycles, &done));
            if (!done) {
                // the queued update and defect were skipped: more cycles, then those
                while (!done) {
                    arm_iter(h);
                    Enq c1{q.st, 0.0};
                    MG_HIPS(run_unit(h, 4, o, false, graphs, c1, 1));
                    MG_HIPS(read_iter(h, cycles + 1, q.st, &cycles, &done));
                }
                MG_HIPS(queue_update_defect(k));
            }
            q.bytes += cycle_bytes * cycles + 20.0 * n + 92.0 * n;
            st.cycles += cycles;
            h->inner_pred[slot] = cycles;
            last = cycles;
            st.outer_steps = k;
            queued = ahead(k + 1);
            if (queued) MG_HIPS(queue_step(k + 1));
        }
        if (result == MG_OK) h->outer_prev = st.outer_steps;
    }
    if (!direct) {
        MG_HIPS(launch_copy<double>(F.x64, dev_x, n, q.st));
        q.bytes += 16.0 * n;
    } else if (zg && st.outer_steps == 0 && bn != 0.0) {
        // no update wrote the caller's x: the result is the zero guess
        MG_HIPS(launch_fill<double>(X64, n, 0.0, q.st));
        q.bytes += 8.0 * n;
    }
    // Later work on the caller's stream runs after the solve's.  The mixed
    // solve's last write of x came before the defect whose norm the host
    // has read, so only the others wait here for their final copy.
    MG_HIPS(hipEventRecord(gc->ev_out, q.st));
    MG_HIPS(hipStreamWaitEvent((hipStream_t)stream, gc->ev_out, 0));
    if (!direct || result != MG_OK || bn == 0.0) MG_HIPS(hipStreamSynchronize(q.st));
    st.status = result;
    st.alg_bytes = q.bytes;
    st.seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (stats) *stats = st;
    return result;
}

// ---------------------------------------------------------------- tiles
namespace mg {
// The post- and pre-smoothing pass of level l as a solve runs them, on h's own
// work vectors (which no solve reads before writing).
template <typename T>
static hipError_t tile_pair(mg_hierarchy* h, int l, hipStream_t st) {
    Level &v = h->lv[l], &c = h->lv[l - 1];
    const bool finest = l == h->L;
    const T om = T(0.7);
    MG_TRY(launch_pre<T>(v, LV<T>::bands(v), LV<T>::x(v), !finest, LV<T>::b(v), om, LV<T>::t(v),
                         LV<T>::b(c), h->dmask, st));
    return launch_post<T>(v, LV<T>::bands(v), LV<T>::t(v), LV<T>::x(c), LV<T>::b(v), om,
                          LV<T>::x(v), finest ? h->partials : nullptr, h->scal, SC_USER, nullptr,
                          st);
}
}  // namespace mg

// Sec. 3: the thread-block partition of the GPU kernels is a runtime
// parameter.  For every level on which the hierarchy's V(2,2) cycle runs
// fused passes, time the FP32 pre- and post-smoothing passes (as the mixed
// solve runs them: the finest level's pre pass from a given iterate and its
// post pass with the residual norm, the others from zero and without) for
// each candidate tile and keep the fastest in the tile table under one
// problem where it beats the rule.
extern "C" mg_status mg_hierarchy_autotune(mg_hierarchy* h, int reps, mg_tile_choice* out,
                                           int out_cap, int* n_out) {
    if (n_out) *n_out = 0;
    if (!h) return fail(MG_ERR_INVALID, "null hierarchy");
    if (!h->assembled) return fail(MG_ERR_INVALID, "hierarchy not assembled");
    if (reps < 1 || reps > 1000) return fail(MG_ERR_INVALID, "reps must lie in [1, 1000]");
    if (out_cap < 0 || (out_cap > 0 && !out)) return fail(MG_ERR_INVALID, "bad output array");
    const TraceRange trace("mg_hierarchy_autotune");
    static const int kRows[] = {4, 8, 12, 16, 24, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256};
    static const int kWidths[] = {64, 128, 192, 256};
    MG_HIP(hipSetDevice(h->ctx->device));
    GraphCache* gc = cache(h);
    if (!gc->st) MG_HIP(hipStreamCreateWithFlags(&gc->st, hipStreamNonBlocking));
    hipStream_t st = gc->st;
    struct Guard {
        hipEvent_t a = nullptr, b = nullptr;
        ~Guard() {
            set_single_trial(0, 0, 0);
            if (a) (void)hipEventDestroy(a);
            if (b) (void)hipEventDestroy(b);
        }
    } g;
    MG_HIP(hipEventCreate(&g.a));
    MG_HIP(hipEventCreate(&g.b));
    std::vector<mg_tile_choice> rows;
    for (int l = h->L; l > h->Lc; --l) {
        if (!(l > tail_max_level() || l == h->L)) continue;
        const int N = h->lv[l].N;
        // reps pairs of passes with a tile, in ms
        auto time_pairs = [&](const std::array<int, 3>& c, bool fp64, float* ms) -> hipError_t {
            auto pair = [&] { return fp64 ? tile_pair<double>(h, l, st) : tile_pair<float>(h, l, st); };
            set_single_trial(N, c[1], c[0], c[2]);
            for (int w = 0; w < 2; ++w) MG_TRY(pair());
            MG_TRY(hipEventRecord(g.a, st));
            for (int r = 0; r < reps; ++r) MG_TRY(pair());
            MG_TRY(hipEventRecord(g.b, st));
            MG_TRY(hipEventSynchronize(g.b));
            return hipEventElapsedTime(ms, g.a, g.b);
        };
        // marching tiles (width x rows), then block tiles on small levels
        std::vector<std::array<int, 3>> cand;
        for (int bt : kWidths)
            for (int rh : kRows) cand.push_back({bt, rh, 0});
        if (N <= dev::BLK_MAX_N)
            for (int s = 1; s <= dev::BLK_SHAPES; ++s)
                cand.push_back({64 * dev::BLK_TAG_WAVES, dev::block_rows(s), dev::BLK_TAG});
        std::array<int, 3> best{};
        float best_ms = 0.0f;
        for (const auto& c : cand) {
            float ms = 0.0f;
            MG_HIP(time_pairs(c, false, &ms));
            if (best_ms == 0.0f || ms < best_ms) {
                best = c;
                best_ms = ms;
            }
        }
        // An entry replaces the rule in both types, and the rule's tiles differ by
        // type (FP32 L = 10 and 11, L = 12: 16 rows, block tiles, another march).
        // It is stored only if, timed in turn with the rule, it is faster in FP32
        // and not slower in FP64: stored regardless, FP64 passes went 30.5 -> 33.5
        // us at L = 10 and 461 -> 473 at L = 12, the FP64 solve 5281 -> 5383.
        bool keep = true, same = true;
        for (const bool fp64 : {false, true}) {
            const dev::FusedGeom r = single_rule(N, fp64 ? 8 : 4);
            const std::array<int, 3> rule =
                r.blk ? std::array<int, 3>{64 * dev::BLK_TAG_WAVES, r.rh, dev::BLK_TAG}
                      : std::array<int, 3>{r.bt, r.rh, 0};
            if (rule == best) continue;
            same = false;
            float mine = 0.0f, ruled = 0.0f;
            for (int turn = 0; turn < 3; ++turn) {
                float a = 0.0f, b = 0.0f;
                MG_HIP(time_pairs(rule, fp64, &a));
                MG_HIP(time_pairs(best, fp64, &b));
                ruled += a;
                mine += b;
            }
            if (mine > ruled) keep = false;
        }
        keep = keep && !same;
        set_single_trial(0, 0, 0);
        if (keep)
            tile_table_set(l, 1, best[1], best[0], best[2]);
        else
            tile_table_erase(l, 1);
        const double us = 1e3 * best_ms / reps;
        rows.push_back({l, 1, best[1], best[0] / 64, best[2], keep ? us : -us});
    }
    const int n = std::min<int>(out_cap, (int)rows.size());
    for (int i = 0; i < n; ++i) out[i] = rows[i];
    if (n_out) *n_out = (int)rows.size();
    return MG_OK;
}
