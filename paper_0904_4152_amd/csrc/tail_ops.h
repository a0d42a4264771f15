// Coarse end of the V-cycle: the coarsest solve by one wavefront, and the
// coarse tail, the sub-cycle over levels of at most 33 x 33 nodes in one
// workgroup.
//
// Both are bound by the latency of a chain of dependent steps, not by bytes
// or operations (60 KB of FP32 bands, 5 k nodes visited per cycle), so the
// layout serves the length of that chain:
//   - a thread keeps the bands, the right-hand side and the iterate of its
//     own nodes in registers (loaded once, every load in flight at once); only
//     the iterate that neighbours read goes through LDS, so a band product
//     reads nine LDS values per node or fewer and no band;
//   - on the 33 x 33 level a thread owns three nodes of a column, whose nine
//     products share five rows (15 LDS reads instead of 27, three independent
//     fma chains), so the level needs six wavefronts and not seventeen;
//   - levels of 9 x 9 nodes and below, and the coarsest solve, run in
//     wavefront 0 alone: LDS operations of one wavefront are executed in
//     order, so no barrier stands between their steps;
//   - the first sweep of a level (from a zero iterate, pointwise) is taken by
//     the thread that restricts the node's right-hand side, in that step;
//   - level sizes are compile-time constants (no run-time division).
// Per-node arithmetic and order are those of the separate kernels: same bits.
// Measured per launch in the solves (levels 5..1, V(2,2), MI355X kernel trace): FP32 8.4 us,
// FP64 10.1 us, FP32 with a CG coarse grid of level 2 13.1 us; one 1024-thread
// workgroup with every band in LDS and a barrier per step took 19.8, 21.0 and
// 33.8 us.
#pragma once

#include "device_ops.h"

namespace mg {
namespace dev {

constexpr int TAIL_MAX = 5;
// 33 columns x 11 groups of three rows, in whole wavefronts
constexpr int TAIL_THREADS = 384;

// Orders this wavefront's LDS accesses before and after it (they execute in
// order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- coarsest
// LDS of a coarse solve: the matrix (CG: nine bands, Cholesky: the factor's
// band up to level 3; at level 4 the factor's 44 KB stay in global memory),
// and a vector with N + 1 zeros on either side.
struct CoarseLds {
    double mat[9 * COARSE_MAX_UNKNOWNS];
    double v[COARSE_MAX_UNKNOWNS + 2 * (COARSE_MAX_N + 1)];
};

// The matrix into LDS, by threads tid = 0 .. threads - 1; the caller's barrier
// (or wave_sync for one wavefront) stands before its use.
template <int LEVEL>
__device__ __forceinline__ void coarse_stage_level(const CoarseSolver& cs, CoarseLds& w, int tid,
                                                   int threads) {
    constexpr int N = (1 << LEVEL) + 1, n = N * N;
    if (cs.cg) {
        for (int p = tid; p < n; p += threads) {
            double r[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) r[k] = cs.bands[k * cs.bs + p];
#pragma unroll
            for (int k = 0; k < 9; ++k) w.mat[k * n + p] = r[k];
        }
        for (int e = tid; e < N + 1; e += threads) w.v[e] = w.v[N + 1 + n + e] = 0.0;
    } else if (LEVEL < COARSE_MAX_LEVEL) {
        // rows of the factor's band: columns r - bw .. r, bw = N + 1
        // (unknowns in node order: nothing lies further off the diagonal)
        for (int e = tid; e < cs.m * (N + 2); e += threads) {
            const int r = e / (N + 2), k = r - (N + 1) + e % (N + 2);
            w.mat[e] = k >= 0 ? cs.chol[r * cs.m + k] : 0.0;
        }
    }
}
__device__ __forceinline__ void coarse_stage(const CoarseSolver& cs, int Lc, CoarseLds& w,
                                             int tid, int threads) {
    switch (Lc) {
        case 1: coarse_stage_level<1>(cs, w, tid, threads); break;
        case 2: coarse_stage_level<2>(cs, w, tid, threads); break;
        case 3: coarse_stage_level<3>(cs, w, tid, threads); break;
        default: coarse_stage_level<4>(cs, w, tid, threads); break;
    }
}

// Forward and back substitution with the banded factor, L(r, k) = f[r ld + k],
// by one wavefront; x in place of b (Dirichlet rows are identity rows).
// Forward: once z[k] is known the lanes subtract its terms from the rows
// below, so each row's terms go off in increasing k as in a row sweep; back:
// every lane carries the same row sum.
template <typename T, int LEVEL, typename F>
__device__ __forceinline__ void coarse_cholesky(const CoarseSolver& cs, T* __restrict__ a,
                                                double* __restrict__ z, F f, int ld) {
    constexpr int N = (1 << LEVEL) + 1, n = N * N, bw = N + 1;
    const int lane = (int)(threadIdx.x & 63);
    const int m = cs.m;
    // the unknowns are a rectangle of nodes, numbered in node order
    const int i0 = cs.dmask & 1, j0 = (cs.dmask >> 2) & 1;
    const int wd = N - i0 - ((cs.dmask >> 1) & 1);
    auto unknown = [&](int p) { return (p / N - j0) * wd + p % N - i0; };
    if (m == 1) {  // the usual level 1: one unknown, two divisions
        const double d = f[0];
        if (lane == 0) a[j0 * N + i0] = (T)((double)a[j0 * N + i0] / d / d);
        wave_sync();
        return;
    }
#pragma unroll
    for (int p = lane; p < n; p += 64)
        if (!is_dirichlet(N, p % N, p / N, cs.dmask)) z[unknown(p)] = (double)a[p];
    wave_sync();
    for (int k = 0; k < m; ++k) {
        const double zk = z[k] / f[k * ld + k];
        const int r = k + 1 + lane;
        if (lane < bw && r < m) z[r] = fma(-f[r * ld + k], zk, z[r]);
        if (lane == 63) z[k] = zk;
        wave_sync();
    }
    for (int r = m - 1; r >= 0; --r) {
        double s = z[r];
        const int hi = min(m, r + bw + 1);
        for (int k = r + 1; k < hi; ++k) s = fma(-f[k * ld + r], z[k], s);
        s = s / f[r * ld + r];
        wave_sync();
        if (lane == 0) z[r] = s;
        wave_sync();
    }
#pragma unroll
    for (int p = lane; p < n; p += 64)
        if (!is_dirichlet(N, p % N, p / N, cs.dmask)) a[p] = (T)z[unknown(p)];
    wave_sync();
}

// u . v over a lane's S nodes in index order, then the fixed butterfly over
// the lanes (every lane gets the total).
template <int S>
__device__ __forceinline__ double cg_dot(const double (&u)[S], const double (&v)[S], int n) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < S; ++k)
        if ((int)(threadIdx.x & 63) + 64 * k < n) s = fma(u[k], v[k], s);
    return wave_sum(s);
}

// Unpreconditioned conjugate gradients (Hestenes and Stiefel) on the
// coarsest level from a zero iterate, in FP64: q = A p, alpha = (r.r)/(p.q),
// x += alpha p, r -= alpha q, beta = (r'.r')/(r.r), p = r' + beta p; stops
// before a step once ||r|| <= tol ||b|| or after max_iter steps.  Dirichlet
// rows keep their zero start (identity rows, zero right-hand side).  One
// wavefront; lane l owns the nodes l, l + 64, ... (S of them), x in place of b.
template <typename T, int LEVEL>
__device__ __forceinline__ void coarse_cg(const CoarseSolver& cs, T* __restrict__ a,
                                          CoarseLds& w) {
    constexpr int N = (1 << LEVEL) + 1, n = N * N, S = (n + 63) / 64;
    const int lane = (int)(threadIdx.x & 63);
    double* const p = w.v + N + 1;
    double xs[S], r[S], q[S], pv[S];
#pragma unroll
    for (int k = 0; k < S; ++k) {
        const int i = lane + 64 * k;
        const double bi = i < n ? (double)a[i] : 0.0;
        xs[k] = 0.0;
        r[k] = pv[k] = bi;
        q[k] = 0.0;
        if (i < n) p[i] = bi;
    }
    wave_sync();
    double rr = cg_dot<S>(r, r, n);
    const double stop = cs.tol * sqrt(rr);
    for (int step = 0; step < cs.max_iter && sqrt(rr) > stop; ++step) {
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const int i = lane + 64 * k;
            // at 17 x 17 nodes the bands stay in LDS, read node by node (kept
            // in registers they spill)
            if (S > 2) asm volatile("" ::: "memory");
            if (i < n) {
                double acc = 0.0;
#pragma unroll
                for (int kb = 0; kb < 9; ++kb)
                    acc = fma(w.mat[kb * n + i], p[i + (kb / 3 - 1) * N + (kb % 3 - 1)], acc);
                q[k] = acc;
            }
        }
        wave_sync();
        const double alpha = rr / cg_dot<S>(pv, q, n);
#pragma unroll
        for (int k = 0; k < S; ++k) {
            xs[k] = fma(alpha, pv[k], xs[k]);
            r[k] = fma(-alpha, q[k], r[k]);
        }
        const double rr_new = cg_dot<S>(r, r, n);
        const double beta = rr_new / rr;
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const int i = lane + 64 * k;
            pv[k] = fma(beta, pv[k], r[k]);
            if (i < n) p[i] = pv[k];
        }
        wave_sync();
        rr = rr_new;
    }
#pragma unroll
    for (int k = 0; k < S; ++k) {
        const int i = lane + 64 * k;
        if (i < n) a[i] = (T)xs[k];
    }
    wave_sync();
}

template <typename T, int LEVEL>
__device__ __forceinline__ void coarse_level(const CoarseSolver& cs, T* __restrict__ a,
                                             CoarseLds& w) {
    constexpr int N = (1 << LEVEL) + 1;
    if (cs.cg)
        coarse_cg<T, LEVEL>(cs, a, w);
    else if (LEVEL < COARSE_MAX_LEVEL)
        coarse_cholesky<T, LEVEL>(cs, a, w.v, w.mat + (N + 1), N + 1);
    else
        coarse_cholesky<T, LEVEL>(cs, a, w.v, cs.chol, cs.m);
}

// The coarsest solve by the configured method, by one wavefront, in place on
// the LDS vector a (the matrix staged before by coarse_stage).
template <typename T>
__device__ __forceinline__ void coarse_wave(const CoarseSolver& cs, int Lc, T* __restrict__ a,
                                            CoarseLds& w) {
    switch (Lc) {
        case 1: coarse_level<T, 1>(cs, a, w); break;
        case 2: coarse_level<T, 2>(cs, a, w); break;
        case 3: coarse_level<T, 3>(cs, a, w); break;
        default: coarse_level<T, 4>(cs, a, w); break;
    }
}

// x = A^-1 b on the coarsest level (N nodes per side), global vectors, one
// workgroup of any size; wavefront 0 works.
template <typename T>
__device__ __forceinline__ void coarse_block(const CoarseSolver& cs, int N, const T* b, T* x) {
    __shared__ CoarseLds w;
    __shared__ T a[COARSE_MAX_UNKNOWNS];
    const int Lc = 31 - __clz(N - 1);
    __syncthreads();  // a previous item of this workgroup is done with LDS
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        coarse_stage(cs, Lc, w, lane, 64);
        for (int p = lane; p < N * N; p += 64) a[p] = b[p];
        wave_sync();
        coarse_wave<T>(cs, Lc, a, w);
        for (int p = lane; p < N * N; p += 64) x[p] = a[p];
    }
    __syncthreads();
}

// ---------------------------------------------------------------- tail

template <typename T>
struct TailLevel {
    const T* bands;
    T* x;
    T* b;
    int64_t bs;
};

template <typename T>
struct TailLevels {
    TailLevel<T> lv[TAIL_MAX + 1];  // index = level
    CoarseSolver cs;                // coarsest solve; cs.dmask: the Dirichlet sides
    int top;  // highest level of the tail; entered with a zero iterate
    int Lc;
    int nu_pre, nu_post;
};

// LDS of level l: two work vectors, each with N + 1 zeros on either side
// (they stand for the neighbours outside the grid, whose bands are zero).
__host__ __device__ constexpr int tail_vec(int l) {
    return ((1 << l) + 1) * ((1 << l) + 1) + 2 * ((1 << l) + 2);
}
__host__ __device__ constexpr int tail_off(int l) {
    int e = 0;
    for (int m = 1; m < l; ++m) e += 2 * tail_vec(m);
    return e;
}

template <typename T>
struct TailLds {
    alignas(16) T v[(tail_off(TAIL_MAX + 1) + 3) / 4 * 4];
    CoarseLds cs;
    int stop;
};

// The nodes of level l a thread owns, with their bands, right-hand side and
// iterate.  Level 5: three rows of a column; level 4: one node; levels 3..1:
// wavefront 0, nodes lane, lane + 64.
template <typename T, int l>
struct TailNodes {
    static constexpr int N = (1 << l) + 1, n = N * N;
    static constexpr int S = l == 5 ? 3 : l == 3 ? 2 : 1;
    T bk[S][9], b[S], x[S];

    static __device__ __forceinline__ int node(int s) {
        const int t = (int)threadIdx.x;
        return l == 5 ? (3 * (t / N) + s) * N + t % N : t + 64 * s;
    }
    static __device__ __forceinline__ bool own(int s) {
        const int t = (int)threadIdx.x;
        return l == 5 ? t < N * (N / 3) : t + 64 * s < n;
    }
    // vector 0 or 1 of the level
    static __device__ __forceinline__ T* vec(T* lds, int which) {
        return lds + tail_off(l) + which * tail_vec(l) + N + 1;
    }
    static __device__ __forceinline__ void sync() {
        if (l >= 4)
            __syncthreads();
        else
            wave_sync();
    }

    __device__ __forceinline__ void load(const TailLevel<T>& g, bool bands, bool rhs) {
        // the first sweep needs the diagonal and b alone: they go out first
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const unsigned p = own(s) ? node(s) : 0;
            if (bands) bk[s][4] = (g.bands + 4 * g.bs)[p];
            if (rhs) b[s] = g.b[p];
        }
        if (!bands) return;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const unsigned p = own(s) ? node(s) : 0;
#pragma unroll
            for (int k = 0; k < 9; ++k)
                if (k != 4) bk[s][k] = (g.bands + k * g.bs)[p];
        }
    }
    // b = P^T d (weights 1, 1/2, 1/4; zero on the Dirichlet sides), d the
    // finer level's defect in LDS
    __device__ __forceinline__ void restrict_from(T* lds, int which, int dmask) {
        constexpr int Nf = 2 * N - 1;
        const T* d = TailNodes<T, l + 1>::vec(lds, which);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int p = own(s) ? node(s) : 0;
            const int I = p % N, J = p / N;
            const T* c = d + 2 * J * Nf + 2 * I;
            const bool lo = I > 0, hi = I < N - 1;
            auto at = [&](int di, int dj) -> T {
                const T v = c[dj * Nf + di];
                return (di < 0 && !lo) || (di > 0 && !hi) ? T(0) : v;
            };
            const T corner = (at(-1, -1) + at(1, -1)) + (at(-1, 1) + at(1, 1));
            const T edge = (at(0, -1) + at(0, 1)) + (at(-1, 0) + at(1, 0));
            const T r = at(0, 0) + T(0.5) * edge + T(0.25) * corner;
            b[s] = is_dirichlet(N, I, J, dmask) ? T(0) : r;
        }
    }
    // band products of the own nodes with an LDS vector
    __device__ __forceinline__ void product(const T* v, T (&acc)[S]) const {
        if (l == 5) {
            const T* c = v + (own(0) ? node(0) : 0);
            T r[S + 2][3];
#pragma unroll
            for (int i = 0; i < S + 2; ++i)
#pragma unroll
                for (int e = 0; e < 3; ++e) r[i][e] = c[(i - 1) * N + e - 1];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                acc[s] = T(0);
#pragma unroll
                for (int k = 0; k < 9; ++k) acc[s] = fma(bk[s][k], r[s + k / 3][k % 3], acc[s]);
            }
        } else {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const T* c = v + (own(s) ? node(s) : 0);
                acc[s] = T(0);
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    acc[s] = fma(bk[s][k], c[(k / 3 - 1) * N + (k % 3 - 1)], acc[s]);
            }
        }
    }
    __device__ __forceinline__ void put(T* v, const T (&r)[S]) const {
#pragma unroll
        for (int s = 0; s < S; ++s)
            if (own(s)) v[node(s)] = r[s];
    }
    // one damped Jacobi sweep of x (in vector `at` of LDS) into the other
    // vector; at = the vector that then holds x
    __device__ __forceinline__ void sweep(T* lds, int& at, T omega) {
        T acc[S];
        product(vec(lds, at), acc);
#pragma unroll
        for (int s = 0; s < S; ++s) x[s] = x[s] + jacobi_div(omega * (b[s] - acc[s]), bk[s][4]);
        at ^= 1;
        put(vec(lds, at), x);
        sync();
    }
    // pre-smoothing from a zero iterate and the defect, which ends up in the
    // vector returned
    __device__ __forceinline__ int down(T* lds, T omega, int nu) {
        int at = 0;
#pragma unroll
        for (int s = 0; s < S; ++s)
            x[s] = nu > 0 ? jacobi_div(omega * b[s], bk[s][4]) : T(0);
        put(vec(lds, 0), x);
        sync();
        for (int k = 1; k < nu; ++k) sweep(lds, at, omega);
        T acc[S];
        product(vec(lds, at), acc);
#pragma unroll
        for (int s = 0; s < S; ++s) acc[s] = b[s] - acc[s];
        at ^= 1;
        put(vec(lds, at), acc);
        sync();
        return at;
    }
    // x + P x_c and post-smoothing; cat: the vector of the coarser level
    // holding x_c.  The last sweep's values stay in x; they go to LDS too
    // unless the level is the tail's last (out: its global iterate).
    __device__ __forceinline__ int up(T* lds, int cat, T omega, int nu, T* out) {
        constexpr int Nc = (N >> 1) + 1;
        const T* xc = TailNodes<T, l - 1>::vec(lds, cat);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int p = own(s) ? node(s) : 0;
            const int i = p % N, j = p / N;
            const T* c = xc + (j >> 1) * Nc + (i >> 1);
            const T k0 = c[0], k1 = c[1], k2 = c[Nc], k3 = c[Nc + 1];
            const T row = (i & 1) ? T(0.5) * (k0 + k1) : k0;
            const T odd = (i & 1) ? T(0.25) * ((k0 + k1) + (k2 + k3)) : T(0.5) * (k0 + k2);
            x[s] += (j & 1) ? odd : row;
        }
        int at = 0;
        put(vec(lds, 0), x);
        sync();
        for (int k = 0; k < nu; ++k) {
            if (out && k == nu - 1) {
                T acc[S];
                product(vec(lds, at), acc);
#pragma unroll
                for (int s = 0; s < S; ++s)
                    x[s] = x[s] + jacobi_div(omega * (b[s] - acc[s]), bk[s][4]);
            } else {
                sweep(lds, at, omega);
            }
        }
        if (out) put(out, x);
        return at;
    }
};

// The V(nu_pre, nu_post) sub-cycle from a zero iterate over levels top..Lc
// of one problem, one workgroup of TAIL_THREADS threads: x_top = V(b_top).
// NU > 0: both smoothing counts are NU (tl's are not read).  A guard that is not
// null and not zero ends the cycle before it writes: one thread reads it while
// the loads are out, and every wavefront takes that thread's word (a guard that
// changes meanwhile must not split the workgroup).
template <typename T, int NU>
__device__ void tail_cycle(TailLds<T>& m, const TailLevels<T>& tl, T omega,
                           const double* __restrict__ guard = nullptr) {
    if (guard && threadIdx.x == 0) m.stop = *guard != 0.0;
    const int top = tl.top, Lc = tl.Lc, dmask = tl.cs.dmask;
    const int pre = NU > 0 ? NU : tl.nu_pre, post = NU > 0 ? NU : tl.nu_post;
    const bool wave0 = threadIdx.x < 64;
    TailNodes<T, 5> n5;
    TailNodes<T, 4> n4;
    TailNodes<T, 3> n3;
    TailNodes<T, 2> n2;
    TailNodes<T, 1> n1;
    // every load of the cycle, in the order of use
    if (top >= 5) n5.load(tl.lv[5], true, true);
    if (top >= 4) n4.load(tl.lv[4], Lc < 4, top == 4);
    if (wave0) {
        if (top >= 3 && Lc <= 3) n3.load(tl.lv[3], Lc < 3, top == 3);
        if (top >= 2 && Lc <= 2) n2.load(tl.lv[2], Lc < 2, top == 2);
        if (Lc == 1 && top == 1) n1.load(tl.lv[1], false, true);
    }
    {
        constexpr int VE = 16 / (int)sizeof(T), NV = (tail_off(TAIL_MAX + 1) + VE - 1) / VE;
        const typename V16<T>::type zero = {};
        for (int e = threadIdx.x; e < NV; e += TAIL_THREADS)
            reinterpret_cast<typename V16<T>::type*>(m.v)[e] = zero;
    }
    __syncthreads();
    if (guard && m.stop) return;
    T* const lds = m.v;
    int at = 0;  // vector of the level just finished: a defect, or an iterate
    if (top >= 5) at = n5.down(lds, omega, pre);
    if (top >= 4) {
        if (top > 4) n4.restrict_from(lds, at, dmask);
        if (Lc < 4) {
            at = n4.down(lds, omega, pre);
        } else {
            n4.put(n4.vec(lds, 0), n4.b);
            __syncthreads();
        }
    }
    if (wave0) {
        if (Lc <= 3 && top >= 3) {
            if (top > 3) n3.restrict_from(lds, at, dmask);
            if (Lc < 3) {
                at = n3.down(lds, omega, pre);
            } else {
                n3.put(n3.vec(lds, 0), n3.b);
                wave_sync();
            }
        }
        if (Lc <= 2 && top >= 2) {
            if (top > 2) n2.restrict_from(lds, at, dmask);
            if (Lc < 2) {
                at = n2.down(lds, omega, pre);
            } else {
                n2.put(n2.vec(lds, 0), n2.b);
                wave_sync();
            }
        }
        if (Lc == 1) {
            if (top > 1) n1.restrict_from(lds, at, dmask);
            n1.put(n1.vec(lds, 0), n1.b);
        }
    } else {
        // meanwhile the other wavefronts fetch the coarsest level's matrix
        coarse_stage(tl.cs, Lc, m.cs, (int)threadIdx.x - 64, TAIL_THREADS - 64);
    }
    __syncthreads();
    if (wave0) {
        T* const ac = Lc == 1 ? n1.vec(lds, 0) : Lc == 2 ? n2.vec(lds, 0)
                    : Lc == 3 ? n3.vec(lds, 0) : n4.vec(lds, 0);
        coarse_wave<T>(tl.cs, Lc, ac, m.cs);
        if (top == Lc) {
            const int n = ((1 << Lc) + 1) * ((1 << Lc) + 1);
            for (int p = threadIdx.x; p < n; p += 64) tl.lv[top].x[p] = ac[p];
        }
        at = 0;  // the coarsest solve's vector
        if (Lc < 2 && top >= 2) at = n2.up(lds, at, omega, post, top == 2 ? tl.lv[2].x : nullptr);
        if (Lc < 3 && top >= 3) at = n3.up(lds, at, omega, post, top == 3 ? tl.lv[3].x : nullptr);
    }
    if (top < 4) return;
    __syncthreads();
    at = Lc < 3 ? post & 1 : 0;  // where wavefront 0 left level 3 (or the coarsest level)
    if (Lc < 4) at = n4.up(lds, at, omega, post, top == 4 ? tl.lv[4].x : nullptr);
    if (top >= 5) n5.up(lds, at, omega, post, tl.lv[5].x);
}

}  // namespace dev
}  // namespace mg
