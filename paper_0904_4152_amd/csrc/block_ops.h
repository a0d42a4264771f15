// Block tiles of the fused smoothing passes, for levels on which a marching
// tile (fused_ops.h) is bound by its chain of row steps and not by bytes.
//
// A tile owns BLK_OWN columns by 4 (W - 2) rows; its workgroup of W wavefronts
// covers the tile and a halo of 4 rows and columns on every side, lane l of
// wavefront w owning the nodes of column l in rows 4 w .. 4 w + 3 of the region.
// Bands, right-hand side and iterate of a thread's four nodes stay in
// registers: the five stored upper bands are loaded once, the lower ones are
// the neighbours' upper ones (the row above in the same thread, the column to
// the left or right one lane away).  A band product takes the left and right
// neighbours' values of the iterate from the adjacent lanes and the rows
// above and below from the thread itself; only a wavefront's first and last
// row go through LDS, with one barrier per step.  So a pass costs one memory
// latency and a few short steps, and LDS carries four values per thread and
// step (with the region's bands and iterates in LDS a product read 18 values
// per node, and L = 9 was LDS-bound).
//
// The steps, the per-node arithmetic and the layout and summation order of
// the norm partials are those of pre_tile and post_tile: same bits.  (Nodes of
// the region that no owned result depends on hold unspecified values; nodes
// outside the grid hold zeros.)
#pragma once

#include "fused_ops.h"

namespace mg {
namespace dev {

// Value of the lane to the left / right (0 beyond the wavefront).
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                         0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <typename T>
__device__ __forceinline__ T from_left(T v) {
    return lane_shift<0x138>(v);  // wave_shr:1
}
template <typename T>
__device__ __forceinline__ T from_right(T v) {
    return lane_shift<0x130>(v);  // wave_shl:1
}

// Guarded passes (*guard not zero: do nothing).  A test before the loads puts a
// memory latency of its own in front of theirs, 0.6 to 0.8 us in a pass of 3 to 5
// us.  So on levels of up to BLK_GUARD_N nodes per side the guard is read among
// the other loads and withholds the stores (a skipped pass then runs its 4 us);
// larger levels, whose passes are longer, test first.
constexpr int BLK_GUARD_N = 513;
static __device__ double zero_guard;  // stands for no guard (a select, not a branch around the load)
__device__ __forceinline__ bool pass_over(const double* guard, int N) {
    return N > BLK_GUARD_N && guard && *(const volatile double*)guard != 0.0;
}

// LDS of a block pass: the wavefronts' first and last rows, two steps of them
// in turn (so one barrier per step separates writers and readers), and with
// the norm each column's sum over a wavefront's four rows.
template <typename T, int W>
struct BlockLds {
    T edge[2][W][2][64];
    double ns[W][64];
};

// H: halo rows and columns on every side, a multiple of four (whole wavefronts).
template <typename T, int W, int H = F_HALO>
struct BlockTile {
    static constexpr int OWN = 64 - 2 * H;          // owned columns
    static constexpr int ROWS = 4 * W - 2 * H;      // owned rows
    static constexpr int W0 = H / 4, W1 = W - W0;   // wavefronts of owned rows
    BlockLds<T, W>& s;
    const int N, lane, w;
    int col, row0;      // this thread's column and first row
    int r0, r1, c0, c1; // owned rows and columns
    int turn = 0;       // edge buffer of the next exchange
    T bk[4][9], b[4];
    bool in[4];         // node inside the grid
    bool go = true;     // not a skipped pass
    bool own;           // this lane's column owned, and not a skipped pass

    __device__ BlockTile(BlockLds<T, W>& s_, int N_, int strip, int chunk)
        : s(s_), N(N_), lane((int)threadIdx.x & 63),
          w(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) {
        c0 = strip * OWN;
        c1 = min(c0 + OWN, N);
        r0 = chunk * ROWS;
        r1 = min(r0 + ROWS, N);
        col = c0 - H + lane;
        own = in_range(col, c0, c1);
        row0 = r0 - H + 4 * w;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            in[r] = in_range(col, 0, N) && in_range(row0 + r, 0, N);
    }
    // Store nothing if the pass is to be skipped.
    __device__ __forceinline__ void heed(const double* guard) {
        if (__builtin_constant_p(guard) && !guard) return;
        go = !(*(guard ? guard : &zero_guard) != 0.0);
        own &= go;
    }
    __device__ __forceinline__ uint32_t off(int r) const {
        return in[r] ? node_off(row0 + r, N, col, sizeof(T)) : OFF_NONE;
    }
    // Every load of the bands and b, then the lower bands.
    __device__ __forceinline__ void load(const T* bands, int64_t bs, const T* bb) {
        const int64_t n = (int64_t)N * N;
        const RowRsrc<T> R(bands, bs, bb, n);
        T up[3];  // bands 6, 7, 8 of the row above
        const bool uin = in_range(col, 0, N) && in_range(row0 - 1, 0, N);
        const uint32_t uo = uin ? node_off(row0 - 1, N, col, sizeof(T)) : OFF_NONE;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t o = off(r);
#pragma unroll
            for (int k = 4; k < 9; ++k) bk[r][k] = bload<T>(R.band[k], o);
            b[r] = bload<T>(R.b, o);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) up[k] = bload<T>(R.band[6 + k], uo);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            bk[r][0] = from_left(r ? bk[r - 1][8] : up[2]);
            bk[r][1] = r ? bk[r - 1][7] : up[1];
            bk[r][2] = from_right(r ? bk[r - 1][6] : up[0]);
            bk[r][3] = from_left(bk[r][5]);
        }
    }
    // The rows of v above and below this wavefront's.
    __device__ __forceinline__ void exchange(const T (&v)[4], T& up, T& dn) {
        s.edge[turn][w][0][lane] = v[0];
        s.edge[turn][w][1][lane] = v[3];
        __syncthreads();
        up = s.edge[turn][w > 0 ? w - 1 : 0][1][lane];
        dn = s.edge[turn][w < W - 1 ? w + 1 : w][0][lane];
        turn ^= 1;
    }
    // Band products of the own nodes: the fma chain of stencil_tile.
    __device__ __forceinline__ void product(const T (&v)[4], T (&acc)[4]) {
        T c[6], l[6], r[6];
        exchange(v, c[0], c[5]);
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i + 1] = v[i];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            l[i] = from_left(c[i]);
            r[i] = from_right(c[i]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            T a = T(0);
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const int i = q + k / 3;
                a = fma(bk[q][k], k % 3 == 0 ? l[i] : k % 3 == 1 ? c[i] : r[i], a);
            }
            acc[q] = a;
        }
    }
    // One damped Jacobi sweep in place.
    __device__ __forceinline__ void sweep(T (&v)[4], T omega) {
        T acc[4];
        product(v, acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const T x = v[r] + jacobi_div(omega * (b[r] - acc[r]), bk[r][4]);
            v[r] = in[r] ? x : T(0);
        }
    }
    __device__ __forceinline__ void store(T* out, const T (&v)[4]) const {
        if (!own || w < W0 || w >= W1) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (in[r]) out[(int64_t)(row0 + r) * N + col] = v[r];
    }
    // v = x + P x_c (the arithmetic of prolong_elem), with every load of the
    // tile.
    __device__ __forceinline__ void start(const T* bands, int64_t bs, const T* x, const T* xc,
                                          const T* bb, T (&v)[4]) {
        const int Nc = (N >> 1) + 1;
        T k0[3], k1[3];
        const rsrc_t Rx = make_rsrc(x, (int64_t)N * N * (int64_t)sizeof(T));
        const rsrc_t Rc = make_rsrc(xc, (int64_t)Nc * Nc * (int64_t)sizeof(T));
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = bload<T>(Rx, off(r));
        // the coarse values around rows row0 .. row0 + 3 (row0 is even)
        const int I = col >> 1, J = row0 >> 1;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const bool ok = in_range(J + q, 0, Nc);
            const uint32_t o = (uint32_t)((J + q) * Nc + I) * (uint32_t)sizeof(T);
            k0[q] = bload<T>(Rc, ok && in_range(I, 0, Nc) ? o : OFF_NONE);
            k1[q] = bload<T>(Rc, ok && in_range(I + 1, 0, Nc) ? o + (uint32_t)sizeof(T) : OFF_NONE);
        }
        load(bands, bs, bb);
        const bool c_even = !(col & 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int q = r >> 1;
            T p;
            if (r & 1)
                p = c_even ? T(0.5) * (k0[q] + k0[q + 1])
                           : T(0.25) * ((k0[q] + k1[q]) + (k0[q + 1] + k1[q + 1]));
            else
                p = c_even ? k0[q] : T(0.5) * (k0[q] + k1[q]);
            v[r] = in[r] ? v[r] + p : T(0);
        }
    }
    // The defect of v, restricted to the owned coarse nodes (row0 and c0 are
    // even, as every node there).
    __device__ __forceinline__ void restrict_defect(const T (&v)[4], T* bc, int dmask) {
        T d[4], up, dn;
        product(v, d);
#pragma unroll
        for (int r = 0; r < 4; ++r) d[r] = in[r] ? b[r] - d[r] : T(0);
        exchange(d, up, dn);
        const int Nc = (N >> 1) + 1;
        const T row[5] = {up, d[0], d[1], d[2], d[3]};
        T l[5], r[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            l[i] = from_left(row[i]);
            r[i] = from_right(row[i]);
        }
        if ((lane & 1) || !own || w < W0 || w >= W1) return;
#pragma unroll
        for (int i = 1; i < 5; i += 2) {
            const int j = row0 + i - 1;
            if (j < r1) {
                const T corner = (l[i - 1] + r[i - 1]) + (l[i + 1] + r[i + 1]);
                const T edge = (row[i - 1] + row[i + 1]) + (l[i] + r[i]);
                const T res = row[i] + T(0.5) * edge + T(0.25) * corner;
                const int I = col >> 1, J = j >> 1;
                bc[(int64_t)J * Nc + I] = is_dirichlet(Nc, I, J, dmask) ? T(0) : res;
            }
        }
    }
    // The norm partials of the residual e on owned nodes: each column's sum
    // over the wavefront's rows (one group of F_NORM_ROWS), rows in increasing
    // order, then the segments' eight column sums.
    __device__ __forceinline__ void norm_partials(const T (&e)[4], double* rowpart) {
        static_assert(F_NORM_ROWS == 4 && OWN % F_NORM_COLS == 0 && ROWS % F_NORM_ROWS == 0,
                      "a wavefront's rows are one group");
        if (w < W0 || w >= W1) return;
        double acc2 = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (row0 + r < r1) acc2 += own ? (double)e[r] * (double)e[r] : 0.0;
        s.ns[w][lane] = acc2;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int nseg = (N + F_NORM_COLS - 1) / F_NORM_COLS, m = lane;
        if (go && m < OWN / F_NORM_COLS && c0 + m * F_NORM_COLS < c1 && row0 < r1) {
            const double* n = s.ns[w] + H + m * F_NORM_COLS;
            const double s8 = ((n[0] + n[1]) + (n[2] + n[3])) + ((n[4] + n[5]) + (n[6] + n[7]));
            rowpart[(int64_t)(row0 / F_NORM_ROWS) * nseg + c0 / F_NORM_COLS + m] = s8;
        }
    }
};

// Pre-smoothing block: NU sweeps (the first from a zero iterate with XZERO),
// the defect and its restriction, as pre_tile for the same owned nodes.
template <typename T, bool XZERO, int W, int NU>
__device__ __forceinline__ void pre_block(BlockLds<T, W>& s, const T* __restrict__ bands,
                                          int64_t bs, int N, const T* __restrict__ x,
                                          const T* __restrict__ b, T omega, T* __restrict__ x2out,
                                          T* __restrict__ bc, int dmask, int strip, int chunk,
                                          const double* __restrict__ guard = nullptr) {
    static_assert(NU + 2 <= F_HALO, "halo of the sweeps, the defect and the restriction");
    BlockTile<T, W> t(s, N, strip, chunk);
    t.heed(guard);
    T v[4];
    if (!XZERO) {
        const rsrc_t Rx = make_rsrc(x, (int64_t)N * N * (int64_t)sizeof(T));
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = bload<T>(Rx, t.off(r));
    }
    t.load(bands, bs, b);
    if (XZERO) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const T x1 = jacobi_div(omega * t.b[r], t.bk[r][4]);
            v[r] = t.in[r] ? x1 : T(0);
        }
    }
#pragma unroll
    for (int k = XZERO ? 1 : 0; k < NU; ++k) t.sweep(v, omega);
    t.store(x2out, v);
    t.restrict_defect(v, bc, dmask);
}

// Post-smoothing block: x + P x_c, NU sweeps and with NORM the sums of squares
// of the defect, as post_tile for the same owned nodes.
template <typename T, bool NORM, int W, int NU>
__device__ __forceinline__ void post_block(BlockLds<T, W>& s, const T* __restrict__ bands,
                                           int64_t bs, int N, const T* __restrict__ x,
                                           const T* __restrict__ xc, const T* __restrict__ b,
                                           T omega, T* __restrict__ xout,
                                           double* __restrict__ rowpart, int strip, int chunk,
                                           const double* __restrict__ guard = nullptr) {
    static_assert(NU + 1 <= F_HALO, "halo of the sweeps and the norm");
    BlockTile<T, W> t(s, N, strip, chunk);
    t.heed(guard);
    T v[4];
    t.start(bands, bs, x, xc, b, v);
#pragma unroll
    for (int k = 0; k < NU; ++k) t.sweep(v, omega);
    t.store(xout, v);
    if (!NORM) return;
    T d[4];
    t.product(v, d);
#pragma unroll
    for (int r = 0; r < 4; ++r) d[r] = t.b[r] - d[r];
    t.norm_partials(d, rowpart);
}

// Halo of a merged block pass: six steps, in whole wavefronts of rows, and in
// columns as many (whole norm segments owned).
constexpr int BLK_MID_HALO = 8;
static_assert((64 - 2 * BLK_MID_HALO) % F_NORM_COLS == 0, "");

// Merged pass (see mid_ops.h) in a block tile: post_block with the norm and
// pre_block of the next cycle, the third sweep from the product of the norm.
template <typename T, int W>
__device__ __forceinline__ void mid_block(BlockLds<T, W>& s, const T* __restrict__ bands,
                                          int64_t bs, int N, const T* __restrict__ x,
                                          const T* __restrict__ xc, const T* __restrict__ b,
                                          T omega, T* __restrict__ xpost, T* __restrict__ x2,
                                          T* __restrict__ bc, int dmask,
                                          double* __restrict__ rowpart, int strip, int chunk,
                                          const double* __restrict__ guard) {
    BlockTile<T, W, BLK_MID_HALO> t(s, N, strip, chunk);
    t.heed(guard);
    T v[4], e[4];
    t.start(bands, bs, x, xc, b, v);
    t.sweep(v, omega);
    t.sweep(v, omega);
    t.store(xpost, v);
    t.product(v, e);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        e[r] = t.b[r] - e[r];
        const T x3 = v[r] + jacobi_div(omega * e[r], t.bk[r][4]);
        v[r] = t.in[r] ? x3 : T(0);
    }
    t.norm_partials(e, rowpart);
    t.sweep(v, omega);
    t.store(x2, v);
    t.restrict_defect(v, bc, dmask);
}

}  // namespace dev
}  // namespace mg
