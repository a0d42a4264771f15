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

// LDS of a block pass: the wavefronts' first and last rows, two steps of them
// in turn (so one barrier per step separates writers and readers), and with
// the norm each column's sum over a wavefront's four rows.
template <typename T, int W>
struct BlockLds {
    T edge[2][W][2][64];
    double ns[W][64];
};

template <typename T, int W>
struct BlockTile {
    BlockLds<T, W>& s;
    const int N, lane, w;
    int col, row0;      // this thread's column and first row
    int r0, r1, c0, c1; // owned rows and columns
    int turn = 0;       // edge buffer of the next exchange
    T bk[4][9], b[4];
    bool in[4];         // node inside the grid

    __device__ BlockTile(BlockLds<T, W>& s_, int N_, int strip, int chunk)
        : s(s_), N(N_), lane((int)threadIdx.x & 63),
          w(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) {
        constexpr int BR = 4 * (W - 2);
        c0 = strip * BLK_OWN;
        c1 = min(c0 + BLK_OWN, N);
        r0 = chunk * BR;
        r1 = min(r0 + BR, N);
        col = c0 - F_HALO + lane;
        row0 = r0 - F_HALO + 4 * w;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            in[r] = in_range(col, 0, N) && in_range(row0 + r, 0, N);
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
        if (!in_range(col, c0, c1) || w == 0 || w == W - 1) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (in[r]) out[(int64_t)(row0 + r) * N + col] = v[r];
    }
};

// Pre-smoothing block: NU sweeps (the first from a zero iterate with XZERO),
// the defect and its restriction, as pre_tile for the same owned nodes.
template <typename T, bool XZERO, int W, int NU>
__device__ __forceinline__ void pre_block(BlockLds<T, W>& s, const T* __restrict__ bands,
                                          int64_t bs, int N, const T* __restrict__ x,
                                          const T* __restrict__ b, T omega, T* __restrict__ x2out,
                                          T* __restrict__ bc, int dmask, int strip, int chunk) {
    static_assert(NU + 2 <= F_HALO, "halo of the sweeps, the defect and the restriction");
    BlockTile<T, W> t(s, N, strip, chunk);
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
    T d[4];
    t.product(v, d);
#pragma unroll
    for (int r = 0; r < 4; ++r) d[r] = t.in[r] ? t.b[r] - d[r] : T(0);
    // restriction at the even rows and columns (row0 and c0 are even)
    T up, dn;
    t.exchange(d, up, dn);
    const int Nc = (N >> 1) + 1;
    const T row[5] = {up, d[0], d[1], d[2], d[3]};
    T l[5], r[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        l[i] = from_left(row[i]);
        r[i] = from_right(row[i]);
    }
    if ((t.lane & 1) || !in_range(t.col, t.c0, t.c1) || t.w == 0 || t.w == W - 1) return;
#pragma unroll
    for (int i = 1; i < 5; i += 2) {
        const int j = t.row0 + i - 1;
        if (j < t.r1) {
            const T corner = (l[i - 1] + r[i - 1]) + (l[i + 1] + r[i + 1]);
            const T edge = (row[i - 1] + row[i + 1]) + (l[i] + r[i]);
            const T res = row[i] + T(0.5) * edge + T(0.25) * corner;
            const int I = t.col >> 1, J = j >> 1;
            bc[(int64_t)J * Nc + I] = is_dirichlet(Nc, I, J, dmask) ? T(0) : res;
        }
    }
}

// Post-smoothing block: x + P x_c, NU sweeps and with NORM the sums of squares
// of the defect, as post_tile for the same owned nodes.
template <typename T, bool NORM, int W, int NU>
__device__ __forceinline__ void post_block(BlockLds<T, W>& s, const T* __restrict__ bands,
                                           int64_t bs, int N, const T* __restrict__ x,
                                           const T* __restrict__ xc, const T* __restrict__ b,
                                           T omega, T* __restrict__ xout,
                                           double* __restrict__ rowpart, int strip, int chunk) {
    static_assert(NU + 1 <= F_HALO && F_NORM_ROWS == 4 && BLK_OWN % F_NORM_COLS == 0,
                  "halo of the sweeps and the norm; a wavefront's rows are one group");
    BlockTile<T, W> t(s, N, strip, chunk);
    const int Nc = (N >> 1) + 1;
    T v[4], k0[3], k1[3];
    {
        const rsrc_t Rx = make_rsrc(x, (int64_t)N * N * (int64_t)sizeof(T));
        const rsrc_t Rc = make_rsrc(xc, (int64_t)Nc * Nc * (int64_t)sizeof(T));
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = bload<T>(Rx, t.off(r));
        // the coarse values around rows row0 .. row0 + 3 (row0 is even)
        const int I = t.col >> 1, J = t.row0 >> 1;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const bool ok = in_range(J + q, 0, Nc);
            const uint32_t o = (uint32_t)((J + q) * Nc + I) * (uint32_t)sizeof(T);
            k0[q] = bload<T>(Rc, ok && in_range(I, 0, Nc) ? o : OFF_NONE);
            k1[q] = bload<T>(Rc, ok && in_range(I + 1, 0, Nc) ? o + (uint32_t)sizeof(T) : OFF_NONE);
        }
    }
    t.load(bands, bs, b);
    const bool c_even = !(t.col & 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int q = r >> 1;
        T p;
        if (r & 1)
            p = c_even ? T(0.5) * (k0[q] + k0[q + 1])
                       : T(0.25) * ((k0[q] + k1[q]) + (k0[q + 1] + k1[q + 1]));
        else
            p = c_even ? k0[q] : T(0.5) * (k0[q] + k1[q]);
        v[r] = t.in[r] ? v[r] + p : T(0);
    }
#pragma unroll
    for (int k = 0; k < NU; ++k) t.sweep(v, omega);
    t.store(xout, v);
    if (!NORM) return;
    T d[4];
    t.product(v, d);
    if (t.w == 0 || t.w == W - 1) return;
    // the column's sum over the wavefront's rows (one group of F_NORM_ROWS),
    // rows in increasing order, then the segments' eight column sums
    const bool own = in_range(t.col, t.c0, t.c1);
    double acc2 = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const T e = t.b[r] - d[r];
        if (t.row0 + r < t.r1) acc2 += own ? (double)e * (double)e : 0.0;
    }
    s.ns[t.w][t.lane] = acc2;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int nseg = (N + F_NORM_COLS - 1) / F_NORM_COLS, m = t.lane;
    if (m < BLK_OWN / F_NORM_COLS && t.c0 + m * F_NORM_COLS < t.c1 && t.row0 < t.r1) {
        const double* n = s.ns[t.w] + F_HALO + m * F_NORM_COLS;
        const double s8 = ((n[0] + n[1]) + (n[2] + n[3])) + ((n[4] + n[5]) + (n[6] + n[7]));
        rowpart[(int64_t)(t.row0 / F_NORM_ROWS) * nseg + t.c0 / F_NORM_COLS + m] = s8;
    }
}

}  // namespace dev
}  // namespace mg
