// Merged pass (marching tiles) on the finest level between two V(2,2) cycles: the post pass of
// one (prolongation, two sweeps, residual norm) and the pre pass of the next
// (two sweeps, defect, restriction) in one march.
//
// Bound by bytes first: apart, the two passes read the bands, b and the
// iterate twice (16 words a node in all, 7 of them again); merged, each is
// read once (5 bands, b, the iterate; two iterates written: 9 words), and the
// third sweep shares its band product with the norm.  At L = 12 the pair took
// 482 us in FP64 and 237 us in FP32, near the rate cold copies reach; merged
// 320 and 163 us.  Memory would take 270 and 135 us with the halo; a row step is
// about 270 (FP64) and 190 (FP32) instructions a wavefront, LDS is busy 43 and
// 50 % of the time, and two or three wavefronts a SIMD (249 and 149 registers)
// spend half of theirs waiting.
#pragma once

#include <utility>

#include "fused_ops.h"

namespace mg {
namespace dev {

// Columns / rows a tile recomputes per side: one for each of the two
// post-smoothing sweeps, the two pre-smoothing sweeps, the defect and the
// restriction.
constexpr int MID_HALO = 6;

// Strips of at most bt - 2 MID_HALO columns (whole norm segments), and as many
// chunks as fill `resident` workgroups once: every workgroup then runs at the
// same time, and a second wave would start with most of the chip idle (L = 12
// in FP64, 24 strips: 21 chunks 5.24 ms a solve, 26 chunks 6.6 ms).  Chunk
// heights are multiples of F_NORM_ROWS.
__host__ __device__ inline FusedGeom mid_geom(int N, int bt, int resident) {
    FusedGeom g;
    g.bt = bt;
    const int cmax = (bt - 2 * MID_HALO) / F_NORM_COLS * F_NORM_COLS;
    g.nstrips = (N + cmax - 1) / cmax;
    g.cw = (N + g.nstrips - 1) / g.nstrips;
    g.cw = (g.cw + F_NORM_COLS - 1) / F_NORM_COLS * F_NORM_COLS;
    const int chunks = resident / g.nstrips > 1 ? resident / g.nstrips : 1;
    g.rh = (N + chunks - 1) / chunks;
    g.rh = (g.rh + F_NORM_ROWS - 1) / F_NORM_ROWS * F_NORM_ROWS;
    g.nchunks = (N + g.rh - 1) / g.rh;
    g.blk = 0;
    return g;
}

// A store past the buffer is dropped, as a load from there returns zero: no
// lane is switched off around it.
template <int AUX>
__device__ __forceinline__ void bstore(rsrc_t r, uint32_t off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)off, 0, AUX);
}
template <int AUX>
__device__ __forceinline__ void bstore(rsrc_t r, uint32_t off, double v) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, (int)off, 0, AUX);
}

// f(0), f(1), .. f(U - 1) with constant arguments (register arrays indexed by
// them stay registers whatever the size of the body).
template <class F, int... I>
__device__ __forceinline__ void unrolled_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int U, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    unrolled_impl(f, std::make_integer_sequence<int, U>{});
}
#define MG_INLINE __attribute__((always_inline))

// On owned nodes: x_post = J(J(x + P x_c)) with the norm partials of
// post_tile, x2 = J(J(x_post)) and bc = P^T (b - A x2).  The same arithmetic
// per node, and the same partials, as post_tile and pre_tile: same bits.  x2
// must not alias x.
//
// One step (x row jx entering) takes two phases, a barrier before each; the
// stages of a phase are independent of each other:
//   A: sweep 1 at row jx-1, sweep 3 and the norm at jx-4, defect at jx-7
//   B: sweep 2 (x_post) at row jx-2, sweep 4 (x2) at jx-5, restriction at jx-8
// (five phases apart; three when sweep 3 followed sweep 2 in the step: 5.37 ->
// 5.24 ms in FP64, 4.66 -> 4.60 ms in mixed precision, a whole solve at L = 12).
// A stage of phase A reads what phase B of earlier steps wrote and the other
// way round, so every LDS ring of three rows has its oldest row rewritten only
// after a barrier that follows its last read.
//
// Bands of rows jx-7 .. jx+1 and b live in a ring of U register slots (the loop
// is unrolled by U, a multiple of two and three: LDS slots, coarse rows and
// register slots are constants of the phase); one band row, two rows of x and
// one coarse row are in flight.  More rows in flight measured slower (FP64 two:
// 5.26, three: 5.37 ms): loads are not what a step waits for, and registers
// decide how many workgroups a compute unit holds.  For the same reason the
// own column stays in LDS (in registers: FP64 spills, FP32 no change).  One
// wavefront per strip with lane shifts instead of LDS and barriers took 416 us
// (FP64) and 221 us (FP32) at L = 12: its halo is a third of its columns.
//
// Rows and columns of the tile that no owned result depends on hold unspecified
// values; nodes outside the grid hold zeros.
template <typename T, int BT>
__device__ __forceinline__ void mid_tile(const T* __restrict__ bands, int64_t bs, int N,
                                         const T* __restrict__ x, const T* __restrict__ xc,
                                         const T* __restrict__ b, T omega, T* __restrict__ xpost,
                                         T* __restrict__ x2, T* __restrict__ bc, int dmask,
                                         double* __restrict__ rowpart, int strip, int chunk,
                                         int rh, int cw) {
    constexpr int U = 12;
    constexpr int AHEAD = 1;   // band rows loaded before they enter
    constexpr int XAHEAD = 2;  // x rows
    constexpr int CAHEAD = 4;  // fine rows by which a coarse row is ahead
    __shared__ T X[3][BT + 2], S1[3][BT + 2], S2[3][BT + 2], S3[3][BT + 2], S4[3][BT + 2],
        D[3][BT + 2];
    __shared__ T U5[BT + 2], U6[2][BT + 2], U8[2][BT + 2];
    __shared__ double NS[BT];
    const int t = threadIdx.x + 1;  // LDS column; 0 and BT+1 are guards
    const int c0 = strip * cw, c1 = min(c0 + cw, N);
    const int r0 = chunk * rh, r1 = min(r0 + rh, N);
    const int col = c0 - MID_HALO + (int)threadIdx.x;
    const bool cval = col >= 0 && col < N;
    const bool c_own = in_range(col, c0, c1);
    const bool c_even = !(threadIdx.x & 1);  // c0 and the halo are even
    const int Nc = (N >> 1) + 1;
    const int64_t bytes = (int64_t)N * N * (int64_t)sizeof(T);
    const int64_t cbytes = (int64_t)Nc * Nc * (int64_t)sizeof(T);
    const RowRsrc<T> R(bands, bs, b, (int64_t)N * N);
    const rsrc_t Rx = make_rsrc(x, bytes), Rc = make_rsrc(xc, cbytes);
    const rsrc_t Rpost = make_rsrc(xpost, bytes), R2 = make_rsrc(x2, bytes);
    const rsrc_t Rbc = make_rsrc(bc, cbytes);
    if (threadIdx.x < 2) {
        const int g = threadIdx.x ? BT + 1 : 0;
        for (int s = 0; s < 3; ++s)
            X[s][g] = S1[s][g] = S2[s][g] = S3[s][g] = S4[s][g] = D[s][g] = T(0);
        U5[g] = U6[0][g] = U6[1][g] = U8[0][g] = U8[1][g] = T(0);
    }
    T bk[U][9], bb[U], px[U];      // slot (row - js) mod U
    T k0[U / 2], k1[U / 2];        // coarse values left and right of the column
    unrolled<U>([&](auto q) MG_INLINE {
        constexpr int i = decltype(q)::value;
        bk[i][0] = bk[i][1] = bk[i][2] = bk[i][3] = bk[i][4] = T(0);
        bk[i][5] = bk[i][6] = bk[i][7] = bk[i][8] = T(0);
        bb[i] = px[i] = k0[i / 2] = k1[i / 2] = T(0);
    });
    double nacc = 0.0;  // this lane's column sum over the current row group
    const int nseg = (N + F_NORM_COLS - 1) / F_NORM_COLS;
    const bool lead = c_own && ((col - c0) % F_NORM_COLS) == 0;
    const int js = r0 - MID_HALO;    // even, as r0
    const int xend = r1 + MID_HALO;  // end of the x rows needed
    const int jlast = r1 + 7;        // step of restriction row r1 - 1
    auto in_grid = [&](int j) MG_INLINE { return cval & ((unsigned)j < (unsigned)N); };
    auto own_row = [&](int j) MG_INLINE { return in_win(j, r0, r1); };
    auto load_x = [&](int j) MG_INLINE {
        const bool use = in_grid(j) && j < xend;
        return bload<T>(Rx, use ? node_off(j, N, col, sizeof(T)) : OFF_NONE);
    };
    auto load_coarse = [&](int j, T& a, T& c) MG_INLINE {  // coarse row j/2, j even
        const bool use = in_grid(j) && j < xend + 1;
        const uint32_t o = use ? node_off(j >> 1, Nc, col >> 1, sizeof(T)) : OFF_NONE;
        a = bload<T>(Rc, o);
        c = bload<T>(Rc, o + (uint32_t)sizeof(T));
    };
    auto load_bands = [&](int j, T(&q)[9], T& bv) MG_INLINE {
        const bool use = in_grid(j) && j < xend - 1;
        const uint32_t o = use ? node_off(j, N, col, sizeof(T)) : OFF_NONE;
        q[4] = bload<T, AUX_NT>(R.band[4], o);
        q[5] = bload<T, AUX_NT>(R.band[5], o);
        q[6] = bload<T, AUX_NT>(R.band[6], o);
        q[7] = bload<T, AUX_NT>(R.band[7], o);
        q[8] = bload<T, AUX_NT>(R.band[8], o);
        bv = bload<T>(R.b, o);
    };
    unrolled<CAHEAD>([&](auto q) MG_INLINE {
        constexpr int i = decltype(q)::value;
        if constexpr (i < XAHEAD) px[i] = load_x(js + i);
        if constexpr (!(i & 1)) load_coarse(js + i, k0[i / 2], k1[i / 2]);
        if constexpr (i < AHEAD) load_bands(js + i, bk[i], bb[i]);
    });
#pragma unroll 1
    for (int jb = js; jb <= jlast; jb += U) {
        unrolled<U>([&](auto phase) MG_INLINE {
            constexpr int ph = decltype(phase)::value;
            const int jx = jb + ph;
            // slots of row jx - k in LDS and in registers
            constexpr auto s3 = [](int k) constexpr { return (ph + U - k) % 3; };
            constexpr auto sl = [](int k) constexpr { return (ph + U - k) % U; };
            {
                // x + P x_c (the arithmetic of prolong_elem; both column
                // parities evaluated, one selected)
                constexpr int i = ph / 2, i2 = (ph / 2 + 1) % (U / 2);
                T v;
                if constexpr (ph & 1)
                    v = c_even ? T(0.5) * (k0[i] + k0[i2])
                               : T(0.25) * ((k0[i] + k1[i]) + (k0[i2] + k1[i2]));
                else
                    v = c_even ? k0[i] : T(0.5) * (k0[i] + k1[i]);
                X[s3(0)][t] = in_grid(jx) ? px[ph] + v : T(0);
            }
            U5[t] = bk[sl(1)][5];
            U6[(ph + 1) & 1][t] = bk[sl(1)][6];
            U8[(ph + 1) & 1][t] = bk[sl(1)][8];
            px[(ph + XAHEAD) % U] = load_x(jx + XAHEAD);
            if constexpr (((ph + CAHEAD) & 1) == 0)
                load_coarse(jx + CAHEAD, k0[((ph + CAHEAD) % U) / 2],
                            k1[((ph + CAHEAD) % U) / 2]);
            load_bands(jx + AHEAD, bk[(ph + AHEAD) % U], bb[(ph + AHEAD) % U]);
            __syncthreads();
            // ---- phase A
            int group = -1;  // row group whose column sums went to NS (uniform)
            {
                // the lower bands of row jx-1 (see LowerBands), first sweep
                T(&q)[9] = bk[sl(1)];
                q[0] = U8[ph & 1][t - 1];
                q[1] = bk[sl(2)][7];
                q[2] = U6[ph & 1][t + 1];
                q[3] = U5[t - 1];
                const T acc = band_row_product(q, X[s3(2)], X[s3(1)], X[s3(0)], t);
                const T v = X[s3(1)][t] + jacobi_div(omega * (bb[sl(1)] - acc), q[4]);
                S1[s3(1)][t] = in_grid(jx - 1) ? v : T(0);
            }
            {
                // residual of x_post and third sweep
                const T(&q)[9] = bk[sl(4)];
                const T acc = band_row_product(q, S2[s3(5)], S2[s3(4)], S2[s3(3)], t);
                const T d = bb[sl(4)] - acc;
                const T v = S2[s3(4)][t] + jacobi_div(omega * d, q[4]);
                S3[s3(4)][t] = in_grid(jx - 4) ? v : T(0);
                const int j = jx - 4;
                if (own_row(j)) {
                    nacc += c_own ? (double)d * (double)d : 0.0;
                    if ((j % F_NORM_ROWS) == F_NORM_ROWS - 1 || j == r1 - 1) {
                        NS[threadIdx.x] = nacc;
                        nacc = 0.0;
                        group = j / F_NORM_ROWS;
                    }
                }
            }
            {
                const T(&q)[9] = bk[sl(7)];
                const T acc = band_row_product(q, S4[s3(8)], S4[s3(7)], S4[s3(6)], t);
                D[s3(7)][t] = in_grid(jx - 7) ? bb[sl(7)] - acc : T(0);
            }
            __syncthreads();
            // ---- phase B
            if (group >= 0 && lead) {
                const double* v = NS + threadIdx.x;
                const double s8 =
                    ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
                rowpart[(int64_t)group * nseg + col / F_NORM_COLS] = s8;
            }
            {
                const T(&q)[9] = bk[sl(2)];
                const T acc = band_row_product(q, S1[s3(3)], S1[s3(2)], S1[s3(1)], t);
                T v = S1[s3(2)][t] + jacobi_div(omega * (bb[sl(2)] - acc), q[4]);
                v = in_grid(jx - 2) ? v : T(0);
                S2[s3(2)][t] = v;
                if (own_row(jx - 2))
                    bstore<AUX_NT>(Rpost, c_own ? node_off(jx - 2, N, col, sizeof(T)) : OFF_NONE,
                                   v);
            }
            {
                const T(&q)[9] = bk[sl(5)];
                const T acc = band_row_product(q, S3[s3(6)], S3[s3(5)], S3[s3(4)], t);
                T v = S3[s3(5)][t] + jacobi_div(omega * (bb[sl(5)] - acc), q[4]);
                v = in_grid(jx - 5) ? v : T(0);
                S4[s3(5)][t] = v;
                if (own_row(jx - 5))
                    bstore<AUX_NT>(R2, c_own ? node_off(jx - 5, N, col, sizeof(T)) : OFF_NONE, v);
            }
            if constexpr (!(ph & 1)) {
                const int jr = jx - 8;  // even
                if (own_row(jr)) {
                    const int I = col >> 1, J = jr >> 1;
                    const T* u = D[s3(9)];
                    const T* c = D[s3(8)];
                    const T* o = D[s3(7)];
                    const T corner = (u[t - 1] + u[t + 1]) + (o[t - 1] + o[t + 1]);
                    const T edge = (u[t] + o[t]) + (c[t - 1] + c[t + 1]);
                    const T s = c[t] + T(0.5) * edge + T(0.25) * corner;
                    bstore<0>(Rbc, c_own && c_even ? node_off(J, Nc, I, sizeof(T)) : OFF_NONE,
                              is_dirichlet(Nc, I, J, dmask) ? T(0) : s);
                }
            }
        });
    }
}
#undef MG_INLINE

}  // namespace dev
}  // namespace mg
