// Fused smoothing passes of the V(2,2) cycle.  One workgroup owns a strip
// of grid columns and a chunk of grid rows and marches down the rows; each
// row of bands, x and b is read from HBM once and kept (bands in a register
// ring of six rows, iterates in LDS rings of three rows) while every
// fused step that needs it runs:
//   pre  : two damped Jacobi sweeps (the first possibly from a zero
//          iterate), the defect of the result and its restriction P^T d to
//          the next coarser level;
//   post : prolongation and correction x + P x_c, two damped Jacobi sweeps,
//          and optionally the sum of squares of the final defect.
// Each node's arithmetic is the one of the unfused kernels (same operands,
// same operation order), so fused and unfused cycles give identical bits.
// Strips overlap by F_HALO columns and chunks by F_HALO rows; the overlap is
// recomputed and only owned nodes are written.
//
// Rows of x and of bands are loaded two to three steps ahead of their use,
// so that enough bytes are in flight per wavefront to cover HBM latency.
// Row bookkeeping of one step of the pre pass: the x row jx enters; after a
// first barrier the first sweep runs at row jx-1 and the defect at jx-4,
// after a second barrier the second sweep at jx-2 and the restriction at
// jx-5.  The post pass runs the first sweep at jx-1, the second at jx-2 and
// the norm at jx-3, a barrier before each.  With j0 the first row of the
// march, an iterate row j lives
// in LDS slot (j - j0) mod 3 and a band row in register slot (j - j0) mod 6;
// the loop is unrolled by six so every slot index is a compile-time
// constant.  The march starts at the first row that is needed and runs
// whole blocks of six steps past the last one (the extra steps compute
// nothing that is kept).
#pragma once

#include "device_ops.h"
#include "mgfem.h"

namespace mg {
namespace dev {

constexpr int F_HALO = 4;           // columns / rows recomputed per side
constexpr int F_MIN_THREADS = 64;   // workgroup widths: 64, 128, 192 or 256 threads,
constexpr int F_MAX_THREADS = 256;  // one grid column per thread

// Columns of one segment of the residual-norm partials (see post_tile);
// strips own whole segments.
constexpr int F_NORM_COLS = 8;

struct FusedGeom {
    int bt;       // threads per workgroup
    int cw;       // owned columns per strip (a multiple of F_NORM_COLS, at most bt - 2 F_HALO)
    int nstrips;  // strips of cw columns (the last one may be narrower)
    int nchunks;  // chunks of rh rows
    int rh;       // owned rows per chunk (even)
    int blk;      // 0: marching tiles; else a block tile shape (block_geom)
};

// Strips of equal width (rounded up to a multiple of F_NORM_COLS) as few as
// bt threads allow.
__host__ __device__ inline FusedGeom fused_geom(int N, int bt, int rh) {
    FusedGeom g;
    g.bt = bt;
    g.rh = rh;
    const int cmax = bt - 2 * F_HALO;  // a multiple of F_NORM_COLS
    g.nstrips = (N + cmax - 1) / cmax;
    g.cw = (N + g.nstrips - 1) / g.nstrips;
    g.cw = (g.cw + F_NORM_COLS - 1) / F_NORM_COLS * F_NORM_COLS;
    g.nchunks = (N + rh - 1) / rh;
    g.blk = 0;
    return g;
}

// Block tiles (block_ops.h): shape s in 1..BLK_SHAPES owns 4 << s rows (8, 16
// or 32) by BLK_OWN columns, run by block_waves(s) wavefronts; 0 is no block
// shape.  In the tile table and the ABI a block tile is marked by BLK_TAG in
// the place of the columns and BLK_TAG_WAVES (or 0) in that of the wavefronts.
constexpr int BLK_SHAPES = 3;
constexpr int BLK_TAG = 32;
constexpr int BLK_TAG_WAVES = 4;
constexpr int BLK_OWN = 64 - 2 * F_HALO;
// Largest level side the autotuners try block tiles on.
constexpr int BLK_MAX_N = 1025;
__host__ __device__ constexpr int block_rows(int shape) { return 4 << shape; }
__host__ __device__ constexpr int block_waves(int shape) { return block_rows(shape) / 4 + 2; }
__host__ __device__ inline int block_shape(int rows, int cols) {
    if (cols != BLK_TAG) return 0;
    for (int s = 1; s <= BLK_SHAPES; ++s)
        if (rows == block_rows(s)) return s;
    return 0;
}
__host__ __device__ inline FusedGeom block_geom(int N, int shape) {
    FusedGeom g;
    g.bt = 64 * block_waves(shape);
    g.rh = block_rows(shape);
    g.cw = BLK_OWN;
    g.nstrips = (N + g.cw - 1) / g.cw;
    g.nchunks = (N + g.rh - 1) / g.rh;
    g.blk = shape;
    return g;
}

__device__ __forceinline__ bool in_range(int v, int lo, int hi) { return v >= lo && v < hi; }

// v in [lo, hi) for lo <= hi, with one compare.
__device__ __forceinline__ bool in_win(int v, int lo, int hi) {
    return (unsigned)(v - lo) < (unsigned)(hi - lo);
}

// The 9-term band product at one node from the rows j-1, j, j+1 of an
// iterate held in LDS, around LDS column t: the fma chain of stencil_tile.
template <typename T>
__device__ __forceinline__ T band_row_product(const T (&bk)[9], const T* __restrict__ rm,
                                              const T* __restrict__ rc,
                                              const T* __restrict__ rp, int t) {
    const T* rows[3] = {rm, rc, rp};
    T acc = T(0);
#pragma unroll
    for (int k = 0; k < 9; ++k) acc = fma(bk[k], rows[k / 3][t + k % 3 - 1], acc);
    return acc;
}

// Raw buffer resources: one per band array, for b and for x.  A load
// whose byte offset falls outside [0, bytes) returns zero, so rows above and
// below the grid need no checks (negative offsets wrap to huge unsigned ones).
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int RSRC_WORD3 = 0x00020000;  // raw (untyped) buffer access on CDNA
constexpr int AUX_NT = 2;               // non-temporal

// A pass over more than the last-level cache holds (STREAM, see
// pass_streams) loads the bands and stores its iterate non-temporally, so
// that b, x and the coarse vectors stay cached; a smaller pass finds all of
// it in the cache from the pass before.
template <bool STREAM, typename T>
__device__ __forceinline__ void pass_store(T* p, T v) {
    if (STREAM)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0,
                                             (int)(uint32_t)bytes, RSRC_WORD3);
}

template <typename T, int AUX>
struct BufLoad;
template <int AUX>
struct BufLoad<float, AUX> {
    static __device__ __forceinline__ float get(rsrc_t r, uint32_t off) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, AUX));
    }
};
template <int AUX>
struct BufLoad<double, AUX> {
    static __device__ __forceinline__ double get(rsrc_t r, uint32_t off) {
        return __builtin_bit_cast(double,
                                  __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, AUX));
    }
};
template <typename T, int AUX = 0>
__device__ __forceinline__ T bload(rsrc_t r, uint32_t off) {
    return BufLoad<T, AUX>::get(r, off);
}

template <typename T>
struct RowRsrc {
    rsrc_t band[9];
    rsrc_t b;
    __device__ RowRsrc(const T* bands, int64_t bs, const T* bb, int64_t n) {
#pragma unroll
        for (int k = 0; k < 9; ++k) band[k] = make_rsrc(bands + k * bs, n * (int64_t)sizeof(T));
        b = make_rsrc(bb, n * (int64_t)sizeof(T));
    }
};

// Byte offset past every buffer: a load from it returns zero.  The largest
// buffer (an FP64 vector at the finest admitted level, 16385^2 x 8 B) is
// just over 2 GiB, so the offset sits at 3 GiB, with room below 2^32 for the
// small strides added to it.
constexpr uint32_t OFF_NONE = 0xC0000000u;
static_assert((uint64_t)((1 << MG_MAX_LEVEL) + 1) * ((1 << MG_MAX_LEVEL) + 1) * sizeof(double) <
                  (uint64_t)OFF_NONE,
              "out-of-range offset inside a buffer");

// The diagonal and upper bands (4..8) and b of one node at byte offset off,
// zeros when !need; the lower bands are rebuilt from the neighbours' upper
// bands (see LowerBands).  The loads are issued on every lane (an unneeded
// lane reads past the buffer), so no branch separates a load from its later
// use and the compiler's wait counting stays exact across the loop.
template <bool STREAM, typename T>
__device__ __forceinline__ void load_upper(const RowRsrc<T>& R, uint32_t off, bool need,
                                           T (&bk)[9], T& bb) {
    const uint32_t o = need ? off : OFF_NONE;
#pragma unroll
    for (int k = 4; k < 9; ++k) bk[k] = bload<T, STREAM ? AUX_NT : 0>(R.band[k], o);
    bb = bload<T>(R.b, o);
}

// The assembled matrix is symmetric bit for bit (each entry and its mirror
// sum the same element terms in the same order), so the lower bands of a
// row are upper bands of its neighbours:
//   A[p][p-1]   = band 5 at p-1      (same row, left column)
//   A[p][p-N-1] = band 8 at p-N-1    (previous row, left column)
//   A[p][p-N]   = band 7 at p-N      (previous row, same column)
//   A[p][p-N+1] = band 6 at p-N+1    (previous row, right column).
// A tile reads 5 of the 9 band streams; bands 5, 6 and 8 of each row pass
// through LDS to the neighbouring columns (6 and 8 kept for two rows), band
// 7 of the previous row is still in the thread's register ring.  Columns
// and rows outside the grid read as zero, as the stored lower bands are.
template <typename T, int BT>
struct LowerBands {
    T* u5;  // band 5 of the row being completed
    T* u6;  // band 6 of two consecutive rows (slot = relative row parity)
    T* u8;  // band 8, likewise
    __device__ void init() {
        if (threadIdx.x < 2) {
            const int g = threadIdx.x ? BT + 1 : 0;
            u5[g] = u6[g] = u6[(BT + 2) + g] = u8[g] = u8[(BT + 2) + g] = T(0);
        }
    }
    // Before a barrier: publish the upper bands of row r (slot par).
    __device__ __forceinline__ void publish(const T (&bk)[9], int par, int t) {
        u5[t] = bk[5];
        u6[par * (BT + 2) + t] = bk[6];
        u8[par * (BT + 2) + t] = bk[8];
    }
    // After it: complete row r from its own and row r-1's published bands
    // (row r-1 in slot prev, its band 7 in bkp).
    __device__ __forceinline__ void complete(T (&bk)[9], const T (&bkp)[9], int prev, int t) {
        bk[0] = u8[prev * (BT + 2) + t - 1];
        bk[1] = bkp[7];
        bk[2] = u6[prev * (BT + 2) + t + 1];
        bk[3] = u5[t - 1];
    }
};

__device__ __forceinline__ uint32_t node_off(int j, int N, int col, int size) {
    return (uint32_t)(j * N + col) * (uint32_t)size;
}

// Pre-smoothing tile (strip, chunk) on a level with N nodes per side:
// x2 = J(J(x)) on owned nodes and bc = P^T (b - A x2) on the owned coarse
// nodes (0 at coarse nodes on the Dirichlet sides of dmask).  With XZERO the
// first sweep starts from a zero iterate and x is not read.  Band rows live
// in a ring of six register slots (the loop is unrolled by six): the load of
// row jx+2 goes out in step jx as soon as the defect has freed its slot, two
// and a half steps before the row is first used; x rows go out three steps
// ahead.
//
// One step (x row jx entering) runs in two barrier-separated phases: phase A
// takes the first sweep at row jx-1 (from the x rows written before the
// first barrier) and the defect at row jx-4 (from second-sweep rows of
// earlier steps); phase B takes the second sweep at row jx-2 (from the
// first-sweep row of phase A) and the restriction at row jx-5 (from the
// defect row of phase A).  Every LDS row ring has three slots: a slot is
// rewritten only in a window that no reader of its old row shares.
template <typename T, bool XZERO, int BT, bool STREAM>
__device__ void pre_tile(const T* __restrict__ bands, int64_t bs, int N, const T* __restrict__ x,
                         const T* __restrict__ b, T omega, T* __restrict__ x2out,
                         T* __restrict__ bc, int dmask, int strip, int chunk, int rh, int cw) {
    __shared__ T X[3][BT + 2], A[3][BT + 2], B[3][BT + 2], D[3][BT + 2];
    __shared__ T U5[BT + 2], U6[2][BT + 2], U8[2][BT + 2];
    LowerBands<T, BT> lower{U5, &U6[0][0], &U8[0][0]};
    const int t = threadIdx.x + 1;  // LDS column; 0 and BT+1 are guards
    const int c0 = strip * cw, c1 = min(c0 + cw, N);
    const int r0 = chunk * rh, r1 = min(r0 + rh, N);
    const int col = c0 - F_HALO + (int)threadIdx.x;
    const bool cval = col >= 0 && col < N;
    // column / row ranges where each step is needed (rows clipped to the
    // grid: rows outside it hold zeros)
    const bool c_op1 = cval && in_range(col, c0 - 3, c1 + 3);
    const bool c_op2 = cval && in_range(col, c0 - 2, c1 + 2);
    const bool c_op3 = cval && in_range(col, c0 - 1, c1 + 1);
    const bool c_own = in_range(col, c0, c1);
    const bool c_coarse = c_own && !(col & 1);
    const int lo1 = max(r0 - 3, 0), hi1 = min(r1 + 3, N);
    const int lo2 = max(r0 - 2, 0), hi2 = min(r1 + 2, N);
    const int lo3 = max(r0 - 1, 0), hi3 = min(r1 + 1, N);
    const int Nc = (N >> 1) + 1;
    const int64_t n = (int64_t)N * N;
    const RowRsrc<T> R(bands, bs, b, n);
    const rsrc_t Rx = make_rsrc(x, n * (int64_t)sizeof(T));
    if (threadIdx.x < 2) {
        const int g = threadIdx.x ? BT + 1 : 0;
#pragma unroll
        for (int s = 0; s < 3; ++s) X[s][g] = A[s][g] = B[s][g] = D[s][g] = T(0);
    }
    lower.init();
    T bk[6][9], bb[6];  // band rows, slot (r - js) mod 6
    T pfx[3];           // x rows, slot (r - js) mod 3 (LDS rows likewise)
    // The first x row any sweep needs (r0 - F_HALO) enters LDS before the
    // loop, whose first step brings in the next; the last restriction row
    // leaves last.
    const int js = r0 - F_HALO + 1;
    const int jend = r1 + 5;
    auto xload = [&](int j) -> T {
        if (XZERO) return T(0);
        return bload<T>(Rx, cval && j < r1 + 4 ? node_off(j, N, col, sizeof(T)) : OFF_NONE);
    };
    // upper bands and b: the rows the first sweep needs and the one above
    // (its lower bands come from there), on every column of the tile (the
    // halo columns' bands complete their neighbours' rows)
    auto needb = [&](int j) { return cval && in_range(j, r0 - 4, r1 + 3); };
    if (!XZERO) X[2][t] = xload(js - 1);  // slot of row js - 1
    pfx[0] = xload(js);
    pfx[1] = xload(js + 1);
    pfx[2] = xload(js + 2);
    load_upper<STREAM>(R, node_off(js - 1, N, col, sizeof(T)), needb(js - 1), bk[5], bb[5]);
    load_upper<STREAM>(R, node_off(js, N, col, sizeof(T)), needb(js), bk[0], bb[0]);
    load_upper<STREAM>(R, node_off(js + 1, N, col, sizeof(T)), needb(js + 1), bk[1], bb[1]);
#pragma unroll 1
    for (int jb = js; jb < jend; jb += 6) {
#pragma unroll
        for (int ph = 0; ph < 6; ++ph) {
            const int jx = jb + ph;  // x row entering: LDS slot x3
            const int x3 = ph % 3;
            const int j1 = jx - 1, j2 = jx - 2, jd = jx - 4, jr = jx - 5;
            const int b1 = (ph + 5) % 6, b2 = (ph + 4) % 6, bd = (ph + 2) % 6;
            // LDS slots: x3 holds rows jx, jx-3, jx-6; l1 rows jx-1, jx-4;
            // l2 rows jx-2, jx-5
            const int l1 = (x3 + 2) % 3, l2 = (x3 + 1) % 3;
            // x row jx and the upper bands of row jx-1 into LDS; prefetch x
            // row jx+3 into the register just freed
            if (!XZERO) X[x3][t] = pfx[x3];
            lower.publish(bk[b1], (ph + 1) & 1, t);
            pfx[x3] = xload(jx + 3);
            __syncthreads();
            // ---- phase A
            lower.complete(bk[b1], bk[b2], ph & 1, t);
            // Every lane computes each step (lanes and rows outside a step's
            // window select zero), so the steps run without divergent
            // branches.
            // first sweep at row j1
            {
                T v;
                if (XZERO) {
                    v = jacobi_div(omega * bb[b1], bk[b1][4]);
                } else {
                    const T acc = band_row_product(bk[b1], X[l2], X[l1], X[x3], t);
                    v = X[l1][t] + jacobi_div(omega * (bb[b1] - acc), bk[b1][4]);
                }
                A[l1][t] = (c_op1 & in_win(j1, lo1, hi1)) ? v : T(0);
            }
            // defect at row jd from second-sweep rows jd-1, jd, jd+1
            {
                const T acc = band_row_product(bk[bd], B[l2], B[l1], B[x3], t);
                D[l1][t] = (c_op3 & in_win(jd, lo3, hi3)) ? bb[bd] - acc : T(0);
            }
            // the bands of row jx+2 into the slot row jd no longer needs
            load_upper<STREAM>(R, node_off(jx + 2, N, col, sizeof(T)), needb(jx + 2), bk[bd], bb[bd]);
            __syncthreads();
            // ---- phase B
            // second sweep at row j2 (written on owned nodes)
            {
                const T acc = band_row_product(bk[b2], A[x3], A[l2], A[l1], t);
                T v = A[l2][t] + jacobi_div(omega * (bb[b2] - acc), bk[b2][4]);
                v = (c_op2 & in_win(j2, lo2, hi2)) ? v : T(0);
                if (in_win(j2, r0, r1) && c_own)
                    pass_store<STREAM>(x2out + (int64_t)j2 * N + col, v);
                B[l2][t] = v;
            }
            // restriction of defect rows jr-1, jr, jr+1 to coarse row jr/2
            if (in_win(jr, r0, r1) && !(jr & 1)) {
                const int I = col >> 1, J = jr >> 1;
                // defect columns and rows outside the grid are zero in LDS
                const T* u = D[x3];  // row jr - 1
                const T* c = D[l2];  // row jr
                const T* o = D[l1];  // row jr + 1
                const T corner = (u[t - 1] + u[t + 1]) + (o[t - 1] + o[t + 1]);
                const T edge = (u[t] + o[t]) + (c[t - 1] + c[t + 1]);
                const T s = c[t] + T(0.5) * edge + T(0.25) * corner;
                if (c_coarse) bc[(int64_t)J * Nc + I] = is_dirichlet(Nc, I, J, dmask) ? T(0) : s;
            }
        }
    }
}

// Grid rows per residual partial of a fused post pass; chunk heights are
// multiples of it, so no group of rows straddles two tiles.
constexpr int F_NORM_ROWS = 4;

// Partial sums of squares a fused post pass with NORM writes on a level of
// N nodes per side: one per (group of F_NORM_ROWS grid rows, segment of
// F_NORM_COLS grid columns), row groups outer.  The layout depends on N
// alone, not on the tiling.
__host__ __device__ inline int64_t fused_norm_parts(int N) {
    return (int64_t)((N + F_NORM_ROWS - 1) / F_NORM_ROWS) * ((N + F_NORM_COLS - 1) / F_NORM_COLS);
}

// Post-smoothing tile: x_out = J(J(x + P x_c)) on owned nodes.  With NORM
// also rowpart[G * NSEG + m] = the sum of (b - A x_out)^2 over rows 4G ..
// 4G+3 and columns 8m .. 8m+7 (NSEG segments per row), in one fixed order:
// each column's rows in increasing order, then the eight column sums as
// ((c0 + c1) + (c2 + c3)) + ((c4 + c5) + (c6 + c7)).  Neither the chunk
// heights nor the strip widths change a bit of it.  Same register ring as
// pre_tile; a barrier before each of the first sweep (row jx-1), the second
// (row jx-2) and the norm (row jx-3).
template <typename T, bool NORM, int BT, bool STREAM>
__device__ void post_tile(const T* __restrict__ bands, int64_t bs, int N, const T* __restrict__ x,
                          const T* __restrict__ xc, const T* __restrict__ b, T omega,
                          T* __restrict__ xout, double* __restrict__ rowpart, int strip, int chunk,
                          int rh, int cw) {
    __shared__ T X[3][BT + 2], A[3][BT + 2], B[3][BT + 2];
    __shared__ T U5[BT + 2], U6[2][BT + 2], U8[2][BT + 2];
    LowerBands<T, BT> lower{U5, &U6[0][0], &U8[0][0]};
    constexpr int H = NORM ? 3 : 2;  // halo the last step needs
    const int t = threadIdx.x + 1;
    const int c0 = strip * cw, c1 = min(c0 + cw, N);
    const int r0 = chunk * rh, r1 = min(r0 + rh, N);
    const int col = c0 - F_HALO + (int)threadIdx.x;
    const bool cval = col >= 0 && col < N;
    const bool c_x = cval && in_range(col, c0 - H, c1 + H);
    const bool c_op1 = cval && in_range(col, c0 - (H - 1), c1 + (H - 1));
    const bool c_op2 = cval && in_range(col, c0 - (H - 2), c1 + (H - 2));
    const bool c_own = in_range(col, c0, c1);
    const int lo1 = max(r0 - (H - 1), 0), hi1 = min(r1 + (H - 1), N);
    const int lo2 = max(r0 - (H - 2), 0), hi2 = min(r1 + (H - 2), N);
    const int64_t n = (int64_t)N * N;
    const RowRsrc<T> R(bands, bs, b, n);
    const rsrc_t Rx = make_rsrc(x, n * (int64_t)sizeof(T));
    if (threadIdx.x < 2) {
        const int g = threadIdx.x ? BT + 1 : 0;
#pragma unroll
        for (int s = 0; s < 3; ++s) X[s][g] = A[s][g] = B[s][g] = T(0);
    }
    lower.init();
    T bk[6][9], bb[6];
    // x and the four coarse values around each x row in flight (slot r mod 3)
    T pfx[3], pc0[3], pc1[3], pc2[3], pc3[3];
    // Norm partials: at the end of a row group every lane leaves its
    // column's sum in NS; after the next barrier the lane at the first
    // column of each owned segment adds the segment's eight sums.
    __shared__ double NS[BT];
    double nacc = 0.0;  // this lane's column sum over the current row group
    int pend = -1;      // row group whose sums wait in NS (uniform), or -1
    const int nseg = (N + F_NORM_COLS - 1) / F_NORM_COLS;
    const bool lead = c_own && ((col - c0) % F_NORM_COLS) == 0;
    auto flush = [&]() {
        if (lead) {
            const double* v = NS + threadIdx.x;
            const double s8 = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            rowpart[(int64_t)pend * nseg + col / F_NORM_COLS] = s8;
        }
    };
    // first x row needed .. last row of the last step (the norm, or the
    // second sweep)
    const int jstart = r0 - H;
    const int jend = r1 + (NORM ? 3 : 2);
    // x row j plus its coarse correction P x_c (the arithmetic of
    // prolong_elem): the x value and the four coarse values around the node
    // are loaded ahead and combined when the row enters
    const int Nc = (N >> 1) + 1;
    const rsrc_t Rc = make_rsrc(xc, (int64_t)Nc * Nc * (int64_t)sizeof(T));
    auto x_use = [&](int j) { return c_x && in_range(j, r0 - H, r1 + H) && in_range(j, 0, N); };
    auto xrow_load = [&](int j, T& xv, T& c0, T& c1, T& c2, T& c3) {
        const bool use = x_use(j);
        const uint32_t ox = use ? node_off(j, N, col, sizeof(T)) : OFF_NONE;
        const uint32_t oc =
            use ? (uint32_t)((j >> 1) * Nc + (col >> 1)) * (uint32_t)sizeof(T) : OFF_NONE;
        xv = bload<T>(Rx, ox);
        c0 = bload<T>(Rc, oc);
        c1 = bload<T>(Rc, oc + (uint32_t)sizeof(T));
        c2 = bload<T>(Rc, oc + (uint32_t)(Nc * sizeof(T)));
        c3 = bload<T>(Rc, oc + (uint32_t)((Nc + 1) * sizeof(T)));
    };
    const bool c_even = !(col & 1);
    auto xrow_value = [&](int j, T xv, T c0, T c1, T c2, T c3) -> T {
        // every case is evaluated and one selected (no divergent branch)
        const T v_row = c_even ? c0 : T(0.5) * (c0 + c1);  // even grid row
        const T v_odd = c_even ? T(0.5) * (c0 + c2) : T(0.25) * ((c0 + c1) + (c2 + c3));
        const T v = (j & 1) ? v_odd : v_row;
        return x_use(j) ? xv + v : T(0);
    };
    // upper bands and b: the first sweep's rows and the one above, on every
    // column of the tile (see pre_tile)
    auto needb = [&](int j) { return cval && in_range(j, r0 - H, r1 + (H - 1)); };
    // Without NORM no step reads row jx-3 and the register ring has room to
    // load bands and x one row further ahead (three rows in flight).
    constexpr int AHEAD = NORM ? 2 : 3;
    xrow_load(jstart, pfx[0], pc0[0], pc1[0], pc2[0], pc3[0]);
    xrow_load(jstart + 1, pfx[1], pc0[1], pc1[1], pc2[1], pc3[1]);
    if (AHEAD == 3) xrow_load(jstart + 2, pfx[2], pc0[2], pc1[2], pc2[2], pc3[2]);
    load_upper<STREAM>(R, node_off(jstart - 1, N, col, sizeof(T)), needb(jstart - 1), bk[5], bb[5]);
    load_upper<STREAM>(R, node_off(jstart, N, col, sizeof(T)), needb(jstart), bk[0], bb[0]);
    if (AHEAD == 3)
        load_upper<STREAM>(R, node_off(jstart + 1, N, col, sizeof(T)), needb(jstart + 1), bk[1], bb[1]);
#pragma unroll 1
    for (int jb = jstart; jb < jend; jb += 6) {
#pragma unroll
        for (int ph = 0; ph < 6; ++ph) {
            const int jx = jb + ph;
            const int x3 = ph % 3;
            const int j1 = jx - 1, j2 = jx - 2, j3 = jx - 3;
            const int b1 = (ph + 5) % 6, b2 = (ph + 4) % 6, b3 = (ph + 3) % 6;
            const int l1 = (x3 + 2) % 3, l2 = (x3 + 1) % 3;
            X[x3][t] = xrow_value(jx, pfx[x3], pc0[x3], pc1[x3], pc2[x3], pc3[x3]);
            lower.publish(bk[b1], (ph + 1) & 1, t);
            {
                // x row jx+AHEAD into its slot (the one just written to LDS
                // when three rows are in flight)
                const int xs = (x3 + AHEAD) % 3;
                xrow_load(jx + AHEAD, pfx[xs], pc0[xs], pc1[xs], pc2[xs], pc3[xs]);
            }
            load_upper<STREAM>(R, node_off(jx + AHEAD - 1, N, col, sizeof(T)), needb(jx + AHEAD - 1),
                       bk[(ph + AHEAD - 1) % 6], bb[(ph + AHEAD - 1) % 6]);
            __syncthreads();
            if (NORM && pend >= 0) {
                flush();
                pend = -1;
            }
            lower.complete(bk[b1], bk[b2], ph & 1, t);
            // every lane computes each sweep (lanes and rows outside the
            // sweep's window select zero): no divergent branches
            {
                const T acc = band_row_product(bk[b1], X[l2], X[l1], X[x3], t);
                const T v = X[l1][t] + jacobi_div(omega * (bb[b1] - acc), bk[b1][4]);
                A[l1][t] = (c_op1 & in_win(j1, lo1, hi1)) ? v : T(0);
            }
            __syncthreads();
            {
                const T acc = band_row_product(bk[b2], A[x3], A[l2], A[l1], t);
                T v = A[l2][t] + jacobi_div(omega * (bb[b2] - acc), bk[b2][4]);
                v = (c_op2 & in_win(j2, lo2, hi2)) ? v : T(0);
                if (in_win(j2, r0, r1) && c_own)
                    pass_store<STREAM>(xout + (int64_t)j2 * N + col, v);
                if (NORM) B[l2][t] = v;
            }
            if (NORM) __syncthreads();
            if (NORM && in_win(j3, r0, r1)) {
                {
                    const T acc = band_row_product(bk[b3], B[l1], B[x3], B[l2], t);
                    const T d = bb[b3] - acc;
                    nacc += c_own ? (double)d * (double)d : 0.0;
                }
                if ((j3 % F_NORM_ROWS) == F_NORM_ROWS - 1 || j3 == r1 - 1) {
                    NS[threadIdx.x] = nacc;
                    nacc = 0.0;
                    pend = j3 / F_NORM_ROWS;
                }
            }
        }
    }
    if (NORM && pend >= 0) {
        __syncthreads();
        flush();
    }
}

}  // namespace dev
}  // namespace mg
