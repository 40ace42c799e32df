// FT-GCR device kernels for gfx950 (MI355X).
//
// One inner step of Algorithm 1 (FT-GCR(k), arXiv 2103.07210) runs as three
// streaming passes over HBM and two one-block reductions (where the columns
// fit the registers of the chip, the resident kernel takes their place):
//
//   update_thomas   r+ = r + beta L(p^nu), <r+, r+> partials, e = P^{-1} r+
//   stencil_dots    L(e) and the partials of <L(e), L(p^l)>, l = 0..nu
//                   (launched before the step's decision: it writes only
//                   its partials and reads nothing the decision changes)
//     finish_step   exit test, monotone-norm fault test, backup or rollback
//                   (Algorithm 1, red part), then
//                   alpha_l = -<L(e), L(p^l)> / <L(p^l), L(p^l)>
//   dir_update      L(p^{nu+1}) (L(e) recomputed), the next beta's inner
//                   products, and at the end of a cycle p^k and the deferred
//                   iterate update phi += sum_l beta_l p^l, both summed over
//                   the cycle's basis p^0, e^1 .. e^k
//     finish_beta   beta, pass and cycle bookkeeping
//
// A step with faults to inject into e takes the decision in a launch of its
// own (finish_col) so the injection can follow it, then finish_alpha after
// the dots pass: the same arithmetic in the same order.
//
// The reductions are separate launches on purpose: a grid-wide "last block
// finishes" scheme needs a device-scope fence and a same-address atomic per
// block, which across the eight XCDs (eight L2s) of MI355X costs far more
// than a launch.  Every reduction is deterministic: fixed per-block partition
// and order, butterfly wave sums (bitwise equal on every lane), fixed
// cross-wave order, then a fixed-order sum over the block partials.  The
// detector's <r, r> is therefore a function of r alone, as the equality case
// of the test needs.
//
// Storage type T is double (FP64 solve) or float (mixed precision: binary32
// vectors, FP64 arithmetic in registers, FP64 inner products and iterate).
#include <hip/hip_ext.h>

#include "device.h"

namespace ftgcr {

enum { MODE_STEP = 0, MODE_INIT = 1, MODE_DEBUG = 2, MODE_GM = 3 };
enum { GM_INIT = 0, GM_CHECK = 1, GM_REDO = 2 };

// Fixed-order sums of values 0..nv-1 over an instance's block partials
// (value-major: a value's partials are contiguous, value q in row row0 + q),
// by one RED_THREADS block:
// thread t adds blocks t, t + RED_THREADS, ... in order, then the waves are
// summed in a fixed order.  Values are taken G at a time, and each thread
// issues the loads of U of its blocks for all G values before the first add,
// so up to G * U * RED_THREADS partials cost one round trip to memory; the
// order of the additions is the same for every (G, U).  The returned LDS
// array holds the nv sums; out, if not null, gets the first two of them in
// registers.  Both are valid in every thread.
// `first`: the first partial's place in its row.
template <int G, int U, typename I>
__device__ __forceinline__ const double* sum_partials(const I& in, int nblk, int row0, int nv, double* out,
                                                      int first = 0)
{
    constexpr int NW = RED_THREADS / 64;
    __shared__ double sh[NV_MAX][NW];
    __shared__ double res[NV_MAX];
    const gptr<double> part = as_global(in.part) + first;
    const long long stride = in.pstride;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int q0 = 0; q0 < nv; q0 += G) {
        double acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = 0.0;
        for (int b0 = threadIdx.x; b0 < nblk; b0 += U * RED_THREADS) {
            double v[U][G];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int b = b0 + u * RED_THREADS;
#pragma unroll
                for (int g = 0; g < G; ++g)
                    v[u][g] = (b < nblk && q0 + g < nv) ? part[(long long)(row0 + q0 + g) * stride + b] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (b0 + u * RED_THREADS < nblk) {
#pragma unroll
                    for (int g = 0; g < G; ++g) acc[g] += v[u][g];
                }
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (q0 + g < nv) {
                const double t = wave_sum(acc[g]);
                if (lane == 0) sh[q0 + g][w] = t;
            }
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < nv) {
        double t = 0.0;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) t += sh[threadIdx.x][ww];
        res[threadIdx.x] = t;
    }
    __syncthreads();
    if (out != nullptr)
        for (int q = 0; q < 2 && q < nv; ++q) out[q] = res[q];
    return res;
}

// (A x) at levels k0 .. k0+KC-1 of column (i, j) (i, j clamped in range,
// k0 < nz), for a whole block: a block is a 64 x 4 tile of columns, one
// wavefront per row (lane = i - tile start), so most neighbours are values
// other lanes already loaded:
//   west / east  the adjacent lanes' centre values, moved by DPP; the row
//                segment's two edge values (one of them the periodic wrap)
//                come from one load instruction, lanes 0..KC-1 west and
//                32..32+KC-1 east, broadcast by readlane;
//   south/north  FP64: the adjacent rows' centre values through LDS, only
//                the tile's first and last rows load a halo row; binary32:
//                each row loads its own south and north rows;
//   below/above  registers (each thread holds its KC levels and one more on
//                either side).
// All loads use clamped in-range addresses and are issued before the first
// is used; missing neighbours (beyond the poles, bottom, top) are selected
// to 0 (a select, not a product, so a NaN at a clamped address cannot leak)
// and carry weight 0.  Entries at levels >= nz or in clamped columns are
// garbage and must be masked by the caller.  `centre`, if given, receives
// x at the KC levels (as loaded).  Every thread of the block must call this
// (the FP64 form holds a barrier).
template <typename TI, int KC>
__device__ __forceinline__ void stencil_chunk(const Geo& g, const TI* __restrict__ x, int i, int j,
                                              int k0, double (&out)[KC], double* centre = nullptr)
{
    static_assert(ST_TX == 64 && ST_TY * ST_TX == ST_THREADS, "one wavefront per tile row");
    static_assert(KC <= 32, "edge lanes");
    using AT = TI;   // arithmetic type: FP64 for FP64 vectors, binary32 for binary32
    __shared__ AT s_row[ST_TY][KC][ST_TX];
    const typename RowOf<AT>::type rc = row_consts_for<AT>(g, i, j);
    const int nz = g.nz, nx = g.nx;
    const long long plane = (long long)g.ncols;
    const int lane = threadIdx.x & (ST_TX - 1);
    const int w = threadIdx.x / ST_TX;
    // tile start (lane 0 is never a clamped column) and the last real lane
    const int i0 = __builtin_amdgcn_readlane(i, 0);
    const int last = (nx - 1 - i0 < ST_TX - 1) ? nx - 1 - i0 : ST_TX - 1;
    const int iw0 = (i0 == 0) ? nx - 1 : i0 - 1;
    const int ie0 = (i0 + last + 1 == nx) ? 0 : i0 + last + 1;
    const bool has_s = j > 0, has_n = j < g.ny - 1;
    const long long row = (long long)j * nx;
    AT xv[KC + 2], xs[KC], xn[KC];
#pragma unroll
    for (int t = 0; t < KC + 2; ++t) {
        int k = k0 - 1 + t;
        k = k < 0 ? 0 : (k > nz - 1 ? nz - 1 : k);
        xv[t] = (AT)x[row + i + plane * k];
    }
    AT edge;
    {
        const int t = lane < 32 ? lane : lane - 32;
        int k = k0 + (t < KC ? t : KC - 1);
        k = k > nz - 1 ? nz - 1 : k;
        edge = (AT)x[row + plane * k + (lane < 32 ? iw0 : ie0)];
    }
    if constexpr (sizeof(AT) == 8) {
        // halo rows of the tile (first row: south, last row: north); the
        // inner rows come from the adjacent waves through LDS
        if (w == 0) {
            const long long so = has_s ? -(long long)nx : 0;
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) {
                const int k = (k0 + kk > nz - 1) ? nz - 1 : k0 + kk;
                xs[kk] = (AT)x[row + so + plane * k + i];
            }
        }
        if (w == ST_TY - 1) {
            const long long no = has_n ? (long long)nx : 0;
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) {
                const int k = (k0 + kk > nz - 1) ? nz - 1 : k0 + kk;
                xn[kk] = (AT)x[row + no + plane * k + i];
            }
        }
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) s_row[w][kk][lane] = xv[kk + 1];
        __syncthreads();
        if (w > 0) {
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) xs[kk] = s_row[w - 1][kk][lane];
        }
        if (w < ST_TY - 1) {
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) xn[kk] = s_row[w + 1][kk][lane];
        }
    } else {
        // binary32: every wave loads its south and north rows itself (the
        // adjacent waves' rows, cache hits); no LDS exchange and no barrier,
        // so no wave waits for the tile's slowest (measured faster in
        // binary32; in FP64 the extra values in flight cost occupancy)
        const long long so = has_s ? -(long long)nx : 0;
        const long long no = has_n ? (long long)nx : 0;
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) {
            const int k = (k0 + kk > nz - 1) ? nz - 1 : k0 + kk;
            xs[kk] = (AT)x[row + so + plane * k + i];
            xn[kk] = (AT)x[row + no + plane * k + i];
        }
    }
    AT xw[KC], xe[KC];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const AT up = lane_shift(xv[kk + 1], 1);
        const AT dn = lane_shift(xv[kk + 1], 0);
        const AT we = lane_read(edge, kk);
        const AT ee = lane_read(edge, 32 + kk);
        xw[kk] = (lane == 0) ? we : up;
        xe[kk] = (lane == last) ? ee : dn;
    }
    // vertical face weights of faces k0 .. k0+KC (level k has faces k, k+1)
    AT wf[KC + 1];
#pragma unroll
    for (int t = 0; t <= KC; ++t) {
        const int f = k0 + t;
        const int fq = f > nz ? nz : f;
        wf[t] = vface(rc, (AT)g.gf[fq], f, nz);
    }
    const AT opsig = (AT)g.opsig;
    const AT zero = AT(0);
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const int k = k0 + kk;
        const int kq = (k > nz - 1) ? nz - 1 : k;
        const AT gk = (AT)g.gc[kq];
        const AT wb = wf[kk], wa = wf[kk + 1];
        const AT xsv = has_s ? xs[kk] : zero;
        const AT xnv = has_n ? xn[kk] : zero;
        const AT xb = (k > 0) ? xv[kk] : zero;
        const AT xa = (k + 1 < nz) ? xv[kk + 2] : zero;
        AT t1 = rc.gx * (xw[kk] + xe[kk]);
        t1 = fma(rc.gys, xsv, t1);
        t1 = fma(rc.gyn, xnv, t1);
        AT t2 = rc.cw * xw[kk];
        t2 = fma(rc.ce, xe[kk], t2);
        t2 = fma(rc.cs, xsv, t2);
        t2 = fma(rc.cn, xnv, t2);
        AT off = fma(gk, t2, t1);
        off = fma(wb, xb, off);
        off = fma(wa, xa, off);
        const AT diag = opsig * ((fma(gk, rc.h1, rc.h0) + wb) + wa);
        out[kk] = (double)fma(diag, xv[kk + 1], -off);
        if (centre) centre[kk] = (double)xv[kk + 1];
    }
}

// Depth of the direction-term load pipeline of the direction pass: the
// loads of term l + TERM_PIPE - 1 are issued before term l is used.
// binary32 loads carry half the bytes and the binary32 kernel has registers
// to spare, so it keeps one more term in flight.  One stage more in either
// form is within the noise (FP64 81.5 vs 82.0 us, binary32 47.8 vs 48.0 on
// 512 x 256 x 64; O160 x 51 53.6 vs 54.4).
template <typename T>
constexpr int TERM_PIPE = sizeof(T) == 4 ? 3 : 2;

// Stencil-grid coordinates of this thread: (i, j) clamped into the grid for
// addressing, `col_ok` whether the thread owns a real column.
struct StPos {
    int i, j, k0;
    bool col_ok;
};

// Block lb of a stencil-grid launch of nct column tiles times tz level
// chunks -> its column tile ct and level chunk bz, in block order `ord`
// (ORD_X: ct fastest; ORD_Z: bz fastest; ORD_XCD: bz fastest after
// renumbering, so that the blocks the hardware places on one die (those
// congruent modulo XCDS) take one contiguous range of the order).  A
// bijection on [0, nct * tz) for every order.
__device__ __forceinline__ void block_tile(int lb, int nct, int tz, int ord, int& ct, int& bz)
{
    if (ord == ORD_X) {
        ct = lb % nct;
        bz = lb / nct;
        return;
    }
    if (ord == ORD_XCD) {
        const int n = nct * tz;
        const int q = n / XCDS, r = n % XCDS, d = lb % XCDS;
        lb = d * q + (d < r ? d : r) + lb / XCDS;
    }
    bz = lb % tz;
    ct = lb / tz;
}

// Lat-lon: a block is a 64 x 4 tile of columns times kc levels.
template <typename T>
__device__ __forceinline__ StPos st_pos(const Inst<T>& in, int lb, int kc, int ord)
{
    StPos p;
    int ct, bz;
    block_tile(lb, in.tx * in.ty, (in.g.nz + kc - 1) / kc, ord, ct, bz);
    const int bx = ct % in.tx;
    const int by = ct / in.tx;
    const int i = bx * ST_TX + (threadIdx.x & (ST_TX - 1));
    const int j = by * ST_TY + (threadIdx.x / ST_TX);
    p.col_ok = i < in.g.nx && j < in.g.ny;
    p.i = i < in.g.nx ? i : in.g.nx - 1;
    p.j = j < in.g.ny ? j : in.g.ny - 1;
    p.k0 = bz * kc;
    return p;
}

// Position on either mesh: lat-lon as above; octahedral (nx = points per
// level, ny = 1): ST_THREADS consecutive points per block, i = the point.
template <int MESH, typename T>
__device__ __forceinline__ StPos st_pos_m(const Inst<T>& in, int lb, int kc, int ord)
{
    if constexpr (MESH == FTGCR_MESH_OCTAHEDRAL) {
        StPos p;
        int bx, bz;
        block_tile(lb, in.tx, (in.g.nz + kc - 1) / kc, ord, bx, bz);
        const int i = bx * ST_THREADS + threadIdx.x;
        p.col_ok = i < in.g.nx;
        p.i = p.col_ok ? i : in.g.nx - 1;
        p.j = 0;
        p.k0 = bz * kc;
        return p;
    } else {
        return st_pos(in, lb, kc, ord);
    }
}

// (A x) at levels k0 .. k0+KC-1 of point c of the octahedral mesh, in the
// same operation order as a lat-lon row (off-diagonal sums of metric and
// metric-times-hill terms, combined with g_k; diagonal h0 + g_k h1 plus the
// vertical faces, as the column solve forms it), neighbours gathered through
// the slot tables; an empty slot contributes a selected 0, not a product.
// The arithmetic runs in the vector type (binary32 vectors: binary32 tables
// and arithmetic, as on the lat-lon mesh).
template <typename TI, int KC>
__device__ __forceinline__ void stencil_oct(const Geo& g, const TI* __restrict__ x, int c, int k0,
                                            double (&out)[KC], double* centre = nullptr)
{
    using AT = TI;
    const int nz = g.nz;
    const long long plane = (long long)g.ncols;
    const AT h0 = oct_tab<AT>(g.oh0, g.oh0_32, c), h1 = oct_tab<AT>(g.oh1, g.oh1_32, c);
    const AT gz = oct_tab<AT>(g.ogz, g.ogz32, c), hc = oct_tab<AT>(g.ohc, g.ohc32, c);
    AT xv[KC + 2], t1[KC], t2[KC];
#pragma unroll
    for (int t = 0; t < KC + 2; ++t) {
        int k = k0 - 1 + t;
        k = k < 0 ? 0 : (k > nz - 1 ? nz - 1 : k);
        xv[t] = x[c + plane * k];
    }
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        t1[kk] = AT(0);
        t2[kk] = AT(0);
    }
#pragma unroll
    for (int q = 0; q < NB_OCT; ++q) {
        const long long slot = (long long)q * g.ncols + c;
        const int nb = g.onb[slot];
        const AT gw = oct_tab<AT>(g.ogw, g.ogw32, slot), hw = oct_tab<AT>(g.ohw, g.ohw32, slot);
        const long long base = nb >= 0 ? nb : c;
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) {
            const int k = (k0 + kk > nz - 1) ? nz - 1 : k0 + kk;
            const AT v = x[base + plane * k];
            const AT vs = nb >= 0 ? v : AT(0);
            t1[kk] = fma(gw, vs, t1[kk]);
            t2[kk] = fma(hw, vs, t2[kk]);
        }
    }
    AT wf[KC + 1];
#pragma unroll
    for (int t = 0; t <= KC; ++t) {
        const int f = k0 + t;
        const int fq = f > nz ? nz : f;
        wf[t] = (f > 0 && f < nz) ? gz * fma(hc, (AT)g.gf[fq], AT(1)) : AT(0);
    }
    const AT opsig = (AT)g.opsig;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const int k = k0 + kk;
        const int kq = (k > nz - 1) ? nz - 1 : k;
        const AT gk = (AT)g.gc[kq];
        const AT wb = wf[kk], wa = wf[kk + 1];
        const AT xb = (k > 0) ? xv[kk] : AT(0);
        const AT xa = (k + 1 < nz) ? xv[kk + 2] : AT(0);
        AT off = fma(gk, t2[kk], t1[kk]);
        off = fma(wb, xb, off);
        off = fma(wa, xa, off);
        const AT diag = opsig * ((fma(gk, h1, h0) + wb) + wa);
        out[kk] = (double)fma(diag, xv[kk + 1], -off);
        if (centre) centre[kk] = (double)xv[kk + 1];
    }
}

// The stencil on either mesh.
template <typename TI, int KC, int MESH>
__device__ __forceinline__ void stencil_m(const Geo& g, const TI* __restrict__ x, const StPos& ps, double (&out)[KC],
                                          double* centre = nullptr)
{
    if constexpr (MESH == FTGCR_MESH_OCTAHEDRAL) {
        stencil_oct<TI, KC>(g, x, ps.i, ps.k0, out, centre);
    } else {
        stencil_chunk<TI, KC>(g, x, ps.i, ps.j, ps.k0, out, centre);
    }
}

template <typename T>
__device__ __forceinline__ void write_xor(T* p, int bit);

template <>
__device__ __forceinline__ void write_xor<double>(double* p, int bit)
{
    atomicXor(reinterpret_cast<unsigned long long*>(p), 1ull << bit);
}

template <>
__device__ __forceinline__ void write_xor<float>(float* p, int bit)
{
    atomicXor(reinterpret_cast<unsigned int*>(p), 1u << bit);
}

// ---------------------------------------------------------------------------
// state setup
// ---------------------------------------------------------------------------

template <typename T>
__global__ void k_init_state(Table<T> tb, int k, int ft, int mixed, long long max_steps, double tol2,
                             int reset_counters)
{
    const int m = blockIdx.x;
    if (m >= tb.n || threadIdx.x != 0) return;
    SolveState* st = tb.inst[m].st;
    // a launch that failed has left words of rounds the state does not count
    if (st->res_fail) st->res_seq += RES_ROUNDS;
    st->res_fail = 0;
    if (reset_counters) {
        st->s = 0;
        st->accepted = 0;
        st->cycles = 0;
        st->detections = 0;
        st->stagnation_accepts = 0;
        st->events_applied = 0;
        st->log_len = 0;
    }
    st->last_rb_pos = -1;
    st->events_since_rb = 1;
    st->status = RUNNING;
    st->active = 0;
    st->nu = 0;
    st->k = k;
    st->ft = ft;
    st->mixed = mixed;
    st->max_steps = max_steps;
    st->tol2 = tol2;
    for (int l = 0; l <= KMAX; ++l) {
        st->slot[l] = l;
        st->d[l] = 0.0;
        st->beta[l] = 0.0;
        st->alpha[l] = 0.0;
        st->xc[l] = 0.0;
    }
    for (int l = 0; l <= KMAX + 1; ++l) st->uslot[l] = l;
    st->bm[0][0] = 1.0;
    st->r_cur = 0;
    st->r_dst = 0;
    st->r_bak = 0;
    st->x_base = 0;
    st->x_base_nu = 0;
    st->x_bak = 0;
    st->x_dst = 0;
    st->x_final_hi = -1;
    st->ev_ok = 0;
}

// Tolerance and step cap of an inner round of the mixed-precision
// refinement: exit when <r,r> <= tau^2 <r_t, r_t>.
template <typename T>
__global__ void k_set_round(Table<T> tb, double tol2, long long max_steps)
{
    const int m = blockIdx.x;
    if (m >= tb.n || threadIdx.x != 0) return;
    SolveState* st = tb.inst[m].st;
    st->tol2 = tol2;
    st->max_steps = max_steps;
    st->T = tol2 * (st->mixed ? st->rt2 : st->RR);
}

// r = A x - R (x = caller's FP64 iterate), stored in R[r_dst] when `store`;
// partials of <R, R> and of the unrounded FP64 <r, r>.
template <typename T, int KC, int MESH>
__global__ __launch_bounds__(ST_THREADS) void k_residual(Table<T> tb, int store)
{
    __shared__ double sh[4];
    const int m = find_inst(tb.blk0_st, tb.n, blockIdx.x);
    const Inst<T>& in = tb.inst[m];
    const int lb = blockIdx.x - tb.blk0_st[m];
    const StPos ps = st_pos_m<MESH>(in, lb, in.kc, in.ord_st);
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    T* rout = in.R[in.st->r_dst];
    const double* rhs = in.rhs;
    double ax[KC], b[KC];
    stencil_m<double, KC, MESH>(in.g, in.X[0], ps, ax);
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
        b[kk] = rhs[c0 + plane * kq];
    }
    double rr = 0.0, bb = 0.0;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const bool ok = ps.col_ok && ps.k0 + kk < nz;
        const double r = ok ? ax[kk] - b[kk] : 0.0;
        const double bv = ok ? b[kk] : 0.0;
        if (ok && store) rout[c0 + plane * (ps.k0 + kk)] = (T)r;
        rr = fma(r, r, rr);
        bb = fma(bv, bv, bb);
    }
    const double sb = block_sum(bb, sh);
    const double sr = block_sum(rr, sh);
    if (threadIdx.x == 0) {
        in.part[(long long)(0) * in.pstride + lb] = sb;
        in.part[(long long)(1) * in.pstride + lb] = sr;
    }
}

template <typename T>
__global__ __launch_bounds__(RED_THREADS) void k_finish_residual(Table<T> tb, int set_T)
{
    const Inst<T>& in = tb.inst[blockIdx.x];
    SolveState* st = in.st;
    double v[2];
    sum_partials<2, 8>(in, in.nblk_st, 0, 2, v);
    const double RR = v[0], rt2 = v[1];
    if (threadIdx.x == 0) {
        st->RR = RR;
        st->rt2 = rt2;
        if (set_T) st->T = st->tol2 * (st->mixed ? rt2 : RR);
    }
}

// ---------------------------------------------------------------------------
// update + column preconditioner (+ the step's decision)
// ---------------------------------------------------------------------------
//
// Each column (i, j) is split between two lanes of a wave (lane l and l+32):
// the lower lane eliminates levels 0 .. h-1 upward (Thomas forward sweep),
// the upper lane levels nz-1 .. h downward; they meet at level h-1, exchange
// one pivot pair by a lane shuffle, and each back-substitutes its half.  The
// elimination state of a half column (at most H levels) stays in registers.
// P's rows: a_k e_{k-1} + b_k e_k + u_k e_{k+1} = r_k with b the diagonal of
// A and a, u minus the vertical face weights.
//
// A lane's rows run from its outer end to the middle: row H - 1 is level h - 1
// (lower) or h (upper), so where the halves meet, and every row after the
// first pad_rows(H), is the same in every column, and only those first rows
// are guarded.  Behind a guard on each row's store of r+ the compiler moved
// every row's elimination after all the stores, and a column that did not
// fill its template exactly ran at one or two waves per SIMD with all rows'
// values in registers; settle() keeps a row's results formed beside its
// loads.  The empty rows (levels a half is short of H) read the outermost
// level's address, take no part in the sums and store nothing.
//
// Bound by memory where the solve exceeds the cache: r and L(p) read, r+ and
// e written, 268 MB in 45 us at 512 x 256 x 64 (6 TB/s).  Columns that do not
// fill their template take no longer per byte: O160 x 51 41.8 -> 33.3 us,
// 700 x 333 x 47 83.6 -> 74.5 us against a guard on every row.

// MODE_GM (FT-GMRES, FP64): the current Arnoldi vector U[j] is divided by
// den[j] (normalised, written back in place) and z_j = P^{-1} v_j goes to
// Z[j]; no norms.
// ANY: the launch's columns may be shorter than the template's range (a batch
// of members of different depths), so every row is guarded.
template <typename T, int H, int mode, bool ANY>
__device__ __forceinline__ void update_thomas_body(Table<T> tb, const T* dbg_in, T* dbg_out, const GmInst* gm)
{
    // The column solve runs in the storage precision: FP64 for FP64 solves;
    // binary32 for the mixed form, where e = P^{-1} r only has to be a fixed
    // preconditioner application (L(e) is formed from the stored e).  The
    // update r+ = r + beta L(p) and both norms stay FP64.
    using CT = T;
    __shared__ double sh[4];
    // per half and row: the vertical decay at the level, and at the face
    // towards the middle with a 1 (both 0 at the bottom and top faces and in
    // empty rows)
    __shared__ CT s_lev[2][H], s_face[2][H][2];
    // Half columns longer than 32 levels: the multipliers of the first LH
    // rows (the last ones the back-substitution reads) wait in LDS, the rest
    // in registers, so that the kernel fits two waves per SIMD (all 48
    // levels in registers take about 370 registers in FP64: one wave)
    constexpr int LH = H > 32 ? (sizeof(CT) == 8 ? 19 : 16) : 0;
    constexpr int RH = H - LH;
    constexpr int PAD = ANY ? H : pad_rows(H);
    __shared__ CT s_stk[LH > 0 ? LH : 1][2][COL_THREADS];
    const int m = find_inst(tb.blk0_col, tb.n, blockIdx.x);
    const Inst<T>& in = tb.inst[m];
    const int lb = blockIdx.x - tb.blk0_col[m];
    SolveState* st = in.st;
    if (mode == MODE_STEP || mode == MODE_INIT) {
        if (st->status != RUNNING) return;
        if (mode == MODE_STEP && st->d_cur == 0.0) return;   // the decision records the breakdown
    }
    if (mode == MODE_GM) {
        if (gm->st->status != RUNNING || !gm->st->active) return;
    }
    // everything read from the instance and the state is copied to registers
    // before the first store, so no later access can wait behind a store
    const Geo& g = in.g;
    const int nx = g.nx, nz = g.nz, ncols = g.ncols;
    const int h = (nz + 1) >> 1;   // lower half: levels [0, h), upper half: [h, nz)
    const double opsig = g.opsig;
    // vertical decay tables in LDS (LDS reads do not queue behind stores)
    for (int t = threadIdx.x; t < 2 * H; t += blockDim.x) {
        const int up = t / H, q = t % H;
        const int a = q - (H - (up ? nz - h : h));   // levels from the outer end
        const int k = up ? nz - 1 - a : a, f = up ? k : k + 1;
        const bool inner = a >= 0 && f > 0 && f < nz;
        s_lev[up][q] = a >= 0 ? (CT)g.gc[k] : CT(0);
        s_face[up][q][0] = inner ? (CT)g.gf[f] : CT(0);
        s_face[up][q][1] = inner ? CT(1) : CT(0);
    }
    const CT opsig_c = (CT)opsig;
    const T* rin;
    const T* ap;
    T* rout;
    T* eout;
    double beta = 0.0;
    double den = 1.0;
    if (mode == MODE_DEBUG) {
        rin = dbg_in;
        ap = dbg_in;
        rout = nullptr;
        eout = dbg_out;
    } else if (mode == MODE_GM) {
        const int jj = gm->st->j;
        rin = (const T*)gm->U[jj];
        ap = rin;
        rout = (T*)gm->U[jj];
        eout = (T*)gm->Z[jj];
        den = gm->st->den[jj];
    } else {
        rin = in.R[st->r_cur];
        eout = in.U[st->uslot[mode == MODE_STEP ? st->nu + 1 : 0]];
        ap = rin;
        rout = nullptr;
        if (mode == MODE_STEP) {
            ap = in.AP[st->slot[st->nu]];
            rout = in.R[st->r_dst];
            beta = -st->beta_num / st->d_cur;
        }
    }
    double* part = in.part;
    const long long pstride = in.pstride;
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const int upper = lane >> 5;
    const int col = lb * COLS_PER_BLOCK + (threadIdx.x >> 6) * 32 + (lane & 31);
    double acc_new = 0.0, acc_st = 0.0;
    if (col < ncols) {   // (both lanes of a column or neither)
        const int j = col / nx;
        const int i = col - j * nx;
        const long long plane = (long long)ncols;
        const int nmine = upper ? nz - h : h;
        const int pad = H - nmine;
        // diagonal h0 + g_k h1 + vertical faces, from the same per-column
        // constants and in the same order as the stencil rows (identical)
        const typename RowOf<CT>::type rcst = col_consts_for<CT>(g, i, j);
        const CT h0 = rcst.h0;
        const CT h1 = rcst.h1;
        const CT gz = rcst.gz, hc = rcst.hc;
        auto face = [&](int q) -> CT { return gz * fma(hc, s_face[upper][q][0], s_face[upper][q][1]); };

        // The half column streams in chunks of CH levels, each chunk's loads
        // issued one chunk ahead of its elimination (a two-stage software
        // pipeline), before the previous chunk's stores, so waiting for them
        // never waits for a store.  The elimination is the same instruction
        // stream for both halves.
        // r is loaded with the non-temporal hint: this is its last use in the
        // step (the direction pass reads r+), and the hint leaves the Infinity
        // Cache to what the next passes re-read (e, r+, the L(p^l)).
        // FP64 streams in 4-level chunks: with 8 the half column's registers
        // exceed 256 and the kernel drops to one wave per SIMD.  binary32 values
        // are half the bytes per load, so it streams 16 levels ahead where the
        // half column allows (more bytes in flight per wave)
        constexpr int CHW = sizeof(T) == 8 ? 4 : (H % 16 == 0 ? 16 : (H % 8 == 0 ? 8 : 4));
        constexpr int CH = H < CHW ? H : CHW;
        constexpr int NCH = H / CH;
        static_assert(H % CH == 0, "chunks must tile the half column");
        T bufr[2][CH], bufa[2][CH];
        CT de[RH], ga[RH];
        CT carry_g = 0, carry_d = 0;
        CT w_out = 0;                // face towards the column's end (0 at the bottom and top)
        CT mk = 1, fk = 0;
        // offsets walk one level per row (a fresh induction value, so no row's
        // 64-bit address need stay live), from the outermost level; a half
        // without rows (one level) stays on level 0
        const long long step = upper ? -plane : plane;
        const long long first = (long long)col + (upper && nmine > 0 ? plane * (nz - 1) : 0);
        const int walk = nmine > 0 ? pad : H;   // rows before this one do not move
        gptr<T> rp = as_global(rin) + first;
        // L(p) relative to r: one walking pointer for both
        const long long to_ap = ((long long)ap - (long long)rin) / (long long)sizeof(T);
        gptr_mut<T> rw = as_global_mut((mode == MODE_STEP || mode == MODE_GM) ? rout : eout) + first;
        asm volatile("" : "+v"(rp), "+v"(rw));
        auto load = [&](int q, T& rv, T& av) {
            rv = __builtin_nontemporal_load(rp);
            av = (mode == MODE_STEP) ? rp[to_ap] : T(0);
            if (q + 1 < H) rp += (q < PAD && q < walk) ? 0 : step;
        };
#pragma unroll
        for (int t = 0; t < CH; ++t) load(t, bufr[0][t], bufa[0][t]);
#pragma unroll
        for (int cb = 0; cb < NCH; ++cb) {
            const int b = cb & 1;
            // keep the pipeline depth at one chunk: without this fence the
            // scheduler hoists every chunk's loads and the half column's raw
            // values all sit in registers at once (occupancy 1)
            __builtin_amdgcn_sched_barrier(0);
            if (cb + 1 < NCH) {
#pragma unroll
                for (int t = 0; t < CH; ++t) load((cb + 1) * CH + t, bufr[b ^ 1][t], bufa[b ^ 1][t]);
            }
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const int q = cb * CH + t;
                const bool mine = q >= PAD || q >= pad;
                const double v = (mode == MODE_STEP) ? fma(beta, (double)bufa[b][t], (double)bufr[b][t])
                                 : (mode == MODE_GM) ? (double)bufr[b][t] / den
                                                     : (double)bufr[b][t];
                const T sv = (T)v;
                const double rp_ = (double)sv;
                if (mode == MODE_STEP || mode == MODE_GM) {
                    if (mine) *rw = sv;
                    rw += (q < PAD && q < walk) ? 0 : step;
                }
                // (selected, not multiplied: an empty row's Inf would leave NaN)
                const double vn = mine ? v : 0.0, vs = mine ? rp_ : 0.0;
                acc_new = fma(vn, vn, acc_new);
                acc_st = fma(vs, vs, acc_st);
                const CT w_in = face(q);
                const CT wb = upper ? w_in : w_out;
                const CT wa = upper ? w_out : w_in;
                const CT diag = opsig_c * ((fma(s_lev[upper][q], h1, h0) + wb) + wa);
                mk = diag + w_out * carry_g;
                fk = (CT)sv + w_out * carry_d;
                // binary32 column solve: the hardware reciprocal (about 1 ulp;
                // the preconditioner only has to be a fixed operator); FP64:
                // the correctly rounded quotient
                CT inv;
                if constexpr (sizeof(CT) == 4) inv = __builtin_amdgcn_rcpf(mk);
                else inv = CT(1) / mk;
                // (an empty row leaves 0: the next row's outer face is 0 too)
                carry_g = mine ? -w_in * inv : CT(0);
                carry_d = mine ? fk * inv : CT(0);
                w_out = w_in;
                if (q < LH) {
                    s_stk[q < LH ? q : 0][0][threadIdx.x] = carry_g;
                    s_stk[q < LH ? q : 0][1][threadIdx.x] = carry_d;
                } else {
                    ga[q - LH] = carry_g;
                    de[q - LH] = carry_d;
                    settle(ga[q - LH]);
                    settle(de[q - LH]);
                }
            }
        }
        // meeting row (the lower lane's last): the lower lane gets (zeta_h,
        // eps_h) from its upper partner
        const CT zx = __shfl_xor(carry_g, 32);
        const CT ex = __shfl_xor(carry_d, 32);
        const CT xm = (fk + w_out * ex) / (mk + w_out * zx);
        const CT xl = __shfl_xor(xm, 32);
        // back-substitution: the lower lane from the meeting value at row
        // H - 1 outward, the upper lane from its row H - 1 on
        CT xv = upper ? carry_d - carry_g * xl : xm;
        gptr_mut<T> ep = as_global_mut(eout) + (long long)col + plane * (upper ? h : h - 1);
        asm volatile("" : "+v"(ep));
        if (!(upper && nmine == 0)) *ep = (T)xv;
#pragma unroll
        for (int q = H - 2; q >= 0; --q) {
            CT gq, dq;
            if (q < LH) {
                gq = s_stk[q < LH ? q : 0][0][threadIdx.x];
                dq = s_stk[q < LH ? q : 0][1][threadIdx.x];
            } else {
                gq = ga[q - LH];
                dq = de[q - LH];
            }
            xv = dq - gq * xv;
            ep -= step;
            if (q >= PAD || q >= pad) *ep = (T)xv;
        }
    }
    if (mode == MODE_DEBUG || mode == MODE_GM) return;
    const double sn = block_sum(acc_new, sh);
    const double ss = block_sum(acc_st, sh);
    if (threadIdx.x == 0) {
        part[(long long)(0) * pstride + lb] = sn;
        part[(long long)(1) * pstride + lb] = ss;
    }
}

// Two waves per SIMD (the longest columns need the hint to stay within 256
// registers)
template <typename T, int H, int mode, bool ANY = false>
__global__ __launch_bounds__(COL_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_update_thomas(
    Table<T> tb, const T* dbg_in, T* dbg_out)
{
    update_thomas_body<T, H, mode, ANY>(tb, dbg_in, dbg_out, nullptr);
}

template <int H>
__global__ __launch_bounds__(COL_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void k_update_thomas_gm(
    Table<double> tb, const GmInst* gm)
{
    update_thomas_body<double, H, MODE_GM, false>(tb, nullptr, nullptr, gm);
}

// The binary32 column pass with one lane per column (256 columns per
// block), for columns of at most NZ = 64 levels.  The two-lane kernel above
// needs more registers per lane in binary32 than fit four waves per SIMD, so
// its 4096 waves on 512 x 256 columns take 1.33 rounds of the chip at three
// per SIMD; with one lane per column there are half as many waves, which fit
// in one round at two per SIMD, and every load is a full 256-byte wave
// segment.  settle() beside each row's loads holds it at 155 registers (246
// without: 27.4 -> 24.9 us on 512 x 256 x 64).  Same update, norms, faces, diagonal and elimination as above
// (the lower lane's order, extended to the whole column), so P is the same
// fixed operator up to rounding.
template <typename T, int NZ, int mode>
__global__ __launch_bounds__(COL_THREADS) void k_update_thomas1(Table<T> tb)
{
    static_assert(sizeof(T) == 4 && NZ % 8 == 0, "binary32, whole chunks");
    using CT = T;
    __shared__ double sh[4];
    __shared__ CT s_gc[NZ];
    __shared__ CT s_gf[NZ + 1];
    const int m = find_inst(tb.blk0_col, tb.n, blockIdx.x);
    const Inst<T>& in = tb.inst[m];
    const int lb = blockIdx.x - tb.blk0_col[m];
    SolveState* st = in.st;
    if (st->status != RUNNING) return;
    if (mode == MODE_STEP && st->d_cur == 0.0) return;   // the decision records the breakdown
    const Geo& g = in.g;
    const int nx = g.nx, nz = g.nz, ncols = g.ncols;
    for (int t = threadIdx.x; t < nz; t += blockDim.x) s_gc[t] = (CT)g.gc[t];
    for (int t = threadIdx.x; t <= nz; t += blockDim.x) s_gf[t] = (CT)g.gf[t];
    const CT opsig_c = (CT)g.opsig;
    const T* rin = in.R[st->r_cur];
    const T* ap = rin;
    T* rout = nullptr;
    double beta = 0.0;
    if (mode == MODE_STEP) {
        ap = in.AP[st->slot[st->nu]];
        rout = in.R[st->r_dst];
        beta = -st->beta_num / st->d_cur;
    }
    T* eout = in.U[st->uslot[mode == MODE_STEP ? st->nu + 1 : 0]];
    double* part = in.part;
    const long long pstride = in.pstride;
    __syncthreads();

    const int col = lb * COL_THREADS + threadIdx.x;
    const bool valid = col < ncols;
    const int colc = valid ? col : 0;
    const int j = colc / nx;
    const int i = colc - j * nx;
    const long long plane = (long long)ncols;
    const RowCf rcst = col_consts_for<float>(g, i, j);
    const CT h0 = rcst.h0;
    const CT h1 = rcst.h1;
    const CT gz = rcst.gz, hc = rcst.hc;

    // levels stream in 8-level chunks, each chunk's loads issued one chunk
    // ahead (as in the two-lane kernel); r is read with the non-temporal
    // hint (its last use in the step)
    constexpr int CH = 8;
    constexpr int NCH = NZ / CH;
    T bufr[2][CH], bufa[2][CH];
    CT de[NZ], ga[NZ];
    double acc_new = 0.0, acc_st = 0.0;
    CT carry_g = 0, carry_d = 0;
    CT w_near = 0;   // face below level 0
    gptr_mut<T> rw = as_global_mut(mode == MODE_STEP ? rout : eout) + (long long)colc;
    asm volatile("" : "+v"(rw));
#pragma unroll
    for (int t = 0; t < CH; ++t) {
        const int k = t > nz - 1 ? nz - 1 : t;
        const long long o = (long long)colc + plane * k;
        bufr[0][t] = __builtin_nontemporal_load(&rin[o]);
        bufa[0][t] = (mode == MODE_STEP) ? ap[o] : T(0);
    }
#pragma unroll
    for (int cb = 0; cb < NCH; ++cb) {
        const int b = cb & 1;
        __builtin_amdgcn_sched_barrier(0);
        if (cb + 1 < NCH) {
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                int k = (cb + 1) * CH + t;
                k = k > nz - 1 ? nz - 1 : k;
                const long long o = (long long)colc + plane * k;
                bufr[b ^ 1][t] = __builtin_nontemporal_load(&rin[o]);
                bufa[b ^ 1][t] = (mode == MODE_STEP) ? ap[o] : T(0);
            }
        }
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            const int q = cb * CH + t;   // level
            const bool mine = q < nz;
            const int k = q > nz - 1 ? nz - 1 : q;
            const double v = (mode == MODE_STEP) ? fma(beta, (double)bufa[b][t], (double)bufr[b][t])
                                                 : (double)bufr[b][t];
            const T sv = (T)v;
            const double rp = (double)sv;
            const CT rc = (CT)sv;
            if (mine && valid) {
                if (mode == MODE_STEP) *rw = sv;
                acc_new = fma(v, v, acc_new);
                acc_st = fma(rp, rp, acc_st);
            }
            rw += plane;
            const int f = k + 1;
            const CT gff = s_gf[f];
            const CT w_far = (f > 0 && f < nz) ? gz * fma(hc, gff, CT(1)) : CT(0);
            const CT wb = w_near, wa = w_far;
            w_near = w_far;
            const CT diag = opsig_c * ((fma(s_gc[k], h1, h0) + wb) + wa);
            const CT near = -wb;
            const CT far = -wa;
            const CT mk = (q == 0) ? diag : diag - near * carry_g;
            const CT fk = (q == 0) ? rc : rc - near * carry_d;
            const CT inv = __builtin_amdgcn_rcpf(mk);
            const CT g_new = far * inv;
            const CT d_new = fk * inv;
            if (mine) {
                carry_g = g_new;
                carry_d = d_new;
            }
            ga[q] = g_new;
            de[q] = d_new;
            settle(ga[q]);
            settle(de[q]);
        }
    }
    // back-substitution from the top level down
    CT xv = carry_d;
    gptr_mut<T> ep = as_global_mut(eout) + (long long)colc + plane * (nz - 1);
    asm volatile("" : "+v"(ep));
    if (valid) *ep = (T)xv;
    ep -= plane;
#pragma unroll
    for (int q = NZ - 2; q >= 0; --q) {
        if (q < nz - 1) {
            xv = de[q] - ga[q] * xv;
            if (valid) *ep = (T)xv;
            ep -= plane;
        }
    }
    const double sn = block_sum(acc_new, sh);
    const double ss = block_sum(acc_st, sh);
    if (threadIdx.x == 0) {
        part[(long long)(0) * pstride + lb] = sn;
        part[(long long)(1) * pstride + lb] = ss;
    }
}

// No preconditioner (P = I): the column pass's update, stored r+ and norms,
// with e = r+ (MODE_GM: v_j normalised and z_j = v_j; MODE_DEBUG: out = in).
// It runs on the column grid (cpb columns per block, all their levels), so
// the decision kernels read the same partial rows.
template <typename T, int mode>
__global__ __launch_bounds__(COL_THREADS) void k_update_copy(Table<T> tb, const T* dbg_in, T* dbg_out,
                                                             const GmInst* gm, int cpb)
{
    __shared__ double sh[4];
    const int m = find_inst(tb.blk0_col, tb.n, blockIdx.x);
    const Inst<T>& in = tb.inst[m];
    const int lb = blockIdx.x - tb.blk0_col[m];
    SolveState* st = in.st;
    if (mode == MODE_STEP || mode == MODE_INIT) {
        if (st->status != RUNNING) return;
        if (mode == MODE_STEP && st->d_cur == 0.0) return;   // the decision records the breakdown
    }
    if (mode == MODE_GM) {
        if (gm->st->status != RUNNING || !gm->st->active) return;
    }
    const T* rin;
    const T* ap = nullptr;
    T* rout = nullptr;
    T* eout;
    double beta = 0.0, den = 1.0;
    if (mode == MODE_DEBUG) {
        rin = dbg_in;
        eout = dbg_out;
    } else if (mode == MODE_GM) {
        const int jj = gm->st->j;
        rin = (const T*)gm->U[jj];
        rout = (T*)gm->U[jj];
        eout = (T*)gm->Z[jj];
        den = gm->st->den[jj];
    } else {
        rin = in.R[st->r_cur];
        eout = in.U[st->uslot[mode == MODE_STEP ? st->nu + 1 : 0]];
        if (mode == MODE_STEP) {
            ap = in.AP[st->slot[st->nu]];
            rout = in.R[st->r_dst];
            beta = -st->beta_num / st->d_cur;
        }
    }
    const int ncols = in.g.ncols, nz = in.g.nz;
    const long long plane = (long long)ncols;
    const int c0 = lb * cpb;
    const int cols = ncols - c0 < cpb ? ncols - c0 : cpb;
    double acc_new = 0.0, acc_st = 0.0;
    for (int t = threadIdx.x; t < cpb * nz; t += COL_THREADS) {
        const int q = t % cpb, k = t / cpb;
        if (q >= cols) continue;
        const long long o = (long long)(c0 + q) + plane * k;
        const double v = (mode == MODE_STEP) ? fma(beta, (double)ap[o], (double)rin[o])
                         : (mode == MODE_GM) ? (double)rin[o] / den
                                             : (double)rin[o];
        const T sv = (T)v;
        const double rp = (double)sv;
        if (mode == MODE_STEP || mode == MODE_GM) rout[o] = sv;
        eout[o] = sv;
        acc_new = fma(v, v, acc_new);
        acc_st = fma(rp, rp, acc_st);
    }
    if (mode == MODE_DEBUG || mode == MODE_GM) return;
    const double sn = block_sum(acc_new, sh);
    const double ss = block_sum(acc_st, sh);
    if (threadIdx.x == 0) {
        in.part[(long long)(0) * in.pstride + lb] = sn;
        in.part[(long long)(1) * in.pstride + lb] = ss;
    }
}

template <typename T>
__global__ __launch_bounds__(RED_THREADS) void k_finish_col(Table<T> tb, int mode)
{
    const Inst<T>& in = tb.inst[blockIdx.x];
    SolveState* st = in.st;
    if (st->status != RUNNING) return;
    double v[2];
    sum_partials<2, 8>(in, in.nblk_col, 0, 2, v);
    const double rn = v[0], rs = v[1];
    if (threadIdx.x == 0) {
        if (mode == MODE_STEP) decide_step(st, st->log, rn, rs, in.hist, in.hist_cap);
        else decide_init(st, rn, rs);
    }
}

// <r, r> and the backup's <r, r>, summed as the column pass sums them (cpb
// columns per block; two lanes per column from its ends at COLS_PER_BLOCK,
// else one upward), after steps of the resident kernel, which adds in another
// order: a step that leaves r unchanged (beta = 0 after an overflow) has to
// find its norm unchanged to the last bit.
template <typename T>
__global__ __launch_bounds__(COL_THREADS) void k_norms(Table<T> tb, int cpb)
{
    __shared__ double sh[4];
    const Inst<T>& in = tb.inst[0];
    const SolveState* st = in.st;
    if (st->status != RUNNING) return;
    const int lb = blockIdx.x, lane = threadIdx.x & 63;
    const int ncols = in.g.ncols, nz = in.g.nz;
    const bool two = cpb == COLS_PER_BLOCK;
    const bool upper = two && lane >= 32;
    const int col = lb * cpb + (two ? (threadIdx.x >> 6) * 32 + (lane & 31) : threadIdx.x);
    const int h = (nz + 1) >> 1;
    const int rows = col < ncols ? (!two ? nz : (upper ? nz - h : h)) : 0;
    const T* r = in.R[st->r_cur];
    const T* b = in.R[st->r_bak];
    double ar = 0.0, ab = 0.0;
    for (int q = 0; q < rows; ++q) {
        const long long o = (long long)col + (long long)ncols * (upper ? nz - 1 - q : q);
        const double rv = (double)r[o], bv = (double)b[o];
        ar = fma(rv, rv, ar);
        ab = fma(bv, bv, ab);
    }
    const double sr = block_sum(ar, sh);
    const double sb = block_sum(ab, sh);
    if (threadIdx.x == 0) {
        in.part[lb] = sr;
        in.part[in.pstride + lb] = sb;
    }
}

template <typename T>
__global__ __launch_bounds__(RED_THREADS) void k_finish_norms(Table<T> tb)
{
    const Inst<T>& in = tb.inst[0];
    SolveState* st = in.st;
    if (st->status != RUNNING) return;
    double v[2];
    sum_partials<2, 8>(in, in.nblk_col, 0, 2, v);
    if (threadIdx.x == 0) {
        st->rr_old = v[0];
        st->b_rr = v[1];
    }
}

// ---------------------------------------------------------------------------
// L(e) and orthogonalisation inner products (+ alpha)
// ---------------------------------------------------------------------------

// spec = 1: launched before the step's decision (k_finish_step takes it
// afterwards); it runs whenever the column pass ran, and its partials are
// discarded if the step is rejected or ends the solve.  Nothing it reads
// (nu, the slots, e, the L(p^l)) is changed by the decision.
template <typename T, int KC, int MESH>
__global__ __launch_bounds__(ST_THREADS) void k_stencil_dots(Table<T> tb, int spec)
{
    __shared__ double sh[KMAX + 1][4];
    __shared__ const T* s_ap[KMAX + 1];
    const int m = find_inst(tb.blk0_st, tb.n, blockIdx.x);
    const Inst<T>& in = tb.inst[m];
    const int lb = blockIdx.x - tb.blk0_st[m];
    SolveState* st = in.st;
    if (st->status != RUNNING || (spec ? st->d_cur == 0.0 : !st->active)) return;
    const int nu = st->nu;
    if ((int)threadIdx.x <= nu) s_ap[threadIdx.x] = in.AP[st->slot[threadIdx.x]];
    __syncthreads();
    const StPos ps = st_pos_m<MESH>(in, lb, in.kc, in.ord_st);
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    double le[KC];
    stencil_m<T, KC, MESH>(in.g, in.U[st->uslot[nu + 1]], ps, le);
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const bool ok = ps.col_ok && ps.k0 + kk < nz;
        // octahedral mesh: L(e) kept for the direction pass (exact in T: the
        // stencil rounds to T's precision, so the direction pass starts from
        // the same value as if it had formed L(e) itself)
        if constexpr (MESH == FTGCR_MESH_OCTAHEDRAL)
            if (ok) in.LE[c0 + plane * (ps.k0 + kk)] = (T)le[kk];
        if (!ok) le[kk] = 0.0;
    }
    // every <L(e), L(p^l)>, one uniform branch per l; the loads of term
    // l + 1 are issued before term l's values are used (a two-stage
    // pipeline), so the terms cost one memory round trip together, not one
    // each
    // (two buffers alternating with the parity of l, which is a compile-time
    // constant after unrolling: no register copies, so the wait for term l
    // comes after term l + 1's loads are issued)
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // PD - 1 terms in flight ahead of the one in use (a deeper pipeline
    // costs this pass occupancy without a gain, measured in both forms).  On
    // the octahedral mesh the pass is a chain of round trips (state, slot
    // tables, gathers, terms) at two waves per SIMD: O160 x 51 in FP64 68 us
    // for 236 MB.  More waves by fewer registers spill (81 us at three, 130 at
    // four), 4 levels a block take 66, the tables held over a loop of level
    // chunks 74 to 84.
    constexpr int PD = 2;
    T buf[PD][KC];
#pragma unroll
    for (int l0 = 0; l0 < PD - 1; ++l0) {
        if (l0 == 0 || l0 <= nu) {   // nu >= 0 here
            const gptr<T> apn = as_global(s_ap[l0]);
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) {
                const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                buf[l0][kk] = apn[c0 + plane * kq];
            }
        }
    }
#pragma unroll
    for (int l = 0; l <= KMAX; ++l) {
        if (l <= nu) {
            double acc = 0.0;
            const int ln = l + PD - 1;
            if (ln <= KMAX && ln <= nu) {
                const gptr<T> apn = as_global(s_ap[ln]);
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                    buf[ln % PD][kk] = apn[c0 + plane * kq];
                }
            }
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) {
                const bool ok = ps.col_ok && ps.k0 + kk < nz;
                acc = fma(le[kk], ok ? (double)buf[l % PD][kk] : 0.0, acc);
            }
            // this term's wave sum now, while the next term's loads are in
            // flight (binary32 dots 27.4 -> 26.6 us on 512 x 256 x 64)
            const double v = wave_sum(acc);
            if (lane == 0) sh[l][w] = v;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x <= nu) {
        const int l = threadIdx.x;
        in.part[(long long)(DOT_ROW0 + l) * in.pstride + lb] = ((sh[l][0] + sh[l][1]) + sh[l][2]) + sh[l][3];
    }
}

// The partials of a large grid's dots (dir = 0) or direction pass (1) to
// RED_FOLD per value, kept behind them in their rows, before the one-block
// reduction: one CU takes in about 42 GB/s of partials, whatever it keeps in
// flight.  On 1024 x 512 x 96 (24576 and 49152 blocks) the two reductions take
// 10 us and this 9, against 35 in one block each (a step 1206 -> 1186 us, in
// binary32 685 -> 667); on 1024 x 512 x 36 (18432 blocks in the direction pass
// alone) a step 483.6 -> 481.2.
// Block (x, y): part x of value y.
template <typename T>
__global__ __launch_bounds__(ST_THREADS) void k_fold(Table<T> tb, int dir)
{
    __shared__ double sh[4];
    const Inst<T>& in = tb.inst[0];
    const SolveState* st = in.st;
    if (st->status != RUNNING) return;
    const int nblk = dir ? in.nblk_dir : in.nblk_st, parts = dir ? in.fold_dir : in.fold_st;
    const int q = blockIdx.y;
    if (q >= (dir ? 2 : st->nu + 1)) return;
    double* row = in.part + (long long)((dir ? 0 : DOT_ROW0) + q) * in.pstride;
    const gptr<double> from = as_global((const double*)row);
    const int per = (nblk + parts - 1) / parts;
    const int b1 = min(nblk, ((int)blockIdx.x + 1) * per);
    double acc = 0.0;
    constexpr int U = 4;
    for (int b = blockIdx.x * per + threadIdx.x; b < b1; b += U * ST_THREADS) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = b + u * ST_THREADS < b1 ? from[b + u * ST_THREADS] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (b + u * ST_THREADS < b1) acc += v[u];
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) row[nblk + blockIdx.x] = acc;
}

// alpha_l = -<L(e), L(p^l)> / <L(p^l), L(p^l)>, the new direction over the
// basis (p^{nu+1} = e + sum_l alpha_l p^l), at a cycle's end the iterate
// update over the basis, and the iterate buffer the direction pass writes;
// every thread of the block calls it.
template <typename T>
__device__ __forceinline__ void finish_alpha_body(const Inst<T>& in, SolveState* st)
{
    const int nu = st->nu;
    const double* v = sum_partials<4, 4>(in, in.fold_st ? in.fold_st : in.nblk_st, DOT_ROW0, nu + 1, nullptr,
                                         in.fold_st ? in.nblk_st : 0);
    if ((int)threadIdx.x <= nu) st->alpha[threadIdx.x] = -v[threadIdx.x] / st->d[threadIdx.x];
    __syncthreads();
    basis_row(st, nu, threadIdx.x);
    if (threadIdx.x == 0) st->x_dst = (st->x_base == st->x_bak) ? 1 - st->x_base : st->x_base;
}

template <typename T>
__global__ __launch_bounds__(RED_THREADS) void k_finish_alpha(Table<T> tb)
{
    const Inst<T>& in = tb.inst[blockIdx.x];
    SolveState* st = in.st;
    if (st->status != RUNNING || !st->active) return;
    finish_alpha_body(in, st);
}

// The step's decision (k_finish_col) and, if the step goes on, its alpha
// (k_finish_alpha) in one launch, after a speculative dots pass.
template <typename T>
__global__ __launch_bounds__(RED_THREADS) void k_finish_step(Table<T> tb)
{
    __shared__ SolveState s_st;
    const Inst<T>& in = tb.inst[blockIdx.x];
    SolveState* gst = in.st;
    // the state's words and the column pass's partials in one round trip
    // (the partials of a solve that is no longer running are read and
    // ignored)
    const long long word = state_word_load(gst);
    const int status = gst->status;   // not the staged one: thread 0 changes that one below, without a barrier
    double v[2];
    sum_partials<2, 8>(in, in.nblk_col, 0, 2, v);
    state_word_stage(&s_st, word);
    __syncthreads();
    SolveState* st = &s_st;
    if (status != RUNNING) return;
    if (threadIdx.x == 0) decide_step(st, gst->log, v[0], v[1], in.hist, in.hist_cap);
    __syncthreads();
    if (st->status == RUNNING && st->active) finish_alpha_body(in, st);
    __syncthreads();
    state_word_store(gst, st);
}

// ---------------------------------------------------------------------------
// new direction, its image, next beta's inner products, deferred iterate
// ---------------------------------------------------------------------------

// The directions are not formed step by step: p^{nu+1} = e + sum_l alpha_l p^l
// is a row of bm over the cycle's basis, so the pass forms L(p^{nu+1}) alone
// and, in the last pass of a cycle, p^k (which opens the next cycle) and the
// iterate from the basis at once: nu + 4 vectors a pass and k + 3 a cycle,
// against 2 nu + 6 and 2 with every p^l stored and summed.
//
// Cache hints: the basis vectors, the iterate and p^k are next touched a
// whole step later or more (more than the Infinity Cache holds in between), so
// they are loaded and stored with the non-temporal hint, leaving the cache
// to e, r+ and L(p^{nu+1}), which the next passes read within the step.
// NTAP extends the hint to the L(p^l) loads: set when the solve's k + 1
// images of A p do not fit the cache anyway (otherwise the next dots pass
// finds them there).
//
// Bound by memory.  On 512 x 256 x 64 at k = 4, in FP64, this pass takes 82.0
// us against 100.4 with stored directions; the dots and column passes 49.7 and
// 45.3 against 46.2 and 42.8, since e now goes to k + 2 buffers in turn and
// the cache absorbs fewer of its writes (a solve 72.5 -> 68.0 ms; binary32
// vectors 1.10x).
template <typename T, int KC, bool NTAP, int MESH>
__global__ __launch_bounds__(ST_THREADS) void k_dir_update(Table<T> tb, int init)
{
    __shared__ double sh[4];
    __shared__ const T* s_u[KMAX + 1];
    __shared__ const T* s_ap[KMAX + 1];
    __shared__ double s_al[KMAX + 1];
    __shared__ double s_pk[KMAX + 1];
    __shared__ double s_xc[KMAX + 1];
    const int m = find_inst(tb.blk0_dir, tb.n, blockIdx.x);
    const Inst<T>& in = tb.inst[m];
    const int lb = blockIdx.x - tb.blk0_dir[m];
    SolveState* st = in.st;
    if (st->status != RUNNING) return;
    if (!init && !st->active) return;
    const int nu = init ? -1 : st->nu;
    const bool last = !init && (nu == st->k - 1);
    const T* ein = in.U[st->uslot[nu + 1]];
    T* pout = in.U[st->uslot[last ? nu + 2 : 0]];
    T* apout = in.AP[st->slot[nu + 1]];
    const T* rv = in.R[st->r_cur];
    const double* xb = in.X[st->x_base];
    double* xo = in.X[st->x_dst];
    if ((int)threadIdx.x <= nu) {
        s_u[threadIdx.x] = in.U[st->uslot[threadIdx.x]];
        s_ap[threadIdx.x] = in.AP[st->slot[threadIdx.x]];
        s_al[threadIdx.x] = st->alpha[threadIdx.x];
        s_pk[threadIdx.x] = last ? st->bm[nu + 1][threadIdx.x] : 0.0;
        s_xc[threadIdx.x] = last ? st->xc[threadIdx.x] : 0.0;
    }
    __syncthreads();
    const StPos ps = st_pos_m<MESH>(in, lb, in.kc_dir, in.ord_dir);
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    double a[KC], p[KC], r[KC];
    // On the octahedral mesh the step's dots pass has stored L(e): it is
    // loaded instead of gathering six neighbours again (the first direction
    // of a solve or round, with no dots pass before it, forms it)
    bool formed = false;
    if constexpr (MESH == FTGCR_MESH_OCTAHEDRAL) {
        if (!init) {
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) {
                const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                const long long c = c0 + plane * kq;
                p[kk] = last ? (double)ein[c] : 0.0;
                a[kk] = (double)in.LE[c];
            }
            formed = true;
        }
    }
    // p starts from e: the stencil's own centre values (no second load)
    if (!formed) stencil_m<T, KC, MESH>(in.g, ein, ps, a, p);
    // r is needed only for the next beta's products at the end: binary32
    // loads it there (the registers it frees give that kernel a sixth wave
    // per SIMD); FP64 loads it here (there a late load is slower, the
    // occupancy being the same)
    constexpr bool R_LATE = sizeof(T) == 4;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
        if constexpr (!R_LATE) r[kk] = (double)rv[c0 + plane * kq];
    }
    // sums over l in ascending order; term l + 1's loads are issued before
    // term l's values are used (two-stage pipeline, as in the dots pass)
    constexpr int PD = TERM_PIPE<T>;
    T ab[PD][KC];
#pragma unroll
    for (int l0 = 0; l0 < PD - 1; ++l0) {
        if (l0 <= nu) {
            const gptr<T> apn = as_global(s_ap[l0]);
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) {
                const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                ab[l0][kk] = NTAP ? __builtin_nontemporal_load(&apn[c0 + plane * kq]) : apn[c0 + plane * kq];
            }
        }
    }
#pragma unroll
    for (int l = 0; l < KMAX; ++l) {
        if (l <= nu) {
            const double al = s_al[l];
            const int ln = l + PD - 1;
            if (ln < KMAX && ln <= nu) {
                const gptr<T> apn = as_global(s_ap[ln]);
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                    ab[ln % PD][kk] = NTAP ? __builtin_nontemporal_load(&apn[c0 + plane * kq])
                                           : apn[c0 + plane * kq];
                }
            }
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) a[kk] = fma(al, (double)ab[l % PD][kk], a[kk]);
        }
    }
    if constexpr (R_LATE) {
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) {
            const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
            r[kk] = (double)rv[c0 + plane * kq];
        }
    }
    double acc_num = 0.0, acc_d = 0.0;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const bool ok = ps.col_ok && ps.k0 + kk < nz;
        const T as_ = (T)a[kk];
        if (ok) apout[c0 + plane * (ps.k0 + kk)] = as_;
        const double ad = ok ? (double)as_ : 0.0;
        const double rd = ok ? r[kk] : 0.0;
        acc_num = fma(rd, ad, acc_num);
        acc_d = fma(ad, ad, acc_d);
    }
    if (last) {
        // p^k and the iterate: sums over the basis in ascending order, the
        // iterate's update by itself, so that it is rounded once a cycle and
        // not once a term
        double xa[KC], xd[KC];
        T ub[2][KC];
        const gptr<T> u0 = as_global(s_u[0]);
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) {
            const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
            xa[kk] = __builtin_nontemporal_load(&xb[c0 + plane * kq]);
            xd[kk] = 0.0;
            ub[0][kk] = __builtin_nontemporal_load(&u0[c0 + plane * kq]);
        }
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
            if (j <= nu) {
                if (j + 1 < KMAX && j + 1 <= nu) {
                    const gptr<T> un = as_global(s_u[j + 1]);
#pragma unroll
                    for (int kk = 0; kk < KC; ++kk) {
                        const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                        ub[(j + 1) & 1][kk] = __builtin_nontemporal_load(&un[c0 + plane * kq]);
                    }
                }
                const double pj = s_pk[j], xj = s_xc[j];
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    p[kk] = fma(pj, (double)ub[j & 1][kk], p[kk]);
                    xd[kk] = fma(xj, (double)ub[j & 1][kk], xd[kk]);
                }
            }
        }
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) {
            if (ps.col_ok && ps.k0 + kk < nz) {
                const long long c = c0 + plane * (ps.k0 + kk);
                __builtin_nontemporal_store((T)p[kk], &pout[c]);
                __builtin_nontemporal_store(xa[kk] + xd[kk], &xo[c]);
            }
        }
    }
    const double sn = block_sum(acc_num, sh);
    const double sd = block_sum(acc_d, sh);
    if (threadIdx.x == 0) {
        in.part[(long long)(0) * in.pstride + lb] = sn;
        in.part[(long long)(1) * in.pstride + lb] = sd;
    }
}

template <typename T>
__global__ __launch_bounds__(RED_THREADS) void k_finish_beta(Table<T> tb, int init)
{
    __shared__ SolveState s_st;
    const Inst<T>& in = tb.inst[blockIdx.x];
    SolveState* gst = in.st;
    const long long word = state_word_load(gst);
    const int status = gst->status, active = gst->active;   // not the staged ones: see k_finish_step
    double v[2];
    sum_partials<2, 8>(in, in.fold_dir ? in.fold_dir : in.nblk_dir, 0, 2, v, in.fold_dir ? in.nblk_dir : 0);
    state_word_stage(&s_st, word);
    __syncthreads();
    SolveState* st = &s_st;
    if (status != RUNNING || (!init && !active)) return;
    if (threadIdx.x == 0) decide_beta(st, v[0], v[1], init);
    __syncthreads();
    state_word_store(gst, st);
}

// x = x_base + sum_{l = x_base_nu .. x_final_hi} beta_l p^l (over the basis),
// into X[0].
template <typename T, int KC, int MESH>
__global__ __launch_bounds__(ST_THREADS) void k_finalize_x(Table<T> tb)
{
    const int m = find_inst(tb.blk0_st, tb.n, blockIdx.x);
    const Inst<T>& in = tb.inst[m];
    const int lb = blockIdx.x - tb.blk0_st[m];
    const SolveState* st = in.st;
    const int lo = st->x_base_nu, hi = st->x_final_hi;
    if (st->x_base == 0 && hi < lo) return;
    __shared__ double s_c[KMAX + 1];
    __shared__ const T* s_u[KMAX + 1];
    if ((int)threadIdx.x <= hi) {
        s_c[threadIdx.x] = basis_coef(st, threadIdx.x, lo, hi);
        s_u[threadIdx.x] = in.U[st->uslot[threadIdx.x]];
    }
    __syncthreads();
    const StPos ps = st_pos_m<MESH>(in, lb, in.kc, in.ord_st);
    if (!ps.col_ok) return;
    const double* xb = in.X[st->x_base];
    double* xo = in.X[0];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        if (ps.k0 + kk < in.g.nz) {
            const long long c = (long long)ps.i + (long long)in.g.nx * ps.j + (long long)in.g.ncols * (ps.k0 + kk);
            double xd = 0.0;
            if (hi >= lo)
                for (int j = 0; j <= hi; ++j) xd = fma(s_c[j], (double)as_global(s_u[j])[c], xd);
            xo[c] = xb[c] + xd;
        }
    }
}

// ---------------------------------------------------------------------------
// fault events (harness): prepare target buffers, copy-on-write, flip bits
// ---------------------------------------------------------------------------
//
// The working vectors share buffers with the backup where that is free
// (the backup of p^0 / L(p^0) is the slot itself; x and r keep their
// cycle-start buffer).  A flip must never reach the backup, so when the
// current vector still is the backup's buffer it is first copied.  A flip of
// p^nu, nu > 0, first forms p^nu from the basis in the buffer of u_nu (which
// no earlier direction contains): it takes u_nu's place in the basis.

template <typename T>
__global__ void k_event_prep(Table<T> tb, int vec)
{
    if (threadIdx.x != 0) return;
    SolveState* st = tb.inst[0].st;
    // e events run between the step's decision and its stencil pass: they
    // apply when the step passed its tests (its e feeds the new direction);
    // e belongs to no backup, so nothing is copied first
    st->ev_ok = (vec == FTGCR_V_E) ? st->e_ok : (st->status == RUNNING);
    if (!st->ev_ok) return;
    st->ev_vec = vec;
    st->ev_copy = 0;
    if (vec == FTGCR_V_E) return;
    const int nu = st->nu;
    if (vec == FTGCR_V_X) {
        // materialise the iterate of this step: x_base + sum_{l < nu} beta_l p^l
        const int src = st->x_base;
        const int dst = (st->x_base == st->x_bak) ? 1 - st->x_base : st->x_base;
        st->ev_src = src;
        st->ev_dst = dst;
        st->ev_lo = st->x_base_nu;
        st->ev_hi = nu;
        st->ev_copy = (src != dst) || (nu > st->x_base_nu);
        st->x_base = dst;
        st->x_base_nu = nu;
    } else if (vec == FTGCR_V_R) {
        if (st->r_cur == st->r_bak) {
            const int dst = other_r(st->r_cur, st->r_dst);
            st->ev_src = st->r_cur;
            st->ev_dst = dst;
            st->ev_copy = 1;
            st->r_cur = dst;
            if (nu > 0) st->r_dst = dst;
        }
    } else {
        if (nu == 0 && st->slot[0] == st->b_slot0) {
            const int src = st->slot[0];
            const int dst = st->slot[1];
            st->ev_src = src;
            st->ev_dst = dst;
            st->ev_copy = 1;
            st->slot[0] = dst;
            st->slot[1] = src;
            const int last = st->k + 1;
            st->ev_usrc = st->uslot[0];
            st->ev_udst = st->uslot[last];
            st->uslot[0] = st->ev_udst;
            st->uslot[last] = st->ev_usrc;
        } else if (nu > 0 && vec == FTGCR_V_P) {
            st->ev_copy = 2;
        }
    }
}

template <typename T>
__global__ void k_event_copy(Table<T> tb)
{
    const Inst<T>& in = tb.inst[0];
    const SolveState* st = in.st;
    if (!st->ev_ok || !st->ev_copy) return;
    const long long n = in.g.n;
    const int vec = st->ev_vec;
    const int nu = st->nu;
    __shared__ double s_c[KMAX + 1];
    if ((int)threadIdx.x <= KMAX) {
        const int j = threadIdx.x;
        s_c[j] = vec == FTGCR_V_X ? basis_coef(st, j, st->ev_lo, st->ev_hi - 1)
                 : (st->ev_copy == 2 && j <= nu) ? st->bm[nu][j] : 0.0;
    }
    __syncthreads();
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += stride) {
        if (vec == FTGCR_V_X) {
            double xd = 0.0;
            if (st->ev_hi > st->ev_lo)
                for (int j = 0; j < st->ev_hi; ++j) xd = fma(s_c[j], (double)in.U[st->uslot[j]][c], xd);
            in.X[st->ev_dst][c] = in.X[st->ev_src][c] + xd;
        } else if (vec == FTGCR_V_R) {
            in.R[st->ev_dst][c] = in.R[st->ev_src][c];
        } else if (st->ev_copy == 2) {
            T* u = in.U[st->uslot[nu]];
            double pa = (double)u[c];
            for (int j = 0; j < nu; ++j) pa = fma(s_c[j], (double)in.U[st->uslot[j]][c], pa);
            u[c] = (T)pa;
        } else {
            in.U[st->ev_udst][c] = in.U[st->ev_usrc][c];
            in.AP[st->ev_dst][c] = in.AP[st->ev_src][c];
        }
    }
}

template <typename T>
__global__ void k_event_inject(Table<T> tb, const long long* idx, const unsigned char* bits, long long count,
                               long long start, int bit0, int again)
{
    const Inst<T>& in = tb.inst[0];
    SolveState* st = in.st;
    if (!st->ev_ok) return;
    const int vec = st->ev_vec;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += stride) {
        const long long at = idx ? idx[t] : start + t;
        const int bit = bits ? (int)bits[t] : bit0;
        if (vec == FTGCR_V_X) write_xor<double>(in.X[st->x_base] + at, bit);
        else if (vec == FTGCR_V_R) write_xor<T>(in.R[st->r_cur] + at, bit);
        else if (vec == FTGCR_V_P) write_xor<T>(in.U[st->uslot[st->nu]] + at, bit);
        else if (vec == FTGCR_V_AP) write_xor<T>(in.AP[st->slot[st->nu]] + at, bit);
        else write_xor<T>(in.U[st->uslot[st->nu + 1]] + at, bit);
    }
    if (!again && blockIdx.x == 0 && threadIdx.x == 0) {
        st->events_applied += 1;
        st->events_since_rb = 1;
        if (vec == FTGCR_V_P && st->ev_copy == 2)   // the basis holds p^nu itself now
            for (int j = 0; j < st->nu; ++j) st->bm[st->nu][j] = 0.0;
    }
}

// <r, L p^nu> and <L p^nu, L p^nu> recomputed after a flip in r or L(p^nu).
template <typename T, int MESH>
__global__ __launch_bounds__(ST_THREADS) void k_beta_dots(Table<T> tb)
{
    __shared__ double sh[4];
    const Inst<T>& in = tb.inst[0];
    SolveState* st = in.st;
    if (!st->ev_ok) return;
    const int lb = blockIdx.x;
    const StPos ps = st_pos_m<MESH>(in, lb, in.kc, in.ord_st);
    double an = 0.0, ad = 0.0;
    if (ps.col_ok) {
        const T* r = in.R[st->r_cur];
        const T* ap = in.AP[st->slot[st->nu]];
        for (int kk = 0; kk < in.kc; ++kk) {
            if (ps.k0 + kk < in.g.nz) {
                const long long c = (long long)ps.i + (long long)in.g.nx * ps.j + (long long)in.g.ncols * (ps.k0 + kk);
                const double a = (double)ap[c];
                an = fma((double)r[c], a, an);
                ad = fma(a, a, ad);
            }
        }
    }
    const double sn = block_sum(an, sh);
    const double sd = block_sum(ad, sh);
    if (threadIdx.x == 0) {
        in.part[(long long)(0) * in.pstride + lb] = sn;
        in.part[(long long)(1) * in.pstride + lb] = sd;
    }
}

template <typename T>
__global__ __launch_bounds__(RED_THREADS) void k_finish_beta_dots(Table<T> tb)
{
    const Inst<T>& in = tb.inst[0];
    SolveState* st = in.st;
    if (!st->ev_ok) return;
    double v[2];
    sum_partials<2, 8>(in, in.nblk_st, 0, 2, v);
    const double num = v[0], dn = v[1];
    if (threadIdx.x == 0) {
        st->beta_num = num;
        st->d_cur = dn;
        st->d[st->nu] = dn;
    }
}

// ---------------------------------------------------------------------------
// parity entry points
// ---------------------------------------------------------------------------

template <int KC, int MESH>
__global__ __launch_bounds__(ST_THREADS) void k_debug_apply_A(Table<double> tb, const double* x, double* y)
{
    const Inst<double>& in = tb.inst[0];
    const StPos ps = st_pos_m<MESH>(in, blockIdx.x, in.kc, in.ord_st);
    double ax[KC];
    stencil_m<double, KC, MESH>(in.g, x, ps, ax);
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
        if (ps.col_ok && ps.k0 + kk < in.g.nz)
            y[(long long)ps.i + (long long)in.g.nx * ps.j + (long long)in.g.ncols * (ps.k0 + kk)] = ax[kk];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

#define FTGCR_KC_SWITCH(kc, CALL)                         \
    switch (kc) {                                         \
    case 1: { constexpr int KCV = 1; CALL; } break;       \
    case 2: { constexpr int KCV = 2; CALL; } break;       \
    case 4: { constexpr int KCV = 4; CALL; } break;       \
    case 8: { constexpr int KCV = 8; CALL; } break;       \
    default: { constexpr int KCV = 16; CALL; } break;     \
    }

// A launch whose start and stop times, if events are given, are taken by
// the dispatch itself (no separate event packets on the stream).
#define FTGCR_TIMED_LAUNCH(E0, E1, KERNEL, GRID, BLOCK, S, ...)                       \
    do {                                                                              \
        if (E0)                                                                       \
            hipExtLaunchKernelGGL(KERNEL, GRID, BLOCK, 0, S, E0, E1, 0, __VA_ARGS__); \
        else                                                                          \
            hipLaunchKernelGGL(KERNEL, GRID, BLOCK, 0, S, __VA_ARGS__);               \
    } while (0)

#define FTGCR_H_SWITCH(H, CALL)                           \
    switch (H) {                                          \
    case 4: { constexpr int HV = 4; CALL; } break;        \
    case 8: { constexpr int HV = 8; CALL; } break;        \
    case 16: { constexpr int HV = 16; CALL; } break;      \
    case 24: { constexpr int HV = 24; CALL; } break;      \
    case 28: { constexpr int HV = 28; CALL; } break;      \
    case 32: { constexpr int HV = 32; CALL; } break;      \
    case 40: { constexpr int HV = 40; CALL; } break;      \
    default: { constexpr int HV = 48; CALL; } break;      \
    }

// Half-column depth of the column pass: the smallest template depth that
// holds (nz + 1) / 2 levels (28 serves the paper's 51-level O_N columns,
// half columns of 26, with 8 phantom rows instead of 12 at 32: 44.5 ->
// 41.4 us per launch on O160 x 51).
int thomas_depth(int nz)
{
    const int h = (nz + 1) / 2;
    const int depths[] = {4, 8, 16, 24, 28, 32, 40, 48};
    for (int d : depths)
        if (h <= d) return d;
    return -1;
}

template <typename T>
void Launch<T>::init_state(const Table<T>& tb, int k, int ft, int mixed, long long max_steps, double tol2,
                           int reset_counters, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_init_state<T>, dim3(grid), dim3(64), 0, s, tb, k, ft, mixed, max_steps, tol2,
                       reset_counters);
}

template <typename T>
void Launch<T>::set_round(const Table<T>& tb, double tol2, long long max_steps, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_round<T>, dim3(tb.n), dim3(64), 0, s, tb, tol2, max_steps);
}

// A stencil-pass launch on the table's mesh.
#define FTGCR_MESH_LAUNCH(tb, LAUNCH0, LAUNCH1)                                   \
    do {                                                                          \
        if ((tb).mesh == FTGCR_MESH_OCTAHEDRAL) {                                 \
            constexpr int MESHV = FTGCR_MESH_OCTAHEDRAL;                          \
            LAUNCH1;                                                              \
        } else {                                                                  \
            constexpr int MESHV = FTGCR_MESH_LATLON;                              \
            LAUNCH0;                                                              \
        }                                                                         \
    } while (0)

template <typename T>
void Launch<T>::residual(const Table<T>& tb, int total, int kc, int store, int set_T, hipStream_t s)
{
    FTGCR_MESH_LAUNCH(tb,
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_residual<T, KCV, MESHV>), dim3(total), dim3(ST_THREADS), 0, s, tb,
                                               store)),
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_residual<T, KCV, MESHV>), dim3(total), dim3(ST_THREADS), 0, s, tb,
                                               store)));
    hipLaunchKernelGGL(k_finish_residual<T>, dim3(tb.n), dim3(RED_THREADS), 0, s, tb, set_T);
}

template <typename T>
void Launch<T>::update_thomas(const Table<T>& tb, int total, int H, int mode, hipStream_t s, hipEvent_t e0,
                              hipEvent_t e1)
{
    if (tb.precond == FTGCR_PRECOND_NONE) {
        const int cpb = col_block_cols((int)sizeof(T), H);
        if (mode == MODE_STEP)
            FTGCR_TIMED_LAUNCH(e0, e1, (k_update_copy<T, MODE_STEP>), dim3(total), dim3(COL_THREADS), s, tb,
                               (const T*)nullptr, (T*)nullptr, (const GmInst*)nullptr, cpb);
        else
            hipLaunchKernelGGL((k_update_copy<T, MODE_INIT>), dim3(total), dim3(COL_THREADS), 0, s, tb,
                               (const T*)nullptr, (T*)nullptr, (const GmInst*)nullptr, cpb);
        return;
    }
    if constexpr (sizeof(T) == 4) {
        if (col_block_cols((int)sizeof(T), H) == COL_THREADS) {
            // one lane per column: NZ = 2H levels at most (H <= 32)
#define FTGCR_T1(HH)                                                                                        \
    if (mode == MODE_STEP)                                                                                  \
        FTGCR_TIMED_LAUNCH(e0, e1, (k_update_thomas1<T, 2 * HH, MODE_STEP>), dim3(total), dim3(COL_THREADS), \
                           s, tb);                                                                          \
    else                                                                                                    \
        hipLaunchKernelGGL((k_update_thomas1<T, 2 * HH, MODE_INIT>), dim3(total), dim3(COL_THREADS), 0, s, tb);
            switch (H) {
            case 4: FTGCR_T1(4) break;
            case 8: FTGCR_T1(8) break;
            case 16: FTGCR_T1(16) break;
            case 24: FTGCR_T1(24) break;
            case 28: FTGCR_T1(28) break;
            default: FTGCR_T1(32) break;
            }
#undef FTGCR_T1
            return;
        }
    }
    if constexpr (sizeof(T) == 8) {
        if (tb.mixed_depth) {
            if (mode == MODE_STEP)
                FTGCR_H_SWITCH(H, FTGCR_TIMED_LAUNCH(e0, e1, (k_update_thomas<T, HV, MODE_STEP, true>), dim3(total),
                                                     dim3(COL_THREADS), s, tb, (const T*)nullptr, (T*)nullptr))
            else
                FTGCR_H_SWITCH(H, hipLaunchKernelGGL((k_update_thomas<T, HV, MODE_INIT, true>), dim3(total),
                                                     dim3(COL_THREADS), 0, s, tb, (const T*)nullptr, (T*)nullptr))
            return;
        }
    }
    if (mode == MODE_STEP)
        FTGCR_H_SWITCH(H, FTGCR_TIMED_LAUNCH(e0, e1, (k_update_thomas<T, HV, MODE_STEP>), dim3(total),
                                             dim3(COL_THREADS), s, tb, (const T*)nullptr, (T*)nullptr))
    else
        FTGCR_H_SWITCH(H, hipLaunchKernelGGL((k_update_thomas<T, HV, MODE_INIT>), dim3(total), dim3(COL_THREADS), 0,
                                             s, tb, (const T*)nullptr, (T*)nullptr))
}

template <typename T>
void Launch<T>::finish_col(const Table<T>& tb, int mode, hipStream_t s)
{
    hipLaunchKernelGGL(k_finish_col<T>, dim3(tb.n), dim3(RED_THREADS), 0, s, tb, mode);
}

template <typename T>
void Launch<T>::norms(const Table<T>& tb, int total, int H, hipStream_t s)
{
    hipLaunchKernelGGL(k_norms<T>, dim3(total), dim3(COL_THREADS), 0, s, tb, col_block_cols((int)sizeof(T), H));
    hipLaunchKernelGGL(k_finish_norms<T>, dim3(1), dim3(RED_THREADS), 0, s, tb);
}

template <typename T>
void Launch<T>::finish_alpha(const Table<T>& tb, hipStream_t s)
{
    hipLaunchKernelGGL(k_finish_alpha<T>, dim3(tb.n), dim3(RED_THREADS), 0, s, tb);
}

template <typename T>
void Launch<T>::fold(const Table<T>& tb, int dir, int parts, int values, hipStream_t s)
{
    hipLaunchKernelGGL(k_fold<T>, dim3(parts, values), dim3(ST_THREADS), 0, s, tb, dir);
}

template <typename T>
void Launch<T>::finish_beta(const Table<T>& tb, int init, hipStream_t s)
{
    hipLaunchKernelGGL(k_finish_beta<T>, dim3(tb.n), dim3(RED_THREADS), 0, s, tb, init);
}

template <typename T>
void Launch<T>::stencil_dots(const Table<T>& tb, int total, int kc, int spec, hipStream_t s, hipEvent_t e0,
                             hipEvent_t e1)
{
    FTGCR_MESH_LAUNCH(tb,
        FTGCR_KC_SWITCH(kc, FTGCR_TIMED_LAUNCH(e0, e1, (k_stencil_dots<T, KCV, MESHV>), dim3(total),
                                               dim3(ST_THREADS), s, tb, spec)),
        FTGCR_KC_SWITCH(kc, FTGCR_TIMED_LAUNCH(e0, e1, (k_stencil_dots<T, KCV, MESHV>), dim3(total),
                                               dim3(ST_THREADS), s, tb, spec)));
}

template <typename T>
void Launch<T>::finish_step(const Table<T>& tb, hipStream_t s)
{
    hipLaunchKernelGGL(k_finish_step<T>, dim3(tb.n), dim3(RED_THREADS), 0, s, tb);
}

template <typename T>
void Launch<T>::dir_update(const Table<T>& tb, int total, int kc, int init, bool nt_ap, hipStream_t s,
                           hipEvent_t e0, hipEvent_t e1)
{
    if (nt_ap)
        FTGCR_MESH_LAUNCH(tb,
            FTGCR_KC_SWITCH(kc, FTGCR_TIMED_LAUNCH(e0, e1, (k_dir_update<T, KCV, true, MESHV>), dim3(total),
                                                   dim3(ST_THREADS), s, tb, init)),
            FTGCR_KC_SWITCH(kc, FTGCR_TIMED_LAUNCH(e0, e1, (k_dir_update<T, KCV, true, MESHV>), dim3(total),
                                                   dim3(ST_THREADS), s, tb, init)));
    else
        FTGCR_MESH_LAUNCH(tb,
            FTGCR_KC_SWITCH(kc, FTGCR_TIMED_LAUNCH(e0, e1, (k_dir_update<T, KCV, false, MESHV>), dim3(total),
                                                   dim3(ST_THREADS), s, tb, init)),
            FTGCR_KC_SWITCH(kc, FTGCR_TIMED_LAUNCH(e0, e1, (k_dir_update<T, KCV, false, MESHV>), dim3(total),
                                                   dim3(ST_THREADS), s, tb, init)));
}

template <typename T>
void Launch<T>::finalize_x(const Table<T>& tb, int total, int kc, hipStream_t s)
{
    FTGCR_MESH_LAUNCH(tb,
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_finalize_x<T, KCV, MESHV>), dim3(total), dim3(ST_THREADS), 0, s, tb)),
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_finalize_x<T, KCV, MESHV>), dim3(total), dim3(ST_THREADS), 0, s,
                                               tb)));
}

template <typename T>
void Launch<T>::event_prep(const Table<T>& tb, int vec, hipStream_t s)
{
    hipLaunchKernelGGL(k_event_prep<T>, dim3(1), dim3(64), 0, s, tb, vec);
}

template <typename T>
void Launch<T>::event_copy(const Table<T>& tb, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_event_copy<T>, dim3(grid), dim3(256), 0, s, tb);
}

template <typename T>
void Launch<T>::event_inject(const Table<T>& tb, int grid, const long long* idx, const unsigned char* bits,
                             long long count, long long start, int bit, bool again, hipStream_t s)
{
    hipLaunchKernelGGL(k_event_inject<T>, dim3(grid), dim3(256), 0, s, tb, idx, bits, count, start, bit, again ? 1 : 0);
}

template <typename T>
void Launch<T>::beta_dots(const Table<T>& tb, int total, hipStream_t s)
{
    FTGCR_MESH_LAUNCH(tb, hipLaunchKernelGGL((k_beta_dots<T, MESHV>), dim3(total), dim3(ST_THREADS), 0, s, tb),
                      hipLaunchKernelGGL((k_beta_dots<T, MESHV>), dim3(total), dim3(ST_THREADS), 0, s, tb));
    hipLaunchKernelGGL(k_finish_beta_dots<T>, dim3(1), dim3(RED_THREADS), 0, s, tb);
}

template <typename T>
void Launch<T>::debug_apply_A(const Table<T>&, int, int, const double*, double*, hipStream_t)
{
}

template <>
void Launch<double>::debug_apply_A(const Table<double>& tb, int total, int kc, const double* in, double* out,
                                   hipStream_t s)
{
    FTGCR_MESH_LAUNCH(tb,
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_debug_apply_A<KCV, MESHV>), dim3(total), dim3(ST_THREADS), 0, s, tb,
                                               in, out)),
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_debug_apply_A<KCV, MESHV>), dim3(total), dim3(ST_THREADS), 0, s, tb,
                                               in, out)));
}

template <typename T>
void Launch<T>::debug_pinv(const Table<T>&, int, int, const double*, double*, hipStream_t)
{
}

template <>
void Launch<double>::debug_pinv(const Table<double>& tb, int total, int H, const double* in, double* out,
                                hipStream_t s)
{
    if (tb.precond == FTGCR_PRECOND_NONE) {
        hipLaunchKernelGGL((k_update_copy<double, MODE_DEBUG>), dim3(total), dim3(COL_THREADS), 0, s, tb, in, out,
                           (const GmInst*)nullptr, COLS_PER_BLOCK);
        return;
    }
    FTGCR_H_SWITCH(H, hipLaunchKernelGGL((k_update_thomas<double, HV, MODE_DEBUG>), dim3(total), dim3(COL_THREADS),
                                         0, s, tb, in, out));
}

// Status and step count of every instance into a small device array (one
// read-back per poll of a batched solve).
template <typename T>
__global__ void k_gather_status(Table<T> tb, long long* out)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= tb.n) return;
    const SolveState* st = tb.inst[m].st;
    out[2 * m] = st->res_fail == RES_BROKEN ? BROKEN : st->status;
    out[2 * m + 1] = st->s;
}

// Clears RES_LATE and leaves the words of that launch's round behind.
template <typename T>
__global__ void k_resident_late(Table<T> tb)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= tb.n) return;
    SolveState* st = tb.inst[m].st;
    if (st->res_fail != RES_LATE) return;
    st->res_fail = 0;
    st->res_seq += 2;
}

template <typename T>
void Launch<T>::resident_late(const Table<T>& tb, hipStream_t s)
{
    hipLaunchKernelGGL(k_resident_late<T>, dim3((tb.n + 63) / 64), dim3(64), 0, s, tb);
}

template <typename T>
void Launch<T>::gather_status(const Table<T>& tb, long long* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_gather_status<T>, dim3((tb.n + 63) / 64), dim3(64), 0, s, tb, out);
}

template struct Launch<double>;
template struct Launch<float>;

// ---------------------------------------------------------------------------
// FT-GMRES(k): the fault layer of Algorithm 1 on restarted GMRES(k)
// ---------------------------------------------------------------------------
//
// Right-preconditioned restarted GMRES with classical Gram-Schmidt and Givens
// rotations; the residual-norm test after every step (on the rotated
// right-hand side |g_{j+1}|, the minimised residual norm of the cycle) and on
// the explicit residual at the end of every cycle, the backup [x, |s|^2] of
// each cycle that passes, the rollback and the stagnation rule of FT-GCR.
// Per cycle the host enqueues: residual s = R - A x (into U[0]), restart (the
// cycle-end decisions, then g_0 = |s|); k steps of
//   precond      v_j = U[j] / den[j] (written back), z_j = P^{-1} v_j
//   stencil      w = A z_j (stored) and the partials of <w, v_i>, i <= j
//   finish_h     h_ij
//   orth         w - sum_i h_ij v_i into U[j+1], partials of its norm
//   finish_step  h_{j+1,j}, rotations, |g_{j+1}|^2, exit and fault tests
// then xupd (x + sum_i y_i z_i, y from the triangular system) and finish_x.
// Every step kernel returns at once once the cycle is inactive (ended,
// rolled back or the solve finished), so a cycle is a fixed launch sequence.

__device__ __forceinline__ StPos gm_pos(const GmInst& in, int lb)
{
    StPos p;
    int ct, bz;
    block_tile(lb, in.tx * in.ty, in.tz, in.ord, ct, bz);
    if (in.g.mesh == FTGCR_MESH_OCTAHEDRAL) {   // ST_THREADS consecutive points per block
        const int i = ct * ST_THREADS + threadIdx.x;
        p.col_ok = i < in.g.nx;
        p.i = p.col_ok ? i : in.g.nx - 1;
        p.j = 0;
        p.k0 = bz * in.kc;
        return p;
    }
    const int bx = ct % in.tx;
    const int by = ct / in.tx;
    const int i = bx * ST_TX + (threadIdx.x & (ST_TX - 1));
    const int j = by * ST_TY + (threadIdx.x / ST_TX);
    p.col_ok = i < in.g.nx && j < in.g.ny;
    p.i = i < in.g.nx ? i : in.g.nx - 1;
    p.j = j < in.g.ny ? j : in.g.ny - 1;
    p.k0 = bz * in.kc;
    return p;
}

__global__ void k_gm_init(const GmInst* gi, int k, int ft, long long max_steps, double tol2)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    GmState* st = gi->st;
    st->status = RUNNING;
    st->active = 0;
    st->j = 0;
    st->k = k;
    st->ft = ft;
    st->phase = GM_INIT;
    st->jdone = 0;
    st->cycle_end = 0;
    st->capped = 0;
    st->x_cur = 0;
    st->x_bak = 0;
    st->x_dst = 0;
    st->detections = 0;
    st->stagnation_accepts = 0;
    st->events_applied = 0;
    st->events_since_rb = 1;
    st->log_len = 0;
    st->ev_ok = 0;
    st->s = 0;
    st->max_steps = max_steps;
    st->accepted = 0;
    st->cycles = 0;
    st->last_rb_pos = -1;
    st->b_accepted = 0;
    st->tol2 = tol2;
}

// s = R - A x into U[0]; partials of <R, R> (row 0) and <s, s> (row 1).
template <int KC, int MESH>
__global__ __launch_bounds__(ST_THREADS) void k_gm_residual(const GmInst* gi)
{
    __shared__ double sh[4];
    const GmInst& in = *gi;
    const GmState* st = in.st;
    if (st->status != RUNNING) return;
    const StPos ps = gm_pos(in, blockIdx.x);
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    double ax[KC], b[KC];
    stencil_m<double, KC, MESH>(in.g, in.X[st->x_cur], ps, ax);
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
        b[kk] = in.rhs[c0 + plane * kq];
    }
    double ss = 0.0, bb = 0.0;
    double* u0 = in.U[0];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const bool ok = ps.col_ok && ps.k0 + kk < nz;
        const double r = ok ? b[kk] - ax[kk] : 0.0;
        const double bv = ok ? b[kk] : 0.0;
        if (ok) u0[c0 + plane * (ps.k0 + kk)] = r;
        ss = fma(r, r, ss);
        bb = fma(bv, bv, bb);
    }
    const double sb = block_sum(bb, sh);
    const double sr = block_sum(ss, sh);
    if (threadIdx.x == 0) {
        in.part[blockIdx.x] = sb;
        in.part[in.pstride + blockIdx.x] = sr;
    }
}

__device__ void gm_log(GmState* st, long long step, int nu, int action, double rr_old, double rr_new)
{
    st->detections += 1;
    if (st->log_len < LOG_CAP) {
        DetectRec& rec = st->log[st->log_len++];
        rec.step = step;
        rec.nu = nu;
        rec.action = action;
        rec.rr_old = rr_old;
        rec.rr_new = rr_new;
    }
}

// The explicit residual's decisions (first pass: the initial state; after
// a cycle: exit test, then the fault test against the backup, then the new
// backup; after a rollback: none), then a new cycle from |s|.
__global__ __launch_bounds__(RED_THREADS) void k_gm_restart(const GmInst* gi)
{
    const GmInst& in = *gi;
    GmState* st = in.st;
    if (st->status != RUNNING) return;
    double v[2];
    sum_partials<2, 8>(in, in.nblk_st, 0, 2, v);
    if (threadIdx.x != 0) return;
    const double rho2 = v[1];
    st->rho2 = rho2;
    if (st->phase == GM_INIT) {
        st->RR = v[0];
        st->T = st->tol2 * v[0];
        if (rho2 <= st->T) {
            st->status = FTGCR_CONVERGED;
            return;
        }
        st->x_bak = st->x_cur;
        st->b_rho2 = rho2;
        st->b_accepted = 0;
    } else if (st->phase == GM_CHECK) {
        if (st->capped || (st->s >= st->max_steps && rho2 > st->T)) {
            st->status = FTGCR_MAX_STEPS;
            return;
        }
        if (rho2 <= st->T) {
            st->status = FTGCR_CONVERGED;
            return;
        }
        if (st->ft && !(rho2 < st->b_rho2)) {   // NaN included
            const long long pos = 2 * st->accepted + 1;
            const int stag = (pos == st->last_rb_pos) && !st->events_since_rb;
            gm_log(st, st->s, -1, stag, st->b_rho2, rho2);
            if (!stag) {
                st->x_cur = st->x_bak;
                st->accepted = st->b_accepted;
                st->last_rb_pos = pos;
                st->events_since_rb = 0;
                st->phase = GM_REDO;
                st->active = 0;
                st->cycle_end = 0;
                return;   // the next residual pass is that of the restored x
            }
            st->stagnation_accepts += 1;
        }
        if (st->ft) {
            st->x_bak = st->x_cur;
            st->b_rho2 = rho2;
            st->b_accepted = st->accepted;
        }
    }
    if (st->s >= st->max_steps) {
        st->status = FTGCR_MAX_STEPS;
        return;
    }
    const double rho = sqrt(rho2);
    st->den[0] = rho;
    st->g[0] = rho;
    for (int i = 1; i <= st->k; ++i) st->g[i] = 0.0;
    st->rr_old = rho2;
    st->j = 0;
    st->jdone = 0;
    st->cycle_end = 0;
    st->capped = 0;
    st->active = 1;
    st->phase = GM_CHECK;
}

// The partials of <w, v_i>, i <= j, of a block's cells (rows DOT_ROW0 + i).
// The loop over i is unrolled to KMAX with a uniform guard, and the loads of
// v_{i+1} are issued before v_i's values are used (two buffers alternating
// with the parity of i), so the terms cost one memory round trip together
// rather than one each.
// NT: the Arnoldi vectors are loaded with the non-temporal hint (gm_nt_hint:
// the cycle's vectors do not fit the Infinity Cache, which is then left to
// z_j, w and v_{j+1}, read again within the step: FT-GMRES(16) on 512 x 256 x
// 64 308.6 -> 271.5 ms, the stencil pass 150 -> 130 us, orthogonalisation 124
// -> 108, column solve 44 -> 36).
template <bool NT>
__device__ __forceinline__ double gm_load(const double* p)
{
    return NT ? __builtin_nontemporal_load(p) : *p;
}

template <int KC, bool NT>
__device__ __forceinline__ void gm_dots(const GmInst& in, const StPos& ps, const double (&w)[KC], int j)
{
    __shared__ double sh[KMAX + 1][4];
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double buf[2][KC];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
        buf[0][kk] = gm_load<NT>(&in.U[0][c0 + plane * kq]);
    }
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
        if (i <= j) {
            if (i + 1 < KMAX && i + 1 <= j) {
                const double* vn = in.U[i + 1];
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                    buf[(i + 1) & 1][kk] = gm_load<NT>(&vn[c0 + plane * kq]);
                }
            }
            double acc = 0.0;
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) {
                const bool ok = ps.col_ok && ps.k0 + kk < nz;
                acc = fma(w[kk], ok ? buf[i & 1][kk] : 0.0, acc);
            }
            const double t = wave_sum(acc);
            if (lane == 0) sh[i][wv] = t;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x <= j) {
        const int i = threadIdx.x;
        in.part[(long long)(DOT_ROW0 + i) * in.pstride + blockIdx.x] = ((sh[i][0] + sh[i][1]) + sh[i][2]) + sh[i][3];
    }
}

// w = A z_j into W; with DOTS also the partials of <w, v_i>.
template <int KC, int DOTS, int MESH, bool NT>
__global__ __launch_bounds__(ST_THREADS) void k_gm_stencil(const GmInst* gi)
{
    const GmInst& in = *gi;
    const GmState* st = in.st;
    if (st->status != RUNNING || !st->active) return;
    const int j = st->j;
    const StPos ps = gm_pos(in, blockIdx.x);
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    double w[KC];
    stencil_m<double, KC, MESH>(in.g, in.Z[j], ps, w);
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const bool ok = ps.col_ok && ps.k0 + kk < nz;
        if (ok) in.W[c0 + plane * (ps.k0 + kk)] = w[kk];
        else w[kk] = 0.0;
    }
    if (DOTS) gm_dots<KC, NT>(in, ps, w, j);
}

// The partials of <w, v_i> from the stored w (after a fault event on it).
template <int KC>
__global__ __launch_bounds__(ST_THREADS) void k_gm_dots(const GmInst* gi)
{
    const GmInst& in = *gi;
    const GmState* st = in.st;
    if (st->status != RUNNING || !st->active) return;
    const StPos ps = gm_pos(in, blockIdx.x);
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    double w[KC];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const bool ok = ps.col_ok && ps.k0 + kk < nz;
        const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
        const double v = in.W[c0 + plane * kq];
        w[kk] = ok ? v : 0.0;
    }
    gm_dots<KC, false>(in, ps, w, st->j);
}

__global__ __launch_bounds__(RED_THREADS) void k_gm_finish_h(const GmInst* gi)
{
    const GmInst& in = *gi;
    GmState* st = in.st;
    if (st->status != RUNNING || !st->active) return;
    const int j = st->j;
    const double* v = sum_partials<4, 4>(in, in.nblk_st, DOT_ROW0, j + 1, nullptr);
    if ((int)threadIdx.x <= j) st->H[threadIdx.x * KMAX + j] = v[threadIdx.x];
}

// U[j+1] = w - sum_i h_ij v_i (ascending i); partials of its squared norm.
// Each cell takes the same operations in the same order as a loop over i
// per cell; the loop over i runs outside (unrolled to KMAX, uniform guard)
// with v_{i+1}'s loads issued before v_i is used.
template <int KC, bool NT>
__global__ __launch_bounds__(ST_THREADS) void k_gm_orth(const GmInst* gi)
{
    __shared__ double sh[4];
    __shared__ double s_h[KMAX + 1];
    const GmInst& in = *gi;
    const GmState* st = in.st;
    if (st->status != RUNNING || !st->active) return;
    const int j = st->j;
    if ((int)threadIdx.x <= j) s_h[threadIdx.x] = st->H[threadIdx.x * KMAX + j];
    __syncthreads();
    const StPos ps = gm_pos(in, blockIdx.x);
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    double* un = in.U[j + 1];
    double w[KC], buf[2][KC];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
        const long long c = c0 + plane * kq;
        w[kk] = in.W[c];
        buf[0][kk] = gm_load<NT>(&in.U[0][c]);
    }
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
        if (i <= j) {
            if (i + 1 < KMAX && i + 1 <= j) {
                const double* vn = in.U[i + 1];
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                    buf[(i + 1) & 1][kk] = gm_load<NT>(&vn[c0 + plane * kq]);
                }
            }
            const double h = s_h[i];
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) w[kk] = w[kk] - h * buf[i & 1][kk];
        }
    }
    double acc = 0.0;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const bool ok = ps.col_ok && ps.k0 + kk < nz;
        if (ok) un[c0 + plane * (ps.k0 + kk)] = w[kk];
        const double wd = ok ? w[kk] : 0.0;
        acc = fma(wd, wd, acc);
    }
    const double sw = block_sum(acc, sh);
    if (threadIdx.x == 0) in.part[blockIdx.x] = sw;
}

// h_{j+1,j}, the rotations, the step's residual norm |g_{j+1}|^2, then the
// exit test and the fault test of the step.
__global__ __launch_bounds__(RED_THREADS) void k_gm_finish_step(const GmInst* gi)
{
    const GmInst& in = *gi;
    GmState* st = in.st;
    if (st->status != RUNNING || !st->active) return;
    double v[2];
    sum_partials<2, 8>(in, in.nblk_st, 0, 1, v);
    if (threadIdx.x != 0) return;
    const int j = st->j;
    double* H = st->H;
    const double hn = sqrt(v[0]);
    H[(j + 1) * KMAX + j] = hn;
    for (int i = 0; i < j; ++i) {
        const double a = H[i * KMAX + j], b = H[(i + 1) * KMAX + j];
        H[i * KMAX + j] = st->cs[i] * a + st->sn[i] * b;
        H[(i + 1) * KMAX + j] = -st->sn[i] * a + st->cs[i] * b;
    }
    {
        const double a = H[j * KMAX + j], b = H[(j + 1) * KMAX + j];
        const double den = sqrt(a * a + b * b);
        st->cs[j] = a / den;
        st->sn[j] = b / den;
        H[j * KMAX + j] = den;
        H[(j + 1) * KMAX + j] = 0.0;
        st->g[j + 1] = -st->sn[j] * st->g[j];
        st->g[j] = st->cs[j] * st->g[j];
    }
    const double rr_new = st->g[j + 1] * st->g[j + 1];
    st->s += 1;
    const long long s = st->s;
    if (j == 0) st->cycles += 1;
    if (s <= in.hist_cap) in.hist[s - 1] = rr_new;
    st->jdone = j + 1;
    if (rr_new <= st->T) {   // exit test first: the cycle ends, the check follows
        st->accepted += 1;
        st->rr_old = rr_new;
        st->cycle_end = 1;
        st->active = 0;
        return;
    }
    if (st->ft && !(rr_new < st->rr_old)) {   // NaN included
        const long long pos = 2 * (st->accepted + 1);
        const int stag = (pos == st->last_rb_pos) && !st->events_since_rb;
        gm_log(st, s, j, stag, st->rr_old, rr_new);
        if (!stag) {
            st->x_cur = st->x_bak;
            st->accepted = st->b_accepted;
            st->last_rb_pos = pos;
            st->events_since_rb = 0;
            st->phase = GM_REDO;
            st->active = 0;
            st->cycle_end = 0;
            return;
        }
        st->stagnation_accepts += 1;
    }
    st->accepted += 1;
    st->rr_old = rr_new;
    if (hn == 0.0 || j + 1 == st->k) {   // the cycle is complete (or its space holds the solution)
        st->cycle_end = 1;
        st->active = 0;
        return;
    }
    st->den[j + 1] = hn;
    st->j = j + 1;
    if (s >= st->max_steps) {   // the next step would pass the cap
        st->capped = 1;
        st->cycle_end = 1;
        st->active = 0;
    }
}

// The cycle's correction: y from the rotated triangular system over the
// steps done, then x + sum_i y_i z_i (ascending i) into a buffer that is not
// the backup.
template <int KC, bool NT>
__global__ __launch_bounds__(ST_THREADS) void k_gm_xupd(const GmInst* gi)
{
    __shared__ double y[KMAX];
    const GmInst& in = *gi;
    const GmState* st = in.st;
    if (st->status != RUNNING || !st->cycle_end) return;
    const int jd = st->jdone;
    if (threadIdx.x == 0) {
        const double* H = st->H;
        for (int i = jd - 1; i >= 0; --i) {
            double acc = st->g[i];
            for (int l = i + 1; l < jd; ++l) acc = acc - H[i * KMAX + l] * y[l];
            y[i] = acc / H[i * KMAX + i];
        }
    }
    __syncthreads();
    const StPos ps = gm_pos(in, blockIdx.x);
    if (!ps.col_ok) return;
    const int nz = in.g.nz;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    const int xs = st->x_cur;
    const int xd = (st->x_cur == st->x_bak) ? 1 - st->x_cur : st->x_cur;
    const double* xsrc = in.X[xs];
    double* xdst = in.X[xd];
    // per cell x + y_0 z_0 + y_1 z_1 + ... in ascending i, the loop over i
    // outside (unrolled to KMAX, uniform guard) with z_{i+1}'s loads issued
    // before z_i is used
    double xv[KC], buf[2][KC];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
        const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
        const long long c = c0 + plane * kq;
        xv[kk] = xsrc[c];
        buf[0][kk] = jd > 0 ? gm_load<NT>(&in.Z[0][c]) : 0.0;
    }
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
        if (i < jd) {
            if (i + 1 < KMAX && i + 1 < jd) {
                const double* zn = in.Z[i + 1];
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    const int kq = (ps.k0 + kk > nz - 1) ? nz - 1 : ps.k0 + kk;
                    buf[(i + 1) & 1][kk] = gm_load<NT>(&zn[c0 + plane * kq]);
                }
            }
            const double yi = y[i];
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) xv[kk] = xv[kk] + yi * buf[i & 1][kk];
        }
    }
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
        if (ps.k0 + kk < nz) xdst[c0 + plane * (ps.k0 + kk)] = xv[kk];
}

__global__ void k_gm_finish_x(const GmInst* gi)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    GmState* st = gi->st;
    if (st->status != RUNNING || !st->cycle_end) return;
    st->x_cur = (st->x_cur == st->x_bak) ? 1 - st->x_cur : st->x_cur;
}

// The returned iterate into the caller's buffer X[0].
template <int KC>
__global__ __launch_bounds__(ST_THREADS) void k_gm_finalize(const GmInst* gi)
{
    const GmInst& in = *gi;
    const GmState* st = in.st;
    if (st->x_cur == 0) return;
    const StPos ps = gm_pos(in, blockIdx.x);
    if (!ps.col_ok) return;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    for (int kk = 0; kk < KC; ++kk) {
        if (ps.k0 + kk >= in.g.nz) break;
        in.X[0][c0 + plane * (ps.k0 + kk)] = in.X[st->x_cur][c0 + plane * (ps.k0 + kk)];
    }
}

// Fault events of executed step `step` (they apply only if that step is the
// one about to run, in an active cycle).  X: x at the start of the step,
// copied first if it still is the backup's buffer; R: v_j at the start of
// the step, stored normalised first (the flip acts on v_j itself); P and E:
// z_j after the preconditioner; AP: w = A z_j before the inner products.
__global__ void k_gm_event_prep(const GmInst* gi, int vec, long long step)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    GmState* st = gi->st;
    st->ev_ok = (st->status == RUNNING && st->active && st->s + 1 == step);
    st->ev_vec = vec;
    st->ev_copy = 0;
    if (!st->ev_ok) return;
    if (vec == FTGCR_V_X && st->x_cur == st->x_bak) {
        st->ev_copy = 1;
        st->ev_src = st->x_cur;
        st->ev_dst = 1 - st->x_cur;
        st->x_cur = st->ev_dst;
    } else if (vec == FTGCR_V_R && st->den[st->j] != 1.0) {
        st->ev_copy = 1;
    }
}

template <int KC>
__global__ __launch_bounds__(ST_THREADS) void k_gm_event_copy(const GmInst* gi)
{
    const GmInst& in = *gi;
    const GmState* st = in.st;
    if (!st->ev_ok || !st->ev_copy) return;
    const StPos ps = gm_pos(in, blockIdx.x);
    if (!ps.col_ok) return;
    const long long plane = (long long)in.g.ncols;
    const long long c0 = (long long)ps.i + (long long)in.g.nx * ps.j;
    const int j = st->j;
    const double den = st->den[j];
    for (int kk = 0; kk < KC; ++kk) {
        if (ps.k0 + kk >= in.g.nz) break;
        const long long c = c0 + plane * (ps.k0 + kk);
        if (st->ev_vec == FTGCR_V_X) in.X[st->ev_dst][c] = in.X[st->ev_src][c];
        else in.U[j][c] = in.U[j][c] / den;
    }
}

__global__ void k_gm_event_inject(const GmInst* gi, const long long* idx, const unsigned char* bits, long long count,
                                  long long start, int bit0)
{
    const GmInst& in = *gi;
    GmState* st = in.st;
    if (!st->ev_ok) return;
    const int vec = st->ev_vec;
    const int j = st->j;
    double* target = vec == FTGCR_V_X ? in.X[st->x_cur]
                   : vec == FTGCR_V_R ? in.U[j]
                   : vec == FTGCR_V_AP ? in.W : in.Z[j];
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += stride) {
        const long long at = idx ? idx[t] : start + t;
        const int bit = bits ? (int)bits[t] : bit0;
        write_xor<double>(target + at, bit);
    }
    // the grid's last use of the prepared state is above; the one-thread
    // bookkeeping below touches fields no thread reads here
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->events_applied += 1;
        st->events_since_rb = 1;
        if (vec == FTGCR_V_R) st->den[j] = 1.0;   // v_j is stored normalised now
    }
}

void GmLaunch::init(const GmInst* gi, int k, int ft, long long max_steps, double tol2, hipStream_t s)
{
    hipLaunchKernelGGL(k_gm_init, dim3(1), dim3(64), 0, s, gi, k, ft, max_steps, tol2);
}

void GmLaunch::residual(const GmInst* gi, int nblk, int kc, int mesh, hipStream_t s)
{
    if (mesh == FTGCR_MESH_OCTAHEDRAL)
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_residual<KCV, FTGCR_MESH_OCTAHEDRAL>), dim3(nblk),
                                               dim3(ST_THREADS), 0, s, gi))
    else
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_residual<KCV, FTGCR_MESH_LATLON>), dim3(nblk),
                                               dim3(ST_THREADS), 0, s, gi))
}

void GmLaunch::restart(const GmInst* gi, hipStream_t s)
{
    hipLaunchKernelGGL(k_gm_restart, dim3(1), dim3(RED_THREADS), 0, s, gi);
}

void GmLaunch::precond(const Table<double>& tb, const GmInst* gi, int nblk_col, int H, hipStream_t s)
{
    if (tb.precond == FTGCR_PRECOND_NONE) {
        hipLaunchKernelGGL((k_update_copy<double, MODE_GM>), dim3(nblk_col), dim3(COL_THREADS), 0, s, tb,
                           (const double*)nullptr, (double*)nullptr, gi, COLS_PER_BLOCK);
        return;
    }
    FTGCR_H_SWITCH(H, hipLaunchKernelGGL((k_update_thomas_gm<HV>), dim3(nblk_col), dim3(COL_THREADS), 0, s, tb,
                                             gi))
}

void GmLaunch::stencil(const GmInst* gi, int nblk, int kc, int dots, int mesh, bool nt, hipStream_t s)
{
#define FTGCR_GM_STENCIL(MV, DV, NTV) \
    FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_stencil<KCV, DV, MV, NTV>), dim3(nblk), dim3(ST_THREADS), 0, s, gi))
#define FTGCR_GM_STENCIL_MESH(MV)                     \
    if (!dots) FTGCR_GM_STENCIL(MV, 0, false)         \
    else if (nt) FTGCR_GM_STENCIL(MV, 1, true)        \
    else FTGCR_GM_STENCIL(MV, 1, false)
    if (mesh == FTGCR_MESH_OCTAHEDRAL) {
        FTGCR_GM_STENCIL_MESH(FTGCR_MESH_OCTAHEDRAL)
    } else {
        FTGCR_GM_STENCIL_MESH(FTGCR_MESH_LATLON)
    }
#undef FTGCR_GM_STENCIL_MESH
#undef FTGCR_GM_STENCIL
}

void GmLaunch::dots(const GmInst* gi, int nblk, int kc, hipStream_t s)
{
    FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_dots<KCV>), dim3(nblk), dim3(ST_THREADS), 0, s, gi));
}

void GmLaunch::finish_h(const GmInst* gi, hipStream_t s)
{
    hipLaunchKernelGGL(k_gm_finish_h, dim3(1), dim3(RED_THREADS), 0, s, gi);
}

void GmLaunch::orth(const GmInst* gi, int nblk, int kc, bool nt, hipStream_t s)
{
    if (nt)
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_orth<KCV, true>), dim3(nblk), dim3(ST_THREADS), 0, s, gi))
    else
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_orth<KCV, false>), dim3(nblk), dim3(ST_THREADS), 0, s, gi))
}

void GmLaunch::finish_step(const GmInst* gi, hipStream_t s)
{
    hipLaunchKernelGGL(k_gm_finish_step, dim3(1), dim3(RED_THREADS), 0, s, gi);
}

void GmLaunch::xupd(const GmInst* gi, int nblk, int kc, bool nt, hipStream_t s)
{
    if (nt)
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_xupd<KCV, true>), dim3(nblk), dim3(ST_THREADS), 0, s, gi))
    else
        FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_xupd<KCV, false>), dim3(nblk), dim3(ST_THREADS), 0, s, gi))
}

void GmLaunch::finish_x(const GmInst* gi, hipStream_t s)
{
    hipLaunchKernelGGL(k_gm_finish_x, dim3(1), dim3(64), 0, s, gi);
}

void GmLaunch::finalize(const GmInst* gi, int nblk, int kc, hipStream_t s)
{
    FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_finalize<KCV>), dim3(nblk), dim3(ST_THREADS), 0, s, gi));
}

void GmLaunch::event_prep(const GmInst* gi, int vec, long long step, hipStream_t s)
{
    hipLaunchKernelGGL(k_gm_event_prep, dim3(1), dim3(64), 0, s, gi, vec, step);
}

void GmLaunch::event_copy(const GmInst* gi, int nblk, int kc, hipStream_t s)
{
    FTGCR_KC_SWITCH(kc, hipLaunchKernelGGL((k_gm_event_copy<KCV>), dim3(nblk), dim3(ST_THREADS), 0, s, gi));
}

void GmLaunch::event_inject(const GmInst* gi, int grid, const long long* idx, const unsigned char* bits,
                            long long count, long long start, int bit, hipStream_t s)
{
    hipLaunchKernelGGL(k_gm_event_inject, dim3(grid), dim3(256), 0, s, gi, idx, bits, count, start, bit);
}

// ---------------------------------------------------------------------------
// bandwidth probe: a plain streaming copy, the reference for what a kernel
// that reads and writes each byte once can reach on this device
// ---------------------------------------------------------------------------

// Each thread moves COPY_UNROLL 16-byte vectors, a block's vectors
// contiguous per unrolled step (full 1 KiB wave segments); all loads of a
// thread are issued before its first store.
constexpr int COPY_UNROLL = 4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_bw_copy(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                 long long nvec)
{
    const long long base = (long long)blockIdx.x * (256 * COPY_UNROLL) + threadIdx.x;
    u32x4 v[COPY_UNROLL];
#pragma unroll
    for (int u = 0; u < COPY_UNROLL; ++u) {
        const long long q = base + (long long)u * 256;
        const long long qc = q < nvec ? q : nvec - 1;   // clamped: branch-free loads
        v[u] = __builtin_nontemporal_load(&src[qc]);
    }
#pragma unroll
    for (int u = 0; u < COPY_UNROLL; ++u) {
        const long long q = base + (long long)u * 256;
        if (q < nvec) __builtin_nontemporal_store(v[u], &dst[q]);
    }
}

void launch_bw_copy(const void* src, void* dst, long long bytes, hipStream_t s)
{
    const long long nvec = bytes / 16;
    const long long blocks = (nvec + 256 * COPY_UNROLL - 1) / (256 * COPY_UNROLL);
    hipLaunchKernelGGL(k_bw_copy, dim3((unsigned)blocks), dim3(256), 0, s, (const u32x4*)src, (u32x4*)dst, nvec);
}

}  // namespace ftgcr
