// Device code shared by the step kernels and the resident kernel: wave
// reductions, row constants of both meshes, and the decisions of Algorithm 1
// on the solve's control state.
#pragma once

#include <cstddef>

#include "ftgcr_internal.h"

namespace ftgcr {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ int find_inst(const int* blk0, int n, int b)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (blk0[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Pointers that pass through LDS (per-block tables of the direction
// vectors) or through an empty asm statement come back as generic pointers,
// and accesses through them compile to flat instructions, which count
// against both the memory and the LDS counters: every LDS access and wave
// shuffle after them would wait for all outstanding HBM traffic.  The
// vectors are in global memory; these views say so.
template <typename T>
using gptr = const __attribute__((address_space(1))) T*;

template <typename T>
using gptr_mut = __attribute__((address_space(1))) T*;

template <typename T>
__device__ __forceinline__ gptr<T> as_global(const T* p)
{
    return (gptr<T>)p;
}

template <typename T>
__device__ __forceinline__ gptr_mut<T> as_global_mut(T* p)
{
    return (gptr_mut<T>)p;
}

// The value is formed here: its arithmetic is not moved to where it is used
// (which would keep all operands instead of the result), and what follows from
// it is not formed once before the step loop (and kept).
template <typename V>
__device__ __forceinline__ void settle(V& v)
{
    asm volatile("" : "+v"(v));
}

template <int CTRL>
__device__ __forceinline__ double dpp_mov_f64(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double lane_read(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the 64 lanes as a pairwise tree in lane order,
// ((v0 + v1) + (v2 + v3)) + ..., bitwise equal in every lane: DPP moves
// pair lanes l ^ 1 and l ^ 2 (quad permutes), then quads and half rows
// (half-row and row mirrors: every lane of a quad, then of a half row,
// holds the same value, so a mirror pairs the right partial sums; a + b and
// b + a round alike); the four row sums are read by readlane.  No LDS
// traffic.  Every lane must be active.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_mov_f64<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_mov_f64<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_mov_f64<0x141>(v);   // row_half_mirror
    v += dpp_mov_f64<0x140>(v);   // row_mirror
    return (lane_read(v, 0) + lane_read(v, 16)) + (lane_read(v, 32) + lane_read(v, 48));
}

// Sum over a 256-thread block; every thread gets the result.
__device__ __forceinline__ double block_sum(double v, double* sh)
{
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    return ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// Most empty rows of a half column in the template of depth H (the next
// smaller depth holds anything shorter).
constexpr int pad_rows(int H)
{
    return H == 4 ? 4 : H == 8 ? 5 : H == 16 ? 9 : H == 24 ? 9 : H == 28 ? 5 : H == 32 ? 5 : 9;
}

// Per-column constants: hill_amp * h at the five horizontal positions and
// the metric factors of the faces.
struct ColW {
    double hw, he, hs, hn, hc;
    double gx, gys, gyn, gz;
};

__device__ __forceinline__ ColW col_weights(const Geo& g, int i, int j)
{
    ColW c;
    const int iw = (i == 0) ? g.nx - 1 : i - 1;
    c.hw = g.hx[(long long)j * g.nx + iw];
    c.he = g.hx[(long long)j * g.nx + i];
    c.hs = g.hy[(long long)j * g.nx + i];
    c.hn = g.hy[(long long)(j + 1) * g.nx + i];
    c.hc = g.hc[(long long)j * g.nx + i];
    c.gx = g.Gx[j];
    c.gys = g.Gy[j];
    c.gyn = g.Gy[j + 1];
    c.gz = g.Gz[j];
    return c;
}

// Per-column constants of a row of A.  A horizontal face weight is
// G * (1 + h * g_k) (metric G, hill term h, vertical decay g_k at the cell's
// level), so the horizontal part of a row splits into a level-independent
// sum and a second one scaled by g_k:
//   sum_f W_f x_f = (Gx (x_w + x_e) + Gy_s x_s + Gy_n x_n)
//                 + g_k (Gx h_w x_w + Gx h_e x_e + Gy_s h_s x_s + Gy_n h_n x_n)
// and the horizontal part of the diagonal is h0 + g_k h1.  The column solve
// forms the same diagonal from the same constants, so P's diagonal is A's
// bit for bit.
struct RowC {
    double gx, gys, gyn;     // face metrics
    double cw, ce, cs, cn;   // metric * hill term of the four side faces
    double h0, h1;           // horizontal diagonal = h0 + g_k h1
    double gz, hc;           // vertical face weight = gz (1 + hc g_face)
};

__device__ __forceinline__ RowC row_consts(const ColW& c)
{
    RowC r;
    r.gx = c.gx;
    r.gys = c.gys;
    r.gyn = c.gyn;
    r.cw = c.gx * c.hw;
    r.ce = c.gx * c.he;
    r.cs = c.gys * c.hs;
    r.cn = c.gyn * c.hn;
    r.h0 = ((c.gx + c.gx) + c.gys) + c.gyn;
    r.h1 = ((c.gx * (c.hw + c.he) + c.gys * c.hs) + c.gyn * c.hn);
    r.gz = c.gz;
    r.hc = c.hc;
    return r;
}

// Vertical face weight of face f (between levels f-1 and f); 0 at the
// bottom (f = 0) and top (f = nz) faces.
__device__ __forceinline__ double vface(const RowC& r, double gf, int f, int nz)
{
    return (f > 0 && f < nz) ? r.gz * fma(r.hc, gf, 1.0) : 0.0;
}

// The same constants in binary32, for the stencil and column solve of the
// mixed form (binary32 vectors): there L(e) is stored in binary32, so
// forming it in binary32 arithmetic changes it by the order of that
// rounding, at half the vector-ALU cost of FP64 (row_consts32 below).
struct RowCf {
    float gx, gys, gyn, cw, ce, cs, cn, h0, h1, gz, hc;
};

template <typename AT>
struct RowOf;
template <>
struct RowOf<double> {
    using type = RowC;
};
template <>
struct RowOf<float> {
    using type = RowCf;
};

// The binary32 row constants straight from the binary32 hill tables (the
// per-row metric factors rounded from FP64), in the same operation order as
// row_consts: the binary32 stencil and column solve read half the table
// bytes, and their diagonals agree with each other as the FP64 ones do.
__device__ __forceinline__ RowCf row_consts32(const Geo& g, int i, int j)
{
    const int iw = (i == 0) ? g.nx - 1 : i - 1;
    const float hw = g.hx32[(long long)j * g.nx + iw];
    const float he = g.hx32[(long long)j * g.nx + i];
    const float hs = g.hy32[(long long)j * g.nx + i];
    const float hn = g.hy32[(long long)(j + 1) * g.nx + i];
    RowCf r;
    r.gx = (float)g.Gx[j];
    r.gys = (float)g.Gy[j];
    r.gyn = (float)g.Gy[j + 1];
    r.cw = r.gx * hw;
    r.ce = r.gx * he;
    r.cs = r.gys * hs;
    r.cn = r.gyn * hn;
    r.h0 = ((r.gx + r.gx) + r.gys) + r.gyn;
    r.h1 = ((r.gx * (hw + he) + r.gys * hs) + r.gyn * hn);
    r.gz = (float)g.Gz[j];
    r.hc = g.hc32[(long long)j * g.nx + i];
    return r;
}

template <typename AT>
__device__ __forceinline__ typename RowOf<AT>::type row_consts_for(const Geo& g, int i, int j)
{
    if constexpr (sizeof(AT) == 4) return row_consts32(g, i, j);
    else return row_consts(col_weights(g, i, j));
}

// Row constants of the column solve on either mesh: the octahedral mesh
// reads its per-point sums (only h0, h1, gz and hc are used by the solve).
template <typename AT>
__device__ __forceinline__ typename RowOf<AT>::type col_consts_for(const Geo& g, int i, int j)
{
    if (g.mesh == FTGCR_MESH_OCTAHEDRAL) {
        typename RowOf<AT>::type r = {};
        if constexpr (sizeof(AT) == 8) {
            r.h0 = g.oh0[i];
            r.h1 = g.oh1[i];
            r.gz = g.ogz[i];
            r.hc = g.ohc[i];
        } else {
            r.h0 = g.oh0_32[i];
            r.h1 = g.oh1_32[i];
            r.gz = g.ogz32[i];
            r.hc = g.ohc32[i];
        }
        return r;
    }
    return row_consts_for<AT>(g, i, j);
}

__device__ __forceinline__ float vface(const RowCf& r, float gf, int f, int nz)
{
    return (f > 0 && f < nz) ? r.gz * fmaf(r.hc, gf, 1.0f) : 0.0f;
}

// Wavefront shifts by one lane (DPP): lane l receives lane l-1's value
// (shift_up) or lane l+1's (shift_down); lanes with no source get 0.  Every
// lane of the wavefront must be active.
__device__ __forceinline__ double lane_shift(double v, int ctrl_up)
{
    const long long b = __double_as_longlong(v);
    int lo, hi;
    if (ctrl_up) {
        lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x138, 0xF, 0xF, false);        // wave_shr:1
        hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xF, 0xF, false);
    } else {
        lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x130, 0xF, 0xF, false);        // wave_shl:1
        hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xF, 0xF, false);
    }
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ float lane_shift(float v, int ctrl_up)
{
    const int b = __float_as_int(v);
    const int r = ctrl_up ? __builtin_amdgcn_update_dpp(0, b, 0x138, 0xF, 0xF, false)
                          : __builtin_amdgcn_update_dpp(0, b, 0x130, 0xF, 0xF, false);
    return __int_as_float(r);
}

__device__ __forceinline__ float lane_read(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// A table entry of the octahedral mesh in the arithmetic type: the FP64
// table, or its binary32 copy (rounded to nearest) for binary32 arithmetic.
template <typename AT>
__device__ __forceinline__ AT oct_tab(const double* d, const float* f, long long q)
{
    if constexpr (sizeof(AT) == 8) return d[q];
    else return f[q];
}

__device__ __forceinline__ int other_r(int a, int b)
{
    for (int q = 0; q < 3; ++q)
        if (q != a && q != b) return q;
    return 0;
}

__device__ __forceinline__ void assign_slots(SolveState* st, int k)
{
    const int s0 = st->slot[0];
    int q = 1;
    for (int l = 0; l <= k; ++l)
        if (l != s0) st->slot[q++] = l;
}

// Basis buffers after uslot[0], `last` at the end: the first pass of a cycle
// writes its e (uslot[1]) before the decision that retires the backup, so
// the previous cycle's p^0 must not come first.
__device__ __forceinline__ void assign_uslots(SolveState* st, int k, int last)
{
    const int s0 = st->uslot[0];
    int q = 1;
    for (int l = 0; l <= k + 1; ++l)
        if (l != s0 && l != last) st->uslot[q++] = l;
    if (last != s0) st->uslot[q] = last;
}

// sum_{l = lo .. hi} beta_l p^l over the basis: the coefficient of u_j.
__device__ __forceinline__ double basis_coef(const SolveState* st, int j, int lo, int hi)
{
    double c = 0.0;
    for (int l = lo > j ? lo : j; l <= hi; ++l) c = fma(st->beta[l], st->bm[l][j], c);
    return c;
}

// ---------------------------------------------------------------------------
// decisions (single thread of the last block)
// ---------------------------------------------------------------------------

// The control state staged in LDS for a reduction block.  Every field read
// by the decision logic would otherwise be a dependent round trip to memory
// (and a read after a store to another field of the same type must go
// back to memory); instead each of the first ST_WORDS threads loads one
// 8-byte word of the state (all fields before the detection log) together
// with the block's other loads, the decision runs on the LDS copy, and the
// words are stored back once.  Barriers separate the word-wise copies from
// the field accesses.
constexpr int ST_WORDS = (int)(offsetof(SolveState, log) / 8);
static_assert(offsetof(SolveState, log) % 8 == 0, "state words");
static_assert(ST_WORDS <= RED_THREADS, "one word per thread");

__device__ __forceinline__ long long state_word_load(const SolveState* g)
{
    const gptr<long long> w = as_global(reinterpret_cast<const long long*>(g));
    return ((int)threadIdx.x < ST_WORDS) ? w[threadIdx.x] : 0;
}

__device__ __forceinline__ void state_word_stage(SolveState* s, long long w)
{
    if ((int)threadIdx.x < ST_WORDS) reinterpret_cast<long long*>(s)[threadIdx.x] = w;
}

__device__ __forceinline__ void state_word_store(SolveState* g, const SolveState* s)
{
    if ((int)threadIdx.x < ST_WORDS)
        as_global_mut(reinterpret_cast<long long*>(g))[threadIdx.x] = reinterpret_cast<const long long*>(s)[threadIdx.x];
}

__device__ inline void rollback(SolveState* st)
{
    st->slot[0] = st->b_slot0;
    assign_slots(st, st->k);
    st->uslot[0] = st->b_uslot0;
    assign_uslots(st, st->k, st->b_uslot0);
    st->r_cur = st->r_bak;
    st->r_dst = other_r(st->r_cur, st->r_cur);
    st->x_base = st->x_bak;
    st->x_base_nu = 0;
    st->rr_old = st->b_rr;
    st->beta_num = st->b_beta_num;
    st->d_cur = st->b_d0;
    st->d[0] = st->b_d0;
    st->accepted = st->b_accepted;
    st->nu = 0;
}

// After the initial residual and P^{-1} r^0: <r^0, r^0>, the exit test, and
// the initial known-good state.
__device__ inline void decide_init(SolveState* st, double rn, double rs)
{
    st->rr_new = rn;
    st->rr_old = rs;
    if (rs <= st->T) {
        st->status = FTGCR_CONVERGED;
        st->x_final_hi = -1;
    }
    st->b_rr = rs;
    st->b_accepted = st->accepted;
    st->b_slot0 = st->slot[0];
    st->b_uslot0 = st->uslot[0];
    st->r_bak = st->r_cur;
    st->x_bak = st->x_base;
}

// One step's decision: exit test first, then the monotone residual-norm
// fault test with rollback to the backup, else (first pass of a cycle) the
// new backup.  rn: <r+, r+> of the unrounded update (detector), rs: of the
// stored r+ (exit test and next reference); equal in FP64.
// `log` is the state's detection log (st itself may be a staged copy
// without one), or null where another block keeps it.
__device__ inline void decide_step(SolveState* st, DetectRec* log, double rn, double rs, double* hist,
                            long long hist_cap)
{
    const int nu = st->nu;
    st->s += 1;
    st->e_ok = 0;
    const long long s = st->s;
    if (st->d_cur == 0.0) {   // <L p, L p> = 0: beta undefined
        st->status = FTGCR_BREAKDOWN;
        st->x_final_hi = nu - 1;
        st->active = 0;
        return;
    }
    if (nu == 0) st->cycles += 1;
    if (s <= hist_cap) hist[s - 1] = rn;
    st->beta[nu] = -st->beta_num / st->d_cur;
    st->rr_new = rn;
    if (rs <= st->T) {
        st->accepted += 1;
        st->rr_old = rs;
        st->r_cur = st->r_dst;
        st->status = FTGCR_CONVERGED;
        st->x_final_hi = nu;
        st->active = 0;
        return;
    }
    if (st->ft && !(rn < st->rr_old)) {   // the norm did not decrease (NaN included)
        const long long pos = st->accepted + 1;
        const int stag = (pos == st->last_rb_pos) && !st->events_since_rb;
        st->detections += 1;
        if (st->log_len < LOG_CAP) {
            const int at = st->log_len++;
            if (log != nullptr) {
                DetectRec& rec = log[at];
                rec.step = s;
                rec.nu = nu;
                rec.action = stag;
                rec.rr_old = st->rr_old;
                rec.rr_new = rn;
            }
        }
        if (!stag) {
            rollback(st);
            st->last_rb_pos = pos;
            st->events_since_rb = 0;
            st->active = 0;
            if (s >= st->max_steps) {
                st->status = FTGCR_MAX_STEPS;
                st->x_final_hi = -1;
            }
            return;
        }
        st->stagnation_accepts += 1;
    }
    if (st->ft && nu == 0) {   // this pass opens a cycle: it becomes the backup
        st->b_rr = st->rr_old;
        st->b_beta_num = st->beta_num;
        st->b_d0 = st->d_cur;
        st->b_accepted = st->accepted;
        st->b_slot0 = st->slot[0];
        st->b_uslot0 = st->uslot[0];
        st->r_bak = st->r_cur;
        st->x_bak = st->x_base;
    }
    st->accepted += 1;
    st->rr_old = rs;
    st->r_cur = st->r_dst;
    st->active = 1;
    st->e_ok = 1;
    if (s >= st->max_steps) {
        st->status = FTGCR_MAX_STEPS;
        st->x_final_hi = nu;
        st->active = 0;
    }
}

// Pass and cycle bookkeeping after a step's new direction (p^k opens the next
// cycle); it depends on no product, so it can run before they are known.
__device__ inline void next_pass(SolveState* st)
{
    const int nu = st->nu;
    if (nu + 1 == st->k) {
        st->x_base = st->x_dst;
        st->x_base_nu = 0;
        st->slot[0] = st->slot[st->k];
        assign_slots(st, st->k);
        const int old = st->uslot[0];
        st->uslot[0] = st->uslot[st->k + 1];
        assign_uslots(st, st->k, old);
        st->nu = 0;
        st->r_dst = other_r(st->r_cur, st->r_bak);
    } else {
        st->nu = nu + 1;
        st->r_dst = st->r_cur;
    }
}

// After the new direction: the next beta's inner products, then the
// bookkeeping.
__device__ inline void decide_beta(SolveState* st, double num, double dn, int init)
{
    st->beta_num = num;
    st->d_cur = dn;
    if (init) {
        st->d[0] = dn;
        st->b_beta_num = num;
        st->b_d0 = dn;
        st->r_dst = other_r(st->r_cur, st->r_bak);
        return;
    }
    next_pass(st);
    st->d[st->nu] = dn;
}

// The new direction p^{nu+1} = e + sum_l alpha_l p^l over the basis and, in a
// cycle's last pass, the iterate update: thread t <= nu + 1 of a block forms
// coefficient t.
__device__ inline void basis_row(SolveState* st, int nu, int t)
{
    if (t <= nu) {
        double c = 0.0;
        for (int l = t; l <= nu; ++l) c = fma(st->alpha[l], st->bm[l][t], c);
        st->bm[nu + 1][t] = c;
        if (nu + 1 == st->k) st->xc[t] = basis_coef(st, t, st->x_base_nu, nu);
    } else if (t == nu + 1) {
        st->bm[nu + 1][nu + 1] = 1.0;
    }
}

}  // namespace ftgcr
