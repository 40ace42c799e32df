// Internal types shared by the FT-GCR kernels and the host engine.
//
// One solve ("instance") keeps all of its control state on the device in a
// SolveState; the step kernels read it to find the pass index nu, the buffer
// roles and the scalars of Algorithm 1, so a step is the same fixed kernel
// sequence whatever happened before (rollbacks included) and can be enqueued
// or replayed without reading anything back.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/ftgcr.h"

namespace ftgcr {

constexpr int KMAX = FTGCR_KMAX;
constexpr int LOG_CAP = FTGCR_LOG_CAP;
constexpr int NV_MAX = KMAX + 2;     // reduction values per block
constexpr int DOT_ROW0 = 2;          // first partials row of the dots pass (rows 0, 1:
                                     // the column pass's, still unread when a
                                     // speculative dots pass runs)
constexpr int RUNNING = -1;

// Block shapes.  Column kernels: 256 threads = 4 waves, each wave owns 32
// columns (lanes 0..31 the lower half of each column, 32..63 the upper half).
constexpr int COL_THREADS = 256;
constexpr int COLS_PER_BLOCK = 128;

// Columns per block of the column pass: the binary32 form with half columns
// of at most 32 levels uses one lane per column (k_update_thomas1), the
// others two lanes per column.
inline int col_block_cols(int elem_bytes, int H)
{
    return (elem_bytes == 4 && H <= 32) ? COL_THREADS : COLS_PER_BLOCK;
}
// Stencil kernels: 64 longitudes x 4 latitudes per block, KC levels each.
constexpr int ST_TX = 64;
constexpr int ST_TY = 4;
constexpr int ST_THREADS = ST_TX * ST_TY;
constexpr int RED_THREADS = 1024;
// Partials per value after folding, and the blocks beyond which it pays (the
// whole reduction of 8192 blocks takes 4.8 us, a fold alone 4.7; at 18432 a step
// gains 2.4)
constexpr int RED_FOLD = 32;
constexpr int FOLD_BLOCKS = 16384;
// Octahedral mesh: neighbour slots per point (the triangulation's valence
// is at most 6); a block of the stencil kernels covers ST_THREADS
// consecutive points.
constexpr int NB_OCT = 6;
// Block orders of the stencil-grid launches (a block is a column tile times
// a chunk of levels; FTGCR_ORDER_* minus 1): tiles of a level chunk in a row
// (X); a tile's level chunks in a row (Z); as Z, with each accelerator die
// given one contiguous range of blocks (XCD).  Consecutive workgroups are
// placed on the XCDS dies round robin, each die with its own L2.
enum { ORD_X = 0, ORD_Z = 1, ORD_XCD = 2 };
constexpr int XCDS = 8;

struct DetectRec {
    long long step;
    int nu;
    int action;
    double rr_old, rr_new;
};

// Per-solve control state (device memory, written by single-thread kernel
// sections only).
struct SolveState {
    int res_fail;        // RES_LATE, RES_BROKEN: a resident kernel's block waited in vain
    unsigned res_seq;    // rounds of exchanges the resident kernels of this handle have run
    unsigned long long res_ticks[3];   // the last resident launch's timed rounds (100 MHz)
    int res_counts[3];
    unsigned res_gate;   // the last resident launch's verdict: its first round's number, doubled, + 1 if it went on
    int status;          // RUNNING or an FTGCR_* outcome
    int active;          // 1: this step goes on to P^{-1}, L and the new direction
    int nu;              // pass index of the current step
    int k;
    int ft;
    int mixed;
    int detections, stagnation_accepts, events_applied, events_since_rb;
    long long s;         // executed steps
    long long max_steps; // stop when s reaches this (global or round cap)
    long long accepted;
    long long cycles;
    long long last_rb_pos;
    double tol2;         // tol^2 (FP64) or inner tol^2 (mixed round)
    double T;            // exit threshold on <r,r>
    double RR;           // <R,R>
    double rt2;          // <r_t, r_t> of the last true-residual pass
    double rr_old, rr_new;
    double beta_num;     // <r, L p^nu>
    double d_cur;        // <L p^nu, L p^nu>
    double d[KMAX + 1];
    double beta[KMAX + 1];
    double alpha[KMAX + 1];
    // p^l = sum_{j <= l} bm[l][j] u_j over the cycle's basis u_0 = p^0,
    // u_j = e of its j-th step (bm[l][l] = 1): the directions after p^0 are
    // never stored, only p^k of a cycle's end, which opens the next one
    double bm[KMAX + 1][KMAX + 1];
    double xc[KMAX + 1]; // the cycle's iterate update sum_l beta_l p^l over the basis
    int slot[KMAX + 1];  // buffer index of L(p^l)
    int uslot[KMAX + 2]; // buffer index of u_l, l = 0..k; [k + 1]: where p^k is formed
    int r_cur, r_dst, r_bak;
    int x_base, x_base_nu, x_bak, x_dst;
    int x_final_hi;      // materialise x with beta_l p^l for l <= this at the end (basis sums)
    int b_slot0, b_uslot0;
    long long b_accepted;
    double b_rr, b_beta_num, b_d0;
    // fault-event staging (set by the event preparation kernel)
    int ev_ok;           // the event applies (solve still running)
    int ev_vec;
    int ev_copy;         // 1: copy src -> dst buffer before flipping; 2: form p^nu in u_nu's
    int ev_src, ev_dst;  // buffer indices for the copy
    int ev_usrc, ev_udst;   // and of p^0 with that of L(p^0)
    int ev_lo, ev_hi;    // x materialisation: beta terms l in [lo, hi)
    int log_len;
    int e_ok;            // 1: this step passed its tests, its e feeds a new direction
    DetectRec log[LOG_CAP];
};

// Geometry / coefficient tables of one grid (device, FP64).
struct Geo {
    int nx, ny, nz;
    int ncols;               // nx * ny
    long long n;             // nx * ny * nz
    double opsig;            // 1 + helmholtz
    const double* hx;        // [ny][nx]    hill_amp * h at east face (i+1/2, j)
    const double* hy;        // [ny+1][nx]  hill_amp * h at face (i, j-1/2)
    const double* hc;        // [ny][nx]    hill_amp * h at centre (i, j)
    const double* gc;        // [nz]        exp(-zeta_k / decay)
    const double* gf;        // [nz+1]      exp(-zeta_{k-1/2} / decay)
    const double* Gx;        // [ny]        dlat dz / (cos(lat_j) dlon)
    const double* Gy;        // [ny+1]      cos(lat_{j-1/2}) dlon dz / dlat, 0 at poles
    const double* Gz;        // [ny]        cos(lat_j) dlon dlat / dz
    // binary32 copies of the per-column hill tables, read by the binary32
    // stencil and column solve (half the bytes of the FP64 ones)
    const float* hx32;
    const float* hy32;
    const float* hc32;
    // octahedral mesh (mesh == FTGCR_MESH_OCTAHEDRAL; then nx = points per
    // level, ny = 1): per point and neighbour slot q (slot-major, [q][point])
    // the neighbour (-1: empty slot), the metric part of the face weight and
    // that times hill_amp * h at the face centre; per point the sums of both
    // over its slots, the vertical face metric (control area / dz) and
    // hill_amp * h at the point
    int mesh;
    const int* onb;
    const double* ogw;
    const double* ohw;
    const double* oh0;
    const double* oh1;
    const double* ogz;
    const double* ohc;
    // binary32 copies of the octahedral tables (rounded to nearest), read by
    // the binary32 stencil and column solve of the mixed form
    const float* ogw32;
    const float* ohw32;
    const float* oh0_32;
    const float* oh1_32;
    const float* ogz32;
    const float* ohc32;
};

// Everything one instance's kernels need (device copy per solve).
template <typename T>
struct Inst {
    Geo g;
    T* U[KMAX + 2];          // the cycle's basis: p^0 and every e since (SolveState::bm)
    T* AP[KMAX + 1];
    T* R[3];
    // octahedral mesh: L(e) of the step, stored by the dots pass and read by
    // the direction pass instead of a second indirect stencil (null on the
    // lat-lon mesh)
    T* LE;
    double* X[2];            // X[0]: caller's x, X[1]: workspace
    const double* rhs;
    SolveState* st;
    double* part;            // block partials [NV_MAX][pstride] (value-major)
    long long pstride;       // >= blocks of either grid
    double* hist;
    long long hist_cap;
    int nblk_col;            // blocks of the column grid
    int nblk_st;             // blocks of the stencil grid
    int kc;                  // stencil levels per block
    int tx, ty, tz;          // stencil tiles per dimension
    // the direction pass (the most registers per level) has its own level
    // tiling over the same columns
    int nblk_dir, kc_dir, tz_dir;
    // partials per value that the two grids' are folded to before the one-block
    // reductions (0: they read the blocks' own)
    int fold_st, fold_dir;
    // block orders (ORD_*) of the stencil grid and of the direction grid
    int ord_st, ord_dir;
    // the resident kernel's exchange words, blocks and tiles in x
    unsigned long long* xw;
    int nblk_res, rtx;
    // of a batch's launch (ResidentArgs::s_stop < 0): this member's
    int res_new_norms, res_leave;
    long long res_stop;
};

// FT-GMRES(k) control state of one solve (device memory; written by single
// threads of the one-block kernels, and by the event preparation kernel).
struct GmState {
    int status;          // RUNNING or an FTGCR_* outcome
    int active;          // 1: the cycle's steps run
    int j;               // step index inside the cycle
    int k, ft;
    int phase;           // next restart pass: GM_INIT, GM_CHECK (a cycle ended), GM_REDO (after a rollback)
    int jdone;           // steps of this cycle that count
    int cycle_end;       // 1: the cycle is complete, its correction is pending
    int capped;          // 1: the step cap cut the cycle
    int x_cur, x_bak, x_dst;
    int detections, stagnation_accepts, events_applied, events_since_rb;
    int log_len;
    int ev_ok, ev_vec, ev_copy, ev_src, ev_dst;
    long long s, max_steps, accepted, cycles, last_rb_pos, b_accepted;
    double tol2, T, RR;
    double rho2;         // explicit |R - A x|^2 of the cycle's start (or of the last check)
    double b_rho2;       // the backup's
    double rr_old;       // |g_j|^2 of the previous step (the detector's reference)
    double den[KMAX + 1];            // stored U[i] = den[i] * v_i (1 once stored normalised)
    double H[(KMAX + 1) * KMAX];     // Hessenberg, row-major with row stride KMAX, rotated in place
    double cs[KMAX], sn[KMAX];       // Givens rotations
    double g[KMAX + 1];              // rotated right-hand side, g_0 = |s|
    DetectRec log[LOG_CAP];
};

// Everything the FT-GMRES kernels of one solve need (device copy per solve).
struct GmInst {
    Geo g;
    double* U[KMAX + 1];     // Arnoldi vectors v_i (v_0 = s / |s|), stored scaled by den[i] until normalised
    double* Z[KMAX];         // z_i = P^{-1} v_i
    double* W;               // A z_j, then the orthogonalised vector
    double* X[2];            // X[0]: caller's x, X[1]: workspace
    const double* rhs;
    GmState* st;
    double* part;
    long long pstride;
    double* hist;
    long long hist_cap;
    int nblk_st, kc, tx, ty, tz;
    int ord;                 // block order (ORD_*) of the stencil kernels
};

// Launch table for combined (batched) launches: block b of a launch belongs
// to instance inst_of(b); blk0[m] is the first block of instance m.
template <typename T>
struct Table {
    const Inst<T>* inst;
    const int* blk0_col;     // n + 1 prefix sums (column grid)
    const int* blk0_st;      // n + 1 prefix sums (stencil grid)
    const int* blk0_dir;     // n + 1 prefix sums (direction-pass grid)
    int n;
    int mesh = 0;            // every instance's mesh (FTGCR_MESH_*)
    int precond = FTGCR_PRECOND_COLUMN;   // every instance's preconditioner
    // 1: some instance's columns belong to a smaller template depth than the
    // launch's (thomas_depth)
    int mixed_depth = 0;
};

// The resident kernel (resident.hip): whole columns kept in registers by
// blocks that stay on the GPU for many steps.  RES_COLS columns per wavefront
// (two lanes each), at most RES_WAVES wavefronts per block, at most
// RES_BLOCKS blocks.
constexpr int RES_COLS = 32;
constexpr int RES_WAVES = 8;
constexpr int RES_BLOCKS = 256;
// exchange words of a handle: two rounds in turn, each in RES_COPIES copies
// (every block writes all and reads one, so fewer blocks poll the same
// memory: 2.8 -> 2.5 us a round on 256 blocks), NV_MAX values per block, two
// tagged words a value
constexpr int RES_COPIES = 4;
constexpr size_t RES_WORDS = 2 * (size_t)RES_COPIES * NV_MAX * RES_BLOCKS * 2;
// Steps a launch runs at most before the host looks at the state, and more
// rounds than it exchanges (three a step and two before them)
constexpr long long RES_STEPS = 4096;
constexpr unsigned RES_ROUNDS = 3 * RES_STEPS + 4;
// SolveState::res_fail: a launch whose blocks did not all start in time has
// changed nothing but its exchange words; one that came apart later has
// broken the solve (gather_status then reports BROKEN for its status)
enum { RES_LATE = FTGCR_RESIDENT_LATE, RES_BROKEN = FTGCR_RESIDENT_BROKEN };
constexpr int BROKEN = -2;

// Wavefronts per block with which the resident kernel takes a problem of
// half columns of depth H on at most `cus` blocks (0: it does not), and its
// tile counts.
int resident_waves(int mesh, int nx, int ny, int H, int elem_bytes, int cus, int* rtx, int* nblk);
// The same for a given number of wavefronts per block (false: it does not).
bool resident_shape(int mesh, int nx, int ny, int H, int elem_bytes, int cus, int waves, int* rtx, int* nblk);
// About the microseconds a step takes there.
double resident_step_us(int mesh, int H, int elem_bytes, int waves);
// Whether the device can hold the kernel's blocks all at once.
template <typename T> bool resident_fits(int mesh, int H, int waves, int nblk, int k);
// What a launch runs: steps until every instance has left RUNNING or executed
// s_stop of them.
struct ResidentArgs {
    long long s_stop;  // < 0: each instance's own (Inst::res_stop, res_new_norms, res_leave)
    int nvmax;         // k + 1: the most sums in a round
    int new_norms;     // 1: form the state's norms of r anew first
    int time_mask, time_stride;   // options.profile_kernels
    int leave;         // RES_LATE, RES_BROKEN: all blocks leave so (ftgcr_debug_resident), 0: none
};
template <typename T>
hipError_t resident_run(const Table<T>& tb, const int* blk0, int total_blocks, int mesh, int H, int waves,
                        ResidentArgs arg, hipStream_t s);

// Kernel launchers (kernels.hip).
template <typename T> struct Launch {
    static void init_state(const Table<T>& tb, int k, int ft, int mixed, long long max_steps, double tol2,
                           int reset_counters, int grid, hipStream_t s);
    static void set_round(const Table<T>& tb, double tol2, long long max_steps, hipStream_t s);
    static void residual(const Table<T>& tb, int total_st_blocks, int kc, int store, int set_T, hipStream_t s);
    // update_thomas, stencil_dots and dir_update take optional events that
    // the dispatch itself stamps with its start and stop times
    static void update_thomas(const Table<T>& tb, int total_col_blocks, int H, int mode, hipStream_t s,
                              hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
    static void finish_col(const Table<T>& tb, int mode, hipStream_t s);
    // the state's norms in the column pass's order (single instance)
    static void norms(const Table<T>& tb, int total_col_blocks, int H, hipStream_t s);
    // spec = 1: before the step's decision, followed by finish_step
    static void stencil_dots(const Table<T>& tb, int total_st_blocks, int kc, int spec, hipStream_t s,
                             hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
    static void finish_step(const Table<T>& tb, hipStream_t s);   // finish_col + finish_alpha
    static void finish_alpha(const Table<T>& tb, hipStream_t s);
    static void finish_beta(const Table<T>& tb, int init, hipStream_t s);
    static void fold(const Table<T>& tb, int dir, int parts, int values, hipStream_t s);
    // after a resident launch that ended RES_LATE: before the next one
    static void resident_late(const Table<T>& tb, hipStream_t s);
    // nt_ap: load the L(p^l) with the non-temporal hint (nt_ap_hint)
    static void dir_update(const Table<T>& tb, int total_st_blocks, int kc, int init, bool nt_ap, hipStream_t s,
                           hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
    static void finalize_x(const Table<T>& tb, int total_st_blocks, int kc, hipStream_t s);
    // fault events (single instance)
    static void event_prep(const Table<T>& tb, int vec, hipStream_t s);
    static void event_copy(const Table<T>& tb, int grid, hipStream_t s);
    // again: a flip already counted, taken out or put back
    static void event_inject(const Table<T>& tb, int grid, const long long* idx, const unsigned char* bits,
                             long long count, long long start, int bit, bool again, hipStream_t s);
    static void beta_dots(const Table<T>& tb, int total_st_blocks, hipStream_t s);
    static void gather_status(const Table<T>& tb, long long* out, hipStream_t s);
    // parity entry points (FP64 only)
    static void debug_apply_A(const Table<T>& tb, int total_st_blocks, int kc, const double* in, double* out, hipStream_t s);
    static void debug_pinv(const Table<T>& tb, int total_col_blocks, int H, const double* in, double* out, hipStream_t s);
};

// FT-GMRES(k) launchers (kernels.hip); gi is the device copy of the solve's
// GmInst, `tb` the handle's single-instance table (geometry and column grid)
// for the column pass.
struct GmLaunch {
    static void init(const GmInst* gi, int k, int ft, long long max_steps, double tol2, hipStream_t s);
    static void residual(const GmInst* gi, int nblk_st, int kc, int mesh, hipStream_t s);
    static void restart(const GmInst* gi, hipStream_t s);
    static void precond(const Table<double>& tb, const GmInst* gi, int nblk_col, int H, hipStream_t s);
    // dots = 0: store A z_j only (the dots follow a fault event on it)
    // nt: the basis does not fit the cache (gm_nt_hint)
    static void stencil(const GmInst* gi, int nblk_st, int kc, int dots, int mesh, bool nt, hipStream_t s);
    static void dots(const GmInst* gi, int nblk_st, int kc, hipStream_t s);
    static void finish_h(const GmInst* gi, hipStream_t s);
    static void orth(const GmInst* gi, int nblk_st, int kc, bool nt, hipStream_t s);
    static void finish_step(const GmInst* gi, hipStream_t s);
    static void xupd(const GmInst* gi, int nblk_st, int kc, bool nt, hipStream_t s);
    static void finish_x(const GmInst* gi, hipStream_t s);
    static void finalize(const GmInst* gi, int nblk_st, int kc, hipStream_t s);
    static void event_prep(const GmInst* gi, int vec, long long step, hipStream_t s);
    static void event_copy(const GmInst* gi, int nblk_st, int kc, hipStream_t s);
    static void event_inject(const GmInst* gi, int grid, const long long* idx, const unsigned char* bits,
                             long long count, long long start, int bit, hipStream_t s);
};

// Plain streaming copy of `bytes` (a multiple of 16, 16-byte aligned
// pointers): the bandwidth probe.
void launch_bw_copy(const void* src, void* dst, long long bytes, hipStream_t s);

// Smallest supported register-array depth H >= levels per column half.
int thomas_depth(int nz);

// Whether the direction pass should load the L(p^l) with the non-temporal
// hint: when the k + 1 images of A p of all solves in flight (n_total
// entries of elem bytes each) exceed most of the 256 MB Infinity Cache, so
// the next dots pass would not find them there anyway.
inline bool nt_ap_hint(int k, long long n_total, int elem)
{
    return (double)(k + 1) * (double)n_total * elem > 192.0 * 1024 * 1024;
}

// Whether FT-GMRES should load its Krylov vectors so: when besides they are so
// long that the few a step writes and reads again (z_j, w, v_{j+1}) do not stay
// cached behind the others.  Below 32 MiB a vector the others are still found
// there in part: microseconds a step without and with the hint, k = 16, 300 x 150
// x 40 (14 MB a vector) 98, 108; O_90 x 51 (15) 97, 112; 430 x 215 x 40 (30) 184,
// 193; 480 x 240 x 40 (37) 218, 206; 480 x 240 x 60 (55) 325, 298; k = 8, 430 x
// 215 x 40 138, 146; 480 x 240 x 40 157, 156; 480 x 240 x 60 239, 223.
inline bool gm_nt_hint(int k, long long n)
{
    return nt_ap_hint(k, n, 8) && (double)n * 8.0 > 32.0 * 1024 * 1024;
}

}  // namespace ftgcr
