// The resident kernel: many steps of Algorithm 1 in one launch, for problems
// whose columns fit the registers of the GPU.
//
// On grids of up to a few million cells a step of the streaming kernels
// (kernels.hip) is five launches that each last a few microseconds: launch,
// drain and memory latency, not bytes.  Here one block per CU keeps its tile of
// whole columns for the whole solve (r, L(p^nu) and the column solve's pivots
// in registers), so that a step is three exchanges between the blocks and
// otherwise local work:
//
//   1  r+ = r + beta L(p^nu), e = P^{-1} r+; <r+, r+> and the tile's rim of e
//   2  L(e) and <L(e), L(p^l)>
//   3  L(p^{nu+1}); <r+, L(p^{nu+1})>, <L(p^{nu+1}), L(p^{nu+1})>
//
// and every block takes the step's decisions itself, on its own copy of the
// control state, from the same sums added in the same order.
//
// Exchanges go through memory with agent-scope atomic loads and stores
// (write-through, read from the point of coherence) and without fences: a
// release or acquire fence writes back or drops a die's whole L2 (32 us a
// round on 256 blocks, against 2.8 us).  A block's partial sum is published as
// two 64-bit words, each half of the value under the round's number, so the
// reader polls the data themselves.  The rim of e is written to an r buffer
// not otherwise in use (R[r_dst]; the kernel reaches the R buffers through
// such loads and stores only) and has arrived there before the block
// publishes its round-1 words.  Two sets of words in turn suffice: a block
// that publishes round n + 2 has seen every block's round n + 1, which they
// publish after reading round n.
//
// Measured, us a step (streaming kernels -> here): 64 x 32 x 8 FP64 22.9 -> 8.8
// (of them about 6 in the three exchanges), 256 x 128 x 32 FP64 42 -> 22,
// O40 x 51 FP64 41.6 -> 26, 301 x 151 x 41 binary32 55.6 -> 34, O80 x 51 binary32
// 46.8 -> 30.  What bounds a step here: the exchanges' round trips to the
// point of coherence, the rim's (a write, then neighbours' reads: 5-9 us on
// 256 blocks), and instruction issue at one or two wavefronts per SIMD.
//
// All blocks of a launch have to run at once: the launch is cooperative, one
// block per CU at most, and every wait is bounded (a wait that ends in vain
// sets SolveState::res_fail and the block leaves).  Before anything else all
// blocks come to one verdict on whether they are all there: where another
// stream's work keeps blocks from starting that long, the launch ends with the
// solve as it was (RES_LATE) and the host goes on in the streaming kernels.
#include <algorithm>

#include "device.h"

namespace ftgcr {

namespace {

typedef unsigned long long u64;

// LDS of a CU
constexpr size_t RES_LDS = 160 * 1024;

// wall_clock64 ticks (100 MHz) a block waits for the others: 5 s
constexpr u64 WAIT_TICKS = 500000000ull;

__device__ __forceinline__ u64 word_load(const u64* p)
{
    return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void word_store(u64* p, u64 v)
{
    __hip_atomic_store(as_global_mut(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether the pivots wait in LDS: where the half column's five vectors leave
// the registers short (512 a lane at up to four wavefronts a block, else 256)
constexpr bool pivots_in_lds(int elem, int H, int maxw) { return H * elem >= (maxw == 8 ? 64 : 192); }

// A wave-uniform pointer held in scalar registers.
template <typename P>
__device__ __forceinline__ P* uniform(P* p)
{
    const u64 b = (u64)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return (P*)(((u64)hi << 32) | lo);
}

// The element `at` bytes into a field, through a scalar base.
template <typename T>
__device__ __forceinline__ gptr<T> elem(const T* base, unsigned at)
{
    return (gptr<T>)((gptr<char>)as_global((const char*)base) + at);
}

template <typename T>
__device__ __forceinline__ gptr_mut<T> elem_mut(T* base, unsigned at)
{
    return (gptr_mut<T>)((gptr_mut<char>)as_global_mut((char*)base) + at);
}

// The same, at the point of coherence.
template <typename T>
__device__ __forceinline__ T far_load(const T* base, unsigned at)
{
    return __hip_atomic_load(elem(base, at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ void far_store(T* base, unsigned at, T v)
{
    __hip_atomic_store(elem_mut(base, at), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Where a block's words of a round lie: [parity][copy][value][block][half].
__device__ __forceinline__ size_t word_at(unsigned seq, int copy, int value, int block)
{
    return ((((size_t)(seq & 1) * RES_COPIES + copy) * NV_MAX + value) * RES_BLOCKS + block) * 2;
}

// Whether all blocks of the launch run: an exchange of round `seq` without
// values, and one verdict on it for all blocks, which the first block that knows
// sets (one that has seen every block for it, one that has waited in vain
// against).  Every thread of the block calls it; -1: the verdict was for it, but
// the words did not come.  (Out of line: inlined it moves the step loop's
// registers about, 256 x 128 x 32 22.5 -> 22.9 us a step.)
__device__ __noinline__ int all_there(u64* xw, unsigned* gate, unsigned seq, int lb, int nblk, bool none, int* sh)
{
    const int tid = threadIdx.x;
    if (tid < RES_COPIES) word_store(xw + word_at(seq, tid, 0, lb), (u64)seq << 32);
    for (int turn = 0;; ++turn) {
        if (tid == 0) sh[0] = none ? 0 : 1;
        __syncthreads();
        if (!none) {
            u64 began = 0;
            for (int b = tid; b < nblk; b += blockDim.x) {
                const u64* p = xw + word_at(seq, lb & (RES_COPIES - 1), 0, b);
                for (int spin = 0; (unsigned)(word_load(p) >> 32) != seq; ++spin) {
                    if ((spin & 255) != 255) continue;
                    const u64 now = wall_clock64();
                    if (began == 0) began = now;
                    if (now - began > WAIT_TICKS) {
                        sh[0] = 0;
                        break;
                    }
                }
            }
        }
        __syncthreads();
        const int all = sh[0];
        if (tid == 0) {
            const unsigned mine = (seq << 1) | (unsigned)all;
            unsigned u = __hip_atomic_load(as_global(gate), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            while ((u >> 1) != (mine >> 1)) {
                const unsigned v = atomicCAS(gate, u, mine);
                u = v == u ? mine : v;
            }
            sh[1] = (int)(u & 1);
        }
        __syncthreads();
        if (!sh[1]) return 0;
        if (all) return 1;
        if (turn > 0) return -1;   // (another block has read them all: the second time they are there)
        __syncthreads();
    }
}

// Nothing moves across: without it the scheduler starts the loads of all
// rows at once and spills what they return.
__device__ __forceinline__ void fence_rows()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace

// A wavefront holds RES_COLS columns, lanes 0..31 their lower halves, lanes
// 32..63 the upper ones: the column solve's ownership, used for every pass.
// A half's rows run from its outer end to the middle of the column, row H - 1
// being the lower half's top level or the upper half's bottom one; a half of
// fewer than H levels starts with empty rows, which hold 0, have weights 0
// and address the first level (a store there comes before that level's own).
// Lat-lon: the wavefronts of a block are consecutive rows of the same 32
// longitudes; octahedral: a block is consecutive points.  Lanes without a
// column follow the last one's addresses, store nothing and are left out of
// the sums.
template <typename T, int H, int MESH, int MAXW>
__global__ __launch_bounds__(64 * MAXW) void k_resident(const Inst<T>* insts, const int* blk0, int n,
                                                        ResidentArgs arg, int ncache)
{
    using CT = T;
    constexpr bool OCT = MESH == FTGCR_MESH_OCTAHEDRAL;
    // rows whose neighbour loads are in flight together
    constexpr int HH = H % 2 == 0 && H > 16 ? H / 2 : H;
    constexpr int CH = OCT ? (H <= 8 ? H : (H % 8 == 0 ? 8 : 7)) : (MAXW == 4 ? HH : (H <= 8 ? H : (H % 8 == 0 ? 8 : 7)));
    static_assert(H % CH == 0, "chunks tile the half column");
    __shared__ long long s_words[ST_WORDS];   // the state before its log
    SolveState& s_st = *reinterpret_cast<SolveState*>(s_words);
    __shared__ double s_wp[NV_MAX][MAXW];
    __shared__ double s_sum[NV_MAX];
    // per half and row: the vertical decay at the face towards the middle with
    // a 1 (both 0 at the bottom and top faces and in empty rows), the decay at
    // the level with a 1 (0 in empty rows)
    __shared__ CT s_face[2][H][2], s_lev[2][H][2];
    __shared__ T* s_R[3];
    __shared__ T* s_U[KMAX + 2];
    __shared__ T* s_AP[KMAX + 1];
    __shared__ T* s_ap[KMAX + 1];   // this step's L(p^l) and basis
    __shared__ T* s_u[KMAX + 2];
    __shared__ int s_fail, s_there[2];
    // the blocks' partials of up to arg.nvmax sums, e of the tile, the pivots where
    // registers are short, then L(p^l) of the first `ncache` l (read twice a
    // step)
    constexpr bool INV_LDS = pivots_in_lds((int)sizeof(T), H, MAXW);
    extern __shared__ double s_dyn[];

    const int m = find_inst(blk0, n, blockIdx.x);
    const Inst<T>& in = insts[m];
    const int lb = blockIdx.x - blk0[m];
    SolveState* gst = in.st;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nthr >> 6;
    const int nblk = in.nblk_res;
    const int lgb = 32 - __builtin_clz(nblk - 1 > 0 ? nblk - 1 : 1);   // blocks of a value: 1 << lgb slots
    u64* const xw = (u64*)in.xw;
    const int leave = arg.s_stop < 0 ? in.res_leave : arg.leave;
    const Geo& g = in.g;
    const int nx = g.nx, ny = g.ny, nz = g.nz, ncols = g.ncols;
    const CT opsig = (CT)g.opsig;
    const int h = (nz + 1) >> 1;

    for (int q = tid; q < ST_WORDS; q += nthr)
        s_words[q] = as_global(reinterpret_cast<const long long*>(gst))[q];
    for (int t = tid; t < 2 * H; t += nthr) {
        const int up = t / H, q = t % H;
        const int a = q - (H - (up ? nz - h : h));   // levels from the outer end
        const int k = up ? nz - 1 - a : a, f = up ? k : k + 1;
        const bool real = a >= 0, inner = real && f > 0 && f < nz;
        s_face[up][q][0] = inner ? (CT)g.gf[f] : CT(0);
        s_face[up][q][1] = inner ? CT(1) : CT(0);
        s_lev[up][q][0] = real ? (CT)g.gc[k] : CT(0);
        s_lev[up][q][1] = real ? CT(1) : CT(0);
    }
    if (tid <= KMAX + 1) {
        s_U[tid] = in.U[tid];
        if (tid <= KMAX) s_AP[tid] = in.AP[tid];
        if (tid < 3) s_R[tid] = in.R[tid];
    }
    if (tid == 0) s_fail = 0;
    double* const hist = in.hist;
    const long long hist_cap = lb == 0 ? in.hist_cap : 0;   // one block keeps the history and the log
    DetectRec* const log = lb == 0 ? gst->log : nullptr;
    double* const s_sv = s_dyn;                                // [sum][block]
    T* const s_e = reinterpret_cast<T*>(s_dyn + arg.nvmax * RES_BLOCKS);   // [wavefront][row][lane]
    CT* const s_inv = reinterpret_cast<CT*>(s_e + nw * H * 64) + w * H * 64 + lane;
    T* const s_cache = s_e + nw * H * 64 * (INV_LDS ? 2 : 1) + w * H * 64 + lane;   // [l][wavefront][row][lane]
    const int cache_step = nw * H * 64;
    __syncthreads();

    unsigned seq = s_st.res_seq;
    if (s_st.status == RUNNING) {   // before anything is written
        seq += 1;
        const int there = all_there(xw, &gst->res_gate, seq, lb, nblk, leave == RES_LATE, s_there);
        if (there <= 0) {
            if (tid == 0) atomicMax(&gst->res_fail, there < 0 ? RES_BROKEN : RES_LATE);
            return;
        }
    }

    // this lane's column and its half
    const int upper = lane >> 5;
    const int l32 = lane & 31;
    int i, j, last = 31;
    bool valid;
    if constexpr (OCT) {
        const int p = lb * (RES_COLS * nw) + w * RES_COLS + l32;
        valid = p < nx;
        i = valid ? p : nx - 1;
        j = 0;
    } else {
        const int bx = lb % in.rtx, by = lb / in.rtx;
        const int ii = bx * RES_COLS + l32, jj = by * nw + w;
        valid = ii < nx && jj < ny;
        i = ii < nx ? ii : nx - 1;
        j = jj < ny ? jj : ny - 1;
        const int left = nx - 1 - bx * RES_COLS;
        last = left < 31 ? left : 31;
    }
    const int nmine = upper ? nz - h : h;
    const bool stores = valid && nmine > 0;
    // element offsets of the rows (bytes, by T's and by the iterate's size)
    unsigned at[H];
    {
        const int col = OCT ? i : j * nx + i;
#pragma unroll
        for (int q = 0; q < H; ++q) {
            int a = q - (H - nmine);
            a = a < 0 ? 0 : a;
            const int k = nmine == 0 ? 0 : (upper ? nz - 1 - a : a);
            at[q] = (unsigned)(col + ncols * k) * (unsigned)sizeof(T);
        }
    }
    const typename RowOf<CT>::type rc = col_consts_for<CT>(g, i, j);
    auto face = [&](int q) -> CT { return rc.gz * fma(rc.hc, s_face[upper][q][0], s_face[upper][q][1]); };
    auto diagonal = [&](int q, CT w_out, CT w_in) -> CT {
        return opsig * ((fma(s_lev[upper][q][0], rc.h1, rc.h0) + w_out) + w_in);
    };
    // octahedral: the neighbours (an empty slot: this point, weights 0)
    int nd[OCT ? NB_OCT : 1];
    CT ngw[OCT ? NB_OCT : 1], nhw[OCT ? NB_OCT : 1];
    if constexpr (OCT) {
#pragma unroll
        for (int q = 0; q < NB_OCT; ++q) {
            const long long slot = (long long)q * ncols + i;
            const int nb = g.onb[slot];
            nd[q] = nb >= 0 ? (nb - i) * (int)sizeof(T) : 0;
            ngw[q] = nb >= 0 ? oct_tab<CT>(g.ogw, g.ogw32, slot) : CT(0);
            nhw[q] = nb >= 0 ? oct_tab<CT>(g.ohw, g.ohw32, slot) : CT(0);
        }
    }

    // the column's pivots: elimination from both ends to the lower half's top
    // row, as the streaming column pass does it (reciprocals kept)
    CT inv[INV_LDS ? 1 : H];
    auto pivot = [&](int q) -> CT {
        if constexpr (INV_LDS) return s_inv[q * 64];
        else return inv[q];
    };
    CT meet_den;
    {
        CT carry = 0, w_out = 0, mm = 1, mw = 0;
#pragma unroll
        for (int q = 0; q < H; ++q) {
            const CT w_in = face(q);
            const CT mk = diagonal(q, w_out, w_in) + w_out * carry;
            if (q == H - 1) {
                mm = mk;
                mw = w_in;
            }
            CT iv;
            if constexpr (sizeof(CT) == 4) iv = __builtin_amdgcn_rcpf(mk);
            else iv = CT(1) / mk;
            iv = q >= H - nmine ? iv : CT(0);
            carry = -w_in * iv;
            w_out = w_in;
            settle(iv);
            if constexpr (INV_LDS) s_inv[q * 64] = iv;
            else inv[q] = iv;
            if (q % 4 == 3) fence_rows();
        }
        const CT zx = __shfl_xor(carry, 32);
        meet_den = mm + mw * zx;
    }

    fence_rows();
    T r[H], ap[H];
    auto load_state = [&]() {   // r and L(p^nu) as the state names them
        const T* rp = uniform(s_R[s_st.r_cur]);
        const int nu = s_st.nu;
        for (int l = 0; l < nu && l < ncache; ++l) {
            const T* al = uniform(s_AP[s_st.slot[l]]);
#pragma unroll
            for (int q = 0; q < H; ++q) s_cache[l * cache_step + q * 64] = *elem(al, at[q]);
        }
        const T* app = uniform(s_AP[s_st.slot[nu]]);
#pragma unroll
        for (int q = 0; q < H; ++q) {
            r[q] = far_load(rp, at[q]);
            ap[q] = *elem(app, at[q]);
        }
        if (nu < ncache) {
#pragma unroll
            for (int q = 0; q < H; ++q) s_cache[nu * cache_step + q * 64] = ap[q];
        }
#pragma unroll
        for (int q = 0; q < H; ++q) {
            r[q] = q >= H - nmine ? r[q] : T(0);
            ap[q] = q >= H - nmine ? ap[q] : T(0);
            settle(r[q]);
            settle(ap[q]);
        }
    };
    load_state();

    // Publish the block's partials (s_wp summed over its wavefronts) as the
    // next round; collect() waits for every block's and leaves the sums in
    // s_sum.
    auto publish = [&](int nv) {
        __syncthreads();
        seq += 1;
        int first = tid;
        settle(first);
        for (int t = first; t < nv * RES_COPIES; t += nthr) {
            const int q = t / RES_COPIES, copy = t % RES_COPIES;
            double v = 0.0;
            for (int z = 0; z < nw; ++z) v += s_wp[q][z];
            const u64 b = (u64)__double_as_longlong(v), tag = (u64)seq << 32;
            u64* p = xw + word_at(seq, copy, q, lb);
            word_store(p, tag | (b & 0xffffffffull));
            word_store(p + 1, tag | (b >> 32));
        }
    };
    auto collect = [&](int nv) -> bool {
        const u64* base = xw + word_at(seq, lb & (RES_COPIES - 1), 0, 0);
        const int items = nv << lgb, mask = (1 << lgb) - 1;
        constexpr int G = 4;
        int first = tid;
        settle(first);   // (no address of these is kept across the steps)
        for (int t0 = first; t0 < items; t0 += G * nthr) {
            u64 a[G], b[G];
            int slot[G];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const int t = t0 + u * nthr;
                const bool is = t < items && (t & mask) < nblk;
                slot[u] = is ? (t >> lgb) * RES_BLOCKS + (t & mask) : -1;
                a[u] = b[u] = (u64)seq << 32;
            }
            u64 began = 0;
            for (int spin = 0;; ++spin) {
                bool all = true;
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    if (slot[u] >= 0) {
                        const u64* p = base + 2 * (size_t)slot[u];
                        a[u] = word_load(p);
                        b[u] = word_load(p + 1);
                    }
                }
#pragma unroll
                for (int u = 0; u < G; ++u)
                    all = all && (unsigned)(a[u] >> 32) == seq && (unsigned)(b[u] >> 32) == seq;
                if (all) break;
                if ((spin & 255) == 255) {
                    const u64 now = wall_clock64();
                    if (began == 0) began = now;
                    else if (now - began > WAIT_TICKS) {
                        s_fail = 1;
                        break;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (slot[u] >= 0)
                    s_sv[slot[u]] = __longlong_as_double((long long)((a[u] & 0xffffffffull) | (b[u] << 32)));
        }
        __syncthreads();
        if (s_fail) return false;
        for (int q = w; q < nv; q += nw) {
            double v = 0.0;
            for (int b = lane; b < nblk; b += 64) v += s_sv[q * RES_BLOCKS + b];
            v = wave_sum(v);
            if (lane == 0) s_sum[q] = v;
        }
        __syncthreads();
        return true;
    };
    auto gave_up = [&](int how) {
        if (tid == 0) atomicMax(&gst->res_fail, how);
    };
    auto decide = [&](double rn, double rs) {   // thread 0, on this block's copy of the state
        decide_step(&s_st, log, rn, rs, hist, hist_cap);
    };
    // L(p^l), l < nu, of this step
    auto row_of = [&](int l, T (&v)[H]) {
        if (l < ncache) {
#pragma unroll
            for (int q = 0; q < H; ++q) v[q] = s_cache[l * cache_step + q * 64];
        } else {
            const T* const al = uniform((const T*)s_ap[l]);
#pragma unroll
            for (int q = 0; q < H; ++q) v[q] = *elem(al, at[q]);
        }
    };
    // a lane's part of sum q of this block
    auto partial = [&](int q, double v) {
        v = wave_sum(valid ? v : 0.0);
        if (lane == 0) s_wp[q][w] = v;
    };

    // The detector compares norms of r summed in one order: where these two (of
    // r and of the backup's) come from the streaming kernels, they are formed
    // anew here.
    if (s_st.status == RUNNING && (arg.s_stop < 0 ? in.res_new_norms : arg.new_norms) != 0) {
        const T* rp = uniform(s_R[s_st.r_bak]);
        double a0 = 0.0, a1 = 0.0;
#pragma unroll
        for (int q = 0; q < H; ++q) {
            a0 = fma((double)r[q], (double)r[q], a0);
            const double b = q >= H - nmine ? (double)far_load(rp, at[q]) : 0.0;
            a1 = fma(b, b, a1);
            settle(a0);
            settle(a1);
        }
        partial(0, a0);
        partial(1, a1);
        publish(2);
        if (!collect(2)) return gave_up(RES_BROKEN);
        if (tid == 0) {
            s_st.rr_old = s_sum[0];
            s_st.b_rr = s_sum[1];
        }
        __syncthreads();
    }

    // kernel timing (options.profile_kernels): the three rounds' durations on
    // block 0, in the records of the streaming kernels they stand for
    u64 tick = 0, ticks[3] = {0, 0, 0};
    int counts[3] = {0, 0, 0};
    auto timed = [&](int phase, long long step) {
        if (!arg.time_mask) return;
        const u64 now = wall_clock64();
        if (phase >= 0 && (arg.time_mask & (2 << phase)) && (arg.time_stride < 2 || step % arg.time_stride == 0)) {
            ticks[phase] += now - tick;
            counts[phase] += 1;
        }
        tick = now;
    };

    const long long s_stop = arg.s_stop < 0 ? in.res_stop : arg.s_stop;
    while (s_st.status == RUNNING && s_st.s < s_stop) {
        const long long step = s_st.s + 1;
        timed(-1, step);
        const int nu = __builtin_amdgcn_readfirstlane(s_st.nu);
        const double d_cur = s_st.d_cur;
        if (d_cur == 0.0) {   // the decision records the breakdown
            __syncthreads();
            if (tid == 0) decide(0.0, 0.0);
            __syncthreads();
            continue;
        }
        const double beta = -s_st.beta_num / d_cur;
        const bool lastp = nu == s_st.k - 1;
        T* const rim = uniform(s_R[s_st.r_dst]);
        // the decision below may move the slots (rollback): this step's now
        if (tid <= KMAX + 1) {
            s_u[tid] = s_U[s_st.uslot[tid]];
            if (tid <= KMAX) s_ap[tid] = s_AP[s_st.slot[tid]];
        }
        if (nu == 0) {   // the cycle's r, the backup if this pass stands
            T* const rold = uniform(s_R[s_st.r_cur]);
            if (stores) {
#pragma unroll
                for (int q = 0; q < H; ++q) far_store(rold, at[q], r[q]);
            }
        }

        // 1: update and column solve
        T e[H];
        double acc_new = 0.0, acc_st = 0.0;
        {
            CT w_out = 0, carry = 0, fk = 0;
#pragma unroll
            for (int q = 0; q < H; ++q) {
                const double v = fma(beta, (double)ap[q], (double)r[q]);
                const T sv = (T)v;
                r[q] = sv;
                acc_new = fma(v, v, acc_new);
                acc_st = fma((double)sv, (double)sv, acc_st);
                if (q % 8 == 0) {
                    fence_rows();
                    settle(acc_new);
                    settle(acc_st);
                }
                fk = (CT)sv + w_out * carry;
                w_out = face(q);
                carry = fk * pivot(q);
                e[q] = carry;
                settle(r[q]);
                settle(e[q]);
            }
            const CT ex = __shfl_xor(carry, 32);
            const CT xm = (fk + w_out * ex) / meet_den;
            const CT xl = __shfl_xor(xm, 32);
            const CT xu = e[H - 1] + w_out * pivot(H - 1) * xl;
            CT xv = upper ? xu : xm;
            e[H - 1] = xv;
#pragma unroll
            for (int q = H - 2; q >= 0; --q) {
                if (q % 8 == 7) fence_rows();
                xv = e[q] + face(q) * pivot(q) * xv;
                e[q] = xv;
                settle(e[q]);
            }
        }
        // the rim to memory, the tile to LDS
        {
            fence_rows();
            bool out = stores;
            if constexpr (!OCT) out = out && (w == 0 || w == nw - 1 || l32 == 0 || l32 == last);
            {
#pragma unroll
                for (int q = 0; q < H; ++q) s_e[(w * H + q) * 64 + lane] = e[q];
            }
            if (out) {
#pragma unroll
                for (int q = 0; q < H; ++q) far_store(rim, at[q], e[q]);
            }
        }
        partial(0, acc_new);
        partial(1, acc_st);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the rim has arrived
        publish(2);
        {
            T* const ub = uniform(s_u[nu + 1]);
            if (stores) {
#pragma unroll
                for (int q = 0; q < H; ++q) *elem_mut(ub, at[q]) = e[q];
            }
        }
        if (!collect(2)) return gave_up(RES_BROKEN);
        const double rn = s_sum[0], rs = s_sum[1];
        timed(0, step);

        // 2: L(e) and its products
        T le[H];
        {
            const T partner = __shfl_xor(e[H - 1], 32);   // across the halves' meeting face
            CT w_out = 0;
#pragma unroll
            for (int c0 = 0; c0 < H; c0 += CH) {
                fence_rows();
                CT t1[CH], t2[CH];
                if constexpr (OCT) {
                    // neighbours in this block from LDS, then the others from
                    // memory (all in flight together)
                    T v[NB_OCT][CH];
#pragma unroll
                    for (int s = 0; s < NB_OCT; ++s) {
                        int d = nd[s];
                        settle(d);
                        const int p = w * RES_COLS + l32 + d / (int)sizeof(T);   // the neighbour in the block's points
                        const bool here = p >= 0 && p < RES_COLS * nw;
                        const int hl = here ? ((p >> 5) * H) * 64 + (p & 31) + (lane & 32) : lane;
#pragma unroll
                        for (int c = 0; c < CH; ++c) v[s][c] = s_e[hl + (c0 + c) * 64];
                    }
#pragma unroll
                    for (int s = 0; s < NB_OCT; ++s) {
                        int d = nd[s];
                        settle(d);
                        const int p = w * RES_COLS + l32 + d / (int)sizeof(T);
                        if (p < 0 || p >= RES_COLS * nw) {
#pragma unroll
                            for (int c = 0; c < CH; ++c) v[s][c] = far_load(rim, at[c0 + c] + (unsigned)d);
                        }
                    }
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        t1[c] = CT(0);
                        t2[c] = CT(0);
#pragma unroll
                        for (int s = 0; s < NB_OCT; ++s) {
                            t1[c] = fma(ngw[s], v[s][c], t1[c]);
                            t2[c] = fma(nhw[s], v[s][c], t2[c]);
                        }
                    }
                } else {
                    // vx: the tile's west edge value in lane 0 of a half, its
                    // east one in the lane after the last column, or in lane
                    // 31 if that is the last
                    T vs[CH], vn[CH], vx[CH];
                    const bool west = l32 == 0, east = l32 == (last < 31 ? last + 1 : 31);
                    if (j > 0) {
                        if (w == 0) {
#pragma unroll
                            for (int c = 0; c < CH; ++c) vs[c] = far_load(rim - nx, at[c0 + c]);
                        } else {
#pragma unroll
                            for (int c = 0; c < CH; ++c) vs[c] = s_e[((w - 1) * H + c0 + c) * 64 + lane];
                        }
                    } else {
#pragma unroll
                        for (int c = 0; c < CH; ++c) vs[c] = T(0);
                    }
                    if (j < ny - 1) {
                        if (w == nw - 1) {
#pragma unroll
                            for (int c = 0; c < CH; ++c) vn[c] = far_load(rim + nx, at[c0 + c]);
                        } else {
#pragma unroll
                            for (int c = 0; c < CH; ++c) vn[c] = s_e[((w + 1) * H + c0 + c) * 64 + lane];
                        }
                    } else {
#pragma unroll
                        for (int c = 0; c < CH; ++c) vn[c] = T(0);
                    }
#pragma unroll
                    for (int c = 0; c < CH; ++c) vx[c] = T(0);
                    if (west || east) {
                        const int i_first = i - (l32 < last ? l32 : last), i_last = i_first + last;
                        const int di = west ? (i_first == 0 ? nx - 1 : -1) : (i_last == nx - 1 ? 0 : i_last + 1) - i;
                        unsigned d = (unsigned)(di * (int)sizeof(T));
                        settle(d);
#pragma unroll
                        for (int c = 0; c < CH; ++c)
                            vx[c] = far_load(rim, at[c0 + c] + d);
                    }
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const int q = c0 + c;
                        const T up = lane_shift(e[q], 1), dn = lane_shift(l32 > last ? vx[c] : e[q], 0);
                        const CT xwv = west ? vx[c] : up;
                        const CT xev = (l32 == 31) ? vx[c] : dn;
                        CT a1 = rc.gx * (xwv + xev);
                        a1 = fma(rc.gys, vs[c], a1);
                        a1 = fma(rc.gyn, vn[c], a1);
                        CT a2 = rc.cw * xwv;
                        a2 = fma(rc.ce, xev, a2);
                        a2 = fma(rc.cs, vs[c], a2);
                        a2 = fma(rc.cn, vn[c], a2);
                        t1[c] = a1;
                        t2[c] = a2;
                    }
                }
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const int q = c0 + c;
                    const CT w_in = face(q);
                    const CT x_out = (q > 0) ? e[q > 0 ? q - 1 : 0] : CT(0);
                    const CT x_in = (q == H - 1) ? partner : e[q + 1 < H ? q + 1 : q];
                    CT o = fma(s_lev[upper][q][0], t2[c], t1[c]);
                    o = fma(w_out, x_out, o);
                    o = fma(w_in, x_in, o);
                    le[q] = s_lev[upper][q][1] * fma(diagonal(q, w_out, w_in), e[q], -o);
                    w_out = w_in;
                    settle(le[q]);
                }
            }
        }
        fence_rows();
        for (int l = 0; l < nu; ++l) {
            T v[H];
            row_of(l, v);
            double a0 = 0.0, a1 = 0.0;
#pragma unroll
            for (int q = 0; q < H; q += 2) {
                a0 = fma((double)le[q], (double)v[q], a0);
                a1 = fma((double)le[q + 1], (double)v[q + 1], a1);
            }
            partial(l, a0 + a1);
        }
        {
            double a0 = 0.0, a1 = 0.0;
#pragma unroll
            for (int q = 0; q < H; q += 2) {
                a0 = fma((double)le[q], (double)ap[q], a0);
                a1 = fma((double)le[q + 1], (double)ap[q + 1], a1);
            }
            partial(nu, a0 + a1);
        }
        publish(nu + 1);
        if (tid == 0) decide(rn, rs);   // while the products travel
        if (!collect(nu + 1)) return gave_up(RES_BROKEN);
        timed(1, step);
        if (s_st.status != RUNNING || !s_st.active) {
            if (s_st.status == RUNNING) load_state();   // rolled back: the restored r and L(p^0)
            continue;
        }
        if (tid <= nu) s_st.alpha[tid] = -s_sum[tid] / s_st.d[tid];
        if (tid == 0) s_st.x_dst = (s_st.x_base == s_st.x_bak) ? 1 - s_st.x_base : s_st.x_base;
        __syncthreads();

        // 3: L(p^{nu+1}) and its products
        fence_rows();
        {
            double a[H];
#pragma unroll
            for (int q = 0; q < H; ++q) a[q] = (double)le[q];
            for (int l = 0; l < nu; ++l) {
                const double al = s_st.alpha[l];
                T v[H];
                row_of(l, v);
#pragma unroll
                for (int q = 0; q < H; ++q) a[q] = fma(al, (double)v[q], a[q]);
            }
            const double al = s_st.alpha[nu];
            double a_num = 0.0, a_d = 0.0;
#pragma unroll
            for (int q = 0; q < H; ++q) {
                ap[q] = s_lev[upper][q][1] * (T)fma(al, (double)ap[q], a[q]);
                settle(ap[q]);
                a_num = fma((double)r[q], (double)ap[q], a_num);
                a_d = fma((double)ap[q], (double)ap[q], a_d);
            }
            partial(0, a_num);
            partial(1, a_d);
        }
        publish(2);
        basis_row(&s_st, nu, tid);
        {
            T* const aout = uniform(s_ap[nu + 1]);
            const int l = lastp ? 0 : nu + 1;   // its place in the next step
            if (l < ncache) {
#pragma unroll
                for (int q = 0; q < H; ++q) s_cache[l * cache_step + q * 64] = ap[q];
            }
            if (stores) {
#pragma unroll
                for (int q = 0; q < H; ++q) *elem_mut(aout, at[q]) = ap[q];
            }
        }
        __syncthreads();
        // p^k and the iterate from the basis: its update is summed by itself,
        // so the iterate is rounded once a cycle and not once a term
        if (lastp) {
            const double* const xb = uniform(in.X[s_st.x_base]);
            double* const xo = uniform(in.X[s_st.x_dst]);
            const T* const ue = uniform((const T*)s_u[nu + 1]);
            T* const pout = uniform(s_u[nu + 2]);
            // x is loaded with the chunk's first values where registers allow,
            // else after its sums: 120 x 60 x 60 25.5 -> 25.2 us a step, 256 x 128
            // x 32 22.65 -> 22.56, but 301 x 151 x 41 binary32 (eight wavefronts)
            // 42.8 -> 43.9
            constexpr bool XF = MAXW == 4;
            constexpr unsigned XS = sizeof(double) / sizeof(T);
            constexpr int CL = MAXW == 4 && H <= 16 ? H : (H <= 8 ? H : (H % 8 == 0 ? 8 : 7));
#pragma unroll
            for (int c0 = 0; c0 < H; c0 += CL) {
                fence_rows();
                double p[CL], d[CL], x[CL];
                unsigned ax[CL];
                T v[2][CL], ev[CL];
                const T* u0 = uniform((const T*)s_u[0]);
#pragma unroll
                for (int c = 0; c < CL; ++c) {
                    ax[c] = at[c0 + c];
                    settle(ax[c]);
                    ax[c] *= XS;
                    v[0][c] = *elem(u0, at[c0 + c]);
                    if (XF) x[c] = *elem(xb, ax[c]);
                    ev[c] = *elem(ue, at[c0 + c]);
                }
#pragma unroll
                for (int c = 0; c < CL; ++c) {
                    p[c] = (double)ev[c];
                    d[c] = 0.0;
                }
                for (int q = 0; q <= nu; q += 2) {
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        if (q + b <= nu) {
                            if (q + b + 1 <= nu) {
                                const T* const un = uniform((const T*)s_u[q + b + 1]);
#pragma unroll
                                for (int c = 0; c < CL; ++c) v[b ^ 1][c] = *elem(un, at[c0 + c]);
                            }
                            const double pj = s_st.bm[nu + 1][q + b], xj = s_st.xc[q + b];
#pragma unroll
                            for (int c = 0; c < CL; ++c) {
                                p[c] = fma(pj, (double)v[b][c], p[c]);
                                d[c] = fma(xj, (double)v[b][c], d[c]);
                            }
                        }
                    }
                }
                if (!XF)
#pragma unroll
                    for (int c = 0; c < CL; ++c) x[c] = *elem(xb, ax[c]);
                if (stores) {
#pragma unroll
                    for (int c = 0; c < CL; ++c) {
                        // (xo may be xb: a level is updated by its own row
                        // alone, an empty row of an earlier chunk would add
                        // its increment once more)
                        const int q = c0 + c;
                        if (q < pad_rows(H) && q < H - nmine) continue;
                        *elem_mut(pout, at[q]) = (T)p[c];
                        *elem_mut(xo, ax[c]) = x[c] + d[c];
                    }
                }
            }
        }
        __syncthreads();   // bm, xc and the bases are read before the slots move
        if (tid == 0) next_pass(&s_st);
        if (!collect(2)) return gave_up(RES_BROKEN);
        if (tid == 0) {
            s_st.beta_num = s_sum[0];
            s_st.d_cur = s_sum[1];
            s_st.d[s_st.nu] = s_sum[1];
        }
        timed(2, step);
        __syncthreads();
    }
    if (leave == RES_BROKEN) return gave_up(RES_BROKEN);
    // r back to its buffer, the state to memory (one block's copy: all agree)
    if (stores) {
        T* const rp = uniform(s_R[s_st.r_cur]);
#pragma unroll
        for (int q = 0; q < H; ++q) far_store(rp, at[q], r[q]);
    }
    if (lb == 0) {
        __syncthreads();
        if (tid == 0) {
            as_global_mut(gst)->res_seq = seq;
            for (int q = 0; q < 3; ++q) {
                s_st.res_ticks[q] = ticks[q];
                s_st.res_counts[q] = counts[q];
            }
        }
        __syncthreads();
        // (not the first word: another block may still set res_fail there)
        static_assert(offsetof(SolveState, res_ticks) == 8, "res_fail and res_seq are the first word");
        for (int q = tid + 1; q < ST_WORDS; q += nthr)
            as_global_mut(reinterpret_cast<long long*>(gst))[q] = s_words[q];
    }
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------

// Registers bound the depth: a half column of H levels holds five vectors of
// H values per lane (r, L(p), the pivots, e, L(e)), 512 registers at one
// wavefront per SIMD (four to a block), 256 at two; the deepest of each spill
// some (resident_step_us).
bool resident_shape(int mesh, int nx, int ny, int H, int elem_bytes, int cus, int waves, int* rtx, int* nblk)
{
    const int hmax = waves <= 4 ? (elem_bytes == 4 ? 48 : 32) : (elem_bytes == 4 ? 28 : 16);
    const int most = cus < RES_BLOCKS ? cus : RES_BLOCKS;
    if (H > hmax) return false;
    const bool oct = mesh == FTGCR_MESH_OCTAHEDRAL;
    const long long wide = oct ? (long long)RES_COLS * waves : RES_COLS;
    const long long tx = (nx + wide - 1) / wide;
    const long long blocks = tx * (oct ? 1 : (ny + waves - 1) / waves);
    if (blocks > most) return false;
    *rtx = (int)tx;
    *nblk = (int)blocks;
    return true;
}

int resident_waves(int mesh, int nx, int ny, int H, int elem_bytes, int cus, int* rtx, int* nblk)
{
    for (int w = 1; w <= RES_WAVES; w *= 2)
        if (resident_shape(mesh, nx, ny, H, elem_bytes, cus, w, rtx, nblk)) return w;
    return 0;
}

// Measured at k = 3 (MI355X), a step by template depth (4, 8, 16, 24, 28, 32, 40,
// 48) and wavefronts per block (1, 2, 4, 8).  It hardly depends on the grid: a
// block runs its columns' rows in sequence whatever the number of blocks.  What
// steps up between the columns of a row is registers: at eight wavefronts FP64
// halves of 16 rows spill 113 to 202 vector registers beyond their 256, binary32
// ones of 24 and 28 rows 117 to 224; at four FP64 ones of 32 rows up to 16,
// binary32 ones of 40 rows 26 and of 48 rows 65.  (Binary32 halves of 32 rows at
// eight spilled 288: 78 us lat-lon and 84 octahedral, where the largest grid of
// that form streams in 75.)
double resident_step_us(int mesh, int H, int elem_bytes, int waves)
{
    static const unsigned char us[2][2][4][8] = {   // mesh; FP64, binary32; wavefronts; depth
        {{{11, 12, 15, 18, 20, 21}, {13, 14, 18, 21, 23, 25}, {14, 16, 22, 27, 30, 31}, {18, 22, 37}},
         {{11, 12, 14, 17, 19, 20, 23, 28}, {13, 14, 17, 20, 22, 23, 28, 33}, {14, 15, 19, 24, 26, 28, 34, 42},
          {16, 19, 25, 41, 60}}},
        {{{11, 12, 15, 19, 22, 24}, {13, 15, 19, 24, 26, 29}, {14, 17, 25, 29, 36, 41}, {19, 25, 50}},
         {{12, 12, 15, 19, 21, 22, 27, 33}, {13, 14, 18, 22, 25, 26, 33, 40}, {14, 16, 19, 24, 28, 30, 38, 46},
          {16, 19, 25, 50, 68}}}};
    const int depths[] = {4, 8, 16, 24, 28, 32, 40, 48};
    int d = 0, w = 0;
    while (d < 7 && depths[d] < H) ++d;
    while (w < 3 && (1 << w) < waves) ++w;
    return us[mesh == FTGCR_MESH_OCTAHEDRAL ? 1 : 0][elem_bytes == 4 ? 1 : 0][w][d];
}

namespace {

template <typename T>
const void* resident_kernel(int mesh, int H, int waves)
{
#define FTGCR_RES(HV)                                                                                     \
    case HV:                                                                                              \
        if (waves <= 4)                                                                                   \
            return mesh == FTGCR_MESH_OCTAHEDRAL ? (const void*)k_resident<T, HV, FTGCR_MESH_OCTAHEDRAL, 4> \
                                                 : (const void*)k_resident<T, HV, FTGCR_MESH_LATLON, 4>;  \
        if constexpr (HV <= (sizeof(T) == 4 ? 28 : 16))                                                   \
            return mesh == FTGCR_MESH_OCTAHEDRAL ? (const void*)k_resident<T, HV, FTGCR_MESH_OCTAHEDRAL, 8> \
                                                 : (const void*)k_resident<T, HV, FTGCR_MESH_LATLON, 8>;  \
        return nullptr;
    switch (H) {
        FTGCR_RES(4)
        FTGCR_RES(8)
        FTGCR_RES(16)
        FTGCR_RES(24)
        FTGCR_RES(28)
        FTGCR_RES(32)
    case 40:
        if constexpr (sizeof(T) == 4) {
            if (waves <= 4)
                return mesh == FTGCR_MESH_OCTAHEDRAL ? (const void*)k_resident<T, 40, FTGCR_MESH_OCTAHEDRAL, 4>
                                                     : (const void*)k_resident<T, 40, FTGCR_MESH_LATLON, 4>;
        }
        return nullptr;
    case 48:
        if constexpr (sizeof(T) == 4) {
            if (waves <= 4)
                return mesh == FTGCR_MESH_OCTAHEDRAL ? (const void*)k_resident<T, 48, FTGCR_MESH_OCTAHEDRAL, 4>
                                                     : (const void*)k_resident<T, 48, FTGCR_MESH_LATLON, 4>;
        }
        return nullptr;
    default: return nullptr;
    }
#undef FTGCR_RES
}

}  // namespace

namespace {

// Dynamic LDS of a launch: the partials of k + 1 sums, then vectors of the
// block's tile: e, the pivots of deep FP64 halves, and as many L(p^l) as the
// CU's LDS still holds beside the kernel's own, at most k.
size_t resident_lds(const void* f, int H, int waves, int elem, int k, int* ncache)
{
    const size_t vec = (size_t)waves * H * 64 * elem;
    const size_t fixed = (size_t)(k + 1) * RES_BLOCKS * sizeof(double) + vec * (pivots_in_lds(elem, H, waves <= 4 ? 4 : 8) ? 2 : 1);
    hipFuncAttributes fa;
    *ncache = 0;
    if (hipFuncGetAttributes(&fa, f) != hipSuccess) {
        (void)hipGetLastError();
        return fixed;
    }
    const size_t used = fa.sharedSizeBytes + fixed;
    if (used < RES_LDS) *ncache = (int)std::min<size_t>((size_t)k, (RES_LDS - used) / vec);
    return fixed + *ncache * vec;
}

}  // namespace

template <typename T>
bool resident_fits(int mesh, int H, int waves, int nblk, int k)
{
    const void* f = resident_kernel<T>(mesh, H, waves);
    if (!f) return false;
    int dev = 0, coop = 0, cus = 0, per = 0, nc = 0;
    const size_t lds = resident_lds(f, H, waves, (int)sizeof(T), k, &nc);
    hipFuncAttributes fa;
    // (the limit of a launch's dynamic LDS belongs to the function, not to a
    // handle: all there is beside the kernel's own, whatever this one needs)
    if (hipGetDevice(&dev) != hipSuccess || hipFuncGetAttributes(&fa, f) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(RES_LDS - fa.sharedSizeBytes)) !=
            hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, waves * 64, lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return (long long)per * cus >= nblk;
}

template <typename T>
hipError_t resident_run(const Table<T>& tb, const int* blk0, int total_blocks, int mesh, int H, int waves,
                        ResidentArgs arg, hipStream_t s)
{
    const void* f = resident_kernel<T>(mesh, H, waves);
    const Inst<T>* inst = tb.inst;
    int n = tb.n, nc = 0;
    const size_t lds = resident_lds(f, H, waves, (int)sizeof(T), arg.nvmax - 1, &nc);
    void* args[] = {(void*)&inst, (void*)&blk0, (void*)&n, (void*)&arg, (void*)&nc};
    return hipLaunchCooperativeKernel(f, dim3(total_blocks), dim3(waves * 64), args, (unsigned)lds, s);
}

template bool resident_fits<double>(int, int, int, int, int);
template bool resident_fits<float>(int, int, int, int, int);
template hipError_t resident_run<double>(const Table<double>&, const int*, int, int, int, int, ResidentArgs,
                                          hipStream_t);
template hipError_t resident_run<float>(const Table<float>&, const int*, int, int, int, int, ResidentArgs,
                                          hipStream_t);

}  // namespace ftgcr
