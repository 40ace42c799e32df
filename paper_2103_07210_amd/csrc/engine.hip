// Host engine and C ABI of libftgcr (see include/ftgcr.h).
//
// The engine builds the FP64 coefficient tables once per handle, lays the
// working vectors out in the caller's workspace, and drives a solve as a
// sequence of step launches on the handle's stream, or of launches of the
// resident kernel with many steps each.  All decisions of
// Algorithm 1 (exit, fault test, backup, rollback, cycle restart) are taken
// on the device; the host only enqueues steps, inserts the harness's fault
// events before the step they belong to, and reads one status word every
// `poll_steps` steps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <map>
#include <mutex>
#include <tuple>
#include <cstdio>
#include <cstddef>
#include <cstring>
#include <new>
#include <set>
#include <string>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "ftgcr_internal.h"

using namespace ftgcr;

namespace {

constexpr double kPi = 3.14159265358979323846;

// A named range on the ROCm tracer's timeline (rocprofv3 --marker-trace):
// solves, batches, autotuning and refinement rounds.  The allocation-free
// solve opens none.
struct TraceRange {
    explicit TraceRange(const char* name) { roctxRangePushA(name); }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange&) = delete;
    TraceRange& operator=(const TraceRange&) = delete;
};

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

thread_local std::string g_create_error;

}  // namespace

struct ftgcr_handle {
    ftgcr_grid grid{};
    ftgcr_coeffs co{};
    int precond = FTGCR_PRECOND_COLUMN;
    int precision = FTGCR_FP64;
    int kmax = 1;
    int device = 0;
    hipStream_t stream = nullptr;
    ftgcr_options opt{};
    std::string err;

    Geo geo{};
    double* tables = nullptr;       // device coefficient tables
    SolveState* st = nullptr;       // device control state
    void* inst = nullptr;           // device Inst<T> of the storage type
    Inst<double>* inst_dbg = nullptr;  // device Inst<double> for the parity entry points
    int* blk0 = nullptr;            // device {0, nblk_col, 0, nblk_st, 0, nblk_dir, 0, nblk_res}
    SolveState* st_host = nullptr;  // pinned copy for reading back
    hipEvent_t ev_start = nullptr, ev_stop = nullptr;

    long long* ev_idx = nullptr;    // device staging of fault-event entries
    unsigned char* ev_bits = nullptr;
    size_t ev_cap = 0;

    void* ws = nullptr;
    size_t ws_bytes = 0;

    // captured step sequence: `graph_steps` steps replayed as one graph
    hipStream_t cap_stream = nullptr;
    hipGraphExec_t graph = nullptr;
    int graph_steps = 0;
    bool graph_nt_ap = false;
    bool nt_ap = false;   // this solve's L(p^l) load hint (nt_ap_hint)

    // the resident kernel's shape (res_waves 0: this grid does not take it) and
    // exchange words (device)
    int res_waves = 0, nblk_res = 0, rtx = 0;
    double res_gain = 0.0;    // microseconds a step it gains, about
    int cus = 0;              // of the device
    bool no_resident = false; // a tuner is timing the streaming kernels
    unsigned long long* xw = nullptr;
    int test_launch = 0, test_outcome = 0;   // ftgcr_debug_resident

    int nblk_col = 0, nblk_st = 0, nblk_dir = 0;
    int fold_st = 0, fold_dir = 0;   // Inst's
    int kc = 1, tx = 1, ty = 1, tz = 1, H = 4, kc_dir = 1, tz_dir = 1;
    int tuned_kc = 0;   // from ftgcr_autotune (0: none)
    // block orders (ORD_*) of the stencil and direction grids, and
    // ftgcr_autotune's choice of them (-1: none)
    int ord_st = ORD_X, ord_dir = ORD_X;
    int tuned_ord_st = -1, tuned_ord_dir = -1;
    int tuned_batch_kc = 0;   // options.batch_levels_per_block as ftgcr_autotune_batch left it

    // kernel timing (options.profile_kernels)
    struct Pending {
        int cls;
        long long step;   // executed-step number the launch belongs to
        hipEvent_t a, b;
    };
    std::vector<hipEvent_t> ev_pool;
    size_t ev_next = 0;
    std::vector<Pending> pending;
    double kt_ms[3] = {0, 0, 0};
    long long kt_n[3] = {0, 0, 0};

    // FT-GMRES(k) control state (device), its instance record and a pinned
    // host copy, allocated with the handle
    GmState* gm_st = nullptr;
    GmInst* gm_inst = nullptr;
    GmState* gm_host = nullptr;

    // batched solves led by this handle: device tables kept between calls
    // (grown, never per call) and the captured step chunk of the last
    // launch table shape
    struct Batch {
        int cap = 0;
        Inst<double>* inst = nullptr;   // launch table (running members)
        int* blk0 = nullptr;            // its col, st and dir prefixes (cap+1 each)
        long long* status = nullptr;    // 2 per member
        Inst<double>* all = nullptr;    // every member, in order
        int* blk0_all = nullptr;
        hipGraphExec_t graph = nullptr;
        long long graph_key[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    } batch;
};

namespace {

ftgcr_status fail(ftgcr_handle* h, ftgcr_status code, const std::string& msg)
{
    if (h) h->err = msg;
    else g_create_error = msg;
    return code;
}

#define HIP_TRY(h, call)                                                                         \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess)                                                                    \
            return fail((h), FTGCR_E_HIP, std::string(#call) + ": " + hipGetErrorString(e_));     \
    } while (0)

// Great-circle distance to the hill centre in the haversine form, and the
// hill h = exp(-(gc / width)^2) (used only to tabulate the coefficients).
double hill_height(const ftgcr_coeffs& c, double lon, double lat)
{
    const double a = std::sin(0.5 * (lat - c.hill_lat));
    const double b = std::sin(0.5 * (lon - c.hill_lon));
    double root = std::sqrt(a * a + std::cos(lat) * std::cos(c.hill_lat) * b * b);
    root = std::min(root, 1.0);
    const double q = 2.0 * std::asin(root) / c.hill_width;
    return std::exp(-q * q);
}

// Autotuned levels per stencil block and block orders, per (mesh, nlon,
// nlat, nz, precision).
using TuneKey = std::tuple<int, int, int, int, int>;
struct Tuned {
    int kc = 0, ord_st = -1, ord_dir = -1;
};
std::mutex g_tune_mutex;
std::map<TuneKey, Tuned> g_tuned;

TuneKey tune_key(const ftgcr_handle* h)
{
    return TuneKey{h->geo.mesh, h->geo.nx, h->geo.ny, h->geo.nz, h->precision};
}

Tuned tuned_for(const ftgcr_handle* h)
{
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    auto it = g_tuned.find(tune_key(h));
    return it == g_tuned.end() ? Tuned{} : it->second;
}

int tuned_levels(const ftgcr_handle* h) { return tuned_for(h).kc; }

long long part_stride(const ftgcr_handle* h);

// Levels per stencil block: as many as keep >= 1024 blocks in flight (8 at
// most: deeper chunks raise register pressure more than they save halo).
// On the octahedral mesh the dots pass at 8 levels holds 181 registers, two
// waves per SIMD, against four waves at 4, and a point's tables are read once
// per 8 levels instead of 4: the waves win on a grid of a few rounds of the
// chip, the reads on a larger one.  Microseconds a step at 4 and 8 levels,
// FP64 and binary32 (blocks at 8 levels): O110 x 40 (1025) 75.6, 78.8 and
// 54.9, 56.0; O160 x 51 (2961) 169.3, 170.3 and 92.9, 94.8; O200 x 51 (4578)
// 271.9, 273.0 and 142.1, 138.1; O320 x 51 (11396) 693, 689 and 373, 359.
int auto_levels_per_block(int mesh, int tx, int ty, int nz)
{
    const long long cols = (long long)tx * ty;
    const int cand[] = {8, 4, 2};
    for (int kc : cand) {
        const long long blocks = cols * ((nz + kc - 1) / kc);
        if (blocks >= (mesh == FTGCR_MESH_OCTAHEDRAL && kc == 8 ? 4096 : 1024) && kc <= nz) return kc;
    }
    return 1;
}

// The direction pass takes at most 4 levels per block: at 8 its FP64 form needs
// 163 registers with the basis sums of a cycle's end and drops to three waves
// per SIMD (512x256x64: FP64 83.7 vs 82.0 us, binary32 50.6 vs 48.0; O160x51
// 58.2 vs 54.4), while the dots pass is fastest at 8 on the lat-lon mesh.
void dir_tiling(int kc, int nz, int tx, int ty, int& kc_dir, int& tz_dir, int& nblk_dir)
{
    kc_dir = kc < 4 ? kc : 4;
    tz_dir = (nz + kc_dir - 1) / kc_dir;
    nblk_dir = tx * ty * tz_dir;
}

void set_tiling(ftgcr_handle* h)
{
    const Geo& g = h->geo;
    const int cpb = col_block_cols(h->precision == FTGCR_MIXED ? 4 : 8, h->H);
    h->nblk_col = (g.ncols + cpb - 1) / cpb;
    if (g.mesh == FTGCR_MESH_OCTAHEDRAL) {   // ST_THREADS consecutive points per block
        h->tx = (g.nx + ST_THREADS - 1) / ST_THREADS;
        h->ty = 1;
    } else {
        h->tx = (g.nx + ST_TX - 1) / ST_TX;
        h->ty = (g.ny + ST_TY - 1) / ST_TY;
    }
    int kc = h->opt.levels_per_block;
    if (kc != 1 && kc != 2 && kc != 4 && kc != 8 && kc != 16) kc = h->tuned_kc ? h->tuned_kc : tuned_levels(h);
    if (kc != 1 && kc != 2 && kc != 4 && kc != 8 && kc != 16) kc = auto_levels_per_block(g.mesh, h->tx, h->ty, g.nz);
    h->kc = kc;
    h->tz = (g.nz + kc - 1) / kc;
    h->nblk_st = h->tx * h->ty * h->tz;
    dir_tiling(kc, g.nz, h->tx, h->ty, h->kc_dir, h->tz_dir, h->nblk_dir);
    auto fold = [&](int nblk) { return nblk > FOLD_BLOCKS && nblk + RED_FOLD <= part_stride(h) ? RED_FOLD : 0; };
    h->fold_st = fold(h->nblk_st);
    h->fold_dir = fold(h->nblk_dir);
    // block orders: the option, else the tuned choice, else the mesh's
    // default (octahedral: XCD-aware level chunks in a row, measured 18%
    // faster on O160 x 51 than tiles in a row, its slot tables and neighbour
    // gathers then being re-read from the die's L2; lat-lon: tiles in a row)
    const Tuned tu = tuned_for(h);
    const int def = g.mesh == FTGCR_MESH_OCTAHEDRAL ? ORD_XCD : ORD_X;
    auto pick = [&](int opt, int mine, int cached) {
        if (opt >= FTGCR_ORDER_X && opt <= FTGCR_ORDER_XCD) return opt - 1;
        if (mine >= 0) return mine;
        return cached >= 0 ? cached : def;
    };
    h->ord_st = pick(h->opt.order_stencil, h->tuned_ord_st, tu.ord_st);
    h->ord_dir = pick(h->opt.order_dir, h->tuned_ord_dir, tu.ord_dir);
}

size_t elem_bytes(const ftgcr_handle* h) { return h->precision == FTGCR_MIXED ? 4 : 8; }

// Room for block partials of either grid at any levels-per-block (1 level
// per block is the most blocks), so batched solves may pick their own tiling.
long long part_stride(const ftgcr_handle* h)
{
    return std::max<long long>(h->nblk_col, (long long)h->tx * h->ty * h->geo.nz);
}

struct Layout {
    size_t vec, xvec, part, hist, total;
};

Layout layout(const ftgcr_handle* h)
{
    Layout L;
    const size_t n = (size_t)h->geo.n;
    L.vec = align256(n * elem_bytes(h));
    L.xvec = align256(n * sizeof(double));
    L.part = align256((size_t)part_stride(h) * NV_MAX * sizeof(double));
    L.hist = align256((size_t)std::max<long long>(h->opt.hist_cap, 1) * sizeof(double));
    // U (kmax + 2), AP (kmax + 1), three r, and on the octahedral mesh L(e)
    const int nvec = 2 * (h->kmax + 1) + 4 + (h->geo.mesh == FTGCR_MESH_OCTAHEDRAL ? 1 : 0);
    L.total = (size_t)nvec * L.vec + L.xvec + L.part + L.hist;
    return L;
}

template <typename T>
Inst<T> make_inst(const ftgcr_handle* h, const double* rhs, double* x, void* ws)
{
    Inst<T> in;
    std::memset(&in, 0, sizeof in);
    in.g = h->geo;
    const Layout L = layout(h);
    char* p = (char*)ws;
    for (int l = 0; l <= h->kmax + 1; ++l) { in.U[l] = (T*)p; p += L.vec; }
    for (int l = 0; l <= h->kmax; ++l) { in.AP[l] = (T*)p; p += L.vec; }
    for (int q = 0; q < 3; ++q) { in.R[q] = (T*)p; p += L.vec; }
    if (h->geo.mesh == FTGCR_MESH_OCTAHEDRAL) {
        in.LE = (T*)p;
        p += L.vec;
    }
    in.X[0] = x;
    in.X[1] = (double*)p; p += L.xvec;
    in.part = (double*)p; p += L.part;
    in.pstride = part_stride(h);
    in.hist = (double*)p;
    in.hist_cap = h->opt.hist_cap;
    in.rhs = rhs;
    in.st = h->st;
    in.nblk_col = h->nblk_col;
    in.nblk_st = h->nblk_st;
    in.kc = h->kc;
    in.tx = h->tx;
    in.ty = h->ty;
    in.tz = h->tz;
    in.nblk_dir = h->nblk_dir;
    in.kc_dir = h->kc_dir;
    in.tz_dir = h->tz_dir;
    in.fold_st = h->fold_st;
    in.fold_dir = h->fold_dir;
    in.ord_st = h->ord_st;
    in.ord_dir = h->ord_dir;
    in.xw = h->xw;
    in.nblk_res = h->nblk_res;
    in.rtx = h->rtx;
    return in;
}

// About the microseconds a step of a single solve takes in the streaming
// kernels, measured at k = 3 as resident_step_us: launches, and passes over
// vectors that the cache holds (grids that the resident kernel takes).
double streaming_step_us(const ftgcr_handle* h)
{
    const double m = 1e-6 * (double)h->geo.n;
    if (h->precision == FTGCR_MIXED) return (h->H <= 32 ? 33.0 : 31.0) + 10.0 * m;
    return h->geo.mesh == FTGCR_MESH_OCTAHEDRAL ? 27.0 + 20.0 * m : 28.0 + 18.0 * m;
}

// Decide whether solves of this handle run in the resident kernel, and give
// it its exchange words.  A grid it does not take, a device without cooperative
// launches, or a form of the kernel that takes longer than the streaming
// kernels on this grid leaves the handle to those.  Such forms are the ones
// that spill: us a step, streaming and resident, binary32 O_87 x 33 44, 47 (but
// O_119 x 33 54, 52), O_12 x 96 31, 33; FP64 O_87 x 17 40, 47 (but O_119 x 32 67,
// 59).
ftgcr_status setup_resident(ftgcr_handle* h)
{
    if (h->precond != FTGCR_PRECOND_COLUMN) return FTGCR_OK;
    const bool mixed = h->precision == FTGCR_MIXED;
    const Geo& g = h->geo;
    HIP_TRY(h, hipDeviceGetAttribute(&h->cus, hipDeviceAttributeMultiprocessorCount, h->device));
    const int w = resident_waves(g.mesh, g.nx, g.ny, h->H, mixed ? 4 : 8, h->cus, &h->rtx, &h->nblk_res);
    if (w == 0 || !(mixed ? resident_fits<float>(g.mesh, h->H, w, h->nblk_res, h->kmax)
                          : resident_fits<double>(g.mesh, h->H, w, h->nblk_res, h->kmax)))
        return FTGCR_OK;
    h->res_gain = streaming_step_us(h) - resident_step_us(g.mesh, h->H, mixed ? 4 : 8, w);
    if (h->res_gain <= 0.0) return FTGCR_OK;
    HIP_TRY(h, hipMalloc(&h->xw, RES_WORDS * sizeof(unsigned long long)));
    HIP_TRY(h, hipMemset(h->xw, 0, RES_WORDS * sizeof(unsigned long long)));
    h->res_waves = w;
    return FTGCR_OK;
}

// A tiling asked for in the options means the streaming kernels.
bool use_resident(const ftgcr_handle* h)
{
    return h->res_waves > 0 && !h->no_resident && h->opt.levels_per_block == 0 && h->opt.order_stencil == FTGCR_ORDER_AUTO &&
           h->opt.order_dir == FTGCR_ORDER_AUTO;
}

// What this handle's next resident launch is made to end as (0: nothing).
int forced_outcome(ftgcr_handle* h)
{
    if (h->test_launch > 1) {
        h->test_launch -= 1;
        return 0;
    }
    return h->test_launch == 1 ? h->test_outcome : 0;
}

// options.profile_kernels, bits 0-7: 1 times all three step kernels, any
// other nonzero value is a mask (bit 1 update_thomas, bit 2 stencil_dots, bit 3
// dir_update); bits 8-15: a stride s > 1 times only the steps whose number is
// a multiple of s (for s coprime with k the sample covers every pass index
// alike).
int profile_mask(const ftgcr_handle* h)
{
    const int sel = h->opt.profile_kernels & 0xFF;
    return sel == 1 ? 0xE : sel;
}

int profile_stride(const ftgcr_handle* h) { return (h->opt.profile_kernels >> 8) & 0xFF; }

ftgcr_status upload_tables(ftgcr_handle* h)
{
    const int nx = h->grid.nlon, ny = h->grid.nlat, nz = h->grid.nz;
    const double dlon = 2.0 * kPi / nx, dlat = kPi / ny, dz = h->grid.shell_depth / nz;
    const ftgcr_coeffs& c = h->co;
    const size_t nhx = (size_t)nx * ny, nhy = (size_t)nx * (ny + 1), nhc = (size_t)nx * ny;
    const size_t total = nhx + nhy + nhc + nz + (nz + 1) + ny + (ny + 1) + ny;
    std::vector<double> t(total, 0.0);
    double* hx = t.data();
    double* hy = hx + nhx;
    double* hc = hy + nhy;
    double* gc = hc + nhc;
    double* gf = gc + nz;
    double* Gx = gf + (nz + 1);
    double* Gy = Gx + ny;
    double* Gz = Gy + (ny + 1);
    auto lon_c = [&](int i) { return (i + 0.5) * dlon; };
    auto lon_e = [&](int i) { return (i + 1.0) * dlon; };
    auto lat_c = [&](int j) { return -0.5 * kPi + (j + 0.5) * dlat; };
    auto lat_s = [&](int j) { return -0.5 * kPi + j * dlat; };
    for (int j = 0; j < ny; ++j)
        for (int i = 0; i < nx; ++i) {
            hx[(size_t)j * nx + i] = c.hill_amp * hill_height(c, lon_e(i), lat_c(j));
            hc[(size_t)j * nx + i] = c.hill_amp * hill_height(c, lon_c(i), lat_c(j));
        }
    for (int j = 1; j < ny; ++j)
        for (int i = 0; i < nx; ++i) hy[(size_t)j * nx + i] = c.hill_amp * hill_height(c, lon_c(i), lat_s(j));
    for (int k = 0; k < nz; ++k) gc[k] = std::exp(-((k + 0.5) / nz) / c.decay_z);
    for (int k = 0; k <= nz; ++k) gf[k] = std::exp(-((double)k / nz) / c.decay_z);
    for (int j = 0; j < ny; ++j) {
        Gx[j] = dlat * dz / (std::cos(lat_c(j)) * dlon);
        Gz[j] = std::cos(lat_c(j)) * dlon * dlat / dz;
    }
    for (int j = 1; j < ny; ++j) Gy[j] = std::cos(lat_s(j)) * dlon * dz / dlat;   // poles stay exactly 0
    // binary32 copies of hx, hy, hc (rounded to nearest) after the FP64 tables
    const size_t n32 = nhx + nhy + nhc;
    std::vector<float> t32(n32);
    for (size_t q = 0; q < n32; ++q) t32[q] = (float)t[q];
    HIP_TRY(h, hipMalloc(&h->tables, total * sizeof(double) + n32 * sizeof(float)));
    HIP_TRY(h, hipMemcpy(h->tables, t.data(), total * sizeof(double), hipMemcpyHostToDevice));
    float* tab32 = reinterpret_cast<float*>(h->tables + total);
    HIP_TRY(h, hipMemcpy(tab32, t32.data(), n32 * sizeof(float), hipMemcpyHostToDevice));
    Geo& g = h->geo;
    g.mesh = FTGCR_MESH_LATLON;
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.ncols = nx * ny;
    g.n = (long long)nx * ny * nz;
    g.opsig = 1.0 + c.helmholtz;
    g.hx = h->tables;
    g.hy = g.hx + nhx;
    g.hc = g.hy + nhy;
    g.gc = g.hc + nhc;
    g.gf = g.gc + nz;
    g.Gx = g.gf + (nz + 1);
    g.Gy = g.Gx + ny;
    g.Gz = g.Gy + (ny + 1);
    g.hx32 = tab32;
    g.hy32 = g.hx32 + nhx;
    g.hc32 = g.hy32 + nhy;
    return FTGCR_OK;
}

// ---------------------------------------------------------------------------
// octahedral reduced Gaussian grid O_N: host tables
// ---------------------------------------------------------------------------

// Points per level of O_N and of its ring j (0 = southernmost).
long long oct_points(int N) { return 4LL * N * (N + 9); }
int oct_ring(int N, int j) { return 4 * (j < N ? j + 1 : 2 * N - j) + 16; }

// Gauss-Legendre nodes of order n (ascending) by Newton's method on the
// Legendre recurrence, started from Tricomi's asymptotic estimate.
std::vector<double> gauss_nodes(int n)
{
    std::vector<double> mu(n);
    for (int l = 1; l <= n; ++l) {
        const double th = kPi * (4.0 * l - 1.0) / (4.0 * n + 2.0);
        double x = (1.0 - (n - 1.0) / (8.0 * n * n * n)) * std::cos(th);
        for (int it = 0; it < 50; ++it) {
            double pm = 1.0, p = x;   // P_0, P_1
            for (int m = 2; m <= n; ++m) {
                const double pn = ((2 * m - 1) * x * p - (m - 1) * pm) / m;
                pm = p;
                p = pn;
            }
            const double dpdx = n * (pm - x * p) / (1.0 - x * x);
            const double step = p / dpdx;
            x -= step;
            if (std::fabs(step) <= 1e-16 * std::fabs(x) + 1e-300) break;
        }
        mu[n - l] = x;   // the l-th largest root
    }
    return mu;
}

ftgcr_status upload_tables_oct(ftgcr_handle* h)
{
    const int N = h->grid.nlat, nz = h->grid.nz, nr = 2 * N;
    const long long np = oct_points(N);
    const double dz = h->grid.shell_depth / nz;
    const ftgcr_coeffs& co = h->co;
    const std::vector<double> mu = gauss_nodes(nr);
    std::vector<long long> first(nr + 1, 0);
    for (int j = 0; j < nr; ++j) first[j + 1] = first[j] + oct_ring(N, j);
    if (first[nr] != np) return fail(h, FTGCR_E_HIP, "octahedral point count");
    std::vector<double> px(np), py(np), pz(np), plon(np), plat(np);
    for (int j = 0; j < nr; ++j) {
        const int n = oct_ring(N, j);
        const double lat = std::asin(mu[j]);
        for (int q = 0; q < n; ++q) {
            const long long a = first[j] + q;
            const double lon = (2.0 * kPi / n) * q;
            plon[a] = lon;
            plat[a] = lat;
            px[a] = std::cos(lat) * std::cos(lon);
            py[a] = std::cos(lat) * std::sin(lon);
            pz[a] = std::sin(lat);
        }
    }
    // neighbour slots: ids (-1 empty) and accumulated cotangent weights
    std::vector<int> nb((size_t)np * NB_OCT, -1);
    std::vector<double> cw((size_t)np * NB_OCT, 0.0);
    auto slot = [&](long long a, long long b) -> long long {
        for (int q = 0; q < NB_OCT; ++q) {
            const size_t at = (size_t)a * NB_OCT + q;
            if (nb[at] == (int)b) return (long long)at;
            if (nb[at] < 0) {
                nb[at] = (int)b;
                return (long long)at;
            }
        }
        return -1;
    };
    bool overflow = false;
    // a triangle adds half the cotangent of each corner to the opposite edge
    auto triangle = [&](long long a, long long b, long long c) {
        const long long v[3] = {a, b, c};
        for (int r = 0; r < 3; ++r) {
            const long long o = v[r], e1 = v[(r + 1) % 3], e2 = v[(r + 2) % 3];
            const double ux = px[e1] - px[o], uy = py[e1] - py[o], uz = pz[e1] - pz[o];
            const double vx = px[e2] - px[o], vy = py[e2] - py[o], vz = pz[e2] - pz[o];
            const double dot = ux * vx + uy * vy + uz * vz;
            const double crx = uy * vz - uz * vy, cry = uz * vx - ux * vz, crz = ux * vy - uy * vx;
            const double half_cot = 0.5 * dot / std::sqrt(crx * crx + cry * cry + crz * crz);
            const long long s1 = slot(e1, e2), s2 = slot(e2, e1);
            if (s1 < 0 || s2 < 0) {
                overflow = true;
                return;
            }
            cw[s1] += half_cot;
            cw[s2] += half_cot;
        }
    };
    for (int j = 0; j + 1 < nr; ++j) {
        const long long n = oct_ring(N, j), n2 = oct_ring(N, j + 1);
        long long a = 0, b = 0;
        // eastward: the ring whose next point comes first adds a triangle
        // ((a+1)/n <= (b+1)/n2 in exact integer form; the southern ring on a tie)
        while (a < n || b < n2) {
            if (a < n && (b >= n2 || (a + 1) * n2 <= (b + 1) * n)) {
                triangle(first[j] + a % n, first[j] + (a + 1) % n, first[j + 1] + b % n2);
                ++a;
            } else {
                triangle(first[j] + a % n, first[j + 1] + b % n2, first[j + 1] + (b + 1) % n2);
                ++b;
            }
        }
    }
    if (overflow) return fail(h, FTGCR_E_HIP, "octahedral mesh: a point has more than NB_OCT neighbours");
    // per point: slot tables (slot-major), sums, circumcentric area, hills
    const size_t nq = (size_t)NB_OCT * np;
    std::vector<int> onb(nq);
    std::vector<double> ogw(nq), ohw(nq), oh0(np), oh1(np), ogz(np), ohc(np);
    for (long long a = 0; a < np; ++a) {
        double area = 0.0, s0 = 0.0, s1 = 0.0;
        for (int q = 0; q < NB_OCT; ++q) {
            const size_t at = (size_t)a * NB_OCT + q;
            const size_t to = (size_t)q * np + a;
            const int b = nb[at];
            onb[to] = b;
            ogw[to] = 0.0;
            ohw[to] = 0.0;
            if (b < 0) continue;
            const double dx = px[a] - px[b], dy = py[a] - py[b], dzz = pz[a] - pz[b];
            area += 0.25 * cw[at] * (dx * dx + dy * dy + dzz * dzz);
            // hill at the edge's centre: the chord's midpoint, back on the sphere
            const double mx = px[a] + px[b], my = py[a] + py[b], mz = pz[a] + pz[b];
            const double mr = std::sqrt(mx * mx + my * my + mz * mz);
            const double he = co.hill_amp * hill_height(co, std::atan2(my, mx), std::asin(mz / mr));
            ogw[to] = dz * cw[at];
            ohw[to] = ogw[to] * he;
            s0 += ogw[to];
            s1 += ohw[to];
        }
        oh0[a] = s0;
        oh1[a] = s1;
        ogz[a] = area / dz;
        ohc[a] = co.hill_amp * hill_height(co, plon[a], plat[a]);
    }
    std::vector<double> gc(nz), gf(nz + 1);
    for (int k = 0; k < nz; ++k) gc[k] = std::exp(-((k + 0.5) / nz) / co.decay_z);
    for (int k = 0; k <= nz; ++k) gf[k] = std::exp(-((double)k / nz) / co.decay_z);
    // one device allocation: doubles first, then the slot ids, then binary32
    // copies of the weight and per-point tables (the mixed form's)
    const size_t nd = 2 * nq + 4 * (size_t)np + nz + (nz + 1);
    const size_t n32 = 2 * nq + 4 * (size_t)np;
    HIP_TRY(h, hipMalloc(&h->tables, nd * sizeof(double) + nq * sizeof(int) + n32 * sizeof(float)));
    double* t = h->tables;
    auto put = [&](const double* src, size_t cnt) -> double* {
        double* at = t;
        t += cnt;
        return hipMemcpy(at, src, cnt * sizeof(double), hipMemcpyHostToDevice) == hipSuccess ? at : nullptr;
    };
    Geo& g = h->geo;
    g.mesh = FTGCR_MESH_OCTAHEDRAL;
    g.nx = (int)np;
    g.ny = 1;
    g.nz = nz;
    g.ncols = (int)np;
    g.n = np * nz;
    g.opsig = 1.0 + co.helmholtz;
    g.ogw = put(ogw.data(), nq);
    g.ohw = put(ohw.data(), nq);
    g.oh0 = put(oh0.data(), np);
    g.oh1 = put(oh1.data(), np);
    g.ogz = put(ogz.data(), np);
    g.ohc = put(ohc.data(), np);
    g.gc = put(gc.data(), nz);
    g.gf = put(gf.data(), nz + 1);
    int* ids = reinterpret_cast<int*>(t);
    HIP_TRY(h, hipMemcpy(ids, onb.data(), nq * sizeof(int), hipMemcpyHostToDevice));
    g.onb = ids;
    std::vector<float> t32;
    t32.reserve(n32);
    for (const std::vector<double>* v : {&ogw, &ohw, &oh0, &oh1, &ogz, &ohc})
        for (double d : *v) t32.push_back((float)d);
    float* f32 = reinterpret_cast<float*>(ids + nq);
    HIP_TRY(h, hipMemcpy(f32, t32.data(), n32 * sizeof(float), hipMemcpyHostToDevice));
    g.ogw32 = f32;
    g.ohw32 = g.ogw32 + nq;
    g.oh0_32 = g.ohw32 + nq;
    g.oh1_32 = g.oh0_32 + np;
    g.ogz32 = g.oh1_32 + np;
    g.ohc32 = g.ogz32 + np;
    if (!g.ogw || !g.ohw || !g.oh0 || !g.oh1 || !g.ogz || !g.ohc || !g.gc || !g.gf)
        return fail(h, FTGCR_E_HIP, "octahedral table upload failed");
    return FTGCR_OK;
}

ftgcr_status upload_debug_inst(ftgcr_handle* h)
{
    Inst<double> in;
    std::memset(&in, 0, sizeof in);
    in.g = h->geo;
    in.st = h->st;
    in.nblk_col = h->nblk_col;
    in.nblk_st = h->nblk_st;
    in.kc = h->kc;
    in.tx = h->tx;
    in.ty = h->ty;
    in.tz = h->tz;
    in.nblk_dir = h->nblk_dir;
    in.kc_dir = h->kc_dir;
    in.tz_dir = h->tz_dir;
    in.ord_st = h->ord_st;
    in.ord_dir = h->ord_dir;
    HIP_TRY(h, hipMemcpy(h->inst_dbg, &in, sizeof in, hipMemcpyHostToDevice));
    const int blk0[8] = {0, h->nblk_col, 0, h->nblk_st, 0, h->nblk_dir, 0, h->nblk_res};
    HIP_TRY(h, hipMemcpy(h->blk0, blk0, sizeof blk0, hipMemcpyHostToDevice));
    return FTGCR_OK;
}

// ---------------------------------------------------------------------------
// one solve
// ---------------------------------------------------------------------------

struct DevEvent {
    long long step;
    int vec, bit;
    long long count, start;
    const long long* idx;        // device or null
    const unsigned char* bits;   // device or null
};


const char* const kKernelNames[3] = {"update_thomas", "stencil_dots", "dir_update"};

hipEvent_t take_event(ftgcr_handle* h)
{
    if (h->ev_next == h->ev_pool.size()) {
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        h->ev_pool.push_back(e);
    }
    return h->ev_pool[h->ev_next++];
}

// Resolve the event pairs recorded since the last synchronisation.  Steps
// numbered above `last_step` were enqueued after the solve had ended (they
// returned at once) and are not counted.
void collect_times(ftgcr_handle* h, long long last_step)
{
    for (const auto& p : h->pending) {
        if (p.step > last_step) continue;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
            h->kt_ms[p.cls] += ms;
            h->kt_n[p.cls] += 1;
        }
    }
    h->pending.clear();
    h->ev_next = 0;
}

template <typename T>
void inject_event(const Table<T>& tb, const DevEvent& ev, long long n, hipStream_t s)
{
    using L = Launch<T>;
    L::event_prep(tb, ev.vec, s);
    if (ev.vec != FTGCR_V_E) L::event_copy(tb, (int)std::min<long long>((n + 255) / 256, 8192), s);
    L::event_inject(tb, (int)std::max<long long>(1, std::min<long long>((ev.count + 255) / 256, 8192)), ev.idx, ev.bits,
                    ev.count, ev.start, ev.bit, false, s);
}

// The state's norms in the streaming kernels' order, after a resident launch
// that did not run.  on_r: this step's events on r, already injected: they are
// taken out meanwhile (a flip is its own inverse), since the detector compares
// with the norm of r before them.
template <typename T>
void streaming_norms(const Table<T>& tb, const std::vector<const DevEvent*>& on_r, int nblk_col, int H, hipStream_t s)
{
    using L = Launch<T>;
    auto flip = [&]() {
        for (const DevEvent* ev : on_r) {
            L::event_prep(tb, FTGCR_V_R, s);   // (r is no longer in the backup's buffer: no copy)
            L::event_inject(tb, (int)std::max<long long>(1, std::min<long long>((ev->count + 255) / 256, 8192)), ev->idx,
                            ev->bits, ev->count, ev->start, ev->bit, true, s);
        }
    };
    flip();
    L::norms(tb, nblk_col, H, s);
    flip();
}

template <typename T>
struct Runner {
    using L = Launch<T>;
    ftgcr_handle* h;
    Table<T> tb;
    hipStream_t s;
    // no allocation of any kind: no graph capture or instantiation, no
    // timing events (kernel timing and graph replay are skipped)
    bool noalloc = false;
    // a resident launch's blocks did not start together: this solve streams
    // (in all its refinement rounds, so that it waits for them once)
    bool late = false;

    long long cur_step = 0;

    template <class F>
    void timed(int cls, F&& launch)
    {
        const int mask = noalloc ? 0 : profile_mask(h);
        const int stride = profile_stride(h);
        if (!(mask & (2 << cls)) || (stride > 1 && cur_step % stride != 0)) {
            launch(nullptr, nullptr);
            return;
        }
        hipEvent_t a = take_event(h), b = take_event(h);
        if (!a || !b) {
            launch(nullptr, nullptr);
            return;
        }
        // the dispatch stamps a and b itself: the kernel's own execution
        // time, with no event packets between it and its neighbours
        launch(a, b);
        h->pending.push_back({cls, cur_step, a, b});
    }

    // Replay `n` steps as one captured graph (captured on first use; the
    // graph holds kernel launches only and every argument is fixed for the
    // handle: the per-solve data live in the device-side instance record).
    ftgcr_status replay(int n)
    {
        if (!h->graph || h->graph_steps != n || h->graph_nt_ap != h->nt_ap) {
            if (h->graph) {
                (void)hipGraphExecDestroy(h->graph);
                h->graph = nullptr;
            }
            Runner cap{h, tb, h->cap_stream};
            HIP_TRY(h, hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeRelaxed));
            for (int q = 0; q < n; ++q) cap.step(0);
            hipGraph_t g = nullptr;
            HIP_TRY(h, hipStreamEndCapture(h->cap_stream, &g));
            hipError_t e = hipGraphInstantiate(&h->graph, g, nullptr, nullptr, 0);
            (void)hipGraphDestroy(g);
            if (e != hipSuccess) {
                h->graph = nullptr;
                return fail(h, FTGCR_E_HIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
            }
            h->graph_steps = n;
            h->graph_nt_ap = h->nt_ap;
        }
        HIP_TRY(h, hipGraphLaunch(h->graph, s));
        return FTGCR_OK;
    }

    // One inner step; `mid` are the step's e events (injected after the
    // column solve's decision, before the stencil pass reads e).
    void step(long long number, const std::vector<const DevEvent*>* mid = nullptr)
    {
        cur_step = number;
        timed(0, [&](hipEvent_t a, hipEvent_t b) { L::update_thomas(tb, h->nblk_col, h->H, 0, s, a, b); });
        if (mid && !mid->empty()) {
            // e events go between the decision and the dots pass
            L::finish_col(tb, 0, s);
            for (const DevEvent* ev : *mid) event(*ev);
            timed(1, [&](hipEvent_t a, hipEvent_t b) { L::stencil_dots(tb, h->nblk_st, h->kc, 0, s, a, b); });
            if (h->fold_st) L::fold(tb, 0, h->fold_st, h->kmax, s);
            L::finish_alpha(tb, s);
        } else {
            // dots pass first, then decision and alpha in one launch
            timed(1, [&](hipEvent_t a, hipEvent_t b) { L::stencil_dots(tb, h->nblk_st, h->kc, 1, s, a, b); });
            if (h->fold_st) L::fold(tb, 0, h->fold_st, h->kmax, s);
            L::finish_step(tb, s);
        }
        timed(2, [&](hipEvent_t a, hipEvent_t b) { L::dir_update(tb, h->nblk_dir, h->kc_dir, 0, h->nt_ap, s, a, b); });
        if (h->fold_dir) L::fold(tb, 1, h->fold_dir, 2, s);
        L::finish_beta(tb, 0, s);
    }

    void start_round()
    {
        L::update_thomas(tb, h->nblk_col, h->H, 1, s);
        L::finish_col(tb, 1, s);
        L::dir_update(tb, h->nblk_dir, h->kc_dir, 1, h->nt_ap, s);
        if (h->fold_dir) L::fold(tb, 1, h->fold_dir, 2, s);
        L::finish_beta(tb, 1, s);
    }

    void event(const DevEvent& ev)
    {
        inject_event<T>(tb, ev, h->geo.n, s);
        if (ev.vec == FTGCR_V_R || ev.vec == FTGCR_V_AP) {
            L::beta_dots(tb, h->nblk_st, s);
        }
    }

    ftgcr_status read_state()
    {
        HIP_TRY(h, hipGetLastError());
        HIP_TRY(h, hipMemcpyAsync(h->st_host, h->st, sizeof(SolveState), hipMemcpyDeviceToHost, s));
        HIP_TRY(h, hipStreamSynchronize(s));
        collect_times(h, h->st_host->s);
        return FTGCR_OK;
    }

    ftgcr_status read_status(int* status)
    {
        HIP_TRY(h, hipGetLastError());
        // the status, the counters and the norms the next chunk is sized from
        HIP_TRY(h, hipMemcpyAsync(h->st_host, h->st, offsetof(SolveState, rr_new) + sizeof(double),
                                  hipMemcpyDeviceToHost, s));
        HIP_TRY(h, hipStreamSynchronize(s));
        collect_times(h, h->st_host->s);
        *status = h->st_host->status;
        return FTGCR_OK;
    }

    // Whether a resident launch of the steps before event `next` pays: it loads
    // the state and forms the columns' pivots, and where the event's step is not
    // resident (e) the norms have to be formed anew on both sides.  (Before an
    // event of another kind the next launch gains that step too.)
    // Microseconds a step, streaming and resident, 64 x 32 x 8, 256 x 128 x 32
    // and O_40 x 51, k = 3: flips in x every step 58, 58; 72, 80; 64, 84; every
    // second 44, 34; 62, 52; 55, 56; every fourth 36, 22; 55, 38; 50, 42; flips
    // in e every second 43, 50; 60, 70; 54, 73; every fourth 35, 31; 54, 47; 48,
    // 51; every eighth 30, 21; 50, 36; 45, 39.
    bool pays_until(const std::vector<DevEvent>& evs, size_t next, long long launched, bool event_now) const
    {
        const double entry = 12.0 + 1.2 * h->H;
        bool leaves = false;
        size_t after = next;   // the event after it
        for (; after < evs.size() && evs[after].step == evs[next].step; ++after)
            leaves = leaves || evs[after].vec == FTGCR_V_E;
        const long long gap = evs[next].step - 1 - launched;
        if (leaves) return (double)gap * h->res_gain > entry + 0.8 * h->H;
        const bool stays = after == evs.size() || (double)(evs[after].step - evs[next].step) * h->res_gain > entry;
        return (double)(gap + (stays && !event_now ? 1 : 0)) * h->res_gain > entry;
    }

    // Enqueue steps until the device reports an outcome.  `launched` is the
    // number of steps executed so far (the device's s).
    ftgcr_status run_steps(int k, long long launched, long long cap, const std::vector<DevEvent>& evs)
    {
        size_t evp = 0;
        const int chunk = std::max(1, h->opt.poll_steps);
        const long long guard = cap + std::max<long long>(chunk, RES_STEPS) + 16;
        long long issued = 0;
        // Chunks after the first are sized from the observed convergence
        // rate: steps past the exit are launched and return at once, so the
        // last chunk should end near it.  A rate estimate that is too short
        // only costs one more status read.
        long long want = chunk;
        double rr_prev = -1.0;
        long long s_prev = 0;
        bool resident_norms = false;   // the state's norms are the resident kernel's
        std::vector<const DevEvent*> on_r;   // events on r before the launch
        auto back_to_streaming = [&]() {     // the launch did not run
            if (resident_norms) streaming_norms<T>(tb, on_r, h->nblk_col, h->H, s);
            resident_norms = false;
        };
        while (true) {
            while (evp < evs.size() && evs[evp].step <= launched) ++evp;
            const bool event_now = evp < evs.size() && evs[evp].step == launched + 1;
            bool resident = use_resident(h) && !late;
            size_t next = evp;   // the first event of a later step
            while (next < evs.size() && evs[next].step <= launched + 1) ++next;
            if (resident && next < evs.size()) resident = pays_until(evs, next, launched, event_now);
            if (event_now && resident) {
                // events at the start of a step come between two launches of
                // the resident kernel; one inside a step (e), or one on r
                // while the state's norms are the streaming kernels', leaves
                // that step to the streaming kernels
                for (size_t q = evp; q < evs.size() && evs[q].step == launched + 1; ++q)
                    if (evs[q].vec == FTGCR_V_E || (evs[q].vec == FTGCR_V_R && !resident_norms)) resident = false;
            }
            if (resident_norms && !resident) {
                L::norms(tb, h->nblk_col, h->H, s);
                resident_norms = false;
            }
            if (event_now && !resident) {
                std::vector<const DevEvent*> mid;
                for (; evp < evs.size() && evs[evp].step == launched + 1; ++evp) {
                    if (evs[evp].vec == FTGCR_V_E) mid.push_back(&evs[evp]);
                    else event(evs[evp]);
                }
                step(launched + 1, &mid);
                launched += 1;
                issued += 1;
            } else if (resident) {
                on_r.clear();
                for (; evp < evs.size() && evs[evp].step == launched + 1; ++evp) {
                    if (evs[evp].vec == FTGCR_V_R) on_r.push_back(&evs[evp]);
                    event(evs[evp]);
                }
                // to the next event or the outcome, in one launch
                long long cnt = RES_STEPS;
                if (evp < evs.size()) cnt = std::min<long long>(cnt, evs[evp].step - 1 - launched);
                const int forced = forced_outcome(h);
                const ResidentArgs arg{launched + cnt, k + 1, resident_norms ? 0 : 1, noalloc ? 0 : profile_mask(h),
                                       profile_stride(h), forced};
                const hipError_t e =
                    forced == FTGCR_RESIDENT_REFUSED
                        ? hipErrorCooperativeLaunchTooLarge
                        : resident_run<T>(tb, h->blk0 + 6, h->nblk_res, h->geo.mesh, h->H, h->res_waves, arg, s);
                if (e != hipSuccess) {   // the device does not take the launch: the streaming kernels from here
                    (void)hipGetLastError();
                    h->res_waves = 0;
                    back_to_streaming();
                    continue;
                }
                launched += cnt;
                issued += cnt;
            } else {
                long long cnt = want;
                if (evp < evs.size()) cnt = std::min<long long>(cnt, evs[evp].step - 1 - launched);
                cnt = std::max<long long>(cnt, 1);
                if (cnt == chunk && h->opt.use_graphs && !h->opt.profile_kernels && !noalloc) {
                    ftgcr_status rc = replay(chunk);
                    if (rc != FTGCR_OK) return rc;
                } else {
                    for (long long q = 0; q < cnt; ++q) step(launched + 1 + q);
                }
                launched += cnt;
                issued += cnt;
            }
            int status = RUNNING;
            ftgcr_status rc = read_status(&status);
            if (rc != FTGCR_OK) return rc;
            if (h->st_host->res_fail == RES_BROKEN)
                return fail(h, FTGCR_E_HIP, "the resident kernel's blocks did not run together");
            if (h->st_host->res_fail == RES_LATE) {   // nothing has changed since the last read
                L::resident_late(tb, s);
                late = true;
                back_to_streaming();
                launched = h->st_host->s;
                continue;
            }
            resident_norms = resident_norms || resident;
            if (resident) {
                for (int q = 0; q < 3; ++q) {
                    h->kt_ms[q] += 1e-5 * (double)h->st_host->res_ticks[q];
                    h->kt_n[q] += h->st_host->res_counts[q];
                }
            }
            if (status != RUNNING) return FTGCR_OK;
            if (issued > guard) return fail(h, FTGCR_E_HIP, "step loop did not terminate");
            const SolveState& hs = *h->st_host;
            want = chunk;
            if (rr_prev > 0.0 && hs.s > s_prev && hs.rr_old > hs.T && hs.rr_old < rr_prev) {
                // per-step factor of <r, r> since the last read
                const double rate = std::pow(hs.rr_old / rr_prev, 1.0 / (double)(hs.s - s_prev));
                if (rate < 1.0 && rate > 0.0) {
                    const double left = std::log(hs.T / hs.rr_old) / std::log(rate);
                    if (left >= 0.0 && left < (double)chunk) want = std::max<long long>(1, (long long)std::ceil(left) + 1);
                }
            }
            rr_prev = hs.rr_old;
            s_prev = hs.s;
        }
    }
};

// Copy a fault plan's entry lists to the device.  staging == nullptr: into
// the handle's staging buffers (grown with hipMalloc when too small); else
// into `staging` (staging_bytes of device memory), with no allocation.
ftgcr_status stage_events(ftgcr_handle* h, const ftgcr_fault_plan* plan, std::vector<DevEvent>& out,
                          void* staging = nullptr, size_t staging_bytes = 0)
{
    out.clear();
    if (!plan || plan->n_events <= 0) return FTGCR_OK;
    if (!plan->events) return fail(h, FTGCR_E_INVALID, "plan has events == NULL");
    const long long n = h->geo.n;
    const int maxbit = (h->precision == FTGCR_MIXED) ? 31 : 63;
    size_t need = 0;
    for (int q = 0; q < plan->n_events; ++q) {
        const ftgcr_fault_event& e = plan->events[q];
        if (e.vec < FTGCR_V_X || e.vec > FTGCR_V_E) return fail(h, FTGCR_E_INVALID, "event vec out of range");
        if (e.count < 0) return fail(h, FTGCR_E_INVALID, "event count < 0");
        const int bmax = (e.vec == FTGCR_V_X) ? 63 : maxbit;
        if (!e.bits && (e.bit < 0 || e.bit > bmax)) return fail(h, FTGCR_E_INVALID, "event bit out of range");
        if (!e.idx && (e.start < 0 || e.start + e.count > n)) return fail(h, FTGCR_E_INVALID, "event range out of bounds");
        for (long long t = 0; t < e.count; ++t) {
            if (e.idx && (e.idx[t] < 0 || e.idx[t] >= n)) return fail(h, FTGCR_E_INVALID, "event index out of bounds");
            if (e.bits && e.bits[t] > bmax) return fail(h, FTGCR_E_INVALID, "event bit out of range");
        }
        if (e.idx || e.bits) need += (size_t)e.count;
    }
    long long* ev_idx = h->ev_idx;
    unsigned char* ev_bits = h->ev_bits;
    if (staging) {
        if (need * (sizeof(long long) + 1) > staging_bytes)
            return fail(h, FTGCR_E_WORKSPACE, "fault plan entries exceed the scratch memory left by the workspace");
        ev_idx = (long long*)staging;
        ev_bits = (unsigned char*)(ev_idx + need);
    } else if (need > h->ev_cap) {
        if (h->ev_idx) (void)hipFree(h->ev_idx);
        if (h->ev_bits) (void)hipFree(h->ev_bits);
        h->ev_idx = nullptr;
        h->ev_bits = nullptr;
        h->ev_cap = 0;
        HIP_TRY(h, hipMalloc(&h->ev_idx, need * sizeof(long long)));
        HIP_TRY(h, hipMalloc(&h->ev_bits, need));
        h->ev_cap = need;
        ev_idx = h->ev_idx;
        ev_bits = h->ev_bits;
    }
    size_t off = 0;
    for (int q = 0; q < plan->n_events; ++q) {
        const ftgcr_fault_event& e = plan->events[q];
        DevEvent d;
        d.step = e.step;
        d.vec = e.vec;
        d.bit = e.bit;
        d.count = e.count;
        d.start = e.start;
        d.idx = nullptr;
        d.bits = nullptr;
        if (e.idx && e.count > 0) {
            HIP_TRY(h, hipMemcpy(ev_idx + off, e.idx, (size_t)e.count * sizeof(long long), hipMemcpyHostToDevice));
            d.idx = ev_idx + off;
        }
        if (e.bits && e.count > 0) {
            HIP_TRY(h, hipMemcpy(ev_bits + off, e.bits, (size_t)e.count, hipMemcpyHostToDevice));
            d.bits = ev_bits + off;
        }
        if (e.idx || e.bits) off += (size_t)e.count;
        if (e.count > 0 && e.step >= 1) out.push_back(d);
    }
    std::stable_sort(out.begin(), out.end(), [](const DevEvent& a, const DevEvent& b) { return a.step < b.step; });
    return FTGCR_OK;
}

void fill_stats(ftgcr_handle* h, const SolveState& st, int refinements, float ms, ftgcr_stats* stats)
{
    if (!stats) return;
    stats->status = st.status;
    stats->detections = st.detections;
    stats->stagnation_accepts = st.stagnation_accepts;
    stats->events_applied = st.events_applied;
    stats->steps_executed = st.s;
    stats->steps_accepted = st.accepted;
    stats->steps_wasted = st.s - st.accepted;
    stats->cycles = st.cycles;
    stats->refinements = refinements;
    stats->rhs_norm2 = st.RR;
    stats->rr_final = st.rr_old;
    stats->rel_res_recursive = st.RR > 0 ? std::sqrt(st.rr_old / st.RR) : 0.0;
    stats->rel_res_true = st.RR > 0 ? std::sqrt(st.rt2 / st.RR) : 0.0;
    stats->time_ms = ms;
    stats->log_len = 0;
    if (stats->log && stats->log_cap > 0) {
        const int nlog = std::min(std::min(st.log_len, LOG_CAP), stats->log_cap);
        for (int q = 0; q < nlog; ++q) {
            stats->log[q].step = st.log[q].step;
            stats->log[q].nu = st.log[q].nu;
            stats->log[q].action = st.log[q].action;
            stats->log[q].rr_old = st.log[q].rr_old;
            stats->log[q].rr_new = st.log[q].rr_new;
        }
        stats->log_len = nlog;
    }
    stats->hist_len = 0;
    (void)h;
}

// One solve with the working vectors in `ws` (layout(h).total bytes).
// staging != nullptr: the fault plan's entry lists go there and nothing is
// allocated (no graphs, no timing events): the allocation-free entry point.
template <typename T>
ftgcr_status solve_impl(ftgcr_handle* h, const double* rhs, double* x, double tol, int k,
                        const ftgcr_fault_plan* plan, ftgcr_stats* stats, void* ws,
                        void* staging = nullptr, size_t staging_bytes = 0)
{
    using L = Launch<T>;
    hipStream_t s = h->stream;
    std::vector<DevEvent> evs;
    ftgcr_status rc = stage_events(h, plan, evs, staging, staging_bytes);
    if (rc != FTGCR_OK) return rc;

    Inst<T> in = make_inst<T>(h, rhs, x, ws);
    h->nt_ap = nt_ap_hint(k, h->geo.n, (int)sizeof(T));
    HIP_TRY(h, hipMemcpyAsync(h->inst, &in, sizeof in, hipMemcpyHostToDevice, s));
    HIP_TRY(h, hipStreamSynchronize(s));
    Runner<T> run{h,
                  Table<T>{(const Inst<T>*)h->inst, h->blk0, h->blk0 + 2, h->blk0 + 4, 1, h->geo.mesh, h->precond},
                  s};
    run.noalloc = staging != nullptr;
    const Table<T>& tb = run.tb;
    const bool mixed = h->precision == FTGCR_MIXED;
    const long long max_steps = h->opt.max_steps;
    int refinements = 0;
    int inner_outcome_final = FTGCR_CONVERGED;

    HIP_TRY(h, hipEventRecord(h->ev_start, s));
    if (!mixed) {
        L::init_state(tb, k, h->opt.ft, 0, max_steps, tol * tol, 1, 1, s);
        L::residual(tb, h->nblk_st, h->kc, 1, 1, s);
        run.start_round();
        rc = run.run_steps(k, 0, max_steps, evs);
        if (rc != FTGCR_OK) return rc;
        L::finalize_x(tb, h->nblk_st, h->kc, s);
    } else {
        // iterative refinement: FP64 true residual outside, FT-GCR with
        // binary32 vectors inside, the correction accumulated into FP64 x
        bool first = true;
        int inner_outcome = FTGCR_CONVERGED;
        while (true) {
            // a fresh round state first (it names the buffer the true
            // residual is written to), then r_t = A x - R in FP64
            L::init_state(tb, k, h->opt.ft, 1, max_steps, 0.0, first ? 1 : 0, 1, s);
            first = false;
            L::residual(tb, h->nblk_st, h->kc, 1, 0, s);
            rc = run.read_state();
            if (rc != FTGCR_OK) return rc;
            const SolveState& hs = *h->st_host;
            if (hs.rt2 <= tol * tol * hs.RR) break;                 // converged (true residual)
            if (hs.s >= max_steps || refinements >= h->opt.max_refinements) break;
            // 10% margin for the gap binary32 rounding leaves between the
            // inner recursive residual and the true one (measured below 3%)
            double tau = std::max(h->opt.inner_tol, 0.9 * tol * std::sqrt(hs.RR / hs.rt2));
            tau = std::min(tau, 0.5);
            const long long cap = std::min<long long>(max_steps, hs.s + h->opt.inner_max_steps);
            const long long s0 = hs.s;
            L::set_round(tb, tau * tau, cap, s);
            if (!run.noalloc) roctxRangePushA("ftgcr refinement round");
            run.start_round();
            rc = run.run_steps(k, s0, cap, evs);
            if (!run.noalloc) roctxRangePop();
            if (rc != FTGCR_OK) return rc;
            L::finalize_x(tb, h->nblk_st, h->kc, s);
            refinements += 1;
            inner_outcome = h->st_host->status;   // from the last status read
            inner_outcome_final = inner_outcome;
            if (inner_outcome == FTGCR_BREAKDOWN) break;
        }
    }
    // FP64 true residual of the returned x
    L::residual(tb, h->nblk_st, h->kc, 0, 0, s);
    HIP_TRY(h, hipEventRecord(h->ev_stop, s));
    rc = run.read_state();
    if (rc != FTGCR_OK) return rc;
    float ms = 0.f;
    HIP_TRY(h, hipEventElapsedTime(&ms, h->ev_start, h->ev_stop));
    SolveState st = *h->st_host;
    if (mixed) {
        // the outer loop decides convergence on the true residual
        if (st.rt2 <= tol * tol * st.RR) st.status = FTGCR_CONVERGED;
        else if (inner_outcome_final == FTGCR_BREAKDOWN) st.status = FTGCR_BREAKDOWN;
        else st.status = FTGCR_MAX_STEPS;
    }
    fill_stats(h, st, refinements, ms, stats);
    if (stats && stats->hist && stats->hist_cap > 0) {
        const long long nh = std::min<long long>(std::min<long long>(st.s, h->opt.hist_cap), stats->hist_cap);
        if (nh > 0) HIP_TRY(h, hipMemcpy(stats->hist, in.hist, (size_t)nh * sizeof(double), hipMemcpyDeviceToHost));
        stats->hist_len = nh;
    }
    return FTGCR_OK;
}

// ---------------------------------------------------------------------------
// FT-GMRES(k) solve
// ---------------------------------------------------------------------------

// The GMRES working vectors inside the FP64 workspace layout: v_0..v_kmax in
// the basis slots, z_0..z_{kmax-1} and w in the image slots.
GmInst make_gm_inst(const ftgcr_handle* h, const double* rhs, double* x, void* ws)
{
    const Inst<double> in = make_inst<double>(h, rhs, x, ws);
    GmInst gi;
    std::memset(&gi, 0, sizeof gi);
    gi.g = in.g;
    for (int l = 0; l <= h->kmax; ++l) gi.U[l] = in.U[l];
    for (int l = 0; l < h->kmax; ++l) gi.Z[l] = in.AP[l];
    gi.W = in.AP[h->kmax];
    gi.X[0] = in.X[0];
    gi.X[1] = in.X[1];
    gi.rhs = rhs;
    gi.st = h->gm_st;
    gi.part = in.part;
    gi.pstride = in.pstride;
    gi.hist = in.hist;
    gi.hist_cap = in.hist_cap;
    gi.nblk_st = h->nblk_st;
    gi.kc = h->kc;
    gi.tx = h->tx;
    gi.ty = h->ty;
    gi.tz = h->tz;
    // the option, else the mesh's default (the autotuner's choice is made
    // for the FT-GCR passes)
    const int os = h->opt.order_stencil;
    gi.ord = (os >= FTGCR_ORDER_X && os <= FTGCR_ORDER_XCD) ? os - 1
                                                           : (h->geo.mesh == FTGCR_MESH_OCTAHEDRAL ? ORD_XCD : ORD_X);
    return gi;
}

ftgcr_status gm_solve_impl(ftgcr_handle* h, const double* rhs, double* x, double tol, int k,
                           const ftgcr_fault_plan* plan, ftgcr_stats* stats, void* ws, void* staging = nullptr,
                           size_t staging_bytes = 0)
{
    using G = GmLaunch;
    hipStream_t s = h->stream;
    std::vector<DevEvent> evs;
    ftgcr_status rc = stage_events(h, plan, evs, staging, staging_bytes);
    if (rc != FTGCR_OK) return rc;
    const GmInst gi = make_gm_inst(h, rhs, x, ws);
    HIP_TRY(h, hipMemcpyAsync(h->gm_inst, &gi, sizeof gi, hipMemcpyHostToDevice, s));
    HIP_TRY(h, hipStreamSynchronize(s));
    const GmInst* d = h->gm_inst;
    // geometry and the column grid of the two-lane FP64 column kernel
    const Table<double> tb{h->inst_dbg, h->blk0, h->blk0 + 2, h->blk0 + 4, 1, h->geo.mesh, h->precond};
    const int nblk_col = (h->geo.ncols + COLS_PER_BLOCK - 1) / COLS_PER_BLOCK;
    const int nst = h->nblk_st, kc = h->kc;
    const bool nt = gm_nt_hint(k, h->geo.n);
    GmState* hs = h->gm_host;
    auto read_head = [&]() -> ftgcr_status {
        HIP_TRY(h, hipGetLastError());
        HIP_TRY(h, hipMemcpyAsync(hs, h->gm_st, offsetof(GmState, den), hipMemcpyDeviceToHost, s));
        HIP_TRY(h, hipStreamSynchronize(s));
        return FTGCR_OK;
    };
    auto inject = [&](const DevEvent& ev, long long t) {
        G::event_prep(d, ev.vec, t, s);
        if (ev.vec == FTGCR_V_X || ev.vec == FTGCR_V_R) G::event_copy(d, nst, kc, s);
        const int grid = (int)std::max<long long>(1, std::min<long long>((ev.count + 255) / 256, 8192));
        G::event_inject(d, grid, ev.idx, ev.bits, ev.count, ev.start, ev.bit, s);
    };
    // one Arnoldi step; `at` are the fault events of executed step t
    auto step = [&](const std::vector<const DevEvent*>& at, long long t) {
        for (const DevEvent* ev : at)
            if (ev->vec == FTGCR_V_X || ev->vec == FTGCR_V_R) inject(*ev, t);
        G::precond(tb, d, nblk_col, h->H, s);
        bool ap = false;
        for (const DevEvent* ev : at) {
            if (ev->vec == FTGCR_V_P || ev->vec == FTGCR_V_E) inject(*ev, t);
            ap = ap || ev->vec == FTGCR_V_AP;
        }
        if (ap) {
            G::stencil(d, nst, kc, 0, h->geo.mesh, nt, s);
            for (const DevEvent* ev : at)
                if (ev->vec == FTGCR_V_AP) inject(*ev, t);
            G::dots(d, nst, kc, s);
        } else {
            G::stencil(d, nst, kc, 1, h->geo.mesh, nt, s);
        }
        G::finish_h(d, s);
        G::orth(d, nst, kc, nt, s);
        G::finish_step(d, s);
    };
    HIP_TRY(h, hipEventRecord(h->ev_start, s));
    G::init(d, k, h->opt.ft, h->opt.max_steps, tol * tol, s);
    size_t evp = 0;
    const std::vector<const DevEvent*> none;
    const long long guard = 4 * (h->opt.max_steps + 16) + 64;
    for (long long iter = 0;; ++iter) {
        if (iter > guard) return fail(h, FTGCR_E_HIP, "GMRES cycle loop did not terminate");
        G::residual(d, nst, kc, h->geo.mesh, s);
        G::restart(d, s);
        rc = read_head();
        if (rc != FTGCR_OK) return rc;
        if (hs->status != RUNNING) break;
        if (!hs->active) continue;   // rolled back at the cycle's end: the restored x's residual next
        while (evp < evs.size() && evs[evp].step <= hs->s) ++evp;
        if (evp < evs.size() && evs[evp].step <= hs->s + k) {
            // a fault event falls in this cycle: step by step, reading the
            // executed-step count before each step
            for (int j = 0; j < k; ++j) {
                if (j > 0) {
                    rc = read_head();
                    if (rc != FTGCR_OK) return rc;
                    if (hs->status != RUNNING || !hs->active) break;
                }
                const long long t = hs->s + 1;
                while (evp < evs.size() && evs[evp].step < t) ++evp;
                std::vector<const DevEvent*> at;
                for (size_t q = evp; q < evs.size() && evs[q].step == t; ++q) at.push_back(&evs[q]);
                step(at, t);
            }
        } else {
            for (int j = 0; j < k; ++j) step(none, 0);
        }
        G::xupd(d, nst, kc, nt, s);
        G::finish_x(d, s);
    }
    G::finalize(d, nst, kc, s);
    HIP_TRY(h, hipEventRecord(h->ev_stop, s));
    HIP_TRY(h, hipGetLastError());
    HIP_TRY(h, hipMemcpyAsync(hs, h->gm_st, sizeof(GmState), hipMemcpyDeviceToHost, s));
    HIP_TRY(h, hipStreamSynchronize(s));
    float ms = 0.f;
    HIP_TRY(h, hipEventElapsedTime(&ms, h->ev_start, h->ev_stop));
    if (stats) {
        stats->status = hs->status;
        stats->detections = hs->detections;
        stats->stagnation_accepts = hs->stagnation_accepts;
        stats->events_applied = hs->events_applied;
        stats->steps_executed = hs->s;
        stats->steps_accepted = hs->accepted;
        stats->steps_wasted = hs->s - hs->accepted;
        stats->cycles = hs->cycles;
        stats->refinements = 0;
        stats->rhs_norm2 = hs->RR;
        stats->rr_final = hs->rho2;
        stats->rel_res_recursive = hs->RR > 0 ? std::sqrt(hs->rho2 / hs->RR) : 0.0;
        stats->rel_res_true = stats->rel_res_recursive;
        stats->time_ms = ms;
        stats->log_len = 0;
        if (stats->log && stats->log_cap > 0) {
            const int nlog = std::min(std::min(hs->log_len, LOG_CAP), stats->log_cap);
            for (int q = 0; q < nlog; ++q) {
                stats->log[q].step = hs->log[q].step;
                stats->log[q].nu = hs->log[q].nu;
                stats->log[q].action = hs->log[q].action;
                stats->log[q].rr_old = hs->log[q].rr_old;
                stats->log[q].rr_new = hs->log[q].rr_new;
            }
            stats->log_len = nlog;
        }
        stats->hist_len = 0;
        if (stats->hist && stats->hist_cap > 0) {
            const long long nh = std::min<long long>(std::min<long long>(hs->s, h->opt.hist_cap), stats->hist_cap);
            if (nh > 0) HIP_TRY(h, hipMemcpy(stats->hist, gi.hist, (size_t)nh * sizeof(double), hipMemcpyDeviceToHost));
            stats->hist_len = nh;
        }
    }
    return FTGCR_OK;
}

// ---------------------------------------------------------------------------
// batched solve
// ---------------------------------------------------------------------------
//
// Members step together: each launch of a step kernel covers the blocks of
// every unfinished member (block -> member by a prefix search), and the
// one-block reductions run one block per member.  All members share one
// Thomas depth and one stencil tiling.  Finished members are dropped from the
// launch table at the next status read.

// Device tables of a batch of n members on the leading handle, grown when n
// exceeds what earlier calls needed (the only allocation of a batched solve).
ftgcr_status batch_tables(ftgcr_handle* h0, int n)
{
    auto& B = h0->batch;
    if (n <= B.cap) return FTGCR_OK;
    if (B.graph) (void)hipGraphExecDestroy(B.graph);
    (void)hipFree(B.inst);
    (void)hipFree(B.blk0);
    (void)hipFree(B.status);
    (void)hipFree(B.all);
    (void)hipFree(B.blk0_all);
    B = ftgcr_handle::Batch{};
    const size_t pre = 3 * (size_t)(n + 1) * sizeof(int);
    if (hipMalloc(&B.inst, n * sizeof(Inst<double>)) != hipSuccess || hipMalloc(&B.blk0, pre) != hipSuccess ||
        hipMalloc(&B.status, 2 * n * sizeof(long long)) != hipSuccess ||
        hipMalloc(&B.all, n * sizeof(Inst<double>)) != hipSuccess || hipMalloc(&B.blk0_all, pre) != hipSuccess) {
        (void)hipFree(B.inst);
        (void)hipFree(B.blk0);
        (void)hipFree(B.status);
        (void)hipFree(B.all);
        (void)hipFree(B.blk0_all);
        B = ftgcr_handle::Batch{};
        return fail(h0, FTGCR_E_NOMEM, "batch table allocation failed");
    }
    B.cap = n;
    return FTGCR_OK;
}

// Launch-table shape of the running members: blocks of the three grids.
struct BatchShape {
    int n = 0, cols = 0, sts = 0, dirs = 0;
};

// Upload the members' instance records and block prefixes into `inst` /
// `blk0` (device, capacity for members.size()).
ftgcr_status upload_batch(ftgcr_handle* h0, const std::vector<Inst<double>>& ins, const std::vector<int>& members,
                          int H, Inst<double>* inst, int* blk0, BatchShape& sh, Table<double>& tb)
{
    const int na = (int)members.size();
    std::vector<Inst<double>> act(na);
    std::vector<int> pre(3 * (na + 1), 0);
    bool mixed_depth = false;
    for (int q = 0; q < na; ++q) {
        act[q] = ins[members[q]];
        mixed_depth = mixed_depth || thomas_depth(act[q].g.nz) != H;
        pre[q + 1] = pre[q] + act[q].nblk_col;
        pre[na + 1 + q + 1] = pre[na + 1 + q] + act[q].nblk_st;
        pre[2 * (na + 1) + q + 1] = pre[2 * (na + 1) + q] + act[q].nblk_dir;
    }
    HIP_TRY(h0, hipMemcpy(inst, act.data(), na * sizeof(Inst<double>), hipMemcpyHostToDevice));
    HIP_TRY(h0, hipMemcpy(blk0, pre.data(), pre.size() * sizeof(int), hipMemcpyHostToDevice));
    sh.n = na;
    sh.cols = pre[na];
    sh.sts = pre[2 * na + 1];
    sh.dirs = pre[3 * na + 2];
    tb = Table<double>{inst, blk0, blk0 + na + 1, blk0 + 2 * (na + 1), na, h0->geo.mesh, h0->precond,
                       mixed_depth ? 1 : 0};
    return FTGCR_OK;
}

// One batched step over the launch table; `mid` are the step's e events
// (member, event), injected by `apply` between the decision and the dots
// pass.
template <class Apply>
void batch_step(const Table<double>& tb, const BatchShape& sh, int H, int kc, bool nt_ap, hipStream_t s,
                const std::vector<std::pair<int, const DevEvent*>>& mid, Apply&& apply)
{
    using L = Launch<double>;
    L::update_thomas(tb, sh.cols, H, 0, s);
    if (!mid.empty()) {
        L::finish_col(tb, 0, s);
        for (const auto& me : mid) apply(me.first, *me.second);
        L::stencil_dots(tb, sh.sts, kc, 0, s);
        L::finish_alpha(tb, s);
    } else {
        L::stencil_dots(tb, sh.sts, kc, 1, s);
        L::finish_step(tb, s);
    }
    L::dir_update(tb, sh.dirs, kc < 4 ? kc : 4, 0, nt_ap, s);
    L::finish_beta(tb, 0, s);
}

// How a batch runs in the resident kernel: its members by template depth, a
// number of wavefronts per block for each depth.  A launch takes one block per
// CU at most, so members of a depth go together as far as their blocks fit:
// the fewest wavefronts per block with which all of them do (the quickest
// step), else the most the depth allows (the most cells in flight: two
// 256 x 128 x 32 members at 8 wavefronts take 41 us a step together, one at 4
// takes 22).
struct ResidentBatch {
    struct Depth {
        int H, waves;
        std::vector<int> members;
    };
    std::vector<Depth> depths;
    std::vector<int> rtx, nblk;   // per member
};

// Launches of members with these blocks: first fit by falling counts, at most
// `most` blocks in each.  bins: the indices into `blocks` of each launch.
void first_fit(const std::vector<int>& blocks, int most, std::vector<std::vector<int>>& bins)
{
    std::vector<int> order(blocks.size()), room;
    for (size_t q = 0; q < order.size(); ++q) order[q] = (int)q;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return blocks[a] > blocks[b]; });
    bins.clear();
    for (int q : order) {
        size_t b = 0;
        while (b < bins.size() && room[b] < blocks[q]) ++b;
        if (b == bins.size()) {
            bins.emplace_back();
            room.push_back(most);
        }
        bins[b].push_back(q);
        room[b] -= blocks[q];
    }
}

// About the microseconds a step of the planned members with take(m) takes in
// the resident kernel, and one of all members in streaming launches, with all of
// them running.  Measured at k = 3 to 16 on 2 to 16 equal members of 25 sizes on
// both meshes: launches of the resident kernel take 3% more per k beyond 3;
// streaming launches 25 us, 5 a member (less on the smallest) and 18
// (octahedral mesh: 21) a million cells, tiles counted whole, at the bytes of k =
// 3, in proportion to a step's bytes.  The two come
// out on the wrong side of each other where they differ by a tenth at most.
template <class Take>
double batch_resident_us(const ResidentBatch& rb, int mesh, int k, int most, Take&& take)
{
    double us = 0.0;
    for (const auto& d : rb.depths) {
        std::vector<int> blocks;
        for (int m : d.members)
            if (take(m)) blocks.push_back(rb.nblk[m]);
        std::vector<std::vector<int>> bins;
        first_fit(blocks, most, bins);
        us += (double)bins.size() * resident_step_us(mesh, d.H, 8, d.waves);
    }
    return us * (1.0 + 0.03 * (k - 3));
}

double batch_streaming_us(ftgcr_handle* const* hs, int n, int k)
{
    const bool oct = hs[0]->geo.mesh == FTGCR_MESH_OCTAHEDRAL;
    const double per = (oct ? 21.0 : 18.0) * (10.0 + k + 3.0 / k) / 14.0;
    double us = 25.0;
    for (int m = 0; m < n; ++m) {
        const double cells = 1e-6 * (double)hs[m]->tx * hs[m]->ty * ST_THREADS * hs[m]->geo.nz;   // whole tiles
        us += std::min(2.0 * per * cells, 5.0 + per * cells);
    }
    return us;
}

// Whether the batch runs there (else it streams): every member has to, and the
// launches of one block per CU at most have to be quicker than streaming ones
// over all members, which they are not where each holds a single member or two
// of a million cells or less.  Microseconds a member and step, streaming and
// resident, k = 3: 12 of 480 x 100 x 5 11, 16; 12 of 384 x 128 x 24 29, 36; 12 of
// O_80 x 20 19, 26; 4 of O_60 x 17 17, 23; but 2 of them 23, 24, 2 of 384 x 128 x
// 24 39, 38, 12 of 512 x 128 x 16 27, 24 and 12 of 128 x 64 x 16 7, 3.
bool plan_resident_batch(ftgcr_handle* const* hs, int n, int k, ResidentBatch& rb)
{
    // a tiling asked for in the options means the streaming kernels
    const int bkc = hs[0]->opt.batch_levels_per_block;
    if (bkc != hs[0]->tuned_batch_kc && (bkc == 1 || bkc == 2 || bkc == 4 || bkc == 8 || bkc == 16)) return false;
    rb.rtx.assign(n, 0);
    rb.nblk.assign(n, 0);
    std::map<int, std::vector<int>> by_depth;
    for (int m = 0; m < n; ++m) {
        if (!use_resident(hs[m])) return false;
        by_depth[hs[m]->H].push_back(m);
    }
    const int cus = hs[0]->cus, mesh = hs[0]->geo.mesh;
    const int most = std::min(cus, RES_BLOCKS);
    for (const auto& d : by_depth) {
        const int H = d.first;
        int waves = 0;
        for (int w = 1; w <= RES_WAVES; w *= 2) {
            long long total = 0;
            bool fits = true;
            for (int m : d.second) {
                const Geo& g = hs[m]->geo;
                int tx = 0, nb = 0;
                fits = fits && resident_shape(mesh, g.nx, g.ny, H, 8, cus, w, &tx, &nb);
                total += nb;
            }
            if (!fits || !resident_fits<double>(mesh, H, w, most, k)) continue;
            waves = w;
            if (total <= most) break;
        }
        if (waves == 0) return false;
        for (int m : d.second) {
            const Geo& g = hs[m]->geo;
            resident_shape(mesh, g.nx, g.ny, H, 8, cus, waves, &rb.rtx[m], &rb.nblk[m]);
        }
        rb.depths.push_back({H, waves, d.second});
    }
    return n == 1 || batch_resident_us(rb, mesh, k, most, [](int) { return true; }) < batch_streaming_us(hs, n, k);
}

// Whether a planned batch takes its steps up to the last fault event in
// streaming launches, all members together, before it goes on in the resident
// kernel: there the members with events run ahead of the others from event to
// event, a round of launches and a status read each (175 us), and a step with
// an event in e is the member's alone; here a step with events costs a status
// read (45 us).  Estimated over the steps a solve usually takes (50 a decade).
// Microseconds a member and step over 100 steps, streaming and resident, 16 of
// 64 x 32 x 8: flips in x in one member every second step 4.5, 7.2, every 16th
// 2.8, 2.5; in e in all members every 8th 4.6, 7.5, every 50th 2.7, 2.1; 8 of
// O_20 x 51: in x in one member every 4th 10.7, 12.9, every 50th 8.2, 7.5.
bool stream_events_first(ftgcr_handle* const* hs, int n, int k, const ResidentBatch& rb,
                         const std::vector<std::vector<DevEvent>>& evs, const double* tol)
{
    const int mesh = hs[0]->geo.mesh, most = std::min(hs[0]->cus, RES_BLOCKS);
    std::set<long long> steps;   // with events
    long long rounds = 0, events = 0, last = 0;
    double alone = 0.0;   // members' own streaming steps
    bool others = false;
    std::vector<char> has(n, 0);
    for (int m = 0; m < n; ++m) {
        const long long usual = (long long)(50.0 * std::max(1.0, -std::log10(tol[m])));
        long long mine = 0, at = 0, e_at = 0;
        for (const DevEvent& ev : evs[m]) {
            if (ev.step > usual) break;
            if (ev.step != at) mine += 1;
            at = ev.step;
            if (ev.vec == FTGCR_V_E && ev.step != e_at) {   // that step, then a launch again
                e_at = ev.step;
                mine += 1;
                alone += 33.0 + 18e-6 * (double)hs[m]->geo.n;
            }
            steps.insert(at);
            events += 1;
        }
        has[m] = mine > 0;
        others = others || mine == 0;
        rounds = std::max(rounds, mine);
        last = std::max(last, at);
    }
    if (events == 0) return false;
    const double ahead = batch_resident_us(rb, mesh, k, most, [&](int m) { return has[m] != 0; });
    const double all = batch_resident_us(rb, mesh, k, most, [](int) { return true; });
    const double resident = 175.0 * rounds + 10.0 * events + alone + ahead * last;
    const double streaming = 45.0 * steps.size() + 7.5 * (events - (long long)steps.size()) +
                             (batch_streaming_us(hs, n, k) - (others ? all : 0.0)) * last;
    return streaming < resident;
}

// The steps of a batch planned by plan_resident_batch, from every member's
// state to its outcome.  Members with fault events ahead run first, each to
// the step before its next one; once none is left, all run to their end.  When
// a launch does not run (its blocks do not start together, or the device does
// not take it), the members still running are left to the streaming kernels:
// `left`, with the steps each has executed in `base` and its next event in
// `evp`.
// inst, blk0, status: device tables with room for n members; single(m) the
// member's own launch table, apply(m, event) injects an event.
template <class Single, class Apply>
ftgcr_status run_resident_batch(ftgcr_handle* const* hs, int n, int k, const ResidentBatch& rb,
                                const std::vector<Inst<double>>& ins, const std::vector<std::vector<DevEvent>>& evs,
                                const Table<double>& tb_all, long long* status, Inst<double>* inst, int* blk0,
                                std::vector<int>& left, std::vector<long long>& base, std::vector<size_t>& evp,
                                Single&& single, Apply&& apply)
{
    using L = Launch<double>;
    ftgcr_handle* h0 = hs[0];
    hipStream_t s = h0->stream;
    const int most = std::min(h0->cus, RES_BLOCKS);
    std::vector<char> resident_norms(n, 0);   // the member's state holds the resident kernel's norms
    std::vector<long long> host(2 * n), before(n, -1);
    std::vector<char> launched(n, 0), norms_before(n, 0);
    std::vector<std::vector<const DevEvent*>> on_r(n);   // events on r before the member's launch
    while (true) {
        L::gather_status(tb_all, status, s);
        HIP_TRY(h0, hipMemcpyAsync(host.data(), status, 2 * n * sizeof(long long), hipMemcpyDeviceToHost, s));
        HIP_TRY(h0, hipStreamSynchronize(s));
        bool any = false, ahead = false, stream_on = false;
        for (int m = 0; m < n; ++m) {
            if (host[2 * m] == BROKEN) return fail(h0, FTGCR_E_HIP, "the resident kernel's blocks did not run together");
            if (host[2 * m] != RUNNING) continue;
            any = true;
            if (launched[m] && host[2 * m + 1] <= before[m]) {   // nothing of it has changed
                resident_norms[m] = norms_before[m];
                stream_on = true;
            } else {
                on_r[m].clear();
            }
            while (evp[m] < evs[m].size() && evs[m][evp[m]].step <= host[2 * m + 1]) ++evp[m];
            ahead = ahead || evp[m] < evs[m].size();
        }
        if (!any) return FTGCR_OK;
        if (stream_on) {
            L::resident_late(tb_all, s);
            for (int m = 0; m < n; ++m) {
                if (host[2 * m] != RUNNING) continue;
                if (resident_norms[m])
                    streaming_norms<double>(single(m), on_r[m], ins[m].nblk_col, hs[m]->H, s);
                left.push_back(m);
                base[m] = host[2 * m + 1];
            }
            return FTGCR_OK;
        }
        std::fill(launched.begin(), launched.end(), 0);
        std::vector<Inst<double>> act;
        std::vector<int> pre;
        struct Go {
            const ResidentBatch::Depth* d;
            int first, at, count, blocks;
        };
        std::vector<Go> gos;
        bool streamed = false;
        for (const auto& d : rb.depths) {
            std::vector<Inst<double>> go_in;
            for (int m : d.members) {
                if (host[2 * m] != RUNNING || (ahead && evp[m] >= evs[m].size())) continue;
                const long long next = host[2 * m + 1] + 1;
                bool now = evp[m] < evs[m].size() && evs[m][evp[m]].step == next, stream = false;
                if (now) {
                    size_t end = evp[m];
                    for (; end < evs[m].size() && evs[m][end].step == next; ++end)
                        stream = stream || evs[m][end].vec == FTGCR_V_E ||
                                 (evs[m][end].vec == FTGCR_V_R && !resident_norms[m]);
                    if (stream) {   // this step in the streaming kernels
                        const Table<double> t1 = single(m);
                        if (resident_norms[m]) L::norms(t1, ins[m].nblk_col, hs[m]->H, s);
                        resident_norms[m] = 0;
                        std::vector<std::pair<int, const DevEvent*>> mid;
                        for (; evp[m] < end; ++evp[m]) {
                            if (evs[m][evp[m]].vec == FTGCR_V_E) mid.push_back({m, &evs[m][evp[m]]});
                            else apply(m, evs[m][evp[m]]);
                        }
                        BatchShape one;
                        one.n = 1;
                        one.cols = ins[m].nblk_col;
                        one.sts = ins[m].nblk_st;
                        one.dirs = ins[m].nblk_dir;
                        batch_step(t1, one, hs[m]->H, ins[m].kc, nt_ap_hint(k, hs[m]->geo.n, 8), s, mid, apply);
                        streamed = true;
                        continue;
                    }
                    for (; evp[m] < end; ++evp[m]) {
                        if (evs[m][evp[m]].vec == FTGCR_V_R) on_r[m].push_back(&evs[m][evp[m]]);
                        apply(m, evs[m][evp[m]]);
                    }
                }
                Inst<double> in = ins[m];
                in.rtx = rb.rtx[m];
                in.nblk_res = rb.nblk[m];
                in.res_new_norms = resident_norms[m] ? 0 : 1;
                in.res_leave = forced_outcome(hs[m]);
                in.res_stop = next - 1 + RES_STEPS;
                if (evp[m] < evs[m].size()) in.res_stop = std::min<long long>(in.res_stop, evs[m][evp[m]].step - 1);
                norms_before[m] = resident_norms[m];
                resident_norms[m] = 1;
                before[m] = next - 1;
                launched[m] = 1;
                go_in.push_back(in);
            }
            std::vector<int> blocks;
            for (const auto& in : go_in) blocks.push_back(in.nblk_res);
            std::vector<std::vector<int>> bins;   // members of one launch
            first_fit(blocks, most, bins);
            for (const auto& bin : bins) {
                Go go{&d, (int)pre.size(), (int)act.size(), (int)bin.size(), 0};
                pre.push_back(0);
                for (int q : bin) {
                    act.push_back(go_in[q]);
                    go.blocks += go_in[q].nblk_res;
                    pre.push_back(go.blocks);
                }
                gos.push_back(go);
            }
        }
        if (act.empty() && !streamed) return fail(h0, FTGCR_E_HIP, "batched step loop did not terminate");
        if (act.empty()) continue;
        HIP_TRY(h0, hipMemcpyAsync(inst, act.data(), act.size() * sizeof(Inst<double>), hipMemcpyHostToDevice, s));
        HIP_TRY(h0, hipMemcpyAsync(blk0, pre.data(), pre.size() * sizeof(int), hipMemcpyHostToDevice, s));
        for (const Go& go : gos) {
            Table<double> t{};
            t.inst = inst + go.at;
            t.n = go.count;
            bool refused = false;
            for (int q = go.at; q < go.at + go.count; ++q) refused = refused || act[q].res_leave == FTGCR_RESIDENT_REFUSED;
            if (refused || resident_run<double>(t, blk0 + go.first, go.blocks, h0->geo.mesh, go.d->H, go.d->waves,
                                                ResidentArgs{-1, k + 1, 0, 0, 0, 0}, s) != hipSuccess) {
                (void)hipGetLastError();
                break;   // its members are found unchanged
            }
        }
        HIP_TRY(h0, hipStreamSynchronize(s));   // act and pre are read until here
    }
}

// Members step together: each launch of a step kernel covers the blocks of
// every member of the launch table (block -> member by a prefix search),
// and the one-block reductions run one block per member.  All members share
// one Thomas depth and one stencil tiling.  Steps without fault events are
// replayed from a captured graph of `poll_steps` steps (options.use_graphs
// of the leading handle), captured again only when the launch table changes
// shape.  A member that finishes does no work in later launches (every step
// kernel returns at once for a solve that is no longer running); finished
// members are compacted out of the table at a status read once their blocks
// are an eighth of the table's or more.
ftgcr_status solve_batch_impl(ftgcr_handle* const* hs, int n, const double* const* rhs, double* const* x,
                              const double* tol, int k, const ftgcr_fault_plan* plans, ftgcr_stats* stats)
{
    using L = Launch<double>;
    ftgcr_handle* h0 = hs[0];
    hipStream_t s = h0->stream;
    // common tiling: Thomas depth of the deepest member; stencil levels per
    // block from the first member's batch option (ftgcr_autotune_batch), else
    // those of the largest member
    int H = 4, kc = 1;
    long long biggest = -1;
    for (int m = 0; m < n; ++m) {
        H = std::max(H, hs[m]->H);
        if (hs[m]->geo.n > biggest) {
            biggest = hs[m]->geo.n;
            kc = hs[m]->kc;
        }
    }
    const int bkc = h0->opt.batch_levels_per_block;
    if (bkc == 1 || bkc == 2 || bkc == 4 || bkc == 8 || bkc == 16) kc = bkc;
    std::vector<Inst<double>> ins(n);
    std::vector<std::vector<DevEvent>> evs(n);
    for (int m = 0; m < n; ++m) {
        ftgcr_handle* h = hs[m];
        ins[m] = make_inst<double>(h, rhs[m], x[m], h->ws);
        ins[m].fold_st = ins[m].fold_dir = 0;
        ins[m].kc = kc;
        ins[m].tz = (h->geo.nz + kc - 1) / kc;
        ins[m].nblk_st = ins[m].tx * ins[m].ty * ins[m].tz;
        dir_tiling(kc, h->geo.nz, ins[m].tx, ins[m].ty, ins[m].kc_dir, ins[m].tz_dir, ins[m].nblk_dir);
        ftgcr_status rc = stage_events(h, plans ? &plans[m] : nullptr, evs[m]);
        if (rc != FTGCR_OK) {
            if (m) h0->err = h->err;
            return rc;
        }
    }
    ftgcr_status rc = batch_tables(h0, n);
    if (rc != FTGCR_OK) return rc;
    auto& B = h0->batch;
    std::vector<int> members(n);
    for (int m = 0; m < n; ++m) members[m] = m;
    // the full table (every member, in order) for the passes before and
    // after the steps, and the per-member single tables of the fault-event
    // kernels
    BatchShape sh_all;
    Table<double> tb_all{};
    rc = upload_batch(h0, ins, members, H, B.all, B.blk0_all, sh_all, tb_all);
    if (rc != FTGCR_OK) return rc;
    BatchShape sh;
    Table<double> tb{};
    rc = upload_batch(h0, ins, members, H, B.inst, B.blk0, sh, tb);
    if (rc != FTGCR_OK) return rc;
    auto single = [&](int m) {
        return Table<double>{B.all + m, hs[m]->blk0, hs[m]->blk0 + 2, hs[m]->blk0 + 4, 1, h0->geo.mesh,
                             h0->precond};
    };

    hipEvent_t e0 = h0->ev_start, e1 = h0->ev_stop;
    (void)hipEventRecord(e0, s);
    for (int m = 0; m < n; ++m)
        L::init_state(single(m), k, hs[m]->opt.ft, 0, hs[m]->opt.max_steps, tol[m] * tol[m], 1, 1, s);
    L::residual(tb, sh.sts, kc, 1, 1, s);
    L::update_thomas(tb, sh.cols, H, 1, s);
    L::finish_col(tb, 1, s);
    long long n_total = 0;
    for (int m = 0; m < n; ++m) n_total += hs[m]->geo.n;
    const bool nt_ap = nt_ap_hint(k, n_total, (int)sizeof(double));
    L::dir_update(tb, sh.dirs, kc < 4 ? kc : 4, 1, nt_ap, s);
    L::finish_beta(tb, 1, s);

    const int chunk = std::max(1, h0->opt.poll_steps);
    long long launched = 0, max_cap = 0;
    for (int m = 0; m < n; ++m) max_cap = std::max<long long>(max_cap, hs[m]->opt.max_steps);
    std::vector<size_t> evp(n, 0);
    std::vector<long long> host_status(2 * n);
    auto apply = [&](int m, const DevEvent& ev) {
        const Table<double> t1 = single(m);
        inject_event<double>(t1, ev, hs[m]->geo.n, s);
        if (ev.vec == FTGCR_V_R || ev.vec == FTGCR_V_AP) L::beta_dots(t1, ins[m].nblk_st, s);
    };
    const std::vector<std::pair<int, const DevEvent*>> no_mid;
    // replay `chunk` steps from the graph of this launch-table shape
    // (captured first when the shape is new)
    auto replay = [&]() -> ftgcr_status {
        const long long key[8] = {sh.n, sh.cols, sh.sts, sh.dirs, kc, H, nt_ap ? 1 : 0, chunk};
        if (!B.graph || std::memcmp(key, B.graph_key, sizeof key) != 0) {
            if (B.graph) {
                (void)hipGraphExecDestroy(B.graph);
                B.graph = nullptr;
            }
            HIP_TRY(h0, hipStreamBeginCapture(h0->cap_stream, hipStreamCaptureModeRelaxed));
            for (int q = 0; q < chunk; ++q) batch_step(tb, sh, H, kc, nt_ap, h0->cap_stream, no_mid, apply);
            hipGraph_t g = nullptr;
            HIP_TRY(h0, hipStreamEndCapture(h0->cap_stream, &g));
            const hipError_t e = hipGraphInstantiate(&B.graph, g, nullptr, nullptr, 0);
            (void)hipGraphDestroy(g);
            if (e != hipSuccess) {
                B.graph = nullptr;
                return fail(h0, FTGCR_E_HIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
            }
            std::memcpy(B.graph_key, key, sizeof key);
        }
        HIP_TRY(h0, hipGraphLaunch(B.graph, s));
        return FTGCR_OK;
    };
    ResidentBatch rb;
    std::vector<long long> base(n, 0);   // a member's steps before `launched` counts
    bool resident = plan_resident_batch(hs, n, k, rb);
    bool events_first = resident && stream_events_first(hs, n, k, rb, evs, tol);
    while (!members.empty()) {
        if (events_first) {
            events_first = false;
            for (int m : members) events_first = events_first || evp[m] < evs[m].size();
        }
        if (resident && !events_first) {
            resident = false;
            members.clear();
            launched = 0;
            rc = run_resident_batch(hs, n, k, rb, ins, evs, tb_all, B.status, B.inst, B.blk0, members, base, evp, single,
                                    apply);
            if (rc != FTGCR_OK) return rc;
            if (members.empty()) break;
            rc = upload_batch(h0, ins, members, H, B.inst, B.blk0, sh, tb);
            if (rc != FTGCR_OK) return rc;
        }
        // fault events of the next step, member by member: x, r, p, L(p)
        // events now, e events between the step's decision and its stencil
        // pass
        bool any_event = false;
        std::vector<std::pair<int, const DevEvent*>> mid;
        for (int m : members) {
            const long long at = base[m] + launched;
            while (evp[m] < evs[m].size() && evs[m][evp[m]].step <= at) ++evp[m];
            while (evp[m] < evs[m].size() && evs[m][evp[m]].step == at + 1) {
                const DevEvent& ev = evs[m][evp[m]++];
                if (ev.vec == FTGCR_V_E) mid.push_back({m, &ev});
                else apply(m, ev);
                any_event = true;
            }
        }
        long long cnt = any_event ? 1 : chunk;
        for (int m : members)
            if (evp[m] < evs[m].size())
                cnt = std::min<long long>(cnt, std::max<long long>(1, evs[m][evp[m]].step - 1 - base[m] - launched));
        if (cnt == chunk && !any_event && h0->opt.use_graphs) {
            rc = replay();
            if (rc != FTGCR_OK) return rc;
        } else {
            for (long long q = 0; q < cnt; ++q) batch_step(tb, sh, H, kc, nt_ap, s, mid, apply);   // cnt == 1 if mid
        }
        launched += cnt;
        L::gather_status(tb, B.status, s);
        if (hipMemcpyAsync(host_status.data(), B.status, 2 * members.size() * sizeof(long long),
                           hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return fail(h0, FTGCR_E_HIP, "batch status read failed");
        std::vector<int> still;
        long long done_blocks = 0;
        for (size_t q = 0; q < members.size(); ++q) {
            if (host_status[2 * q] == RUNNING) still.push_back(members[q]);
            else done_blocks += ins[members[q]].nblk_st;
        }
        if (still.empty()) break;
        if (8 * done_blocks >= sh.sts) {
            members.swap(still);
            rc = upload_batch(h0, ins, members, H, B.inst, B.blk0, sh, tb);
            if (rc != FTGCR_OK) return rc;
        }
        if (launched > max_cap + chunk + 16) return fail(h0, FTGCR_E_HIP, "batched step loop did not terminate");
    }
    L::finalize_x(tb_all, sh_all.sts, kc, s);
    L::residual(tb_all, sh_all.sts, kc, 0, 0, s);
    (void)hipEventRecord(e1, s);
    if (hipStreamSynchronize(s) != hipSuccess) return fail(h0, FTGCR_E_HIP, "batch synchronisation failed");
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    for (int m = 0; m < n; ++m) {
        ftgcr_handle* h = hs[m];
        if (hipMemcpy(h->st_host, h->st, sizeof(SolveState), hipMemcpyDeviceToHost) != hipSuccess)
            return fail(h0, FTGCR_E_HIP, "batch state read failed");
        if (stats) {
            fill_stats(h, *h->st_host, 0, ms, &stats[m]);
            if (stats[m].hist && stats[m].hist_cap > 0) {
                const long long nh = std::min<long long>(std::min<long long>(h->st_host->s, h->opt.hist_cap),
                                                         stats[m].hist_cap);
                if (nh > 0 && hipMemcpy(stats[m].hist, ins[m].hist, (size_t)nh * sizeof(double),
                                        hipMemcpyDeviceToHost) != hipSuccess)
                    return fail(h0, FTGCR_E_HIP, "batch history read failed");
                stats[m].hist_len = nh;
            }
        }
    }
    return FTGCR_OK;
}

// ---------------------------------------------------------------------------
// scratch of the allocation-free entry point
// ---------------------------------------------------------------------------

std::mutex g_scratch_mutex;
std::map<int, void*> g_scratch_ptr;   // device -> address of `scratch` there

}  // namespace

// Working vectors and fault-plan staging of ftgcr_solve_noalloc.  Every GPU
// the library runs on holds its own copy at its own address until the process
// ends; in host code `scratch` is only a stand-in for the symbol, never a
// device address: host code uses the address hipGetSymbolAddress returns.
static __device__ __align__(256) unsigned char scratch[FTGCR_NOALLOC_SCRATCH_BYTES];

namespace {

// Device address of `scratch` on device `dev`, which must be current: looked
// up on the first call on that device, then kept.
ftgcr_status scratch_on_device(ftgcr_handle* h, int dev, void** out)
{
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    auto it = g_scratch_ptr.find(dev);
    if (it == g_scratch_ptr.end()) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || ptr == nullptr)
            return fail(h, FTGCR_E_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        it = g_scratch_ptr.emplace(dev, ptr).first;
    }
    *out = it->second;
    return FTGCR_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------

extern "C" {

void ftgcr_default_options(ftgcr_options* opt)
{
    if (!opt) return;
    std::memset(opt, 0, sizeof *opt);
    opt->ft = 1;
    opt->poll_steps = 16;
    opt->max_steps = 100000;
    opt->inner_tol = 3e-5;
    opt->max_refinements = 20;
    opt->inner_max_steps = 5000;
    opt->hist_cap = 65536;
    opt->use_graphs = 1;
    opt->levels_per_block = 0;
    opt->profile_kernels = 0;
}

ftgcr_status ftgcr_create(const ftgcr_grid* grid, const ftgcr_coeffs* coeffs, ftgcr_precond precond,
                          ftgcr_precision precision, int32_t kmax, void* hip_stream, ftgcr_handle** out)
{
    if (!out) return fail(nullptr, FTGCR_E_INVALID, "out == NULL");
    *out = nullptr;
    if (!grid || !coeffs) return fail(nullptr, FTGCR_E_INVALID, "grid or coeffs == NULL");
    if (grid->mesh != FTGCR_MESH_LATLON && grid->mesh != FTGCR_MESH_OCTAHEDRAL)
        return fail(nullptr, FTGCR_E_INVALID, "grid.mesh must be FTGCR_MESH_LATLON or FTGCR_MESH_OCTAHEDRAL");
    const bool oct = grid->mesh == FTGCR_MESH_OCTAHEDRAL;
    if (!oct && (grid->nlon < 3 || grid->nlat < 1 || grid->nz < 1))
        return fail(nullptr, FTGCR_E_INVALID, "grid needs nlon >= 3, nlat >= 1, nz >= 1");
    if (oct && (grid->nlat < 1 || grid->nlat > 4000 || grid->nz < 1))
        return fail(nullptr, FTGCR_E_INVALID, "octahedral grid needs N = nlat in 1..4000 and nz >= 1");
    if (!(grid->shell_depth > 0)) return fail(nullptr, FTGCR_E_INVALID, "shell_depth must be > 0");
    if (!(coeffs->hill_width > 0) || !(coeffs->decay_z > 0) || !(coeffs->hill_amp >= 0) || !(coeffs->helmholtz > 0))
        return fail(nullptr, FTGCR_E_INVALID, "coefficients need hill_width > 0, decay_z > 0, hill_amp >= 0, helmholtz > 0");
    if (kmax < 1 || kmax > FTGCR_KMAX) return fail(nullptr, FTGCR_E_INVALID, "kmax out of range");
    if (precision != FTGCR_FP64 && precision != FTGCR_MIXED) return fail(nullptr, FTGCR_E_INVALID, "bad precision");
    if (precond != FTGCR_PRECOND_COLUMN && precond != FTGCR_PRECOND_NONE)
        return fail(nullptr, FTGCR_E_INVALID, "precond must be FTGCR_PRECOND_COLUMN or FTGCR_PRECOND_NONE");
    if (thomas_depth(grid->nz) < 0) return fail(nullptr, FTGCR_E_UNSUPPORTED, "nz > 96 is not supported");
    const long long ncols = oct ? oct_points(grid->nlat) : (long long)grid->nlon * grid->nlat;
    if (ncols > (1LL << 30) || ncols * grid->nz > (1LL << 40)) return fail(nullptr, FTGCR_E_UNSUPPORTED, "grid too large");

    ftgcr_handle* h = new (std::nothrow) ftgcr_handle();
    if (!h) return fail(nullptr, FTGCR_E_NOMEM, "host allocation failed");
    h->grid = *grid;
    h->co = *coeffs;
    h->precond = precond;
    h->precision = precision;
    h->kmax = kmax;
    h->stream = (hipStream_t)hip_stream;
    ftgcr_default_options(&h->opt);
    auto bail = [&](ftgcr_status code) {
        g_create_error = h->err;
        ftgcr_destroy(h);
        return code;
    };
    if (hipGetDevice(&h->device) != hipSuccess) {
        h->err = "hipGetDevice failed";
        return bail(FTGCR_E_HIP);
    }
    ftgcr_status rc = oct ? upload_tables_oct(h) : upload_tables(h);
    if (rc != FTGCR_OK) return bail(rc);
    h->H = thomas_depth(grid->nz);
    set_tiling(h);
    rc = setup_resident(h);
    if (rc != FTGCR_OK) return bail(rc);
    if (hipMalloc(&h->st, sizeof(SolveState)) != hipSuccess ||
        hipMemset(h->st, 0, sizeof(SolveState)) != hipSuccess ||
        hipMalloc(&h->inst, std::max(sizeof(Inst<double>), sizeof(Inst<float>))) != hipSuccess ||
        hipMalloc(&h->inst_dbg, sizeof(Inst<double>)) != hipSuccess ||
        hipMalloc(&h->blk0, 8 * sizeof(int)) != hipSuccess ||
        hipHostMalloc(&h->st_host, sizeof(SolveState)) != hipSuccess ||
        hipMalloc(&h->gm_st, sizeof(GmState)) != hipSuccess || hipMalloc(&h->gm_inst, sizeof(GmInst)) != hipSuccess ||
        hipHostMalloc(&h->gm_host, sizeof(GmState)) != hipSuccess ||
        hipEventCreate(&h->ev_start) != hipSuccess || hipEventCreate(&h->ev_stop) != hipSuccess) {
        h->err = "device allocation failed";
        return bail(FTGCR_E_NOMEM);
    }
    rc = upload_debug_inst(h);
    if (rc != FTGCR_OK) return bail(rc);
    if (hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking) != hipSuccess) {
        h->err = "hipStreamCreate failed";
        return bail(FTGCR_E_HIP);
    }
    *out = h;
    return FTGCR_OK;
}

ftgcr_status ftgcr_set_options(ftgcr_handle* h, const ftgcr_options* opt)
{
    if (!h || !opt) return FTGCR_E_INVALID;
    if (opt->poll_steps < 1 || opt->max_steps < 0 || opt->hist_cap < 0 || opt->max_refinements < 0 ||
        opt->inner_max_steps < 1 || !(opt->inner_tol > 0) || !(opt->inner_tol < 1) ||
        (opt->method != FTGCR_METHOD_GCR && opt->method != FTGCR_METHOD_GMRES) || opt->order_stencil < 0 ||
        opt->order_stencil > FTGCR_ORDER_XCD || opt->order_dir < 0 || opt->order_dir > FTGCR_ORDER_XCD)
        return fail(h, FTGCR_E_INVALID, "invalid options");
    if (opt->method == FTGCR_METHOD_GMRES && h->precision != FTGCR_FP64)
        return fail(h, FTGCR_E_UNSUPPORTED, "FT-GMRES is built for FP64 handles");
    if (opt->batch_levels_per_block != h->tuned_batch_kc) h->tuned_batch_kc = 0;
    h->opt = *opt;
    set_tiling(h);
    if (h->graph) {
        (void)hipGraphExecDestroy(h->graph);
        h->graph = nullptr;
        h->graph_steps = 0;
    }
    return upload_debug_inst(h);
}

ftgcr_status ftgcr_get_options(const ftgcr_handle* h, ftgcr_options* opt)
{
    if (!h || !opt) return FTGCR_E_INVALID;
    *opt = h->opt;
    return FTGCR_OK;
}

ftgcr_status ftgcr_set_stream(ftgcr_handle* h, void* hip_stream)
{
    if (!h) return FTGCR_E_INVALID;
    h->stream = (hipStream_t)hip_stream;
    return FTGCR_OK;
}

size_t ftgcr_workspace_bytes(const ftgcr_handle* h)
{
    if (!h) return 0;
    return layout(h).total;
}

ftgcr_status ftgcr_set_workspace(ftgcr_handle* h, void* dev_ptr, size_t bytes)
{
    if (!h) return FTGCR_E_INVALID;
    if (!dev_ptr) return fail(h, FTGCR_E_WORKSPACE, "workspace pointer is NULL");
    if (((uintptr_t)dev_ptr & 255) != 0) return fail(h, FTGCR_E_WORKSPACE, "workspace must be 256-byte aligned");
    if (bytes < layout(h).total) return fail(h, FTGCR_E_WORKSPACE, "workspace smaller than ftgcr_workspace_bytes()");
    h->ws = dev_ptr;
    h->ws_bytes = bytes;
    return FTGCR_OK;
}

ftgcr_status ftgcr_solve(ftgcr_handle* h, const double* rhs_dev, double* x_dev, double tol, int32_t k,
                         const ftgcr_fault_plan* plan, ftgcr_stats* stats)
{
    if (!h) return FTGCR_E_INVALID;
    if (!rhs_dev || !x_dev) return fail(h, FTGCR_E_INVALID, "rhs or x is NULL");
    if (!(tol > 0) || !std::isfinite(tol)) return fail(h, FTGCR_E_INVALID, "tol must be finite and > 0");
    if (k < 1 || k > h->kmax) return fail(h, FTGCR_E_INVALID, "k must be in [1, kmax]");
    if (!h->ws) return fail(h, FTGCR_E_WORKSPACE, "no workspace set");
    if (h->ws_bytes < layout(h).total) return fail(h, FTGCR_E_WORKSPACE, "workspace smaller than required by the current options");
    HIP_TRY(h, hipSetDevice(h->device));
    if (h->opt.method == FTGCR_METHOD_GMRES) {
        TraceRange tr("ftgcr_solve FT-GMRES");
        return gm_solve_impl(h, rhs_dev, x_dev, tol, k, plan, stats, h->ws);
    }
    if (h->precision == FTGCR_MIXED) {
        TraceRange tr("ftgcr_solve FT-GCR mixed");
        return solve_impl<float>(h, rhs_dev, x_dev, tol, k, plan, stats, h->ws);
    }
    TraceRange tr("ftgcr_solve FT-GCR FP64");
    return solve_impl<double>(h, rhs_dev, x_dev, tol, k, plan, stats, h->ws);
}

ftgcr_status ftgcr_solve_noalloc(ftgcr_handle* h, const double* rhs_dev, double* x_dev, double tol, int32_t k,
                                 const ftgcr_fault_plan* plan, ftgcr_stats* stats)
{
    if (!h) return FTGCR_E_INVALID;
    if (!rhs_dev || !x_dev) return fail(h, FTGCR_E_INVALID, "rhs or x is NULL");
    if (!(tol > 0) || !std::isfinite(tol)) return fail(h, FTGCR_E_INVALID, "tol must be finite and > 0");
    if (k < 1 || k > h->kmax) return fail(h, FTGCR_E_INVALID, "k must be in [1, kmax]");
    const size_t need = align256(layout(h).total);
    if (need > (size_t)FTGCR_NOALLOC_SCRATCH_BYTES)
        return fail(h, FTGCR_E_WORKSPACE, "the allocation-free solve needs " + std::to_string(need) +
                                              " bytes of scratch for this grid and kmax; it has " +
                                              std::to_string((size_t)FTGCR_NOALLOC_SCRATCH_BYTES));
    HIP_TRY(h, hipSetDevice(h->device));
    void* base = nullptr;
    ftgcr_status rc = scratch_on_device(h, h->device, &base);
    if (rc != FTGCR_OK) return rc;
    // the fault plan's entry lists follow the working vectors
    char* staging = (char*)base + need;
    const size_t staging_bytes = (size_t)FTGCR_NOALLOC_SCRATCH_BYTES - need;
    if (h->opt.method == FTGCR_METHOD_GMRES)
        return gm_solve_impl(h, rhs_dev, x_dev, tol, k, plan, stats, base, staging, staging_bytes);
    if (h->precision == FTGCR_MIXED)
        return solve_impl<float>(h, rhs_dev, x_dev, tol, k, plan, stats, base, staging, staging_bytes);
    return solve_impl<double>(h, rhs_dev, x_dev, tol, k, plan, stats, base, staging, staging_bytes);
}

ftgcr_status ftgcr_solve_batch(ftgcr_handle* const* hs, int32_t n, const double* const* rhs, double* const* x,
                               const double* tol, int32_t k, const ftgcr_fault_plan* plans, ftgcr_stats* stats)
{
    if (!hs || n < 1 || !rhs || !x || !tol) return FTGCR_E_INVALID;
    TraceRange tr("ftgcr_solve_batch");
    for (int m = 0; m < n; ++m) {
        ftgcr_handle* h = hs[m];
        if (!h) return FTGCR_E_INVALID;
        if (h->precision != FTGCR_FP64) return fail(hs[0], FTGCR_E_UNSUPPORTED, "batched solves are FP64 only");
        if (h->opt.method != FTGCR_METHOD_GCR)
            return fail(hs[0], FTGCR_E_UNSUPPORTED, "batched solves run FT-GCR (options.method of every member)");
        if (h->geo.mesh != hs[0]->geo.mesh)
            return fail(hs[0], FTGCR_E_UNSUPPORTED, "batch members on different meshes");
        if (h->precond != hs[0]->precond)
            return fail(hs[0], FTGCR_E_INVALID, "batch members with different preconditioners");
        if (!rhs[m] || !x[m]) return fail(hs[0], FTGCR_E_INVALID, "rhs or x is NULL");
        if (!(tol[m] > 0) || !std::isfinite(tol[m])) return fail(hs[0], FTGCR_E_INVALID, "tol must be finite and > 0");
        if (k < 1 || k > h->kmax) return fail(hs[0], FTGCR_E_INVALID, "k must be in [1, kmax] of every member");
        if (!h->ws || h->ws_bytes < layout(h).total) return fail(hs[0], FTGCR_E_WORKSPACE, "member without a large enough workspace");
        if (h->device != hs[0]->device) return fail(hs[0], FTGCR_E_INVALID, "members on different devices");
        for (int q = 0; q < m; ++q)
            if (hs[q] == h) return fail(hs[0], FTGCR_E_INVALID, "a handle appears twice in the batch");
    }
    HIP_TRY(hs[0], hipSetDevice(hs[0]->device));
    return solve_batch_impl(hs, n, rhs, x, tol, k, plans, stats);
}

ftgcr_status ftgcr_autotune(ftgcr_handle* h, const double* rhs_dev, double* x_scratch_dev, int32_t k,
                            int32_t steps, int32_t* chosen)
{
    if (!h) return FTGCR_E_INVALID;
    TraceRange tr("ftgcr_autotune");
    if (!rhs_dev || !x_scratch_dev) return fail(h, FTGCR_E_INVALID, "rhs or x is NULL");
    if (k < 1 || k > h->kmax || steps < 1) return fail(h, FTGCR_E_INVALID, "bad k or steps");
    if (!h->ws || h->ws_bytes < layout(h).total) return fail(h, FTGCR_E_WORKSPACE, "no workspace set");
    HIP_TRY(h, hipSetDevice(h->device));
    Tuned tu = tuned_for(h);
    const ftgcr_options saved = h->opt;
    // one timed run of `steps` steps from x = 0 (the tolerance is never met)
    auto run = [&](ftgcr_stats* st) -> ftgcr_status {
        HIP_TRY(h, hipMemsetAsync(x_scratch_dev, 0, (size_t)h->geo.n * sizeof(double), h->stream));
        std::memset(st, 0, sizeof *st);
        return ftgcr_solve(h, rhs_dev, x_scratch_dev, 1e-300, k, nullptr, st);
    };
    if (tu.kc == 0) {
        float best_ms = 0.f;
        const int cand[] = {2, 4, 8};
        for (int kc : cand) {
            if (kc > h->geo.nz) continue;
            ftgcr_options o = saved;
            o.levels_per_block = kc;
            o.max_steps = steps;
            o.profile_kernels = 0;
            ftgcr_status rc = ftgcr_set_options(h, &o);
            float ms_min = 0.f;
            for (int rep = 0; rep < 2 && rc == FTGCR_OK; ++rep) {
                ftgcr_stats st;
                rc = run(&st);
                if (rc == FTGCR_OK && (rep == 0 || st.time_ms < ms_min)) ms_min = (float)st.time_ms;
            }
            if (rc != FTGCR_OK) {
                ftgcr_set_options(h, &saved);
                return rc;
            }
            if (tu.kc == 0 || ms_min < best_ms) {
                tu.kc = kc;
                best_ms = ms_min;
            }
        }
    }
    if ((tu.ord_st < 0 || tu.ord_dir < 0) && saved.method == FTGCR_METHOD_GCR) {
        // block orders at that tiling: every pair for the dots pass and the
        // direction pass, by the two kernels' own mean launch times (the
        // pair, since one pass's order changes what the other finds cached).
        // The mesh's default pair stays unless another is at least 1%
        // faster, so that timing noise does not pick between equals.  The
        // handle's kernel-time totals are kept aside meanwhile.
        const int def = h->geo.mesh == FTGCR_MESH_OCTAHEDRAL ? ORD_XCD : ORD_X;
        double kt_ms[3], best_t = 0.0, def_t = 0.0;
        long long kt_n[3];
        std::memcpy(kt_ms, h->kt_ms, sizeof kt_ms);
        std::memcpy(kt_n, h->kt_n, sizeof kt_n);
        ftgcr_status rc = FTGCR_OK;
        for (int os = ORD_X; os <= ORD_XCD && rc == FTGCR_OK; ++os) {
            for (int od = ORD_X; od <= ORD_XCD && rc == FTGCR_OK; ++od) {
                ftgcr_options o = saved;
                o.levels_per_block = tu.kc;
                o.max_steps = steps;
                o.profile_kernels = 0xC;   // stencil_dots and dir_update
                o.order_stencil = os + 1;
                o.order_dir = od + 1;
                rc = ftgcr_set_options(h, &o);
                double t_min = 0.0;
                for (int rep = 0; rep < 2 && rc == FTGCR_OK; ++rep) {
                    for (int q = 0; q < 3; ++q) {
                        h->kt_ms[q] = 0.0;
                        h->kt_n[q] = 0;
                    }
                    ftgcr_stats st;
                    rc = run(&st);
                    double t = 0.0;
                    for (int q = 1; q < 3; ++q)
                        if (h->kt_n[q]) t += h->kt_ms[q] / (double)h->kt_n[q];
                    if (rep == 0 || t < t_min) t_min = t;
                }
                if (rc == FTGCR_OK && (tu.ord_st < 0 || t_min < best_t)) {
                    tu.ord_st = os;
                    tu.ord_dir = od;
                    best_t = t_min;
                }
                if (os == def && od == def) def_t = t_min;
            }
        }
        if (rc == FTGCR_OK && !(best_t < 0.99 * def_t)) {
            tu.ord_st = def;
            tu.ord_dir = def;
        }
        std::memcpy(h->kt_ms, kt_ms, sizeof kt_ms);
        std::memcpy(h->kt_n, kt_n, sizeof kt_n);
        if (rc != FTGCR_OK) {
            ftgcr_set_options(h, &saved);
            return rc;
        }
    }
    {
        std::lock_guard<std::mutex> lock(g_tune_mutex);
        g_tuned[tune_key(h)] = tu;
    }
    h->tuned_kc = tu.kc;
    h->tuned_ord_st = tu.ord_st;
    h->tuned_ord_dir = tu.ord_dir;
    ftgcr_status rc0 = ftgcr_set_options(h, &saved);
    if (rc0 != FTGCR_OK) return rc0;
    if (h->graph) {
        (void)hipGraphExecDestroy(h->graph);
        h->graph = nullptr;
        h->graph_steps = 0;
    }
    ftgcr_status rc = upload_debug_inst(h);
    if (rc != FTGCR_OK) return rc;
    if (chosen) *chosen = h->kc;
    return FTGCR_OK;
}

ftgcr_status ftgcr_get_tiling(const ftgcr_handle* h, int32_t* levels_per_block, int32_t* levels_per_block_dir,
                              int32_t* order_stencil, int32_t* order_dir)
{
    if (!h) return FTGCR_E_INVALID;
    if (levels_per_block) *levels_per_block = h->kc;
    if (levels_per_block_dir) *levels_per_block_dir = h->kc_dir;
    if (order_stencil) *order_stencil = h->ord_st + 1;
    if (order_dir) *order_dir = h->ord_dir + 1;
    return FTGCR_OK;
}

ftgcr_status ftgcr_autotune_batch(ftgcr_handle* const* hs, int32_t n, const double* const* rhs,
                                  double* const* x_scratch, int32_t k, int32_t steps, int32_t* chosen)
{
    if (!hs || n < 1 || !rhs || !x_scratch || steps < 1) return FTGCR_E_INVALID;
    TraceRange tr("ftgcr_autotune_batch");
    for (int m = 0; m < n; ++m)
        if (!hs[m] || !x_scratch[m]) return FTGCR_E_INVALID;
    HIP_TRY(hs[0], hipSetDevice(hs[0]->device));
    int nz_max = 1;
    for (int m = 0; m < n; ++m) nz_max = std::max(nz_max, hs[m]->geo.nz);
    std::vector<ftgcr_options> saved(n);
    for (int m = 0; m < n; ++m) saved[m] = hs[m]->opt;
    auto restore = [&]() {
        for (int m = 0; m < n; ++m) {
            hs[m]->no_resident = false;
            (void)ftgcr_set_options(hs[m], &saved[m]);
        }
    };
    for (int m = 0; m < n; ++m) {
        ftgcr_options o = saved[m];
        o.max_steps = steps;
        o.profile_kernels = 0;
        hs[m]->no_resident = true;   // the tiling of the streaming kernels is what is timed
        ftgcr_status rc = ftgcr_set_options(hs[m], &o);
        if (rc != FTGCR_OK) {
            restore();
            return rc;
        }
    }
    const std::vector<double> tol(n, 1e-300);   // never met: every member runs `steps` steps
    int best = 0;
    double best_ms = 0.0;
    const int cand[] = {2, 4, 8};
    for (int kc : cand) {
        if (kc > nz_max && kc != cand[0]) continue;
        hs[0]->opt.batch_levels_per_block = kc;
        double ms_min = 0.0;
        for (int rep = 0; rep < 2; ++rep) {
            for (int m = 0; m < n; ++m) {
                const hipError_t e = hipMemsetAsync(x_scratch[m], 0, (size_t)hs[m]->geo.n * sizeof(double),
                                                    hs[0]->stream);
                if (e != hipSuccess) {
                    restore();
                    return fail(hs[0], FTGCR_E_HIP, std::string("hipMemsetAsync: ") + hipGetErrorString(e));
                }
            }
            const auto t0 = std::chrono::steady_clock::now();
            const ftgcr_status rc = ftgcr_solve_batch(hs, n, rhs, x_scratch, tol.data(), k, nullptr, nullptr);
            const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
            if (rc != FTGCR_OK) {
                const std::string err = hs[0]->err;
                restore();
                hs[0]->err = err;
                return rc;
            }
            if (rep == 0 || ms < ms_min) ms_min = ms;
        }
        if (best == 0 || ms_min < best_ms) {
            best = kc;
            best_ms = ms_min;
        }
    }
    restore();
    hs[0]->opt.batch_levels_per_block = hs[0]->tuned_batch_kc = best;
    if (chosen) *chosen = best;
    return FTGCR_OK;
}

ftgcr_status ftgcr_kernel_times(const ftgcr_handle* h, ftgcr_kernel_time* out, int32_t cap, int32_t* n_out)
{
    if (!h || (!out && cap > 0)) return FTGCR_E_INVALID;
    const int n = 3;
    for (int q = 0; q < n && q < cap; ++q) {
        std::memset(out[q].name, 0, sizeof out[q].name);
        std::strncpy(out[q].name, kKernelNames[q], sizeof out[q].name - 1);
        out[q].launches = h->kt_n[q];
        out[q].total_ms = h->kt_ms[q];
    }
    if (n_out) *n_out = n;
    return FTGCR_OK;
}

ftgcr_status ftgcr_reset_kernel_times(ftgcr_handle* h)
{
    if (!h) return FTGCR_E_INVALID;
    for (int q = 0; q < 3; ++q) {
        h->kt_ms[q] = 0.0;
        h->kt_n[q] = 0;
    }
    return FTGCR_OK;
}

void ftgcr_destroy(ftgcr_handle* h)
{
    if (!h) return;
    for (hipEvent_t e : h->ev_pool) (void)hipEventDestroy(e);
    if (h->graph) (void)hipGraphExecDestroy(h->graph);
    if (h->cap_stream) (void)hipStreamDestroy(h->cap_stream);
    if (h->tables) (void)hipFree(h->tables);
    if (h->st) (void)hipFree(h->st);
    if (h->inst) (void)hipFree(h->inst);
    if (h->inst_dbg) (void)hipFree(h->inst_dbg);
    if (h->blk0) (void)hipFree(h->blk0);
    if (h->xw) (void)hipFree(h->xw);
    if (h->st_host) (void)hipHostFree(h->st_host);
    if (h->ev_start) (void)hipEventDestroy(h->ev_start);
    if (h->ev_stop) (void)hipEventDestroy(h->ev_stop);
    if (h->ev_idx) (void)hipFree(h->ev_idx);
    if (h->ev_bits) (void)hipFree(h->ev_bits);
    if (h->gm_st) (void)hipFree(h->gm_st);
    if (h->gm_inst) (void)hipFree(h->gm_inst);
    if (h->gm_host) (void)hipHostFree(h->gm_host);
    if (h->batch.graph) (void)hipGraphExecDestroy(h->batch.graph);
    (void)hipFree(h->batch.inst);
    (void)hipFree(h->batch.blk0);
    (void)hipFree(h->batch.status);
    (void)hipFree(h->batch.all);
    (void)hipFree(h->batch.blk0_all);
    delete h;
}

ftgcr_status ftgcr_bw_probe(const void* src_dev, void* dst_dev, size_t bytes, int32_t reps, void* hip_stream,
                            double* gbs)
{
    if (!src_dev || !dst_dev || !gbs) return fail(nullptr, FTGCR_E_INVALID, "src, dst or gbs is NULL");
    if (bytes == 0 || (bytes & 15) != 0 || reps < 1)
        return fail(nullptr, FTGCR_E_INVALID, "bytes must be a positive multiple of 16 and reps >= 1");
    if ((((uintptr_t)src_dev) | ((uintptr_t)dst_dev)) & 15)
        return fail(nullptr, FTGCR_E_INVALID, "src and dst must be 16-byte aligned");
    const uintptr_t s0 = (uintptr_t)src_dev, d0 = (uintptr_t)dst_dev;
    if (s0 < d0 + bytes && d0 < s0 + bytes) return fail(nullptr, FTGCR_E_INVALID, "src and dst overlap");
    hipStream_t s = (hipStream_t)hip_stream;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return fail(nullptr, FTGCR_E_HIP, "hipEventCreate failed");
    }
    launch_bw_copy(src_dev, dst_dev, (long long)bytes, s);   // warm-up
    hipError_t e = hipEventRecord(e0, s);
    for (int q = 0; q < reps && e == hipSuccess; ++q) launch_bw_copy(src_dev, dst_dev, (long long)bytes, s);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) return fail(nullptr, FTGCR_E_HIP, std::string("bandwidth probe: ") + hipGetErrorString(e));
    *gbs = 2.0 * (double)bytes * reps / (ms * 1e-3) / 1e9;
    return FTGCR_OK;
}

const char* ftgcr_last_error(const ftgcr_handle* h)
{
    return h ? h->err.c_str() : g_create_error.c_str();
}

ftgcr_status ftgcr_debug_apply_A(ftgcr_handle* h, const double* in_dev, double* out_dev)
{
    if (!h) return FTGCR_E_INVALID;
    if (!in_dev || !out_dev) return fail(h, FTGCR_E_INVALID, "in or out is NULL");
    HIP_TRY(h, hipSetDevice(h->device));
    Table<double> tb{h->inst_dbg, h->blk0, h->blk0 + 2, h->blk0 + 4, 1, h->geo.mesh, h->precond};
    Launch<double>::debug_apply_A(tb, h->nblk_st, h->kc, in_dev, out_dev, h->stream);
    HIP_TRY(h, hipGetLastError());
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    return FTGCR_OK;
}

ftgcr_status ftgcr_debug_resident(ftgcr_handle* h, int32_t launch, int32_t outcome)
{
    if (!h) return FTGCR_E_INVALID;
    if (launch < 0 || (launch > 0 && (outcome < FTGCR_RESIDENT_LATE || outcome > FTGCR_RESIDENT_REFUSED)))
        return fail(h, FTGCR_E_INVALID, "launch or outcome out of range");
    h->test_launch = launch;
    h->test_outcome = outcome;
    return FTGCR_OK;
}

ftgcr_status ftgcr_debug_apply_Pinv(ftgcr_handle* h, const double* in_dev, double* out_dev)
{
    if (!h) return FTGCR_E_INVALID;
    if (!in_dev || !out_dev) return fail(h, FTGCR_E_INVALID, "in or out is NULL");
    HIP_TRY(h, hipSetDevice(h->device));
    Table<double> tb{h->inst_dbg, h->blk0, h->blk0 + 2, h->blk0 + 4, 1, h->geo.mesh, h->precond};
    // the FP64 two-lane kernel, whatever the handle's own column tiling
    Launch<double>::debug_pinv(tb, (h->geo.ncols + COLS_PER_BLOCK - 1) / COLS_PER_BLOCK, h->H, in_dev, out_dev,
                               h->stream);
    HIP_TRY(h, hipGetLastError());
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    return FTGCR_OK;
}

}  // extern "C"
