// Host side of the C ABI declared in include/lbm.h: contexts, parameter
// mapping, launches, diagnostics, tables, checkpoints and the tile tuner.
#include "lbm.h"
#include "lbm_contact.hpp"
#include "lbm_hostcopy.hpp"
#include "lbm_kernels.hpp"
#include "lbm_launch.hpp"
#include "lbm_params.hpp"
#include "lbm_plan.hpp"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

using namespace lbm;

struct lbm_ctx {
    int nx = 0, ny = 0, storage = 0;
    unsigned flags = 0;
    long long N = 0;
    int device = 0;
    hipStream_t stream = nullptr;
    hipStream_t own_stream = nullptr;
    void *buf[2] = {nullptr, nullptr};
    bool ext_buf = false;  // buf[] belongs to the caller (lbm_create_ex)
    int cur = 0;  // buffer holding the post-collision set of the previous step
    uint8_t *d_solid = nullptr;
    double *d_tmp = nullptr;  // staging: fields (4N doubles) or populations (18N)
    size_t tmp_bytes = 0;
    double *d_partials = nullptr;
    size_t partials_cap = 0;
    double *d_out = nullptr;  // 8 reduction results + 6 contact-angle results
    std::vector<uint8_t> solid;
    long long n_fluid = 0;
    double Gc = 0, Gw1 = 0, Gw2 = 0, delta = 0.8, tau = 1.0;
    double acc[2][2] = {{0, 0}, {0, 0}};
    double rho0[2] = {0, 0};
    double uw[2][2] = {{0, 0}, {0, 0}};  // wall velocity: rows y < ny/2, the others
    std::vector<double> inlet;           // [2][ny] inlet velocity (LBM_INLET)
    double *d_inlet = nullptr;
    // the populations were just set (init_fields, set_populations): the
    // next pull reproduces them as given, without the open or moving
    // boundary conditions
    bool fresh = false;
    bool have_geom = false, have_params = false, have_fields = false;
    long t = 0;
    lbm_host::Tile dflt = {256, 0, 0};  // the storage's default
    lbm_host::Tile tile = {256, 0, 0};  // set by lbm_set_tile, the fastest that lbm_autotune timed, or the default
    bool own_tile = false;              // steps run in `tile`, else as the library chooses
    int diag_every = 0;
    int cus = 0;
    long diag_t = -1;
    lbm_host::HostCopier copier;  // large arrays to host memory
    std::string err;
};

namespace lbm_host {

int set_err(lbm_ctx *c, int code, const char *fmt, ...)
{
    if (c) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        c->err = buf;
    }
    return code;
}

#define HIPCHK(c, call)                                                                            \
    do {                                                                                           \
        hipError_t e_ = (call);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return lbm_host::set_err((c), LBM_EDEVICE, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)

size_t elem_size(int storage) { return storage == LBM_F64 ? 8 : storage == LBM_F32 ? 4 : 2; }

bool valid_block(int b) { return b == 64 || b == 128 || b == 256; }

int ensure_tmp(lbm_ctx *c, size_t bytes)
{
    if (c->tmp_bytes >= bytes) return LBM_OK;
    if (c->d_tmp) (void)hipFree(c->d_tmp);
    c->d_tmp = nullptr;
    c->tmp_bytes = 0;
    if (hipMalloc(&c->d_tmp, bytes) != hipSuccess)
        return set_err(c, LBM_ENOMEM, "device allocation of %zu bytes failed", bytes);
    c->tmp_bytes = bytes;
    return LBM_OK;
}

int ensure_partials(lbm_ctx *c, size_t nparts)
{
    if (c->partials_cap >= nparts) return LBM_OK;
    if (c->d_partials) (void)hipFree(c->d_partials);
    c->d_partials = nullptr;
    c->partials_cap = 0;
    if (hipMalloc(&c->d_partials, nparts * 8 * sizeof(double)) != hipSuccess)
        return set_err(c, LBM_ENOMEM, "partials allocation failed");
    c->partials_cap = nparts;
    return LBM_OK;
}

bool moving_walls(const lbm_ctx *c)
{
    return c->uw[0][0] != 0.0 || c->uw[0][1] != 0.0 || c->uw[1][0] != 0.0 || c->uw[1][1] != 0.0;
}

// Open or moving boundaries are on.  Right after the populations were set
// the first step must pull them as given while the second applies the
// boundary conditions, so that step runs alone.
bool boundary_steps(const lbm_ctx *c)
{
    return (c->flags & (LBM_INLET | LBM_OUTFLOW)) || moving_walls(c);
}

template <class C>
KParams<C> make_params(const lbm_ctx *c, const void *A, void *B, const Tile &t, int halo = 2)
{
    KParams<C> p;
    std::memset(&p, 0, sizeof p);
    p.A = A;
    p.B = B;
    p.nx = c->nx;
    p.ny = c->ny;
    p.flags = c->flags;
    tile_counts(t.block, t.seg_rows, c->nx, c->ny, &p.n_strips, &p.n_segs, t.sched,
                (int)(128 / elem_size(c->storage)), &p.strip_w, halo);
    p.band_order = (t.sched & SCHED_BANDS) ? 1 : 0;
    p.xcd_slabs = 0;
    p.n_units = p.n_strips * p.n_segs;
    p.item0 = 0;
    p.tick = (unsigned)c->t;
    p.N = c->N;
    fill_physics<C>(p, c->flags, c->Gc, c->Gw1, c->Gw2, c->delta, c->tau, c->acc, c->rho0, c->storage != LBM_F64);
    for (int w = 0; w < 2; ++w)
        for (int a = 0; a < 2; ++a) p.uw[w][a] = (C)c->uw[w][a];
    p.moving = moving_walls(c) ? 1 : 0;
    p.plain = c->fresh ? 1 : 0;
    p.inlet = c->d_inlet;
    return p;
}

int grid_of(int strips, int segs) { return ((strips * segs + 7) / 8) * 8; }


int compute_units(const lbm_ctx *c) { return c->cus; }

PlanInput plan_input(const lbm_ctx *c) { return {c->nx, c->ny, c->storage, c->tau, boundary_steps(c), c->cus}; }

// The tile of the marching kernels: the caller's, or the rule of lbm_plan.hpp so
// long as the caller has set or tuned none.
Tile march_tile(const lbm_ctx *c, bool two, bool record = false)
{
    return c->own_tile ? c->tile : march_tile(plan_input(c), c->dflt, two, record);
}

// Workgroups of the step kernel that fit on the device at once.
template <int S>
int resident_capacity(lbm_ctx *c, int block)
{
    return step_occupancy<S>(block) * compute_units(c);
}

// Bricks for the steps of this lattice: the rule of lbm_plan.hpp; a tile that
// the caller has set or tuned always marches.
BrickPlan brick_plan(const lbm_ctx *c) { return c->own_tile ? BrickPlan{0, 0} : brick_plan(plan_input(c)); }

// Rows per segment of the field, diagnostic and table passes: the tile's, or
// as few as give every compute unit a workgroup where the tile leaves some idle
// (a segment is a serial march, about 3.4 us per row: 400 x 400 nodes took 34
// workgroups of 24 rows, 86 us in FP32, and take 200 of 4 rows, 26 us).
int field_rows(lbm_ctx *c)
{
    const int own = c->own_tile ? c->tile.seg_rows : c->dflt.seg_rows, rows = own > 0 ? own : 64;
    const int strips = (c->nx + 251) / 252;
    const long long fill = (long long)c->ny * strips / compute_units(c);
    return (int)std::min<long long>(rows, std::max<long long>(fill, 4));
}

// Launch one pass reading buf[cur].  P_STEP* write buf[cur^1] (the caller
// flips cur).  Returns the number of partial records in *nparts.
template <int S>
int run_pass_t(lbm_ctx *c, Pass pass, double *fields, uint8_t *link, uint8_t *nw, int32_t *src, int *nparts,
               double *partials = nullptr, int max_parts = 0)
{
    using C = typename Traits<S>::C;
    const bool two = pass == P_STEP2 || pass == P_STEP2_RED1 || pass == P_STEP2_RED2;
    const bool stepping = pass == P_STEP || pass == P_STEP_REDUCE || two;
    Tile t = march_tile(c, two, pass == P_STEP_REDUCE);
    const bool persistent = t.seg_rows == 0;
    if (persistent) t.seg_rows = 64;
    if (!stepping) t = {256, field_rows(c), c->own_tile ? c->tile.sched : c->dflt.sched};
    KParams<C> p = make_params<C>(c, c->buf[c->cur], c->buf[c->cur ^ 1], t, two ? 5 : 2);
    if ((t.sched & SCHED_XCD_SLABS) && stepping) {
        // one unit per (strip, row slab); the grid is 8 * strips so that
        // workgroup b lands on XCD b % 8 = its slab
        p.xcd_slabs = 1;
        p.band_order = 0;
        p.n_segs = 8;
        p.n_units = 8 * p.n_strips;
    } else if (persistent && stepping) {
        // persistent: one unit per resident workgroup, balanced rows per unit
        const int cap = resident_capacity<S>(c, t.block);
        const long long rows = (long long)p.n_strips * c->ny;
        p.n_units = (int)std::max(1LL, std::min((long long)cap, rows));
    }
    const int grid = ((p.n_units + 7) / 8) * 8;
    if (nparts) *nparts = grid;
    if (partials) {
        // a caller-provided partials area (no allocation)
        if (grid > max_parts)
            return set_err(c, LBM_EINVAL, "%d workgroup partials exceed the %d the scratch array holds", grid,
                           max_parts);
        p.partials = partials;
    } else if (pass == P_STEP_REDUCE || pass == P_STEP2_RED1 || pass == P_STEP2_RED2 ||
               pass == P_REDUCE) {
        int rc = ensure_partials(c, (size_t)grid);
        if (rc) return rc;
        p.partials = c->d_partials;
    }
    if (fields) {
        p.out_rho1 = fields;
        p.out_rho2 = fields + c->N;
        p.out_ux = fields + 2 * c->N;
        p.out_uy = fields + 3 * c->N;
    }
    p.tab_link = link;
    p.tab_nw = nw;
    p.tab_src = src;
    if (pass == P_TABLES) p.plain = 1;  // link bits: plain unavailability of each source
    const bool sr = (S == ST_F16 || S == ST_BF16) && (c->flags & LBM_ROUND_STOCHASTIC);
    const hipError_t e = launch_pass<S>(p, pass, t.block, sr, boundary_steps(c), c->stream, (t.sched & SCHED_REPULL) != 0);
    if (e != hipSuccess) return set_err(c, LBM_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
    return LBM_OK;
}

int run_pass(lbm_ctx *c, Pass pass, double *fields, uint8_t *link, uint8_t *nw, int32_t *src, int *nparts,
             double *partials = nullptr, int max_parts = 0)
{
    switch (c->storage) {
    case LBM_F64: return run_pass_t<ST_F64>(c, pass, fields, link, nw, src, nparts, partials, max_parts);
    case LBM_F32: return run_pass_t<ST_F32>(c, pass, fields, link, nw, src, nparts, partials, max_parts);
    case LBM_F16: return run_pass_t<ST_F16>(c, pass, fields, link, nw, src, nparts, partials, max_parts);
    default: return run_pass_t<ST_BF16>(c, pass, fields, link, nw, src, nparts, partials, max_parts);
    }
}

// Write the post-collision set whose streaming gives f(t) (from `fsrc`
// [2][9][N] FP64, or from `rho` [2][N] at rest) into buf[cur].
template <int S>
int inverse_stream_t(lbm_ctx *c, const double *fsrc, const double *rho)
{
    using C = typename Traits<S>::C;
    KParams<C> p = make_params<C>(c, nullptr, c->buf[c->cur], {256, 64, 0});
    const long long blocks = (c->N + 255) / 256;
    hipLaunchKernelGGL((k_inverse_stream<S>), dim3((unsigned)blocks), dim3(256), 0, c->stream, p, c->d_solid, fsrc, rho);
    HIPCHK(c, hipGetLastError());
    return LBM_OK;
}

int inverse_stream(lbm_ctx *c, const double *fsrc, const double *rho)
{
    switch (c->storage) {
    case LBM_F64: return inverse_stream_t<ST_F64>(c, fsrc, rho);
    case LBM_F32: return inverse_stream_t<ST_F32>(c, fsrc, rho);
    case LBM_F16: return inverse_stream_t<ST_F16>(c, fsrc, rho);
    default: return inverse_stream_t<ST_BF16>(c, fsrc, rho);
    }
}

template <int S>
int pull_window_t(lbm_ctx *c, int x0, int y0, int w, int h, double *out)
{
    using C = typename Traits<S>::C;
    KParams<C> p = make_params<C>(c, c->buf[c->cur], nullptr, {256, 64, 0});
    const long long blocks = ((long long)w * h + 255) / 256;
    hipLaunchKernelGGL((k_pull_window<S>), dim3((unsigned)blocks), dim3(256), 0, c->stream, p, x0, y0, w, h, out);
    HIPCHK(c, hipGetLastError());
    return LBM_OK;
}

int pull_window(lbm_ctx *c, int x0, int y0, int w, int h, double *out)
{
    switch (c->storage) {
    case LBM_F64: return pull_window_t<ST_F64>(c, x0, y0, w, h, out);
    case LBM_F32: return pull_window_t<ST_F32>(c, x0, y0, w, h, out);
    case LBM_F16: return pull_window_t<ST_F16>(c, x0, y0, w, h, out);
    default: return pull_window_t<ST_BF16>(c, x0, y0, w, h, out);
    }
}

// One launch of the brick kernel: `steps` steps from buf[cur] to buf[cur ^ 1].
template <int S>
int run_bricks_t(lbm_ctx *c, int region, int steps)
{
    using C = typename Traits<S>::C;
    const KParams<C> p = make_params<C>(c, c->buf[c->cur], c->buf[c->cur ^ 1], {256, 64, 0});
    const bool sr = (S == ST_F16 || S == ST_BF16) && (c->flags & LBM_ROUND_STOCHASTIC);
    const hipError_t e = launch_brick<S>(p, region, steps, sr, boundary_steps(c), c->stream);
    if (e != hipSuccess) return set_err(c, LBM_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
    return LBM_OK;
}

int run_bricks(lbm_ctx *c, int region, int steps)
{
    switch (c->storage) {
    case LBM_F64: return run_bricks_t<ST_F64>(c, region, steps);
    case LBM_F32: return run_bricks_t<ST_F32>(c, region, steps);
    case LBM_F16: return run_bricks_t<ST_F16>(c, region, steps);
    default: return run_bricks_t<ST_BF16>(c, region, steps);
    }
}

// n device arrays of `bytes` each to the caller's memory (null: skipped).
int copy_out(lbm_ctx *c, void *const *dst, const void *const *src, size_t bytes, int n)
{
    HIPCHK(c, c->copier.copy(c->device, c->stream, dst, src, bytes, n));
    return LBM_OK;
}
int copy_out(lbm_ctx *c, void *dst, const void *src, size_t bytes) { return copy_out(c, &dst, &src, bytes, 1); }

int ready(lbm_ctx *c)
{
    if (!c) return LBM_EINVAL;
    if (!c->have_geom) return set_err(c, LBM_ESTATE, "set_geometry first");
    if (!c->have_params) return set_err(c, LBM_ESTATE, "set_params first");
    if (!c->have_fields) return set_err(c, LBM_ESTATE, "init_fields or set_populations first");
    return LBM_OK;
}

int check_adhesion(lbm_ctx *c, double Gw1, double Gw2, double delta)
{
    if (!(delta > 0.0) || !std::isfinite(delta)) return set_err(c, LBM_EINVAL, "delta must be > 0");
    if (!std::isfinite(Gw1) || !std::isfinite(Gw2)) return set_err(c, LBM_EINVAL, "non-finite adhesion parameter");
    if (!(c->flags & LBM_SCHEME_ORIGINAL) && Gw1 + Gw2 == 0.0)
        return set_err(c, LBM_EINVAL, "improved scheme needs G_w1 + G_w2 != 0");
    return LBM_OK;
}

// The diagnostics alone into d_out[0..7]: no field is written (32 B per node,
// half the pass's traffic in FP32).
int reduce_only(lbm_ctx *c)
{
    int nparts = 0;
    const int rc = run_pass(c, P_REDUCE, nullptr, nullptr, nullptr, nullptr, &nparts);
    if (rc) return rc;
    hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(256), 0, c->stream, c->d_partials, nparts, c->d_out);
    HIPCHK(c, hipGetLastError());
    return LBM_OK;
}

// The fields into d_tmp (4N doubles); the diagnostics are reduce_only's.
int fields_only(lbm_ctx *c)
{
    const int rc = ensure_tmp(c, (size_t)c->N * 4 * sizeof(double));
    return rc ? rc : run_pass(c, P_FIELDS, c->d_tmp, nullptr, nullptr, nullptr, nullptr);
}

// ---------------------------------------------------------------------------
// Device scratch of the allocation-free diagnostics (lbm_reduce_noalloc):
// the workgroup partials of the reduction pass live in this file-scope
// array, one copy per device, for the life of the process.  Its host-side
// name is not a device address: kernels get the address that
// hipGetSymbolAddress returns for the current device.
// ---------------------------------------------------------------------------
constexpr int NOALLOC_MAX_PARTS = 16384;  // workgroup records of 8 doubles: 1 MiB
static __device__ __align__(256) double scratch[NOALLOC_MAX_PARTS * 8];

constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static double *g_scratch_ptr[MAX_DEVICES];

// Address of this device's scratch array (looked up once per device, with
// that device current).
int scratch_of(lbm_ctx *c, double **out)
{
    if (c->device < 0 || c->device >= MAX_DEVICES) return set_err(c, LBM_EDEVICE, "device index %d out of range", c->device);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[c->device]) {
        int cur = -1;
        HIPCHK(c, hipGetDevice(&cur));
        if (cur != c->device) HIPCHK(c, hipSetDevice(c->device));
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (cur != c->device) (void)hipSetDevice(cur);
        if (e != hipSuccess || !ptr)
            return set_err(c, LBM_EDEVICE, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
        g_scratch_ptr[c->device] = (double *)ptr;
    }
    *out = g_scratch_ptr[c->device];
    return LBM_OK;
}

// Diagnostics with no field output: sets out[5], out[6] to 0 on a lattice
// without fluid nodes (as lbm_reduce does on the host).
static __global__ void k_reduce_no_fluid(double *out)
{
    if (threadIdx.x == 0) {
        out[5] = 0.0;
        out[6] = 0.0;
    }
}

}  // namespace lbm_host

using namespace lbm_host;

extern "C" {

int lbm_reduce_noalloc(lbm_ctx *c, double *d_out)
{
    int rc = ready(c);
    if (rc) return rc;
    if (!d_out || ((uintptr_t)d_out % alignof(double)) != 0)
        return set_err(c, LBM_EINVAL, "d_out must be an aligned device pointer to 8 doubles");
    double *parts = nullptr;
    rc = scratch_of(c, &parts);
    if (rc) return rc;
    int nparts = 0;
    rc = run_pass(c, P_REDUCE, nullptr, nullptr, nullptr, nullptr, &nparts, parts, NOALLOC_MAX_PARTS);
    if (rc) return rc;
    hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(256), 0, c->stream, (const double *)parts, nparts, d_out);
    if (c->n_fluid == 0) hipLaunchKernelGGL(k_reduce_no_fluid, dim3(1), dim3(64), 0, c->stream, d_out);
    HIPCHK(c, hipGetLastError());
    return LBM_OK;
}

static int create_ctx(lbm_ctx **out, int nx, int ny, int storage, unsigned flags, void *ext_a, void *ext_b,
                      size_t ext_bytes)
{
    if (!out) return LBM_EINVAL;
    *out = nullptr;
    if (nx < 5 || ny < 5 || (long long)nx * ny > (1LL << 30)) return LBM_EINVAL;
    if (storage < LBM_F64 || storage > LBM_BF16) return LBM_EINVAL;
    if (flags & ~(unsigned)FL_ALL) return LBM_EINVAL;
    if ((flags & (LBM_INLET | LBM_OUTFLOW)) && (flags & LBM_PERIODIC_X)) return LBM_EINVAL;
    if ((flags & LBM_ROUND_STOCHASTIC) && (flags & LBM_ROUND_NEAREST)) return LBM_EINVAL;
    flags = resolve_rounding(flags, storage);
    // one component's 9 direction arrays are addressed through a 32-bit range
    if ((long long)nx * ny * 9 * (long long)elem_size(storage) >= (1LL << 32)) return LBM_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return LBM_EDEVICE;
    lbm_ctx *c = new (std::nothrow) lbm_ctx();
    if (!c) return LBM_ENOMEM;
    c->nx = nx;
    c->ny = ny;
    c->storage = storage;
    c->flags = flags;
    c->N = (long long)nx * ny;
    if (hipGetDevice(&c->device) != hipSuccess) {
        delete c;
        return LBM_EDEVICE;
    }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, c->device) != hipSuccess || std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
        delete c;
        return LBM_EDEVICE;
    }
    c->cus = prop.multiProcessorCount;
    const size_t bytes = (size_t)c->N * 18 * elem_size(storage);
    if (ext_a || ext_b) {
        // the caller's buffers: device memory of this device, distinct,
        // not overlapping, aligned and large enough
        bool good = ext_a && ext_b && ext_bytes >= bytes && ((uintptr_t)ext_a % 256) == 0 &&
                    ((uintptr_t)ext_b % 256) == 0;
        if (good) {
            uintptr_t a = (uintptr_t)ext_a, b = (uintptr_t)ext_b;
            good = a + bytes <= b || b + bytes <= a;
        }
        for (void *p : {ext_a, ext_b}) {
            hipPointerAttribute_t at;
            if (good && (hipPointerGetAttributes(&at, p) != hipSuccess || at.type != hipMemoryTypeDevice ||
                         at.device != c->device))
                good = false;
        }
        (void)hipGetLastError();  // a failed attribute query leaves no error behind
        if (!good) {
            delete c;
            return LBM_EINVAL;
        }
        c->buf[0] = ext_a;
        c->buf[1] = ext_b;
        c->ext_buf = true;
    }
    if (hipStreamCreateWithFlags(&c->own_stream, hipStreamNonBlocking) != hipSuccess) {
        delete c;
        return LBM_EDEVICE;
    }
    c->stream = c->own_stream;
    bool ok = (c->ext_buf || (hipMalloc(&c->buf[0], bytes) == hipSuccess && hipMalloc(&c->buf[1], bytes) == hipSuccess)) &&
              hipMalloc(&c->d_solid, (size_t)c->N) == hipSuccess && hipMalloc(&c->d_out, 32 * sizeof(double)) == hipSuccess &&
              hipMalloc(&c->d_inlet, (size_t)ny * 2 * sizeof(double)) == hipSuccess;
    if (!ok) {
        lbm_destroy(c);
        return LBM_ENOMEM;
    }
    c->inlet.assign((size_t)ny * 2, 0.0);
    if (hipMemcpy(c->d_inlet, c->inlet.data(), (size_t)ny * 2 * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
        lbm_destroy(c);
        return LBM_EDEVICE;
    }
    c->solid.assign((size_t)c->N, 0);
    // measured defaults on the 16384 x 2048 channel: FP32 fuses two steps
    // per launch (128-thread strips, 24-row segments in row bands); so do
    // FP16 and BF16 in 64-thread strips of 32-row segments, their packed
    // row state keeping three waves per SIMD (with stochastic rounding FP16
    // 50.5 GLUPS against 47.3 one step per launch at (256, 16), BF16 48.1
    // against 46.9; with round-to-nearest FP16 58.0 against 48.2, BF16 50.5
    // against 47.4).  FP64 fuses two steps too, in 64-thread strips of
    // 48-row segments at one wave per SIMD (20.9 GLUPS against 12.7 one
    // step per launch in 256-thread aligned strips of 16 rows), with open
    // x edges as well.
    // With open x edges the steps run in the boundary instances (FP32: 220
    // VGPRs against 195; 16-bit states unpacked), which run best in narrower
    // strips: FP32 64 threads (2.4 % over 128); BF16 and FP16 with
    // stochastic rounding one step in 128 threads (BF16 with round-to-
    // nearest: 42.8 GLUPS against 39.8 for two fused steps in 64)
    const bool open_x = (flags & (LBM_INLET | LBM_OUTFLOW)) != 0;
    const bool sr = (c->flags & LBM_ROUND_STOCHASTIC) != 0;
    const unsigned fused = SCHED_TWO_STEP | SCHED_BANDS;
    if (storage == LBM_F32) c->dflt = {open_x ? 64 : 128, 24, fused};
    else if (storage == LBM_F64) c->dflt = {64, 48, fused};
    else if (!(open_x && (sr || storage == LBM_BF16))) c->dflt = {64, 32, fused};
    else c->dflt = {128, 16, SCHED_BANDS};
    c->tile = c->dflt;
    *out = c;
    return LBM_OK;
}

int lbm_create(lbm_ctx **out, int nx, int ny, int storage, unsigned flags)
{
    return create_ctx(out, nx, ny, storage, flags, nullptr, nullptr, 0);
}

int lbm_create_ex(lbm_ctx **out, int nx, int ny, int storage, unsigned flags, void *buf_a, void *buf_b,
                  size_t bytes_each)
{
    if (!buf_a || !buf_b) {
        if (out) *out = nullptr;
        return LBM_EINVAL;
    }
    return create_ctx(out, nx, ny, storage, flags, buf_a, buf_b, bytes_each);
}

size_t lbm_population_bytes(int nx, int ny, int storage)
{
    if (nx < 5 || ny < 5 || storage < LBM_F64 || storage > LBM_BF16) return 0;
    return (size_t)nx * (size_t)ny * 18 * elem_size(storage);
}

int lbm_current_buffer(const lbm_ctx *c)
{
    if (!c) return LBM_EINVAL;
    return c->cur;
}

unsigned lbm_get_flags(const lbm_ctx *c) { return c ? c->flags : 0u; }

void lbm_destroy(lbm_ctx *c)
{
    if (!c) return;
    if (c->stream) (void)hipStreamSynchronize(c->stream);
    if (c->buf[0] && !c->ext_buf) (void)hipFree(c->buf[0]);
    if (c->buf[1] && !c->ext_buf) (void)hipFree(c->buf[1]);
    if (c->d_solid) (void)hipFree(c->d_solid);
    if (c->d_tmp) (void)hipFree(c->d_tmp);
    if (c->d_partials) (void)hipFree(c->d_partials);
    if (c->d_out) (void)hipFree(c->d_out);
    if (c->d_inlet) (void)hipFree(c->d_inlet);
    if (c->own_stream) (void)hipStreamDestroy(c->own_stream);
    delete c;
}

const char *lbm_last_error(const lbm_ctx *c) { return c ? c->err.c_str() : "null context"; }

int lbm_set_stream(lbm_ctx *c, void *hip_stream)
{
    if (!c) return LBM_EINVAL;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->stream = hip_stream ? (hipStream_t)hip_stream : c->own_stream;
    return LBM_OK;
}

int lbm_set_geometry(lbm_ctx *c, const uint8_t *solid)
{
    if (!c || !solid) return LBM_EINVAL;
    long long nf = 0;
    for (long long i = 0; i < c->N; ++i) {
        c->solid[(size_t)i] = solid[i] ? 1 : 0;
        nf += solid[i] ? 0 : 1;
    }
    HIPCHK(c, hipMemcpyAsync(c->d_solid, c->solid.data(), (size_t)c->N, hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->n_fluid = nf;
    c->have_geom = true;
    c->have_fields = false;
    return LBM_OK;
}

int lbm_set_params(lbm_ctx *c, double G_c, double G_ads, double tau)
{
    if (!c) return LBM_EINVAL;
    if (!(tau > 0.5) || !std::isfinite(tau)) return set_err(c, LBM_EINVAL, "tau must be > 0.5");
    if (!std::isfinite(G_c) || !std::isfinite(G_ads)) return set_err(c, LBM_EINVAL, "non-finite parameter");
    const double Gw2 = G_c, Gw1 = G_c + 2.0 * G_ads;
    if (!(c->flags & LBM_SCHEME_ORIGINAL) && !(Gw2 != 0.0 && Gw1 / Gw2 > 0.0))
        return set_err(c, LBM_EINVAL, "lambda = 1 + 2 G_ads / G_c must be > 0");
    int rc = check_adhesion(c, Gw1, Gw2, 0.8);
    if (rc) return rc;
    c->Gc = G_c;
    c->Gw1 = Gw1;
    c->Gw2 = Gw2;
    c->delta = 0.8;
    c->tau = tau;
    c->have_params = true;
    return LBM_OK;
}

int lbm_set_adhesion(lbm_ctx *c, double G_w1, double G_w2, double delta)
{
    if (!c) return LBM_EINVAL;
    if (!c->have_params) return set_err(c, LBM_ESTATE, "set_params first");
    int rc = check_adhesion(c, G_w1, G_w2, delta);
    if (rc) return rc;
    c->Gw1 = G_w1;
    c->Gw2 = G_w2;
    c->delta = delta;
    return LBM_OK;
}

int lbm_set_body_accel(lbm_ctx *c, double g1x, double g1y, double g2x, double g2y)
{
    if (!c) return LBM_EINVAL;
    if (!std::isfinite(g1x) || !std::isfinite(g1y) || !std::isfinite(g2x) || !std::isfinite(g2y))
        return set_err(c, LBM_EINVAL, "non-finite acceleration");
    c->acc[0][0] = g1x;
    c->acc[0][1] = g1y;
    c->acc[1][0] = g2x;
    c->acc[1][1] = g2y;
    return LBM_OK;
}

int lbm_set_wall_velocity(lbm_ctx *c, double ubx, double uby, double utx, double uty)
{
    if (!c) return LBM_EINVAL;
    if (!std::isfinite(ubx) || !std::isfinite(uby) || !std::isfinite(utx) || !std::isfinite(uty))
        return set_err(c, LBM_EINVAL, "non-finite wall velocity");
    c->uw[0][0] = ubx;
    c->uw[0][1] = uby;
    c->uw[1][0] = utx;
    c->uw[1][1] = uty;
    return LBM_OK;
}

int lbm_set_inlet_velocity(lbm_ctx *c, const double *ux, const double *uy)
{
    if (!c || !ux || !uy) return LBM_EINVAL;
    for (int y = 0; y < c->ny; ++y)
        if (!std::isfinite(ux[y]) || !std::isfinite(uy[y]) || !(ux[y] < 1.0))
            return set_err(c, LBM_EINVAL, "inlet velocity must be finite with u_x < 1");
    for (int y = 0; y < c->ny; ++y) {
        c->inlet[(size_t)y] = ux[y];
        c->inlet[(size_t)(c->ny + y)] = uy[y];
    }
    HIPCHK(c, hipStreamSynchronize(c->stream));
    HIPCHK(c, hipMemcpy(c->d_inlet, c->inlet.data(), (size_t)c->ny * 2 * sizeof(double), hipMemcpyHostToDevice));
    return LBM_OK;
}

int lbm_init_fields(lbm_ctx *c, const double *rho1, const double *rho2)
{
    if (!c || !rho1 || !rho2) return LBM_EINVAL;
    if (!c->have_geom) return set_err(c, LBM_ESTATE, "set_geometry first");
    double s[2] = {0, 0};
    for (long long i = 0; i < c->N; ++i) {
        if (c->solid[(size_t)i]) continue;
        if (!std::isfinite(rho1[i]) || !std::isfinite(rho2[i])) return set_err(c, LBM_EINVAL, "non-finite density");
        s[0] += rho1[i];
        s[1] += rho2[i];
    }
    c->rho0[0] = c->n_fluid ? s[0] / (double)c->n_fluid : 0.0;
    c->rho0[1] = c->n_fluid ? s[1] / (double)c->n_fluid : 0.0;
    int rc = ensure_tmp(c, (size_t)c->N * 2 * sizeof(double));
    if (rc) return rc;
    HIPCHK(c, hipMemcpyAsync(c->d_tmp, rho1, (size_t)c->N * sizeof(double), hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipMemcpyAsync(c->d_tmp + c->N, rho2, (size_t)c->N * sizeof(double), hipMemcpyHostToDevice, c->stream));
    const size_t bytes = (size_t)c->N * 18 * elem_size(c->storage);
    HIPCHK(c, hipMemsetAsync(c->buf[0], 0xff, bytes, c->stream));
    HIPCHK(c, hipMemsetAsync(c->buf[1], 0xff, bytes, c->stream));
    c->cur = 0;
    rc = inverse_stream(c, nullptr, c->d_tmp);
    if (rc) return rc;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->have_fields = true;
    c->fresh = true;
    c->t = 0;
    c->diag_t = -1;
    return LBM_OK;
}

int lbm_set_populations(lbm_ctx *c, const double *f)
{
    if (!c || !f) return LBM_EINVAL;
    if (!c->have_geom) return set_err(c, LBM_ESTATE, "set_geometry first");
    double s[2] = {0, 0};
    for (int k = 0; k < 2; ++k)
        for (int i = 0; i < 9; ++i)
            for (long long z = 0; z < c->N; ++z) {
                if (c->solid[(size_t)z]) continue;
                const double v = f[(size_t)(k * 9 + i) * c->N + z];
                if (!std::isfinite(v)) return set_err(c, LBM_EINVAL, "non-finite population");
                s[k] += v;
            }
    c->rho0[0] = c->n_fluid ? s[0] / (double)c->n_fluid : 0.0;
    c->rho0[1] = c->n_fluid ? s[1] / (double)c->n_fluid : 0.0;
    int rc = ensure_tmp(c, (size_t)c->N * 18 * sizeof(double));
    if (rc) return rc;
    HIPCHK(c, hipMemcpyAsync(c->d_tmp, f, (size_t)c->N * 18 * sizeof(double), hipMemcpyHostToDevice, c->stream));
    const size_t bytes = (size_t)c->N * 18 * elem_size(c->storage);
    HIPCHK(c, hipMemsetAsync(c->buf[0], 0xff, bytes, c->stream));
    HIPCHK(c, hipMemsetAsync(c->buf[1], 0xff, bytes, c->stream));
    c->cur = 0;
    rc = inverse_stream(c, c->d_tmp, nullptr);
    if (rc) return rc;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->have_fields = true;
    c->fresh = true;
    c->t = 0;
    return LBM_OK;
}

int lbm_get_populations(lbm_ctx *c, double *f)
{
    int rc = ready(c);
    if (rc) return rc;
    if (!f) return set_err(c, LBM_EINVAL, "null output");
    rc = ensure_tmp(c, (size_t)c->N * 18 * sizeof(double));
    if (rc) return rc;
    rc = pull_window(c, 0, 0, c->nx, c->ny, c->d_tmp);
    if (rc) return rc;
    return copy_out(c, f, c->d_tmp, (size_t)c->N * 18 * sizeof(double));
}

int lbm_get_populations_window(lbm_ctx *c, int x0, int y0, int w, int h, double *f)
{
    int rc = ready(c);
    if (rc) return rc;
    if (!f || w < 1 || h < 1) return set_err(c, LBM_EINVAL, "bad window");
    const bool px = c->flags & LBM_PERIODIC_X, py = c->flags & LBM_PERIODIC_Y;
    if ((!px && (x0 < 0 || (long long)x0 + w > c->nx)) || (!py && (y0 < 0 || (long long)y0 + h > c->ny)) ||
        (long long)w * h > c->N * 4)
        return set_err(c, LBM_EINVAL, "window leaves the domain");
    const size_t bytes = (size_t)w * h * 18 * sizeof(double);
    rc = ensure_tmp(c, bytes);
    if (rc) return rc;
    rc = pull_window(c, x0, y0, w, h, c->d_tmp);
    if (rc) return rc;
    return copy_out(c, f, c->d_tmp, bytes);
}

int lbm_step(lbm_ctx *c, int n)
{
    int rc = ready(c);
    if (rc) return rc;
    if (n < 0) return set_err(c, LBM_EINVAL, "negative step count");
    const BrickPlan plan = brick_plan(c);
    const bool two = (march_tile(c, true).sched & SCHED_TWO_STEP) != 0 && !plan.steps;
    for (int s = 0; s < n; ++s) {
        const bool diag_now = c->diag_every > 0 && c->t % c->diag_every == 0;
        const bool diag_next = c->diag_every > 0 && (c->t + 1) % c->diag_every == 0;
        const bool alone = c->fresh && boundary_steps(c);
        if (plan.steps && !diag_now) {
            // as many steps as the plan's bricks take, up to the next record
            long k = alone ? 1 : std::min(plan.steps, n - s);
            if (c->diag_every > 0) k = std::min(k, c->diag_every - c->t % c->diag_every);
            rc = run_bricks(c, plan.region, (int)k);
            if (rc) return rc;
            c->cur ^= 1;
            c->t += k;
            c->fresh = false;
            s += (int)k - 1;
            continue;
        }
        if (two && !alone && !(diag_now && diag_next) && n - s >= 2) {
            // two fused steps, recording the diagnostics of whichever of
            // them is due
            const Pass pass = diag_now ? P_STEP2_RED1 : diag_next ? P_STEP2_RED2 : P_STEP2;
            int nparts = 0;
            rc = run_pass(c, pass, nullptr, nullptr, nullptr, nullptr, &nparts);
            if (rc) return rc;
            if (pass != P_STEP2) {
                hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(256), 0, c->stream, c->d_partials, nparts,
                                   c->d_out + 16);
                HIPCHK(c, hipGetLastError());
                c->diag_t = diag_now ? c->t : c->t + 1;
            }
            c->cur ^= 1;
            c->t += 2;
            c->fresh = false;
            ++s;
            continue;
        }
        if (diag_now) {
            int nparts = 0;
            rc = run_pass(c, P_STEP_REDUCE, nullptr, nullptr, nullptr, nullptr, &nparts);
            if (rc) return rc;
            hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(256), 0, c->stream, c->d_partials, nparts, c->d_out + 16);
            HIPCHK(c, hipGetLastError());
            c->diag_t = c->t;
        } else {
            rc = run_pass(c, P_STEP, nullptr, nullptr, nullptr, nullptr, nullptr);
            if (rc) return rc;
        }
        c->cur ^= 1;
        c->t += 1;
        c->fresh = false;
    }
    return LBM_OK;
}

int lbm_set_diag_interval(lbm_ctx *c, int every)
{
    if (!c) return LBM_EINVAL;
    if (every < 0) return set_err(c, LBM_EINVAL, "interval must be >= 0");
    c->diag_every = every;
    return LBM_OK;
}

int lbm_get_diag(lbm_ctx *c, double out[8], long *t_diag)
{
    if (!c || !out) return LBM_EINVAL;
    if (c->diag_t < 0) return set_err(c, LBM_ESTATE, "no diagnostic record yet");
    HIPCHK(c, hipMemcpyAsync(out, c->d_out + 16, 8 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (t_diag) *t_diag = c->diag_t;
    return LBM_OK;
}

int lbm_synchronize(lbm_ctx *c)
{
    if (!c) return LBM_EINVAL;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return LBM_OK;
}

long lbm_time(const lbm_ctx *c) { return c ? c->t : -1; }

int lbm_get_fields(lbm_ctx *c, double *rho1, double *rho2, double *ux, double *uy)
{
    int rc = ready(c);
    if (rc) return rc;
    rc = fields_only(c);
    if (rc) return rc;
    void *const outs[4] = {rho1, rho2, ux, uy};
    const void *src[4];
    for (int q = 0; q < 4; ++q) src[q] = c->d_tmp + (size_t)q * c->N;
    return copy_out(c, outs, src, (size_t)c->N * sizeof(double), 4);
}

int lbm_reduce(lbm_ctx *c, double out[8])
{
    int rc = ready(c);
    if (rc) return rc;
    if (!out) return set_err(c, LBM_EINVAL, "null output");
    rc = reduce_only(c);
    if (rc) return rc;
    HIPCHK(c, hipMemcpyAsync(out, c->d_out, 8 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (c->n_fluid == 0) {
        out[5] = 0.0;
        out[6] = 0.0;
    }
    return LBM_OK;
}

int lbm_contact_angle(lbm_ctx *c, int wall_kind, const double wall[3], double *theta_deg)
{
    int rc = ready(c);
    if (rc) return rc;
    if (!wall || !theta_deg || (wall_kind != LBM_WALL_FLAT && wall_kind != LBM_WALL_CYLINDER))
        return set_err(c, LBM_EINVAL, "bad wall description");
    rc = fields_only(c);
    if (rc) return rc;
    const WallDesc wd = {wall_kind, wall[0], wall[1], wall[2]};
    const RunSet rs = {nullptr, nullptr, c->nx, c->ny, 1};
    // labels and link list in the velocity half of the field staging
    if (region_bytes(c->N, 1, 2) > (size_t)c->N * 2 * sizeof(double)) return set_err(c, LBM_ENOMEM, "no room for the labels");
    const RegionMem m = region_mem(c->d_tmp + 2 * c->N, c->N, 1, 2);
    const double *r1 = c->d_tmp, *r2 = c->d_tmp + c->N;
    const dim3 lg = link_grid(c->N, 1);
    HIPCHK(c, launch_regions(c->stream, rs, 1, c->N, r1, r2, c->d_solid, m));
    hipLaunchKernelGGL(k_cc_links, lg, dim3(256), 0, c->stream, rs, m, r1, r2, (const WallDesc *)nullptr, wd);
    hipLaunchKernelGGL(k_cc_list<2>, lg, dim3(256), 0, c->stream, rs, m);
    hipLaunchKernelGGL(k_contact_angle, dim3(1), dim3(256), 0, c->stream, rs, m, (int)lg.x, r1, r2,
                       (const WallDesc *)nullptr, wd, c->d_out + 8);
    HIPCHK(c, hipGetLastError());
    double res[6] = {0, 0, 0, 0, 0, 0};
    HIPCHK(c, hipMemcpyAsync(res, c->d_out + 8, 6 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (res[5] == 1.0) return set_err(c, LBM_EUNSTABLE, "fewer than 3 interface points");
    if (res[5] != 0.0) return set_err(c, LBM_EUNSTABLE, "circle fit failed");
    *theta_deg = res[0];
    return LBM_OK;
}

int lbm_get_tables(lbm_ctx *c, uint8_t *link, int32_t *nw_list, int32_t *nw_src, int *n_nw)
{
    if (!c) return LBM_EINVAL;
    if (!c->have_geom || !c->have_fields)
        return set_err(c, LBM_ESTATE, "tables are derived from an initialised lattice");
    const size_t N = (size_t)c->N;
    int rc = ensure_tmp(c, N * (2 + 24 * sizeof(int32_t)) + 64);
    if (rc) return rc;
    uint8_t *d_link = (uint8_t *)c->d_tmp;
    uint8_t *d_nw = d_link + N;
    int32_t *d_src = (int32_t *)(((uintptr_t)(d_nw + N) + 63) & ~(uintptr_t)63);
    HIPCHK(c, hipMemsetAsync(d_link, 0, 2 * N, c->stream));
    rc = run_pass(c, P_TABLES, nullptr, d_link, d_nw, d_src, nullptr);
    if (rc) return rc;
    std::vector<uint8_t> h_link(N), h_nw(N);
    std::vector<int32_t> h_src;
    HIPCHK(c, hipMemcpyAsync(h_link.data(), d_link, N, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipMemcpyAsync(h_nw.data(), d_nw, N, hipMemcpyDeviceToHost, c->stream));
    if (nw_list && nw_src) {
        h_src.resize(N * 24);
        HIPCHK(c, hipMemcpyAsync(h_src.data(), d_src, N * 24 * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    }
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (link) std::memcpy(link, h_link.data(), N);
    int count = 0;
    for (size_t z = 0; z < N; ++z) {
        if (!h_nw[z]) continue;
        if (nw_list) {
            nw_list[count] = (int32_t)z;
            if (nw_src) std::memcpy(nw_src + (size_t)count * 24, h_src.data() + z * 24, 24 * sizeof(int32_t));
        }
        ++count;
    }
    if (n_nw) *n_nw = count;
    return LBM_OK;
}

int lbm_set_tile(lbm_ctx *c, int block, int seg_rows, unsigned sched)
{
    if (!c) return LBM_EINVAL;
    if (!valid_block(block) || seg_rows < 0 || (sched & ~31u))
        return set_err(c, LBM_EINVAL, "block must be 64/128/256, seg_rows >= 0 (0: persistent), sched in 0..31");
    if ((sched & SCHED_REPULL) && !(sched & SCHED_TWO_STEP))
        return set_err(c, LBM_EINVAL, "LBM_SCHED_REPULL needs LBM_SCHED_TWO_STEP");
    if ((sched & SCHED_TWO_STEP) && c->storage == LBM_F64 && block == 256)
        return set_err(c, LBM_EINVAL, "two fused steps in FP64 take block 64 or 128");
    c->tile = {block, seg_rows, sched};
    c->own_tile = true;
    return LBM_OK;
}

int lbm_get_tile(const lbm_ctx *c, int *block, int *seg_rows, unsigned *sched)
{
    if (!c) return LBM_EINVAL;
    if (block) *block = c->tile.block;
    if (seg_rows) *seg_rows = c->tile.seg_rows;
    if (sched) *sched = c->tile.sched;
    return LBM_OK;
}

int lbm_autotune(lbm_ctx *c, int steps)
{
    int rc = ready(c);
    if (rc) return rc;
    if (steps < 1) return set_err(c, LBM_EINVAL, "steps must be >= 1");
    const size_t bytes = (size_t)c->N * 18 * elem_size(c->storage);
    void *backup = nullptr;
    if (hipMalloc(&backup, bytes) != hipSuccess) return set_err(c, LBM_ENOMEM, "autotune backup allocation failed");
    const int cur0 = c->cur;
    const long t0 = c->t, diag_t0 = c->diag_t;
    hipError_t e = hipMemcpyAsync(backup, c->buf[cur0], bytes, hipMemcpyDeviceToDevice, c->stream);
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (e == hipSuccess) e = hipEventCreate(&ev0);
    if (e == hipSuccess) e = hipEventCreate(&ev1);
    const bool fresh0 = c->fresh;
    const int blocks[3] = {64, 128, 256};
    const int rows[10] = {0, 8, 16, 24, 32, 48, 64, 128, 256, 512};
    const Tile cur = c->tile;
    const bool cur_own = c->own_tile;
    Tile best = cur;
    float best_ms = 1e30f, plan_ms = 1e30f;
    // candidate -2 is the library's own choice, while no tile is set; -1 is the
    // incumbent tile; the rest need a 2 % margin to win.
    // Each block x rows x schedule is tried with one step per launch and
    // with two fused steps per launch (FP64: 64- and 128-thread strips).
    const int n_two = 2;
    for (int cand = cur_own ? -1 : -2; cand < 3 * 10 * 6 * n_two && e == hipSuccess && rc == LBM_OK; ++cand) {
        int cb = cur.block, cr = cur.seg_rows;
        unsigned sc = cur.sched;
        if (cand >= 0) {
            const int tw = cand / 180, bi = (cand / 60) % 3, ri = (cand / 6) % 10;
            sc = (unsigned)(cand % 6);  // 0-3: align/bands bits; 4, 5: XCD slabs (+ align)
            if (rows[ri] > c->ny && ri > 1) continue;
            if (rows[ri] == 0 && (sc & SCHED_BANDS)) continue;  // bands need fixed segments
            if ((sc & SCHED_XCD_SLABS) && ri != 0) continue;   // slabs ignore seg_rows
            if (tw) sc |= SCHED_TWO_STEP;
            if (tw && c->storage == LBM_F64 && blocks[bi] == 256) continue;  // FP64 fuses in 64 or 128 threads
            cb = blocks[bi];
            cr = rows[ri];
        }
        c->tile = {cb, cr, sc};
        c->own_tile = cand >= -1;
        rc = lbm_step(c, 1);  // warm-up
        if (rc) break;
        e = hipEventRecord(ev0, c->stream);
        if (e != hipSuccess) break;
        rc = lbm_step(c, steps);
        if (rc) break;
        e = hipEventRecord(ev1, c->stream);
        if (e == hipSuccess) e = hipEventSynchronize(ev1);
        float ms = 0;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, ev0, ev1);
        if (e != hipSuccess) break;
        if (cand == -2) {
            plan_ms = ms;
        } else if (cand == -1 || ms < 0.98f * best_ms) {
            best_ms = ms;
            best = c->tile;
        }
    }
    if (e == hipSuccess) e = hipMemcpyAsync(c->buf[cur0], backup, bytes, hipMemcpyDeviceToDevice, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (ev0) (void)hipEventDestroy(ev0);
    if (ev1) (void)hipEventDestroy(ev1);
    (void)hipFree(backup);
    c->cur = cur0;
    c->t = t0;
    c->fresh = fresh0;
    c->diag_t = diag_t0;
    // the library's choice goes on unless a tile beats it; `tile` is the fastest
    // tile either way, to be set on a lattice like this one
    c->tile = best;
    c->own_tile = cur_own || best_ms < 0.98f * plan_ms;
    if (rc) return rc;
    if (e != hipSuccess) return set_err(c, LBM_EDEVICE, "autotune failed: %s", hipGetErrorString(e));
    return LBM_OK;
}

// Checkpoint file: header, then the raw post-collision buffer.
struct CkptHeader {
    char magic[8];
    int version, nx, ny, storage;
    unsigned flags;
    long long t;
    double Gc, Gw1, Gw2, delta, tau, acc[4], rho0[2];
};
// version 2 appends this block (and, after the populations, the inlet
// velocity [2][ny] FP64)
struct CkptBoundary {
    int fresh, pad;
    double uw[4];
};

int lbm_save(lbm_ctx *c, const char *path)
{
    int rc = ready(c);
    if (rc) return rc;
    if (!path) return set_err(c, LBM_EINVAL, "null path");
    const size_t bytes = (size_t)c->N * 18 * elem_size(c->storage);
    std::vector<char> host(bytes);
    rc = copy_out(c, host.data(), c->buf[c->cur], bytes);
    if (rc) return rc;
    CkptHeader h;
    std::memset(&h, 0, sizeof h);
    std::memcpy(h.magic, "LBM2CPK", 8);
    h.version = 2;
    h.nx = c->nx;
    h.ny = c->ny;
    h.storage = c->storage;
    h.flags = c->flags;
    h.t = c->t;
    h.Gc = c->Gc;
    h.Gw1 = c->Gw1;
    h.Gw2 = c->Gw2;
    h.delta = c->delta;
    h.tau = c->tau;
    h.acc[0] = c->acc[0][0];
    h.acc[1] = c->acc[0][1];
    h.acc[2] = c->acc[1][0];
    h.acc[3] = c->acc[1][1];
    h.rho0[0] = c->rho0[0];
    h.rho0[1] = c->rho0[1];
    CkptBoundary hb;
    std::memset(&hb, 0, sizeof hb);
    hb.fresh = c->fresh ? 1 : 0;
    hb.uw[0] = c->uw[0][0];
    hb.uw[1] = c->uw[0][1];
    hb.uw[2] = c->uw[1][0];
    hb.uw[3] = c->uw[1][1];
    FILE *fp = std::fopen(path, "wb");
    if (!fp) return set_err(c, LBM_EIO, "cannot open %s", path);
    bool ok = std::fwrite(&h, sizeof h, 1, fp) == 1 && std::fwrite(&hb, sizeof hb, 1, fp) == 1 &&
              std::fwrite(c->solid.data(), 1, (size_t)c->N, fp) == (size_t)c->N &&
              std::fwrite(host.data(), 1, bytes, fp) == bytes &&
              std::fwrite(c->inlet.data(), sizeof(double), c->inlet.size(), fp) == c->inlet.size();
    ok = (std::fclose(fp) == 0) && ok;
    if (!ok) return set_err(c, LBM_EIO, "write to %s failed", path);
    return LBM_OK;
}

int lbm_load(lbm_ctx *c, const char *path)
{
    if (!c || !path) return LBM_EINVAL;
    FILE *fp = std::fopen(path, "rb");
    if (!fp) return set_err(c, LBM_EIO, "cannot open %s", path);
    CkptHeader h;
    const size_t bytes = (size_t)c->N * 18 * elem_size(c->storage);
    std::vector<uint8_t> sol((size_t)c->N);
    std::vector<char> host(bytes);
    bool ok = std::fread(&h, sizeof h, 1, fp) == 1;
    if (ok && (std::memcmp(h.magic, "LBM2CPK", 8) != 0 || (h.version != 1 && h.version != 2) || h.nx != c->nx ||
               h.ny != c->ny || h.storage != c->storage || h.flags != c->flags)) {
        std::fclose(fp);
        return set_err(c, LBM_EINVAL, "checkpoint does not match this context");
    }
    CkptBoundary hb;
    std::memset(&hb, 0, sizeof hb);  // version 1: no open or moving boundaries
    std::vector<double> inl((size_t)c->ny * 2, 0.0);
    if (ok && h.version == 2) ok = std::fread(&hb, sizeof hb, 1, fp) == 1;
    ok = ok && std::fread(sol.data(), 1, (size_t)c->N, fp) == (size_t)c->N && std::fread(host.data(), 1, bytes, fp) == bytes;
    if (ok && h.version == 2) ok = std::fread(inl.data(), sizeof(double), inl.size(), fp) == inl.size();
    std::fclose(fp);
    if (!ok) return set_err(c, LBM_EIO, "short read from %s", path);
    int rc = lbm_set_geometry(c, sol.data());
    if (rc) return rc;
    c->Gc = h.Gc;
    c->Gw1 = h.Gw1;
    c->Gw2 = h.Gw2;
    c->delta = h.delta;
    c->tau = h.tau;
    c->acc[0][0] = h.acc[0];
    c->acc[0][1] = h.acc[1];
    c->acc[1][0] = h.acc[2];
    c->acc[1][1] = h.acc[3];
    c->rho0[0] = h.rho0[0];
    c->rho0[1] = h.rho0[1];
    c->uw[0][0] = hb.uw[0];
    c->uw[0][1] = hb.uw[1];
    c->uw[1][0] = hb.uw[2];
    c->uw[1][1] = hb.uw[3];
    c->have_params = true;
    rc = lbm_set_inlet_velocity(c, inl.data(), inl.data() + c->ny);
    if (rc) return rc;
    HIPCHK(c, hipMemcpyAsync(c->buf[0], host.data(), bytes, hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipMemsetAsync(c->buf[1], 0xff, bytes, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->cur = 0;
    c->t = (long)h.t;
    c->fresh = hb.fresh != 0;
    c->have_fields = true;
    return LBM_OK;
}

long lbm_fluid_nodes(const lbm_ctx *c) { return c ? (long)c->n_fluid : -1; }

int lbm_bytes_per_update(const lbm_ctx *c)
{
    if (!c) return LBM_EINVAL;
    return (int)(2 * 9 * 2 * elem_size(c->storage) + 1);
}

}  // extern "C"
