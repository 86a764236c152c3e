// C-ABI host layer: argument validation, buffer layout and launch sequencing
// for the kernels in lb_kernels.hip.  See include/lb.h for the contract.
#include "lb.h"

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <new>

#include "lb_internal.h"

namespace {

thread_local char g_err[512] = "";

lb_status fail(lb_status st, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

lb_status hip_fail(hipError_t e, const char* what)
{
    return fail(LB_EHIP, "%s: %s", what, hipGetErrorString(e));
}

constexpr size_t kAlign = 256;
constexpr int kAdjComponents = 2 * LB_NVEL + 1;  // lambda_f, lambda_g, lambda_phi
constexpr int kAdjScratchComponents = 5;         // a, b_x, b_y, b_z, c
constexpr int kAdjScratchForce = 8;              // ... and dL/dF (force coupling)

// Elements per component in a time level: N rounded up to 256, plus 4352
// (4096 + 256) of padding between the f region, the g region and phi_c, so
// those streams do not start at the same offset modulo large powers of two
// (HBM channel and bank interleave; measured on MI355X with one array per
// component, 2-4% faster than 256 or none).
size_t stride_for(long long n)
{
    const size_t r = (size_t(n) + 255) / 256 * 256;
    return r + 4352;
}

bool aligned(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) % kAlign) == 0; }

// Sites a component of a time level holds: the lattice's, plus (x-slab
// shard) two halo planes on each side.
long long level_sites(const lb_params* p)
{
    return (long long)(p->nx + (p->halo_x ? 4 : 0)) * p->ny * p->nz;
}

lb_status validate(const lb_params* p)
{
    if (!p) return fail(LB_EINVAL, "params is NULL");
    if (p->nx < 1 || p->ny < 1 || p->nz < 1)
        return fail(LB_ESHAPE, "extents must be >= 1 (got %d x %d x %d)", p->nx, p->ny, p->nz);
    if (p->halo_x != 0 && p->halo_x != 1) return fail(LB_EINVAL, "halo_x must be 0 or 1");
    const long long n = level_sites(p);
    // element offsets in the kernels are 32-bit: component * stride + site with
    // up to 39 components (an adjoint level)
    if ((long long)(stride_for(n)) * 39 >= (1LL << 32))
        return fail(LB_ESHAPE, "lattice of %lld sites is too large (limit ~1.1e8 sites)", n);
    // one x-plane of the row-blocked f or g region is addressed with 32-bit
    // byte offsets (FP64: ny*nz < ~2.8e7)
    const long long elem = p->precision == LB_FP32_DEV ? 4 : 8;
    if ((long long)p->ny * p->nz * LB_NVEL * elem >= (1LL << 32))
        return fail(LB_ESHAPE, "x-plane of %lld sites is too large (ny*nz*19*%lld bytes >= 4 GiB)",
                    (long long)p->ny * p->nz, elem);
    if (!(p->tau_f > 0.5) || !(p->tau_g > 0.5))
        return fail(LB_EINVAL, "tau_f and tau_g must exceed 1/2 (got %g, %g)", p->tau_f, p->tau_g);
    if (!(p->rho0 > 0.0)) return fail(LB_EINVAL, "rho0 must be positive (got %g)", p->rho0);
    if (p->precision != LB_FP64 && p->precision != LB_FP32_DEV)
        return fail(LB_EINVAL, "unknown precision %d", p->precision);
    if (p->kernel != LB_KERNEL_FUSED && p->kernel != LB_KERNEL_TWO_PASS &&
        p->kernel != LB_KERNEL_STREAM)
        return fail(LB_EINVAL, "unknown kernel variant %d", p->kernel);
    if (p->kernel == LB_KERNEL_STREAM &&
        (p->coupling != LB_COUPLING_STRESS || p->order_param != LB_OP_LB))
        return fail(LB_EINVAL, "LB_KERNEL_STREAM is the twin of the LB_OP_LB stress-coupled step");
    if (p->layout < LB_LAYOUT_ROWS || p->layout > LB_LAYOUT_AOSOA)
        return fail(LB_EINVAL, "unknown layout %d", p->layout);
    if (p->coupling != LB_COUPLING_STRESS && p->coupling != LB_COUPLING_FORCE)
        return fail(LB_EINVAL, "unknown coupling %d", p->coupling);
    if (p->order_param != LB_OP_LB && p->order_param != LB_OP_FD)
        return fail(LB_EINVAL, "unknown order_param %d", p->order_param);
    if (p->halo_x) {
        if (p->nx < 2) return fail(LB_ESHAPE, "an x-slab shard needs nx >= 2 (got %d)", p->nx);
        if (p->order_param != LB_OP_LB || p->coupling != LB_COUPLING_STRESS ||
            (p->kernel != LB_KERNEL_FUSED && p->kernel != LB_KERNEL_STREAM))
            return fail(LB_EINVAL, "x-slab shards (halo_x) run the single-pass LB_OP_LB step "
                                   "with LB_COUPLING_STRESS only");
    }
    if (p->layout == LB_LAYOUT_AOSOA) {
        const int v = p->aosoa_len;
        if (v < 1 || (v & (v - 1)) != 0 || p->nz % v != 0)
            return fail(LB_ESHAPE, "aosoa_len %d must be a power of two dividing nz = %d", v,
                        p->nz);
    }
    return LB_OK;
}

// The kernels' view of the parameters, with every field that the tiling and the
// choice of a step's form read: the sizes that lb_query_sizes gives and the
// steps of the context that lb_create makes follow from the same one.
lbk::KParams kernel_params(const lb_params* p)
{
    lbk::KParams k{};
    k.nx = p->nx;
    k.ny = p->ny;
    k.nz = p->nz;
    k.nsites = p->nx * p->ny * p->nz;
    k.stride = unsigned(stride_for(level_sites(p)));
    lbk::set_layout(k, p->layout, p->aosoa_len);
    k.A = p->A;
    k.B = p->B;
    k.kappa = p->kappa;
    k.gamma = p->gamma;
    k.omega_f = 1.0 / p->tau_f;
    k.omega_g = 1.0 / p->tau_g;
    k.rho0 = p->rho0;
    k.force = p->coupling == LB_COUPLING_FORCE;
    k.fd = p->order_param == LB_OP_FD;
    k.mobility = p->gamma * (p->tau_g - 0.5);
    k.xh = p->halo_x ? 2 : 0;
    return k;
}

}  // namespace

struct lb_ctx {
    lb_params p;
    lb_sizes sz;
    lb_buffers b;
    hipStream_t stream;
    lbk::KParams kp;
    lbk::TileCfg tc;
    bool fp32;
    int cur;      // time level holding the current state
    int other;    // what state[1 - cur] holds: 0 a level (or nothing yet), else the
                  // form of the compact level there (kCompactSrc, kCompactF)
    bool shared;  // other contexts start from state[0] (lb_share_levels)
    int adj_cur;  // adjoint level holding the current lambda
    bool has_adj;
};

// ---- allocation-free lb_step_sums --------------------------------------
// The reduction partials of lb_step_sums_noalloc live in this array instead
// of the caller's scratch buffer: one copy per GPU the library runs on, held
// until the process ends.  On the host the name `scratch` is only a stand-in
// for the symbol, never a device address: host code takes the address of
// each GPU's copy from hipGetSymbolAddress (with that GPU current) and uses
// only that.  Every block of a reducing step writes its own five slots
// before the final pass reads them, so nothing has to start at zero.
static __device__ __align__(256) double scratch[LB_NOALLOC_MAX_PARTIALS * 5];

namespace {

static_assert(lbk::kMaxStepPartials <= LB_NOALLOC_MAX_PARTIALS, "every two-pass step fits");

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_dev[kMaxDevices] = {};

// Device address of the current GPU's copy of `scratch` (looked up once per
// device, then reused).
lb_status noalloc_scratch(lb_ctx* ctx, double** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "lb_step_sums_noalloc (hipGetDevice)");
    if (dev < 0 || dev >= kMaxDevices)
        return fail(LB_ESTATE, "lb_step_sums_noalloc: device %d is beyond the %d the library "
                               "tracks", dev, kMaxDevices);
    if (ctx->stream) {
        int sdev = -1;
        e = hipStreamGetDevice(ctx->stream, &sdev);
        if (e != hipSuccess) return hip_fail(e, "lb_step_sums_noalloc (hipStreamGetDevice)");
        if (sdev != dev)
            return fail(LB_ESTATE, "lb_step_sums_noalloc: the current device (%d) is not the "
                                   "context stream's (%d)", dev, sdev);
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "lb_step_sums_noalloc (hipGetSymbolAddress)");
        g_scratch_dev[dev] = static_cast<double*>(ptr);
    }
    *out = g_scratch_dev[dev];
    return LB_OK;
}

}  // namespace

extern "C" {

int32_t lb_abi_version(void) { return LB_ABI_VERSION; }

const char* lb_status_string(lb_status s)
{
    switch (s) {
        case LB_OK: return "ok";
        case LB_EINVAL: return "invalid argument";
        case LB_ESHAPE: return "invalid lattice shape";
        case LB_EALIGN: return "device pointer not 256-byte aligned";
        case LB_EHIP: return "HIP runtime error";
        case LB_ESTATE: return "call not valid in this state";
    }
    return "unknown status";
}

const char* lb_last_error(void) { return g_err; }

lb_status lb_query_sizes(const lb_params* p, lb_sizes* out)
{
    lb_status st = validate(p);
    if (st != LB_OK) return st;
    if (!out) return fail(LB_EINVAL, "out is NULL");
    const size_t e = p->precision == LB_FP64 ? 8 : 4;
    const lbk::KParams k = kernel_params(p);
    const size_t stride = k.stride;
    out->elem_bytes = e;
    out->stride_elems = stride;
    const bool fd = p->order_param == LB_OP_FD;
    if (fd) {
        // f, then the FP64 phi field; work fields mu, u_x, u_y, u_z
        out->state_bytes = LB_NVEL * stride * e + stride * 8;
        out->phi_bytes = 4 * stride * 8;
    } else {
        // f and g, plus the 32-bit reference order parameter in FP32 mode
        out->state_bytes = 2 * LB_NVEL * stride * e + (p->precision == LB_FP32_DEV ? stride * 4 : 0);
        // FP64 work field: phi
        out->phi_bytes = stride * 8;
    }
    // block partials of the reductions: 5 FP64 per block of the largest grid
    const bool fp32 = p->precision == LB_FP32_DEV;
    const lbk::TileCfg tc = lbk::tile_config(k, p->segment_x, fp32);
    const lbk::TileCfg rows = lbk::row_tile_config(k, p->segment_x, fp32);
    size_t nparts = std::max<size_t>(size_t(tc.ntiles) * tc.nseg, lbk::kMaxPartialBlocks);
    nparts = std::max<size_t>(nparts, size_t(rows.ntiles) * rows.nseg);
    // a two-pass step reduces over at most this many blocks
    if (!fd) nparts = std::max<size_t>(nparts, lbk::kMaxStepPartials);
    if (fd) nparts = std::max<size_t>(nparts, size_t(lbk::fd_step_partial_blocks(k, p->segment_x)));
    else if (p->coupling == LB_COUPLING_FORCE)
        nparts = std::max<size_t>(nparts, size_t(lbk::force_sums_blocks(k, p->segment_x)));
    out->scratch_bytes = nparts * 5 * 8;
    out->adj_bytes = size_t(kAdjComponents) * stride * e;
    out->face_bytes = p->halo_x ? lbk::face_bytes(k, p->precision == LB_FP32_DEV) : 0;
    out->adj_scratch_bytes =
        size_t(p->coupling == LB_COUPLING_FORCE ? kAdjScratchForce : kAdjScratchComponents) *
        stride * e;
    return LB_OK;
}

lb_status lb_create(const lb_params* p, const lb_buffers* b, void* hip_stream, lb_ctx** out)
{
    if (!out) return fail(LB_EINVAL, "out is NULL");
    *out = nullptr;
    lb_sizes sz;
    lb_status st = lb_query_sizes(p, &sz);
    if (st != LB_OK) return st;
    if (!b) return fail(LB_EINVAL, "buffers is NULL");
    const void* req[] = {b->state[0], b->state[1], b->phi, b->scratch};
    for (const void* q : req) {
        if (!q) return fail(LB_EINVAL, "state[0], state[1], phi and scratch are required");
        if (!aligned(q)) return fail(LB_EALIGN, "buffer %p is not 256-byte aligned", q);
    }
    const bool any_adj = b->adj[0] || b->adj[1] || b->adj_scratch;
    const bool all_adj = b->adj[0] && b->adj[1] && b->adj_scratch;
    if (any_adj && !all_adj)
        return fail(LB_EINVAL, "adj[0], adj[1] and adj_scratch must be given together");
    if (all_adj && (!aligned(b->adj[0]) || !aligned(b->adj[1]) || !aligned(b->adj_scratch)))
        return fail(LB_EALIGN, "adjoint buffers must be 256-byte aligned");
    if (b->state[0] == b->state[1]) return fail(LB_EINVAL, "state[0] and state[1] alias");

    lb_ctx* c = new (std::nothrow) lb_ctx;
    if (!c) return fail(LB_EINVAL, "out of host memory");
    c->p = *p;
    c->sz = sz;
    c->b = *b;
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->fp32 = p->precision == LB_FP32_DEV;
    c->cur = 0;
    c->other = 0;
    c->shared = false;
    c->adj_cur = 0;
    c->has_adj = all_adj;
    c->kp = kernel_params(p);
    c->tc = lbk::tile_config(c->kp, p->segment_x, c->fp32);
    *out = c;
    return LB_OK;
}

void lb_destroy(lb_ctx* ctx) { delete ctx; }

lb_status lb_set_stream(lb_ctx* ctx, void* hip_stream)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    ctx->stream = static_cast<hipStream_t>(hip_stream);
    return LB_OK;
}

lb_status lb_init_phi(lb_ctx* ctx, const double* phi0_dev)
{
    if (!ctx || !phi0_dev) return fail(LB_EINVAL, "ctx and phi0_dev are required");
    ctx->cur = 0;
    ctx->other = 0;
    hipError_t e = ctx->kp.fd
                       ? lbk::launch_fd_init(ctx->kp, ctx->fp32, ctx->b.state[0], phi0_dev, ctx->stream)
                       : lbk::launch_init(ctx->kp, ctx->fp32, ctx->b.state[0], phi0_dev, ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_init_phi");
}

// One step from src to dst with the context's scheme; partials (may be null)
// takes the block partials of src's conserved sums.
static hipError_t one_step(lb_ctx* ctx, const void* src, void* dst, double* partials,
                           double* phi_src_out = nullptr, int compact = 0,
                           const double* compact_src_phi = nullptr)
{
    double* work = static_cast<double*>(ctx->b.phi);
    if (ctx->kp.fd)
        return lbk::launch_fd_step(ctx->kp, ctx->tc, ctx->fp32, ctx->p.kernel, src, dst, work,
                                   partials, ctx->stream);
    return lbk::launch_step(ctx->kp, ctx->tc, ctx->fp32, ctx->p.kernel, src, dst, work, partials,
                            phi_src_out, ctx->stream, compact, compact_src_phi);
}

// The partial blocks this context's steps reduce over.
static size_t sums_blocks(const lb_ctx* ctx)
{
    return size_t(ctx->kp.fd
                      ? lbk::fd_sums_blocks(ctx->kp, ctx->tc, ctx->fp32, ctx->p.kernel)
                      : lbk::step_sums_blocks(ctx->kp, ctx->tc, ctx->fp32, ctx->p.kernel));
}

// Those of the marching kernels over row tiles: what lb_step_sums_noalloc's
// limit is stated for, whichever form of the step runs.
static size_t march_blocks(const lb_ctx* ctx)
{
    const lbk::TileCfg tc = lbk::row_tile_config(ctx->kp, ctx->p.segment_x, ctx->fp32);
    if (ctx->p.kernel == LB_KERNEL_TWO_PASS) return 0;
    if (ctx->kp.fd) return size_t(lbk::fd_march_blocks(ctx->kp, tc));
    if (ctx->kp.force) return size_t(lbk::force_sums_blocks(ctx->kp, ctx->p.segment_x));
    return size_t(tc.ntiles) * tc.nseg;
}

// part holds the block partials of `rows` blocks: the steps leave theirs one
// after the other, and one launch sums those of as many steps as fit.
static lb_status step_n(lb_ctx* ctx, int32_t nsteps, double* sums_dev, const char* name,
                        double* part = nullptr, size_t rows = 0)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    if (nsteps < 0) return fail(LB_EINVAL, "nsteps must be >= 0 (got %d)", nsteps);
    if (ctx->kp.xh && nsteps > 1)
        return fail(LB_EINVAL, "an x-slab shard advances one step per call (its halo planes "
                               "are exchanged between steps); got nsteps = %d", nsteps);
    // Levels 1 .. last between this call's steps are compact; where the buffers
    // are shared, not the last one if it stays in state[0].
    int32_t last = nsteps - 1 - (ctx->shared ? (ctx->cur + nsteps) & 1 : 0);
    if (!lbk::can_compact(ctx->kp, ctx->tc, ctx->fp32, ctx->p.kernel)) last = 0;
    const bool f_too = last > 0 && lbk::compact_f(ctx->kp, ctx->fp32, sums_dev != nullptr);
    auto from_compact = [&](int32_t t) { return t > 0 && t <= last; };
    auto to_compact = [&](int32_t t) { return t < last; };
    // partial blocks of a step between full levels, of one that collides one
    // site per thread, and of one from a level with f's moments
    size_t nb_full = 0, nb_collide = 0, nb_moments = 0;
    if (sums_dev) {
        nb_full = sums_blocks(ctx);
        if (last > 0) nb_collide = lbk::collide_grid(ctx->kp, true);
        if (f_too) nb_moments = lbk::compact_step_tiles(ctx->kp, ctx->fp32).blocks();
        const size_t most = std::max({nb_full, nb_collide, nb_moments});
        if (most > rows)
            return fail(LB_ESTATE, "%s: a step reduces over %zu partial blocks, the array holds %zu",
                        name, most, rows);
    }
    auto blocks = [&](int32_t t) {
        return from_compact(t) && f_too ? nb_moments
               : from_compact(t) || to_compact(t) ? nb_collide : nb_full;
    };
    int32_t held = 0;  // steps whose partials wait in part, nb blocks each
    size_t nb = blocks(0);
    for (int32_t t = 0; t < nsteps; t++) {
        int compact = (from_compact(t) ? lbk::kCompactSrc : 0) | (to_compact(t) ? lbk::kCompactDst : 0);
        if (compact && f_too) compact |= lbk::kCompactF;
        hipError_t e = one_step(ctx, ctx->b.state[ctx->cur], ctx->b.state[1 - ctx->cur],
                                sums_dev ? part + size_t(held) * 5 * nb : nullptr, nullptr, compact);
        if (e != hipSuccess) return hip_fail(e, name);
        ctx->cur = 1 - ctx->cur;
        ctx->other = from_compact(t) ? compact & (lbk::kCompactF | lbk::kCompactSrc) : 0;
        if (!sums_dev) continue;
        held++;
        const size_t next = blocks(t + 1);
        if (t + 1 < nsteps && next == nb && held < std::min<size_t>(rows / nb, 4096)) continue;
        e = lbk::launch_sums_final(part, int(nb), 5, held, sums_dev + 5 * size_t(t + 1 - held),
                                   ctx->stream);
        if (e != hipSuccess) return hip_fail(e, name);
        held = 0;
        nb = next;
    }
    return LB_OK;
}

lb_status lb_step(lb_ctx* ctx, int32_t nsteps) { return step_n(ctx, nsteps, nullptr, "lb_step"); }

lb_status lb_step_sums(lb_ctx* ctx, int32_t nsteps, double* sums_dev)
{
    if (!sums_dev) return fail(LB_EINVAL, "sums_dev is required");
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    return step_n(ctx, nsteps, sums_dev, "lb_step_sums", static_cast<double*>(ctx->b.scratch),
                  ctx->sz.scratch_bytes / (5 * sizeof(double)));
}

lb_status lb_step_sums_noalloc(lb_ctx* ctx, int32_t nsteps, double* sums_dev)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    if (!sums_dev) return fail(LB_EINVAL, "sums_dev is required");
    if (nsteps < 0) return fail(LB_EINVAL, "nsteps must be >= 0 (got %d)", nsteps);
    // the partial blocks this context's steps reduce over
    const size_t need = std::max(sums_blocks(ctx), march_blocks(ctx));
    if (need > size_t(LB_NOALLOC_MAX_PARTIALS))
        return fail(LB_EINVAL, "lb_step_sums_noalloc: this lattice reduces over %zu partial "
                               "blocks, the library's array holds %d (use lb_step_sums)",
                    need, LB_NOALLOC_MAX_PARTIALS);
    double* part = nullptr;
    lb_status st = noalloc_scratch(ctx, &part);
    if (st != LB_OK) return st;
    return step_n(ctx, nsteps, sums_dev, "lb_step_sums_noalloc", part, LB_NOALLOC_MAX_PARTIALS);
}

lb_status lb_step_from(lb_ctx* ctx, const void* src_dev, void* dst_dev)
{
    if (!ctx || !src_dev || !dst_dev) return fail(LB_EINVAL, "ctx, src_dev and dst_dev are required");
    if (src_dev == dst_dev) return fail(LB_EINVAL, "src_dev and dst_dev must differ");
    if (!aligned(src_dev) || !aligned(dst_dev))
        return fail(LB_EALIGN, "src_dev and dst_dev must be 256-byte aligned");
    hipError_t e = one_step(ctx, src_dev, dst_dev, nullptr);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_step_from");
}

lb_status lb_step_from_phi(lb_ctx* ctx, const void* src_dev, void* dst_dev, double* phi_dev)
{
    if (!ctx || !phi_dev) return fail(LB_EINVAL, "ctx and phi_dev are required");
    if (ctx->kp.xh) return fail(LB_ESTATE, "lb_step_from_phi is not available on a shard");
    if (ctx->kp.fd)
        return fail(LB_EINVAL, "lb_step_from_phi is for LB_OP_LB (LB_OP_FD holds phi in the "
                               "level itself)");
    if (!aligned(phi_dev)) return fail(LB_EALIGN, "phi_dev is not 256-byte aligned");
    if (!src_dev || !dst_dev) return fail(LB_EINVAL, "src_dev and dst_dev are required");
    if (src_dev == dst_dev) return fail(LB_EINVAL, "src_dev and dst_dev must differ");
    if (!aligned(src_dev) || !aligned(dst_dev))
        return fail(LB_EALIGN, "src_dev and dst_dev must be 256-byte aligned");
    hipError_t e = one_step(ctx, src_dev, dst_dev, nullptr, phi_dev);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_step_from_phi");
}

// The checks of a chain of steps through the caller's levels.
static lb_status check_chain(lb_ctx* ctx, const void* src_dev, void* const* levels_dev,
                             double* const* phis_dev, int32_t nsteps)
{
    if (!ctx || !src_dev) return fail(LB_EINVAL, "ctx and src_dev are required");
    if (nsteps < 0) return fail(LB_EINVAL, "nsteps must be >= 0 (got %d)", nsteps);
    if (nsteps > 0 && !levels_dev) return fail(LB_EINVAL, "levels_dev is required");
    if (ctx->kp.xh && nsteps > 1)
        return fail(LB_EINVAL, "an x-slab shard advances one step per call; got nsteps = %d", nsteps);
    if (!aligned(src_dev)) return fail(LB_EALIGN, "src_dev is not 256-byte aligned");
    for (int32_t t = 0; t < nsteps; t++) {
        const void* src = t ? levels_dev[t - 1] : src_dev;
        if (!levels_dev[t]) return fail(LB_EINVAL, "levels_dev[%d] is NULL", t);
        if (levels_dev[t] == src) return fail(LB_EINVAL, "levels_dev[%d] is the level it steps from", t);
        if (!aligned(levels_dev[t])) return fail(LB_EALIGN, "levels_dev[%d] is not 256-byte aligned", t);
        const double* phi = phis_dev ? phis_dev[t] : nullptr;
        if (!phi) continue;
        if (ctx->kp.xh) return fail(LB_ESTATE, "phi of a level is not available on a shard");
        if (ctx->kp.fd) return fail(LB_EINVAL, "phis_dev is for LB_OP_LB");
        if (!aligned(phi)) return fail(LB_EALIGN, "phis_dev[%d] is not 256-byte aligned", t);
    }
    return LB_OK;
}

lb_status lb_step_chain(lb_ctx* ctx, const void* src_dev, void* const* levels_dev,
                        double* const* phis_dev, int32_t nsteps)
{
    lb_status st = check_chain(ctx, src_dev, levels_dev, phis_dev, nsteps);
    if (st != LB_OK) return st;
    for (int32_t t = 0; t < nsteps; t++) {
        hipError_t e = one_step(ctx, t ? levels_dev[t - 1] : src_dev, levels_dev[t], nullptr,
                                phis_dev ? phis_dev[t] : nullptr);
        if (e != hipSuccess) return hip_fail(e, "lb_step_chain");
    }
    return LB_OK;
}

lb_status lb_step_segment(lb_ctx* ctx, const void* src_dev, void* const* levels_dev,
                          double* const* phis_dev, int32_t nsteps, int32_t last_state)
{
    lb_status st = check_chain(ctx, src_dev, levels_dev, phis_dev, nsteps);
    if (st != LB_OK) return st;
    for (int32_t t = 1; phis_dev && t < nsteps; t++)
        if (phis_dev[t] && phis_dev[t] == phis_dev[t - 1])
            return fail(LB_EINVAL, "phis_dev[%d] is that of the step before", t);
    const bool compact = lbk::can_compact(ctx->kp, ctx->tc, ctx->fp32, ctx->p.kernel);
    for (int32_t t = 0; t < nsteps; t++) {
        const int form = !compact ? 0
                                  : (t > 0 ? lbk::kCompactSrc : 0) |
                                        (t + 1 < nsteps || !last_state ? lbk::kCompactDst : 0);
        hipError_t e = one_step(ctx, t ? levels_dev[t - 1] : src_dev, levels_dev[t], nullptr,
                                phis_dev ? phis_dev[t] : nullptr, form,
                                phis_dev && t ? phis_dev[t - 1] : nullptr);
        if (e != hipSuccess) return hip_fail(e, "lb_step_segment");
    }
    return LB_OK;
}

lb_status lb_level_phi(lb_ctx* ctx, const void* level_dev, double* phi_dev)
{
    if (!ctx || !level_dev || !phi_dev) return fail(LB_EINVAL, "ctx, level_dev and phi_dev are required");
    if (ctx->kp.xh) return fail(LB_ESTATE, "lb_level_phi is not available on a shard");
    if (!aligned(level_dev) || !aligned(phi_dev))
        return fail(LB_EALIGN, "level_dev and phi_dev must be 256-byte aligned");
    hipError_t e = ctx->kp.fd
                       ? lbk::launch_fd_phi(ctx->kp, ctx->fp32, level_dev, phi_dev, ctx->stream)
                       : lbk::launch_phi(ctx->kp, ctx->fp32, level_dev, phi_dev, ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_level_phi");
}

// Moments of the current level, and with part block partials of its sums.
static hipError_t moments(lb_ctx* ctx, double* rho, double* u, double* phi, double* part, int* nb)
{
    if (ctx->kp.fd)
        return lbk::launch_fd_moments(ctx->kp, ctx->fp32, ctx->b.state[ctx->cur], rho, u, phi, part,
                                      nb, ctx->stream);
    return lbk::launch_moments(ctx->kp, ctx->fp32, ctx->b.state[ctx->cur], rho, u, phi,
                               static_cast<double*>(ctx->b.phi), part, nb, ctx->stream);
}

lb_status lb_moments(lb_ctx* ctx, double* rho_dev, double* u_dev, double* phi_dev)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    if (!rho_dev && !u_dev && !phi_dev) return LB_OK;
    int nb = 0;
    hipError_t e = moments(ctx, rho_dev, u_dev, phi_dev, nullptr, &nb);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_moments");
}

lb_status lb_sums(lb_ctx* ctx, double* out5_dev)
{
    if (!ctx || !out5_dev) return fail(LB_EINVAL, "ctx and out5_dev are required");
    int nb = 0;
    double* part = static_cast<double*>(ctx->b.scratch);
    hipError_t e = moments(ctx, nullptr, nullptr, nullptr, part, &nb);
    if (e != hipSuccess) return hip_fail(e, "lb_sums (partials)");
    e = lbk::launch_sums_final(part, nb, 5, 1, out5_dev, ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_sums (final)");
}

lb_status lb_get_state(lb_ctx* ctx, void* dst_dev)
{
    if (!ctx || !dst_dev) return fail(LB_EINVAL, "ctx and dst_dev are required");
    hipError_t e = hipMemcpyAsync(dst_dev, ctx->b.state[ctx->cur], ctx->sz.state_bytes,
                                  hipMemcpyDeviceToDevice, ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_get_state");
}

lb_status lb_set_state(lb_ctx* ctx, const void* src_dev)
{
    if (!ctx || !src_dev) return fail(LB_EINVAL, "ctx and src_dev are required");
    hipError_t e = hipMemcpyAsync(ctx->b.state[ctx->cur], src_dev, ctx->sz.state_bytes,
                                  hipMemcpyDeviceToDevice, ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_set_state");
}

lb_status lb_share_levels(lb_ctx* ctx, void* tmp_dev)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    void* level0 = ctx->b.state[0];
    if (ctx->cur == 1 && ctx->other) {
        if (!tmp_dev) return fail(LB_ESTATE, "state[0] holds no level: a buffer is needed to make one");
        if (!aligned(tmp_dev)) return fail(LB_EALIGN, "tmp_dev is not 256-byte aligned");
        if (tmp_dev == level0 || tmp_dev == ctx->b.state[1])
            return fail(LB_EINVAL, "tmp_dev is one of the context's levels");
        const bool moments = ctx->other & lbk::kCompactF;
        hipError_t e = ctx->kp.force ? lbk::launch_full_level_force(ctx->kp, ctx->fp32, moments, level0,
                                                                    tmp_dev, ctx->stream)
                                     : lbk::launch_full_level_f64(ctx->kp, moments, level0, tmp_dev,
                                                                  ctx->stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(level0, tmp_dev, ctx->sz.state_bytes, hipMemcpyDeviceToDevice,
                               ctx->stream);
        if (e != hipSuccess) return hip_fail(e, "lb_share_levels");
        ctx->other = 0;
    }
    ctx->shared = true;
    return LB_OK;
}

lb_status lb_export_dist(lb_ctx* ctx, double* f_dev, double* g_dev)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    if (ctx->kp.fd && g_dev) return fail(LB_EINVAL, "LB_OP_FD has no g: g_dev must be NULL");
    if (!f_dev && !g_dev) return LB_OK;
    hipError_t e = ctx->kp.fd ? lbk::launch_fd_export(ctx->kp, ctx->fp32, ctx->b.state[ctx->cur],
                                                      f_dev, ctx->stream)
                              : lbk::launch_export(ctx->kp, ctx->fp32, ctx->b.state[ctx->cur],
                                                   f_dev, g_dev, ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_export_dist");
}

lb_status lb_import_dist(lb_ctx* ctx, const double* f_dev, const double* g_dev)
{
    if (!ctx || !f_dev) return fail(LB_EINVAL, "ctx and f_dev are required");
    if (ctx->kp.xh)
        return fail(LB_ESTATE, "a shard cannot import post-propagation values: the populations "
                               "leaving it are its neighbours'");
    hipError_t e;
    if (ctx->kp.fd) {
        if (g_dev) return fail(LB_EINVAL, "LB_OP_FD has no g: g_dev must be NULL");
        e = lbk::launch_fd_import(ctx->kp, ctx->fp32, ctx->b.state[ctx->cur], f_dev, ctx->stream);
    } else {
        if (!g_dev) return fail(LB_EINVAL, "g_dev is required");
        e = lbk::launch_import(ctx->kp, ctx->fp32, ctx->b.state[ctx->cur], f_dev, g_dev,
                               ctx->stream);
    }
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_import_dist");
}

lb_status lb_adjoint_seed(lb_ctx* ctx, const double* dphi_dev)
{
    if (!ctx || !dphi_dev) return fail(LB_EINVAL, "ctx and dphi_dev are required");
    if (!ctx->has_adj) return fail(LB_ESTATE, "context was created without adjoint buffers");
    if (ctx->p.kernel == LB_KERNEL_STREAM)
        return fail(LB_ESTATE, "LB_KERNEL_STREAM (free streaming) has no reverse mode");
    if (ctx->kp.xh) return fail(LB_ESTATE, "x-slab shards have no reverse mode");
    ctx->adj_cur = 0;
    hipError_t e = lbk::launch_adj_seed(ctx->kp, ctx->fp32, ctx->b.adj[0], ctx->b.adj[1], dphi_dev,
                                        ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_adjoint_seed");
}

static lb_status adjoint_step(lb_ctx* ctx, const void* state_t_dev, const double* phi_t_dev,
                              double* dtheta3_dev);

lb_status lb_adjoint_step(lb_ctx* ctx, const void* state_t_dev, double* dtheta3_dev)
{
    return adjoint_step(ctx, state_t_dev, nullptr, dtheta3_dev);
}

lb_status lb_adjoint_step_phi(lb_ctx* ctx, const void* state_t_dev, const double* phi_t_dev,
                              double* dtheta3_dev)
{
    if (!ctx || !phi_t_dev) return fail(LB_EINVAL, "ctx and phi_t_dev are required");
    if (ctx->kp.fd) return fail(LB_EINVAL, "lb_adjoint_step_phi is for LB_OP_LB");
    if (!aligned(phi_t_dev)) return fail(LB_EALIGN, "phi_t_dev is not 256-byte aligned");
    return adjoint_step(ctx, state_t_dev, phi_t_dev, dtheta3_dev);
}

static lb_status adjoint_step(lb_ctx* ctx, const void* state_t_dev, const double* phi_t_dev,
                              double* dtheta3_dev)
{
    if (!ctx || !state_t_dev) return fail(LB_EINVAL, "ctx and state_t_dev are required");
    if (!ctx->has_adj) return fail(LB_ESTATE, "context was created without adjoint buffers");
    if (ctx->p.kernel == LB_KERNEL_STREAM)
        return fail(LB_ESTATE, "LB_KERNEL_STREAM (free streaming) has no reverse mode");
    if (ctx->kp.xh) return fail(LB_ESTATE, "x-slab shards have no reverse mode");
    if (!aligned(state_t_dev)) return fail(LB_EALIGN, "state_t_dev is not 256-byte aligned");
    double* part = static_cast<double*>(ctx->b.scratch);
    // FD scheme: phi is part of the level
    hipError_t e =
        ctx->kp.fd ? lbk::launch_fd_adj_step(ctx->kp, ctx->fp32, state_t_dev,
                                             static_cast<double*>(ctx->b.phi),
                                             ctx->b.adj[ctx->adj_cur], ctx->b.adj[1 - ctx->adj_cur],
                                             ctx->b.adj_scratch, part, dtheta3_dev, ctx->stream)
                   : lbk::launch_adj_step(ctx->kp, ctx->fp32, state_t_dev, phi_t_dev,
                                          static_cast<double*>(ctx->b.phi),
                                          ctx->b.adj[ctx->adj_cur], ctx->b.adj[1 - ctx->adj_cur],
                                          ctx->b.adj_scratch, part, dtheta3_dev, ctx->stream);
    if (e != hipSuccess) return hip_fail(e, "lb_adjoint_step");
    ctx->adj_cur = 1 - ctx->adj_cur;
    return LB_OK;
}

lb_status lb_adjoint_chain(lb_ctx* ctx, const void* const* levels_dev,
                           const double* const* phis_dev, int32_t nsteps, double* dtheta3_dev)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    if (nsteps < 0) return fail(LB_EINVAL, "nsteps must be >= 0 (got %d)", nsteps);
    if (nsteps > 0 && !levels_dev) return fail(LB_EINVAL, "levels_dev is required");
    for (int32_t t = 0; t < nsteps; t++) {
        if (!levels_dev[t]) return fail(LB_EINVAL, "levels_dev[%d] is NULL", t);
        if (!aligned(levels_dev[t])) return fail(LB_EALIGN, "levels_dev[%d] is not 256-byte aligned", t);
        if (!phis_dev || !phis_dev[t]) continue;
        if (ctx->kp.fd) return fail(LB_EINVAL, "phis_dev is for LB_OP_LB");
        if (!aligned(phis_dev[t])) return fail(LB_EALIGN, "phis_dev[%d] is not 256-byte aligned", t);
    }
    for (int32_t t = 0; t < nsteps; t++) {
        lb_status st = adjoint_step(ctx, levels_dev[t], phis_dev ? phis_dev[t] : nullptr, dtheta3_dev);
        if (st != LB_OK) return st;
    }
    return LB_OK;
}

lb_status lb_adjoint_phi0(lb_ctx* ctx, double* dphi0_dev)
{
    if (!ctx || !dphi0_dev) return fail(LB_EINVAL, "ctx and dphi0_dev are required");
    if (!ctx->has_adj) return fail(LB_ESTATE, "context was created without adjoint buffers");
    hipError_t e = lbk::launch_adj_phi0(ctx->kp, ctx->fp32, ctx->b.adj[ctx->adj_cur], dphi0_dev,
                                        ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_adjoint_phi0");
}

static lb_status faces(lb_ctx* ctx, void* lo, void* hi, bool pack, const char* name)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    if (!ctx->kp.xh) return fail(LB_ESTATE, "%s: the context is not an x-slab shard", name);
    if ((lo && !aligned(lo)) || (hi && !aligned(hi)))
        return fail(LB_EALIGN, "%s: face buffers must be 256-byte aligned", name);
    if (lo && lo == hi) return fail(LB_EINVAL, "%s: the two face buffers alias", name);
    hipError_t e = lbk::launch_faces(ctx->kp, ctx->fp32, ctx->b.state[ctx->cur], lo, hi, pack,
                                     ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, name);
}

lb_status lb_pack_faces(lb_ctx* ctx, void* send_lo_dev, void* send_hi_dev)
{
    return faces(ctx, send_lo_dev, send_hi_dev, true, "lb_pack_faces");
}

lb_status lb_unpack_faces(lb_ctx* ctx, const void* recv_lo_dev, const void* recv_hi_dev)
{
    return faces(ctx, const_cast<void*>(recv_lo_dev), const_cast<void*>(recv_hi_dev), false,
                 "lb_unpack_faces");
}

lb_status lb_adjoint_export(lb_ctx* ctx, double* df_dev, double* dg_dev)
{
    if (!ctx) return fail(LB_EINVAL, "ctx is NULL");
    if (!ctx->has_adj) return fail(LB_ESTATE, "context was created without adjoint buffers");
    if (ctx->kp.fd && dg_dev) return fail(LB_EINVAL, "LB_OP_FD has no g: dg_dev must be NULL");
    if ((df_dev && !aligned(df_dev)) || (dg_dev && !aligned(dg_dev)))
        return fail(LB_EALIGN, "df_dev and dg_dev must be 256-byte aligned");
    if (!df_dev && !dg_dev) return LB_OK;
    hipError_t e = lbk::launch_adj_export(ctx->kp, ctx->fp32, ctx->b.adj[ctx->adj_cur], df_dev,
                                          dg_dev, ctx->stream);
    return e == hipSuccess ? LB_OK : hip_fail(e, "lb_adjoint_export");
}

}  // extern "C"
