// Internal interface between the C-ABI host layer (lb_api.cpp) and the HIP
// kernels (lb_kernels.hip).  Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

namespace lbk {

constexpr int NV = 19;

// Kernel-side view of the parameters, passed by value.
struct KParams {
    int nx, ny, nz;
    int nsites;            // nx*ny*nz
    unsigned stride;       // elements per distribution component; every element
                           // offset in a kernel (component * stride + site, at
                           // most 39 components) fits in 32 bits
    // layout of the f and g regions: element (i, x, y, z) at
    //   x*plane_e + y*ry + (z >> vs)*zb + (z & vm) + i*cs
    unsigned plane_e, ry, zb, vs, vm, cs;
    double A, B, kappa, gamma;
    double omega_f, omega_g;  // 1/tau
    double rho0;
    int xh;     // x-slab shard: planes of halo on each side of the F and G
                // regions (2; the phi_c field has 1), x not periodic; 0: periodic
    int force;  // force coupling: -div Pi as a body force
    int fd;           // finite-difference order parameter (no g)
    double mobility;  // M = Gamma (tau_g - 1/2) of the finite-difference update
};

// Launch geometry of the single-pass step: (y, z) tiles times x segments.
struct TileCfg {
    int tz;                // tile width along z (128 or 64), or 0: flat tiles
    int nty, ntz, ntiles;  // tiles along y, along z, total
    int sx, nseg;          // planes per x segment, number of segments
    int seg_req;           // segment length asked for (<= 0: automatic)
};

// A time level's regions (LB order parameter): F and G of 19*stride
// elements of T each and, in FP32 mode, phi_c (stride 32-bit words: the high
// word of each site's reference order parameter, see lb_device.h).
template <typename T>
struct Lvl {
    T* F;
    T* G;
    unsigned* phic;  // FP32 mode only
};

template <typename T>
inline Lvl<T> level(void* state, const KParams& p, bool ref)
{
    T* base = static_cast<T*>(state);
    Lvl<T> l;
    l.F = base;
    l.G = base + size_t(NV) * p.stride;
    l.phic = ref ? reinterpret_cast<unsigned*>(base + size_t(2 * NV) * p.stride) : nullptr;
    return l;
}

// segment_x <= 0 picks the segment length automatically.  row_tile_config:
// the row tiling, whatever tile_config picks.
TileCfg tile_config(const KParams& p, int segment_x, bool fp32);
// rounds of workgroups * (planes + 2): what a tiling's march takes, in planes
long long march_cost(const TileCfg& tc);
TileCfg row_tile_config(const KParams& p, int segment_x, bool fp32);

// Fills the layout fields of k (nx, ny, nz and stride set) for an lb_layout.
void set_layout(KParams& k, int layout, int aosoa_len);

// Block size of the kernels that run one site per thread: single waves while
// they do not fill the CUs (us per FP64 two-pass step, blocks of 256 / 64:
// 16^3 7.1 / 5.8, 32^3 8.3 / 7.4, 40^3 10.5 / 10.4).
inline int site_block(const KParams& p) { return p.nsites <= 65536 ? 64 : 256; }

// Whether a step's stores of a level of ncomp components are non-temporal: a
// component's rows are whole 64-byte pieces and the level is larger than `mb`
// MiB, about what the 256 MB Infinity Cache carries over to the next step (the
// reasons and figures are at stc() in lb_step.h and FdFused in lb_fd.hip).
inline bool nt_stores(const KParams& p, int ncomp, size_t elem, int mb)
{
    return p.cs * elem % 64 == 0 && size_t(ncomp) * p.nsites * elem > (size_t(mb) << 20);
}
// Those of a march: also on the smallest lattices it runs on, where a
// workgroup's next plane waits behind its stores (us per 100 steps, non-temporal
// / plain: FD FP32 48^3 1124 / 1230, FP64 40^3 1152 / 1213, LB FP32 40^3 1041 /
// 1101).
inline bool march_nt(const KParams& p, int ncomp, int elem, int mb)
{
    return p.nsites <= 120000 || nt_stores(p, ncomp, elem, mb);
}

// All launchers enqueue on `s` and return hipGetLastError().
// `fp32` selects the FP32 deviation-storage instantiation; otherwise FP64.
// A time level (`state`) is an F region and a G region of 19*stride elements
// each (laid out per KParams) and, in FP32 mode, phi_c[stride] (32-bit
// words, site order).  Order-parameter fields (`phi`) are FP64.
hipError_t launch_init(const KParams& p, bool fp32, void* state, const double* phi0, hipStream_t s);
// variant 0: single-pass fused step (or what step_variant picks for it);
// 1: phi pass (phi into phi_work, and in FP32 mode the new level's phi_c) +
// collision pass; 2: the single pass's memory-only twin.
// If partials is non-null, the step also leaves the block partials of the 5
// FP64 conserved sums [rho, phi, jx, jy, jz] of the source level there
// (step_sums_blocks blocks of 5), for launch_sums_final.
// phi_src_out (may be null): also store phi of src there (N FP64 values in
// site order, bit-identical to launch_phi's).
// Boxes of the smallest lattices' step (variant kStepBox).
constexpr int kBox = 4, kStepBox = 3;
struct BoxCfg {
    int nbx, nby, nbz;
    int blocks() const { return nbx * nby * nbz; }
};
inline BoxCfg box_cfg(const KParams& p)
{
    return {(p.nx + kBox - 1) / kBox, (p.ny + kBox - 1) / kBox, (p.nz + kBox - 1) / kBox};
}
// The kernels a step of `variant` runs, with or without sums.
int step_variant(const KParams& p, const TileCfg& tc, bool fp32, int variant, bool sums);
// The number of partial blocks the LB-scheme step of `variant` reduces over.
int step_sums_blocks(const KParams& p, const TileCfg& tc, bool fp32, int variant);
hipError_t launch_step(const KParams& p, const TileCfg& tc, bool fp32, int variant,
                       const void* src, void* dst, double* phi_work, double* partials,
                       double* phi_src_out, hipStream_t s, int compact = 0,
                       const double* compact_src_phi = nullptr);
// Whether a step of `variant` can start from or leave a compact level
// (lb_compact.h); launch_step's `compact`: kCompactSrc if src is compact (its
// phi in compact_src_phi if that is given: the phi_src_out of the step that
// made it), kCompactDst if dst is to be.
// kCompactF: those compact levels hold f's moments, too (compact_f).
constexpr int kCompactSrc = 1, kCompactDst = 2, kCompactF = 4;
bool compact_f(const KParams& p, bool fp32, bool sums);
bool can_compact(const KParams& p, const TileCfg& tc, bool fp32, int variant);
hipError_t launch_phi_compact_f64(const KParams& p, const void* state, const double* cphi,
                                  double* phi, hipStream_t s);
hipError_t launch_phi_compact_force(const KParams& p, bool fp32, const void* state,
                                    const double* cphi, double* phi, void* next, hipStream_t s);
// The march's tile: 12 x 32 sites and their ring are 8 waves of cells, two
// workgroups of which fill a CU's LDS in FP64 (us per step of 256^3 FP64, the
// collision's 1073 included: 8 x 64 1312, 8 x 48 1310, 4 x 64 1323, 16 x 32
// 1335, 12 x 32 1312; of 151 x 105 x 150 207, 203, 210, 208, 199).
constexpr int kCompactTY = 12, kCompactTZ = 32;
constexpr int kCompactThreads = ((kCompactTY + 2) * (kCompactTZ + 2) + 63) / 64 * 64;
constexpr int kCompactResident = 2 * 256;


// The march's tiles along y and z, and its segments of sx planes.
struct CompactTiles {
    int nty, ntz, sx, nseg;
    int blocks() const { return nty * ntz * nseg; }
};
CompactTiles compact_tiles(const KParams& p, int resident);
// Those of the collision pass.
CompactTiles compact_step_tiles(const KParams& p, bool fp32);
// Whether the phi pass from a compact level marches.
bool compact_march(const KParams& p, bool fp32);
hipError_t launch_step_compact_f64(const KParams& p, const void* src, void* dst, bool to_full,
                                   const double* phi, double* partials, hipStream_t s);
hipError_t launch_step_compact_force(const KParams& p, bool fp32, const void* src, void* dst,
                                     bool to_full, const double* phi, double* partials,
                                     hipStream_t s);
// The full level `dst` of the compact level `src` (moments: with f's moments).
hipError_t launch_full_level_f64(const KParams& p, bool moments, const void* src, void* dst,
                                 hipStream_t s);
hipError_t launch_full_level_force(const KParams& p, bool fp32, bool moments, const void* src,
                                   void* dst, hipStream_t s);
// launch_step's kernels of the stress coupling, by storage precision; phi64
// is the field that variant 1's phi pass left.  launch_phi_*: phi of `state`,
// and if `next` is not null the phi_c of that level (FP32 mode).
hipError_t launch_step_f32(const KParams& p, const TileCfg& tc, int variant, int compact,
                           const void* src, void* dst, double* phi64, double* partials,
                           double* phi_src_out, hipStream_t s);
hipError_t launch_step_f64(const KParams& p, const TileCfg& tc, int variant, int compact,
                           const void* src, void* dst, double* phi64, double* partials,
                           double* phi_src_out, hipStream_t s);
hipError_t launch_phi_f32(const KParams& p, const void* state, double* phi, void* next,
                          hipStream_t s);
hipError_t launch_phi_f64(const KParams& p, const void* state, double* phi, void* next,
                          hipStream_t s);
// Force coupling: the forcing collision from src to dst.  variant 0: the
// whole step in one pass over (y, z) tiles marching along x (its own 8 x 64
// tiling, segments as tc.seg_req asks), phi summed from the pulled g, Pi in
// LDS; phi of src goes to dst's phi_c field (FP32 mode) and to `phi` if not
// null; with `partials`, the pass also leaves block partials of
// [rho, phi, j + F/2] of src there (force_sums_blocks(p, tc.seg_req) blocks
// of 5).  variant 1: after the phi pass, which left phi (all sites, FP64) of
// src in `phi` and dst's phi_c, one site per thread, Pi formed at each face
// neighbour (partials: collide_grid(p, true) blocks of site_block(p) threads).
// kStepBox: boxes, FP32 storage only.  Bit-identical levels.
hipError_t launch_force_collide(const KParams& p, const TileCfg& tc, bool fp32, int variant,
                                int compact, const void* src, void* dst, double* phi, double* partials,
                                hipStream_t s);
int force_sums_blocks(const KParams& p, int seg_req);
// phi(x) of the post-propagation state held in `state`.
hipError_t launch_phi(const KParams& p, bool fp32, const void* state, double* phi, hipStream_t s);
// Moments of the level (outputs may be null) and, if partials is not null, the
// block partials of its sums, *nblocks_out (at most kMaxPartialBlocks) of 5.
// work: the FP64 phi field the force coupling needs (`stride` long); unused
// otherwise.
hipError_t launch_moments(const KParams& p, bool fp32, const void* state, double* rho, double* u,
                          double* phi, double* work, double* partials, int* nblocks_out,
                          hipStream_t s);
// out[b*ncomp + k] = the sum of component k < ncomp over the nblocks block
// partials of set b < nsets (sets follow one another in `partials`).
hipError_t launch_sums_final(const double* partials, int nblocks, int ncomp, int nsets,
                             double* out, hipStream_t s);
hipError_t launch_export(const KParams& p, bool fp32, const void* state, double* f, double* g,
                         hipStream_t s);
hipError_t launch_import(const KParams& p, bool fp32, void* state, const double* f,
                         const double* g, hipStream_t s);

// Reverse mode.
// Workgroups of the sweeping adjoint kernels: at most 1024 of site_block(p)
// threads, each thread looping over its sites (a few resident rounds at the
// local kernels' 1-3 waves per SIMD; a grid of exactly one round measured no
// faster); the parameter reduction (in the stencil kernel's first workgroups)
// then reads half the partials of 2048 workgroups (measured as a launch of its
// own at 128^3: 9.9 -> 5.5 us, k_adj_local unchanged).
constexpr int kAdjBlocks = 1024;
inline int adj_blocks(const KParams& p)
{
    const int nt = site_block(p), g = (p.nsites + nt - 1) / nt;
    return g < kAdjBlocks ? g : kAdjBlocks;
}
// adj: the level seeded (lf = lg = 0, lp = dphi); other: the second level,
// whose lg is zeroed too when tau_g = 1 (the steps then never touch lg).
hipError_t launch_adj_seed(const KParams& p, bool fp32, void* adj, void* other, const double* dphi,
                           hipStream_t s);
// dtheta (may be null): FP64[3] incremented by the step's d/d(A, B, kappa),
// reduced from block partials in `partials` (3 * 1024 doubles; 6 * 1024
// with the force coupling).  The force coupling needs 8 components of
// adj_scratch (the stencil cotangents, then dL/dF).
// phi_given (may be null): phi of `state` (N FP64 values in site order), so
// that no phi pass is needed.
hipError_t launch_adj_step(const KParams& p, bool fp32, const void* state,
                           const double* phi_given, double* phi,
                           const void* adj_next, void* adj_prev, void* adj_scratch,
                           double* partials, double* dtheta, hipStream_t s);
// lp of adj_prev from the stencil cotangents in adj_scratch (a, b_x, b_y,
// b_z, c): lp = a - sum_a D_a b_a + lap c; with dtheta, also
// dtheta[k] += the sum of the nparts block partials of component k < 3 in
// `partials` and, if not null, in `partials2`.
hipError_t launch_adj_stencil(const KParams& p, bool fp32, const void* adj_scratch,
                              void* adj_prev, const double* partials, const double* partials2,
                              int nparts, double* dtheta, hipStream_t s);
// Force coupling: dL/dF (adj_scratch components 5..7) through Pi at the face
// neighbours into the stencil cotangents (components 0..4) of the FP64 phi
// field `phi`; nblocks workgroups, their partials of d/d(A, B, kappa) in
// partials2 (3 * nblocks).
hipError_t launch_adj_force_pi(const KParams& p, bool fp32, const double* phi, void* adj_scratch,
                               double* partials2, int nblocks, hipStream_t s);
// dL/dphi0 from the level in `adj` (LB scheme: lg_0 + lp; FD scheme: lp).
hipError_t launch_adj_phi0(const KParams& p, bool fp32, const void* adj, double* dphi0,
                           hipStream_t s);
// Dense FP64 (19, nx, ny, nz) copies of the level in `adj`: df = lf and
// (LB scheme; null for FD) dg = lg + lp.  Either pointer may be null.
hipError_t launch_adj_export(const KParams& p, bool fp32, const void* adj, double* df, double* dg,
                             hipStream_t s);

// Finite-difference order parameter (lb_fd.hip).  A time level is F
// (19*stride elements, laid out per KParams) then phi (stride FP64 values).
// variant 0: single-pass step with the tiling of tc; 1: collision pass, then
// update pass, with `work` holding mu, u_x, u_y, u_z (4 fields of `stride`:
// FP64, or FP32 with the force coupling in FP32 storage; 4 FP64 fields of
// space).  With `partials` the step also leaves the block partials of the
// source level's sums there: 5 * fd_sums_blocks doubles, the number of blocks
// of `variant` (at most max(tc.ntiles * tc.nseg, fd_step_partial_blocks)).
int fd_step_partial_blocks(const KParams& p, int segment_x);
int fd_sums_blocks(const KParams& p, const TileCfg& tc, bool fp32, int variant);
// ... and that of its marching pass.
int fd_march_blocks(const KParams& p, const TileCfg& tc);
hipError_t launch_fd_init(const KParams& p, bool fp32, void* state, const double* phi0,
                          hipStream_t s);
hipError_t launch_fd_step(const KParams& p, const TileCfg& tc, bool fp32, int variant,
                          const void* src, void* dst, double* work, double* partials,
                          hipStream_t s);
// Reverse mode of one FD step (stress coupling): adj_prev = J(state)^T adj_next
// in the adjoint-level layout (lf[19], unused g components, lp), with
// `work` (4 FP64 fields of space) taking rho and u of `state`, adj_scratch
// the five stencil cotangents, and dtheta as for launch_adj_step.
hipError_t launch_fd_adj_step(const KParams& p, bool fp32, const void* state, double* work,
                              const void* adj_next, void* adj_prev, void* adj_scratch,
                              double* partials, double* dtheta, hipStream_t s);
// phi of the level `state` (a copy of its phi field)
hipError_t launch_fd_phi(const KParams& p, bool fp32, const void* state, double* phi, hipStream_t s);
hipError_t launch_fd_moments(const KParams& p, bool fp32, const void* state, double* rho,
                             double* u, double* phi, double* partials, int* nblocks_out,
                             hipStream_t s);
hipError_t launch_fd_export(const KParams& p, bool fp32, const void* state, double* f,
                            hipStream_t s);
hipError_t launch_fd_import(const KParams& p, bool fp32, void* state, const double* f,
                            hipStream_t s);

// x-slab shards (lb_halo.hip): bytes of one face buffer, and the copy of the
// faces between the buffers `lo` and `hi` (either may be null) and the level
// `state` -- pack: the boundary planes and the planes behind them into the
// buffers for the lower and the upper neighbour; unpack: theirs into the halo
// planes.
size_t face_bytes(const KParams& p, bool fp32);
hipError_t launch_faces(const KParams& p, bool fp32, void* state, void* lo, void* hi, bool pack,
                        hipStream_t st);

// Upper bounds on the block partials (per component) of a moments or adjoint
// reduction, and of an LB step that reduces in its two-pass collision.
constexpr int kMaxPartialBlocks = 2048;
constexpr int kMaxStepPartials = 4096;

// Workgroups of the two-pass step's collision kernel, one site per thread;
// with sums at most kMaxStepPartials, which then sweep the sites.
inline int collide_grid(const KParams& p, bool sums)
{
    const int g = (p.nsites + site_block(p) - 1) / site_block(p);
    return sums && g > kMaxStepPartials ? kMaxStepPartials : g;
}

}  // namespace lbk
