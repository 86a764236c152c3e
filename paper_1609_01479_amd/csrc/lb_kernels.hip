// Forward kernels (gfx950) of the D3Q19 symmetric binary-fluid LB step.
//
// Here: the initial state, moments and sums, dense import and export, and
// the launches of a step -- which form of it runs (step_variant) and its
// tiling.  The step's own kernels are in lb_step.h (the stress coupling),
// lb_force.hip (the force coupling) and lb_fd.hip (the finite-difference
// order parameter).
#include <algorithm>

#include "lb_compact.h"
#include "lb_device.h"
#include "lb_sweep.h"

namespace lbk {

using namespace dev;

namespace {

// Post-propagation state rho = rho0, u = 0, g_0 = phi0, g_{i>0} = 0.  In FP32
// mode phi_c is phi0's reference, and the stored deviation of direction i at
// y is g_i(y + c_i) - r_i phi_c(y + c_i).  In an x-slab shard phi0 also holds
// the planes -1 and nx (the neighbours'), first and last.
template <typename T, bool DEV, bool REF>
__global__ __launch_bounds__(kBlock) void k_init(KParams p, T* __restrict__ F, T* __restrict__ G,
                                                 unsigned* __restrict__ phic,
                                                 const double* __restrict__ phi0)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= p.nsites) return;
    const Geo q = geo_of(p, s);
    const double* ph = phi0 + (p.xh ? p.ny * p.nz : 0);
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const unsigned d = dist_own(p, q, i);
        F[d] = DEV ? T(0) : T(weight(i) * p.rho0);
        if (REF) {
            const double pd = ph[push_site(p, q, i)];
            G[d] = T((i == 0 ? pd : 0.0) - rweight(i) * phic_round(pd));
        } else {
            G[d] = i == 0 ? T(ph[s]) : T(0);
        }
    }
    if (REF) phic[phic_site(p, q.x, q.y, q.z)] = phic_word(ph[s]);
}

// Dense FP64 moments of the post-propagation state and, if partials is not
// null, block partials of [rho, phi, jx, jy, jz] (FP64 accumulation; the
// sites of each XCD a contiguous eighth, so the rows and planes that its
// pulls share are in its L2).
// With fphi (force coupling: phi of this state, all sites) phi comes from
// there, without a second pull of g, the velocity is (j + F/2)/rho,
// F = -div Pi of this state, and the momentum sums are those of j + F/2.
// Bound by memory: one read of the level, one write of what is asked for.
// Without partials no block reduces them, and the grid is not cut to their
// number; phi alone reads g alone (launch_moments).  Force coupling at 192^3
// FP64: rho, u and phi 732 -> 505 us, the sums 632 -> 463, phi 712 -> 209;
// stress 470 -> 475 (5.1 TB/s), 361 -> 359, 386 -> 207.
template <typename T, bool DEV, bool REF, int NB>
__global__ __launch_bounds__(NB) void k_moments(KParams p, const T* __restrict__ F,
                                                const T* __restrict__ G,
                                                const unsigned* __restrict__ phic,
                                                const double* __restrict__ fphi,
                                                double* __restrict__ rho_out,
                                                double* __restrict__ u_out,
                                                double* __restrict__ phi_out,
                                                double* __restrict__ partials)
{
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (XcdSweep w = xcd_sweep(p.nsites, NB); w.s < w.end; w.s += w.stride) {
        const int s = w.s;
        const Geo q = geo_of(p, s);
        double fv[NV];
#pragma unroll
        for (int i = 0; i < NV; i++) fv[i] = double(F[dist_pull(p, q, i)]);
        const double ph = fphi ? fphi[s] : phi_at<T, REF>(p, q, G, phic);
        double b = 0.0;
#pragma unroll
        for (int i = 0; i < NV; i++) b += fv[i];
        const double rho = DEV ? p.rho0 + b : b;
        double jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
        for (int i = 0; i < NV; i++) {
            jx += CX[i] * fv[i];
            jy += CY[i] * fv[i];
            jz += CZ[i] * fv[i];
        }
        if (fphi) {
            double fo[3];
            force_from_phi(p, q, fphi, fo);
            jx += 0.5 * fo[0];
            jy += 0.5 * fo[1];
            jz += 0.5 * fo[2];
        }
        if (rho_out) rho_out[s] = rho;
        if (u_out) {
            u_out[s] = jx / rho;
            u_out[p.nsites + s] = jy / rho;
            u_out[2LL * p.nsites + s] = jz / rho;
        }
        if (phi_out) phi_out[s] = ph;
        acc[0] += rho;
        acc[1] += ph;
        acc[2] += jx;
        acc[3] += jy;
        acc[4] += jz;
    }
    if (partials) block_partials<5, NB>(acc, partials);
}

// Workgroup (k, b): out[b*ncomp + k] = the sum over nblocks partials of
// component k of the b-th set of partials.  Latency: one workgroup per sum,
// each thread's loads in flight together (one workgroup for the five sums,
// loading one after the other, took some 15 us over 2637 blocks).
__global__ __launch_bounds__(kBlock) void k_sums_final(const double* __restrict__ partials,
                                                       int nblocks, double* __restrict__ out)
{
    const int ncomp = gridDim.x;
    const size_t k = size_t(blockIdx.y) * ncomp + blockIdx.x;
    reduce_partials_block(partials + k * nblocks, nblocks, 1, out + k, false);
}

template <typename T, bool DEV, bool REF>
__global__ __launch_bounds__(kBlock) void k_export(KParams p, const T* __restrict__ F,
                                                   const T* __restrict__ G,
                                                   const unsigned* __restrict__ phic,
                                                   double* __restrict__ f, double* __restrict__ g)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= p.nsites) return;
    const Geo q = geo_of(p, s);
    if (f)
#pragma unroll
        for (int i = 0; i < NV; i++)
            f[(long long)i * p.nsites + s] =
                double(F[dist_pull(p, q, i)]) + (DEV ? weight(i) * p.rho0 : 0.0);
    if (g) {
        double d[NV];
        pull_g<T, REF>(p, q, G, phic, d);
#pragma unroll
        for (int i = 0; i < NV; i++) g[(long long)i * p.nsites + s] = d[i];
    }
}

// FP32 mode, first half of an import: the reference phi_c(x) of
// phi(x) = sum_i g_i(x) of the dense post-propagation input.
__global__ __launch_bounds__(kBlock) void k_import_ref(KParams p, unsigned* __restrict__ phic,
                                                       const double* __restrict__ g)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= p.nsites) return;
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < NV; i++) acc += g[(long long)i * p.nsites + s];
    phic[s] = phic_word(acc);
}

// The stored value of direction i at y is the post-propagation value at
// y + c_i (FP32 mode: minus w_i rho0 for f, minus r_i phi_c(y + c_i) for g).
template <typename T, bool DEV, bool REF>
__global__ __launch_bounds__(kBlock) void k_import(KParams p, T* __restrict__ F, T* __restrict__ G,
                                                   const unsigned* __restrict__ phic,
                                                   const double* __restrict__ f,
                                                   const double* __restrict__ g)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= p.nsites) return;
    const Geo q = geo_of(p, s);
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int d = push_site(p, q, i);
        const long long n = d + (long long)i * p.nsites;
        F[dist_own(p, q, i)] = T(f[n] - (DEV ? weight(i) * p.rho0 : 0.0));
        G[dist_own(p, q, i)] = T(REF ? g[n] - rweight(i) * phic_value(phic[d]) : g[n]);
    }
}

int grid_for(const KParams& p) { return (p.nsites + kBlock - 1) / kBlock; }

// workgroups of a moments pass, with sums at most kMaxPartialBlocks
int moments_grid(const KParams& p, bool sums)
{
    const int g = (p.nsites + site_block(p) - 1) / site_block(p);
    return sums && g > kMaxPartialBlocks ? kMaxPartialBlocks : g;
}

template <typename T>
void moments(const KParams& p, int nb, const void* state, const double* fphi, double* rho,
             double* u, double* phi, double* partials, hipStream_t s)
{
    constexpr bool F32 = sizeof(T) == 4;
    Lvl<T> a = level<T>(const_cast<void*>(state), p, F32);
    const int nt = site_block(p);
    auto k = nt == 64 ? k_moments<T, F32, F32, 64> : k_moments<T, F32, F32, kBlock>;
    k<<<nb, nt, 0, s>>>(p, a.F, a.G, a.phic, fphi, rho, u, phi, partials);
}


// Instantiation dispatch: FP64 mode <double, false, false>, FP32 mode <float, true, true>.
#define LB_DISPATCH(fp32, CALL64, CALL32) \
    do {                                  \
        if (fp32) {                       \
            using T = float;              \
            constexpr bool DEV = true;    \
            constexpr bool REF = true;    \
            (void)DEV;                    \
            CALL32;                       \
        } else {                          \
            using T = double;             \
            constexpr bool DEV = false;   \
            constexpr bool REF = false;   \
            (void)DEV;                    \
            CALL64;                       \
        }                                 \
    } while (0)

}  // namespace

void set_layout(KParams& k, int layout, int aosoa_len)
{
    const unsigned ny = unsigned(k.ny), nz = unsigned(k.nz), nv = unsigned(NV);
    k.vs = 31;  // z >> 31 == 0: no z-blocks
    k.vm = 0xffffffffu;
    k.zb = 0;
    k.plane_e = ny * nz * nv;
    k.ry = nz * nv;
    switch (layout) {
    case 1:  // one array per component
        k.plane_e = ny * nz;
        k.ry = nz;
        k.cs = k.stride;
        break;
    case 2:  // a site's components together
        k.vs = 0;
        k.vm = 0;
        k.zb = nv;
        k.cs = 1;
        break;
    case 3: {  // blocks of V z-sites
        unsigned v = unsigned(aosoa_len), sh = 0;
        while ((1u << sh) < v) sh++;
        k.vs = sh;
        k.vm = v - 1;
        k.zb = nv * v;
        k.cs = v;
        break;
    }
    default:  // row-blocked
        k.cs = nz;
        break;
    }
}

// Number of CUs of an MI355X: with 512-thread workgroups at 2 waves per SIMD,
// one workgroup per CU runs at a time.
constexpr int kCUs = 256;
constexpr int kFused = 512;  // columns of a marching kernel's tile

// Whether the LB step can march over flat tiles (lb_step.h): a plane of at
// least one tile, and a halo of at most one cell per thread -- nz sites before
// and after a tile of whole rows, and in FP32 mode 4 more for any other.
static bool flat_fits(const KParams& p, bool fp32)
{
    if (p.fd || (long long)p.ny * p.nz < kFused) return false;
    return 2 * p.nz + (fp32 && kFused % p.nz ? 4 : 0) <= kFused;
}

long long march_cost(const TileCfg& tc)
{
    return (long long)((tc.ntiles * (long long)tc.nseg + kCUs - 1) / kCUs) * (tc.sx + 2);
}

// Segments of a tiling; the automatic length keeps it within max_blocks
// workgroups (0: any number; one segment always counts as within).
static TileCfg with_segments(const KParams& p, TileCfg tc, int segment_x, long long max_blocks = 0)
{
    tc.ntiles = tc.nty * tc.ntz;
    int sx = segment_x;
    if (sx <= 0) {
        // Segments along x: a workgroup marches sx planes after 2 warm-up
        // planes, and workgroups run in rounds of kCUs.  Pick the segment
        // count minimising rounds * (sx + 2) (fewest workgroups on ties);
        // this fits measured times at 128^3 to 256^3 within 10%.
        long long best = -1;
        for (int nseg = 1; nseg <= p.nx; nseg++) {
            const int s = (p.nx + nseg - 1) / nseg;
            const long long nb = (long long)tc.ntiles * ((p.nx + s - 1) / s);
            if (max_blocks > 0 && nseg > 1 && nb > max_blocks) break;
            const long long rounds = (nb + kCUs - 1) / kCUs;
            const long long cost = rounds * (s + 2);
            if (best < 0 || cost < best) {
                best = cost;
                sx = s;
            }
        }
    }
    if (sx > p.nx) sx = p.nx;
    tc.sx = sx;
    tc.nseg = (p.nx + sx - 1) / sx;
    tc.seg_req = segment_x;
    return tc;
}

static TileCfg row_tiles(const KParams& p, int tz, int segment_x)
{
    TileCfg tc;
    tc.tz = tz;
    const int ty = kFused / tz;
    tc.nty = (p.ny + ty - 1) / ty;
    tc.ntz = (p.nz + tz - 1) / tz;
    return with_segments(p, tc, segment_x);
}

TileCfg row_tile_config(const KParams& p, int segment_x, bool fp32)
{
    // 128 wide unless 64 leaves fewer idle lanes along z
    const long long w128 = 128LL * ((p.nz + 127) / 128), w64 = 64LL * ((p.nz + 63) / 64);
    TileCfg tc = row_tiles(p, w64 < w128 ? 64 : 128, segment_x);
    // FP32 storage with rows of 256 sites: the allocation-free sums take what
    // whole rows in pairs would fit in their array.  The narrower tiles are one
    // more in a plane where ny is odd; there their segments are as long as that
    // takes.
    if (fp32 && !p.fd && p.nz == 256 && tc.ntiles * (long long)tc.nseg > kMaxStepPartials) {
        const TileCfg pairs = row_tiles(p, 256, segment_x);
        if (pairs.ntiles * (long long)pairs.nseg <= kMaxStepPartials) {
            const int most = kMaxStepPartials / tc.ntiles;
            tc.sx = (p.nx + most - 1) / most;
            tc.nseg = (p.nx + tc.sx - 1) / tc.sx;
        }
    }
    return tc;
}

// Flat tiles or row tiles.  Measured (us per step, rows / flat): FP32 128^3
// 132 / 130, 192^3 461 / 451, 100 x 120 x 240 207 / 198, 151 x 105 x 160 198 / 168,
// but 24^3 9.2 / 12.4, 40^3 9.8 / 12.7 (short segments, whose prologue the
// pipelined march of flat tiles lengthens): flat where they march fewer planes,
// or as many in segments of 8 or more.  FP64 192^3 831 / 843, 256^3 1831 / 1905
// (flat tiles re-read more through L2), 100 x 120 x 240 340 / 346, but 96^3
// 119 / 111, 151 x 105 x 150 409 / 354: flat where row tiles leave more than a
// tenth of their lanes idle along z.  Up to 120000 sites, whose segments are
// short, row tiles (shards of 8 x 100 x 100 in FP64 16.5 / 17.4, 10 x 75 x 100 15.5
// / 16.7).  Flat tiles take no more workgroups than the array of the
// allocation-free sums holds partials for, unless row tiles do too: what row
// tiles can sum there, flat tiles can (there are never more flat tiles in a
// plane than row tiles).
TileCfg tile_config(const KParams& p, int segment_x, bool fp32)
{
    const TileCfg rows = row_tile_config(p, segment_x, fp32);
    if (!flat_fits(p, fp32) || p.nsites <= 120000) return rows;
    TileCfg flat = rows;
    flat.tz = 0;
    flat.nty = 1;
    flat.ntz = (p.ny * p.nz + kFused - 1) / kFused;
    flat = with_segments(p, flat, segment_x,
                         std::max((long long)rows.ntiles * rows.nseg, (long long)kMaxStepPartials));
    if (fp32) {
        const long long r = march_cost(rows), f = march_cost(flat);
        return f < r || (f == r && flat.sx >= 8) ? flat : rows;
    }
    return 10LL * p.nz < 9LL * rows.tz * ((p.nz + rows.tz - 1) / rows.tz) ? flat : rows;
}

// Where the march is short, its serial prologue and the idle CUs cost more
// than a second pass over g: two launches with one site per thread are
// faster up to a size that depends on what the passes move.  Measured (us per
// step, march / two passes):
//   stress, FP32 (312 / 404 B per site): 16^3 9.9 / 6.6, 48^3 13.8 / 10.6,
//     64^3 21.5 / 18.2, 90 x 75 x 100 47 / 45, 96^3 64 / 71, 128^3 131 / 170
//   stress, FP64, tau_g = 1 (608 / 632 B: the collision loads no g): 16^3
//     12.5 / 6.1, 64^3 33 / 26, 96^3 111 / 104, 72 x 111 x 150 183 / 159,
//     128^3 248 / 255, 192^3 832 / 861
//   stress, FP64, other tau_g (608 / 784 B): 16^3 12.8 / 6.1, 64^3 33.8 / 31.9,
//     68^3 37.6 / 40.0, 72^3 42 / 46, 80^3 73 / 70, 88^3 98 / 100, 90 x 75 x 100
//     101 / 100, 96^3 112 / 126
//   force, FP32: 16^3 19 / 7.7, 64^3 25 / 21, 96^3 78 / 69, 72 x 111 x 150
//     110 / 111, 128^3 161 / 171, 151 x 105 x 150 219 / 226
//   force, FP64, tau_g = 1: 64^3 43 / 27, 128^3 290 / 275, 192^3 942 / 913,
//     256^3 1999 / 2107; other tau_g: 96^3 155 / 134, 128^3 299 / 319
// With sums, lattices whose collision pass cannot reduce them (a third pass)
// march.
// The smallest lattices take one launch: the first ten or so launches after
// the host has waited cost it 10 us each, later ones 3.5, and two chains from
// launch to store are longer than one.  Measured, us of a whole run (initial
// state, 5 / 100 steps, moments), march / two passes / boxes: stress FP32 16^3
// 73 / 117 / 68 and 993 / 800 / 605, 32^3 74 / 117 / 67 and 1007 / 870 / 781;
// FP64 16^3 89 / 117 / 68 and 1299 / 790 / 596, 32^3 87 / 118 / 74 and 1228 /
// 917 / 956; force FP32 16^3 131 / 125 / 105 and 1925 / 850 / 671, 28^3 (343
// boxes) 125 / 121 / 127 and 1786 / 958 / 1020; force FP64 16^3 135 / 124 / 130
// and 2047 / 871 / 900.  Above that, FP32 storage marches, one launch too, as
// long as the march keeps up with two: 40^3 81 / 117 and 1015 / 1010; further
// where a segment is one plane (5 / 50 steps): 42 x 42 x 44 83 / 128 and 547 /
// 578, 44 x 40 x 50 85 / 117 and 571 / 593, but 17 x 56 x 100 88 / 114 and 607 /
// 588, and with two planes 44^3 103 / 114 and 756 / 605.
// The number of steps does not enter.  In a run of 3 to 5 steps the host's wait
// shows and the march would win further up (us of the run, two passes / march:
// 40^3 FP64 3 steps 101 / 69, 5 114 / 96; 48^3 FP32 105 / 74, 117 / 104), but the
// same steps called alone (44 / 53, 75 / 81; 44 / 58, 78 / 88) or one call after
// another (36 / 42, 56 / 70; 36 / 47, 58 / 77) would lose, and a call does not
// know which it is.
int step_variant(const KParams& p, const TileCfg& tc, bool fp32, int variant, bool sums)
{
    // a segment length asked for is the marching kernel's; shards have no
    // two-pass form
    if (variant != 0 || p.xh || tc.seg_req > 0) return variant;
    if (sums && collide_grid(p, false) > kMaxStepPartials) return 0;
    const bool g1 = !fp32 && p.omega_g == 1.0;
    const int limit = p.force ? (g1 ? 7100000 : fp32 ? 1100000 : 1500000)
                              : (g1 ? 2000000 : fp32 ? 700000 : 300000);
    if (box_cfg(p).blocks() <= (!p.force ? 512 : fp32 ? 256 : 0)) return kStepBox;
    if (!p.force && fp32 && (p.nsites <= 75000 || (p.nsites <= 90000 && march_cost(tc) <= 3)))
        return 0;
    return p.nsites <= limit ? 1 : 0;
}

int step_sums_blocks(const KParams& p, const TileCfg& tc, bool fp32, int variant)
{
    variant = step_variant(p, tc, fp32, variant, true);
    if (variant == kStepBox) return box_cfg(p).blocks();
    if (variant == 1) return collide_grid(p, true);
    if (p.force) return force_sums_blocks(p, tc.seg_req);
    return tc.ntiles * tc.nseg;
}

hipError_t launch_init(const KParams& p, bool fp32, void* state, const double* phi0, hipStream_t s)
{
#define CALL                                                                                   \
    {                                                                                          \
        Lvl<T> l = level<T>(state, p, REF);                                                    \
        k_init<T, DEV, REF><<<grid_for(p), kBlock, 0, s>>>(p, l.F, l.G, l.phic, phi0);        \
    }
    LB_DISPATCH(fp32, CALL, CALL);
#undef CALL
    return hipGetLastError();
}

// The march's segments: the least planes' work for as many segments as fill
// the resident workgroups k times.
CompactTiles compact_tiles(const KParams& p, int resident)
{
    CompactTiles t;
    t.nty = (p.ny + kCompactTY - 1) / kCompactTY;
    t.ntz = (p.nz + kCompactTZ - 1) / kCompactTZ;
    const int tiles = t.nty * t.ntz;
    long long cost = -1;
    for (int k = 1; k <= 8; k++) {
        const int want = std::min(p.nx, std::max(1, k * resident / tiles));
        const int sx = (p.nx + want - 1) / want;
        const int n = (p.nx + sx - 1) / sx;
        const long long c = ((long long)tiles * n + resident - 1) / resident
                          * (sx + 2);
        if (cost >= 0 && c >= cost) continue;
        cost = c;
        t.sx = sx;
        t.nseg = n;
    }
    return t;
}

// with the force coupling in FP64 one workgroup per CU, by its registers
CompactTiles compact_step_tiles(const KParams& p, bool fp32)
{
    return compact_tiles(p, p.force && !fp32 ? kCompactResident / 2 : kCompactResident);
}

// The march runs on lattices that fill it, of at least 4 planes, and that its
// tiles cover with at most 3/4 more cells than sites.  us per step, one site
// per thread / march: FP64 stress 48^3 14.1 / 14.2, 60 x 52 x 70 23.8 / 21.5,
// 96^3 87 / 70; FP64 force 56^3 21.0 / 21.7, 60 x 52 x 70 25.4 / 24.4, 96^3
// 104 / 91; FP32 force 80^3 31.9 / 33.2, 90 x 75 x 100 41.0 / 40.6, 128^3
// 143 / 127; 300 x 40 x 20, 1.9 cells per site, FP64 force 25.7 / 26.5.
bool compact_march(const KParams& p, bool fp32)
{
    const CompactTiles t = compact_tiles(p, kCompactResident);
    const long long plane = (long long)p.ny * p.nz;
    const int limit = fp32 ? 650000 : p.force ? 200000 : 160000;
    return p.nsites >= limit && p.nx >= 4 && 4LL * t.nty * t.ntz * kCompactTY * kCompactTZ <= 7 * plane;
}

// Where f's ten moments between steps beat the 19 populations.  Their pass is
// a march, with the force coupling of one workgroup per CU (its F needs 160
// registers; with sums also in FP32 storage), which loses to one site per
// thread in small or ill-covered lattices.  us per step, populations /
// moments: FP64 stress 64^3 22.2 / 22.1, 7 x 200 x 300 33.1 / 33.4, 90 x 75 x
// 100 49 / 42, 128^3 162 / 126, 256^3 1311 / 982; FP64 force 90 x 75 x 100
// (1.4 cells per site) 54 / 62, 96^3 91 / 61, 128^3 188 / 174, 256^3 1472 /
// 1345; FP32 force 72 x 111 x 150 64 / 73, 112^3 94 / 90, 116^3 112 / 91, 120^3
// 122 / 92, 128^3 126 / 106 (with sums 122 / 128), 151 x 105 x 150 166 / 140, 160^3
// 247 / 242, 168^3 321 / 289, 192^3 417 / 417 (in a later run 416 / 401), 256^3
// 919 / 926.
bool compact_f(const KParams& p, bool fp32, bool sums)
{
    if (p.omega_f != 1.0 || !compact_march(p, fp32)) return false;
    const CompactTiles t = compact_step_tiles(p, fp32);
    if (sums && t.blocks() > kMaxStepPartials) return false;
    if (!p.force) return p.nsites >= 450000;
    if (4LL * t.nty * t.ntz * kCompactTY * kCompactTZ > 5LL * p.ny * p.nz) return false;
    return fp32 ? !sums && p.nsites >= 1500000 && p.nsites < 5000000 : p.nsites >= 800000;
}

// Not FP32 storage with the stress coupling: its collision forms g + (g^eq -
// g), which rounds with g.  Below 40000 sites the launches set the time, and
// the compact phi pass's are the longer ones (us per step, full / compact:
// 16^3 5.8 / 6.2, 32^3 7.4 / 7.5, 40^3 10.5 / 9.8).
bool can_compact(const KParams& p, const TileCfg& tc, bool fp32, int variant)
{
    if (p.fd || p.xh || variant != 0 || tc.seg_req > 0 || p.omega_g != 1.0) return false;
    return p.nsites >= 40000 && (!fp32 || p.force);
}

hipError_t launch_step(const KParams& p, const TileCfg& tc, bool fp32, int variant,
                       const void* src, void* dst, double* phi_work, double* partials,
                       double* phi_src_out, hipStream_t s, int compact,
                       const double* compact_src_phi)
{
    // phi of src goes to phi_src_out if given (the work field otherwise,
    // where a pass needs one), or into the compact level that it is part of
    double* phi64 = phi_src_out ? phi_src_out : phi_work;
    const bool to_compact = compact & kCompactDst;
    if (to_compact && !phi_src_out)
        phi64 = fp32 ? compact_phi(level<float>(dst, p, true).G)
                     : compact_phi(level<double>(dst, p, false).G);
    variant = compact ? 1 : step_variant(p, tc, fp32, variant, partials != nullptr);
    if (variant == 1) {
        // phi (and in FP32 mode the new level's phi_c) for the collision pass
        hipError_t e;
        if (compact & kCompactSrc)
            e = p.force ? launch_phi_compact_force(p, fp32, src, compact_src_phi, phi64,
                                                   to_compact ? nullptr : dst, s)
                        : launch_phi_compact_f64(p, src, compact_src_phi, phi64, s);
        else
            e = fp32 ? launch_phi_f32(p, src, phi64, to_compact ? nullptr : dst, s)
                     : launch_phi_f64(p, src, phi64, dst, s);
        if (e != hipSuccess) return e;
    }
    if ((compact & kCompactF) && (compact & kCompactSrc))
        return p.force ? launch_step_compact_force(p, fp32, src, dst, !to_compact, phi64, partials, s)
                       : launch_step_compact_f64(p, src, dst, !to_compact, phi64, partials, s);
    const int form = !to_compact ? 0 : compact & kCompactF ? 2 : 1;
    if (p.force)
        return launch_force_collide(p, tc, fp32, variant, form, src, dst,
                                    variant == 1 ? phi64 : phi_src_out, partials, s);
    auto step = fp32 ? launch_step_f32 : launch_step_f64;
    return step(p, tc, variant, form, src, dst, phi64, partials, phi_src_out, s);
}

hipError_t launch_phi(const KParams& p, bool fp32, const void* state, double* phi, hipStream_t s)
{
    return fp32 ? launch_phi_f32(p, state, phi, nullptr, s) : launch_phi_f64(p, state, phi, nullptr, s);
}

hipError_t launch_moments(const KParams& p, bool fp32, const void* state, double* rho, double* u,
                          double* phi, double* work, double* partials, int* nblocks_out,
                          hipStream_t s)
{
    // phi alone: its own pass
    if (phi && !rho && !u && !partials) return launch_phi(p, fp32, state, phi, s);
    const int nb = moments_grid(p, partials != nullptr);
    *nblocks_out = nb;
    double* fphi = nullptr;
    if (p.force && (u || partials)) {
        // F of this state: phi into its output or the work field first
        fphi = phi ? phi : work;
        hipError_t e = launch_phi(p, fp32, state, fphi, s);
        if (e != hipSuccess) return e;
    }
    auto m = fp32 ? moments<float> : moments<double>;
    m(p, nb, state, fphi, rho, u, fphi == phi ? nullptr : phi, partials, s);
    return hipGetLastError();
}

hipError_t launch_sums_final(const double* partials, int nblocks, int ncomp, int nsets,
                             double* out, hipStream_t s)
{
    k_sums_final<<<dim3(ncomp, nsets), kBlock, 0, s>>>(partials, nblocks, out);
    return hipGetLastError();
}

hipError_t launch_export(const KParams& p, bool fp32, const void* state, double* f, double* g,
                         hipStream_t s)
{
#define CALL                                                                                  \
    {                                                                                         \
        Lvl<T> a = level<T>(const_cast<void*>(state), p, REF);                                \
        k_export<T, DEV, REF><<<grid_for(p), kBlock, 0, s>>>(p, a.F, a.G, a.phic, f, g);      \
    }
    LB_DISPATCH(fp32, CALL, CALL);
#undef CALL
    return hipGetLastError();
}

hipError_t launch_import(const KParams& p, bool fp32, void* state, const double* f,
                         const double* g, hipStream_t s)
{
#define CALL                                                                                  \
    {                                                                                         \
        Lvl<T> a = level<T>(state, p, REF);                                                   \
        if (REF) k_import_ref<<<grid_for(p), kBlock, 0, s>>>(p, a.phic, g);                   \
        k_import<T, DEV, REF><<<grid_for(p), kBlock, 0, s>>>(p, a.F, a.G, a.phic, f, g);      \
    }
    LB_DISPATCH(fp32, CALL, CALL);
#undef CALL
    return hipGetLastError();
}

}  // namespace lbk
