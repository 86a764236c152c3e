// Kernels of one LB-scheme timestep with the stress coupling, and the phi pass
// the force coupling shares: instantiated for FP32 storage by
// lb_step_f32.hip and for FP64 by lb_step_f64.hip.
//
// Three forms with bit-identical levels, chosen by step_variant():
//
//   k_step_box (lb_box.h), for the smallest lattices.
//
//   k_phi + k_step_2s: a phi pass, then stencil, collision and propagation,
//     one site per thread: the shortest chains from launch to store, for
//     lattices too small (or, where the collision loads no g, not large
//     enough) for the march to pay.
//   k_step_fused_f32 / _f64: the marching single pass.  Each workgroup owns a
//     tile of 512 (y, z) columns and marches along x over a segment of
//     planes.  For plane x it needs phi at planes x-1, x, x+1 (7-point
//     stencil); phi(x+1) is formed from the pulled g of plane x+1, which the
//     same threads keep in registers for plane x+1's own collision one
//     iteration later.  phi on the tile's (y, z) halo ring is formed by extra
//     pulls that mostly hit in cache (the neighbouring tiles read the same
//     lines).  phi planes live in a 4-slot LDS ring.  Every population is
//     read once and written once per step from HBM: the method's minimum
//     traffic, instead of a separate phi pass plus a collision pass.
#pragma once

#include <type_traits>

#include "lb_box.h"
#include "lb_compact.h"
#include "lb_device.h"
#include "lb_sweep.h"

namespace lbk {

using namespace dev;

namespace {

// Tiles of the marching kernel: kFused columns, one per thread.
//   TZ = 0: flat tiles, kFused consecutive sites of a plane in site order
//     (y*nz + z), whatever nz is: every lane of every tile is a site, and a
//     tile's accesses are whole runs of rows.  Its halo is the sites within
//     nz + 1 of it in that order.  The last tile of a plane is shifted back
//     to end with it (both tiles store the same values at the sites they
//     share).  Needs a plane of at least kFused sites and a halo of at most
//     kFused cells (tile_config).
//   TZ = 128 or 64: kFused/TZ rows of TZ contiguous z-sites, for the other
//     lattices: 128 unless 64 covers nz with fewer idle lanes.
constexpr int kFused = 512;
// one thread per halo-ring cell (2 rows, 2 columns, 4 corners)
static_assert(2 * 128 + 2 * (kFused / 128) + 4 <= kFused, "halo ring larger than the workgroup");
static_assert(2 * 64 + 2 * (kFused / 64) + 4 <= kFused, "halo ring larger than the workgroup");

// phi(x) = sum_i g_i(x) of the post-propagation state (FP64); with dphic
// (FP32 mode) also the reference field phi_c of the level a step makes.
template <typename T, bool REF>
__global__ __launch_bounds__(kBlock) void k_phi(KParams p, const T* __restrict__ G,
                                                const unsigned* __restrict__ phic,
                                                double* __restrict__ phi,
                                                unsigned* __restrict__ dphic)
{
    const int s = xcd_block() * int(blockDim.x) + threadIdx.x;
    if (s >= p.nsites) return;
    const Geo q = geo_of(p, s);
    const double v = phi_at<T, REF>(p, q, G, phic);
    phi[s] = v;
    if (REF && dphic) dphic[phic_site(p, q.x, q.y, q.z)] = phic_word(v);
}

// Two-pass form, second pass: stencil + chemical stress + collision, one
// site per thread; phi of the post-propagation source level (all sites)
// comes from k_phi.  G1 (FP64, omega_g = 1): g* = g^eq, so the collision
// loads no g and the two passes move the single pass's 608 bytes per site
// plus phi (776 otherwise).  SUMS: 0, or the block size, for block partials
// of the source level's conserved sums.  COMPACT: 1: the new level is compact
// (lb_compact.h), its phi this step's phi field, written by the phi pass; 2:
// with f's moments.
template <typename T, bool DEV, bool REF, bool G1, int SUMS, int COMPACT = 0>
__global__ __launch_bounds__(kBlock) void k_step_2s(KParams p, const T* __restrict__ sF,
                                                    const T* __restrict__ sG,
                                                    const unsigned* __restrict__ sphic,
                                                    const double* __restrict__ phi,
                                                    T* __restrict__ dF, T* __restrict__ dG,
                                                    double* __restrict__ partials)
{
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    const auto site = [&](int s) {
        const Geo q = geo_of(p, s);
        T f[NV], g[NV];
#pragma unroll
        for (int i = 0; i < NV; i++) {
            f[i] = sF[dist_pull(p, q, i)];
            g[i] = G1 ? T(0) : sG[dist_pull(p, q, i)];
        }
        const double c = phi[s];
        const Stencil st = stencil(c, phi[site_of(p, q.xp, q.y, q.z)], phi[site_of(p, q.xm, q.y, q.z)],
                                   phi[site_of(p, q.x, q.yp, q.z)], phi[site_of(p, q.x, q.ym, q.z)],
                                   phi[site_of(p, q.x, q.y, q.zp)], phi[site_of(p, q.x, q.y, q.zm)]);
        if (SUMS) site_sums<DEV>(p, f, c, nullptr, acc);
        if (REF) {
            const double dphi = c - phic_value(sphic[phic_site(p, q.x, q.y, q.z)]);
#pragma unroll
            for (int i = 0; i < NV; i++) g[i] = pre_collision_dev(i, g[i], dphi);
        }
        if constexpr (COMPACT == 2) {
            FEq<T> e;
            const Vel<T> u = feq_stress<T, DEV>(p, f, st, e);
            compact_mu_u(dG, p)[s] = MuU<T>{chem_potential<T>(p, st), u.x, u.y, u.z};
            store_feq(p, dF, s, e);
            return;
        } else if constexpr (COMPACT == 1) {
            const Vel<T> u = collide_f<T, DEV, !DEV>(p, f, st);
            compact_mu_u(dG, p)[s] = MuU<T>{chem_potential<T>(p, st), u.x, u.y, u.z};
        } else {
            collide<T, DEV, REF, G1>(p, f, g, st);
        }
#pragma unroll
        for (int i = 0; i < NV; i++) {
            dF[dist_own(p, q, i)] = f[i];
            if (!COMPACT)
                dG[dist_own(p, q, i)] = REF ? to_dest_ref(i, g[i], c, phi[push_site(p, q, i)]) : g[i];
        }
    };
    if constexpr (SUMS > 0) {
        for (XcdSweep w = sums_sweep(p.nsites, SUMS); w.s < w.end; w.s += w.stride) site(w.s);
    } else {
        const int s = xcd_block() * int(blockDim.x) + threadIdx.x;
        if (s < p.nsites) site(s);
    }
    if (SUMS) block_partials<5, SUMS ? SUMS : kBlock>(acc, partials);
}

// Register copy the compiler cannot merge away: the source register is free
// once the copy has executed, so a load issued after it can land in that
// register.  The memory clobber keeps later loads after the copy.
__device__ __forceinline__ float vcopy(float v)
{
    float r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(v) : "memory");
    return r;
}
__device__ __forceinline__ unsigned vcopy(unsigned v)
{
    unsigned r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(v) : "memory");
    return r;
}
__device__ __forceinline__ double vcopy(double v)
{
    double r;
    asm volatile("v_mov_b64 %0, %1" : "=v"(r) : "v"(v) : "memory");
    return r;
}

// Wrap a coordinate v in [-2n, 3n) onto [0, n).
__device__ __forceinline__ int wrapg(int v, int n)
{
    if (v < 0) return v + n < 0 ? v + 2 * n : v + n;
    if (v >= n) return v - n >= n ? v - 2 * n : v - n;
    return v;
}

// Addressing (layout of didx()): a thread's (y, z) never changes while it
// marches along x, so the byte offsets of the 9 rows/columns (y - cy, z - cz)
// within a plane are computed once (32-bit: one plane of F or G is under
// 4 GiB, checked at creation); a component adds a uniform in-plane offset
// and a plane a uniform plane offset -- 32-bit when the whole F or G region
// is under 4 GiB (SMALL), else 64-bit, added to the base pointer.
template <bool SMALL>
using OffT = typename std::conditional<SMALL, unsigned, size_t>::type;

template <bool SMALL, typename T>
__device__ __forceinline__ T ldc(const T* __restrict__ base, OffT<SMALL> pl, int i,
                                 unsigned compb, unsigned row)
{
    const char* b = reinterpret_cast<const char*>(base);
    if (SMALL) return *reinterpret_cast<const T*>(b + (unsigned(pl) + unsigned(i) * compb + row));
    // uniform 64-bit pointer to the component's run in the plane, then the row
    const char* bi = b + (size_t(pl) + size_t(i) * compb);
    return *reinterpret_cast<const T*>(bi + row);
}
// Stores are non-temporal (NT) where a component's row is whole 64-byte
// pieces and two levels exceed the 256 MB Infinity Cache: the new level is not
// read again in this launch, so it should not displace the source lines that
// neighbouring tiles still pull through L2.  Smaller levels are better kept
// for the next step, and the pieces that two components or two tiles share
// would go to memory in parts, where plain stores let L2 join them (us per
// step, NT / plain: FP32 151 x 105 x 150, rows of 600 bytes, 228 / 189,
// 90 x 75 x 100 64 / 47, 96^3 64 / 60, 128^3 131 / 136, 256^3 944 / 983; FP64
// 32 x 128 x 128 68 / 71).  The march also stores so on lattices of at most
// 120000 sites, whatever their rows (march_nt).
template <bool SMALL, bool NT, typename T>
__device__ __forceinline__ void stc(T* __restrict__ base, OffT<SMALL> pl, int i, unsigned compb,
                                    unsigned row, T v)
{
    char* b = reinterpret_cast<char*>(base);
    T* q = SMALL ? reinterpret_cast<T*>(b + (unsigned(pl) + unsigned(i) * compb + row))
                 : reinterpret_cast<T*>((b + (size_t(pl) + size_t(i) * compb)) + row);
    if constexpr (NT)
        __builtin_nontemporal_store(v, q);
    else
        *q = v;
}

// byte offsets of the 9 rows/columns (y + dy, z + dz), dy, dz in {-1, 0, 1},
// within a plane of an F or G region
struct Yz9 {
    unsigned o[3][3];
};
template <typename T>
__device__ __forceinline__ Yz9 yz9(const KParams& p, int y, int z)
{
    const int ys[3] = {wrapm(y, p.ny), y, wrapp(y, p.ny)};
    const int zs[3] = {wrapm(z, p.nz), z, wrapp(z, p.nz)};
    Yz9 r;
#pragma unroll
    for (int a = 0; a < 3; a++)
#pragma unroll
        for (int c = 0; c < 3; c++) r.o[a][c] = row_off(p, ys[a], zs[c]) * unsigned(sizeof(T));
    return r;
}

// Single-pass step (see the file comment).  Block -> (segment, tile) with
// an XCD-aware order: consecutive workgroup ids go round-robin over the 8
// XCDs, so ids are remapped to give each XCD a contiguous run of tiles, z
// fastest.  An XCD then owns slabs of whole (y) rows: the cache lines that
// z-shifted pulls and the halo columns share with the z-neighbouring tile,
// and the halo rows shared with y-neighbours, are fetched into the same L2.
//
// FP32 mode: the pull of a site needs only its own phi_c (one 32-bit load
// per site); the store of direction i needs phi at the destination y + c_i, which
// the LDS phi ring already holds (its halo then includes the diagonal (y, z)
// neighbours).  G1 (FP64, omega_g = 1): g* = g^eq, as in the two-pass form.
// COLL = false is the kernel's memory-only twin (LB_KERNEL_STREAM): every
// load, LDS ring, phi sum and store of the step, with the collision left out,
// so the populations stream freely, f_i(x + c_i, t+1) = f_i(x, t).
template <typename T, bool DEV, bool REF, bool SMALL, bool PIPE, int TZ, bool COLL, bool G1, bool NT>
__device__ __forceinline__ void step_fused_body(const KParams& p, const TileCfg& tc,
                                                const T* __restrict__ sF,
                                                const T* __restrict__ sG,
                                                const unsigned* __restrict__ sphic,
                                                T* __restrict__ dF, T* __restrict__ dG,
                                                unsigned* __restrict__ dphic,
                                                double* __restrict__ phi_out,
                                                double* __restrict__ partials)
{
    constexpr bool FLAT = TZ == 0;
    constexpr int TW = FLAT ? kFused : TZ, TY = kFused / TW;
    // LDS cells of a plane of phi: the tile with a ring around it, or (flat)
    // the tile and up to kFused halo cells
    constexpr int PZ = TW + 2, NPH = FLAT ? 2 * kFused : (TY + 2) * PZ;
    __shared__ double ph[4][NPH];
    // value kept per direction between the phi pull and the collision: the
    // stored FP32 deviation (FP32 mode) or the FP64 population
    using K = typename std::conditional<REF, T, double>::type;
    using O = OffT<SMALL>;
    const unsigned compb = p.cs * unsigned(sizeof(T));   // one component step
    const O planeb = O(p.plane_e) * O(sizeof(T));        // one plane of F or G

    const int b = xcd_block();
    const int tile = b % tc.ntiles, seg = b / tc.ntiles;
    const int x0 = seg * tc.sx;
    const int x1 = min(x0 + tc.sx, p.nx);
    const int plane = p.ny * p.nz;
    const int y0 = FLAT ? 0 : (tile / tc.ntz) * TY, z0 = FLAT ? 0 : (tile % tc.ntz) * TW;
    const int tya = min(TY, p.ny - y0), tza = min(TW, p.nz - z0);
    // flat tile: its first site in the plane (the last tile's shifted back)
    const int s0 = FLAT ? min(tile * kFused, plane - kFused) : 0;
    const int lz = threadIdx.x % TW, ly = threadIdx.x / TW;
    const bool active = FLAT || (lz < tza && ly < tya);
    // lanes outside the lattice hold a valid site's offsets and do nothing;
    // rowsite is the in-plane site index (for phi_c)
    const int sy = FLAT ? (s0 + lz) / p.nz : (active ? y0 + ly : 0);
    const int sz = FLAT ? s0 + lz - sy * p.nz : (active ? z0 + lz : 0);
    const Yz9 row = yz9<T>(p, sy, sz);
    const unsigned rowsite = unsigned(sy * p.nz + sz);
    // sites whose conserved quantities this tile counts
    const bool counted = !FLAT || s0 + lz >= tile * kFused;

    // Halo ring.  Row tiles: rows y0-1 and y0+tya, columns z0-1 and z0+tza,
    // and in FP32 mode the 4 corners.  A tile that spans the whole periodic z
    // extent pulls only the two rows: its halo columns are its own last and
    // first columns, which put() below copies into LDS columns 0 and tza + 1
    // as it stores them (the corners with the rows' cells).
    // Flat tiles: the hw = nz sites before and after the tile, which hold its
    // y neighbours, and its z neighbours across a row's periodic end (nz - 1
    // sites away).  In FP32 mode the diagonal neighbours need a site more at
    // each end, and, across a row's end, the site 2 nz - 1 ahead of the
    // tile's last row start and the one as far behind its first row end,
    // which have a cell of their own each after the window; a tile of whole
    // rows has them all within nz.
    const bool rows = FLAT && kFused % p.nz == 0;
    const int hw = p.nz + (REF && !rows ? 1 : 0);
    const int nwin = kFused + 2 * hw;  // window cells
    const bool fullz = !FLAT && tza == p.nz;
    const int nside = fullz ? 2 * tza : 2 * tza + 2 * tya;
    const int nring = FLAT ? 2 * hw + (REF && !rows ? 2 : 0) : nside + (REF && !fullz ? 4 : 0);
    // ring cell k: its LDS cell, and its (y, z)
    auto ring_cell = [&](int k, int& li, int& y, int& z) {
        if (FLAT) {
            int w = k < hw ? k : k + kFused;  // window cell
            li = w;
            // (li of the two extra cells: nwin and nwin + 1, which k + kFused is)
            if (k == 2 * hw) w = hw + (s0 + p.nz - 1) / p.nz * p.nz - s0 - 1 - (2 * p.nz - 1);
            if (k == 2 * hw + 1) w = hw + (s0 + kFused - 1) / p.nz * p.nz - s0 + 2 * p.nz - 1;
            const int s = wrap_any(s0 - hw + w, plane);
            y = s / p.nz;
            z = s - y * p.nz;
            return;
        }
        int a, c;
        if (k < tza) { a = 0; c = k + 1; }
        else if (k < 2 * tza) { a = tya + 1; c = k - tza + 1; }
        else if (k < 2 * tza + tya) { a = k - 2 * tza + 1; c = 0; }
        else if (k < nside) { a = k - 2 * tza - tya + 1; c = tza + 1; }
        else { a = ((k - nside) & 1) ? tya + 1 : 0; c = ((k - nside) & 2) ? tza + 1 : 0; }
        li = a * PZ + c;
        y = wrapg(y0 + a - 1, p.ny);
        z = wrapg(z0 + c - 1, p.nz);
    };
    const bool ring = int(threadIdx.x) < nring;
    int rli, ry, rz;
    ring_cell(ring ? int(threadIdx.x) : 0, rli, ry, rz);
    const Yz9 rrow = yz9<T>(p, ry, rz);
    const unsigned rsite = unsigned(ry * p.nz + rz);
    // LDS cell of the own site, and of the neighbour at (dy, dz) of a site
    // at cell o
    const int own = FLAT ? hw + lz : (ly + 1) * PZ + lz + 1;
    auto nbr = [&](int o, int dy, int dz) __attribute__((always_inline)) {
        if (!FLAT) return o + dy * PZ + dz;
        int n = o + dy * p.nz;
        if (dz > 0) n += sz == p.nz - 1 ? 1 - p.nz : 1;
        if (dz < 0) n += sz == 0 ? p.nz - 1 : -1;
        if (REF && dy < 0 && dz > 0) n = n < 0 ? nwin : n;
        if (REF && dy > 0 && dz < 0) n = n >= nwin ? nwin + 1 : n;
        return n;
    };
    // phi into LDS cell li of slot sl, and into the wrap column of a full-z
    // tile
    auto put = [&](int sl, int li, double v) __attribute__((always_inline)) {
        ph[sl][li] = v;
        if (!FLAT && fullz) {
            const int c = li % PZ;
            if (c == tza) ph[sl][li - tza] = v;
            if (c == 1) ph[sl][li + tza] = v;
        }
    };

    // plane indices run from x0-2 to x1+2 (nx may be 1): wrap without
    // division or branches (valid on [-2nx, 4nx)).  An x-slab shard has no
    // wrap: its regions hold planes -2 .. nx+1 of F and G (the halo planes
    // of the neighbours' populations) and -1 .. nx of phi_c; indices beyond
    // those occur only in the prefetch past a segment's end, whose values
    // go unused, and are clamped onto the last halo plane.
    auto xw = [&](int X) {
        X += X < 0 ? p.nx : 0;
        X += X < 0 ? p.nx : 0;
        X -= X >= p.nx ? p.nx : 0;
        X -= X >= p.nx ? p.nx : 0;
        X -= X >= p.nx ? p.nx : 0;
        return X;
    };
    auto xf = [&](int X) { return p.xh ? min(max(X, -2), p.nx + 1) + 2 : xw(X); };
    auto xc = [&](int X) { return p.xh ? min(max(X, -1), p.nx) + 1 : xw(X); };
    // byte base of plane X in F or G; element base of plane X in phi_c
    auto pbase = [&](int X) { return O(xf(X)) * planeb; };
    auto pcbase = [&](int X) { return unsigned(xc(X) * plane); };
    // pull of plane X for a site with row offsets yz and in-plane index
    // `site`: kept values into kv[] and the site's phi_c word into *pc (if
    // non-null); returns phi
    auto pull_phi = [&](int X, const Yz9& yz, unsigned site, K* kv, unsigned* pc)
                        __attribute__((always_inline)) -> double {
        const O pb[3] = {pbase(X - 1), pbase(X), pbase(X + 1)};
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < NV; i++) {
            const K v = K(ldc<SMALL>(sG, pb[1 - CX[i]], i, compb, yz.o[1 - CY[i]][1 - CZ[i]]));
            if (kv) kv[i] = v;
            acc += double(v);
        }
        if (REF) {
            const unsigned w = sphic[pcbase(X) + site];
            if (pc) *pc = w;
            return phic_value(w) + acc;
        }
        return acc;
    };

    // conserved sums of the source level (FP64), if requested
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};

    // collision of this thread's site at plane x and the stores of its new
    // values, from the pulled f[], the kept g values kc[] (and the site's
    // phi_c word pcc), with phi of planes x-1, x, x+1 in LDS slots sp, sc, sn
    auto update = [&](int x, T* f, const K* kc, unsigned pcc, int sp, int sc, int sn)
                      __attribute__((always_inline)) {
        const int psl[3] = {sp, sc, sn};
        // (flat: the neighbours' cells, a few adds each, are not to be held in
        // registers through the march)
        int o = own;
        if (FLAT) asm volatile("" : "+v"(o));
        const double c = ph[sc][o];
        const Stencil st = stencil(c, ph[sn][o], ph[sp][o], ph[sc][nbr(o, 1, 0)],
                                   ph[sc][nbr(o, -1, 0)], ph[sc][nbr(o, 0, 1)],
                                   ph[sc][nbr(o, 0, -1)]);
        T g[NV];
        if (REF) {
            const double dphi = c - phic_value(pcc);
#pragma unroll
            for (int i = 0; i < NV; i++) g[i] = pre_collision_dev(i, T(kc[i]), dphi);
        } else {
#pragma unroll
            for (int i = 0; i < NV; i++) g[i] = T(kc[i]);
        }
        if (partials) {
            // moments of the stored values, formed in FP64; with FP32 storage
            // from the sums and differences of the direction pairs
            // (2k+1, 2k+2), in short chains (0.5% faster than running sums;
            // FP64 storage keeps the running sums, 0.2% faster there)
            double bs = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
            if constexpr (REF) {
                double v[NV];
#pragma unroll
                for (int i = 0; i < NV; i++) v[i] = double(f[i]);
                double sp[9], dp[9];
#pragma unroll
                for (int k = 0; k < 9; k++) {
                    sp[k] = v[2 * k + 1] + v[2 * k + 2];
                    dp[k] = v[2 * k + 1] - v[2 * k + 2];
                }
                bs = ((v[0] + (sp[0] + sp[1])) + ((sp[2] + sp[3]) + (sp[4] + sp[5])))
                   + ((sp[6] + sp[7]) + sp[8]);
                jx = ((dp[0] + dp[3]) + (dp[4] + dp[5])) + dp[6];
                jy = ((dp[1] + dp[3]) - dp[4]) + (dp[7] + dp[8]);
                jz = ((dp[2] + dp[5]) - dp[6]) + (dp[7] - dp[8]);
            } else {
#pragma unroll
                for (int i = 0; i < NV; i++) {
                    const double v = double(f[i]);
                    bs += v;
                    if (CX[i]) jx += CX[i] * v;
                    if (CY[i]) jy += CY[i] * v;
                    if (CZ[i]) jz += CZ[i] * v;
                }
            }
            if (counted) {
                acc[0] += DEV ? p.rho0 + bs : bs;
                acc[1] += c;
                acc[2] += jx;
                acc[3] += jy;
                acc[4] += jz;
            }
        }
        if (COLL) collide<T, DEV, REF, G1>(p, f, g, st);
        const O pso = pbase(x);
        const unsigned so = row.o[1][1];
#pragma unroll
        for (int i = 0; i < NV; i++) {
            stc<SMALL, NT>(dF, pso, i, compb, so, f[i]);
            const T gi = REF ? to_dest_ref(i, g[i], c,
                                           ph[psl[1 + CX[i]]][nbr(o, CY[i], CZ[i])])
                             : g[i];
            stc<SMALL, NT>(dG, pso, i, compb, so, gi);
        }
        // FP32: the new level's reference field; phi of the source level,
        // if asked for
        if (REF) dphic[pcbase(x) + rowsite] = phic_word(c);
        if (phi_out) phi_out[unsigned(x * plane) + rowsite] = c;
    };

    // Software-pipelined march (full tiles): the loads of plane x+2's g
    // (interior and ring) and phi_c and of plane x+1's f are issued before
    // plane x's collision and stores and consumed one iteration later, so
    // the workgroup keeps them in flight across its arithmetic and stores.
    // The path is branch-free -- every lane of a full tile is a site, the
    // ring cells are spread evenly over all waves (spare lanes repeat a cell
    // of their wave), the last iteration's prefetch of planes beyond the
    // segment is issued and left unused -- so the compiler's completion waits
    // follow the issue order exactly: each wait covers loads issued a whole
    // iteration earlier, never the stores issued since.
    const bool full = FLAT || (tya == TY && tza == TW);
    if (PIPE && full) {
        constexpr int NW = kFused / 64;
        // ring cells per wave (at most 64)
        const int RPW = FLAT ? (nring + NW - 1) / NW : (2 * TW + 2 * TY + 4 + NW - 1) / NW;
        const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
        int qli, qy, qz;
        ring_cell(min(w * RPW + (lane < RPW ? lane : 0), nring - 1), qli, qy, qz);
        const Yz9 qrow = yz9<T>(p, qy, qz);
        const unsigned qsite = unsigned(qy * p.nz + qz);

        T fq[NV], fc[NV];
        K gq[NV], rq[NV], kn[NV], kcur[NV];
        unsigned pq = 0, rpq = 0, pcn = 0, pccur = 0;
        // g and phi_c of plane X+1 (interior, ring); f(X)
        auto issue = [&](int X) __attribute__((always_inline)) {
            const O pf[3] = {pbase(X - 1), pbase(X), pbase(X + 1)};
            const O pg[3] = {pf[1], pf[2], pbase(X + 2)};
            // issue order fixed (scheduling barriers): interior g, ring g,
            // f -- the order in which the next iteration consumes them
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NV; i++)
                gq[i] = K(ldc<SMALL>(sG, pg[1 - CX[i]], i, compb, row.o[1 - CY[i]][1 - CZ[i]]));
            if (REF) pq = sphic[pcbase(X + 1) + rowsite];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NV; i++)
                rq[i] = K(ldc<SMALL>(sG, pg[1 - CX[i]], i, compb, qrow.o[1 - CY[i]][1 - CZ[i]]));
            if (REF) rpq = sphic[pcbase(X + 1) + qsite];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NV; i++)
                fq[i] = ldc<SMALL>(sF, pf[1 - CX[i]], i, compb, row.o[1 - CY[i]][1 - CZ[i]]);
            __builtin_amdgcn_sched_barrier(0);
        };
        put(0, own, pull_phi(x0 - 1, row, rowsite, nullptr, nullptr));
        put(0, qli, pull_phi(x0 - 1, qrow, qsite, nullptr, nullptr));
        put(1, own, pull_phi(x0, row, rowsite, kcur, &pccur));
        put(1, qli, pull_phi(x0, qrow, qsite, nullptr, nullptr));
        issue(x0);
        // enter the loop with these loads completed (an empty asm reading
        // each register makes the compiler wait for it here): the waits at
        // the loop's top then follow its steady state -- loads issued an
        // iteration ago, stores issued since -- not this entry path
#pragma unroll
        for (int i = 0; i < NV; i++) asm volatile("" ::"v"(gq[i]), "v"(rq[i]), "v"(fq[i]));
        asm volatile("" ::"v"(pq), "v"(rpq));
        for (int x = x0; x < x1; x++) {
            const int kk = x - x0 + 2;  // phi slot counter of plane x+1
            const int sn = kk & 3, sc = (kk - 1) & 3, sp = (kk - 2) & 3;
            // phi of plane x+1 from the loads issued one iteration ago, in
            // the index order every kernel uses
            double a = 0.0, b = 0.0;
#pragma unroll
            for (int i = 0; i < NV; i++) a += double(gq[i]);
            put(sn, own, REF ? phic_value(pq) + a : a);
#pragma unroll
            for (int i = 0; i < NV; i++) b += double(rq[i]);
            put(sn, qli, REF ? phic_value(rpq) + b : b);
            lds_barrier();
#pragma unroll
            for (int i = 0; i < NV; i++) {
                fc[i] = vcopy(fq[i]);
                kn[i] = vcopy(gq[i]);
            }
            pcn = vcopy(pq);
            issue(x + 1);
            update(x, fc, kcur, pccur, sp, sc, sn);
#pragma unroll
            for (int i = 0; i < NV; i++) kcur[i] = kn[i];
            pccur = pcn;
        }
    } else {
        // Plain march (FP64, and FP32 ragged row tiles), with the f pull of
        // plane x+1 issued before plane x's collision so that those loads
        // are in flight across its arithmetic and stores.  The registers for
        // them come from parking the kept g values of plane x+1 in LDS (each
        // thread its own slots) between their pull and their collision one
        // iteration later; measured in FP64 at 256^3: 4% faster, now within
        // 1% of the memory-only twin.
        K kcur[NV], knext[NV];
        __shared__ K kst[NV][kFused];
        unsigned pccur = 0, pcnext = 0;
        // warm-up: phi at planes x0-1 (slot 0) and x0 (slot 1), keeping
        // plane x0's populations
        if (active) put(0, own, pull_phi(x0 - 1, row, rowsite, nullptr, nullptr));
        if (ring) put(0, rli, pull_phi(x0 - 1, rrow, rsite, nullptr, nullptr));
        if (active) put(1, own, pull_phi(x0, row, rowsite, kcur, &pccur));
        if (ring) put(1, rli, pull_phi(x0, rrow, rsite, nullptr, nullptr));
        T fn[NV];
        auto pull_f = [&](int X) __attribute__((always_inline)) {
            const O pbx[3] = {pbase(X - 1), pbase(X), pbase(X + 1)};
#pragma unroll
            for (int i = 0; i < NV; i++)
                fn[i] = ldc<SMALL>(sF, pbx[1 - CX[i]], i, compb, row.o[1 - CY[i]][1 - CZ[i]]);
        };
        if (active) pull_f(x0);
        for (int x = x0; x < x1; x++) {
            const int kk = x - x0 + 2;  // phi slot counter of plane x+1
            const int sn = kk & 3, sc = (kk - 1) & 3, sp = (kk - 2) & 3;
            T f[NV];
            if (active) {
                put(sn, own, pull_phi(x + 1, row, rowsite, knext, &pcnext));
#pragma unroll
                for (int i = 0; i < NV; i++) kst[i][threadIdx.x] = knext[i];
            }
            if (ring) put(sn, rli, pull_phi(x + 1, rrow, rsite, nullptr, nullptr));
            lds_barrier();
            if (active) {
#pragma unroll
                for (int i = 0; i < NV; i++) f[i] = vcopy(fn[i]);
                if (x + 1 < x1) pull_f(x + 1);
                update(x, f, kcur, pccur, sp, sc, sn);
#pragma unroll
                for (int i = 0; i < NV; i++) kcur[i] = kst[i][threadIdx.x];
                pccur = pcnext;
            }
        }
    }
    if (partials) block_partials<5, kFused>(acc, partials);
}

// The marching kernel of a storage type (or, coll = false, its free-streaming
// twin) for an offset width (small: regions under 4 GiB), a tile width and
// the kind of stores.
template <typename T>
struct Fused;

// k_step_2s of a storage type by what it reduces and its block.
template <typename T, bool G1, int COMPACT>
decltype(&k_step_2s<T, false, false, G1, 0, COMPACT>) pick_2s(bool sums, int nb)
{
    constexpr bool F32 = std::is_same<T, float>::value;
    if (!sums) return k_step_2s<T, F32, F32, G1, 0, COMPACT>;
    return nb == kBlock ? k_step_2s<T, F32, F32, G1, kBlock, COMPACT>
                        : k_step_2s<T, F32, F32, G1, 64, COMPACT>;
}

// The step of one storage precision.  variant: 0 march, 1 two passes (phi64:
// the phi field between them), 2 the march's free-streaming twin.
template <typename T>
hipError_t launch_step_t(const KParams& p, const TileCfg& tc, int variant, int compact,
                         const void* src, void* dst, double* phi64, double* partials,
                         double* phi_src_out, hipStream_t s)
{
    constexpr bool F32 = std::is_same<T, float>::value;
    constexpr bool CAN_G1 = !F32;
    Lvl<T> a = level<T>(const_cast<void*>(src), p, F32);
    Lvl<T> d = level<T>(dst, p, F32);
    const bool g1 = CAN_G1 && p.omega_g == 1.0;
    if (variant == kStepBox) {
        return launch_box_t<T, CAN_G1, false>(p, g1, src, dst, phi_src_out, partials, s);
    } else if (variant == 1) {
        const int nb = site_block(p);
        auto k = compact == 2   ? pick_2s<T, CAN_G1, CAN_G1 ? 2 : 0>(partials, nb)
                 : compact == 1 ? pick_2s<T, CAN_G1, CAN_G1 ? 1 : 0>(partials, nb)
                 : g1           ? pick_2s<T, CAN_G1, 0>(partials, nb)
                                : pick_2s<T, false, 0>(partials, nb);
        k<<<collide_grid(p, partials), nb, 0, s>>>(p, a.F, a.G, a.phic, phi64, d.F, d.G, partials);
    } else {
        const bool small = size_t(NV) * p.stride * sizeof(T) < (size_t(1) << 32);
        auto k = Fused<T>::get(small, tc.tz, variant == 0, g1, march_nt(p, 2 * NV, sizeof(T), 144));
        k<<<tc.ntiles * tc.nseg, kFused, 0, s>>>(p, tc, a.F, a.G, a.phic, d.F, d.G, d.phic,
                                                 phi_src_out, partials);
    }
    return hipGetLastError();
}

// next (may be null): the level a step makes, whose phi_c the pass stores.
template <typename T>
hipError_t launch_phi_t(const KParams& p, const void* state, double* phi, void* next,
                        hipStream_t s)
{
    constexpr bool F32 = std::is_same<T, float>::value;
    Lvl<T> a = level<T>(const_cast<void*>(state), p, F32);
    unsigned* dphic = next ? level<T>(next, p, F32).phic : nullptr;
    const int nb = site_block(p);
    k_phi<T, F32><<<(p.nsites + nb - 1) / nb, nb, 0, s>>>(p, a.G, a.phic, phi, dphic);
    return hipGetLastError();
}

}  // namespace
}  // namespace lbk
