// The LB-scheme step of the smallest lattices in one launch (variant kStepBox;
// where it is taken, and what it measured: step_variant).
//
// A workgroup owns a box of 4 x 4 x 4 sites.  It forms phi of the box and of
// the cells around it that its stencils reach (one layer, with the force
// coupling two), a cell per thread, and hands it over in LDS; the box's own
// cells, which hold their g by then, collide.  Every form of the step rounds
// alike, so the levels are those of the other forms.  Bound by the chain from
// launch to store, which it has once where the two passes have it twice; it
// pulls g 3.4 times (with the force coupling 8 times).
#pragma once

#include "lb_device.h"

namespace lbk {

using namespace dev;

namespace {

constexpr int box_cells(int h) { return (kBox + 2 * h) * (kBox + 2 * h) * (kBox + 2 * h); }
constexpr int box_threads(int h) { return h == 1 ? 256 : 512; }
static_assert(box_cells(1) <= box_threads(1) && box_cells(2) <= box_threads(2), "a thread per cell");

// This thread's cell of its workgroup's box with H cells around it.
struct BoxCell {
    Geo q;
    int c;        // cell, z fastest
    bool own;     // a site of the box
    bool counts;  // and of no box before this one
};

template <int H>
__device__ __forceinline__ BoxCell box_cell(const KParams& p, const BoxCfg& bc)
{
    constexpr int BY = kBox + 2 * H, BX = BY * BY, NC = box_cells(H);
    const int b = xcd_block(), t = threadIdx.x;
    const int bz = b % bc.nbz, by = b / bc.nbz % bc.nby, bx = b / (bc.nbz * bc.nby);
    // the last boxes along each axis are shifted back to end with it
    const int ex = min(p.nx, kBox), ey = min(p.ny, kBox), ez = min(p.nz, kBox);
    const int x0 = min(bx * kBox, p.nx - ex), y0 = min(by * kBox, p.ny - ey),
              z0 = min(bz * kBox, p.nz - ez);
    BoxCell k;
    k.c = min(t, NC - 1);
    const int lx = k.c / BX - H, ly = k.c / BY % BY - H, lz = k.c % BY - H;
    k.own = t < NC && lx >= 0 && lx < ex && ly >= 0 && ly < ey && lz >= 0 && lz < ez;
    k.counts = k.own && x0 + lx >= bx * kBox && y0 + ly >= by * kBox && z0 + lz >= bz * kBox;
    k.q = geo_xyz(p, wrap_any(x0 + lx, p.nx), wrap_any(y0 + ly, p.ny), wrap_any(z0 + lz, p.nz));
    return k;
}

// F = -div Pi at cell c of a box of phi, as force_from_phi forms it.
template <int BX, int BY>
__device__ __forceinline__ void force_in_box(const KParams& p, const double* phi, int c, double F[3])
{
    // component of Pi_ab in the xx, xy, xz, yy, yz, zz storage
    constexpr int K[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
    constexpr int OFF[3] = {BX, BY, 1};
    auto pi = [&](int n, double t[6]) {
        double mu;
        chem_stress(p, stencil(phi[n], phi[n + BX], phi[n - BX], phi[n + BY], phi[n - BY],
                               phi[n + 1], phi[n - 1]), &mu, t);
    };
    double div[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < 3; b++) {
        double tp[6], tm[6];
        pi(c + OFF[b], tp);
        pi(c - OFF[b], tm);
#pragma unroll
        for (int a = 0; a < 3; a++) div[a] += 0.5 * (tp[K[a][b]] - tm[K[a][b]]);
    }
#pragma unroll
    for (int a = 0; a < 3; a++) F[a] = -div[a];
}

template <typename T, bool DEV, bool REF, bool G1, bool FORCE, bool SUMS>
__global__ __launch_bounds__(box_threads(FORCE ? 2 : 1)) void k_step_box(
    KParams p, BoxCfg bc, const T* __restrict__ sF, const T* __restrict__ sG,
    const unsigned* __restrict__ sphic, T* __restrict__ dF, T* __restrict__ dG,
    unsigned* __restrict__ dphic, double* __restrict__ phi_out, double* __restrict__ partials)
{
    constexpr int H = FORCE ? 2 : 1, BY = kBox + 2 * H, BX = BY * BY;
    __shared__ double s_phi[box_cells(H)];
    const BoxCell k = box_cell<H>(p, bc);
    const Geo& q = k.q;
    const int c = k.c;
    T f[NV], g[NV];
#pragma unroll
    for (int i = 0; i < NV; i++) g[i] = sG[dist_pull(p, q, i)];
    const double pc = REF ? phic_value(sphic[phic_site(p, q.x, q.y, q.z)]) : 0.0;
    if (k.own)
#pragma unroll
        for (int i = 0; i < NV; i++) f[i] = sF[dist_pull(p, q, i)];
    // phi as pull_g forms it
    double sum = 0.0;
#pragma unroll
    for (int i = 0; i < NV; i++) sum += double(g[i]);
    const double v = REF ? pc + sum : sum;
    s_phi[c] = v;
    lds_barrier();
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (k.own) {
        if (phi_out) phi_out[site_of(p, q.x, q.y, q.z)] = v;
        if (REF) {
            if (!FORCE || !G1)
#pragma unroll
                for (int i = 0; i < NV; i++) g[i] = pre_collision_dev(i, g[i], v - pc);
            dphic[phic_site(p, q.x, q.y, q.z)] = phic_word(v);
        }
        if constexpr (FORCE) {
            const double lap = (s_phi[c + BX] + s_phi[c - BX] - 2.0 * v)
                             + (s_phi[c + BY] + s_phi[c - BY] - 2.0 * v)
                             + (s_phi[c + 1] + s_phi[c - 1] - 2.0 * v);
            const double mu = p.A * v + p.B * v * v * v - p.kappa * lap;
            double F[3];
            force_in_box<BX, BY>(p, s_phi, c, F);
            if (SUMS && k.counts) site_sums<DEV>(p, f, v, F, acc);
            collide_force<T, DEV, REF, G1>(p, f, g, v, mu, F);
        } else {
            const Stencil st = stencil(v, s_phi[c + BX], s_phi[c - BX], s_phi[c + BY],
                                       s_phi[c - BY], s_phi[c + 1], s_phi[c - 1]);
            if (SUMS && k.counts) site_sums<DEV>(p, f, v, nullptr, acc);
            collide<T, DEV, REF, G1>(p, f, g, st);
        }
#pragma unroll
        for (int i = 0; i < NV; i++) {
            dF[dist_own(p, q, i)] = f[i];
            dG[dist_own(p, q, i)] =
                REF ? to_dest_ref(i, g[i], v, s_phi[c + CX[i] * BX + CY[i] * BY + CZ[i]]) : g[i];
        }
    }
    if (SUMS) block_partials<5, box_threads(FORCE ? 2 : 1)>(acc, partials);
}

template <typename T, bool CAN_G1, bool FORCE>
hipError_t launch_box_t(const KParams& p, bool g1, const void* src, void* dst, double* phi_src_out,
                        double* partials, hipStream_t s)
{
    constexpr bool F32 = sizeof(T) == 4;
    Lvl<T> a = level<T>(const_cast<void*>(src), p, F32);
    Lvl<T> d = level<T>(dst, p, F32);
    const BoxCfg bc = box_cfg(p);
    auto k = g1 ? (partials ? k_step_box<T, F32, F32, CAN_G1, FORCE, true>
                            : k_step_box<T, F32, F32, CAN_G1, FORCE, false>)
                : (partials ? k_step_box<T, F32, F32, false, FORCE, true>
                            : k_step_box<T, F32, F32, false, FORCE, false>);
    k<<<bc.blocks(), box_threads(FORCE ? 2 : 1), 0, s>>>(p, bc, a.F, a.G, a.phic, d.F, d.G, d.phic,
                                                 phi_src_out, partials);
    return hipGetLastError();
}

}  // namespace
}  // namespace lbk
