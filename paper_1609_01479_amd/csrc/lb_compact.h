// Compact levels between the steps of one call, for omega_g = 1 (tau_g = 1).
//
// There g* = g^eq, a function of phi, mu and u of the site that collided: a
// step that is followed by another in the same call leaves these five numbers
// instead of the 19 populations, in the place of the level's g region (phi:
// stride FP64 values, then mu, u_x, u_y, u_z of each site together), and the
// next step's phi pass forms each population it pulls from its origin's five,
// by the expressions that collide_g and collide_force_g store it with, so
// every phi and every f is bit for bit that of full levels.  f stays as it is.
// The levels that a call starts from and leaves are full.  Per site and step
// that is 392 bytes instead of 608 in FP64 (and 208 of 312 in FP32 storage
// with the force coupling): two passes, the first over five fields.
//
// With omega_f = 1 too, f* is f^eq, and ten moments take the place of its 19
// populations: 248 bytes (FP32 storage 136).
//
// us per step, full / g compact / both: FP64 stress 90 x 75 x 100 86 / 49 /
// 42, 128^3 248 / 162 / 126, 256^3 1830 / 1309 / 982; FP64 force 128^3 274 /
// 188 / 174, 256^3 2083 / 1471 / 1345; FP32 force 128^3 161 / 126 / 106,
// 256^3 1153 / 984.
#pragma once

#include "lb_device.h"

namespace lbk {

using namespace dev;

template <typename T>
struct alignas(4 * sizeof(T) < 16 ? 4 * sizeof(T) : 16) MuU {
    T mu, ux, uy, uz;
};

template <typename T>
__host__ __device__ inline double* compact_phi(T* G) { return reinterpret_cast<double*>(G); }
template <typename T>
__host__ __device__ inline MuU<T>* compact_mu_u(T* G, const KParams& p)
{
    return reinterpret_cast<MuU<T>*>(compact_phi(G) + p.stride);
}

// Two of f^eq's moments of a site; five fields of them in the level's f region.
template <typename T>
struct alignas(2 * sizeof(T)) Pair {
    T a, b;
};

namespace {

template <typename T>
__device__ __forceinline__ FEq<T> load_feq(const KParams& p, const T* __restrict__ F, int s)
{
    const Pair<T>* q = reinterpret_cast<const Pair<T>*>(F) + s;
    const size_t n = p.stride;
    const Pair<T> v0 = q[0], v1 = q[n], v2 = q[2 * n], v3 = q[3 * n], v4 = q[4 * n];
    return FEq<T>{v0.a, v0.b, v1.a, v1.b, v2.a, v2.b, v3.a, v3.b, v4.a, v4.b};
}

template <typename T>
__device__ __forceinline__ void store_feq(const KParams& p, T* __restrict__ F, int s, const FEq<T>& e)
{
    Pair<T>* q = reinterpret_cast<Pair<T>*>(F) + s;
    const size_t n = p.stride;
    q[0] = Pair<T>{e.b, e.ax};
    q[n] = Pair<T>{e.ay, e.az};
    q[2 * n] = Pair<T>{e.xx, e.yy};
    q[3 * n] = Pair<T>{e.zz, e.xy};
    q[4 * n] = Pair<T>{e.xz, e.yz};
}

// g*_i of a site (FP32 mode: its deviation h*) as collide_g<T, REF, true>
// forms it (the same expressions, so that each rounds alike).
template <typename T, bool REF>
__device__ __forceinline__ T geq_stress(const KParams& p, int i, T phi, MuU<T> m)
{
    const T gam = T(p.gamma), mu = m.mu;
    const T ux = m.ux, uy = m.uy, uz = m.uz;
    const T h = T(4.5);
    const T w0 = T(weight(0)), wf = T(weight(1)), we = T(weight(7));
    const T wf3 = T(3.0 * weight(1)), we3 = T(3.0 * weight(7));
    const T uu3 = (ux * ux + uy * uy + uz * uz) * T(1.0 / 3.0);
    const T hp = h * phi;
    static_assert(!REF, "FP32 storage adds g - g to g^eq in the stress coupling");
    const T sg = gam * mu - phi * T(1.0 / 3.0);
    if (i == 0) return w0 * (phi - h * sg - hp * uu3);
    const int odd = i & 1;
    if (i < 7) {
        const T ef = phi - hp * uu3;
        const T p3f = wf3 * phi;
        const T v = i < 3 ? ux : (i < 5 ? uy : uz);
        const T sx = wf * (ef + hp * v * v);
        return odd ? sx + p3f * v : sx - p3f * v;
    }
    const T ee = phi + h * sg - hp * uu3;
    const T p3e = we3 * phi;
    const T c = i < 9 ? ux + uy : i < 11 ? ux - uy : i < 13 ? ux + uz : i < 15 ? ux - uz
              : i < 17 ? uy + uz : uy - uz;
    const T s = we * (ee + hp * c * c);
    return odd ? s + p3e * c : s - p3e * c;
}

// The same as collide_force_g<T, REF, true>.
template <typename T, bool REF>
__device__ __forceinline__ T geq_force(const KParams& p, int i, T phi, MuU<T> m)
{
    const T mu = m.mu, ux = m.ux, uy = m.uy, uz = m.uz;
    const T uu3 = (ux * ux + uy * uy + uz * uz) * T(1.0 / 3.0);
    const T gm = T(p.gamma) * mu, sg = REF ? gm : gm - phi * T(1.0 / 3.0);
    const T w = T(weight(i));
    const T cu = T(CX[i]) * ux + T(CY[i]) * uy + T(CZ[i]) * uz;
    const T q = cu * cu - uu3;
    const T c2m1 = T(CX[i] * CX[i] + CY[i] * CY[i] + CZ[i] * CZ[i] - 1);
    return w * ((REF ? T(0) : phi) + T(3) * phi * cu + T(4.5) * (sg * c2m1 + phi * q));
}

// phi of a compact level at every site (phi_at of the full one); with dphic
// (FP32 mode) also the reference field phi_c of the level the step makes.
template <typename T, bool REF, bool FORCE>
__global__ __launch_bounds__(kBlock) void k_phi_compact(KParams p, const double* __restrict__ cphi,
                                                        const MuU<T>* __restrict__ mu_u,
                                                        double* __restrict__ phi,
                                                        unsigned* __restrict__ dphic)
{
    const int s = xcd_block() * int(blockDim.x) + threadIdx.x;
    if (s >= p.nsites) return;
    const Geo q = geo_of(p, s);
    const double pc = REF ? phic_round(cphi[s]) : 0.0;
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int y = pull_site(p, q, i);
        const double ph = cphi[y];
        const MuU<T> m = mu_u[y];
        T g;
        if constexpr (FORCE)
            g = geq_force<T, REF>(p, i, T(ph), m);
        else
            g = geq_stress<T, REF>(p, i, T(ph), m);
        acc += double(REF ? T(__builtin_fma(rweight(i), ph - pc, double(g))) : g);
    }
    const double v = REF ? pc + acc : acc;
    phi[s] = v;
    if (REF && dphic) dphic[phic_site(p, q.x, q.y, q.z)] = phic_word(v);
}

// LDS of a cell: the 16 populations that leave its column (FP32 mode: their
// deviations, and the phi of the cell).
template <typename T, bool REF, int NC>
struct CompactLds {
    T g[NV - 3][NC];
    double phi[REF ? NC : 1];
};

// A pulled population: FP64 its value, FP32 mode its deviation and the phi of
// its origin, until the reference of the site it arrives at is known.
template <typename T, bool REF>
struct Pulled {
    T h;
    double ph;
    __device__ __forceinline__ double at(int i, double pc) const
    {
        return REF ? double(T(__builtin_fma(rweight(i), ph - pc, double(h)))) : double(h);
    }
};

// k_phi_compact as a march along x.  One site per thread reads five values
// from each of 19 sites, 760 bytes in FP64, and is bound by the caches that
// serve them (256^3 620 us, for 48 bytes per site from memory).  Here a
// workgroup owns a tile of TY x TZ columns over a segment of planes, one
// thread per cell of the tile and the ring around it.  Each cell's populations
// are formed once and handed to their destinations through LDS; those that
// leave for the planes on either side wait in the destination's registers.
// Bound by its arithmetic and LDS traffic together, with 8 waves between two
// barriers: 256^3 239 us.
template <typename T, bool REF, bool FORCE>
__global__ __launch_bounds__(kCompactThreads) void k_phi_compact_march(
    KParams p, int nty, int ntz, int sx, const double* __restrict__ cphi,
    const MuU<T>* __restrict__ mu_u, double* __restrict__ phi, unsigned* __restrict__ dphic)
{
    constexpr int TY = kCompactTY, TZ = kCompactTZ, BZ = TZ + 2, NC = (TY + 2) * BZ;
    __shared__ CompactLds<T, REF, NC> lds;
    const int blk = xcd_block();
    const int tile = blk % (nty * ntz), seg = blk / (nty * ntz);
    // the last tiles of a plane are shifted back to end with it
    const int ey = p.ny < TY ? p.ny : TY, ez = p.nz < TZ ? p.nz : TZ;
    const int y0 = min(tile / ntz * TY, p.ny - ey), z0 = min(tile % ntz * TZ, p.nz - ez);
    const int x0 = seg * sx, x1 = min(x0 + sx, p.nx);
    const int c = threadIdx.x, r = c / BZ, l = c - r * BZ;
    const bool cell = c < NC;
    const bool own = cell && r >= 1 && r <= ey && l >= 1 && l <= ez;
    const int y = wrap_any(y0 + r - 1, p.ny), z = wrap_any(z0 + l - 1, p.nz);
    const int col = y * p.nz + z, plane = p.ny * p.nz;
    double ph = 0.0, below = 0.0;  // phi of this plane's cell and of the one before
    MuU<T> m{};
    {
        const int s = (x0 == 0 ? p.nx - 1 : x0 - 1) * plane + col;
        if (cell) {
            ph = cphi[s];
            m = mu_u[s];
        }
    }
    Pulled<T, REF> up[2][5], mid[9];
    constexpr int UP[5] = {1, 7, 9, 11, 13};
    constexpr int MID[9] = {0, 3, 4, 5, 6, 15, 16, 17, 18};
    for (int X = x0 - 1; X <= x1; X++) {
        T g[NV];
        const double here = ph;
        if constexpr (FORCE)
            collide_force_g<T, REF, true>(p, g, ph, double(m.mu), Vel<T>{m.ux, m.uy, m.uz});
        else
            collide_g<T, REF, true>(p, g, T(ph), m.mu, Vel<T>{m.ux, m.uy, m.uz});
        if (cell) {
#pragma unroll
            for (int i = 3; i < NV; i++) lds.g[i - 3][c] = g[i];
            if (REF) lds.phi[c] = here;
        }
        if (cell && X < x1) {  // the next plane, while this one is exchanged
            const int s = (X + 1 >= p.nx ? X + 1 - p.nx : X + 1) * plane + col;
            ph = cphi[s];
            m = mu_u[s];
        }
        lds_barrier();
        if (own) {
            auto pull = [&](int i) {
                const int o = c - (CY[i] * BZ + CZ[i]);
                return Pulled<T, REF>{lds.g[i - 3][o], REF ? lds.phi[o] : 0.0};
            };
            Pulled<T, REF> down[5];
            down[0] = Pulled<T, REF>{g[2], here};
#pragma unroll
            for (int k = 1; k < 5; k++) down[k] = pull(UP[k] + 1);
            if (X > x0) {
                const double pc = REF ? phic_round(below) : 0.0;
                double acc = 0.0;
                acc += mid[0].at(0, pc);
                acc += up[0][0].at(1, pc);
                acc += down[0].at(2, pc);
#pragma unroll
                for (int k = 1; k < 5; k++) acc += mid[k].at(MID[k], pc);
#pragma unroll
                for (int k = 1; k < 5; k++) {
                    acc += up[0][k].at(UP[k], pc);
                    acc += down[k].at(UP[k] + 1, pc);
                }
#pragma unroll
                for (int k = 5; k < 9; k++) acc += mid[k].at(MID[k], pc);
                const double v = REF ? pc + acc : acc;
                const int s = (X - 1) * plane + col;
                phi[s] = v;
                if (REF && dphic) dphic[phic_site(p, X - 1, y, z)] = phic_word(v);
            }
            mid[0] = Pulled<T, REF>{g[0], here};
#pragma unroll
            for (int k = 1; k < 9; k++) mid[k] = pull(MID[k]);
#pragma unroll
            for (int k = 0; k < 5; k++) {
                up[0][k] = up[1][k];
                up[1][k] = k ? pull(UP[k]) : Pulled<T, REF>{g[1], here};
            }
            below = here;
        }
        lds_barrier();
    }
}

// The collision pass from a compact level with f's moments, as a march of
// k_phi_compact_march's tiles: each cell's f is formed once from its ten
// moments and handed over in LDS (one site per thread would read ten values
// from each of 19 sites).  Bound by memory where two workgroups share a CU
// (256^3 FP64, 200 bytes per site: 743 us, 4.5 TB/s; the pass it replaces
// 1073), with the force coupling by the chain of one.  TO_FULL: the new level
// is full.  SUMS: block partials of the source level's conserved sums.
template <typename T, bool DEV, bool REF, bool FORCE, bool TO_FULL, bool SUMS>
__global__ __launch_bounds__(kCompactThreads) void k_step_compact_march(
    KParams p, int nty, int ntz, int sx, const T* __restrict__ sF, const double* __restrict__ phi,
    T* __restrict__ dF, T* __restrict__ dG, double* __restrict__ partials)
{
    constexpr int TY = kCompactTY, TZ = kCompactTZ, BZ = TZ + 2, NC = (TY + 2) * BZ;
    __shared__ T lds[NV - 3][NC];
    const int blk = xcd_block();
    const int tile = blk % (nty * ntz), seg = blk / (nty * ntz);
    // the last tiles of a plane are shifted back to end with it
    const int ey = p.ny < TY ? p.ny : TY, ez = p.nz < TZ ? p.nz : TZ;
    const int y0 = min(tile / ntz * TY, p.ny - ey), z0 = min(tile % ntz * TZ, p.nz - ez);
    const int x0 = seg * sx, x1 = min(x0 + sx, p.nx);
    const int c = threadIdx.x, r = c / BZ, l = c - r * BZ;
    const bool cell = c < NC;
    const bool own = cell && r >= 1 && r <= ey && l >= 1 && l <= ez;
    const int y = wrap_any(y0 + r - 1, p.ny), z = wrap_any(z0 + l - 1, p.nz);
    const int col = y * p.nz + z, plane = p.ny * p.nz;
    // a site that two tiles share counts in the first one's sums
    const bool counts = own && y0 + r > tile / ntz * TY && z0 + l > tile % ntz * TZ;
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    FEq<T> e{};
    if (cell) e = load_feq(p, sF, (x0 == 0 ? p.nx - 1 : x0 - 1) * plane + col);
    T up[2][5], mid[9];
    constexpr int UP[5] = {1, 7, 9, 11, 13};
    constexpr int MID[9] = {0, 3, 4, 5, 6, 15, 16, 17, 18};
    for (int X = x0 - 1; X <= x1; X++) {
        T h[NV];
        hermite_f<T, !DEV && !FORCE>(e, h);
        if (cell) {
#pragma unroll
            for (int i = 3; i < NV; i++) lds[i - 3][c] = h[i];
        }
        if (cell && X < x1)  // the next plane, while this one is exchanged
            e = load_feq(p, sF, (X + 1 >= p.nx ? X + 1 - p.nx : X + 1) * plane + col);
        const bool here = own && X > x0;  // plane X - 1 is complete now
        Stencil st{};
        double F[3] = {0.0, 0.0, 0.0}, mu_d = 0.0;
        const Geo q = geo_xyz(p, X > x0 ? X - 1 : x0, y, z);
        if (here) {
            const double v = phi[site_of(p, q.x, q.y, q.z)];
            if constexpr (FORCE) {
                const double lap = (phi[site_of(p, q.xp, q.y, q.z)] + phi[site_of(p, q.xm, q.y, q.z)] - 2.0 * v)
                                 + (phi[site_of(p, q.x, q.yp, q.z)] + phi[site_of(p, q.x, q.ym, q.z)] - 2.0 * v)
                                 + (phi[site_of(p, q.x, q.y, q.zp)] + phi[site_of(p, q.x, q.y, q.zm)] - 2.0 * v);
                mu_d = p.A * v + p.B * v * v * v - p.kappa * lap;
                force_from_phi(p, q, phi, F);
                st.phi = v;
            } else {
                st = stencil(v, phi[site_of(p, q.xp, q.y, q.z)], phi[site_of(p, q.xm, q.y, q.z)],
                             phi[site_of(p, q.x, q.yp, q.z)], phi[site_of(p, q.x, q.ym, q.z)],
                             phi[site_of(p, q.x, q.y, q.zp)], phi[site_of(p, q.x, q.y, q.zm)]);
            }
        }
        lds_barrier();
        if (own) {
            auto pull = [&](int i) { return lds[i - 3][c - (CY[i] * BZ + CZ[i])]; };
            T down[5];
            down[0] = h[2];
#pragma unroll
            for (int k = 1; k < 5; k++) down[k] = pull(UP[k] + 1);
            if (here) {
                T f[NV];
                f[0] = mid[0];
#pragma unroll
                for (int k = 0; k < 5; k++) {
                    f[UP[k]] = up[0][k];
                    f[UP[k] + 1] = down[k];
                }
#pragma unroll
                for (int k = 1; k < 9; k++) f[MID[k]] = mid[k];
                if (SUMS && counts) site_sums<DEV>(p, f, st.phi, FORCE ? F : nullptr, acc);
                FEq<T> d;
                Vel<T> u;
                T mu;
                if constexpr (FORCE) {
                    u = feq_force<T, DEV>(p, f, F, d);
                    mu = T(mu_d);
                } else {
                    u = feq_stress<T, DEV>(p, f, st, d);
                    mu = chem_potential<T>(p, st);
                }
                if constexpr (TO_FULL) {
                    T g[NV];
                    hermite_f<T, !DEV && !FORCE>(d, f);
#pragma unroll
                    for (int i = 0; i < NV; i++) dF[dist_own(p, q, i)] = f[i];
                    if constexpr (FORCE)
                        collide_force_g<T, REF, true>(p, g, st.phi, mu_d, u);
                    else
                        collide_g<T, REF, true>(p, g, T(st.phi), mu, u);
#pragma unroll
                    for (int i = 0; i < NV; i++)
                        dG[dist_own(p, q, i)] =
                            REF ? to_dest_ref(i, g[i], st.phi, phi[push_site(p, q, i)]) : g[i];
                } else {
                    const int s = (X - 1) * plane + col;
                    store_feq(p, dF, s, d);
                    compact_mu_u(dG, p)[s] = MuU<T>{mu, u.x, u.y, u.z};
                }
            }
            mid[0] = h[0];
#pragma unroll
            for (int k = 1; k < 9; k++) mid[k] = pull(MID[k]);
#pragma unroll
            for (int k = 0; k < 5; k++) {
                up[0][k] = up[1][k];
                up[1][k] = k ? pull(UP[k]) : h[1];
            }
        }
        lds_barrier();
    }
    if (SUMS) block_partials<5, kCompactThreads>(acc, partials);
}

// The full level of a compact one, as the step that left it would have written
// it: one site per thread, bound by memory (once, when the buffers come to be
// shared).  MOMENTS: f as its ten moments.
template <typename T, bool REF, bool FORCE, bool MOMENTS>
__global__ __launch_bounds__(kBlock) void k_full_level(KParams p, const T* __restrict__ sF,
                                                       const double* __restrict__ cphi,
                                                       const MuU<T>* __restrict__ mu_u,
                                                       T* __restrict__ dF, T* __restrict__ dG,
                                                       unsigned* __restrict__ dphic)
{
    const int s = xcd_block() * int(blockDim.x) + threadIdx.x;
    if (s >= p.nsites) return;
    const Geo q = geo_of(p, s);
    T f[NV], g[NV];
    if constexpr (MOMENTS) {
        hermite_f<T, !REF && !FORCE>(load_feq(p, sF, s), f);
    } else {
#pragma unroll
        for (int i = 0; i < NV; i++) f[i] = sF[dist_own(p, q, i)];
    }
    const double ph = cphi[s];
    const MuU<T> m = mu_u[s];
    if constexpr (FORCE)
        collide_force_g<T, REF, true>(p, g, ph, double(m.mu), Vel<T>{m.ux, m.uy, m.uz});
    else
        collide_g<T, REF, true>(p, g, T(ph), m.mu, Vel<T>{m.ux, m.uy, m.uz});
#pragma unroll
    for (int i = 0; i < NV; i++) {
        dF[dist_own(p, q, i)] = f[i];
        dG[dist_own(p, q, i)] = REF ? to_dest_ref(i, g[i], ph, cphi[push_site(p, q, i)]) : g[i];
    }
    if (REF) dphic[phic_site(p, q.x, q.y, q.z)] = phic_word(ph);
}

// phi of the compact level `state`, its own phi field cphi if that is given;
// next (may be null): the level a step makes, whose phi_c the pass stores.
template <typename T, bool FORCE>
hipError_t launch_phi_compact_t(const KParams& p, const void* state, const double* cphi,
                                double* phi, void* next, hipStream_t s)
{
    constexpr bool F32 = sizeof(T) == 4;
    T* G = level<T>(const_cast<void*>(state), p, F32).G;
    if (!cphi) cphi = compact_phi(G);
    unsigned* dphic = next ? level<T>(next, p, F32).phic : nullptr;
    const CompactTiles t = compact_tiles(p, kCompactResident);
    if (compact_march(p, F32)) {
        k_phi_compact_march<T, F32, FORCE>
            <<<t.blocks(), kCompactThreads, 0, s>>>(
                p, t.nty, t.ntz, t.sx, cphi, compact_mu_u(G, p), phi, dphic);
    } else {
        const int nb = site_block(p);
        k_phi_compact<T, F32, FORCE><<<(p.nsites + nb - 1) / nb, nb, 0, s>>>(
            p, cphi, compact_mu_u(G, p), phi, dphic);
    }
    return hipGetLastError();
}

// A step's collision pass from the compact level src with f's moments; phi:
// that level's phi.
template <typename T, bool FORCE>
hipError_t launch_step_compact_t(const KParams& p, const void* src, void* dst, bool to_full,
                                 const double* phi, double* partials, hipStream_t s)
{
    constexpr bool F32 = sizeof(T) == 4;
    const T* F = level<T>(const_cast<void*>(src), p, F32).F;
    Lvl<T> d = level<T>(dst, p, F32);
    const CompactTiles t = compact_step_tiles(p, F32);
    auto k = partials ? to_full ? k_step_compact_march<T, F32, F32, FORCE, true, true>
                                : k_step_compact_march<T, F32, F32, FORCE, false, true>
             : to_full ? k_step_compact_march<T, F32, F32, FORCE, true, false>
                       : k_step_compact_march<T, F32, F32, FORCE, false, false>;
    k<<<t.blocks(), kCompactThreads, 0, s>>>(p, t.nty, t.ntz, t.sx, F, phi, d.F, d.G, partials);
    return hipGetLastError();
}

template <typename T, bool FORCE>
hipError_t launch_full_level_t(const KParams& p, bool moments, const void* src, void* dst,
                               hipStream_t s)
{
    constexpr bool F32 = sizeof(T) == 4;
    const Lvl<T> a = level<T>(const_cast<void*>(src), p, F32);
    const Lvl<T> d = level<T>(dst, p, F32);
    const int nb = site_block(p);
    auto k = moments ? k_full_level<T, F32, FORCE, true> : k_full_level<T, F32, FORCE, false>;
    k<<<(p.nsites + nb - 1) / nb, nb, 0, s>>>(p, a.F, compact_phi(a.G), compact_mu_u(a.G, p), d.F,
                                              d.G, d.phic);
    return hipGetLastError();
}

}  // namespace
}  // namespace lbk
