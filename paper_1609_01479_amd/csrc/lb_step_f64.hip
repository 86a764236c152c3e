// The LB-scheme step kernels (lb_step.h) in FP64.  Floating-point contraction
// within one source expression only, so that every form of the step rounds
// every expression alike: the compiler's default also fuses across
// statements, and did so differently in different kernels.
#pragma clang fp contract(on)

#include "lb_step.h"

namespace lbk {
namespace {

template <bool SMALL, int TZ, bool COLL, bool G1, bool NT>
__global__ __launch_bounds__(kFused) void k_step_fused_f64(
    KParams p, TileCfg tc, const double* __restrict__ sF, const double* __restrict__ sG,
    const unsigned* __restrict__ sphic, double* __restrict__ dF, double* __restrict__ dG,
    unsigned* __restrict__ dphic, double* __restrict__ phi_out, double* __restrict__ partials)
{
    step_fused_body<double, false, false, SMALL, false, TZ, COLL, G1, NT>(
        p, tc, sF, sG, sphic, dF, dG, dphic, phi_out, partials);
}

template <>
struct Fused<double> {
    using K = decltype(&k_step_fused_f64<true, 128, true, false, true>);
    template <bool SMALL, bool COLL, bool G1, bool NT>
    static K tile(int tz)
    {
        if (tz == 0) return k_step_fused_f64<SMALL, 0, COLL, G1, NT>;
        return tz == 64 ? k_step_fused_f64<SMALL, 64, COLL, G1, NT>
                        : k_step_fused_f64<SMALL, 128, COLL, G1, NT>;
    }
    template <bool SMALL, bool NT>
    static K coll(int tz, bool c, bool g1)
    {
        if (!c) return tile<SMALL, false, false, NT>(tz);
        return g1 ? tile<SMALL, true, true, NT>(tz) : tile<SMALL, true, false, NT>(tz);
    }
    static K get(bool small, int tz, bool c, bool g1, bool nt)
    {
        if (small) return nt ? coll<true, true>(tz, c, g1) : coll<true, false>(tz, c, g1);
        return nt ? coll<false, true>(tz, c, g1) : coll<false, false>(tz, c, g1);
    }
};

}  // namespace

hipError_t launch_step_f64(const KParams& p, const TileCfg& tc, int variant, int compact,
                           const void* src, void* dst, double* phi64, double* partials,
                           double* phi_src_out, hipStream_t s)
{
    return launch_step_t<double>(p, tc, variant, compact, src, dst, phi64, partials, phi_src_out, s);
}

hipError_t launch_phi_f64(const KParams& p, const void* state, double* phi, void* next,
                          hipStream_t s)
{
    return launch_phi_t<double>(p, state, phi, next, s);
}

hipError_t launch_phi_compact_f64(const KParams& p, const void* state, const double* cphi,
                                  double* phi, hipStream_t s)
{
    return launch_phi_compact_t<double, false>(p, state, cphi, phi, nullptr, s);
}

hipError_t launch_step_compact_f64(const KParams& p, const void* src, void* dst, bool to_full,
                                   const double* phi, double* partials, hipStream_t s)
{
    return launch_step_compact_t<double, false>(p, src, dst, to_full, phi, partials, s);
}

hipError_t launch_full_level_f64(const KParams& p, bool moments, const void* src, void* dst,
                                 hipStream_t s)
{
    return launch_full_level_t<double, false>(p, moments, src, dst, s);
}

}  // namespace lbk
