// The LB-scheme step kernels (lb_step.h) in FP32 storage.  Their forms round
// alike with the compiler's own floating-point contraction (the tests compare
// them bit for bit).
#include "lb_step.h"

namespace lbk {
namespace {

template <bool SMALL, int TZ, bool COLL, bool NT>
__global__ __launch_bounds__(kFused) void k_step_fused_f32(
    KParams p, TileCfg tc, const float* __restrict__ sF, const float* __restrict__ sG,
    const unsigned* __restrict__ sphic, float* __restrict__ dF, float* __restrict__ dG,
    unsigned* __restrict__ dphic, double* __restrict__ phi_out, double* __restrict__ partials)
{
    step_fused_body<float, true, true, SMALL, true, TZ, COLL, false, NT>(
        p, tc, sF, sG, sphic, dF, dG, dphic, phi_out, partials);
}

template <>
struct Fused<float> {
    using K = decltype(&k_step_fused_f32<true, 128, true, true>);
    template <bool SMALL, bool COLL, bool NT>
    static K tile(int tz)
    {
        if (tz == 0) return k_step_fused_f32<SMALL, 0, COLL, NT>;
        return tz == 64 ? k_step_fused_f32<SMALL, 64, COLL, NT>
                        : k_step_fused_f32<SMALL, 128, COLL, NT>;
    }
    template <bool SMALL, bool NT>
    static K coll(int tz, bool c)
    {
        return c ? tile<SMALL, true, NT>(tz) : tile<SMALL, false, NT>(tz);
    }
    static K get(bool small, int tz, bool c, bool, bool nt)
    {
        if (small) return nt ? coll<true, true>(tz, c) : coll<true, false>(tz, c);
        return nt ? coll<false, true>(tz, c) : coll<false, false>(tz, c);
    }
};

}  // namespace

hipError_t launch_step_f32(const KParams& p, const TileCfg& tc, int variant, int compact,
                           const void* src, void* dst, double* phi64, double* partials,
                           double* phi_src_out, hipStream_t s)
{
    return launch_step_t<float>(p, tc, variant, compact, src, dst, phi64, partials, phi_src_out, s);
}

hipError_t launch_phi_f32(const KParams& p, const void* state, double* phi, void* next,
                          hipStream_t s)
{
    return launch_phi_t<float>(p, state, phi, next, s);
}

}  // namespace lbk
