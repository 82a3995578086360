// Sweep kernels for one precision and direction (see ls_sweep.h).
#include "ls_sweep.h"

namespace lsk {

template <int NSLOT>
static hipError_t launch_one(const SweepPtrs &p, const SweepArgs &a, int nwaves, hipStream_t st) {
    using PT = PrecF32;
    const int vps = sweep_slot_vgprs(PT::vgpr_per_slot, p.prior != nullptr);
    if (nwaves < 1 || nwaves > max_waves_for(NSLOT, vps, p.prior != nullptr))
        return hipErrorInvalidValue;
    if (a.nblk < 1 || a.r0 < 0 || a.r0 + a.nblk > a.R) return hipErrorInvalidValue;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(a.nblk), dim3(64 * nwaves), 0, st, p.Hr,
                           (const PT::T *)p.emis, p.lu_prefix, p.prior, p.rho, p.coef, p.recipients,
                           (PT::ST *)p.state, p.log_scale, p.status, (PT::IO *)p.snap, a);
    };
    auto pick = [&](auto one) {
        constexpr bool ONE = decltype(one)::value;
        if (p.prior && p.emis) go(&sweep_kernel<PT, NSLOT, 0, false, true, true, ONE>);
        else if (p.prior) go(&sweep_kernel<PT, NSLOT, 0, false, false, true, ONE>);
        else if (p.emis) go(&sweep_kernel<PT, NSLOT, 0, false, true, false, ONE>);
        else go(&sweep_kernel<PT, NSLOT, 0, false, false, false, ONE>);
    };
    if constexpr (NSLOT <= kOneWaveSlots) {
        if (nwaves == 1) pick(std::true_type{});
        else pick(std::false_type{});
    } else {
        pick(std::false_type{});
    }
    return hipGetLastError();
}

hipError_t launch_sweep_f32_fwd(const SweepPtrs &p, const SweepArgs &a, Shape shape, hipStream_t st) {
    switch (shape.nslot) {
#define LS_CASE(n) \
    case n:        \
        return launch_one<n>(p, a, shape.nwaves, st);
        LS_MENU_F32(LS_CASE)
#undef LS_CASE
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace lsk
