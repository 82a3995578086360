// Class sweeps (see ls_csweep.h): FP32, group A of the donor-word menu.
#include "ls_csweep.h"

namespace lsk {

hipError_t launch_csweep_f32_a(const SweepPtrs &p, const ClassPtrs &c, const SweepArgs &a,
                                hipStream_t st) {
    switch (c.nslot) {
#define LS_CASE(n) \
    case n:        \
        return launch_csweep_slots<PrecF32, n>(p, c, a, st);
        LS_MENU_CSLOT_A(LS_CASE)
#undef LS_CASE
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace lsk
