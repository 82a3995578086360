// The class gradient's adjoint (see ls_grad_class.h): FP64.
#include "ls_grad_class.h"

namespace lsk {

hipError_t launch_grad_class_f64(const GradArgs &ga, const GradClassArgs &a, int nslot, int nwaves,
                                 hipStream_t st) {
    return launch_grad_class_menu<PrecF64>(ga, a, nslot, nwaves, st);
}

}  // namespace lsk
