// Instantiations of the step and consensus kernels for float32 parameter storage.
#include "kernels.hpp"

namespace fgd {

bool kernels_f32(int M, int k1, int k2, bool subset, KernelSet *out) {
    return exact_workers(M) ? select_exact<StepSets<ParamF32>>(M, out, k1, k2, subset)
                            : kernels_f32_class(M, k1, k2, subset, out);
}

}  // namespace fgd
