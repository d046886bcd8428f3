// Instantiations of the step and consensus kernels for bf16 parameter storage (float32 arithmetic).
#include "kernels.hpp"

namespace fgd {

bool kernels_bf16(int M, int k1, int k2, bool subset, KernelSet *out) {
    return exact_workers(M) ? select_exact<StepSets<ParamBF16>>(M, out, k1, k2, subset)
                            : kernels_bf16_class(M, k1, k2, subset, out);
}

}  // namespace fgd
