// Step kernels for float32 parameter storage that also apply Mix1 to the optimizer
// state (Appendix B, GlobalM1S variants).
#include "kernels.hpp"

namespace fgd {

bool kernels_f32_ms(int M, int k1, int k2, bool subset, KernelSet *out) {
    return exact_workers(M) ? select_exact<StateStepSets<ParamF32>>(M, out, k1, k2, subset)
                            : kernels_f32_ms_class(M, k1, k2, subset, out);
}

}  // namespace fgd
