// Step kernels of the worker classes (M no power of two) for bf16 parameter
// storage (float32 arithmetic) that also apply Mix1 to the optimizer state
// (Appendix B, GlobalM1S variants).
#include "kernels.hpp"

namespace fgd {

bool kernels_bf16_ms_class(int M, int k1, int k2, bool subset, KernelSet *out) {
    return select_class<StateStepSets<ParamBF16>>(M, out, k1, k2, subset);
}

}  // namespace fgd
