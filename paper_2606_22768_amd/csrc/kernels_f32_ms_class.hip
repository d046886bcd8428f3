// Step kernels of the worker classes (M no power of two) for float32
// parameter storage that also apply Mix1 to the optimizer state (Appendix B,
// GlobalM1S variants).
#include "kernels.hpp"

namespace fgd {

bool kernels_f32_ms_class(int M, int k1, int k2, bool subset, KernelSet *out) {
    return select_class<StateStepSets<ParamF32>>(M, out, k1, k2, subset);
}

}  // namespace fgd
