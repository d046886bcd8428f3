// Step and consensus kernels of the worker classes (M no power of two) for
// bf16 parameter storage (float32 arithmetic).
#include "kernels.hpp"

namespace fgd {

bool kernels_bf16_class(int M, int k1, int k2, bool subset, KernelSet *out) {
    return select_class<StepSets<ParamBF16>>(M, out, k1, k2, subset);
}

}  // namespace fgd
