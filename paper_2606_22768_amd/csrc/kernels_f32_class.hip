// Step and consensus kernels of the worker classes (M no power of two) for
// float32 parameter storage.
#include "kernels.hpp"

namespace fgd {

bool kernels_f32_class(int M, int k1, int k2, bool subset, KernelSet *out) {
    return select_class<StepSets<ParamF32>>(M, out, k1, k2, subset);
}

}  // namespace fgd
