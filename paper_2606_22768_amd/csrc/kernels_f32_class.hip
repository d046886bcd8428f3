// The worker classes' instantiations (M no power of two) of the step and consensus kernels for float32 parameter storage.
#include "kernels.hpp"

namespace fgd {

namespace {
struct Sets {
    template <int MMAX, bool EXACT>
    static KernelSet get(int k1, int k2, bool subset) {
        return make_kernel_set<ParamF32, MMAX, EXACT, lanes_v_f32(MMAX)>(k1, k2, subset);
    }
};
}  // namespace

bool kernels_f32_class(int M, int k1, int k2, bool subset, KernelSet *out) {
    return select_class<Sets>(M, out, k1, k2, subset);
}

}  // namespace fgd
