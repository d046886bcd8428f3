// The worker classes' step kernels (M no power of two) for bf16 parameter storage (float32 arithmetic) that also apply Mix1 to the optimizer
// state (Appendix B, GlobalM1S variants).
#include "kernels.hpp"

namespace fgd {

namespace {
struct Sets {
    template <int MMAX, bool EXACT>
    static KernelSet get(int k1, int k2, bool subset) {
        return make_kernel_set_ms<ParamBF16, MMAX, EXACT, lanes_v_bf16(MMAX)>(k1, k2, subset);
    }
};
}  // namespace

bool kernels_bf16_ms_class(int M, int k1, int k2, bool subset, KernelSet *out) {
    return select_class<Sets>(M, out, k1, k2, subset);
}

}  // namespace fgd
