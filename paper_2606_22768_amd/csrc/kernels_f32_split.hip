// Split-execution kernels for float32 parameter storage: the Mix1 half and the blocking
// half of a round (Appendix A, Algorithm 1).
#include "kernels.hpp"

namespace fgd {

bool split_kernels_f32(int M, int k1, int k2, bool subset, bool mix_state, SplitSet *out) {
    return exact_workers(M) ? select_exact<SplitSets<ParamF32>>(M, out, k1, k2, subset, mix_state)
                            : split_kernels_f32_class(M, k1, k2, subset, mix_state, out);
}

}  // namespace fgd
