// Split-execution kernels of the worker classes (M no power of two) for
// float32 parameter storage: the Mix1 half and the blocking half of a round
// (Appendix A, Algorithm 1).
#include "kernels.hpp"

namespace fgd {

bool split_kernels_f32_class(int M, int k1, int k2, bool subset, bool mix_state, SplitSet *out) {
    return select_class<SplitSets<ParamF32>>(M, out, k1, k2, subset, mix_state);
}

}  // namespace fgd
