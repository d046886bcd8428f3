// Split-execution kernels of the worker classes (M no power of two) for bf16
// parameter storage (float32 arithmetic): the Mix1 half and the blocking half
// of a round (Appendix A, Algorithm 1).
#include "kernels.hpp"

namespace fgd {

bool split_kernels_bf16_class(int M, int k1, int k2, bool subset, bool mix_state, SplitSet *out) {
    return select_class<SplitSets<ParamBF16>>(M, out, k1, k2, subset, mix_state);
}

}  // namespace fgd
