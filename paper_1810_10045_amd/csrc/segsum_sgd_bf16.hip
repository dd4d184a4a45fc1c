// Seg-Sum with the update in it (lm_segsum_sgd), bf16 gradients.
#include "segsum_kernels.hpp"

namespace lmz {

template hipError_t seg_walk<bf16_t, kOpSgd>(SegArgs&, hipStream_t);

}  // namespace lmz
