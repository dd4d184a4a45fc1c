// Seg-Sum with the update in it (lm_segsum_adam), bf16 gradients.
#include "segsum_kernels.hpp"

namespace lmz {

template hipError_t seg_walk<bf16_t, kOpAdam>(SegArgs&, hipStream_t);

}  // namespace lmz
