// Seg-Sum with the update in it (lm_segsum_sgd), fp32 gradients.
#include "segsum_kernels.hpp"

namespace lmz {

template hipError_t seg_walk<float, kOpSgd>(SegArgs&, hipStream_t);
template void seg_fix<kOpSgd>(const SegArgs&, hipStream_t);

}  // namespace lmz
