// Seg-Sum with the update in it (lm_segsum_adam), fp32 gradients.
#include "segsum_kernels.hpp"

namespace lmz {

template hipError_t seg_walk<float, kOpAdam>(SegArgs&, hipStream_t);
template void seg_fix<kOpAdam>(const SegArgs&, hipStream_t);

}  // namespace lmz
