// Seg-Sum written out (lm_segsum, lm_segsum_rows), fp32 gradients; the
// occupancy of these kernels also sizes the chunks of the updates.
#include "segsum_plain.hpp"

namespace lmz {

// The updates' sources call these.
SEG_PLAIN(float, 4, 1, false)
SEG_PLAIN(float, 4, 1, true)
SEG_PLAIN(float, 4, 2, false)
SEG_PLAIN(float, 4, 2, true)
SEG_PLAIN(float, 4, 4, false)
SEG_PLAIN(float, 4, 4, true)
SEG_PLAIN(float, 1, 1, false)

template hipError_t seg_walk<float, kOpStore>(SegArgs&, hipStream_t);
template void seg_fix<kOpStore>(const SegArgs&, hipStream_t);

}  // namespace lmz
