// Seg-Sum written out (lm_segsum, lm_segsum_rows), bf16 gradients; the
// occupancy of these kernels also sizes the chunks of the updates.
#include "segsum_plain.hpp"

namespace lmz {

// The updates' sources call these.
SEG_PLAIN(bf16_t, 8, 1, false)
SEG_PLAIN(bf16_t, 8, 1, true)
SEG_PLAIN(bf16_t, 8, 2, false)
SEG_PLAIN(bf16_t, 8, 2, true)
SEG_PLAIN(bf16_t, 1, 1, false)
SEG_PLAIN(bf16_t, 1, 2, false)
SEG_PLAIN(bf16_t, 1, 4, false)

template hipError_t seg_walk<bf16_t, kOpStore>(SegArgs&, hipStream_t);

}  // namespace lmz
