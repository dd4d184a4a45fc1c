// How many workgroups of the plain walk (kOpStore) fit on a compute unit: the
// definition, for the two sources that hold those kernels.
#pragma once

#include "segsum_kernels.hpp"

namespace lmz {

template <typename GT, int VEC, int NV, int R, bool TAIL>
int plain_blocks(bool fused) {
  // Queried once per kernel.
  static std::atomic<int> cache[2] = {-1, -1};
  int b = cache[fused].load(std::memory_order_relaxed);
  if (b < 0) {
    constexpr int RF = rf_for<NV, R>(), T = t_for<R>();
    b = 0;
    hipError_t e;
    if constexpr (VEC >= 2) {
      e = fused ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                      &b, k_segsum<GT, VEC, NV, RF, R, T, true, kOpStore, TAIL, false>,
                      kSegThreads, 0)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                      &b, k_segsum<GT, VEC, NV, RF, R, T, false, kOpStore, TAIL, false>,
                      kSegThreads, 0);
    } else {
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &b, k_segsum<GT, VEC, NV, RF, R, T, false, kOpStore, TAIL, false>, kSegThreads,
          0);
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      b = 0;
    }
    cache[fused].store(b, std::memory_order_relaxed);
  }
  return b;
}

// The instantiations for every chunk length.
#define SEG_PLAIN(GT, VEC, NV, TAIL)                      \
  template int plain_blocks<GT, VEC, NV, 16, TAIL>(bool);  \
  template int plain_blocks<GT, VEC, NV, 32, TAIL>(bool);  \
  template int plain_blocks<GT, VEC, NV, 64, TAIL>(bool);  \
  template int plain_blocks<GT, VEC, NV, 128, TAIL>(bool); \
  template int plain_blocks<GT, VEC, NV, 256, TAIL>(bool); \
  template int plain_blocks<GT, VEC, NV, 512, TAIL>(bool);

}  // namespace lmz
