// Seg-Sum: what the host code (segsum.hip) and the kernels share. The
// kernels (segsum_kernels.hpp) are compiled once per update and gradient type
// (segsum_<update>_<type>.hip), side by side.
#pragma once

#include "common.hpp"
#include "segsum_plan.hpp"

namespace lmz {

constexpr int kFusedCols = kWave * 4;   // columns of a fused fix-up tile

struct SegArgs {
  const void* grad;
  int64_t ld_grad;
  int K, D;
  const int32_t* perm;
  const int32_t* inverse;
  const int32_t* offsets;
  const int64_t* num_unique;
  int64_t u_cap;
  float* out;
  int64_t ld_out;
  float* part_cont;
  float* part_start;
  int32_t* desc;
  int32_t* npieces;
  uint64_t* flags;   // fused launch: flags[c * tiles + t], the word of chunk c's tile t
  uint64_t tag;      // marks the words of this call
  uint64_t wait_tag;  // the tag the fix-up waits for (with the failure-path test
                      // hook, one no walk writes)
  uint32_t spin_limit;  // polls of a flag before the wait gives up
  int main_blocks, fix_tiles, fused;
  int by_column;           // the walk reads a column per lane (column_per_lane)
  int tiles, tile_cols;    // column tiles of the walk and the columns of one
  int thin;                // TAIL kernels: columns by which the last tile starts earlier
  int R, nchunks, rw, ww;  // cost of a position / of a segment end
  int max_chunks;          // chunks the workspace holds
  int enough;              // chunks below nchunks that still fill the device
  const void* row_ids;     // lm_segsum_rows: type u goes to out row row_ids[u]
  int row_ids64;           //   (int64 ids when nonzero), < out_rows; nullptr: row u
  int64_t out_rows;
  int32_t* dev_err;
  OptParams opt;           // lm_segsum_sgd / _adam: the step (out is the table)
  float* m;                // lm_segsum_adam: the moments, rows of out's stride
  float* v;
};

// What a finished type row becomes: written (lm_segsum, lm_segsum_rows), or
// applied to the table row by SGD or Adam.
constexpr int kOpStore = 0, kOpSgd = 1, kOpAdam = 2;

// Walks (and, in the fused form, fixes up) the chunks of `a`; sets a.nchunks
// and the column tiles.
template <typename GT, int OP>
hipError_t seg_walk(SegArgs& a, hipStream_t st);
// The fix-up as a launch of its own.
template <int OP>
void seg_fix(const SegArgs& a, hipStream_t st);

// Compute units a launch on `st` may use (segsum.hip).
int stream_cus(hipStream_t st);

}  // namespace lmz
