// Seg-Sum: how many chunks a call is cut into. Host arithmetic only, without
// HIP, so that a host test can call it.
#pragma once

#include <stdint.h>

namespace lmz {

constexpr int kMinR = 16, kMaxR = 512;  // shortest and longest chunks

// Chunks of a call (n) and how many are enough where far fewer types turn up
// than it has room for (chunk_plan).
struct ChunkCount {
  int n, enough;
};

// Whole rounds of waves. The walk's waves (chunks x column tiles) of equal
// cost run in rounds of as many waves as fit at once (waves_per_round) on the
// compute units the launch's stream may use (cus). Where a
// last round would be less than half full, its few waves run nearly alone,
// far below the memory system's rate: the chunk count then grows (so the
// chunks shrink) until the last round is full, at most to the workspace's
// capacity (a chunk count above the minimum only shortens chunks).
// Measured at K = 1,048,576, D = 2048 fp32 (two column tiles, room for
// 2,048 waves): 2,088 chunks (4,176 waves) 1,591 us, 3,072 chunks 1,488 us.
// Where the last round was half full or more (the bf16 merge: 10,347 waves
// on room for 4,096) rounding up changed nothing measurable.
// Less than one round is filled up too where chunks are long (R >= 256): a
// wave waits for each batch of its rows, so half as many waves leave the memory
// half idle. Measured, fp32: 524,288 ids over 20K words, D = 512 (1,063 waves
// on room for 2,048) 286 -> 208 us, 200,000 over 20K, D = 256 60 -> 52 us,
// 262,144 over 2M, D = 1024 (2,048 on 4,096) 339 -> 336 us.
// Shorter chunks (R = 32 .. 128) make kFillWaves waves for each compute unit,
// two workgroups, where there would be well below that many and chunks hold no
// fewer than kMinR positions on average, and no more than kEnoughWaves for each
// unless a chunk would exceed R, as every cut may cost a partial
// row. Measured on 256 compute units, waves before -> now: Adam, D = 1792,
// 19,200 ids over 98 43.2 us (1,208) -> 39.7 (1,536 waves 41.6, 2,560 43.8);
// D = 300, 40,000 over 2,000 40.4 (627) -> 25.2; SGD, D = 512, 106,496 over
// 800K 71.7 (1,664) -> 67.5; bf16, D = 1792, 19,200 over 15,437 38.0 (5,058)
// -> 33.6 (2,560). Close to kFillWaves it loses: 30,011 over 50K, D = 650 38.3
// (1,876) -> 40.5. So does it with chunks of 10 rows: 20,000 over 98, D = 200
// 17.2 us (2,048), 13.6 (1,280).
// Rows that are no whole number of vectors (part_vec) write their partial rows
// a column at a time: half as many waves. 21,386 over 2,865, D = 358: 22.2 us
// (2,048), 17.7 (1,024), 18.9 (669 as they come); 60,000 over 500, D = 358
// 45.0, 32.1, 32.2; SGD, 100,000 over 1,000, D = 513 59.6, 51.9, 55.3.
constexpr int kFillWaves = 8, kEnoughWaves = 10;  // for each compute unit

inline ChunkCount whole_rounds(int64_t K, int R, bool part_vec, int tiles, int nchunks,
                               int max_chunks, int64_t waves_per_round, int cus) {
  ChunkCount c{nchunks, nchunks};
  if (waves_per_round <= 0 || tiles <= 0 || cus <= 0) return c;
  const int64_t waves = int64_t(nchunks) * tiles;
  const int64_t last = waves % waves_per_round;
  const int64_t fill = int64_t(cus) * (part_vec ? kFillWaves / 2 : kFillWaves);
  int64_t want = nchunks;
  if (R >= 256 ? last != 0 && (waves < waves_per_round || 2 * last < waves_per_round)
               : waves > waves_per_round && last != 0 && 2 * last < waves_per_round) {
    const int64_t rounds = (waves + waves_per_round - 1) / waves_per_round;
    want = (rounds * waves_per_round + tiles - 1) / tiles;
  } else if (R > kMinR && R < 256 && waves < fill - fill / 8) {
    want = (fill + tiles - 1) / tiles;
    if (want > K / kMinR) want = K / kMinR;
  }
  if (want > max_chunks) want = max_chunks;
  if (want > nchunks) c.n = static_cast<int>(want);
  c.enough = R < 256 ? static_cast<int>((int64_t(cus) * kEnoughWaves + tiles - 1) / tiles) : c.n;
  return c;
}

}  // namespace lmz
