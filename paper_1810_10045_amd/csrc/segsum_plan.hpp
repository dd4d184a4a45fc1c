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
//
// Less than one round, many types (fewer than kFewTokens positions for each
// type there may be). A wave waits for each batch of its rows and for what its
// segment ends need, so too few waves leave the memory half idle.
//   Long chunks (R >= 256) fill the round. Measured on 256 compute units, fp32:
//   524,288 ids over 20K words, D = 512 (1,063 waves on room for 2,048) 286 ->
//   208 us, 200,000 over 20K, D = 256 60 -> 52 us; bf16, 400,000 over 300K,
//   D = 512 (3,125 on 4,096) 132 -> 118.
//   Shorter ones (R = 32 .. 128) make kFillWaves waves for each compute unit,
//   two workgroups, where there would be well below that many and chunks hold
//   no fewer than kMinR positions on average. Waves before -> now: D = 300,
//   40,000 over 2,000, Adam 32 us (627) -> 23; SGD, D = 512, 106,496 over 800K
//   77 (1,664) -> 73. Close to kFillWaves it loses: 30,011 over 50K, D = 650
//   38.3 (1,876) -> 40.5. So does it with chunks of 10 rows: 20,000 over 98,
//   D = 200 17.2 us (2,048), 13.6 (1,280).
//   Rows that are no whole number of vectors (part_vec): half as many waves,
//   which is better with short chunks (R = 32, 64) and not with longer ones. us
//   with kFillWaves / half: 21,386 over 2,865, D = 358 15.3 / 14.3; 40,000 over
//   2,000, D = 301 21.6 / 18.8; but R = 128, 106,496 over 800K, D = 510 63.4 /
//   68.4, and bf16, 100,000 over 5,000, D = 518 33.7 / 39.6.
//
// Less than one round, few types: nearly every cut goes through a long segment
// and costs a partial row, and a head's pieces are summed one after the other.
// So only whole workgroups for each compute unit are filled up: one, or two with
// rows of less than kNarrowBytes, of which a wave has few bytes in flight, while
// chunks keep kFewRows positions; and two where one and a part are needed anyway
// (not with part_vec). us as they come / here / as with many types:
//   bf16, 30,000 ids over 98 characters, D = 1024 (950 waves) 22.7 / 22.7 /
//     31.2; D = 352, 905,469 over 221 (1,769) 124 / 118 (2,048) / 128;
//     D = 512, 100,000 over 500 (786) 32.9 / 29.1 (1,024) / 31.3;
//   fp32, 60,000 over 500, D = 1024 (945) 49.2 / 49.2 / 53.7; 262,144 over 98,
//     D = 1024 (1,025) 174 / 174 / 200; 200,000 over 98, D = 256 (782) 53 / 40
//     (1,024) / 55, D = 128 35 (1,024) / 31 (2,048) / 37; Adam, 19,200 over 98,
//     D = 1792 (1,208) 43.0 / 39.7 (2,048) / 39.7; D = 512 (604) 17.0 / 17.0 / 17.7.
//
// kEnoughWaves for each compute unit are enough with bf16 rows where far fewer
// types turn up than there is room for, unless a chunk would exceed R: room for
// types is counted at four positions each there, so chunks get as short as R / 5,
// and every cut may cost a partial row of twice a row's bytes. 30,011 over 50K,
// D = 1792 (9,380 waves) 55.4 -> 46.7 us (2,560). With fp32 rows chunks keep
// R / 2, and fewer lose their whole rounds: 120,000 over 800K, D = 1500 210 ->
// 220 us, 65,536 over 800K, D = 2048 136 -> 139.
constexpr int kFillWaves = 8, kEnoughWaves = 10;  // for each compute unit
constexpr int kGroupWaves = 4;                    // waves of a workgroup
constexpr int kFewTokens = 32, kFewRows = 64, kNarrowBytes = 1024;

inline ChunkCount whole_rounds(int64_t K, int64_t D, int64_t u_cap, int R, bool bf16, int tiles,
                               int nchunks, int max_chunks, int64_t waves_per_round, int cus) {
  const bool part_vec = D % (bf16 ? 8 : 4) != 0;
  ChunkCount c{nchunks, nchunks};
  if (waves_per_round <= 0 || tiles <= 0 || cus <= 0) return c;
  const int64_t waves = int64_t(nchunks) * tiles;
  int64_t fill = waves, most = max_chunks;  // waves to make, chunks at most
  if (waves > waves_per_round) {
    const int64_t last = waves % waves_per_round;
    if (last != 0 && 2 * last < waves_per_round) fill = waves - last + waves_per_round;
  } else if (K >= kFewTokens * u_cap) {
    const int64_t group = int64_t(cus) * kGroupWaves;
    const bool more = waves > group + group / 8, narrow = D * (bf16 ? 2 : 4) < kNarrowBytes;
    const int64_t want = more || narrow ? 2 * group : group;
    const int rows = more && !narrow ? kMinR : kFewRows;
    const bool may = R > kMinR && (narrow || !more || !part_vec);
    if (may && waves < want - want / 8 && K / rows >= (want + tiles - 1) / tiles) fill = want;
  } else if (R >= 256) {
    fill = waves_per_round;
  } else if (R > kMinR) {
    const int64_t want = int64_t(cus) * (part_vec ? kFillWaves / 2 : kFillWaves);
    if (waves < want - want / 8) fill = want;
    if (most > K / kMinR) most = K / kMinR;
  }
  int64_t want = (fill + tiles - 1) / tiles;
  if (want > most) want = most;
  if (want > nchunks) c.n = static_cast<int>(want);
  c.enough = c.n;
  if (bf16 && R < 256) c.enough = static_cast<int>((int64_t(cus) * kEnoughWaves + tiles - 1) / tiles);
  return c;
}

// Whether the walk reads a column per lane, not 16-byte vectors: rows shorter
// than one, and bf16 rows of up to kMaxHalfCols columns where some vector would
// start between two 4-byte words (grad is the rows' address, ld their stride).
// Such a vector takes longer than eight loads of a column. One call, us, vectors
// / columns: 300,000 ids over 221, SGD, D = 63 53.1 / 32.2, D = 255 82.3 / 47.4;
// 36,886 over 60K, D = 31 16.4 / 14.3, D = 127 18.9 / 16.9; but D = 257 23.2 / 27.9,
// and of even width and stride 300,000 over 221, SGD, D = 14 36.7 / 38.3.
constexpr int kMaxHalfCols = 256;

inline bool column_per_lane(uintptr_t grad, int64_t ld, int64_t D, bool bf16) {
  if (D < (bf16 ? 8 : 4)) return true;
  return bf16 && D <= kMaxHalfCols && (grad % 4 != 0 || ld % 2 != 0 || D % 2 != 0);
}

}  // namespace lmz
