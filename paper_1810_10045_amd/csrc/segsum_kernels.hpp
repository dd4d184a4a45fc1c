// Seg-Sum (Sec. III-A step 2): out[u, :] = sum of grad[perm[i], :] over the
// sorted positions i of type u, accumulated in fp32 in a fixed order.
//
// Work partition (no float atomics, run-to-run bit-identical):
//   The K sorted positions are cut into N chunks of equal cost, one chunk per
//   wave and per column tile of up to 1024 columns. A position costs one row
//   read (rw) and a segment end one row write (ww, weighted per gradient
//   dtype by measurement), so the cost before position p
//   of segment u is rw * p + ww * u; chunk c starts where that reaches c * Q,
//   Q = ceil((rw * K + ww * U) / N). Reads and writes thus balance across
//   waves wherever the heads and the tail of the Zipf law fall in the sorted
//   order (equal-length chunks left the waves of the tail, one write per row,
//   twice as long as those of the heads). The waves of a workgroup find their
//   bounds together (load_window), and every segment end of their chunks from
//   the offsets that leaves in LDS.
//   A segment shorter than T rows belongs entirely to the chunk holding its
//   first position, even where it runs past the chunk end; a longer one is
//   cut at chunk boundaries and every chunk sums its piece into a partial
//   row:
//     part_start[c]  the piece of a long segment that starts in chunk c and
//                    continues past it,
//     part_cont[c]   the piece of a long segment that started before chunk c.
//   Its pieces are part_start[c] and part_cont[c + 1 .. c + P], c + P being
//   the chunk of its last position (from the same cost formula), added in a
//   fixed order: one after the other for a segment of fewer than 16 further
//   pieces, a fixed stride split over the waves of a workgroup and a
//   fixed-order combine in LDS for a head. On the 16-byte vector path (rows of
//   up to LMZ_SEG_FUSED_MAX_D columns) that happens in the walk's own launch
//   (the fused launch below), otherwise in a second one (k_segsum_fix, from
//   the desc[c] and npieces[c] that the walk then writes).
// A chunk holds at most R positions (N is sized for U = min(K, u_cap)) and
// reads at most R + T - 1 rows.
//
// Each wave gathers whole 16-byte column vectors of RF rows at a time
// (RF x NV x 1 KiB in flight), adds them in fp32 registers and writes a row
// as soon as its segment ends; grad is streamed with non-temporal loads.
//
// lm_segsum_rows runs the same kernels with a row map: type u's sum goes to
// row row_ids[u] of the output (the dense table of a SCATTER). The walk
// gathers the row of each window position's type with the types; the
// fix-up looks it up per segment. Without a row map, row u.
//
// lm_segsum_sgd and lm_segsum_adam (the update instantiations, OP) update
// those rows instead of writing them, the sum in the same order and the
// update the same arithmetic as lm_sparse_apply's (sgd_value, adam_value).
// The walk loads the table row (Adam: those of the parameters, m and v) when
// the segment has ended; where SGD finds many short segments (the EARLY
// instantiations, see may_be_early) it closes a gather batch after its
// kEnds-th segment end and loads the table rows of those ends with its
// gradient rows, through buffer resources whose range is empty where no row
// is needed (such a load reads nothing and returns zeros), so an update costs
// no round trip of its own.
#pragma once

#include <atomic>

#include "segsum_args.hpp"
#include "segsum_words.hpp"

namespace lmz {

// Tuning knobs (overridable at build time).
#ifndef LMZ_SEG_TDIV
#define LMZ_SEG_TDIV 2               // long-segment threshold T = R / this (1..64)
#endif
#ifndef LMZ_SEG_RF4
#define LMZ_SEG_RF4 4                // rows per gather batch with 4 vectors per lane
#endif
#ifndef LMZ_SEG_RF2
#define LMZ_SEG_RF2 8                // rows per gather batch with <= 2 vectors per lane
#endif
#ifndef LMZ_SEG_LONG_R
#define LMZ_SEG_LONG_R 512           // from this chunk length on, the *_LONG batches
#endif
#ifndef LMZ_SEG_RF4_LONG
#define LMZ_SEG_RF4_LONG 8           // long chunks walk long enough to keep more rows in flight
#endif
#ifndef LMZ_SEG_RF2_LONG
#define LMZ_SEG_RF2_LONG 16
#endif
#ifndef LMZ_SEG_SGD_ENDS2
#define LMZ_SEG_SGD_ENDS2 4          // early updates: segment ends (table rows) per gather batch
#endif                               // with 2 and 1 vectors per lane
#ifndef LMZ_SEG_SGD_ENDS1
#define LMZ_SEG_SGD_ENDS1 6
#endif
#ifndef LMZ_SEG_ADAM_RF4
#define LMZ_SEG_ADAM_RF4 4           // lm_segsum_adam: most rows per batch with 4 vectors per lane
#endif
#ifndef LMZ_SEG_FIX_RF
#define LMZ_SEG_FIX_RF 16            // partial rows per wave in flight in the fix-up
#endif
constexpr int kSegThreads = 256;     // threads of a workgroup: a chunk per wave
constexpr int kSegWaves = kSegThreads / kWave;
static_assert(kSegWaves == kGroupWaves, "the chunk counts assume it");

// Windows of positions a wave loads up front: [p0 - 1, p0 - 1 + 64 * NW)
// must cover p0 - 1 (to see whether the first segment started earlier), the
// whole walk (at most R + T - 1 rows from p0) and one position past it (to
// see whether the last row ends its segment).
template <int R, int T>
constexpr int windows_for() { return (R + T) / 64 + 1; }

// Chunk bounds. A workgroup walks kSegWaves consecutive chunks, so its bounds
// (targets t of the running cost) lie close together, and it looks for them
// together: a 256-ary search (one probe per thread and round) keeps the types
// that any of its targets can fall into, until they are few enough to load
// their offsets into LDS: one round where there are at most types_cap of
// them, two up to about 100K types. Each wave then finds its own two bounds
// and, from the same offsets, every segment end of its chunk, without another
// load. (A search per wave with 32 probes per target, and the segments from
// inverse[perm[i]] for every position, had cost a chain of nine dependent
// loads before the first gradient row, now five, and a 64-byte line per
// gathered position.)
template <int R>
constexpr int types_cap() { return (kSegWaves * R / kSegThreads + 2) * kSegThreads; }

// The chunks of a call, n <= a.nchunks of equal cost Q: the grid has room for
// u_cap types; where far fewer turn up, n falls to a.enough, as long as no
// chunk exceeds R positions (a cost of rw * R).
struct Plan {
  int n;
  int64_t Q;
};
__device__ __forceinline__ Plan chunk_plan(const SegArgs& a, int U) {
  const int Ub = U < a.u_cap ? U : static_cast<int>(a.u_cap);
  const int64_t cost = int64_t(a.rw) * a.K + int64_t(a.ww) * Ub;
  const int64_t most = int64_t(a.rw) * a.R;
  const int64_t least = U > a.u_cap ? a.nchunks : (cost + most - 1) / most;
  int n = a.enough > least ? a.enough : static_cast<int>(least);
  if (n > a.nchunks) n = a.nchunks;
  return Plan{n, (cost + n - 1) / n};
}

// The types [lo, lo + n) that hold every target from t_first to t_last (n <=
// N), their offsets in s_win[0 .. n]. The cost before position p of segment u
// is rw * p + ww * u, so the type of a target t is the largest u < U with
// f(u) = rw * offsets[u] + ww * u <= t (f(0) = 0). Every thread of the
// workgroup calls it. False where the offsets are inconsistent (the window
// then holds some N types).
template <int N>
__device__ __forceinline__ bool load_window(const int32_t* __restrict__ offsets, int U, int rw,
                                            int ww, int64_t t_first, int64_t t_last,
                                            int (&s_win)[N + 1], int (&s_cnt)[2][kSegWaves],
                                            int& lo_out, int& n_out) {
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  int lo = 0, n = U;
  for (int round = 0; n > N && round < 8; ++round) {
    const int st = (n - 1) / kSegThreads + 1;
    const int64_t u = lo + int64_t(tid + 1) * st;
    const bool in = u < int64_t(lo) + n;
    const int64_t f = in ? int64_t(rw) * offsets[u] + int64_t(ww) * u : 0;
    const uint64_t first = ballot(in && f <= t_first), last = ballot(in && f <= t_last);
    if (lane == 0) {
      s_cnt[0][wave] = __popcll(first);
      s_cnt[1][wave] = __popcll(last);
    }
    __syncthreads();
    int c0 = 0, c1 = 0;
#pragma unroll
    for (int w = 0; w < kSegWaves; ++w) {
      c0 += s_cnt[0][w];
      c1 += s_cnt[1][w];
    }
    __syncthreads();
    c0 = first_lane(c0);
    c1 = first_lane(c1);
    const int64_t end = lo + (int64_t(c1) + 1) * st;
    const int64_t most = int64_t(lo) + n;
    lo += c0 * st;
    n = static_cast<int>((end < most ? end : most) - lo);
    if (n < 1) n = 1;  // only inconsistent offsets
  }
  const bool ok = n <= N;
  if (!ok) n = N;
  for (int i = tid; i <= n; i += kSegThreads) s_win[i] = offsets[lo + i];
  __syncthreads();
  lo_out = lo;
  n_out = n;
  return ok;
}

// The bound of a target: the number of sorted positions whose running cost is
// below t, for t = tA in lanes 0..31 and t = tB in lanes 32..63: with u as
// above, b = offsets[u] + min(ceil((t - f(u)) / rw), len(u)); b = K once
// t >= rw * K + ww * U. A 32-ary search of the window per half-wave. Besides b
// it returns that u and offsets[u], offsets[u + 1]: b lies strictly inside
// segment u exactly when offsets[u] < b < offsets[u + 1].
struct Bound {
  int b, u, o0, o1;
};
template <int N>
__device__ __forceinline__ void chunk_bounds(const int (&s_win)[N + 1], int lo, int n, int U,
                                             int rw, int ww, int K, int64_t tA, int64_t tB,
                                             Bound& A, Bound& B) {
  const int lane = lane_id();
  const bool hi = lane >= 32;
  const int hl = lane & 31;
  const int64_t t = (hi ? tB : tA) - int64_t(ww) * lo;
  int loA = 0, nA = n, loB = 0, nB = n;
  while (nA > 1 || nB > 1) {
    const int sA = (nA + 31) / 32, sB = (nB + 31) / 32;
    const int l = hi ? loB : loA, m = hi ? nB : nA, st = hi ? sB : sA;
    const int u = l + (hl + 1) * st;
    const bool le = m > 1 && u < l + m && int64_t(rw) * s_win[u < n ? u : n] + int64_t(ww) * u <= t;
    const uint64_t b = ballot(le);
    const int cA = __popcll(b & 0xffffffffull), cB = __popcll(b >> 32);
    if (nA > 1) {
      loA += cA * sA;
      nA = nA - cA * sA < sA ? nA - cA * sA : sA;
    }
    if (nB > 1) {
      loB += cB * sB;
      nB = nB - cB * sB < sB ? nB - cB * sB : sB;
    }
  }
  const int u = hi ? loB : loA;
  const int o0 = s_win[u], o1 = s_win[u + 1];
  const int64_t into = (t - (int64_t(rw) * o0 + int64_t(ww) * u) + rw - 1) / rw;
  int b = int64_t(o0) + into < int64_t(o1) ? static_cast<int>(int64_t(o0) + into) : o1;
  if (t + int64_t(ww) * lo >= int64_t(rw) * K + int64_t(ww) * U) b = K;
  A = Bound{first_lane(b), first_lane(u) + lo, first_lane(o0), first_lane(o1)};
  B = Bound{read_lane(b, 32), read_lane(u, 32) + lo, read_lane(o0, 32), read_lane(o1, 32)};
}

// ---------------------------------------------------------------------------
// Fused launch: the fix-up in the walk's launch.
// Partial rows go out as agent-scope stores (coherent across the XCDs' L2s),
// the walk waits for them before it says so in a word per chunk and column
// tile, and they are read with agent-scope loads. A word holds a tag that is
// new for every call (of a per-process counter) above its count and flag, so
// no workspace contents need clearing between calls (segsum_words.hpp).
//   A segment of fewer than kHeadPieces further pieces: the wave that adds the
//   last of its pieces to the count in the word of the segment's first chunk
//   sums them all, in order. No wave waits for another.
//   A longer one (a head of the Zipf law): every piece sets the flag in its
//   own chunk's word, and a fix-up workgroup per column tile of 256, after the
//   walk's workgroups in the same grid, waits for them and sums them with all
//   its waves. Workgroups are dispatched in the order of their index (per
//   XCD), so every walk workgroup holds a slot or has finished before a
//   fix-up workgroup starts; walk workgroups never wait, so a fix-up's wait
//   always ends (bounded all the same: LM_DEVERR_SPIN). A head reaches over
//   the end of the span of kHeadPieces chunks it starts in, so the workgroups
//   of a span find it with one search for that bound, while the walk runs.
// Fix-up workgroups for every segment, each looking after 4 chunks, had cost
// more than the sums: at 30,011 ids over 50K words, D = 650, 8 of 39 us.
// Workgroup b of the walk is column tile b % tiles of chunks (b / tiles) * 4
// ..., and a fix-up tile of 256 columns lies inside one walk tile.
// ---------------------------------------------------------------------------
#ifndef LMZ_SEG_FUSED_RF
#define LMZ_SEG_FUSED_RF 16          // pieces per wave per round in the fused fix-up
#endif
#ifndef LMZ_SEG_FUSED_SLEEP
#define LMZ_SEG_FUSED_SLEEP 8        // s_sleep argument (x 64 cycles) between flag polls
#endif
constexpr int kHeadPieces = 16;  // further pieces from which a segment is a head
static_assert(kHeadPieces <= kCountMask, "a word counts a segment's pieces");
// The memory operations of the words (segsum_words.hpp).
struct AgentWords {
  __device__ __forceinline__ void exchange_if(uint64_t* w, uint64_t seen, uint64_t x) const {
    __hip_atomic_compare_exchange_strong(w, &seen, x, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ uint64_t add(uint64_t* w, uint64_t x) const { return add_agent(w, x); }
};

// The output row of type s: s itself, or row_ids[s] for lm_segsum_rows
// (-1 when that id lies outside [0, out_rows); LM_DEVERR_ID_RANGE is raised
// and the row is not written).
__device__ __forceinline__ int64_t out_row_of(const SegArgs& a, int s) {
  if (!a.row_ids) return s;
  const int64_t r = a.row_ids64 ? static_cast<const int64_t*>(a.row_ids)[s]
                                : static_cast<const int32_t*>(a.row_ids)[s];
  if (r < 0 || r >= a.out_rows) {
    raise_err(a.dev_err, LM_DEVERR_ID_RANGE);
    return -1;
  }
  return r;
}

constexpr int kRawBufferWord3 = 0x00020000;  // buffer resources: 32-bit data format, no swizzle
constexpr int kSc1 = 16;                     // the sc1 bit of buffer accesses: agent scope

// The update instantiations: a buffer resource over row r (D fp32 values)
// of base (the table, m or v, all of out's row stride), or over nothing for
// r < 0: loads through an empty range read no memory and return zeros, so
// a batch loads its table rows unconditionally.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t table_row(const SegArgs& a, float* base,
                                                            int64_t r) {
  return __builtin_amdgcn_make_buffer_rsrc(base + (r >= 0 ? r : 0) * a.ld_out, 0,
                                           r >= 0 ? a.D * 4 : 0, kRawBufferWord3);
}

// VEC fp32 values at column col of the row behind resource rs.
template <int VEC>
__device__ __forceinline__ void table_vec(__amdgpu_buffer_rsrc_t rs, int col, float* v) {
  if constexpr (VEC % 4 == 0) {
#pragma unroll
    for (int i = 0; i < VEC; i += 4) {
      const f32x4 x = __builtin_bit_cast(
          f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (col + i) * 4, 0, 0));
      v[i] = x.x;
      v[i + 1] = x.y;
      v[i + 2] = x.z;
      v[i + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i)
      v[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (col + i) * 4, 0, 0));
  }
}

// VEC columns of a type row, at offset off into the output: written with the
// sums, or (load, then finish) the table row and Adam's moments updated.
template <int VEC, int OP>
struct TableVec {
  float p[OP == kOpStore ? 1 : VEC], m[OP == kOpAdam ? VEC : 1], v[OP == kOpAdam ? VEC : 1];
  __device__ __forceinline__ void load(const SegArgs& a, int64_t off) {
    if constexpr (OP != kOpStore) load_vec<VEC>(a.out + off, p);
    if constexpr (OP == kOpAdam) {
      load_vec<VEC>(a.m + off, m);
      load_vec<VEC>(a.v + off, v);
    }
  }
  __device__ __forceinline__ void finish(const SegArgs& a, int64_t off, const float* sum) {
    if constexpr (OP == kOpSgd) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) sgd_value(p[e], sum[e], a.opt);
    } else if constexpr (OP == kOpAdam) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) adam_value(p[e], m[e], v[e], sum[e], a.opt);
    }
    store_vec<VEC>(a.out + off, OP == kOpStore ? sum : p);
    if constexpr (OP == kOpAdam) {
      store_vec<VEC>(a.m + off, m);
      store_vec<VEC>(a.v + off, v);
    }
  }
};

// Columns. A lane's vector starts at column col; past the last whole vector
// of a row it is the row's last VEC columns instead, so that no load leaves
// the row. Where D is a multiple of VEC such a lane has no column at all and
// stores nothing; otherwise (the TAIL kernels) one lane's vector repeats columns of the
// lane before it. In the walk that lane sits in the same wave (column tiles
// never end on a part of a vector, see seg_walk), so both hold the same values
// for them and both store them.
template <int VEC, bool TAIL>
__device__ __forceinline__ int vec_col(int col, int D) {
  if constexpr (TAIL) return col + VEC <= D ? col : D - VEC;
  return col < D ? col : D - VEC;
}

// Partial rows at agent scope (the rows of the workspace are D values apart):
// pairs of columns or, where D is no multiple of a vector and pairs are not
// aligned (TAIL), 16 bytes at the alignment of a float through a buffer
// resource over n rows. A column at a time had cost 6 of 32 us at 60,000 ids
// over 500, D = 358, and 4 of 22 at 19,200 over 98, D = 517 (fp32). Adam's TAIL
// kernels still load a column at a time, which measured faster where there are
// few pieces (640 ids over 10K, D = 517 17.6 us, 19.0; 65,536 over 800K, D = 513
// 90.4, 94.2).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t part_rows(float* row, int n, int D) {
  return __builtin_amdgcn_make_buffer_rsrc(row, 0, n * D * 4, kRawBufferWord3);
}

template <int VEC, bool TAIL>
__device__ __forceinline__ void store_vec_agent(float* row, int D, int col, const float* v) {
  static_assert(VEC % 4 == 0, "16-byte vectors");
  if constexpr (TAIL) {
    const __amdgpu_buffer_rsrc_t rs = part_rows(row, 1, D);
    asm volatile("" : "+v"(col));  // its byte offset is made here, not kept through the walk
#pragma unroll
    for (int i = 0; i < VEC; i += 4)
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(u32x4, f32x4{v[i], v[i + 1], v[i + 2], v[i + 3]}), rs, (col + i) * 4,
          0, kSc1);
  } else {
#pragma unroll
    for (int i = 0; i < VEC; i += 2)
      st_agent(reinterpret_cast<uint64_t*>(row + col + i),
               uint64_t(__float_as_uint(v[i])) | (uint64_t(__float_as_uint(v[i + 1])) << 32));
  }
}

template <int VEC, bool TAIL>
__device__ __forceinline__ void load_vec_agent(const float* p, float* v) {
  if constexpr (TAIL) {
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      v[e] = __uint_as_float(ld_agent(reinterpret_cast<const uint32_t*>(p) + e));
  } else {
#pragma unroll
    for (int e = 0; e < VEC; e += 2) {
      const uint64_t x = ld_agent(reinterpret_cast<const uint64_t*>(p + e));
      v[e] = __uint_as_float(static_cast<uint32_t>(x));
      v[e + 1] = __uint_as_float(static_cast<uint32_t>(x >> 32));
    }
  }
}

// VEC columns from col, of the row `bytes` after the resource's first.
template <int VEC>
__device__ __forceinline__ void load_part_vec(__amdgpu_buffer_rsrc_t rs, int bytes, int col,
                                              float* v) {
#pragma unroll
  for (int i = 0; i < VEC; i += 4) {
    const f32x4 x = __builtin_bit_cast(
        f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (col + i) * 4, bytes, kSc1));
    v[i] = x.x;
    v[i + 1] = x.y;
    v[i + 2] = x.z;
    v[i + 3] = x.w;
  }
}

// The partial row of piece t of the segment that starts in chunk cs.
__device__ __forceinline__ float* piece_row(const SegArgs& a, int cs, int t) {
  return t == 0 ? a.part_start + static_cast<int64_t>(cs) * a.D
                : a.part_cont + static_cast<int64_t>(cs + t) * a.D;
}

template <int NV>
constexpr int ends_for() {
  return NV == 2 ? LMZ_SEG_SGD_ENDS2 : LMZ_SEG_SGD_ENDS1;
}

// Every lane of the wave calls this; the lanes with need wait until chunk x's
// word (of column tile ct) says that its piece is there. False if the wait
// gave up.
__device__ __forceinline__ bool wait_piece(const SegArgs& a, int x, int ct, bool need) {
  for (uint32_t spin = 0;; ++spin) {
    const uint64_t f = need ? ld_agent(a.flags + size_t(x) * a.tiles + ct) : 0;
    const bool ok = !need || (word_is(f, a.wait_tag) && (f & kPieceFlag));
    if (!ballot(!ok)) return true;
    if (spin >= a.spin_limit) {
      if (lane_id() == 0) raise_err(a.dev_err, LM_DEVERR_SPIN);
      return false;
    }
    __builtin_amdgcn_s_sleep(LMZ_SEG_FUSED_SLEEP);
  }
}

// Fix-up workgroup f: the head, if any, that starts in chunks [c0, c0 +
// kHeadPieces) of span f / fix_tiles, columns of tile f % fix_tiles: wave w
// adds pieces w, w + W, ... in order, and the waves' sums are added in order.
template <int OP, bool TAIL>
__device__ __forceinline__ void fused_fix(const SegArgs& a) {
  constexpr int RF = LMZ_SEG_FUSED_RF;
  constexpr int kTypes = 2 * kSegThreads;
  __shared__ float s_part[kSegWaves][kFusedCols];
  __shared__ int s_win[kTypes + 1];
  __shared__ int s_cnt[2][kSegWaves];
  const int lane = lane_id();
  const int wave = first_lane(static_cast<int>(threadIdx.x >> 6));
  const int f = static_cast<int>(blockIdx.x) - a.main_blocks;
  const int c0 = (f / a.fix_tiles) * kHeadPieces, K = a.K, D = a.D;
  const int tile0 = (f % a.fix_tiles) * kFusedCols, col = tile0 + lane * 4;
  const int col_ld = vec_col<4, TAIL>(col, D);
  const int ct = tile0 / a.tile_cols;  // the walk's column tile that holds this one
  const int64_t U64 = *a.num_unique;
  const int U = first_lane(static_cast<int>(U64 < K ? U64 : K));
  if (U < 1) return;
  // The segment that lies across the end of the span, if any.
  const Plan plan = chunk_plan(a, U);
  const int64_t Q = plan.Q, t_end = int64_t(c0 + kHeadPieces) * Q;
  if (c0 + kHeadPieces >= plan.n) return;
  int lo, nt;
  load_window<kTypes>(a.offsets, U, a.rw, a.ww, t_end, t_end, s_win, s_cnt, lo, nt);
  Bound A, B;
  chunk_bounds<kTypes>(s_win, lo, nt, U, a.rw, a.ww, K, t_end, t_end, A, B);
  const int64_t cs64 = (int64_t(a.rw) * A.o0 + int64_t(a.ww) * A.u) / Q;
  const int64_t ce64 = (int64_t(a.rw) * (A.o1 - 1) + int64_t(a.ww) * A.u) / Q;
  const int last = plan.n - 1;
  const int cs = static_cast<int>(cs64 < c0 ? -1 : (cs64 > last ? last : cs64));
  const int ce = static_cast<int>(ce64 > last ? last : ce64);
  const int P = ce - cs, s = A.u;
  if (A.b <= A.o0 || A.b >= A.o1 || cs < 0 || P < kHeadPieces || s >= a.u_cap) return;
  // The type's row, before the wait (no other workgroup writes these columns).
  const int64_t orow = out_row_of(a, s);
  const int cx = tile0 + static_cast<int>(threadIdx.x);
  TableVec<1, OP> tv;
  if (orow >= 0) tv.load(a, orow * a.ld_out + (cx < D ? cx : D - 1));
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int t0 = wave; t0 <= P; t0 += kSegWaves * RF) {
    const int tl = t0 + (lane < RF ? lane : 0) * kSegWaves;  // lane r: piece t0 + r * W
    wait_piece(a, cs + (tl <= P ? tl : 0), ct, lane < RF && tl <= P);
    asm volatile("" ::: "memory");  // no piece is read before its flag
    float buf[RF][4];
#pragma unroll
    for (int r = 0; r < RF; ++r) {
      const int t = t0 + r * kSegWaves;
      float* const row = piece_row(a, cs, t <= P ? t : t0);
      if constexpr (TAIL && OP != kOpAdam) load_part_vec<4>(part_rows(row, 1, D), 0, col_ld, buf[r]);
      else load_vec_agent<4, TAIL>(row + col_ld, buf[r]);
    }
#pragma unroll
    for (int r = 0; r < RF; ++r)
      if (t0 + r * kSegWaves <= P)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += buf[r][e];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (TAIL) {  // this lane's own columns within the tile
      const int x = col_ld + e - tile0;
      if (x >= lane * 4) s_part[wave][x] = acc[e];
    } else {
      s_part[wave][lane * 4 + e] = acc[e];
    }
  }
  __syncthreads();
  if (cx < D && orow >= 0) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kSegWaves; ++w) sum += s_part[w][threadIdx.x];
    tv.finish(a, orow * a.ld_out + cx, &sum);
  }
}

// Adam in one launch with 4 vectors per lane runs two workgroups on a compute
// unit, also where its registers allow three (168 of them at R = 16 and 32):
// then the walk's 512 workgroups spread evenly and the fix-up's start after
// them. us, three / two: 19,200 ids over 98, D = 1792 39.4 / 37.8, over 15,437
// 82.2 / 76.7; 30,011 over 50K, D = 650 50.7 / 47.9; 65,536 over 800K, D = 1024
// 176.6 / 176.1.
template <typename GT, int VEC, int NV, int RF, int R, int T, bool FUSED, int OP,
          bool TAIL, bool EARLY>
__global__ __launch_bounds__(kSegThreads)
__attribute__((amdgpu_waves_per_eu(1, FUSED && OP == kOpAdam && NV >= 4 ? 2 : 8))) void k_segsum(SegArgs a) {
  if constexpr (FUSED) {
    if (static_cast<int>(blockIdx.x) >= a.main_blocks) {
      fused_fix<OP, TAIL>(a);
      return;
    }
  }
  using RV = RowVec<GT, VEC>;
  using raw_t = typename RV::raw_t;
  constexpr int kColsPerVec = kWave * VEC;
  constexpr int CT = NV * kColsPerVec;
  constexpr int NW = windows_for<R, T>();

  const int lane = lane_id();
  // One chunk and column tile per wave: the fused grid is one-dimensional,
  // column tile = block % tiles; otherwise the tile is blockIdx.y.
  const int blk = FUSED ? static_cast<int>(blockIdx.x) / a.tiles : static_cast<int>(blockIdx.x);
  const int ct = FUSED ? static_cast<int>(blockIdx.x) % a.tiles : static_cast<int>(blockIdx.y);
  const int wave = first_lane(static_cast<int>(threadIdx.x >> 6));
  const int c0 = blk * kSegWaves, c = c0 + wave;
  // Two launches: the long segment that starts in this chunk, for the fix-up.
  auto describe = [&](int s, int np) {
    if constexpr (!FUSED) {
      if (ct == 0 && lane == 0) {
        a.desc[c] = s;
        a.npieces[c] = np;
      }
    }
  };
  const int K = a.K, D = a.D;

  // 0. This chunk's positions [p0, p1): equal shares of the cost rw * K + ww * U.
  const int64_t U64 = *a.num_unique;
  if (U64 > a.u_cap && c == 0 && ct == 0 && lane == 0) raise_err(a.dev_err, LM_DEVERR_CAPACITY);
  const int U = first_lane(static_cast<int>(U64 < K ? U64 : K));
  if (U < 1) {  // K > 0 always has a type: only a bad count gets here
    if (c < a.nchunks) describe(-1, 0);
    if (c == 0 && ct == 0 && lane == 0) raise_err(a.dev_err, LM_DEVERR_CAPACITY);
    return;
  }
  const Plan plan = chunk_plan(a, U);
  const int nchunks = plan.n;
  const int64_t Q = plan.Q;
  if (c0 >= nchunks) {
    if (c < a.nchunks) describe(-1, 0);
    return;
  }
  constexpr int kTypes = types_cap<R>();
  __shared__ int s_win[kTypes + 1];
  __shared__ int s_cnt[2][kSegWaves];
  __shared__ uint32_t s_ends[kSegWaves][2 * NW];
  int lo, nt;
  const int c_last = c0 + kSegWaves < nchunks ? c0 + kSegWaves : nchunks;
  bool bad = !load_window<kTypes>(a.offsets, U, a.rw, a.ww, int64_t(c0) * Q, int64_t(c_last) * Q,
                                  s_win, s_cnt, lo, nt);
  if (c >= nchunks) {  // no barrier below
    if (c < a.nchunks) describe(-1, 0);
    return;
  }
  Bound A, B;
  chunk_bounds<kTypes>(s_win, lo, nt, U, a.rw, a.ww, K, int64_t(c) * Q, int64_t(c + 1) * Q, A, B);
  const int p0 = A.b;
  int p1 = B.b;
  bool cut_after = c < nchunks - 1;  // p1 is a cut of the cost, not the end of the positions
  if (!cut_after) p1 = K;
  if (p1 - p0 > R) {  // only inconsistent offsets: never walk past the windows
    if (lane == 0) raise_err(a.dev_err, LM_DEVERR_CAPACITY);
    p1 = p0 + R;
    cut_after = false;
  }
  if (p1 <= p0) {  // an empty chunk (a segment end cost more than Q)
    describe(-1, 0);
    return;
  }

  // 1. The first and the last segment of the chunk, from the search: the
  //    first started before the chunk when p0 lies strictly inside it, the
  //    last runs on after the chunk when p1 does.
  const bool started_before = p0 > A.o0 && p0 < A.o1;
  const int s_f = A.u, len_f = A.o1 - A.o0;
  const bool cont_after = cut_after && p1 > B.o0 && p1 < B.o1;
  const int s_l = B.u, len_l = B.o1 - B.o0;
  const bool long_f = started_before && len_f >= T;
  const bool long_l = cont_after && len_l >= T;
  const bool starts_long = long_l && !(started_before && s_l == s_f);
  // The chunk of a sorted position p of type s: that of its cost.
  auto chunk_of = [&](int p, int s) {
    const int64_t x = (int64_t(a.rw) * p + int64_t(a.ww) * s) / Q;
    return static_cast<int>(x < 0 ? 0 : (x < nchunks ? x : nchunks - 1));
  };
  if constexpr (!FUSED) {
    const int np = starts_long ? chunk_of(B.o1 - 1, s_l) - c : 0;
    describe(np >= 1 ? s_l : -1, np);
  }
  // Rows this chunk sums: skip a short segment owned by the previous chunk,
  // run a short last segment to its end, stop a long one at p1.
  const int q = started_before && !long_f ? A.o1 : p0;
  int q_end = cont_after && !long_l ? B.o1 : p1;
  const int walk_max = p0 - 1 + NW * kWave - 1;  // last position whose end bit is known
  if (q_end > walk_max) {
    bad = true;  // only inconsistent offsets get here: never walk past the windows
    q_end = walk_max;
  }

  // 2. The permutation of the windows' positions. The loads are unconditional,
  //    at clamped positions: a load under a lane condition makes the compiler
  //    wait for every load before it. The windows cover the longest chunk; past
  //    q_end every lane repeats that position (one line, a cache hit).
  int pw[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    int pos = p0 - 1 + w * kWave + lane;
    pos = pos < q_end ? pos : q_end;
    pw[w] = a.perm[pos < 0 ? 0 : (pos < K ? pos : K - 1)];
  }
  //    The words this wave will add to, to claim them before a piece is done:
  //    its own chunk's (lane 0) and, where a segment of few pieces began
  //    before, that of the chunk it began in (lane 1).
  int cs_f = 0, P_f = 0;
  uint64_t* word = nullptr;
  uint64_t seen = 0;
  bool claims = false;
  if constexpr (FUSED) {
    if (long_f) {
      cs_f = chunk_of(A.o0, s_f);
      P_f = chunk_of(A.o1 - 1, s_f) - cs_f;
    }
    word = a.flags + size_t(lane == 1 ? cs_f : c) * a.tiles + ct;
    claims = lane == 0 ? long_f || long_l : lane == 1 && long_f && P_f < kHeadPieces;
    if (claims) seen = ld_agent(word);
  }
  //    While it flies: ends[w] bit j: position p0-1+64w+j is the last of its
  //    segment, from the offsets in LDS (type A.u + i ends before
  //    offsets[A.u + i + 1]; a chunk holds at most R + 2 types), and sw[w], the
  //    type of each position: A.u plus the ends before it.
#pragma unroll
  for (int i = 0; i < 2 * NW; i += kWave)
    if (lane + i < 2 * NW) s_ends[wave][lane + i] = 0;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int i = 0; i < R + 2; i += kWave) {
    const int u = A.u - lo + i + lane;
    if (u < nt) {
      const int j = s_win[u + 1] - p0;
      if (static_cast<uint32_t>(j) < static_cast<uint32_t>(NW * kWave))
        atomicOr(&s_ends[wave][j >> 5], 1u << (j & 31));
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  uint64_t ends[NW];
  int sw[NW];
  int before = A.u;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const uint32_t e0 = static_cast<uint32_t>(first_lane(s_ends[wave][2 * w]));
    const uint32_t e1 = static_cast<uint32_t>(first_lane(s_ends[wave][2 * w + 1]));
    ends[w] = (uint64_t(e1) << 32) | e0;
    sw[w] = before + popc_below(ends[w]);
    before += __popcll(ends[w]);
  }
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (static_cast<uint32_t>(pw[w]) >= static_cast<uint32_t>(K)) {
      bad = true;
      pw[w] = 0;
    }
  }
  if constexpr (FUSED) {
    if (claims) word_claim(AgentWords{}, word, seen, a.tag);
  }
  // The map of the tokens either side of p0 (the arrays' consistency, below).
  const int at_p0 = a.inverse[lane == 0 ? read_lane(pw[0], 0) : read_lane(pw[0], 1)];
  // lm_segsum_rows: the output row of every position's type, gathered with
  // the windows (the first segment end needs it, not the first row loads);
  // -1 marks an id outside [0, out_rows) (and clamped positions).
  int orw[NW];
  const bool rows = a.row_ids != nullptr;
  if (rows) {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int sv = sw[w] >= 0 && sw[w] < a.u_cap ? sw[w] : 0;
      const int64_t r = a.row_ids64 ? static_cast<const int64_t*>(a.row_ids)[sv]
                                    : static_cast<const int32_t*>(a.row_ids)[sv];
      orw[w] = r >= 0 && r < a.out_rows ? static_cast<int>(r) : -1;
    }
  }

  // 3. Walk rows q .. q_end - 1, window by window. Lanes past the last column
  //    load a valid vector of the same row (col_ld) and never store it, so
  //    the loads need no per-lane guard.
  auto tile_col = [&](int t) {
    if constexpr (!TAIL) return t * CT;
    return t < a.tiles ? t * CT - (t == a.tiles - 1 ? a.thin : 0) : D;
  };
  const int col0 = tile_col(ct) + lane * VEC, col_end = TAIL ? tile_col(ct + 1) : D;
  bool col_ok[NV];
  int col_ld[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int col = col0 + v * kColsPerVec;
    col_ok[v] = col < col_end;
    col_ld[v] = vec_col<VEC, TAIL>(col, D);
  }
  float acc[NV][VEC];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[v][e] = 0.f;
  // Vector v's columns of a partial row.
  auto put_part = [&](float* row, int v) {
    if constexpr (FUSED) {
      store_vec_agent<VEC, TAIL>(row, D, col_ld[v], acc[v]);
    } else {
      store_vec<VEC>(row + col_ld[v], acc[v]);
    }
  };
  // An update not EARLY: the table row at dst (and Adam's moments) updated with acc; every
  // vector is loaded before the first store (lanes may share columns).
  auto update_row = [&](float* dst) {
    if (!dst) return;
    const int64_t off = dst - a.out;
    float p[NV][VEC], m[NV][VEC], s[NV][VEC];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      load_vec<VEC>(dst + col_ld[v], p[v]);
      if constexpr (OP == kOpAdam) {
        load_vec<VEC>(a.m + off + col_ld[v], m[v]);
        load_vec<VEC>(a.v + off + col_ld[v], s[v]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        if constexpr (OP == kOpAdam) adam_value(p[v][e], m[v][e], s[v][e], acc[v][e], a.opt);
        else sgd_value(p[v][e], acc[v][e], a.opt);
      }
      if (!col_ok[v]) continue;
      store_vec<VEC>(dst + col_ld[v], p[v]);
      if constexpr (OP == kOpAdam) {
        store_vec<VEC>(a.m + off + col_ld[v], m[v]);
        store_vec<VEC>(a.v + off + col_ld[v], s[v]);
      }
    }
  };
  const GT* __restrict__ grad = static_cast<const GT*>(a.grad);
  bool bad_row = false;
  // EARLY: segment ends, and so table rows, per batch.
  constexpr int kEnds = !EARLY ? 1 : ends_for<NV>();
  static_assert(kEnds >= 1 && kEnds <= RF, "table rows per batch");

#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const int wbase = p0 - 1 + w * kWave;
    const int lo = q > wbase ? q - wbase : 0;
    const int hi = q_end - wbase < kWave ? q_end - wbase : kWave;
    for (int j0 = lo; j0 < hi;) {
      int n = hi - j0 < RF ? hi - j0 : RF;
      // EARLY: at most kEnds segment ends per batch (bm: their bits), whose
      // table rows load with the batch's gradient rows.
      uint64_t bm = 0;
      float tb[kEnds][NV][VEC];
      if constexpr (EARLY) {
        bm = (ends[w] >> j0) & ((uint64_t(1) << n) - 1);
        uint64_t past = bm;  // the ends after the first kEnds
#pragma unroll
        for (int k = 0; k < kEnds; ++k) past &= past - 1;
        if (past) {
          n = __builtin_ctzll(past);
          bm &= (uint64_t(1) << n) - 1;
        }
        uint64_t mm = bm;
#pragma unroll
        for (int k = 0; k < kEnds; ++k) {
          int64_t orow = -1;  // no row: a partial row, a type past u_cap, a bad id, no end
          if (mm) {
            const int j = j0 + __builtin_ctzll(mm);
            mm &= mm - 1;
            const int s = read_lane(sw[w], j);
            if (!(s == s_f && started_before) && s >= 0 && s < a.u_cap) orow = read_lane(orw[w], j);
          }
          const __amdgpu_buffer_rsrc_t rs = table_row(a, a.out, orow);
#pragma unroll
          for (int v = 0; v < NV; ++v) table_vec<VEC>(rs, col_ld[v], tb[k][v]);
        }
      }
      // Always RF row loads (rows past n repeat row n-1, a cache hit): a load
      // under a condition makes the compiler wait for every earlier load.
      raw_t buf[RF][NV];
#pragma unroll
      for (int r = 0; r < RF; ++r) {
        const int k = read_lane(pw[w], j0 + (r < n ? r : n - 1));
        const GT* row = grad + static_cast<int64_t>(k) * a.ld_grad;
#pragma unroll
        for (int v = 0; v < NV; ++v) buf[r][v] = RV::load(row + col_ld[v]);
      }
      // All RF rows in flight before the first add: keep the scheduler from
      // interleaving the adds of early rows with the loads of later ones.
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < RF; ++r) {
        if (r < n) {
#pragma unroll
          for (int v = 0; v < NV; ++v) RV::add(acc[v], buf[r][v]);
          const int j = j0 + r;
          const bool is_end = (ends[w] >> j) & 1u;
          if (is_end || wbase + j == q_end - 1) {
            // is_end false here means a long last segment stopped at p1.
            const int s = read_lane(sw[w], j);
            float* dst;
            bool part = true;
            if (s == s_f && started_before) dst = a.part_cont + static_cast<int64_t>(c) * D;
            else if (!is_end) dst = a.part_start + static_cast<int64_t>(c) * D;
            else {
              part = false;
              const int64_t orow = rows ? read_lane(orw[w], j) : s;
              bad_row |= rows && orow < 0 && s >= 0 && s < a.u_cap;
              dst = (s >= 0 && s < a.u_cap && orow >= 0) ? a.out + orow * a.ld_out : nullptr;
            }
            if constexpr (EARLY) {
              if (!part) {  // the batch's k-th end: table row k
                const int k = __popcll(bm & ((uint64_t(1) << (j - j0)) - 1));
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                  for (int e = 0; e < VEC; ++e) {
                    float t = tb[0][v][e];
#pragma unroll
                    for (int x = 1; x < kEnds; ++x) t = k == x ? tb[x][v][e] : t;
                    sgd_value(t, acc[v][e], a.opt);
                    acc[v][e] = t;
                  }
              }
            } else if constexpr (OP != kOpStore) {
              if (!part) {
                update_row(dst);
                dst = nullptr;
              }
            }
            if (dst) {
#pragma unroll
              for (int v = 0; v < NV; ++v) {
                if (!col_ok[v]) continue;
                if (part) put_part(dst, v);
                else store_vec<VEC>(dst + col_ld[v], acc[v]);
              }
            }
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
              for (int e = 0; e < VEC; ++e) acc[v][e] = 0.f;
          }
        }
      }
      j0 += n;
    }
  }
  // Report a segment map that disagrees with offsets at the chunk start.
  const int seg_before = p0 > 0 ? read_lane(at_p0, 0) : -2, seg_p0 = read_lane(at_p0, 1);
  if (started_before) bad |= seg_before != s_f || seg_p0 != s_f;
  else bad |= seg_before == seg_p0 || seg_p0 != (p0 == A.o1 ? A.u + 1 : A.u);
  if (ballot(bad) && lane == 0) raise_err(a.dev_err, LM_DEVERR_CAPACITY);
  if (ballot(bad_row) && lane == 0) raise_err(a.dev_err, LM_DEVERR_ID_RANGE);

  // 4. Fused: the pieces this wave wrote (at most two: of the segment it found
  //    running, and of the one it left running). The wait also orders the
  //    claims (lane 1's too) before the additions.
  if constexpr (FUSED) {
    if (!(long_f || long_l)) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint64_t* const first_word = a.flags + ct;
    bool flagged = false;
    auto piece_done = [&](int s, int cs, int P) {
      if (P >= kHeadPieces) {
        if (!flagged && lane == 0)
          word_add(AgentWords{}, first_word + size_t(c) * a.tiles, kPieceFlag);
        flagged = true;  // both pieces may be of heads
        return;
      }
      uint32_t n = 0;
      if (lane == 0)
        n = word_count(word_add(AgentWords{}, first_word + size_t(cs) * a.tiles, 1));
      if (first_lane(n) != P + 1) return;
      asm volatile("" ::: "memory");  // no piece is read before its count
      // The last one: every piece is there.
      constexpr int RP = NV * VEC >= 16 ? 4 : 8;  // pieces in flight
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[v][e] = 0.f;
      if constexpr (TAIL && OP != kOpAdam) {
        // Two resources for all of them, piece 0 and the others.
        float p0[NV][VEC];
        const __amdgpu_buffer_rsrc_t first = part_rows(piece_row(a, cs, 0), 1, D);
        const __amdgpu_buffer_rsrc_t rest = part_rows(piece_row(a, cs, 1), P, D);
#pragma unroll
        for (int v = 0; v < NV; ++v) load_part_vec<VEC>(first, 0, col_ld[v], p0[v]);
        for (int t0 = 1; t0 <= P; t0 += RP) {
          float buf[RP][NV][VEC];
#pragma unroll
          for (int r = 0; r < RP; ++r)
#pragma unroll
            for (int v = 0; v < NV; ++v)
              load_part_vec<VEC>(rest, (t0 + r <= P ? t0 + r - 1 : 0) * D * 4, col_ld[v], buf[r][v]);
          if (t0 == 1)
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
              for (int e = 0; e < VEC; ++e) acc[v][e] += p0[v][e];
#pragma unroll
          for (int r = 0; r < RP; ++r)
            if (t0 + r <= P)
#pragma unroll
              for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[v][e] += buf[r][v][e];
        }
      } else {
        for (int t0 = 0; t0 <= P; t0 += RP) {
          float buf[RP][NV][VEC];
#pragma unroll
          for (int r = 0; r < RP; ++r)
#pragma unroll
            for (int v = 0; v < NV; ++v)
              load_vec_agent<VEC, TAIL>(piece_row(a, cs, t0 + r <= P ? t0 + r : 0) + col_ld[v],
                                  buf[r][v]);
#pragma unroll
          for (int r = 0; r < RP; ++r)
            if (t0 + r <= P)
#pragma unroll
              for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[v][e] += buf[r][v][e];
        }
      }
      if (s >= a.u_cap) return;
      const int64_t orow = out_row_of(a, s);
      if (orow < 0) return;
      float* dst = a.out + orow * a.ld_out;
      if constexpr (OP != kOpStore) {
        update_row(dst);
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v)
          if (col_ok[v]) store_vec<VEC>(dst + col_ld[v], acc[v]);
      }
    };
    if (long_f) piece_done(s_f, cs_f, P_f);
    if (starts_long) piece_done(s_l, c, chunk_of(B.o1 - 1, s_l) - c);
  }
}

// Sum the pieces of every long segment that spans chunks (piece 0 is
// part_start[c], piece t >= 1 is part_cont[c + t], added in order of t).
// Grid: one workgroup of kFixWaves waves per kFixChunks chunks and per
// column tile of 64 * VEC columns. Few chunks start such a segment, so a
// workgroup reads the desc and npieces entries of its chunks with one
// coalesced load and a ballot, and only waves with work touch the partial
// rows (launching a wave per chunk cost more than the sums). The partial
// rows were just written, so the sums are bound by load latency: every wave
// issues all its piece loads before it waits for any. A segment of fewer
// than RF further pieces is summed by one wave; a longer one (a head of the
// Zipf law) by all kFixWaves waves, wave v adding pieces v, v + kFixWaves,
// ... in order, their partial rows then added in wave order through LDS.
// Long segments start at least RF chunks apart, so with kFixChunks <= RF a
// workgroup holds at most one head, and with kFixChunks <= kFixWaves each
// wave at most one shorter segment.
#ifndef LMZ_SEG_FIX_WAVES
#define LMZ_SEG_FIX_WAVES 8          // waves of a fix-up workgroup
#endif
#ifndef LMZ_SEG_FIX_CHUNKS
#define LMZ_SEG_FIX_CHUNKS 8         // chunks a fix-up workgroup looks after
#endif
constexpr int kFixWaves = LMZ_SEG_FIX_WAVES;
constexpr int kFixThreads = kFixWaves * kWave;
constexpr int kFixChunks = LMZ_SEG_FIX_CHUNKS;
static_assert(kFixChunks <= kFixWaves && kFixChunks <= LMZ_SEG_FIX_RF,
              "at most one short segment per wave and one head per workgroup");

template <int VEC, int RF, int OP>
__global__ __launch_bounds__(kFixThreads) void k_segsum_fix(SegArgs a) {
  constexpr int kCols = kWave * VEC;  // columns of a tile
  __shared__ float s_part[kFixWaves][kCols];
  const int lane = lane_id();
  const int wave = first_lane(static_cast<int>(threadIdx.x >> 6));
  const int D = a.D;
  const int U = first_lane(static_cast<int>(*a.num_unique));
  const int c0 = blockIdx.x * kFixChunks;
  const int col = blockIdx.y * kCols + lane * VEC;
  const int col_ld = col < D ? col : D - VEC;  // past the end: a valid, unstored vector

  // Chunks c0 + i that start a long segment (the same masks in every wave).
  const int ci = c0 + lane;
  const bool mine = lane < kFixChunks && ci < a.nchunks;
  const int sd = mine ? a.desc[ci] : -1;
  const int np = mine ? a.npieces[ci] : 0;
  const bool has = sd >= 0 && sd < U && sd < a.u_cap && np >= 1 && np <= a.nchunks - 1 - ci;
  const uint64_t todo = ballot(has);
  if (!todo) return;
  const uint64_t heads = ballot(has && np >= RF);
  const uint64_t shorts = todo & ~heads;
  auto piece = [&](int cs, int t) {
    return (t == 0 ? a.part_start + static_cast<int64_t>(cs) * D
                   : a.part_cont + static_cast<int64_t>(cs + t) * D) + col_ld;
  };

  // This wave's short segment: the wave-th of the mask.
  uint64_t m = shorts;
  for (int j = 0; j < wave && m; ++j) m &= m - 1;
  const int is = m ? __builtin_ctzll(m) : -1;
  const int ss = is >= 0 ? read_lane(sd, is) : -1, sP = is >= 0 ? read_lane(np, is) : 0;
  // The head, if any.
  const int ih = heads ? __builtin_ctzll(heads) : -1;
  const int hs = ih >= 0 ? read_lane(sd, ih) : -1, hP = ih >= 0 ? read_lane(np, ih) : 0;

  float sbuf[RF][VEC], hbuf[RF][VEC];
  if (is >= 0) {
#pragma unroll
    for (int r = 0; r < RF; ++r) load_vec<VEC>(piece(c0 + is, r <= sP ? r : 0), sbuf[r]);
  }
  if (ih >= 0) {
#pragma unroll
    for (int r = 0; r < RF; ++r) {
      const int t = wave + r * kFixWaves;
      load_vec<VEC>(piece(c0 + ih, t <= hP ? t : wave), hbuf[r]);
    }
  }
  if (is >= 0) {
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = sbuf[0][e];
#pragma unroll
    for (int r = 1; r < RF; ++r)
      if (r <= sP)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] += sbuf[r][e];
    const int64_t orow = out_row_of(a, ss);
    if (col < D && orow >= 0) {
      TableVec<VEC, OP> tv;
      tv.load(a, orow * a.ld_out + col);
      tv.finish(a, orow * a.ld_out + col, acc);
    }
  }
  if (ih < 0) return;  // the same in every wave: no barrier below is skipped by only some
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
#pragma unroll
  for (int r = 0; r < RF; ++r)
    if (wave + r * kFixWaves <= hP)
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += hbuf[r][e];
  // Heads longer than kFixWaves * RF pieces: further rounds.
  for (int t0 = wave + kFixWaves * RF; t0 <= hP; t0 += kFixWaves * RF) {
#pragma unroll
    for (int r = 0; r < RF; ++r) {
      const int t = t0 + r * kFixWaves;
      load_vec<VEC>(piece(c0 + ih, t <= hP ? t : t0), hbuf[r]);
    }
#pragma unroll
    for (int r = 0; r < RF; ++r)
      if (t0 + r * kFixWaves <= hP)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] += hbuf[r][e];
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) s_part[wave][lane * VEC + e] = acc[e];
  __syncthreads();
  // Thread x adds column x of the tile over the waves in order.
  const int64_t orow = out_row_of(a, hs);
  for (int x = threadIdx.x; x < kCols; x += kFixThreads) {
    const int cx = blockIdx.y * kCols + x;
    if (cx < D && orow >= 0) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < kFixWaves; ++w) sum += s_part[w][x];
      TableVec<1, OP> tv;
      tv.load(a, orow * a.ld_out + cx);
      tv.finish(a, orow * a.ld_out + cx, &sum);
    }
  }
}

template <int R>
constexpr int t_for() {
  constexpr int t = R / LMZ_SEG_TDIV;
  return t < 1 ? 1 : (t > 64 ? 64 : t);
}

// Rows per gather batch: more for long chunks (R >= LMZ_SEG_LONG_R), whose
// walks are long enough to use the extra rows in flight.
template <int NV, int R>
constexpr int rf_for() {
  return NV >= 4 ? (R >= LMZ_SEG_LONG_R ? LMZ_SEG_RF4_LONG : LMZ_SEG_RF4)
                 : (R >= LMZ_SEG_LONG_R ? LMZ_SEG_RF2_LONG : LMZ_SEG_RF2);
}

// lm_segsum_adam's rows per batch: as lm_segsum's, but for its three table
// rows at most 4 rows of 4 vectors, or 8 of fewer.
template <int NV, int R>
constexpr int rf_adam_for() {
  constexpr int rf = rf_for<NV, R>(), most = NV >= 4 ? LMZ_SEG_ADAM_RF4 : 8;
  return rf > most ? most : rf;
}

// Workgroups of the plain walk (kOpStore) that fit on a compute unit, fused or
// not: defined with the plain kernels, which the update instantiations size
// their chunks by.
template <typename GT, int VEC, int NV, int R, bool TAIL>
int plain_blocks(bool fused);

template <typename GT, int VEC, int NV, int R, int OP, bool TAIL, bool EARLY>
static void launch_one(SegArgs& a, int tiles, hipStream_t st) {
  constexpr int T = t_for<R>();
  constexpr int RF = OP == kOpAdam ? rf_adam_for<NV, R>() : rf_for<NV, R>();
  constexpr int CT = NV * kWave * VEC;
  a.tiles = tiles;
  a.tile_cols = CT;
  // A last tile narrower than a vector would repeat columns of the tile
  // before it, which another wave updates: it then starts one vector earlier
  // (and the fix-up is a launch of its own, as the columns of its workgroups
  // no longer lie inside one tile each).
  const int rest = a.D % CT;
  a.thin = tiles > 1 && rest > 0 && rest < VEC ? VEC : 0;
  if (a.thin) a.fused = 0;
  // The rounds are those of the plain kernel (kOpStore) for the update
  // instantiations too: its occupancy fixes the chunks, and with them the
  // order of every sum, so lm_segsum_sgd and _adam add in lm_segsum's order.
  const bool fused = VEC >= 2 && a.fused;
  const int cus = stream_cus(st);
  const int64_t room = int64_t(plain_blocks<GT, VEC, NV, R, TAIL>(fused)) * kSegWaves * cus;
  const ChunkCount cc = whole_rounds(a.K, a.D, a.u_cap, R, sizeof(GT) == 2, tiles, a.nchunks,
                                     a.max_chunks, room, cus);
  a.nchunks = cc.n;
  a.enough = cc.enough;
  const int blocks = (a.nchunks + kSegWaves - 1) / kSegWaves;
  if constexpr (VEC >= 2) {
    if (fused) {
      a.main_blocks = blocks * tiles;
      const int fix_blocks = (a.nchunks - 1) / kHeadPieces * a.fix_tiles;
      k_segsum<GT, VEC, NV, RF, R, T, true, OP, TAIL, EARLY>
          <<<dim3(a.main_blocks + fix_blocks), kSegThreads, 0, st>>>(a);
      return;
    }
  }
  k_segsum<GT, VEC, NV, RF, R, T, false, OP, TAIL, EARLY>
      <<<dim3(blocks, tiles), kSegThreads, 0, st>>>(a);
}

// Whether an update loads the table rows of a batch's segment ends with the
// batch's gradient rows (early). An end then costs no round trip of its own,
// but a batch closes at its last end and takes more registers. Otherwise (late)
// the walk keeps lm_segsum's batches and waits for the table row at every end.
// Measured, early / late, us per call:
//   SGD fp32, up to 512 columns: 106,496 ids over 800K words, D = 512 72.7 /
//     75.4, 30,011 over 50K, D = 300 18.1 / 19.0, 40,000 over 2,000 21.6 / 20.3;
//     600,000 over 300K (chunks of 512) 469 / 412;
//   wider (4 vectors per lane; early 3 rows and 2 ends per batch): D = 1024,
//     65,536 over 800K 85.4 / 84.6, 200,000 over 100K 220 / 207, over 12,500 193 /
//     181, 262,144 over 2M 383 / 366, 8,192 over 100K 16.9 / 18.1; D = 1792, 19,200
//     over 15,437 53.1 / 51.8; D = 2048, 65,536 over 800K 165 / 162. With Unique
//     beside it on another stream, 65,536 over 800K, D = 1024: a step 110.9 / 102.5
//     (early, four workgroups take every register of a compute unit, and
//     Unique's kernels wait for them);
//   SGD bf16, D = 1024: 100,000 ids over 100K words 93.4 / 84.8;
//   Adam (one end, 2 rows per batch early), D = 1024: 262,144 ids over 2M words
//     954 / 909, 65,536 over 800K 226 / 210, 200,000 over 400K 646 / 494,
//     D = 1792: 19,200 over 98 67 / 39. Late with 2 or 3 rows per batch,
//     or loading the three rows' vectors one or two at a time, measured within
//     2% of 4 rows and all vectors at the large sizes and 1-10% slower at
//     19,200 ids.
// So only SGD with fp32 rows of up to 512 columns, chunks below 512 rows and no
// more than 32 tokens per type it may find (there are at most min(K, rows_cap))
// is early.
template <typename GT, int NV, int OP, int R>
constexpr bool may_be_early() {
  return OP == kOpSgd && sizeof(GT) == 4 && NV <= 2 && R < LMZ_SEG_LONG_R;
}
template <typename GT, int VEC, int NV, int R, int OP, bool TAIL>
static void launch_when(SegArgs& a, int tiles, hipStream_t st) {
  if constexpr (may_be_early<GT, NV, OP, R>()) {
    if (a.K < kFewTokens * a.u_cap) {
      launch_one<GT, VEC, NV, R, OP, TAIL, true>(a, tiles, st);
      return;
    }
  }
  launch_one<GT, VEC, NV, R, OP, TAIL, false>(a, tiles, st);
}

template <typename GT, int VEC, int NV, int OP, bool TAIL>
static hipError_t launch_r(SegArgs& a, hipStream_t st) {
  constexpr int CT = NV * kWave * VEC;
  const int tiles = (a.D + CT - 1) / CT;
  switch (a.R) {
    case 16: launch_when<GT, VEC, NV, 16, OP, TAIL>(a, tiles, st); break;
    case 32: launch_when<GT, VEC, NV, 32, OP, TAIL>(a, tiles, st); break;
    case 64: launch_when<GT, VEC, NV, 64, OP, TAIL>(a, tiles, st); break;
    case 128: launch_when<GT, VEC, NV, 128, OP, TAIL>(a, tiles, st); break;
    case 256: launch_when<GT, VEC, NV, 256, OP, TAIL>(a, tiles, st); break;
    default: launch_when<GT, VEC, NV, 512, OP, TAIL>(a, tiles, st); break;
  }
  return hipGetLastError();
}

// 16-byte vectors wherever a row holds one (4 fp32 or 8 bf16 columns), at any
// alignment, up to 1024 columns of a row per wave; other rows, and bf16 rows
// that column_per_lane names, take a column per lane. A column per lane had
// been the path of every row that is no whole number of aligned vectors: four
// times the load instructions for the same bytes, and a second launch for the
// fix-up. Measured with SGD at 30,011 ids over 50K words, D = 650 fp32: walk and
// fix-up 37.3 + 7.6 us before, 40.1 us in one launch now.
template <typename GT, int OP, bool TAIL>
static hipError_t launch_vec(SegArgs& a, hipStream_t st) {
  constexpr int VEC = 16 / static_cast<int>(sizeof(GT));
  const int nv = (a.D + kWave * VEC - 1) / (kWave * VEC);
  if (nv <= 1) return launch_r<GT, VEC, 1, OP, TAIL>(a, st);
  if constexpr (sizeof(GT) == 4)
    if (nv > 2) return launch_r<GT, VEC, 4, OP, TAIL>(a, st);
  return launch_r<GT, VEC, 2, OP, TAIL>(a, st);
}

template <typename GT, int OP>
hipError_t seg_walk(SegArgs& a, hipStream_t st) {
  constexpr int VEC = 16 / static_cast<int>(sizeof(GT));
  if (a.by_column) {
    if constexpr (sizeof(GT) == 2) {
      if (a.D > 2 * kWave) return launch_r<GT, 1, 4, OP, false>(a, st);
      if (a.D > kWave) return launch_r<GT, 1, 2, OP, false>(a, st);
    }
    return launch_r<GT, 1, 1, OP, false>(a, st);
  }
  return a.D % VEC ? launch_vec<GT, OP, true>(a, st) : launch_vec<GT, OP, false>(a, st);
}

template <int OP>
void seg_fix(const SegArgs& a, hipStream_t st) {
  const uint32_t fix_blocks = static_cast<uint32_t>((a.nchunks + kFixChunks - 1) / kFixChunks);
  if (a.D % 4 == 0)
    k_segsum_fix<4, LMZ_SEG_FIX_RF, OP>
        <<<dim3(fix_blocks, (a.D + 255) / 256), kFixThreads, 0, st>>>(a);
  else
    k_segsum_fix<1, LMZ_SEG_FIX_RF, OP>
        <<<dim3(fix_blocks, (a.D + 63) / 64), kFixThreads, 0, st>>>(a);
}

}  // namespace lmz
