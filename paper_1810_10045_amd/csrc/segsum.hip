// Seg-Sum, the host side: workspace layout, chunk counts and the choice of
// the launch form. The kernels and their design: segsum_kernels.hpp.
#include <atomic>
#include <cstdlib>

#include "segsum_args.hpp"

namespace lmz {

// Tuning knobs (overridable at build time).
#ifndef LMZ_SEG_TARGET_CHUNKS
#define LMZ_SEG_TARGET_CHUNKS 1024   // R = the power of two near K / this (16..512)
#endif
#ifndef LMZ_SEG_WRITE_X2_F32
#define LMZ_SEG_WRITE_X2_F32 2       // fp32 rows: cost of a row written / a row read, times 2
#endif
#ifndef LMZ_SEG_WRITE_X2_BF16
#define LMZ_SEG_WRITE_X2_BF16 4      // bf16 rows: the same ratio, times 2
#endif
#ifndef LMZ_SEG_FUSED
#define LMZ_SEG_FUSED 1              // fix-up workgroups in the walk's launch (one column tile)
#endif
#ifndef LMZ_SEG_FUSED_MAX_D
#define LMZ_SEG_FUSED_MAX_D 4096     // widest rows walked and fixed up in one launch
#endif

struct SegLayout {
  int R, max_chunks;
  size_t cont, start, desc, npieces, flags, total;
};

static inline size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

// Costs: a sorted position (a row read) costs rw = 2 * sizeof(grad) per
// column, a segment end (a row written, always fp32) ww = 4 * X2, where X2 / 2
// is the cost of a written row relative to a read row. Measured on MI355X:
// with fp32 rows a written row is best weighted by its bytes (X2 = 2: 1-5%
// faster Seg-Sum than X2 = 4 on the fp32 workloads), with bf16 rows at twice
// the bytes of a read row (X2 = 4: 3% faster than X2 = 2 on the bf16 merge).
// A call has at most rw * K + ww * min(K, u_cap) of it, at most rw * R per
// chunk.
static inline int read_cost(int gtype) { return gtype == LM_BF16 ? 4 : 8; }
static inline int write_cost(int gtype) {
  return 4 * (gtype == LM_BF16 ? LMZ_SEG_WRITE_X2_BF16 : LMZ_SEG_WRITE_X2_F32);
}
constexpr int kMaxWriteCost =
    4 * (LMZ_SEG_WRITE_X2_BF16 > LMZ_SEG_WRITE_X2_F32 ? LMZ_SEG_WRITE_X2_BF16 : LMZ_SEG_WRITE_X2_F32);
static inline int64_t chunks_for(int64_t K, int R, int rw, int ww, int64_t u_cap) {
  const int64_t ub = u_cap < K ? u_cap : K;
  return (int64_t(rw) * K + int64_t(ww) * ub + int64_t(rw) * R - 1) / (int64_t(rw) * R);
}

static SegLayout seg_layout(int64_t K, int64_t D) {
  SegLayout L{};
  const int64_t want = (K + LMZ_SEG_TARGET_CHUNKS - 1) / LMZ_SEG_TARGET_CHUNKS;
  int R = kMinR;
  while (R < want && R < kMaxR) R *= 2;
  L.R = R;
  L.max_chunks = static_cast<int>(chunks_for(K, R, 4, kMaxWriteCost, K));  // any dtype and capacity
  const size_t n = size_t(L.max_chunks);
  size_t off = 0;
  L.cont = off;     off += a256(n * D * 4);
  L.start = off;    off += a256(n * D * 4);
  L.desc = off;     off += a256(n * 4);
  L.npieces = off;  off += a256(n * 4);
  L.flags = off;    off += a256(n * size_t((D + 1023) / 1024) * 8);  // per chunk and column tile
  L.total = off;
  return L;
}

size_t segsum_workspace_bytes(int64_t K, int64_t D) { return seg_layout(K, D).total; }

// Multiprocessors of the current device (queried once per device).
static int device_cus() {
  static std::atomic<int> cus[64];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return 0;
  }
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Multiprocessors a launch on stream st may use: a stream created with a CU
// mask runs its workgroups on the masked ones only. Any other stream, or a
// failed query, gets the whole device.
int stream_cus(hipStream_t st) {
  const int n = device_cus();
  uint32_t mask[32] = {};
  if (hipExtStreamGetCUMask(st, 32, mask) != hipSuccess) {
    (void)hipGetLastError();
    return n;
  }
  int c = 0;
  for (uint32_t m : mask) c += __builtin_popcount(m);
  return c > 0 && c < n ? c : n;
}

// Whole rounds of waves. The walk's waves (chunks x column tiles) of equal
// cost run in rounds of as many waves as fit at once on the compute units
// the launch's stream may use. Where a
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
// Shorter chunks (R = 32 .. 128) make kWaves waves, two workgroups on each
// compute unit, where there would be well below that many and none gets fewer
// than kMinR rows, and no more than
// kEnoughWaves unless a chunk would exceed R, as every cut may cost a partial
// row. Measured, waves before -> now: Adam, D = 1792, 19,200 ids over 98 43.2
// us (1,208) -> 39.7 (1,536 waves 41.6, 2,560 43.8); D = 300, 40,000 over 2,000
// 40.4 (627) -> 25.2; SGD, D = 512, 106,496 over 800K 71.7 (1,664) -> 67.5;
// bf16, D = 1792, 19,200 over 15,437 38.0 (5,058) -> 33.6 (2,560). Close to
// kWaves it loses: 30,011 over 50K, D = 650 38.3 (1,876) -> 40.5. So does it
// with chunks of 10 rows: 20,000 over 98, D = 200 17.2 us (2,048), 13.6 (1,280).
// Rows that are no whole number of vectors write their partial rows a column
// at a time: half as many waves. 21,386 over 2,865, D = 358: 22.2 us (2,048),
// 17.7 (1,024), 18.9 (669 as they come); 60,000 over 500, D = 358 45.0, 32.1,
// 32.2; SGD, 100,000 over 1,000, D = 513 59.6, 51.9, 55.3.
constexpr int kWaves = 2048, kTailWaves = kWaves / 2, kEnoughWaves = 2560;
void whole_rounds(SegArgs& a, int64_t waves_per_round) {
  a.enough = a.nchunks;
  if (waves_per_round <= 0 || a.tiles <= 0) return;
  const int64_t waves = int64_t(a.nchunks) * a.tiles;
  const int64_t last = waves % waves_per_round;
  const bool tail = a.D % (16 / (a.rw / 2)) != 0;  // rw: twice a column's bytes
  const int fill = tail ? kTailWaves : kWaves;
  int64_t want = a.nchunks;
  if (a.R >= 256 ? last != 0 && (waves < waves_per_round || 2 * last < waves_per_round)
                 : waves > waves_per_round && last != 0 && 2 * last < waves_per_round) {
    const int64_t rounds = (waves + waves_per_round - 1) / waves_per_round;
    want = (rounds * waves_per_round + a.tiles - 1) / a.tiles;
  } else if (a.R > kMinR && a.R < 256 && waves < fill - fill / 8) {
    want = (fill + a.tiles - 1) / a.tiles;
    if (want > a.K / kMinR) want = a.K / kMinR;
  }
  if (want > a.max_chunks) want = a.max_chunks;
  if (want > a.nchunks) a.nchunks = static_cast<int>(want);
  a.enough = a.R < 256 ? (kEnoughWaves + a.tiles - 1) / a.tiles : a.nchunks;
}

template <int OP>
static hipError_t run_op(SegArgs& a, int gtype, hipStream_t st) {
  const hipError_t e =
      gtype == LM_F32 ? seg_walk<float, OP>(a, st) : seg_walk<bf16_t, OP>(a, st);
  if (e != hipSuccess || a.fused) return e;
  seg_fix<OP>(a, st);
  return hipGetLastError();
}

// Test hook for the failure path of the one-launch form: while set, the
// fix-up workgroups wait for a flag value that no walk writes, so every such
// wait gives up after `limit` polls and raises LM_DEVERR_SPIN; the launch
// still drains and stays inside its buffers. Off by default.
static std::atomic<bool> g_force_wait_failure{false};
static std::atomic<uint32_t> g_forced_spin_limit{kSpinLimit};

void segsum_force_wait_failure(bool enable, uint32_t limit) {
  g_forced_spin_limit.store(limit < 1 ? 1u : limit, std::memory_order_relaxed);
  g_force_wait_failure.store(enable, std::memory_order_relaxed);
}

// The host switch to the two-launch form (lm_segsum_set_two_launches):
// -1 until the first call reads LMZIPF_SEGSUM_TWO_LAUNCHES, then 0 or 1.
static std::atomic<int> g_two_launches{-1};

static bool two_launches() {
  int v = g_two_launches.load(std::memory_order_relaxed);
  if (v < 0) {
    const char* e = std::getenv("LMZIPF_SEGSUM_TWO_LAUNCHES");
    const int from_env = (e && e[0] == '1') ? 1 : 0;
    int expected = -1;
    g_two_launches.compare_exchange_strong(expected, from_env, std::memory_order_relaxed);
    v = g_two_launches.load(std::memory_order_relaxed);
  }
  return v == 1;
}

int segsum_set_two_launches(bool enable) {
  const int prev = two_launches() ? 1 : 0;
  g_two_launches.store(enable ? 1 : 0, std::memory_order_relaxed);
  return prev;
}

int segsum_run(const void* grad, int gtype, int64_t K, int64_t D, int64_t ld_grad,
               const int32_t* perm, const int32_t* inverse, const int32_t* offsets,
               const int64_t* num_unique, int64_t u_cap, float* out, int64_t ld_out,
               int32_t* dev_err, void* ws, size_t ws_bytes, hipStream_t st,
               const void* row_ids, int row_ids64, int64_t out_rows, int op,
               const OptParams& opt, float* m, float* v) {
  const SegLayout L = seg_layout(K, D);
  if (ws_bytes < L.total) return LM_E_WORKSPACE;
  if (K == 0 || D == 0 || u_cap == 0) return LM_OK;
  char* w = static_cast<char*>(ws);
  SegArgs a{};
  a.spin_limit = kSpinLimit;
  a.grad = grad;
  a.ld_grad = ld_grad;
  a.K = static_cast<int>(K);
  a.D = static_cast<int>(D);
  a.perm = perm;
  a.inverse = inverse;
  a.offsets = offsets;
  a.num_unique = num_unique;
  a.u_cap = u_cap;
  a.out = out;
  a.ld_out = ld_out;
  a.row_ids = row_ids;
  a.row_ids64 = row_ids64;
  a.out_rows = row_ids ? out_rows : u_cap;
  a.part_cont = reinterpret_cast<float*>(w + L.cont);
  a.part_start = reinterpret_cast<float*>(w + L.start);
  a.desc = reinterpret_cast<int32_t*>(w + L.desc);
  a.npieces = reinterpret_cast<int32_t*>(w + L.npieces);
  a.R = L.R;
  a.rw = read_cost(gtype);
  a.ww = write_cost(gtype);
  a.nchunks = static_cast<int>(chunks_for(K, L.R, a.rw, a.ww, u_cap));
  a.max_chunks = L.max_chunks;
  a.dev_err = dev_err;
  a.opt = opt;
  a.m = m;
  a.v = v;

  // One launch for the walk and the fix-up on the vector path (rows of at
  // least one 16-byte vector, at any alignment). Measured at
  // K = 1,048,576, D = 2048 fp32 (two column tiles): 1,490 us as the walk
  // and a separate fix-up kernel, 1,411 us in one launch, the fix-up
  // workgroups running in the walk's last round.
  a.fused = LMZ_SEG_FUSED != 0 && D >= (gtype == LM_F32 ? 4 : 8) && D <= LMZ_SEG_FUSED_MAX_D &&
            !two_launches();
  // A captured launch would replay with this call's tag every time, and a
  // replay could take the previous replay's pieces for its own: under stream
  // capture the fix-up is a second launch, which keeps no state across calls.
  if (a.fused) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      a.fused = 0;
    }
  }
  if (a.fused) {
    static std::atomic<uint64_t> calls{0x3779b97f4a7ull};  // any start
    a.flags = reinterpret_cast<uint64_t*>(w + L.flags);
    a.tag = calls.fetch_add(1, std::memory_order_relaxed) & ((uint64_t(1) << 44) - 1);
    const bool fail = g_force_wait_failure.load(std::memory_order_relaxed);
    a.wait_tag = fail ? ~a.tag : a.tag;
    a.spin_limit = fail ? g_forced_spin_limit.load(std::memory_order_relaxed) : kSpinLimit;
    a.fix_tiles = static_cast<int>((D + kFusedCols - 1) / kFusedCols);
  }
  return launch_status(op == kOpSgd    ? run_op<kOpSgd>(a, gtype, st)
                       : op == kOpAdam ? run_op<kOpAdam>(a, gtype, st)
                                       : run_op<kOpStore>(a, gtype, st));
}

}  // namespace lmz
