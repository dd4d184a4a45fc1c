// Seg-Sum, the host side: workspace layout, chunk counts and the choice of
// the launch form. The kernels and their design: segsum_kernels.hpp.
#include <atomic>
#include <cstdlib>

#include "segsum_args.hpp"
#include "segsum_words.hpp"

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
#define LMZ_SEG_FUSED 1              // the fix-up in the walk's launch
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

  // One launch for the walk and the fix-up on the vector path. Measured at
  // K = 1,048,576, D = 2048 fp32 (two column tiles): 1,490 us as the walk
  // and a separate fix-up kernel, 1,411 us in one launch, the fix-up
  // workgroups running in the walk's last round.
  a.by_column = column_per_lane(reinterpret_cast<uintptr_t>(grad), ld_grad, D, gtype == LM_BF16);
  a.fused = LMZ_SEG_FUSED != 0 && !a.by_column && D <= LMZ_SEG_FUSED_MAX_D && !two_launches();
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
    static std::atomic<uint64_t> calls{0x9e3779b97f4a7cull};  // any start
    a.flags = reinterpret_cast<uint64_t*>(w + L.flags);
    a.tag = calls.fetch_add(1, std::memory_order_relaxed) & kTagMask;
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
