// Budgeted retention and cache fill (paper eq. 5; Section 3.1.3 "Capped capacity", "Cached prefilling").
//
// One launch.  Workgroups with blockIdx.y < slices own one (sequence, KV head) each, or, where the heads leave most of the chip
// idle, a slice of its kept entries: every one of them selects for itself, writes its slice of the kept positions and
// gathers its slice of the rows.
//   candidates among the out-of-window positions 0 .. n-window-1 are sinks or logits above the threshold;
//   their keys (an order-preserving integer image of the fp32 key, 0 for non-candidates) are read once and
//   stay in registers.  If more than `budget` exist, an exact radix select (up to 4 passes of 8 bits) finds
//   the budget-th largest key, and ties at that key are resolved towards lower positions by an ordered scan.
//   The same ordered scan (wave prefix sums, no atomics on results) writes the kept positions and keys
//   ascending by position, so the result is deterministic; the workgroup then gathers the kept K/V rows into
//   the compact segment.
// Workgroups with blockIdx.y >= slices copy the last min(n, window) tokens and their logits into the ring
// (slot = position % window); that part does not depend on the selection and overlaps with it.
//
// The continuation of a prefill runs the same kernel over its extended sequences (append.hip): an element's key then
// comes from the array of keys that were final before the call or from the fresh logits, by its true position, and kept
// positions are written back as true positions.
#include <type_traits>

#include "ltea_common.h"
#include "ltea_kernels.h"

namespace ltea {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kItems = 4;                        // consecutive positions per thread per chunk
constexpr int kChunk = kSelThreads * kItems;     // positions per chunk
constexpr int kSub = 8;                          // sub-histograms per digit (spreads same-digit LDS atomics)
constexpr int kRingRows = 256;                   // ring rows per copy workgroup

__device__ __forceinline__ float key_of_order_key(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u ^ 0x80000000u) : ~u);
}

// Exclusive prefix sum of `val` over the block (thread order); `total` receives the block sum.
// `scratch` holds kSelWaves+1 ints of LDS. Contains two barriers.
__device__ __forceinline__ int block_exclusive_scan(int val, int* scratch, int& total) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int inc = wave_scan_add(val);
  __syncthreads();  // protect scratch from the previous use
  if (lane == kWave - 1) scratch[wave] = inc;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) {
    int t = scratch[w];
    if (w < wave) before += t;
    all += t;
  }
  total = all;
  return before + inc - val;
}

struct RetainArgs {
  const float* logits; int64_t total; const int32_t* cu; int Hkv, window, budget, sink; float tau; int rho;
  const char* k; const char* v; int64_t tok_bytes, head_bytes; int row_bytes;   // K/V views in bytes
  char* k_win; char* v_win; float* win_score; char* k_ret; char* v_ret;
  float* ret_score; int32_t* ret_pos; int32_t* ret_count; int32_t* n_seen; int32_t* n_scored;
  int slices, slice_rows;   // selection workgroups per head, and the kept entries that each but the last one moves
  AppendPlan plan;      // continuation only
};

// What element e of a sequence is.  A prefill's elements are its positions; an extended sequence of a continuation is
// [pad | kept entries | ring | new tokens], with cu = plan.cu_ext and the fresh logits packed by plan.cu_score.
template <bool APPEND> struct Elements;
template <> struct Elements<false> {
  const float* z;
  __device__ Elements(const RetainArgs& a, int, int h, int64_t, int64_t lo, int) : z(a.logits + (int64_t)h * a.total + lo) {}
  __device__ __forceinline__ float logit(int j) const { return z[j]; }
  __device__ __forceinline__ bool is_sink(const RetainArgs& a, int j) const { return j < a.sink; }
  __device__ __forceinline__ bool exists(int) const { return true; }
  __device__ __forceinline__ int position(const RetainArgs&, int64_t, int j) const { return j; }
  __device__ __forceinline__ int seen(int n) const { return n; }
};
template <> struct Elements<true> {
  const float *key, *fresh;
  int pad, prefix, shift, first_fresh, len;     // true position = element + shift from the prefix on
  __device__ Elements(const RetainArgs& a, int b, int h, int64_t head, int64_t lo, int n) {
    const int n_old = a.plan.n_old[b], w_old = a.plan.w_old[b];
    prefix = a.plan.prefix[b];
    pad = prefix - a.plan.old_count[head];
    shift = n_old - w_old - prefix;
    first_fresh = n_old - a.rho - shift;
    // fresh[e]: the scored rows begin with the last min(w_old, 2 rho) ring tokens
    const int ctx = w_old < 2 * a.rho ? w_old : 2 * a.rho;
    fresh = a.logits + (int64_t)h * a.total + a.plan.cu_score[b] - (prefix + w_old - ctx);
    key = a.plan.ext_key + (int64_t)h * a.plan.total_ext + lo;
    len = n;
  }
  __device__ __forceinline__ float logit(int j) const { return j >= first_fresh && j >= prefix ? fresh[j] : key[j]; }
  __device__ __forceinline__ bool is_sink(const RetainArgs& a, int j) const { return j >= prefix && j + shift < a.sink; }
  __device__ __forceinline__ bool exists(int j) const { return j >= pad; }
  __device__ __forceinline__ int position(const RetainArgs& a, int64_t head, int j) const {
    return j < prefix ? a.plan.sorted_pos[head * a.budget + (j - pad)] : j + shift;
  }
  __device__ __forceinline__ int seen(int n) const { return n + shift; }
};

// Copies one K row and one V row of row_bytes (a multiple of 16) in 16-byte pieces; piece index `pc`.
__device__ __forceinline__ void copy_piece(const RetainArgs& a, int64_t src_off, char* dk, char* dv, int pc) {
  reinterpret_cast<u32x4*>(dk)[pc] = reinterpret_cast<const u32x4*>(a.k + src_off)[pc];
  reinterpret_cast<u32x4*>(dv)[pc] = reinterpret_cast<const u32x4*>(a.v + src_off)[pc];
}

// CH > 0: the (sequence, head)'s out-of-window keys fit CH chunks and are held in registers;
// CH == 0: any length, keys are re-read from memory in every pass.
template <int CH, bool APPEND>
__global__ void __launch_bounds__(kSelThreads)
retain_kernel(const RetainArgs a) {
  __shared__ int scan_scratch[kSelWaves + 1];
  __shared__ __align__(16) int hist[256 * kSub];
  __shared__ int sel_digit, sel_need, sel_total, sel_exact;

  const int b = blockIdx.x / a.Hkv, h = blockIdx.x - b * a.Hkv;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int64_t lo = a.cu[b];
  const int n = (int)(a.cu[b + 1] - lo);
  const int64_t head = (int64_t)b * a.Hkv + h;
  const Elements<APPEND> el(a, b, h, head, lo, n);
  const int pieces = a.row_bytes / 16;

  if ((int)blockIdx.y >= a.slices) {
    // ---- ring rows: slot -> the position it holds after n tokens ----
    const int rows_per_pass = kSelThreads / pieces;
    const int sub = tid / pieces, pc = tid - sub * pieces;
    const int from = ((int)blockIdx.y - a.slices) * kRingRows, row_end = min(from + kRingRows, a.window);
    for (int slot = from + sub; slot < row_end; slot += rows_per_pass) {
      int p;
      if (n >= a.window) {
        const int first = n - a.window;   // oldest position in the window
        p = first + (slot - first % a.window + a.window) % a.window;
      } else {
        p = slot < n ? slot : -1;
      }
      if (p < 0) continue;
      if constexpr (APPEND) {
        // fewer than `window` tokens so far (then nothing is kept and the whole prefix is pad): unused slots
        if (p < el.prefix) {
          if (pc == 0) a.win_score[head * a.window + slot] = __uint_as_float(0x7FC00000u);
          const u32x4 zero4 = {0u, 0u, 0u, 0u};
          reinterpret_cast<u32x4*>(a.k_win + (head * a.window + slot) * a.row_bytes)[pc] = zero4;
          reinterpret_cast<u32x4*>(a.v_win + (head * a.window + slot) * a.row_bytes)[pc] = zero4;
          continue;
        }
      }
      if (pc == 0) a.win_score[head * a.window + slot] = el.logit(p);
      copy_piece(a, (lo + p) * a.tok_bytes + h * a.head_bytes, a.k_win + (head * a.window + slot) * a.row_bytes,
                 a.v_win + (head * a.window + slot) * a.row_bytes, pc);
    }
    return;
  }

  const int n_out = n > a.window ? n - a.window : 0;
  const int slice = (int)blockIdx.y;
  if (h == 0 && tid == 0 && slice == 0) {
    const int seen = el.seen(n);
    a.n_seen[b] = seen;
    a.n_scored[b] = seen > a.rho ? seen - a.rho : 0;
  }
  if (a.budget == 0 || n_out == 0) {
    if (tid == 0 && slice == 0) a.ret_count[head] = 0;
    return;
  }

  // ---- keys: 0 = not a candidate (every candidate's order key is positive) ----
  auto fetch = [&](int j) -> uint32_t {
    if (j >= n_out) return 0u;
    if (!el.exists(j)) return 0u;
    if (el.is_sink(a, j)) return order_key(__uint_as_float(0x7F800000u));
    const float zj = el.logit(j);
    return zj > a.tau ? order_key(zj + 0.0f) : 0u;
  };
  constexpr int kHeld = CH > 0 ? CH : 1;
  uint32_t held[kHeld][kItems];
  if constexpr (CH > 0) {
    // a thread's four logits of a chunk are consecutive: one 16-byte load where the head's row allows it
    static_assert(kItems == 4, "one float4 per thread and chunk");
    const float* z = a.logits + (int64_t)h * a.total + lo;
    const bool quads = !APPEND && (reinterpret_cast<uintptr_t>(z) & 15u) == 0;
    auto key_of = [&](float zj, int j) -> uint32_t {
      return ((j < a.sink) || (zj > a.tau)) ? order_key(select_key(zj, j, a.sink)) : 0u;
    };
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int j0 = c * kChunk + tid * kItems;
      if (quads && j0 + kItems <= n_out) {
        const float4 z4 = *reinterpret_cast<const float4*>(z + j0);
        held[c][0] = key_of(z4.x, j0); held[c][1] = key_of(z4.y, j0 + 1);
        held[c][2] = key_of(z4.z, j0 + 2); held[c][3] = key_of(z4.w, j0 + 3);
      } else {
#pragma unroll
        for (int e = 0; e < kItems; ++e) held[c][e] = fetch(j0 + e);
      }
    }
  }
  const int n_chunks = (n_out + kChunk - 1) / kChunk;
  // A sequence longer than the caller's max_seqlen (which picked CH) does not fit the held registers: its keys are
  // re-read from memory in every pass instead (a workgroup-uniform choice), so the result stays exact.
  const bool use_held = CH > 0 && n_chunks <= CH;
  auto chunk_keys = [&](int c, uint32_t (&u)[kItems]) {
    if (use_held) {
#pragma unroll
      for (int cc = 0; cc < kHeld; ++cc)
        if (cc == c) {
#pragma unroll
          for (int e = 0; e < kItems; ++e) u[e] = held[cc][e];
        }
    } else {
#pragma unroll
      for (int e = 0; e < kItems; ++e) u[e] = fetch(c * kChunk + tid * kItems + e);
    }
  };

  // ---- exact budget-th largest key (only when the cap binds); the first pass also counts the candidates ----
  uint32_t thr = 0;      // keep keys strictly above thr ...
  int need_eq = 0;       // ... plus the first need_eq (by position) equal to thr
  {
    uint32_t prefix = 0;
    int need = a.budget;
    for (int pass = 0; pass < 4; ++pass) {
      const int shift = 24 - 8 * pass;
      hist[tid] = 0;
      hist[tid + kSelThreads] = 0;
      __syncthreads();
#pragma unroll 1
      for (int c = 0; c < n_chunks; ++c) {
        uint32_t u[kItems];
        chunk_keys(c, u);
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
          const bool match = u[e] != 0u && ((pass == 0) || ((u[e] >> (shift + 8)) == prefix));
          if (match) atomicAdd(&hist[((u[e] >> shift) & 255u) * kSub + (lane & (kSub - 1))], 1);
        }
      }
      __syncthreads();
      if (tid < kWave) {
        // lane l owns digits 255-4l .. 252-4l, so lane order is descending digit order
        int cnt[4], mine = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = 255 - 4 * lane - i;
          const int4 x = *reinterpret_cast<const int4*>(&hist[d * kSub]);
          const int4 y = *reinterpret_cast<const int4*>(&hist[d * kSub + 4]);
          cnt[i] = x.x + x.y + x.z + x.w + y.x + y.y + y.z + y.w;
          mine += cnt[i];
        }
        const int inc = wave_scan_add(mine);
        int running = inc - mine;   // elements with a larger digit than this lane's first
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (running < need && need <= running + cnt[i]) {
            sel_digit = 255 - 4 * lane - i;
            sel_need = need - running;
            sel_exact = need == running + cnt[i];   // the whole bucket is kept: the lower digits decide nothing
          }
          running += cnt[i];
        }
        if (lane == kWave - 1) sel_total = inc;
      }
      __syncthreads();
      if (pass == 0 && sel_total <= a.budget) break;   // the cap does not bind: keep every candidate
      prefix = (prefix << 8) | (uint32_t)sel_digit;
      need = sel_need;
      if (pass == 3) { thr = prefix; need_eq = need; }
      else if (sel_exact && (prefix << shift) != 0u) { thr = (prefix << shift) - 1u; break; }   // keep keys >= prefix << shift
      __syncthreads();   // hist and sel_* are rewritten by the next pass
    }
  }

  // ---- ordered compaction: ascending positions ----
  const int s_lo = slice * a.slice_rows, s_rows = slice == a.slices - 1 ? INT32_MAX : a.slice_rows;
  // (one comparison per kept entry, from the slice's first one on: an instruction of every thread is 16 clocks of a SIMD here, and two
  // comparisons 0.1 to 0.3 us of calls whose heads are not shared out)
  const int64_t s_first = head * a.budget + s_lo;
  int32_t* const ret_pos = a.ret_pos + s_first;
  float* const ret_score = a.ret_score + s_first;
  int32_t* const local_pos = APPEND ? a.plan.local_pos + s_first : nullptr;
  int kept_before = 0, eq_before = 0;
#pragma unroll 1
  for (int c = 0; c < n_chunks; ++c) {
    const int j0 = c * kChunk + tid * kItems;
    uint32_t u[kItems];
    chunk_keys(c, u);
    int n_eq = 0;
#pragma unroll
    for (int e = 0; e < kItems; ++e) n_eq += (need_eq > 0 && u[e] == thr);
    int eq_rank = 0, eq_total = 0;
    if (need_eq > 0) eq_rank = eq_before + block_exclusive_scan(n_eq, scan_scratch, eq_total);
    bool keep[kItems];
    int n_keep = 0;
#pragma unroll
    for (int e = 0; e < kItems; ++e) {
      bool kp = false;
      if (u[e] > thr) kp = true;
      else if (need_eq > 0 && u[e] == thr) { kp = eq_rank < need_eq; ++eq_rank; }
      keep[e] = kp;
      n_keep += kp;
    }
    int keep_total;
    int off = kept_before - s_lo + block_exclusive_scan(n_keep, scan_scratch, keep_total);      // from the slice's first entry
#pragma unroll
    for (int e = 0; e < kItems; ++e) {
      if (keep[e]) {
        if ((unsigned)off < (unsigned)s_rows) {
          ret_pos[off] = el.position(a, head, j0 + e);
          if constexpr (APPEND) local_pos[off] = j0 + e - el.prefix;
          ret_score[off] = key_of_order_key(u[e]);
        }
        ++off;
      }
    }
    kept_before += keep_total;
    eq_before += eq_total;
  }
  if (tid == 0 && slice == 0) a.ret_count[head] = kept_before;

  // ---- gather the slice's kept rows (positions written above by this workgroup) ----
  __threadfence_block();
  __syncthreads();
  // four pieces per thread in flight: positions first, then all the row loads, then the stores
  constexpr int kGather = 4;
  const int n_pieces = min(kept_before - s_lo, s_rows) * pieces;
  for (int i0 = tid; i0 < n_pieces; i0 += kGather * kSelThreads) {
    int r[kGather], pc[kGather], p[kGather];
#pragma unroll
    for (int u = 0; u < kGather; ++u) {
      const int i = i0 + u * kSelThreads;
      const int ic = i < n_pieces ? i : i0;          // past the end: this thread's first piece once more, not stored
      const int row = ic / pieces;
      pc[u] = ic - row * pieces;
      r[u] = s_lo + row;
      if constexpr (APPEND) p[u] = a.plan.local_pos[head * a.budget + r[u]] + el.prefix;
      else p[u] = a.ret_pos[head * a.budget + r[u]];
    }
    u32x4 xk[kGather], xv[kGather];
#pragma unroll
    for (int u = 0; u < kGather; ++u) {
      const int64_t src = (lo + p[u]) * a.tok_bytes + h * a.head_bytes;
      xk[u] = reinterpret_cast<const u32x4*>(a.k + src)[pc[u]];
      xv[u] = reinterpret_cast<const u32x4*>(a.v + src)[pc[u]];
    }
#pragma unroll
    for (int u = 0; u < kGather; ++u) {
      if (i0 + u * kSelThreads < n_pieces) {
        reinterpret_cast<u32x4*>(a.k_ret + (head * a.budget + r[u]) * a.row_bytes)[pc[u]] = xk[u];
        reinterpret_cast<u32x4*>(a.v_ret + (head * a.budget + r[u]) * a.row_bytes)[pc[u]] = xv[u];
      }
    }
  }
}

}  // namespace

namespace {

RetainArgs retain_args(const ltea_cfg& cfg, const float* logits, int64_t total, const int32_t* cu, const void* k, const void* v,
                       int64_t stride_tok, int64_t stride_head, int rho, const ltea_cache& c) {
  const int64_t esz = cfg.dtype == LTEA_F32 ? 4 : 2;
  RetainArgs a;
  a.logits = logits; a.total = total; a.cu = cu; a.Hkv = cfg.Hkv; a.window = cfg.window;
  a.budget = cfg.budget; a.sink = cfg.sink; a.tau = cfg.tau_logit; a.rho = rho;
  a.k = static_cast<const char*>(k); a.v = static_cast<const char*>(v);
  a.tok_bytes = stride_tok * esz; a.head_bytes = stride_head * esz; a.row_bytes = (int)(cfg.D * esz);
  a.k_win = static_cast<char*>(c.k_win); a.v_win = static_cast<char*>(c.v_win); a.win_score = c.win_score;
  a.k_ret = static_cast<char*>(c.k_ret); a.v_ret = static_cast<char*>(c.v_ret);
  a.ret_score = c.ret_score; a.ret_pos = c.ret_pos; a.ret_count = c.ret_count; a.n_seen = c.n_seen;
  a.n_scored = c.n_scored;
  a.plan = AppendPlan{};
  return a;
}

template <bool APPEND>
hipError_t run(RetainArgs a, int n_seqs, int64_t longest, hipStream_t stream) {
  const int64_t n_out_max = longest > a.window ? longest - a.window : 0;
  // Slices of at least 64 rows while they and the heads take no more than half of the CUs, which the ring's rows need too.  One CU
  // moves about 40 KB per us.  us per call with one workgroup per head, with four and with eight, a workgroup on every CU, for which
  // the ring waits: 32768 tokens, 32 heads, 1024 kept entries of D = 128 each 45.6, 35.3, 42.7; 4 x 4096 tokens, 8 heads, 512
  // entries of D = 64 12.5, 11.7, 13.1.
  const int64_t heads = (int64_t)n_seqs * a.Hkv, by_cus = heads > 0 ? 128 / heads : 1;
  const int64_t most = ((n_out_max < a.budget ? n_out_max : a.budget) + 63) / 64;
  const int64_t slices = by_cus < most ? by_cus : most;
  a.slices = (int)(slices < 1 ? 1 : slices > 8 ? 8 : slices);
  // divided here: the division in the kernel, in front of the compaction, was 0.13 us of the smallest calls (18.4 and 26.6 us)
  a.slice_rows = (int)(((n_out_max < a.budget ? n_out_max : a.budget) + a.slices - 1) / a.slices);
  const dim3 grid((unsigned)n_seqs * (unsigned)a.Hkv, (unsigned)(a.slices + (a.window + kRingRows - 1) / kRingRows));
  auto go = [&](auto ch) {
    hipLaunchKernelGGL((retain_kernel<decltype(ch)::value, APPEND>), grid, dim3(kSelThreads), 0, stream, a);
  };
  if (n_out_max <= 1 * kChunk) go(std::integral_constant<int, 1>{});
  else if (n_out_max <= 2 * kChunk) go(std::integral_constant<int, 2>{});
  else if (n_out_max <= 4 * kChunk) go(std::integral_constant<int, 4>{});
  else if (n_out_max <= 8 * kChunk) go(std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, 0>{});
  return hipGetLastError();
}

}  // namespace

hipError_t launch_retain(const ltea_cfg& cfg, const float* logits, const void* k, const void* v, int64_t stride_tok,
                         int64_t stride_head, const SeqView& sv, int rho, const ltea_cache& c, hipStream_t stream) {
  if (sv.n_seqs == 0) return hipSuccess;
  const RetainArgs a = retain_args(cfg, logits, sv.total_tokens, sv.cu_seqlens, k, v, stride_tok, stride_head, rho, c);
  return run<false>(a, sv.n_seqs, sv.max_seqlen, stream);
}

hipError_t launch_retain_append(const ltea_cfg& cfg, const AppendBuffers& buf, int n_seqs, int rho, const ltea_cache& c,
                                hipStream_t stream) {
  RetainArgs a = retain_args(cfg, buf.score_logits, buf.total_score, buf.plan.cu_ext, buf.ext_k, buf.ext_v,
                             (int64_t)cfg.Hkv * cfg.D, cfg.D, rho, c);
  a.plan = buf.plan;
  return run<true>(a, n_seqs, buf.max_ext_len, stream);
}

}  // namespace ltea
