// One decode step of the SWA+LTE cache (paper Section 3.1.3: cache replacement, decode attention and
// the deferred scoring of Section 3.1.1 item 2).
//
// One launch per step on the caller's stream.  Its first workgroups score: they finalise the logit of position t-rho of
// every (sequence, KV head) from the 2*rho newest ring rows plus the incoming token (none of them is written by the step).
//   - single-layer bf16 CNNs: one workgroup per (KV head, 16 sequences), the conv over the batch as a small GEMM;
//   - stacks of two or three k = 3 layers with one dilation (the paper's): one workgroup per (KV head, 8 sequences);
//   - others (fp32, unusual stacks): one workgroup per (sequence, head).
// Then one streaming workgroup of 4 or 8 waves per (sequence, KV head), or several (shares of its rows) where there are few
// heads.  It
//   - requests its first rows and, under their flight, decides where the token leaving the window goes (one pass over
//     `budget` keys of the old state);
//   - streams the rows the query must see AFTER this step's cache update, without that update having happened: the row of
//     ring slot t % window is taken from the incoming k_t, v_t, and the compact slot that receives the evicted token from
//     the old ring row;
//   - merges its waves, writes the output rows of the group's query heads and applies the update: evicted row to the compact
//     segment, k_t, v_t to the ring.
// The last workgroup of a sequence advances n_seen / n_scored.
//
// Who is last is counted in the upper bits of ret_count, which the cache contract initialises and which are zero again
// when the step ends: bits 24..31 of a sequence's first word count its workgroups (heads, scoring) and, where a head has
// several shares, bits 16..23 of its word count those; the last share then merges all of them and applies the update.  What
// one workgroup hands to another (share records, the eviction decision) is stored and loaded with relaxed agent-scope
// atomics, which go past the XCD's own L2; a workgroup waits for its stores before it counts itself, and nobody waits for
// anybody: no fences, which write back a whole L2 each, and no spinning.
//
// Measured on the paper's layer (32 query heads on 8, D = 64, 1280 rows), us per eager step of one sequence, per eager step of
// 32 of a rotary model and per lazy step of 32: separate streaming, scoring and finishing launches 28.6, 48.3 and 29.8; one
// streaming launch with the finishing as a launch of its own and nothing counted 14.7, 25.8 and 22.4, with the finishing inside
// 12.3, 23.3 and 20.1, after changes of the merge 12.2, 22.7 and 19.3; with everything that needs no address from memory
// requested before the first wait (scalar words, eviction keys, the scoring's rows and weights, at D = 64 the first block of
// rows of either kind, the rows that move) and the descriptors uniform to the compiler 9.6, 19.8 and 17.4. Handing shares over
// costs about 5 us at the end (stores, count, records, each a trip past the L2), which is why a head is one workgroup when the
// heads alone fill the chip and shared out when its rows are long. Caches that do not fit the counting (no budget, or a budget
// of 2^16 and more, or over 127 KV heads) or whose logit is final at once (rho = 0: the scoring would write the ring slot whose
// old logit the eviction reads) run the finishing as a launch of its own, decode_finish_kernel.
//
// The lazy step (Section 3.1.3, lazy scoring) is the same launch without the scoring: logits are
// produced between steps by the batched scoring of lazy.hip, n_scored is left alone and a token that leaves the window
// unscored is flagged.
#pragma once
#include <string.h>

#include <type_traits>

#include "decode_run.h"

namespace ltea {
namespace {

constexpr int kThreads = 256;     // finishing launch
constexpr int kRowsInFlight = 4;  // rows per lane group per iteration of the VALU streaming loop
constexpr int kPerHead = 1, kDeepRole = 9;   // scoring roles besides the kernel sizes 3, 5, 7 of the single-layer one

struct CnnDev {
  int n_layers;
  int kernel[LTEA_MAX_CNN_LAYERS], c_out[LTEA_MAX_CNN_LAYERS];
  // Per-head scoring: the outputs of a layer that a logit depends on are `unit` positions apart (the greatest common divisor of
  // the dilations after it); dilation and row_step (from one such output to the next) are in rows of the layer's input.
  int unit[LTEA_MAX_CNN_LAYERS], dilation[LTEA_MAX_CNN_LAYERS], row_step[LTEA_MAX_CNN_LAYERS];
  const void* w[LTEA_MAX_CNN_LAYERS];
  const float* bias[LTEA_MAX_CNN_LAYERS];
  const void* w_out;
  const float* b_out;
};

struct StepParams {
  int B, Hq, Hkv, D, window, budget, sink, rho, nsplit;
  float tau, scale;
  // scoring workgroups in front of the streaming ones; per-head scoring: rows of the receptive field are `unit` positions
  // apart (the greatest common divisor of the dilations), LDS rows of lds_row_floats
  int n_score_blocks, unit, lds_row_floats;
  int seq_arrivals;          // streaming and scoring workgroups that read a sequence's counters
  // scores computed before this launch over packed receptive-field windows: the window of sequence b occupies rows
  // b*(2*rho+1) .. of pre_logits[h][.], its first row is position max(0, t - 2*rho)
  const float* pre_logits;
  int64_t pre_total;
  // Lazy mode (scores come from separate batched launches between steps): nothing is scored here, n_scored is
  // left alone, and a token that leaves the window without a final logit is reported through `status`.
  int lazy;
  int32_t* status;
  int fused;                 // the finishing is part of the launch
  uint32_t count_mask;       // the bits of ret_count that are the count
  // rotary models: ring keys are rotated back for the scoring (rope.cos null: no), the incoming token's scoring key is kf_new
  // when given, else k_new rotated back at position t
  RopeDev rope;
  const void* kf_new;
};

// What the workgroups of a head hand to each other or to the finishing launch.
struct Handover { float* partial; float* logit; int32_t* t; int32_t* dst; };

template <typename V> __device__ __forceinline__ void store_shared(V* p, V v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V> __device__ __forceinline__ V load_shared(const V* p) {
  return __hip_atomic_load(const_cast<V*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_for_own_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// One workgroup is done with n_seen / n_scored of the sequence (all its waves have read them): the last one advances them.  In two
// parts, the count and what follows from it, so that the count's trip passes beside other work.
__device__ __forceinline__ unsigned count_arrival(const CacheDev& C, const StepParams& P, int b) {
  unsigned* word = reinterpret_cast<unsigned*>(C.ret_count + (int64_t)b * P.Hkv);
  return P.seq_arrivals > 1 ? atomicAdd(word, 1u << 24) >> 24 : 0u;
}
__device__ __forceinline__ void advance_if_last(const CacheDev& C, const StepParams& P, int b, int t, unsigned before) {
  if (before + 1 != (unsigned)P.seq_arrivals) return;
  if (P.seq_arrivals > 1) atomicSub(reinterpret_cast<unsigned*>(C.ret_count + (int64_t)b * P.Hkv), (unsigned)P.seq_arrivals << 24);
  C.n_seen[b] = t + 1;
  if (!P.lazy) C.n_scored[b] = t + 1 > P.rho ? t + 1 - P.rho : 0;
}

// Whether a key in the receptive field of position t - rho that is rotated back lies past the rotary tables: the newest one does.
__device__ __forceinline__ bool past_tables(const StepParams& P, int t) {
  if (P.rope.cos == nullptr) return false;
  return P.kf_new == nullptr ? t >= P.rope.n_pos : P.rho > 0 && t - 1 >= P.rope.n_pos;
}

// exp used by the softmax: library expf for fp32 storage (1e-5 tolerance), hardware exp2 path for bf16.
template <typename T> __device__ __forceinline__ float soft_exp(float x);
template <> __device__ __forceinline__ float soft_exp<float>(float x) { return expf(x); }
template <> __device__ __forceinline__ float soft_exp<bf16_t>(float x) { return __expf(x); }

template <typename T> struct Piece;  // 16 bytes of a row as fp32 values
template <> struct Piece<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void unpack(const u32x4& r, float (&x)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(r[i]);
  }
  static __device__ __forceinline__ void load(const float* p, float (&x)[4]) {
    const f32x4 r = *reinterpret_cast<const f32x4*>(p);
    x[0] = r[0]; x[1] = r[1]; x[2] = r[2]; x[3] = r[3];
  }
};
template <> struct Piece<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void unpack(const u32x4& r, float (&x)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(r[i] << 16);
      x[2 * i + 1] = __uint_as_float(r[i] & 0xFFFF0000u);
    }
  }
  static __device__ __forceinline__ void load(const bf16_t* p, float (&x)[8]) {
    const u32x4 r = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(r[i] << 16);
      x[2 * i + 1] = __uint_as_float(r[i] & 0xFFFF0000u);
    }
  }
};

// A word that no workgroup changes before all that read it are done with it, through the scalar cache: such a load is not one of
// the vector loads, which return in order, so waiting for it does not wait for rows requested earlier.  read_here: its memory
// changes later, so the value is taken here, once.
template <typename V> __device__ __forceinline__ V load_uniform(const V* p) {
  static_assert(sizeof(V) == 4, "one word");
  return __builtin_bit_cast(V, *reinterpret_cast<const __attribute__((address_space(4))) uint32_t*>(reinterpret_cast<uintptr_t>(p)));
}
template <typename V> __device__ __forceinline__ void read_here(V& x) { asm volatile("" : "+s"(x)); }

// Smallest value over the wave, in all lanes, on the cross-lane paths of the vector ALU: six steps of a few instructions where
// LDS permutes would cost about 100 clocks each.
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long x) {
  auto step = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
    constexpr int kCtrl = decltype(ctrl)::value, kRows = decltype(rows)::value;
    const uint32_t lo = __builtin_amdgcn_update_dpp(~0u, (uint32_t)x, kCtrl, kRows, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(~0u, (uint32_t)(x >> 32), kCtrl, kRows, 0xf, false);
    const unsigned long long o = (unsigned long long)hi << 32 | lo;
    x = o < x ? o : x;
  };
  step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});   // row_shr:1
  step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});   // row_shr:2
  step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});   // row_shr:4
  step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});   // row_shr:8
  step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast:15 into rows 1 and 3
  step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});   // row_bcast:31 into rows 2 and 3
  return (unsigned long long)__builtin_amdgcn_readlane((uint32_t)(x >> 32), kWave - 1) << 32 |
         (uint32_t)__builtin_amdgcn_readlane((uint32_t)x, kWave - 1);
}

// A thread's first entries of a head's compact segment, requested before it is known whether they are needed.
constexpr int kHeldKeys = 2;
struct HeldKeys { float score[kHeldKeys]; int pos[kHeldKeys]; };
template <int NT>
__device__ __forceinline__ HeldKeys load_held_keys(int budget, const float* __restrict__ ret_score, const int32_t* __restrict__ ret_pos) {
  HeldKeys H;
#pragma unroll
  for (int i = 0; i < kHeldKeys; ++i) {
    const int r = (int)threadIdx.x + NT * i, rc = r < budget ? r : budget - 1;
    H.score[i] = ret_score[rc];
    H.pos[i] = ret_pos[rc];
  }
  return H;
}

// Where does the token leaving the window go?  Returns the compact slot that receives it (== cnt for an
// append), or -1 if it is dropped.  A pure function of the state before the step, evaluated identically by
// every workgroup that needs it.  All threads of the block must call it, once per launch; `red` is LDS scratch.
template <int NT>
__device__ __forceinline__ int eviction_target(int t, int window, int budget, int sink, float tau, int cnt, float z_e,
                                               const HeldKeys& held, const float* __restrict__ ret_score,
                                               const int32_t* __restrict__ ret_pos, unsigned long long* red, int* slot_out) {
  constexpr int kWaves = NT / kWave;
  const int e_pos = t - window;
  if (e_pos < 0 || budget <= 0) return -1;
  if (!((e_pos < sink) || (z_e > tau))) return -1;
  if (cnt < budget) return cnt;
  // victim: lowest key, among equal keys the latest position
  const int tid = threadIdx.x;
  unsigned long long best = ~0ull;
  auto look = [&](float key, int pos) {
    const unsigned long long c = ((unsigned long long)order_key(key + 0.0f) << 32) | (0xFFFFFFFFu - (uint32_t)pos);
    best = c < best ? c : best;
  };
#pragma unroll
  for (int i = 0; i < kHeldKeys; ++i)
    if (tid + NT * i < budget) look(held.score[i], held.pos[i]);
  for (int r = tid + NT * kHeldKeys; r < budget; r += NT) look(ret_score[r], ret_pos[r]);
  best = wave_min_u64(best);
  if ((tid & (kWave - 1)) == 0) red[tid / kWave] = best;
  if (tid == 0) *slot_out = -1;
  __syncthreads();
  best = red[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) best = red[w] < best ? red[w] : best;
  const int worst_pos = (int)(0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull));
  // positions are unique; of a caller's duplicates the last slot
#pragma unroll
  for (int i = kHeldKeys - 1; i >= 0; --i)
    if (tid + NT * i < budget && held.pos[i] == worst_pos) atomicMax(slot_out, tid + NT * i);
  for (int r = tid + NT * kHeldKeys; r < budget; r += NT)
    if (ret_pos[r] == worst_pos) atomicMax(slot_out, r);
  __syncthreads();
  const int victim = *slot_out;
  return order_key(select_key(z_e, e_pos, sink)) > (uint32_t)(best >> 32) ? victim : -1;
}

// The finalised logit of position t - rho: straight into the ring when the finishing is part of this launch (its slot is
// not the one whose old logit the eviction reads: rho is at least 1 then), else parked for the finishing launch.
__device__ __forceinline__ void put_logit(const CacheDev& C, const StepParams& P, int64_t head, int t, float z, float* ws_logit) {
  if (P.fused) C.win_score[head * P.window + (t - P.rho) % P.window] = z;
  else ws_logit[head] = z;
}

constexpr int kRoleThreads = 256, kRoleWaves = 4;   // the batched scoring roles; a launch's further waves leave at once

// ---- scoring, one (sequence, KV head) per workgroup: any CNN, fp32 arithmetic ------------------------------------
// One layer over the rows in LDS: KS taps, `dil` rows apart, RR output rows, `step` rows apart, per pass (DENSE: both 1,
// neighbouring outputs share their rows).  A thread owns one (output channel, every lpc-th run of 8 input channels); a run's weights are 8*KS
// consecutive elements of the channel's row ([channel][tap] order), the runs of a channel meet in a shuffle reduction.
template <typename T, int KS, int RR, bool DENSE, int NT>
__device__ __forceinline__ void conv_rows(const T* __restrict__ W, const float* __restrict__ bias, int cin, int cout, int dil,
                                          int step, const float* cur, float* nxt, int row_f, int out_rows, int first_pos,
                                          int unit) {
  const int tid = threadIdx.x, n_runs = cin / 8;
  int lpc = n_runs < kWave ? n_runs : kWave;                    // lanes per channel: a power of two
  lpc = 1 << (31 - __clz(lpc));
  while (lpc > 1 && lpc * cout > NT) lpc >>= 1;
  const int sub = tid & (lpc - 1), c_step = NT / lpc;
  for (int c0 = 0; c0 < cout; c0 += c_step) {
    const int c = c0 + tid / lpc, cc = c < cout ? c : 0;
    for (int r0 = 0; r0 < out_rows; r0 += RR) {
      float acc[RR];
#pragma unroll
      for (int r = 0; r < RR; ++r) acc[r] = 0.f;
      for (int run = sub; run < n_runs; run += lpc) {
        const T* wp = W + ((int64_t)cc * cin + 8 * run) * KS;
        constexpr int EPP = Piece<T>::N, NP = 8 * KS / EPP;
        u32x4 raw[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) raw[i] = reinterpret_cast<const u32x4*>(wp)[i];
        auto weight = [&](int f) {       // element f of the run
          if constexpr (EPP == 4) return __uint_as_float(raw[f / 4][f % 4]);
          else return __uint_as_float(f & 1 ? raw[f / 8][f % 8 / 2] & 0xFFFF0000u : raw[f / 8][f % 8 / 2] << 16);
        };
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          auto x_of = [&](int row) { return *reinterpret_cast<const f32x4*>(cur + row * row_f + 8 * run + 4 * half); };
          if constexpr (DENSE) {
#pragma unroll
            for (int i = 0; i < RR + KS - 1; ++i) {             // input row r0 + i is tap i - r of output r0 + r
              const f32x4 x = x_of(r0 + i < out_rows + KS - 1 ? r0 + i : r0);   // past the last: not used by a stored output
#pragma unroll
              for (int r = 0; r < RR; ++r) {
                const int tap = i - r;
                if (tap < 0 || tap >= KS) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[r] = fmaf(x[e], weight((4 * half + e) * KS + tap), acc[r]);
              }
            }
          } else {
#pragma unroll
            for (int r = 0; r < RR; ++r)
#pragma unroll
              for (int tap = 0; tap < KS; ++tap) {
                const f32x4 x = x_of((r0 + r < out_rows ? r0 + r : r0) * step + tap * dil);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[r] = fmaf(x[e], weight((4 * half + e) * KS + tap), acc[r]);
              }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < RR; ++r)
        for (int off = lpc / 2; off > 0; off >>= 1) acc[r] += __shfl_xor(acc[r], off, kWave);
      if (sub == 0 && c < cout) {
#pragma unroll
        for (int r = 0; r < RR; ++r)
          if (r0 + r < out_rows)     // activations at positions before the sequence start are zero padding, not Swish(bias)
            nxt[(r0 + r) * row_f + c] = first_pos + (r0 + r) * unit >= 0 ? silu_f32(acc[r] + bias[c]) : 0.f;
      }
    }
  }
}

// The same for any kernel size and channel count: a thread owns one (output channel, every lpc-th piece of EPP consecutive
// elements of its row), several pieces in flight.
template <typename T, int EPP, int NT>
__device__ __forceinline__ void conv_rows_any(const T* __restrict__ W, const float* __restrict__ bias, int cin, int cout, int ks,
                                              int dil, int step, const float* cur, float* nxt, int row_f, int out_rows, int first_pos,
                                              int unit) {
  constexpr int kAhead = EPP == 1 ? 8 : 4, RR = 4;
  const int tid = threadIdx.x, n_pieces = cin * ks / EPP;
  int lpc = n_pieces < kWave ? n_pieces : kWave;
  lpc = 1 << (31 - __clz(lpc));
  while (lpc > 1 && lpc * cout > NT) lpc >>= 1;
  const int sub = tid & (lpc - 1), c_step = NT / lpc;
  const int ch_step = lpc * EPP / ks, tap_step = lpc * EPP % ks;
  for (int c0 = 0; c0 < cout; c0 += c_step) {
    const int c = c0 + tid / lpc;
    const T* wr = W + (int64_t)(c < cout ? c : 0) * cin * ks;
    for (int r0 = 0; r0 < out_rows; r0 += RR) {
      float acc[RR];
#pragma unroll
      for (int r = 0; r < RR; ++r) acc[r] = 0.f;
      int m0 = sub * EPP / ks, tap0 = sub * EPP % ks;       // input channel and tap of a piece's first element
      for (int p0 = sub; p0 < n_pieces; p0 += kAhead * lpc) {
        float w[kAhead][EPP];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          const int p = p0 + u * lpc < n_pieces ? p0 + u * lpc : p0;
          if constexpr (EPP == 1) w[u][0] = to_f32(wr[p]);
          else Piece<T>::load(wr + (int64_t)p * EPP, w[u]);
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          if (p0 + u * lpc < n_pieces) {
            int m = m0, tap = tap0;
#pragma unroll
            for (int e = 0; e < EPP; ++e) {
              const float* x = cur + (r0 * step + tap * dil) * row_f + m;
#pragma unroll
              for (int r = 0; r < RR; ++r)
                if (r0 + r < out_rows) acc[r] = fmaf(x[r * step * row_f], w[u][e], acc[r]);
              if (++tap == ks) { tap = 0; ++m; }
            }
          }
          m0 += ch_step;
          tap0 += tap_step;
          if (tap0 >= ks) { tap0 -= ks; ++m0; }
        }
      }
#pragma unroll
      for (int r = 0; r < RR; ++r)
        for (int off = lpc / 2; off > 0; off >>= 1) acc[r] += __shfl_xor(acc[r], off, kWave);
      if (sub == 0 && c < cout) {
#pragma unroll
        for (int r = 0; r < RR; ++r)
          if (r0 + r < out_rows) nxt[(r0 + r) * row_f + c] = first_pos + (r0 + r) * unit >= 0 ? silu_f32(acc[r] + bias[c]) : 0.f;
      }
    }
  }
}

// A single layer: with its inputs staged in the order of a weight row, [channel][tap], an output is one dot product.  A thread
// owns one (output channel, every lpc-th piece of EPP consecutive elements), eight pieces in flight.  k = 9, 128 -> 32 channels,
// one sequence of the paper's other sizes: a step took 102 us with one thread per output and a load per multiply-add, 11.3 in
// this form.
template <typename T, int EPP, int NT>
__device__ __forceinline__ void conv_flat(const T* __restrict__ W, const float* __restrict__ bias, int n_el, int cout,
                                          const float* x, float* out) {
  constexpr int kAhead = 8;
  const int tid = threadIdx.x, n_pieces = n_el / EPP;
  int lpc = n_pieces < kWave ? n_pieces : kWave;
  lpc = 1 << (31 - __clz(lpc));
  while (lpc > 1 && lpc * cout > NT) lpc >>= 1;
  const int sub = tid & (lpc - 1);
  for (int c0 = 0; c0 < cout; c0 += NT / lpc) {
    const int c = c0 + tid / lpc;
    const T* wr = W + (int64_t)(c < cout ? c : 0) * n_el;
    float acc[2] = {0.f, 0.f};
    for (int p0 = sub; p0 < n_pieces; p0 += kAhead * lpc) {
      float w[kAhead][EPP];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int p = p0 + u * lpc < n_pieces ? p0 + u * lpc : p0;
        if constexpr (EPP == 1) w[u][0] = to_f32(wr[p]);
        else Piece<T>::load(wr + (int64_t)p * EPP, w[u]);
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (p0 + u * lpc >= n_pieces) break;
        const float* xp = x + (p0 + u * lpc) * EPP;
        if constexpr (EPP == 1) {
          acc[u & 1] = fmaf(xp[0], w[u][0], acc[u & 1]);
        } else {
#pragma unroll
          for (int e = 0; e < EPP; e += 4) {
            const f32x4 y = *reinterpret_cast<const f32x4*>(xp + e);
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[u & 1] = fmaf(y[i], w[u][e + i], acc[u & 1]);
          }
        }
      }
    }
    float a = acc[0] + acc[1];
    for (int off = lpc / 2; off > 0; off >>= 1) a += __shfl_xor(a, off, kWave);
    if (sub == 0 && c < cout) out[c] = silu_f32(a + bias[c]);
  }
}

// Logit of position t - rho of one (sequence, KV head): any CNN.  The inputs are rows of positions `unit` apart around t - rho;
// `lds` holds two generations of 2*rho/unit + 1 rows.  Of every layer only the rows that the layers after it read are formed (3 + 3
// + 3 taps with dilations 1, 2, 4: 7, 3 and 1 of them instead of 13, 9 and 1; a step of 128 sequences of 8 KV heads 176 -> 74 us,
// of one sequence 47 -> 16, taps more than a row apart one thread per output before).
// Bound: latency, a trip to memory per layer; from some 2000 (sequence, head) pairs on the weights' trips from L2.
template <typename T, int NT>
__device__ __forceinline__ void score_token(const CnnDev& cnn, const StepParams& P, const CacheDev& C, const T* __restrict__ k_new,
                                            const T* __restrict__ v_new, int64_t head, int h, int t, float* lds, float* ws_logit) {
  const int tid = threadIdx.x;
  const int rho = P.rho, D = P.D, window = P.window, row_f = P.lds_row_floats, unit = P.unit;
  const int rows0 = 2 * rho / unit + 1;
  float* cur = lds;
  float* nxt = lds + (size_t)rows0 * row_f;
  // layer-0 features (keys then values), one 16-byte piece per thread per pass
  constexpr int EPP = Piece<T>::N;
  const int ppr = 2 * D / EPP;
  for (int idx = tid; idx < rows0 * ppr; idx += NT) {
    const int r = idx / ppr, m = (idx - r * ppr) * EPP;
    const int p = t - 2 * rho + r * unit;
    u32x4 raw = {0u, 0u, 0u, 0u};
    if (p >= 0) {
      const bool is_v = m >= D;
      const int mm = is_v ? m - D : m;
      const T* row = p == t ? (is_v ? v_new : k_new) + head * D
                            : static_cast<const T*>(is_v ? C.v_win : C.k_win) + (head * window + p % window) * D;
      const bool ready = p == t && P.kf_new != nullptr;         // the key as the CNN wants it
      if (!is_v && ready) row = static_cast<const T*>(P.kf_new) + head * D;
      raw = *reinterpret_cast<const u32x4*>(row + mm);
      if (!is_v && !ready && P.rope.cos != nullptr && p < P.rope.n_pos) raw = unrotate_piece<T>(P.rope, p, mm, raw, row);
    }
    float x[EPP];
    Piece<T>::unpack(raw, x);
    if (cnn.n_layers == 1) {
#pragma unroll
      for (int i = 0; i < EPP; ++i) cur[(m + i) * rows0 + r] = x[i];      // the order of a weight row
    } else {
#pragma unroll
      for (int i = 0; i < EPP; i += 4) *reinterpret_cast<f32x4*>(cur + r * row_f + m + i) = f32x4{x[i], x[i + 1], x[i + 2], x[i + 3]};
    }
  }
  __syncthreads();
  int rows = rows0, cin = 2 * D;
  for (int l = 0; l < cnn.n_layers; ++l) {
    const int ks = cnn.kernel[l], dil = cnn.dilation[l], step = cnn.row_step[l], cout = cnn.c_out[l], apart = cnn.unit[l];
    const int out_rows = (rows - 1 - dil * (ks - 1)) / step + 1;
    const int first_pos = t - rho - (out_rows - 1) / 2 * apart;
    const T* W = static_cast<const T*>(cnn.w[l]) + (int64_t)h * cout * cin * ks;
    const float* bias = cnn.bias[l] + h * cout;
    // whole runs, 16-byte aligned
    const bool aligned = (reinterpret_cast<uintptr_t>(W) & 15u) == 0, runs = cin % 8 == 0 && aligned;
    const bool dense = dil == 1 && step == 1;
    if (cnn.n_layers == 1) {
      if (aligned) conv_flat<T, EPP, NT>(W, bias, cin * ks, cout, cur, nxt);       // 2 D channels: whole pieces
      else conv_flat<T, 1, NT>(W, bias, cin * ks, cout, cur, nxt);
    } else if (runs && ks == 1) {
      conv_rows<T, 1, 1, false, NT>(W, bias, cin, cout, dil, step, cur, nxt, row_f, out_rows, first_pos, apart);
    } else if (runs && ks == 3 && dense && out_rows <= 5) {
      conv_rows<T, 3, 5, true, NT>(W, bias, cin, cout, dil, step, cur, nxt, row_f, out_rows, first_pos, apart);
    } else if (runs && ks == 3) {
      conv_rows<T, 3, 4, false, NT>(W, bias, cin, cout, dil, step, cur, nxt, row_f, out_rows, first_pos, apart);
    } else if (runs && ks == 5) {
      conv_rows<T, 5, 1, false, NT>(W, bias, cin, cout, dil, step, cur, nxt, row_f, out_rows, first_pos, apart);
    } else if (runs && ks == 7) {
      conv_rows<T, 7, 1, false, NT>(W, bias, cin, cout, dil, step, cur, nxt, row_f, out_rows, first_pos, apart);
    } else if (aligned && cin * ks % EPP == 0) {
      conv_rows_any<T, EPP, NT>(W, bias, cin, cout, ks, dil, step, cur, nxt, row_f, out_rows, first_pos, apart);
    } else {
      conv_rows_any<T, 1, NT>(W, bias, cin, cout, ks, dil, step, cur, nxt, row_f, out_rows, first_pos, apart);
    }
    __syncthreads();
    float* tmp = cur; cur = nxt; nxt = tmp;
    rows = out_rows; cin = cout;
  }
  // cur holds one row (position t - rho) of cin channels
  if (tid < kWave) {
    float part = 0.f;
    for (int c = tid; c < cin; c += kWave)
      part = fmaf(cur[c], to_f32(static_cast<const T*>(cnn.w_out)[h * cin + c]), part);
    part = wave_sum(part);  // fixed order: deterministic
    if (tid == 0) put_logit(C, P, head, t, part + cnn.b_out[h], ws_logit);
  }
}

// ---- scoring role, batched over sequences on MFMA (single conv layer, bf16, kernel size KS) ----------------------
// Workgroup = (KV head h, group of 16 sequences).  The conv over the batch is the GEMM
//   out[sequence, channel] = sum_{tap, m} x[sequence][tap][m] * W[channel][m][tap]
// on v_mfma_f32_16x16x32_bf16: one row tile of 16 sequences, 2 column tiles of 16 channels, K = (tap, m) with 32
// input channels per instruction.  The four waves split the input channels; a weight is fetched once per
// workgroup (KS contiguous 16-byte loads per lane cover all taps of its 8 channels); features come straight from the ring
// rows / the incoming token.  Partial sums of the waves meet in LDS.
// Bound: latency, and what it keeps a streaming workgroup out of its slot: the grid holds exactly as many workgroups of
// large batches as the chip has slots, so a scoring workgroup delays one of them by its own life.  16 sequences instead of
// 64 per workgroup: four times as many, a quarter of the life.
// Lane roles: A row / B column = lane % 16, K group kg = lane / 16 supplies 8 consecutive channels;
// accumulator register r of a lane is (row 4*kg + r, column lane % 16).
// ROT: the ring's keys are rotated back (rotary models).
constexpr int kSingleSeqs = 16;
template <int D, int KS, bool ROT>
__device__ __forceinline__ void score_new_tokens_mfma(const CnnDev& cnn, const StepParams& P, const CacheDev& C,
                                                      const bf16_t* __restrict__ k_new, const bf16_t* __restrict__ v_new,
                                                      int h, int b0, float* red /* 2048 floats of LDS */, float* __restrict__ ws_logit) {
  constexpr int C2 = 2 * D;
  constexpr int MCW = C2 / 32 / kRoleWaves;  // 32-channel chunks per wave
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  const int row = lane & 15, kg = lane >> 4;
  const int dil = P.unit, Cout = cnn.c_out[0];
  const int rho = P.rho, window = P.window;
  const uint16_t* W = reinterpret_cast<const uint16_t*>(cnn.w[0]) + (int64_t)h * Cout * C2 * KS;
  const int seq_l = tid / 16, chp = tid % 16;   // finishing thread: sequence seq_l, channels chp, chp+16
  const int b = b0 + row;
  const bool ok = b < P.B;
  const int64_t head = (int64_t)(ok ? b : P.B - 1) * P.Hkv + h;
  const int t = C.n_seen[ok ? b : P.B - 1];
  const int t_l = b0 + seq_l < P.B ? C.n_seen[b0 + seq_l] : 0;
  float bias0 = 0.f, bias1 = 0.f, wo0 = 0.f, wo1 = 0.f;
  if (chp < Cout) { bias0 = cnn.bias[0][h * Cout + chp]; wo0 = to_f32(static_cast<const bf16_t*>(cnn.w_out)[h * Cout + chp]); }
  if (chp + 16 < Cout) { bias1 = cnn.bias[0][h * Cout + chp + 16]; wo1 = to_f32(static_cast<const bf16_t*>(cnn.w_out)[h * Cout + chp + 16]); }
  const float b_out = cnn.b_out[h];
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll 1
  for (int mcw = 0; mcw < MCW; ++mcw) {
    const int m = 32 * (wv * MCW + mcw) + 8 * kg;   // first of this lane's 8 input channels
    // weights of channels m..m+7, all taps, for output channels row and 16+row: KS*8 contiguous elements each
    u32x4 wraw[2][KS];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int c = 16 * nb + row;
      const u32x4* wp = reinterpret_cast<const u32x4*>(W + ((int64_t)(c < Cout ? c : 0) * C2 + m) * KS);
#pragma unroll
      for (int i = 0; i < KS; ++i) wraw[nb][i] = wp[i];
    }
    u32x4 araw[KS];
#pragma unroll
    for (int tap = 0; tap < KS; ++tap) {
      const int p = t - 2 * rho + tap * dil;   // position this tap reads for the token t - rho
      const bool p_ok = p >= 0 && ok;
      const int slot_p = (p_ok ? p : 0) % window;
      const bool is_k = m < D, fresh = p == t;
      const bf16_t* rowp = fresh ? (is_k ? k_new : v_new) + head * D
                                 : static_cast<const bf16_t*>(is_k ? C.k_win : C.v_win) + (head * window + slot_p) * D;
      const int col = is_k ? m : m - D;
      bool rotate = false;
      if constexpr (ROT) {
        const bool ready = fresh && P.kf_new != nullptr;        // the key as the CNN wants it
        if (is_k && ready) rowp = static_cast<const bf16_t*>(P.kf_new) + head * D;
        rotate = is_k && p_ok && !ready;
      }
      araw[tap] = *reinterpret_cast<const u32x4*>(rowp + col);
      if constexpr (ROT) {
        if (rotate && p < P.rope.n_pos) araw[tap] = unrotate_piece<bf16_t>(P.rope, p, col, araw[tap], rowp);
      }
      if (!p_ok) araw[tap] = u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int tap = 0; tap < KS; ++tap)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        // B operand: element e is flat index e*KS + tap of the lane's weight run (zero past the last channel)
        u32x4 bop;
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          const int f0 = (2 * e2) * KS + tap, f1 = (2 * e2 + 1) * KS + tap;
          const uint32_t w0 = wraw[nb][f0 / 8][f0 % 8 / 2], w1 = wraw[nb][f1 / 8][f1 % 8 / 2];
          bop[e2] = ((f0 & 1) ? (w0 >> 16) : (w0 & 0xFFFFu)) | ((f1 & 1) ? (w1 & 0xFFFF0000u) : (w1 << 16));
        }
        if (16 * nb + row >= Cout) bop = u32x4{0u, 0u, 0u, 0u};
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, araw[tap]), __builtin_bit_cast(bf16x8, bop),
                                                          acc[nb], 0, 0, 0);
      }
  }
  // cross-wave sum, bias, Swish, output projection
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[(wv * 16 + 4 * kg + r) * 32 + 16 * nb + row] = acc[nb][r];
  __syncthreads();
  float y0 = bias0, y1 = bias1;
#pragma unroll
  for (int w = 0; w < kRoleWaves; ++w) {
    y0 += red[(w * 16 + seq_l) * 32 + chp];
    y1 += red[(w * 16 + seq_l) * 32 + 16 + chp];
  }
  float z = y0 * __frcp_rn(1.0f + __expf(-y0)) * wo0 + y1 * __frcp_rn(1.0f + __expf(-y1)) * wo1;
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) z += __shfl_xor(z, off, kWave);
  if (chp == 0 && b0 + seq_l < P.B && t_l - rho >= 0) put_logit(C, P, (int64_t)(b0 + seq_l) * P.Hkv + h, t_l, z + b_out, ws_logit);
}

// ---- scoring role for stacks of two or three k = 3 layers with one dilation (bf16, D = 64) ---------------------------
// Workgroup = (KV head, 8 sequences).  The logit of position t - rho depends on 2*L + 1 input positions, dilation apart,
// 2*L - 1 outputs of the first layer, and so on down to one: those are the rows, position * 8 + sequence, of small GEMMs on
// v_mfma_f32_16x16x32_bf16, a wave per 16 output channels (and row tile where a layer has fewer channels); a tap is then 8 rows
// further, and a lane's four accumulator rows are the same four sequences in every layer.
// Inputs are staged in LDS once and rotated back there for rotary models; activations stay in LDS as three bf16 terms whose sum
// is the fp32 activation exactly, each multiplied in its own MFMA: the arithmetic of the per-head scoring.  A lane's weights of 8
// input channels and 3 taps are 24 consecutive elements of its channel's row.
// Bound: latency.  The role is as long as the streaming beside it where sequences are few, so everything it reads is requested
// before anything is waited for: one trip to the token indices, one to rows, table entries, weights, biases and output projection.
// With each of those read where it is used (a row's sequence by a division, a piece's table entries behind the piece, biases at
// a layer's end) the role ended 10.0 us after the launch's start for one sequence, 16.3 for 32 and 19 for 32 of a rotary model;
// now 6.8, 8.3 and 9.6.  The step: one sequence 12.2 -> 10.7 us, 32 of a rotary model 22.7 -> 20.6.
// Earlier forms: the windows of the whole batch packed in the main launch and scored by the prefill kernel in a launch of its own
// took 9-12 us of the step, and scoring each (sequence, head) in the workgroup that streams it 14 us of a 20 us step.
constexpr int kDeepSeqs = 8;
constexpr float kMaxBf16 = 3.3895314e38f;                    // above: infinity in bf16
constexpr int kDeepMaxCh = 64;                              // output channels per layer
constexpr int kDeepXS = 2 * 64 + 8, kDeepAS = kDeepMaxCh + 8;   // row strides: 16-byte reads of 16 rows cover all banks
constexpr int kDeepOffB = kDeepSeqs * 7 * kDeepXS * 2;      // region A: inputs, later layer 2's output; region B: layer 1's
constexpr int kDeepTerms = 3;                               // of an activation
constexpr int kDeepLds = kDeepOffB + kDeepTerms * kDeepSeqs * 5 * kDeepAS * 2;
static_assert(kDeepTerms * kDeepSeqs * 3 * kDeepAS * 2 <= kDeepOffB, "layer 2's output fits region A");

template <int CH> struct DeepWeights { u32x4 w[CH][3]; };   // [32-channel chunk][tap], as B operands
template <int CH> struct DeepRaw { u32x4 w[CH][3]; };       // a lane's 24 consecutive elements of its channel's row per chunk

template <int CH>
__device__ __forceinline__ void load_deep_weights(const CnnDev& cnn, int l, int cin, int h, int ct, int col, int kg, DeepRaw<CH>& R) {
  const uint16_t* base = static_cast<const uint16_t*>(cnn.w[l]) + ((int64_t)(h * cnn.c_out[l] + 16 * ct + col) * cin + 8 * kg) * 3;
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) {
    const u32x4* p = reinterpret_cast<const u32x4*>(base + (32 * ch < cin ? 32 * ch : 0) * 3);
#pragma unroll
    for (int i = 0; i < 3; ++i) R.w[ch][i] = p[i];
  }
}
template <int CH>
__device__ __forceinline__ void sort_deep_weights(const DeepRaw<CH>& R, DeepWeights<CH>& W) {
#pragma unroll
  for (int ch = 0; ch < CH; ++ch) {
    auto raw = [&](int i) { return R.w[ch][i / 4][i % 4]; };
#pragma unroll
    for (int tap = 0; tap < 3; ++tap)
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const int f0 = 2 * e2 * 3 + tap, f1 = f0 + 3;
        const uint32_t lo16 = (f0 & 1) ? (raw(f0 / 2) >> 16) : (raw(f0 / 2) & 0xFFFFu);
        const uint32_t hi16 = (f1 & 1) ? (raw(f1 / 2) & 0xFFFF0000u) : (raw(f1 / 2) << 16);
        W.w[ch][tap][e2] = lo16 | hi16;
      }
  }
}

__device__ __forceinline__ void score_new_tokens_deep(const CnnDev& cnn, const StepParams& P, const CacheDev& C,
                                                      const bf16_t* __restrict__ k_new, const bf16_t* __restrict__ v_new,
                                                      int h, int b0, unsigned char* lds, int* t_lds, float* __restrict__ ws_logit) {
  constexpr int D = 64;
  static_assert(kDeepSeqs == 8 && kRoleThreads == 256, "rows are position * 8 + sequence");
  const int tid = threadIdx.x, lane = tid & (kWave - 1), col = lane & 15, kg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int L = cnn.n_layers, dil = P.unit, rho = P.rho, window = P.window;
  const int n_in = 2 * L + 1;                                      // input positions, rho = L * dil to either side
  const int nc0 = cnn.c_out[0] / 16, nc1 = cnn.c_out[1] / 16, nc_last = cnn.c_out[L - 1] / 16;      // 1, 2 or 4 column tiles
  // ---- requests, in the order in which they are needed: token indices, first layer's weights, then (they wait for the token
  // indices) rows and table entries ----
  // Row i * 8 + seq is position t - rho + (i - L) * dil of sequence b0 + seq.  A thread brings one piece (8 of keys, 8 of values)
  // of every second position of one sequence; t = -1: no such sequence, no position of it is valid.
  const int seq = (tid >> 4) & 7, pc = tid & 15, i_first = tid >> 7;
  const bool there = b0 + seq < P.B;
  int t = C.n_seen[there ? b0 + seq : P.B - 1];
  // rotation: pieces of keys, row (tid >> 3) + 32 * v
  const bool rotates = P.rope.cos != nullptr;
  const int rot_seq = (tid >> 3) & 7, rot_e0 = (tid & 7) * 8, rot_i = tid >> 6;
  int rot_t = -1;
  if (rotates) {
    rot_t = C.n_seen[b0 + rot_seq < P.B ? b0 + rot_seq : P.B - 1];
    if (b0 + rot_seq >= P.B) rot_t = -1;
  }
  DeepRaw<4> raw0;
  load_deep_weights<4>(cnn, 0, 2 * D, h, wv % nc0, col, kg, raw0);
  if (!there) t = -1;
  if (pc == 0 && i_first == 0) t_lds[seq] = t;
  constexpr int kPerThread = 4, kRotPerThread = 2;
  u32x4 piece[kPerThread];
  const int64_t head = (int64_t)(b0 + seq) * P.Hkv + h;
  const bool is_v = pc >= 8;
  const int slot_t = t >= 0 ? (int)((unsigned)t % (unsigned)window) : 0;
  auto position = [&](int i) { return t - (2 * L - i) * dil; };
#pragma unroll
  for (int u = 0; u < kPerThread; ++u) {
    const int i = i_first + 2 * u, back = (2 * L - i) * dil;       // window > 2 rho
    const bf16_t* row;
    if (i == 2 * L) row = (is_v ? v_new : rotates && P.kf_new != nullptr ? static_cast<const bf16_t*>(P.kf_new) : k_new) + head * D;
    else row = static_cast<const bf16_t*>(is_v ? C.v_win : C.k_win) + (head * window + (slot_t - back < 0 ? slot_t - back + window : slot_t - back)) * D;
    if (!(i < n_in && position(i) >= 0 && t >= 0)) row = v_new;    // somewhere readable: not used
    piece[u] = reinterpret_cast<const u32x4*>(row)[pc & 7];
  }
  RopeEntries<bf16_t> entries[kRotPerThread];
  bool rot[kRotPerThread];
  if (rotates) {
#pragma unroll
    for (int v = 0; v < kRotPerThread; ++v) {
      const int i = rot_i + 4 * v, p = rot_t - (2 * L - i) * dil;
      rot[v] = i < n_in && rot_t >= 0 && p >= 0 && p < P.rope.n_pos && rot_e0 < P.rope.rot_dim && (i < 2 * L || P.kf_new == nullptr);
      entries[v] = load_rope_entries<bf16_t>(P.rope, rot[v] ? p : 0, rot[v] ? rot_e0 : 0);
    }
  }
  // what the layers' ends need: all of it on its way now
  const float bias0 = cnn.bias[0][h * cnn.c_out[0] + 16 * (wv % nc0) + col], bias1 = cnn.bias[1][h * cnn.c_out[1] + 16 * (wv % nc1) + col];
  const float bias2 = L == 3 ? cnn.bias[2][h * cnn.c_out[2] + 16 * (wv % nc_last) + col] : 0.f;
  const int cl = cnn.c_out[L - 1];
  float wo[kDeepMaxCh / 16];
#pragma unroll
  for (int j = 0; j < kDeepMaxCh / 16; ++j) wo[j] = to_f32(static_cast<const bf16_t*>(cnn.w_out)[h * cl + (16 * j < cl ? 16 * j : 0) + col]);
  const float b_out = cnn.b_out[h];
  DeepWeights<4> w0;
  sort_deep_weights<4>(raw0, w0);
  bf16_t* xs = reinterpret_cast<bf16_t*>(lds);
#pragma unroll
  for (int u = 0; u < kPerThread; ++u) {
    const int i = i_first + 2 * u;
    if (i < n_in) *reinterpret_cast<u32x4*>(xs + (8 * i + seq) * kDeepXS + pc * 8) = position(i) >= 0 && t >= 0 ? piece[u] : u32x4{0u, 0u, 0u, 0u};
  }
  __syncthreads();
  if (rotates) {
    u32x4 back[kRotPerThread];
#pragma unroll
    for (int v = 0; v < kRotPerThread; ++v) {
      const bf16_t* row = xs + (8 * (rot_i + 4 * v) + rot_seq) * kDeepXS;
      if (rot[v])
        back[v] = rotate_back<bf16_t>(P.rope, rot_e0, entries[v], *reinterpret_cast<const u32x4*>(row + rot_e0),
                                      *reinterpret_cast<const u32x4*>(row + rope_partner(P.rope, rot_e0)));
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kRotPerThread; ++v)
      if (rot[v]) *reinterpret_cast<u32x4*>(xs + (8 * (rot_i + 4 * v) + rot_seq) * kDeepXS + rot_e0) = back[v];
    __syncthreads();
  }
  DeepRaw<2> raw1;
  load_deep_weights<2>(cnn, 1, cnn.c_out[0], h, wv % nc1, col, kg, raw1);

  // one layer: `pos_in` positions in `src` (the terms term_off elements apart; 0: one term) to pos_in - 2 positions in `dst`
  // (three terms) or, from the last layer, fp32 rows of kDeepMaxCh
  auto layer = [&](int l, const auto& W, float bias, int chunks, int pos_in, const bf16_t* src, int stride, int term_off, unsigned char* dst,
                   bool last) __attribute__((always_inline)) {
    constexpr int kCh = sizeof(W.w) / sizeof(W.w[0]);
    const int nc = cnn.c_out[l] / 16, ct = wv % nc, pos_out = pos_in - 2, n_rows = 8 * pos_out, half = (pos_out - 1) / 2;
    const int4 t4 = *reinterpret_cast<const int4*>(t_lds + 4 * (kg & 1));
    const int ts[4] = {t4.x, t4.y, t4.z, t4.w};                    // of the sequences of this lane's four rows
    for (int rt = wv / nc; 16 * rt < n_rows; rt += kRoleWaves / nc) {
      const int r = 16 * rt + col < n_rows ? 16 * rt + col : n_rows - 1;
      const bf16_t* a = src + r * stride + 8 * kg;
      f32x4 acc[kDeepTerms] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int ch = 0; ch < kCh; ++ch) {
        if (ch >= chunks) break;
#pragma unroll
        for (int tap = 0; tap < 3; ++tap) {
          const bf16_t* ap = a + 8 * tap * stride + 32 * ch;
          const bf16x8 w = __builtin_bit_cast(bf16x8, W.w[ch][tap]);
          acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(ap), w, acc[0], 0, 0, 0);
          if (term_off != 0) {
#pragma unroll
            for (int u = 1; u < kDeepTerms; ++u)
              acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(ap + u * term_off), w, acc[u], 0, 0, 0);
          }
        }
      }
      const int pos = 2 * rt + (kg >> 1);
      if (pos >= pos_out) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ro = 16 * rt + 4 * kg + e, so = 4 * (kg & 1) + e;
        float y = acc[0][e];
        if (term_off != 0) y += acc[1][e] + acc[2][e];
        y += bias;
        // activations at positions before the sequence start are zero padding, not Swish(bias)
        const float val = ts[e] - rho + (pos - half) * dil >= 0 ? y * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504f * y)) : 0.f;
        if (last) {
          reinterpret_cast<float*>(dst)[so * kDeepMaxCh + 16 * ct + col] = val;
        } else {
          bf16_t* d = reinterpret_cast<bf16_t*>(dst) + ro * kDeepAS + 16 * ct + col;
          const bf16_t t0 = static_cast<bf16_t>(val);
          const float r1 = fabsf(val) <= kMaxBf16 ? val - to_f32(t0) : 0.f;     // infinite: no lower terms
          const bf16_t t1 = static_cast<bf16_t>(r1);
          d[0] = t0;
          d[n_rows * kDeepAS] = t1;
          d[2 * n_rows * kDeepAS] = static_cast<bf16_t>(r1 - to_f32(t1));
        }
      }
    }
  };
  const bf16_t* region_a = reinterpret_cast<const bf16_t*>(lds);
  const bf16_t* region_b = reinterpret_cast<const bf16_t*>(lds + kDeepOffB);
  layer(0, w0, bias0, 4, n_in, region_a, kDeepXS, 0, lds + kDeepOffB, false);
  DeepWeights<2> w1;
  sort_deep_weights<2>(raw1, w1);
  DeepRaw<2> raw2;
  if (L == 3) load_deep_weights<2>(cnn, 2, cnn.c_out[1], h, wv % nc_last, col, kg, raw2);
  __syncthreads();
  layer(1, w1, bias1, cnn.c_out[0] / 32, n_in - 2, region_b, kDeepAS, kDeepSeqs * (n_in - 2) * kDeepAS, lds, L == 2);
  __syncthreads();
  if (L == 3) {
    DeepWeights<2> w2;
    sort_deep_weights<2>(raw2, w2);
    layer(2, w2, bias2, cnn.c_out[1] / 32, n_in - 4, region_a, kDeepAS, kDeepSeqs * (n_in - 4) * kDeepAS, lds + kDeepOffB, true);
    __syncthreads();
  }
  const float* act = reinterpret_cast<const float*>(L == 2 ? lds : lds + kDeepOffB);
  if (tid < 16 * kDeepSeqs) {
    const int s = tid / 16, b = b0 + s, ts = t_lds[s];
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < kDeepMaxCh / 16; ++j)
      if (16 * j < cl) z = fmaf(act[s * kDeepMaxCh + 16 * j + col], wo[j], z);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) z += __shfl_xor(z, off, kWave);
    if (col == 0 && b < P.B && ts - rho >= 0) put_logit(C, P, (int64_t)b * P.Hkv + h, ts, z + b_out, ws_logit);
  }
}

// ---- the finishing of one (sequence, KV head) ----------------------------------------------------------------------
// Merge of the shares' records into the group's output rows, eight records at a time in flight.  Record per (sequence,
// query head, share): [max, sum, acc[D]].
template <typename T, int D, int NT>
__device__ __forceinline__ void merge_shares(const StepParams& P, const float* __restrict__ partial, T* __restrict__ out, int b,
                                             int h, bool late) {
  const int G = P.Hq / P.Hkv, nsplit = P.nsplit;
  for (int item = threadIdx.x; item < G * D; item += NT) {
    const int g = item / D, d = item - g * D;
    const int64_t bh = (int64_t)b * P.Hq + h * G + g;
    const float* rec = partial + bh * nsplit * (D + 2);
    float M = -INFINITY, L = 0.f, A = 0.f;
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
      float m[8], l[8], a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float* r = rec + (s0 + u < nsplit ? s0 + u : s0) * (D + 2);
        m[u] = load_shared(r);
        l[u] = load_shared(r + 1);
        a[u] = load_shared(r + 2 + d);
      }
      float m_new = M;
#pragma unroll
      for (int u = 0; u < 8; ++u) m_new = fmaxf(m_new, m[u]);
      if (m_new == -INFINITY) continue;          // no share so far saw a row
      const float f0 = soft_exp<T>(M - m_new);
      L *= f0;
      A *= f0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float f = s0 + u < nsplit ? soft_exp<T>(m[u] - m_new) : 0.f;
        L = fmaf(l[u], f, L);
        A = fmaf(a[u], f, A);
      }
      M = m_new;
    }
    out[bh * D + d] = from_f32<T>(late ? __builtin_nanf("") : A / L);
  }
}

// Cache update: evicted row -> compact slot dst (-1: dropped), then token t and the new logit -> ring.  Every thread of the
// workgroup calls it after its last read of this head's state; it begins with a barrier.  thread 0 holds z_e and z_new.
struct MovingRows { u32x4 old_piece, new_piece; };   // this thread's 16-byte piece of the two rows (keys, then values)

template <typename T, int D>
__device__ __forceinline__ MovingRows load_moving_rows(const CacheDev& C, const StepParams& P, const T* __restrict__ k_new,
                                                       const T* __restrict__ v_new, int64_t head, int t) {
  constexpr int pieces = D * (int)sizeof(T) / 16;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));       // (its addresses are worked out here)
  MovingRows m = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
  if (tid < 2 * pieces) {
    const bool k = tid < pieces;
    const int pc = k ? tid : tid - pieces;
    m.old_piece = reinterpret_cast<const u32x4*>(static_cast<const T*>(k ? C.k_win : C.v_win) + (head * P.window + t % P.window) * D)[pc];
    m.new_piece = reinterpret_cast<const u32x4*>((k ? k_new : v_new) + head * D)[pc];
  }
  return m;
}

template <typename T, int D>
__device__ __forceinline__ void update_cache(const CacheDev& C, const StepParams& P, const MovingRows& rows, int64_t head, int t,
                                             int dst, float z_e, float z_new, bool puts_logit) {
  const int tid = threadIdx.x, window = P.window, slot = t % window;
  T* kw = static_cast<T*>(C.k_win) + (head * window + slot) * D;
  T* vw = static_cast<T*>(C.v_win) + (head * window + slot) * D;
  constexpr int pieces = D * (int)sizeof(T) / 16;
  const bool moves_k = tid < pieces, moves_v = tid >= pieces && tid < 2 * pieces;
  const int pc = moves_k ? tid : (moves_v ? tid - pieces : 0);
  const u32x4 old_piece = rows.old_piece, new_piece = rows.new_piece;
  __syncthreads();
  if (dst >= 0) {
    T* kr = static_cast<T*>(C.k_ret) + (head * P.budget + dst) * D;
    T* vr = static_cast<T*>(C.v_ret) + (head * P.budget + dst) * D;
    if (moves_k || moves_v) reinterpret_cast<u32x4*>(moves_k ? kr : vr)[pc] = old_piece;
    if (tid == 0) {
      C.ret_score[head * P.budget + dst] = select_key(z_e, t - window, P.sink);
      C.ret_pos[head * P.budget + dst] = t - window;
    }
  }
  if (moves_k || moves_v) reinterpret_cast<u32x4*>(moves_k ? kw : vw)[pc] = new_piece;
  if (tid == 0 && puts_logit) C.win_score[head * window + ((t - P.rho) % window)] = z_new;
}

// The finalised logit scored outside the step: the position's row in the sequence's scored window.
__device__ __forceinline__ float given_logit(const StepParams& P, int b, int h, int t) {
  const int first = t - 2 * P.rho > 0 ? t - 2 * P.rho : 0;
  return P.pre_logits[(int64_t)h * P.pre_total + (int64_t)b * (2 * P.rho + 1) + (t - P.rho - first)];
}

template <typename T, int D>
__global__ void __launch_bounds__(kThreads)
decode_finish_kernel(CacheDev C, StepParams P, const T* __restrict__ k_new, const T* __restrict__ v_new, Handover H,
                     T* __restrict__ out) {
  const int b = blockIdx.x / P.Hkv, h = blockIdx.x - b * P.Hkv;
  const int64_t head = (int64_t)b * P.Hkv + h;
  // t comes from the workspace copy made by the main launch: n_seen[b] itself is advanced below by the
  // h == 0 workgroup while other workgroups of the same sequence may still be starting.
  const int t = H.t[b];
  const int dst = P.budget > 0 ? H.dst[head] : -1;
  const float z_e = t >= P.window ? C.win_score[head * P.window + t % P.window] : 0.f;
  const bool puts_logit = !P.lazy && t - P.rho >= 0;
  const float z_new = !puts_logit ? 0.f : P.pre_logits != nullptr ? given_logit(P, b, h, t) : H.logit[head];
  const bool late = P.lazy && t >= P.window && C.n_scored[b] <= t - P.window;
  const int cnt_old = P.budget > 0 ? C.ret_count[head] : 0;
  const MovingRows rows = load_moving_rows<T, D>(C, P, k_new, v_new, head, t);
  merge_shares<T, D, kThreads>(P, H.partial, out, b, h, late);
  update_cache<T, D>(C, P, rows, head, t, dst, z_e, z_new, puts_logit);
  if (threadIdx.x == 0) {
    if (dst >= 0 && dst == cnt_old) C.ret_count[head] = cnt_old + 1;
    if (h == 0) {
      C.n_seen[b] = t + 1;
      if (!P.lazy) C.n_scored[b] = t + 1 > P.rho ? t + 1 - P.rho : 0;
      if (late && P.status != nullptr) atomicOr(P.status, LTEA_LATE_SCORING);
    }
  }
}

// ---- streaming for grouped queries (bf16): up to 16 query heads of a KV group per pass, on MFMA --------------------------
// One wave takes 32 ring slots or 32 compact slots at a time, every W-th block of the workgroup's share:
//   S^T[row, head] = K . Q^T     v_mfma_f32_16x16x32_bf16, K rows straight from global memory into the A operand (a lane
//                                holds 8 columns of one row), Q as the B operand (unused columns are zeros)
//   O^T[d, head] += V^T . P^T    V rows pass through 32 rows of LDS of the wave's own (no barrier: a wave's LDS operations
//                                are in order) and come back transposed (ds_read_b64_tr_b16); P goes from the
//                                accumulator registers of S^T into the B operand as three bf16 terms whose sum is the fp32
//                                probability exactly (8 bits of mantissa each): products with bf16 values are exact, so O is
//                                what fp32 multiply-adds give
// Groups of up to 5 query heads (GT = 5) use the columns that they leave empty for the terms: column 5 * term + head of one
// MFMA, every lane working out the probability of its head and keeping its column's term of it.  Wider groups (GT = 16) take
// an MFMA per term.  Paper's layer (4 query heads per KV head), 32 sequences, in us per lazy step: 19.5 with two terms in two
// MFMAs (16 bits), 23.4 with three in three, 20.1 with three in one.
// In the accumulators a lane owns one column (lane % 16) and four rows per tile, so the softmax state is per lane.  The next
// 32 rows are in flight from memory during this block.  Bound: HBM.  With fp32 VALU products instead (one row per 8
// lanes, four heads) the paper's layer at B = 32 took 22.9 us for 84 MB of rows: the unpacking, the four dot products and
// their shuffles were as much VALU time as the rows' flight; the same launch on MFMA 18.3 us.
template <int D> struct MfmaStream {
  static constexpr int QK = D / 32;              // matrix instructions over the head dimension, per 16 rows
  static constexpr int DT = D / 16;              // output tiles
  static constexpr int RPI = 64 / (D / 8);       // rows per wave load instruction of V
  static constexpr int NV = 32 / RPI;
  static constexpr int kTile = 32 * D;           // LDS elements per wave
  struct Rows { u32x4 k[2][QK]; u32x4 v[NV]; };
  // 32-byte chunk c of row r sits at chunk c ^ swz(r): eight consecutive rows of one chunk then cover all 64 banks
  static __device__ __forceinline__ int swz(int r) { return D == 64 ? (r >> 1) & 3 : r & 7; }
};

__device__ __forceinline__ u32x2 read_transposed4(const bf16_t* p) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p)));
}

// GT = query heads of a KV group handled per pass over the rows: every K/V row is loaded once per pass and used for GT
// queries, so grouped-query configurations do not re-stream the cache once per query head.  1, 2 or 4 on the VALU (fp32
// storage, and bf16 with one query head per KV head); up to 5 or up to 16 on MFMA (bf16).
// W = waves per workgroup.  SK = scoring compiled into this instance: 3, 5 or 7 the batched single-layer role of that kernel
// size, kDeepRole the one for stacks, kPerHead one (sequence, KV head) per workgroup, 0 none: one instance holding all
// would carry the largest one's registers.
template <typename T, int D, int GT, int W, int SK>
__global__ void __launch_bounds__(W * kWave, GT >= 5 && D == 128 ? 2 : 4)
decode_step_kernel(CnnDev cnn, CacheDev C, StepParams P, const T* __restrict__ q, const T* __restrict__ k_new,
                   const T* __restrict__ v_new, Handover H, T* __restrict__ out) {
  constexpr int NT = W * kWave;
  constexpr int kHeads = GT >= 5 ? 16 : 1;   // columns merged at once
  extern __shared__ __align__(16) float dyn_lds[];  // per-head scoring: two generations of activation rows
  __shared__ float red_m[W][kHeads], red_l[W][kHeads];
  // merge of the waves; before that the wave-private V tiles of the MFMA stream; the batched scoring roles' scratch.  The 16
  // columns of the MFMA stream write theirs side by side: four words between the rows spread them over all 64 banks (rows of D
  // words meet in 4 of them).  Groups of up to five heads: lazy steps of 32 sequences of the paper's layer 19.1 -> 18.9 us, of a
  // layer with D = 128 37.7 -> 36.9; 8 heads: 26.7 -> 25.8 at D = 128, 18.0 -> 17.6 at D = 64; 16 heads: 20.7 -> 18.8 (8 sequences,
  // D = 128), 16.4 -> 15.7 (32, D = 64).
  constexpr int kRow = GT >= 5 ? D + 4 : D;
  constexpr int kMerge = W * kHeads * kRow, kRole = SK == kDeepRole ? kDeepLds / 4 : SK > 1 ? 2048 : 0;
  __shared__ __align__(16) float scratch[kMerge > kRole ? kMerge : kRole];
  __shared__ unsigned long long red64[W];
  __shared__ int slot_lds;
  __shared__ __align__(16) int t_lds[kDeepSeqs];

  const int Hkv = P.Hkv, window = P.window, budget = P.budget, nsplit = P.nsplit;
  if constexpr (SK != 0) {
    if ((int)blockIdx.x < P.n_score_blocks) {
      int first_seq, n_seqs;                    // whose logits this workgroup finalises
      if constexpr (SK == kPerHead) {
        const int64_t sh = blockIdx.x;
        first_seq = (int)(sh / Hkv);
        n_seqs = 1;
        const int t = C.n_seen[first_seq];
        if (t - P.rho >= 0) score_token<T, NT>(cnn, P, C, k_new, v_new, sh, (int)(sh - (int64_t)first_seq * Hkv), t, dyn_lds, H.logit);
      } else {
        if (threadIdx.x >= kRoleThreads) return;
        n_seqs = SK == kDeepRole ? kDeepSeqs : kSingleSeqs;
        const int h = blockIdx.x % Hkv;
        first_seq = (int)(blockIdx.x / Hkv) * n_seqs;
        if constexpr (SK == kDeepRole)
          score_new_tokens_deep(cnn, P, C, k_new, v_new, h, first_seq, reinterpret_cast<unsigned char*>(scratch), t_lds, H.logit);
        else if (P.rope.cos != nullptr)
          score_new_tokens_mfma<D, SK, true>(cnn, P, C, k_new, v_new, h, first_seq, scratch, H.logit);
        else
          score_new_tokens_mfma<D, SK, false>(cnn, P, C, k_new, v_new, h, first_seq, scratch, H.logit);
      }
      const int b = first_seq + (int)threadIdx.x;
      const bool mine = (int)threadIdx.x < n_seqs && b < P.B;
      const int t = mine ? C.n_seen[b] : 0;
      if (mine && P.status != nullptr && past_tables(P, t)) atomicOr(P.status, LTEA_ROPE_RANGE);
      if (P.fused) {
        __syncthreads();                        // every wave has read the counters
        if (mine) advance_if_last(C, P, b, t, count_arrival(C, P, b));
      }
      return;
    }
  }
  const int work = (int)blockIdx.x - P.n_score_blocks;
  const int split = work % nsplit;
  const int64_t head = work / nsplit;
  const int b = (int)(head / Hkv), h = (int)(head - (int64_t)b * Hkv);
  int t = load_uniform(C.n_seen + b);
  uint32_t count_word = budget > 0 ? (uint32_t)load_uniform(C.ret_count + head) : 0;
  int scored = P.lazy ? load_uniform(C.n_scored + b) : 0;
  const T* kw = static_cast<const T*>(C.k_win) + head * window * D;
  const T* vw = static_cast<const T*>(C.v_win) + head * window * D;
  const int G = P.Hq / Hkv;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);

  using MS = MfmaStream<D>;
  typename MS::Rows cur;
  // V: this lane's row of an instruction and its 16-byte piece
  const int kg = lane >> 4, c16 = lane & 15, v_row = lane / (D / 8), v_piece = lane % (D / 8);
  const uint32_t k_off = (uint32_t)(c16 * D + 8 * kg) * 2u, v_off = (uint32_t)(v_row * D + 8 * v_piece) * 2u;
  // shares: whole blocks of 32 ring slots or 32 compact slots on the matrix path, rows otherwise
  const int ring_blocks = (window + 31) / 32, all_blocks = ring_blocks + (budget + 31) / 32;
  const int blk_chunk = (all_blocks + nsplit - 1) / nsplit, blk_begin = split * blk_chunk;
  const int blk_end = blk_begin + blk_chunk < all_blocks ? blk_begin + blk_chunk : all_blocks;
  const int first = blk_begin + wave;
  const int chunk = (window + budget + nsplit - 1) / nsplit, r_begin = split * chunk;
  const int r_end = r_begin + chunk < window + budget ? r_begin + chunk : window + budget;
  const bool decides = budget > 0 && (GT >= 5 ? blk_end > ring_blocks : r_end > window);      // some of its rows are compact slots
  // 32 rows from ks, vs on, the first `n_rows` of them real (the others read as zeros)
  auto load_rows = [&](const T* ks, const T* vs, int n_rows, typename MS::Rows& R) {
    // (the compiler does not see that these are the same in all lanes: it would put a loop over the lanes' descriptors around each load)
    auto same = [](const T* p) {
      const uint64_t a = reinterpret_cast<uint64_t>(p);
      return reinterpret_cast<T*>((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32 |
                                  (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a));
    };
    const uint32_t bytes = __builtin_amdgcn_readfirstlane((uint32_t)n_rows * (uint32_t)(D * 2));
    const auto rk = __builtin_amdgcn_make_buffer_rsrc(same(ks), 0, bytes, 0x00020000);
    const auto rv = __builtin_amdgcn_make_buffer_rsrc(same(vs), 0, bytes, 0x00020000);
    constexpr int kNonTemporal = 2;
    // the offsets again, known to be small: the constants are then part of the instructions, not six registers kept over the loop
    uint32_t ko = k_off, vo = v_off;
    asm volatile("" : "+v"(ko), "+v"(vo));
    ko &= 4095u;
    vo &= 4095u;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < MS::QK; ++i)
        R.k[j][i] = __builtin_amdgcn_raw_buffer_load_b128(rk, ko + (uint32_t)(16 * j * D + 32 * i) * 2u, 0, kNonTemporal);
#pragma unroll
    for (int i = 0; i < MS::NV; ++i)
      R.v[i] = __builtin_amdgcn_raw_buffer_load_b128(rv, vo + (uint32_t)(MS::RPI * i * D) * 2u, 0, kNonTemporal);
  };
  // Requests, before anything is known of the sequence: the compact segment's keys, where the token leaving the window may go; on
  // the matrix path a wave's first rows, whatever they hold: settle() takes out what is not there yet.  Then the scalar words, the
  // decision and everything up to the stream's loop pass under the rows' flight.  What it replaces: the words as vector loads, each
  // waiting for the rows before it, and the keys requested once the count was known, read a second time for the victim's slot: the
  // decision was there 3 to 4 us after a launch's start.
  HeldKeys held;
  held = load_held_keys<NT>(decides ? budget : 1, decides ? C.ret_score + head * budget : reinterpret_cast<const float*>(C.n_seen),
                            decides ? C.ret_pos + head * budget : C.n_seen);      // (no branch: they would be waited for at its end)
  constexpr int EPL = Piece<T>::N;  // elements per lane
  constexpr int LPR = D / EPL;      // lanes per row
  constexpr int GPW = kWave / LPR;  // row groups per wave
  constexpr int GPB = GPW * W;
  constexpr int RIF = GT >= 5 ? 1 : GT >= 4 ? 2 : kRowsInFlight;   // rows in flight per lane group (registers: GT states per lane)
  const int sub = lane % LPR, grp = lane / LPR, r_first = r_begin + wave * GPW + grp;
  u32x4 kraw[RIF], vraw[RIF];
  // Which first rows are requested ahead.  Matrix path, D = 64: all.  Steps of 1 / 8 / 32 / 128 sequences, 32 query heads on 8, a
  // window of 800, a budget of 512, the paper's stack, us without -> with: full caches 10.2 12.7 19.8 57.7 -> 9.8 13.0 19.5 57.6
  // (lazy 9.7 10.8 18.5 55.8 -> 9.5 10.6 17.8 54.9); sequences of 200 tokens, where most of the rows do not exist yet, 9.0 11.1
  // 12.8 27.1 -> 9.0 11.4 13.6 27.7 (lazy 8.3 9.1 11.1 25.3 -> 8.4 9.4 11.0 24.9); of 40 tokens 9.0 10.3 12.1 24.4 -> 9.0 11.6
  // 13.2 26.5.
  // D = 128, where eight waves' first rows, 128 KB, keep a CU's vector cache for about a microsecond, beside scoring workgroups:
  // none (a window of 1024, k = 5: full 12.0 18.1 36.3 124.9 -> 12.5 19.4 37.3 125.3, 200 tokens 10.2 15.4 22.0 52.1 -> 11.1 15.8
  // 22.8 53.0, 40 tokens 10.2 13.8 20.5 45.1 -> 10.9 15.4 21.7 49.1).  Without scoring, whole heads and halves gain from all of
  // them (32 sequences: full 36.5 -> 35.9, no budget 25.2 -> 23.8; but 40 tokens 15.2 -> 17.6), shares down to a seventh from the
  // ring's (8 sequences: full 17.4 -> 17.0, only the ring full 15.7 -> 14.9; but 40 tokens 11.5 -> 13.2), smaller ones from none
  // (one sequence: full 12.5 -> 12.7, 200 tokens 10.4 -> 11.3).
  // VALU path: if all of a workgroup's first rows are ring slots, once the token index has come.
  constexpr bool kAhead = GT >= 5 && (D == 64 || SK == 0);
  const int ahead = D == 64 || nsplit <= 2 ? all_blocks : nsplit < 8 ? ring_blocks : 0;
  const bool early = GT >= 5 ? kAhead && first < (blk_end < ahead ? blk_end : ahead)
                             : r_begin + GPB * RIF <= window && r_begin + GPB * RIF <= r_end;
  const T* kr = static_cast<const T*>(C.k_ret) + head * budget * D;
  const T* vr = static_cast<const T*>(C.v_ret) + head * budget * D;
  if constexpr (kAhead) {
    if (D == 64 || early) {      // (D = 64: a branch costs more than requests of nothing)
      const bool ring = first < ring_blocks;
      const int row0 = 32 * (ring ? first : first - ring_blocks), left = (ring ? window : budget) - row0;
      load_rows((ring ? kw : kr) + (early ? (int64_t)row0 * D : 0), (ring ? vw : vr) + (early ? (int64_t)row0 * D : 0),
                !early ? 0 : left < 32 ? left : 32, cur);
    }
  }
  read_here(t);
  read_here(count_word);
  read_here(scored);
  const int cnt_old = (int)(count_word & P.count_mask);
  const T* kn = k_new + head * D;
  const T* vn = v_new + head * D;

  // The state after this step, described from the state before it.  Rows are addressed in a fixed slot space
  // [ring slots 0..window) ++ [compact slots 0..budget) split evenly, so a share that holds ring slots only never
  // needs the eviction decision.
  const int slot = t % window;
  const int n_valid = t + 1 < window ? t + 1 : window;
  const T* k_evicted = kw + (int64_t)slot * D;  // old ring row that moves to compact slot dst
  const T* v_evicted = vw + (int64_t)slot * D;
  const bool whole = P.fused && nsplit == 1;      // nothing is handed over
  int dst = -1, cnt = 0;
  MovingRows rows;             // requested when the stream is done: they come beside the merge, like the count of arrivals
  unsigned arrivals_before = 0;
  const bool counts = tid == NT - kWave;      // of the last wave: the answer is waited for at once, and merging begins with the others

  float z_e = t >= window ? load_uniform(C.win_score + head * window + slot) : 0.f;
  // lazy mode: the token leaving the window must have been scored by a batched scoring call
  const bool late = P.lazy && t >= window && scored <= t - window;
  auto decide = [&]() {
    read_here(z_e);      // (not before the VALU path's first rows are requested: they need the token index only)
    if (decides) {   // uniform across the workgroup
      dst = __builtin_amdgcn_readfirstlane(eviction_target<NT>(t, window, budget, P.sink, P.tau, cnt_old, z_e, held,
                                                               C.ret_score + head * budget, C.ret_pos + head * budget, red64,
                                                               &slot_lds));
      cnt = cnt_old + (dst == cnt_old ? 1 : 0);
    }
  };
  // merged row (M: natural-log domain) of one query head and column: output, or a record for whoever finishes the head
  auto put_row = [&](int hq, int d, float M, float L, float A) {
    const int64_t bh = (int64_t)b * P.Hq + hq;
    if (whole) {
      out[bh * D + d] = from_f32<T>(late ? __builtin_nanf("") : A / L);
    } else {
      float* rec = H.partial + (bh * nsplit + split) * (D + 2);
      if (d == 0) { store_shared(rec, M); store_shared(rec + 1, L); }
      store_shared(rec + 2 + d, A);
    }
  };

  if constexpr (GT >= 5) {
    static_assert(sizeof(scratch) >= W * MS::kTile * sizeof(bf16_t), "the V tiles of the four waves");
    bf16_t* vt = reinterpret_cast<bf16_t*>(scratch) + wave * MS::kTile;
    const float scale2 = P.scale * 1.4426950408889634f;
    // V^T operand: 16 lanes point at a 4-row x 16-column block; rows 4*kg.. of either half
    const int tr_row = 4 * kg + (c16 >> 2);
    const bf16_t* v_src = vt + tr_row * D + 4 * (lane & 3);
    // rows of block `blk`: ring or compact slots row0 .., `n_live` of them real (the others read as zeros)
    auto where = [&](int blk, bool& ring, int& row0, int& n_live) {
      ring = blk < ring_blocks;
      row0 = 32 * (ring ? blk : blk - ring_blocks);
      const int left = (ring ? n_valid : cnt) - row0;
      n_live = left < 0 ? 0 : (left < 32 ? left : 32);
    };
    // the one row whose contents after this step are somewhere else: the incoming token's, or the evicted one's
    auto replace = [&](bool ring, int row0, typename MS::Rows& R) {
      const int special = (ring ? slot : dst) - row0;      // dst = -1: none
      if (special >= 0 && special < 32 && (ring || dst >= 0)) {
        const T* ks = ring ? kn : k_evicted;
        const T* vs = ring ? vn : v_evicted;
        int k_at = 8 * kg, v_at = 8 * v_piece;       // (worked out here: addresses of every lane are not kept over the loop)
        asm volatile("" : "+v"(k_at), "+v"(v_at));
#pragma unroll
        for (int j = 0; j < 2; ++j)
          if (16 * j + c16 == special) {
#pragma unroll
            for (int i = 0; i < MS::QK; ++i) R.k[j][i] = *reinterpret_cast<const u32x4*>(ks + 32 * i + k_at);
          }
#pragma unroll
        for (int i = 0; i < MS::NV; ++i)
          if (MS::RPI * i + v_row == special) R.v[i] = *reinterpret_cast<const u32x4*>(vs + v_at);
      }
    };
    auto load = [&](int blk, typename MS::Rows& R) {
      bool ring;
      int row0, n_live;
      where(blk, ring, row0, n_live);
      load_rows((ring ? kw : kr) + (int64_t)row0 * D, (ring ? vw : vr) + (int64_t)row0 * D, n_live, R);
      replace(ring, row0, R);
    };
    // the block requested before anything was known: V rows past the last one that counts are zeros (scores are masked)
    auto settle = [&]() {
      bool ring;
      int row0, n_live;
      where(first, ring, row0, n_live);
      if (n_live < 32) {
#pragma unroll
        for (int i = 0; i < MS::NV; ++i)
          if (MS::RPI * i + v_row >= n_live) cur.v[i] = u32x4{0u, 0u, 0u, 0u};
      }
      replace(ring, row0, cur);
    };
    // this lane's column: a head of the pass and (GT = 5) which term of its probabilities
    constexpr bool kTermColumns = GT == 5;
    const int term = kTermColumns ? c16 / 5 : 0, col_head = kTermColumns ? c16 % 5 : c16;
    const float from_second = term > 0 ? 1.f : 0.f, from_third = term > 1 ? 1.f : 0.f;
    bf16x8 qf[MS::QK];
    auto load_queries = [&](int g0) {
#pragma unroll
      for (int i = 0; i < MS::QK; ++i) {
        const bool real = g0 + col_head < G && term < 3;
        u32x4 x = *reinterpret_cast<const u32x4*>(q + ((int64_t)b * P.Hq + h * G + (real ? g0 + col_head : 0)) * D + 32 * i + 8 * kg);
        if (!real) x = u32x4{0u, 0u, 0u, 0u};
        qf[i] = __builtin_bit_cast(bf16x8, x);
      }
    };
    load_queries(0);
    decide();
    if (early) settle();
    for (int g0 = 0; g0 < G; g0 += GT) {
      const int heads_here = G - g0 < GT ? G - g0 : GT;
      if (g0 > 0) load_queries(g0);
      if (first < blk_end && !(early && g0 == 0)) load(first, cur);
      float m_run, l_run;
      f32x4 o[MS::DT];
      auto value_operand = [&](int d) {
        const u32x2 a0 = read_transposed4(v_src + ((d ^ MS::swz(tr_row)) << 4));
        const u32x2 a1 = read_transposed4(v_src + 16 * D + ((d ^ MS::swz(tr_row)) << 4));
        return __builtin_bit_cast(bf16x8, u32x4{a0[0], a0[1], a1[0], a1[1]});
      };
      auto walk = [&](auto all_terms) {
        m_run = -INFINITY;
        l_run = 0.f;
#pragma unroll
        for (int d = 0; d < MS::DT; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int blk = first; blk < blk_end; blk += W) {
          f32x4 sc[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            sc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < MS::QK; ++i)
              sc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, cur.k[j][i]), qf[i], sc[j], 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < MS::NV; ++i) {
            const int r = MS::RPI * i + v_row;
            *reinterpret_cast<u32x4*>(vt + r * D + (((v_piece >> 1) ^ MS::swz(r)) << 4) + (v_piece & 1) * 8) = cur.v[i];
          }
          if (blk + W < blk_end) load(blk + W, cur);
          bool ring;
          int row0, n_live;
          where(blk, ring, row0, n_live);
          float m_new = m_run;
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              sc[j][r] = 16 * j + 4 * kg + r < n_live ? sc[j][r] * scale2 : -INFINITY;
              m_new = fmaxf(m_new, sc[j][r]);
            }
          m_new = fmaxf(m_new, __shfl_xor(m_new, 16, kWave));
          m_new = fmaxf(m_new, __shfl_xor(m_new, 32, kWave));
          const float m_use = m_new == -INFINITY ? 0.f : m_new;    // nothing live yet: every factor below is 0
          const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
          m_run = m_new;
          l_run *= alpha;
          if constexpr (kTermColumns) {
            // p = top + middle + rest, cut to 8 bits each: the lane's term is what the ones above it leave, cut in turn
            auto top = [](float x) { return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); };
            u32x4 cut;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int r = 0; r < 4; r += 2) {
                uint32_t x[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                  const float p = __builtin_amdgcn_exp2f(sc[j][r + e] - m_use);
                  l_run += p;
                  const float y = fmaf(-from_second, top(p), p);
                  x[e] = __float_as_uint(fmaf(-from_third, top(y), y));
                }
                cut[2 * j + r / 2] = __builtin_amdgcn_perm(x[1], x[0], 0x07060302u);    // upper halves
              }
            const bf16x8 pt = __builtin_bit_cast(bf16x8, cut);
#pragma unroll
            for (int d = 0; d < MS::DT; ++d) {
              o[d] *= alpha;
              o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(value_operand(d), pt, o[d], 0, 0, 0);
            }
          } else {
            bf16x8 hi, mid, lo;                // p = hi + mid + lo, exactly
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float p = __builtin_amdgcn_exp2f(sc[j][r] - m_use);
                l_run += p;
                hi[4 * j + r] = static_cast<bf16_t>(p);
                const float rest = p - to_f32(hi[4 * j + r]);
                mid[4 * j + r] = static_cast<bf16_t>(rest);
                lo[4 * j + r] = static_cast<bf16_t>(rest - to_f32(mid[4 * j + r]));
              }
#pragma unroll
            for (int d = 0; d < MS::DT; ++d) {
              const bf16x8 av = value_operand(d);
              o[d] *= alpha;
              o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, hi, o[d], 0, 0, 0);
              if constexpr (decltype(all_terms)::value) {
                o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, mid, o[d], 0, 0, 0);
                o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, lo, o[d], 0, 0, 0);
              }
            }
          }
        }
      };
      walk(std::true_type{});
      // An infinite value times the lower terms of a probability, zero or of either sign, is not the infinity that the
      // probability itself makes of it: such sums are what the leading terms give.
      if constexpr (!kTermColumns) {
        bool finite = true;
#pragma unroll
        for (int d = 0; d < MS::DT; ++d)
#pragma unroll
          for (int r = 0; r < 4; ++r) finite = finite && fabsf(o[d][r]) < INFINITY;
        if (__builtin_amdgcn_ballot_w64(!finite) != 0ull) {
          f32x4 all[MS::DT];
#pragma unroll
          for (int d = 0; d < MS::DT; ++d) all[d] = o[d];
          load(first, cur);
          walk(std::false_type{});
#pragma unroll
          for (int d = 0; d < MS::DT; ++d)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[d][r] = fabsf(all[d][r]) < INFINITY ? all[d][r] : o[d][r];
        }
      }
      // (in every pass: not kept over the next one; also where the finishing is a launch of its own: a branch around it costs more than
      // the 16 bytes a thread, 32 query heads on 2 of D = 64, 128 sequences 21.7 -> 24.9 us, one sequence of 32 on 8 9.7 -> 10.0)
      rows = load_moving_rows<T, D>(C, P, k_new, v_new, head, t);
      // merge of the waves, fixed order; register r of o[d] is head dimension 16*d + 4*kg + r of column c16
      l_run += __shfl_xor(l_run, 16, kWave);
      l_run += __shfl_xor(l_run, 32, kWave);
      __syncthreads();      // every wave is done with its V tile
      if (whole && g0 == 0 && counts) arrivals_before = count_arrival(C, P, b);
      if (col_head < heads_here && term < 3) {
        if (kg == 0) { red_m[wave][c16] = m_run; red_l[wave][c16] = l_run; }
#pragma unroll
        for (int d = 0; d < MS::DT; ++d) *reinterpret_cast<f32x4*>((scratch + (wave * kHeads + c16) * kRow) + 16 * d + 4 * kg) = o[d];
      }
      __syncthreads();
      for (int item = tid; item < heads_here * D; item += NT) {
        const int g = item / D, d = item - g * D;
        // all of it requested before any is used: one trip to LDS instead of one per wave (0.75 -> 0.4 us of a step with 8 waves)
        constexpr int kParts = kTermColumns ? 3 : 1;
        float mw[W], lw[W], part[W][kParts];
#pragma unroll
        for (int w = 0; w < W; ++w) {
          mw[w] = red_m[w][g];
          lw[w] = red_l[w][g];
#pragma unroll
          for (int u = 0; u < kParts; ++u) part[w][u] = scratch[(w * kHeads + 5 * u + g) * kRow + d];
        }
        __builtin_amdgcn_sched_barrier(0);
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) M = fmaxf(M, mw[w]);
        float L = 0.f, A = 0.f;
        if (M != -INFINITY) {
#pragma unroll
          for (int w = 0; w < W; ++w) {
            const float f = __builtin_amdgcn_exp2f(mw[w] - M);
            L = fmaf(lw[w], f, L);
            float a = part[w][0];
            if constexpr (kTermColumns) a = fabsf(a) < INFINITY ? a + (part[w][1] + part[w][2]) : a;
            A = fmaf(a, f, A);
          }
        }
        put_row(h * G + g0 + g, d, M * 0.6931471805599453f, L, A);
      }
      __syncthreads();
    }
  } else {
    bool live[RIF];
    auto load = [&](int r0) {
#pragma unroll
      for (int u = 0; u < RIF; ++u) {
        // Branch-free row selection so that all loads of the iteration are issued back to back; rows that do
        // not exist re-read the incoming token's row and are masked out of the softmax below.
        const int r = r0 + u * GPB;
        const bool in_ring = r < window;
        const int rr = r - window;
        live[u] = (r < r_end) && (in_ring ? r < n_valid : rr < cnt);
        const T* kp = in_ring ? kw + (int64_t)r * D : kr + (int64_t)rr * D;
        const T* vp = in_ring ? vw + (int64_t)r * D : vr + (int64_t)rr * D;
        const bool is_new = in_ring && r == slot;
        const bool is_moved = !in_ring && rr == dst;
        kp = is_moved ? k_evicted : kp;
        vp = is_moved ? v_evicted : vp;
        kp = (is_new || !live[u]) ? kn : kp;
        vp = (is_new || !live[u]) ? vn : vp;
        kraw[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kp + sub * EPL));
        vraw[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vp + sub * EPL));
      }
    };
    if (early) load(r_first);
    decide();
    for (int g0 = 0; g0 < G; g0 += GT) {
      float qf[GT][EPL];
      float m_run[GT], l_run[GT], acc[GT][EPL];
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        Piece<T>::load(q + ((int64_t)b * P.Hq + h * G + g0 + g) * D + sub * EPL, qf[g]);
        m_run[g] = -INFINITY;
        l_run[g] = 0.f;
#pragma unroll
        for (int i = 0; i < EPL; ++i) { qf[g][i] *= P.scale; acc[g][i] = 0.f; }
      }
      for (int r0 = r_first; r0 < r_end; r0 += GPB * RIF) {
        if (!(early && g0 == 0 && r0 == r_first)) load(r0);
        float s[GT][RIF], m_new[GT];
#pragma unroll
        for (int g = 0; g < GT; ++g) m_new[g] = m_run[g];
#pragma unroll
        for (int u = 0; u < RIF; ++u) {
          float kf[EPL];
          Piece<T>::unpack(kraw[u], kf);
#pragma unroll
          for (int g = 0; g < GT; ++g) {
            float d = 0.f;
#pragma unroll
            for (int i = 0; i < EPL; ++i) d = fmaf(qf[g][i], kf[i], d);
#pragma unroll
            for (int off = LPR / 2; off > 0; off >>= 1) d += __shfl_xor(d, off, kWave);
            s[g][u] = live[u] ? d : -INFINITY;
            m_new[g] = fmaxf(m_new[g], s[g][u]);
          }
        }
        if (m_new[0] == -INFINITY) continue;  // nothing live for this lane group yet (liveness is the same for every g)
        float pr[GT][RIF];
#pragma unroll
        for (int g = 0; g < GT; ++g) {
          const float alpha = soft_exp<T>(m_run[g] - m_new[g]);
          l_run[g] *= alpha;
#pragma unroll
          for (int i = 0; i < EPL; ++i) acc[g][i] *= alpha;
#pragma unroll
          for (int u = 0; u < RIF; ++u) {
            pr[g][u] = soft_exp<T>(s[g][u] - m_new[g]);
            l_run[g] += pr[g][u];
          }
          m_run[g] = m_new[g];
        }
#pragma unroll
        for (int u = 0; u < RIF; ++u) {
          float vf[EPL];
          Piece<T>::unpack(vraw[u], vf);
#pragma unroll
          for (int g = 0; g < GT; ++g)
#pragma unroll
            for (int i = 0; i < EPL; ++i) acc[g][i] = fmaf(pr[g][u], vf[i], acc[g][i]);
        }
      }
      rows = load_moving_rows<T, D>(C, P, k_new, v_new, head, t);      // (as above)
      // merge: the row groups of a wave by lane exchange, then the waves through LDS (fixed order -> deterministic)
#pragma unroll
      for (int g = 0; g < GT; ++g) {
        float m = m_run[g];
#pragma unroll
        for (int off = LPR; off < kWave; off <<= 1) m = fmaxf(m, __shfl_xor(m, off, kWave));
        const float f = m == -INFINITY ? 0.f : soft_exp<T>(m_run[g] - m);
        float l = l_run[g] * f;
#pragma unroll
        for (int i = 0; i < EPL; ++i) acc[g][i] *= f;
#pragma unroll
        for (int off = LPR; off < kWave; off <<= 1) {
          l += __shfl_xor(l, off, kWave);
#pragma unroll
          for (int i = 0; i < EPL; ++i) acc[g][i] += __shfl_xor(acc[g][i], off, kWave);
        }
        if (lane == 0) { red_m[wave][0] = m; red_l[wave][0] = l; }
        if (grp == 0) {
#pragma unroll
          for (int i = 0; i < EPL; ++i) scratch[wave * D + sub * EPL + i] = acc[g][i];
        }
        __syncthreads();
        if (whole && g0 + g == 0 && counts) arrivals_before = count_arrival(C, P, b);
        if (tid < D) {
          float mw[W], lw[W], part[W];
#pragma unroll
          for (int w = 0; w < W; ++w) { mw[w] = red_m[w][0]; lw[w] = red_l[w][0]; part[w] = scratch[w * D + tid]; }
          __builtin_amdgcn_sched_barrier(0);
          float M = -INFINITY;
#pragma unroll
          for (int w = 0; w < W; ++w) M = fmaxf(M, mw[w]);
          float L = 0.f, A = 0.f;
          if (M != -INFINITY) {
#pragma unroll
            for (int w = 0; w < W; ++w) {
              const float fw = soft_exp<T>(mw[w] - M);
              L = fmaf(lw[w], fw, L);
              A = fmaf(part[w], fw, A);
            }
          }
          put_row(h * G + g0 + g, tid, M, L, A);
        }
        __syncthreads();
      }
    }
  }

  const bool puts_logit = P.pre_logits != nullptr && t - P.rho >= 0;    // a scoring role has put its logit there itself
  unsigned* word = reinterpret_cast<unsigned*>(C.ret_count + head);
  if (whole) {
    const float z_new = puts_logit && tid == 0 ? given_logit(P, b, h, t) : 0.f;
    update_cache<T, D>(C, P, rows, head, t, dst, z_e, z_new, puts_logit);
    if (tid == 0) {
      if (dst >= 0 && dst == cnt_old) atomicAdd(word, 1u);
      if (h == 0 && late && P.status != nullptr) atomicOr(P.status, LTEA_LATE_SCORING);
    }
    if (counts) advance_if_last(C, P, b, t, arrivals_before);
    return;
  }
  // ---- hand this share over; the last one of the head to get here finishes it ----
  if (tid == 0) {
    if (split == nsplit - 1) store_shared(H.dst + head, dst);     // this share always touches the compact segment
    if (!P.fused && split == 0 && h == 0) H.t[b] = t;
  }
  if (!P.fused) return;
  wait_for_own_stores();
  __syncthreads();
  if (tid == 0) slot_lds = ((atomicAdd(word, 1u << 16) >> 16) & 255u) + 1 == (unsigned)nsplit;
  __syncthreads();
  if (slot_lds == 0) return;
  if (counts) arrivals_before = count_arrival(C, P, b);      // for the head: its other shares have counted themselves
  dst = load_shared(H.dst + head);
  const float z_new = puts_logit && tid == 0 ? given_logit(P, b, h, t) : 0.f;
  merge_shares<T, D, NT>(P, H.partial, out, b, h, late);
  update_cache<T, D>(C, P, rows, head, t, dst, z_e, z_new, puts_logit);
  if (tid == 0) {
    atomicAdd(word, (dst >= 0 && dst == cnt_old ? 1u : 0u) - ((unsigned)nsplit << 16));
    if (h == 0 && late && P.status != nullptr) atomicOr(P.status, LTEA_LATE_SCORING);
  }
  if (counts) advance_if_last(C, P, b, t, arrivals_before);
}

// Positions between the rows that a logit depends on, of the input of layer `first`: the greatest common divisor of the
// dilations from there on (1 where no layer reaches further than its own row).
int receptive_unit(const ltea_cnn& cnn, int first) {
  int g = 0;
  for (int l = first; l < cnn.n_layers; ++l) {
    int a = cnn.kernel[l] > 1 ? cnn.dilation[l] : 0, b = g;
    while (a != 0) { const int r = b % a; b = a; a = r; }
    g = b;
  }
  return g > 0 ? g : 1;
}

// Whether a logit depends on one output of layer l alone: no later layer reaches past its own row.
bool last_reach(const ltea_cnn& cnn, int l) {
  for (int m = l + 1; m < cnn.n_layers; ++m)
    if (cnn.kernel[m] > 1) return false;
  return true;
}

// Stacks that the deep scoring role takes (see score_new_tokens_deep); its weight loads are 16-byte pieces of the rows.
bool deep_role(const ltea_cfg& cfg, const ltea_cnn& cnn) {
  if (cfg.dtype != LTEA_BF16 || cfg.D != 64 || cnn.n_layers < 2 || cnn.n_layers > 3) return false;
  for (int l = 0; l < cnn.n_layers; ++l) {
    const int c = cnn.c_out[l];
    if (cnn.kernel[l] != 3 || cnn.dilation[l] != cnn.dilation[0] || (c != 16 && c != 32 && c != 64)) return false;
    if (l + 1 < cnn.n_layers && c == 16) return false;               // a later layer contracts 32 channels at a time
    if ((reinterpret_cast<uintptr_t>(cnn.w[l]) & 15u) != 0) return false;
  }
  return true;
}
// Kernel size of the batched single-layer role, 0: not that CNN.
int single_layer_role(const ltea_cfg& cfg, const ltea_cnn& cnn) {
  const int ks = cnn.kernel[0];
  return cfg.dtype == LTEA_BF16 && cnn.n_layers == 1 && cnn.c_out[0] <= 32 && (ks == 3 || ks == 5 || ks == 7) ? ks : 0;
}

// Waves per workgroup: the most with which all workgroups, the scoring ones included, are resident at once (16 waves per
// CU at the kernels' registers, 8 for the matrix stream at D = 128, 256 CUs).
int step_waves(int64_t workgroups, bool wide) { return workgroups <= (wide ? 256 : 512) ? 8 : 4; }

template <typename T, int D>
hipError_t run(const ltea_cfg& cfg, const ltea_cnn* cnn_or_null, const StepInputs& in, const ltea_cache& c, int n_seqs,
               void* workspace, const float* given_logits, int64_t given_total, hipStream_t stream) {
  ltea_cnn none;
  memset(&none, 0, sizeof(none));
  const ltea_cnn& cnn = cnn_or_null ? *cnn_or_null : none;
  CacheDev C{c.k_win, c.v_win, c.win_score, c.k_ret, c.v_ret, c.ret_score, c.ret_pos, c.ret_count, c.n_seen, c.n_scored};
  StepParams P;
  memset(&P, 0, sizeof(P));
  P.B = n_seqs; P.Hq = cfg.Hq; P.Hkv = cfg.Hkv; P.D = cfg.D; P.window = cfg.window; P.budget = cfg.budget;
  P.sink = cfg.sink;
  P.rho = cnn_rho(&cnn);
  P.tau = cfg.tau_logit;
  P.scale = cfg.softmax_scale > 0.f ? cfg.softmax_scale : 1.0f / sqrtf((float)cfg.D);
  P.lazy = cnn_or_null == nullptr ? 1 : 0;
  P.unit = receptive_unit(cnn, 0);
  P.lds_row_floats = lds_row_floats(cfg, cnn);
  P.status = in.status;
  P.rope = rope_dev(in.rope);
  P.kf_new = in.kf;
  P.pre_logits = given_logits;
  P.pre_total = given_total;
  CnnDev cd;
  cd.n_layers = cnn.n_layers;
  for (int l = 0; l < LTEA_MAX_CNN_LAYERS; ++l) {
    const bool on = l < cnn.n_layers;
    cd.kernel[l] = on ? cnn.kernel[l] : 1;
    const int in_unit = receptive_unit(cnn, l), out_unit = receptive_unit(cnn, l + 1);
    cd.unit[l] = last_reach(cnn, l) ? in_unit : out_unit;      // a single row has no spacing
    cd.row_step[l] = cd.unit[l] / in_unit;
    cd.dilation[l] = on && cnn.kernel[l] > 1 ? cnn.dilation[l] / in_unit : 1;
    cd.c_out[l] = on ? cnn.c_out[l] : 0;
    cd.w[l] = on ? cnn.w[l] : nullptr;
    cd.bias[l] = on ? cnn.bias[l] : nullptr;
  }
  cd.w_out = cnn.w_out;
  cd.b_out = cnn.b_out;
  // The finishing runs inside the launch when the counts fit the upper bits of ret_count: a budget below 2^16 leaves the
  // lower half to the count; the workgroups of a sequence and the shares of a head (at most 64) are eight bits each.
  const bool scores = !P.lazy && given_logits == nullptr;
  P.fused = cfg.budget > 0 && cfg.budget < (1 << 16) && 2 * cfg.Hkv <= 255 && (!scores || P.rho >= 1);
  P.count_mask = P.fused ? 0xFFFFu : 0xFFFFFFFFu;
  P.nsplit = decode_num_splits(cfg, n_seqs);
  const int64_t heads = (int64_t)n_seqs * cfg.Hkv;
  Handover H;
  H.partial = static_cast<float*>(workspace);
  H.logit = H.partial + partial_floats(cfg, n_seqs, P.nsplit);
  H.t = reinterpret_cast<int32_t*>(H.logit + heads);
  H.dst = H.t + n_seqs;
  const int G = cfg.Hq / cfg.Hkv;
  const int role = !scores ? 0 : deep_role(cfg, cnn) ? kDeepRole : single_layer_role(cfg, cnn) != 0 ? single_layer_role(cfg, cnn) : kPerHead;
  P.seq_arrivals = scores ? 2 * cfg.Hkv : cfg.Hkv;
  const int per_group = role == kDeepRole ? kDeepSeqs : role == kPerHead ? 1 : kSingleSeqs;
  P.n_score_blocks = role == 0 ? 0 : cfg.Hkv * ((n_seqs + per_group - 1) / per_group);
  const size_t lds_bytes = role == kPerHead ? (size_t)2 * (2 * P.rho / P.unit + 1) * P.lds_row_floats * sizeof(float) : 0;
  auto launch_sk = [&](auto gt, auto waves, auto sk) {
    hipLaunchKernelGGL((decode_step_kernel<T, D, decltype(gt)::value, decltype(waves)::value, decltype(sk)::value>),
                       dim3((unsigned)(P.n_score_blocks + heads * P.nsplit)), dim3(decltype(waves)::value * kWave), lds_bytes, stream,
                       cd, C, P, static_cast<const T*>(in.q), static_cast<const T*>(in.k), static_cast<const T*>(in.v), H,
                       static_cast<T*>(in.out));
  };
  auto launch = [&](auto gt, auto waves) {
    if (role == 0) return launch_sk(gt, waves, std::integral_constant<int, 0>{});
    if constexpr (sizeof(T) == 2) {
      if constexpr (D == 64) {
        if (role == kDeepRole) return launch_sk(gt, waves, std::integral_constant<int, kDeepRole>{});
      }
      if (role == 3) return launch_sk(gt, waves, std::integral_constant<int, 3>{});
      if (role == 5) return launch_sk(gt, waves, std::integral_constant<int, 5>{});
      if (role == 7) return launch_sk(gt, waves, std::integral_constant<int, 7>{});
    }
    launch_sk(gt, waves, std::integral_constant<int, kPerHead>{});
  };
  auto launch_gt = [&](auto gt) {
    constexpr bool kWide = decltype(gt)::value >= 5 && D == 128;
    const int w = step_waves(heads * P.nsplit + P.n_score_blocks, kWide);
    if (w == 8) return launch(gt, std::integral_constant<int, 8>{});
    launch(gt, std::integral_constant<int, 4>{});
  };
  if constexpr (sizeof(T) == 2) {
    // one query head leaves 15 of the 16 matrix columns idle and streams as fast on the VALU
    if (G > 5) launch_gt(std::integral_constant<int, 16>{});
    else if (G > 1) launch_gt(std::integral_constant<int, 5>{});
    else launch_gt(std::integral_constant<int, 1>{});
  } else {
    if (G % 4 == 0) launch_gt(std::integral_constant<int, 4>{});
    else if (G % 2 == 0) launch_gt(std::integral_constant<int, 2>{});
    else launch_gt(std::integral_constant<int, 1>{});
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || P.fused) return e;
  hipLaunchKernelGGL((decode_finish_kernel<T, D>), dim3((unsigned)heads), dim3(kThreads), 0, stream, C, P,
                     static_cast<const T*>(in.k), static_cast<const T*>(in.v), H, static_cast<T*>(in.out));
  return hipGetLastError();
}

}  // namespace
}  // namespace ltea
