// Prefill attention over window + retained set (paper Section 3.1.3) in fp32 arithmetic, for fp32 storage and for bf16
// views beyond the addressing of the bf16 matrix kernel.
//
// One workgroup = 16 consecutive queries of one (sequence, query head); its four waves take the 16-key blocks of the
// tile's keys (window positions, then compact slots) in turn and merge once at the end through LDS.  Products run on
// v_mfma_f32_16x16x4_f32, exact fp32 multiply-adds:
//   S^T[key, query] = K . Q^T      a lane group of 16 contracts its own quarter of the head dimension, so that every
//                                  lane reads D/4 consecutive values of one key row (the order of a sum over d is free)
//   O^T[d, query]  += V^T . P^T    step r contracts the keys 4*g + r of lane group g: exactly the probabilities a lane
//                                  holds in accumulator register r, so P feeds the product without moving
// In the accumulator layout a lane owns one query, so the softmax state is per lane; rows go from global memory to
// registers, one block ahead.  Small problems are what this path sees, so the bound is latency: a tile of window 64 +
// budget 32 is two blocks per wave.  512 tokens x 2 heads (D = 64): 29 us with one wave per query and scalar row loads,
// 7 us in this form (a whole prefill 18.2 us, 18.5 with the test for sums that are not finite).
#include "ltea_common.h"
#include "ltea_kernels.h"

namespace ltea {
namespace {

constexpr int kWaves = 4;
constexpr int kBlock = 16;     // queries per workgroup, and keys per block

// N consecutive elements as fp32, in the widest aligned loads (N * sizeof(T) is a multiple of 8)
template <int N> __device__ __forceinline__ void load_run(const float* p, float (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    const f32x4 y = *reinterpret_cast<const f32x4*>(p + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[i + e] = y[e];
  }
}
template <int N> __device__ __forceinline__ void load_run(const bf16_t* p, float (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    const bf16x4 y = *reinterpret_cast<const bf16x4*>(p + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[i + e] = to_f32(y[e]);
  }
}

template <typename T, int D>
__global__ void __launch_bounds__(kWaves * kWave, 2)
attention_fp32_kernel(const T* __restrict__ q, int64_t q_st, int64_t q_sh, const T* __restrict__ k,
                      const T* __restrict__ v, int64_t kv_st, int64_t kv_sh, const int32_t* __restrict__ cu,
                      int n_seqs, int64_t total, int Hq, int Hkv, int window, int budget, float scale,
                      const T* __restrict__ k_ret, const T* __restrict__ v_ret,
                      const int32_t* __restrict__ ret_pos, const int32_t* __restrict__ ret_count,
                      T* __restrict__ out, float* __restrict__ lse, const int32_t* __restrict__ kv_start,
                      const int32_t* __restrict__ kv_len) {
  constexpr int DK = D / 4;      // values of a key row per lane
  constexpr int DV = D / 16;     // values of a value row per lane
  constexpr int OS = D + 4;      // merge row stride
  __shared__ float m_lds[kWaves][kBlock], l_lds[kWaves][kBlock];
  __shared__ __align__(16) float o_lds[kWaves][kBlock][OS];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int ql = lane & 15, g = lane >> 4;
  const int hq = blockIdx.y, h = hq / (Hq / Hkv);
  int s, tile, lo_q, n;
  if (!locate_tile(cu, n_seqs, kBlock, (int)blockIdx.x, s, tile, lo_q, n)) return;
  // cu packs the query / output rows.  Normally it packs the keys as well; with kv_start / kv_len given, the keys of
  // sequence s are rows kv_start[s] .. kv_start[s] + kv_len[s] - 1 of k / v and the queries are the last
  // cu[s+1] - cu[s] positions of that key sequence (continuation of a prefill).
  int64_t lo = lo_q;
  int q_begin = 0;
  if (kv_start != nullptr) {
    const int nq = n;
    lo = kv_start[s];
    n = kv_len[s];
    q_begin = n - nq;
  }
  const int64_t head = (int64_t)s * Hkv + h;
  const int i0 = q_begin + tile * kBlock;
  const int i_last = (i0 + kBlock < n ? i0 + kBlock : n) - 1;
  const int qi = i0 + ql;                                          // this lane's query position
  const int64_t q_row = lo_q + (qi <= i_last ? qi : i_last) - q_begin;

  float qf[DK];
  load_run<DK>(q + q_row * q_st + (int64_t)hq * q_sh + g * DK, qf);

  const int jlo = i0 - window + 1 > 0 ? i0 - window + 1 : 0;
  const int n_win = (i_last - jlo) / kBlock + 1;                   // blocks of window keys jlo ..
  const int cnt = (budget > 0 && i_last - window >= 0) ? ret_count[head] : 0;
  const int n_blocks = n_win + (cnt + kBlock - 1) / kBlock;
  const T* kb = k + lo * kv_st + (int64_t)h * kv_sh;
  const T* vb = v + lo * kv_st + (int64_t)h * kv_sh;
  const T* krb = k_ret + head * budget * D;
  const T* vrb = v_ret + head * budget * D;
  const int32_t* prb = ret_pos + head * budget;

  // one block's rows: keys row `ql` (this lane's quarter), values rows 4*g + r, and for compact slots their positions
  struct Rows { float k[DK]; float v[4][DV]; int pos[4]; };
  auto load = [&](int blk, Rows& R) {
    const bool win = blk < n_win;
    const int base = win ? jlo + blk * kBlock : (blk - n_win) * kBlock;
    const int last = win ? n - 1 : cnt - 1;
    const T* kp = win ? kb : krb;
    const T* vp = win ? vb : vrb;
    const int64_t st = win ? kv_st : (int64_t)D;
    const int rk = base + ql < last ? base + ql : last;            // rows past the end re-read the last one, masked below
    load_run<DK>(kp + rk * st + g * DK, R.k);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = base + 4 * g + r, rv = row < last ? row : last;
      load_run<DV>(vp + rv * st + ql * DV, R.v[r]);
      R.pos[r] = win ? row : (row < cnt ? prb[rv] : 0x7FFFFFFF);
    }
  };

  float m_run, l_run;
  f32x4 o[DV];
  // The matrix product multiplies every row of a block by its probability, and 0 * V of a masked pair is not zero when V is
  // not finite.  Sums that end up not finite are therefore formed again (exact) from the pairs whose probability is not zero,
  // one by one.  At the end of the walk: finite inputs, the case that is timed, pay one comparison.
  auto walk = [&](const bool exact) {
    m_run = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int e = 0; e < DV; ++e) o[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    Rows cur;
    if (wave < n_blocks) load(wave, cur);
    for (int blk = wave; blk < n_blocks; blk += kWaves) {
      Rows nxt = cur;
      if (blk + kWaves < n_blocks) load(blk + kWaves, nxt);
      f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < DK; ++i) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.k[i], qf[i], sc, 0, 0, 0);
      const bool win = blk < n_win;
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = cur.pos[r];
        const bool valid = win ? (j <= qi && j > qi - window) : j <= qi - window;
        sc[r] = valid ? sc[r] * scale : -INFINITY;
        mx = fmaxf(mx, sc[r]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
      mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
      const float m_new = fmaxf(m_run, mx);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;        // nothing visible so far: every factor below is 0
      const float alpha = expf(m_run - m_use);
      float p[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = expf(sc[r] - m_use);
      l_run = l_run * alpha + ((p[0] + p[1]) + (p[2] + p[3]));     // this lane's keys; the lane groups meet at the end
      m_run = m_new;
#pragma unroll
      for (int e = 0; e < DV; ++e) o[e] *= alpha;
      if (!exact) {
#pragma unroll
        for (int e = 0; e < DV; ++e)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.v[r][e], p[r], o[e], 0, 0, 0);
      } else {
        const int base = win ? jlo + blk * kBlock : (blk - n_win) * kBlock, last = win ? n - 1 : cnt - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          for (int kg = 0; kg < 4; ++kg) {
            const float pk = __shfl(p[r], 16 * kg + ql, kWave);
            const int row = base + 4 * kg + r, rv = row < last ? row : last;
            const T* vp = (win ? vb + rv * kv_st : vrb + (int64_t)rv * D) + DV * 4 * g;
            if (pk == 0.f) continue;
#pragma unroll
            for (int e = 0; e < DV; ++e)
#pragma unroll
              for (int r2 = 0; r2 < 4; ++r2) o[e][r2] = fmaf(pk, to_f32(vp[DV * r2 + e]), o[e][r2]);
          }
      }
      cur = nxt;
    }
  };
  walk(false);
  bool finite = true;
#pragma unroll
  for (int e = 0; e < DV; ++e)
#pragma unroll
    for (int r = 0; r < 4; ++r) finite = finite && fabsf(o[e][r]) < INFINITY;
  if (__builtin_amdgcn_ballot_w64(!finite) != 0ull) walk(true);

  // ---- merge of the waves: register r of o[e] is head dimension DV * (4*g + r) + e of query ql -----------------
  l_run += __shfl_xor(l_run, 16, kWave);
  l_run += __shfl_xor(l_run, 32, kWave);
  if (g == 0) { m_lds[wave][ql] = m_run; l_lds[wave][ql] = l_run; }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int e = 0; e < DV; ++e) o_lds[wave][ql][DV * (4 * g + r) + e] = o[e][r];
  __syncthreads();
  const int row = threadIdx.x / 16, col = (threadIdx.x % 16) * DV;
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) M = fmaxf(M, m_lds[w][row]);
  float L = 0.f, f[kWaves];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    f[w] = expf(m_lds[w][row] - M);                                // 0 for a wave that saw no key of this query
    L = fmaf(l_lds[w][row], f[w], L);
  }
  if (i0 + row > i_last) return;
  const int64_t o_row = lo_q + i0 + row - q_begin;
  const float inv = 1.0f / L;
  T* orow = out + (o_row * Hq + hq) * D + col;
#pragma unroll
  for (int e = 0; e < DV; ++e) {
    float a = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) a = fmaf(o_lds[w][row][col + e], f[w], a);
    orow[e] = from_f32<T>(a * inv);
  }
  if (lse != nullptr && col == 0) lse[(int64_t)hq * total + o_row] = M + logf(L);   // wanted by a backward pass
}

template <typename T, int D>
hipError_t run(const ltea_cfg& cfg, const void* q, int64_t q_st, int64_t q_sh, const void* k, const void* v,
               int64_t kv_st, int64_t kv_sh, const SeqView& sv, const ltea_cache& c, void* out, float scale,
               float* lse, const int32_t* kv_start, const int32_t* kv_len, hipStream_t stream) {
  const dim3 grid((unsigned)((sv.total_tokens + kBlock - 1) / kBlock + sv.n_seqs), (unsigned)cfg.Hq);
  hipLaunchKernelGGL((attention_fp32_kernel<T, D>), grid, dim3(kWaves * kWave), 0, stream,
                     static_cast<const T*>(q), q_st, q_sh, static_cast<const T*>(k), static_cast<const T*>(v), kv_st,
                     kv_sh, sv.cu_seqlens, sv.n_seqs, sv.total_tokens, cfg.Hq, cfg.Hkv, cfg.window, cfg.budget, scale,
                     static_cast<const T*>(c.k_ret), static_cast<const T*>(c.v_ret), c.ret_pos, c.ret_count,
                     static_cast<T*>(out), lse, kv_start, kv_len);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attention_generic(const ltea_cfg& cfg, const void* q, int64_t q_st, int64_t q_sh, const void* k,
                                    const void* v, int64_t kv_st, int64_t kv_sh, const SeqView& sv,
                                    const ltea_cache& c, void* out, hipStream_t stream, float* lse,
                                    const int32_t* kv_start, const int32_t* kv_len) {
  if (sv.total_tokens == 0) return hipSuccess;
  const float scale = cfg.softmax_scale > 0.f ? cfg.softmax_scale : 1.0f / sqrtf((float)cfg.D);
  if (cfg.dtype == LTEA_F32) {
    return cfg.D == 64 ? run<float, 64>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, scale, lse, kv_start, kv_len, stream)
                       : run<float, 128>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, scale, lse, kv_start, kv_len, stream);
  }
  return cfg.D == 64 ? run<bf16_t, 64>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, scale, lse, kv_start, kv_len, stream)
                     : run<bf16_t, 128>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, scale, lse, kv_start, kv_len, stream);
}

}  // namespace ltea
