// What the decode step's launchers (decode.hip) and its kernel (decode_step.h, instantiated per storage type and head size
// in decode_*.hip) share.
#pragma once
#include "ltea_common.h"
#include "ltea_kernels.h"
#include "rope_dev.h"

namespace ltea {

struct CacheDev {
  void *k_win, *v_win;
  float* win_score;
  void *k_ret, *v_ret;
  float* ret_score;
  int32_t *ret_pos, *ret_count, *n_seen, *n_scored;
};

struct StepInputs { const void *q, *k, *v, *kf; const ltea_rope* rope; void* out; int32_t* status; };

inline size_t partial_floats(const ltea_cfg& cfg, int n_seqs, int nsplit) {
  return (size_t)n_seqs * cfg.Hq * nsplit * (cfg.D + 2);
}

inline int widest_row(const ltea_cfg& cfg, const ltea_cnn& cnn) {
  int row_floats = 2 * cfg.D;
  for (int l = 0; l < cnn.n_layers; ++l) row_floats = cnn.c_out[l] > row_floats ? cnn.c_out[l] : row_floats;
  return row_floats;
}
inline int lds_row_floats(const ltea_cfg& cfg, const ltea_cnn& cnn) { return (widest_row(cfg, cnn) + 3) / 4 * 4; }

// The step for one storage type and head size.  cnn_or_null == null: the lazy step; given_logits: scored windows of
// [Hkv][given_total] (see launch_decode_step_scored).
#define LTEA_DECODE_RUN(name)                                                                                              \
  hipError_t name(const ltea_cfg& cfg, const ltea_cnn* cnn_or_null, const StepInputs& in, const ltea_cache& c, int n_seqs, \
                  void* workspace, const float* given_logits, int64_t given_total, hipStream_t stream)
LTEA_DECODE_RUN(decode_run_f32_64);
LTEA_DECODE_RUN(decode_run_f32_128);
LTEA_DECODE_RUN(decode_run_bf16_64);
LTEA_DECODE_RUN(decode_run_bf16_128);

}  // namespace ltea
