// Instances of the decode step: see decode_step.h.
#include "decode_step.h"

namespace ltea {

LTEA_DECODE_RUN(decode_run_f32_64) {
  return run<float, 64>(cfg, cnn_or_null, in, c, n_seqs, workspace, given_logits, given_total, stream);
}

LTEA_DECODE_RUN(decode_run_f32_128) {
  return run<float, 128>(cfg, cnn_or_null, in, c, n_seqs, workspace, given_logits, given_total, stream);
}

}  // namespace ltea
