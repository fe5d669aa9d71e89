// Instances of the decode step: see decode_step.h.
#include "decode_step.h"

namespace ltea {

LTEA_DECODE_RUN(decode_run_bf16_64) {
  return run<bf16_t, 64>(cfg, cnn_or_null, in, c, n_seqs, workspace, given_logits, given_total, stream);
}

}  // namespace ltea
