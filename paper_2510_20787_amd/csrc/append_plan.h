// Device arrays that describe the extended sequences of a continued prefill (see append.hip), written by its build
// kernel and read by the retention kernel.  One entry per sequence unless noted.
#pragma once
#include <stdint.h>

namespace ltea {

struct AppendPlan {
  int32_t* n_old;          // tokens in the cache before the call
  int32_t* w_old;          // min(n_old, window): ring tokens
  int32_t* prefix;         // F: rows in front of the ring (pad + old kept entries)
  int32_t* cu_ext;         // [n_seqs + 1] packing of the extended sequences
  int32_t* cu_score;       // [n_seqs + 1] packing of the rows that are scored
  int32_t* kv_start;       // first row of the ring + new part in the extended buffers
  int32_t* kv_len;         // w_old + new tokens
  int32_t* old_count;      // [n_seqs][Hkv] kept entries before the call (retention sets the cache's own counts)
  int32_t* sorted_pos;     // [n_seqs][Hkv][budget] old kept positions ascending
  int32_t* local_pos;      // [n_seqs][Hkv][budget] kept positions in the ring + new frame (for the attention kernel)
  float* ext_key;          // [Hkv][total_ext] selection keys that were final before the call
  int64_t total_ext;       // rows the extended buffers are sized for
};

}  // namespace ltea
