// A decode plan as the kernels take it (shared by the decode and the mixed launch).
#pragma once

#include "decode_impl.h"
#include "launch.h"

namespace pkv {

inline dec::DecodeWork decode_work(const DecodePlan& p, const int32_t* seq_lens,
                                   int32_t num_seqs) {
  return dec::DecodeWork{seq_lens, p.ordered ? p.order : nullptr, p.by_rank, num_seqs,
                         p.split,  p.max_splits,                  p.max_keys};
}

}  // namespace pkv
