// The rule for one launch (csrc/plan.hpp) as C functions.  use: 0 decode step, 1 top-k on query codes.
#include "plan.hpp"

extern "C" int one_launch_waves(const adamas_config* c, int32_t batch, int64_t max_seq_len, int32_t k, int32_t use, int32_t paged) {
  return adamas::one_launch_waves((adamas::ScanUse)use, c, batch, max_seq_len, k, paged != 0);
}

extern "C" int64_t one_launch_lds(const adamas_config* c, int waves, int64_t max_seq_len, int32_t k, int32_t use, int32_t paged) {
  return (int64_t)(adamas::one_launch_lds(waves, c->head_dim, max_seq_len, k, use == 0, paged != 0) +
                   adamas::one_launch_static_lds(adamas::metric_of(c), c->head_dim));
}
