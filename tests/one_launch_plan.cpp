// The rule for one launch (csrc/plan.hpp) as C functions.  use: 0 decode step, 1 top-k on query codes.
#include "plan.hpp"

extern "C" int one_launch_waves(const adamas_config* c, int32_t batch, int64_t max_seq_len, int32_t k, int32_t use, int32_t paged) {
  const adamas::ScanUse as = (adamas::ScanUse)use;
  return adamas::one_launch_waves(as, c, batch, max_seq_len, k, paged != 0, adamas::make_plan(c, batch, max_seq_len, as));
}

extern "C" int64_t one_launch_lds(const adamas_config* c, int waves, int64_t max_seq_len, int32_t k, int32_t use, int32_t paged) {
  return (int64_t)(adamas::one_launch_lds(waves, c->head_dim, max_seq_len, k, use == 0, paged != 0) +
                   adamas::one_launch_static_lds(adamas::metric_of(c), c->head_dim));
}

extern "C" int one_launch_waves_per_simd(int32_t step, int32_t metric, int32_t head_dim) {
  return adamas::one_launch_waves_per_simd(step != 0, metric, head_dim);
}
