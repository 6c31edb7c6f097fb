// The library's launch plan as a C function: csrc/plan.hpp is plain C++, so a test can ask it for a call's cut.
// use: 0 decode step, 1 top-k on query codes, 2 distances alone, 3 decode step in the static array.
#include "plan.hpp"

extern "C" void scan_plan(const adamas_config* c, int32_t batch, int64_t max_seq_len, int32_t use, int64_t out[4]) {
  const adamas::Plan pl = use == 3 ? adamas::make_plan_within(ADAMAS_STATIC_SCRATCH_BYTES, c, batch, max_seq_len)
                                   : adamas::make_plan(c, batch, max_seq_len, (adamas::ScanUse)use);
  out[0] = pl.tile_tokens;
  out[1] = 1 << pl.g_shift;
  out[2] = pl.n_tiles;
  out[3] = (int64_t)pl.total;
}

extern "C" int heads_per_part(int group, int g_shift) { return adamas::heads_per_part(group, g_shift); }

extern "C" int sparse_parts(int64_t n_heads, int32_t k, int head_dim) {
  const adamas::SparseCut cut = adamas::sparse_cut(n_heads, k, head_dim);
  return cut.wide ? -cut.parts : cut.parts;
}
