// How a call is cut into workgroups and where its scratch lives: plain C++, so that the rules can be looked at without
// a GPU library (a test compiles this header by itself).
#pragma once

#include <cmath>
#include <cstddef>
#include <cstdint>

#include "adamas.h"

namespace adamas {

// Code format and distance estimator, one id for both:
//   kMetricL1   2-bit codes, Eq. 6 (sum of |a - b|, 0..384): the method
//   kMetricL2   2-bit codes, squared differences (Section 4.4 ablation, 0..1152)
//   kMetricB1   1-bit codes, Eq. 6 = Hamming distance (Section 4.4, 0..128)
//   kMetricB3   3-bit codes, Eq. 6 (Section 4.4, 0..896)
constexpr int kMetricL1 = 0, kMetricL2 = 1, kMetricB1 = 2, kMetricB3 = 3;

constexpr int kHistBatch = 16;  // tiles whose histograms the select kernel loads together
constexpr int kMaxParts = 16;   // attention partial slots per head in the workspace
// floats per attention partial of a head of dimension d: m, l, pad, pad, o[d]
constexpr int partial_stride(int d) { return d + 4; }
constexpr int kTargetWorkgroups = 256;  // one per compute unit of an MI355X
constexpr int kSegGranule = 4096;

// How one call is cut into workgroups and where its scratch lives in the workspace.
struct Plan {
  int tile_tokens;   // tokens per scan workgroup (threads = tile_tokens / 4): 1024, 2048 or 4096
  int n_tiles;       // scan tiles per (sequence, KV head)
  int seg_len;       // tokens per select workgroup, kSegGranule times a power of two (a multiple of the tile)
  int n_segs;        // select workgroups per (sequence, query head)
  int metric;        // code format + distance estimator (struct Dist)
  int head_dim;      // one of ADAMAS_FOR_EACH_HEAD_DIM (kernel_set.hpp)
  int g_shift;       // 2^g_shift scan workgroups per (tile, KV head), each with a share of the query group
  int64_t dist_stride;
  size_t off_dist, off_high, off_hist, off_partial, total;
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

inline int code_bits(const adamas_config* c) { return c->code_bits == 0 ? 2 : c->code_bits; }

// Code format + distance estimator id (see struct Dist).
inline int metric_of(const adamas_config* c) {
  if (code_bits(c) == 1) return kMetricB1;
  if (code_bits(c) == 3) return kMetricB3;
  return (c->variant & ADAMAS_VARIANT_L2) ? kMetricL2 : kMetricL1;
}

// Largest distance of a metric (Dist<METRIC, D>::kMaxDist for run-time arguments).
inline int max_dist_of(int metric, int head_dim) {
  const int per_dim = metric == kMetricL1 ? 3 : metric == kMetricL2 ? 9 : metric == kMetricB1 ? 1 : 7;
  return per_dim * head_dim;
}

// 32-bit words of a tile histogram (Dist<METRIC, D>::kPairs)
inline size_t hist_pairs_of(int metric, int head_dim) { return (size_t)(max_dist_of(metric, head_dim) + 2) / 2; }

// Bytes per token of the distance plane, and whether a plane of ninth bits goes
// with it (Dist<METRIC, D>::kDistBytes, kHighPlane).
inline int dist_bytes_of(int metric, int head_dim) { return max_dist_of(metric, head_dim) <= 511 ? 1 : 2; }
inline bool high_plane_of(int metric, int head_dim) {
  const int m = max_dist_of(metric, head_dim);
  return m > 255 && m <= 511;
}

// Offsets for so many tile histograms.
inline void lay_out(Plan* pl, size_t heads, int64_t max_seq_len, size_t histograms) {
  pl->dist_stride = (max_seq_len + 127) & ~(int64_t)127;
  size_t off = 0;
  pl->off_dist = off;
  off = align256(off + heads * (size_t)pl->dist_stride * dist_bytes_of(pl->metric, pl->head_dim));
  pl->off_high = off;
  if (high_plane_of(pl->metric, pl->head_dim)) off = align256(off + heads * (size_t)pl->dist_stride / 8);
  pl->off_hist = off;
  // + kHistBatch: the select kernel reads whole batches of them, also behind the last head's
  off = align256(off + (histograms + kHistBatch) * hist_pairs_of(pl->metric, pl->head_dim) * sizeof(uint32_t));
  pl->off_partial = off;
  off = align256(off + heads * (size_t)kMaxParts * partial_stride(pl->head_dim) * sizeof(float));
  pl->total = off;
}

// Tiles and offsets that follow from tile_tokens, the metric and the head dimension.
inline void lay_out(Plan* pl, const adamas_config* c, int32_t batch, int64_t max_seq_len) {
  const size_t heads = (size_t)batch * c->num_q_heads;
  pl->n_tiles = (int)((max_seq_len + pl->tile_tokens - 1) / pl->tile_tokens);
  lay_out(pl, heads, max_seq_len, heads * (size_t)pl->n_tiles);
}

// Bytes that the calls of these sizes ask for, whatever their plan: never less for more sequences or a longer context, so that a
// workspace for a program's largest call holds all its smaller ones.  (The plans' own totals are not: a smaller call may
// take smaller tiles, which leave more histograms.)  Tiles are of 2048 tokens or more, except where fewer than two of
// 1024 per compute unit exist, or the context is no longer than one.
inline size_t workspace_need(const adamas_config* c, int32_t batch, int64_t max_seq_len) {
  Plan pl{};
  pl.metric = metric_of(c);
  pl.head_dim = c->head_dim;
  const size_t heads = (size_t)batch * c->num_q_heads, group = (size_t)(c->num_q_heads / c->num_kv_heads);
  const size_t large = heads * (size_t)((max_seq_len + 2047) / 2048);
  size_t small = heads * (size_t)((max_seq_len + 1023) / 1024);
  if (small > 2 * kTargetWorkgroups * group) small = 2 * kTargetWorkgroups * group;
  lay_out(&pl, heads, max_seq_len, large > small ? large : small);
  return pl.total;
}

inline Plan make_plan(const adamas_config* c, int32_t batch, int64_t max_seq_len, int32_t k) {
  (void)k;  // the budget does not change the plan: the workspace holds every distance whatever k is
  Plan pl{};
  pl.metric = metric_of(c);
  pl.head_dim = c->head_dim;
  const int64_t planes = (int64_t)batch * c->num_kv_heads;
  // Scan: tokens per workgroup (4, 8 or 16 waves of 256) and the share of the query group that it serves (all, half or a
  // quarter of it, each share reading the rows again).  A compute unit's time goes with the waves that each of its
  // SIMDs gets, times what a wave does: about as much for the rows, the histogram and the prologue as for one head, and a
  // share of encoding the queries, which costs 1.5 of that per query and is spread over the waves.  Below 2.5 waves per
  // SIMD it is the chain of one wave that takes the time.  The select kernel loads the histograms of kHistBatch tiles at
  // once and pays about four such units for each further batch.  Measured (us per layer, 32 query heads, d = 128; tile /
  // parts of the group, chosen *):                2048 / 1  2048 / 2  4096 / 1  4096 / 2  4096 / 4
  //   1 sequence of 20000, group of 4               13.6     12.6*     15.0      13.3      13.1
  //   1 of 32771                                    14.8     15.6      15.3      14.0*     16.3
  //   1 of 100000                                   22.3     24.0      19.2*     22.1
  //   2 of 20011                                    15.2     16.0      16.3      14.7*     17.4
  //   4 of 30000                                    21.8     24.3      20.9*     22.5
  //   8 ragged, up to 16000                         24.2     25.4      22.6*     25.6
  //   16 ragged, up to 32768 (1024 / 1: 44.2)       42.3     47.8      42.1*     53.5
  //   48 ragged, up to 6001 (1024 / 1: 60.3)        58.5*    60.6      60.3      70.4
  //   2 of 60000, group of 8                        21.5     20.6      22.6      19.1*     22.9
  //   4 of 60001, group of 8                        28.2     28.8      26.5*     26.9
  //   1 of 100000, 16 heads, group of 8             20.3     18.0      21.1      17.5      16.7*
  //   1 of 32768, group of 1                        16.8*              17.2
  //   1 of 50000, group of 1                        21.2               20.1*
  // d = 64, 96, 192 and 256 rank alike (six shapes each).
  const int group = c->num_q_heads / c->num_kv_heads;
  auto n_tiles_of = [&](int tile) { return (max_seq_len + tile - 1) / tile; };
  double best = 0.0;
  for (int tile = 4096; tile >= 1024; tile /= 2) {
    if (tile > 1024 && tile >= 2 * max_seq_len) continue;
    // with workgroups for half of the compute units or more, tiles of 1024 lose
    if (tile == 1024 && pl.tile_tokens != 0 && planes * n_tiles_of(2048) >= kTargetWorkgroups / 2) break;
    for (int shift = 0; shift <= 2 && group % (1 << shift) == 0; ++shift) {
      const int64_t n_wg = planes * n_tiles_of(tile) << shift;
      if (shift > 0 && n_wg > kTargetWorkgroups) break;
      // whole rounds while there are few, the average beyond
      const double per_unit = n_wg < 4 * kTargetWorkgroups ? (double)((n_wg + kTargetWorkgroups - 1) / kTargetWorkgroups)
                                                           : (double)n_wg / kTargetWorkgroups;
      const double waves = std::fmax(2.5, per_unit * (tile / 1024)), heads = group >> shift;
      double cost = waves * (1.0 + heads + 1.5 * heads / (tile / 256)) +
                    4.0 * (double)((n_tiles_of(tile) + kHistBatch - 1) / kHistBatch - 1);
      // one head per row is bound by memory, and two workgroups per unit keep that busier than one (32 planes of 32768: see above)
      if (group == 1 && tile == 4096 && n_wg <= kTargetWorkgroups) cost *= 1.1;
      if (pl.tile_tokens == 0 || cost < best) {
        best = cost;
        pl.tile_tokens = tile;
        pl.g_shift = shift;
      }
    }
  }
  // Select + attention: a head is cut into segments, one workgroup each (a
  // single compute unit is too slow to compact a whole 32K-token head or to
  // gather all of its rows), and the segments' attention partials are merged
  // afterwards (by the last segment to finish, or by the merge kernel in staged
  // calls).  With many heads in flight there is parallelism enough
  // already: fewer segments mean fewer re-reads of the head's histograms, and a
  // head that fits one segment needs no merge at all.
  const int64_t n_heads = (int64_t)batch * c->num_q_heads;
  int64_t want = (2 * kTargetWorkgroups + n_heads - 1) / n_heads;
  if (want > kMaxParts) want = kMaxParts;
  // a power of two (the select kernel shifts instead of dividing) and a multiple of every tile size
  int64_t seg = kSegGranule;
  while (seg * want < max_seq_len) seg *= 2;
  pl.seg_len = (int)seg;
  pl.n_segs = (int)((max_seq_len + seg - 1) / seg);
  lay_out(&pl, c, batch, max_seq_len);
  return pl;
}

// The plan of a call whose scratch is an array of a given size: the chosen one where it fits, else the one with the
// fewest histograms (tiles of 4096 tokens), which needs the least.  Not for calls that bring a workspace: these have the cut that
// takes the least time (41 sequences of 2560 tokens, 32 heads over 8 KV heads: 33.4 us a layer, 34.0 with the fewest histograms).
inline Plan make_plan_within(size_t bytes, const adamas_config* c, int32_t batch, int64_t max_seq_len, int32_t k) {
  const Plan chosen = make_plan(c, batch, max_seq_len, k);
  if (chosen.total <= bytes) return chosen;
  Plan least = chosen;
  least.tile_tokens = 4096;
  least.g_shift = 0;
  lay_out(&least, c, batch, max_seq_len);
  return least.total <= bytes ? least : chosen;
}

// Whether the select kernel requests its first K / V lines ahead of the gather
// (SelectParams::early_rows).  Measured on MI355X: it gains 0.25 to 0.6 us
// where at most two workgroups share a compute unit and a segment takes at most
// four passes (contexts of 32K to 128K at batch 1 to 4), is neutral to slightly
// harmful with eight passes per segment (16 ragged sequences, one segment per
// head), and costs 6 us of 48 with 2048 short heads in flight.
inline int early_rows_pay(const Plan& pl, int64_t n_heads) {
  return n_heads * pl.n_segs <= 2 * kTargetWorkgroups && pl.seg_len <= 4 * kSegGranule ? 1 : 0;
}

}  // namespace adamas
