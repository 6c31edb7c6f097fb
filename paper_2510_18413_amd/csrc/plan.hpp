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
  double cost;       // of the cut that choose_cut took (scan_cost)
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

// What a call has the scan do: the decode step (encodes its queries, leaves distances and tile histograms), top-k on
// query codes (the same without the encode), or distances for the caller alone.
enum class ScanUse { kStep, kSelect, kDistances };

// What a cut of the scan costs, in the time that a wave takes for one query head: tiles of `tile` tokens (4, 8 or 16 waves
// of 256) and `parts` workgroups per tile and KV head, each with its share of the group's heads and reading the rows again.
// A compute unit's time goes with the waves that each of its SIMDs gets, times what a wave does: about as much for the rows,
// the histogram and the prologue as for one head, and a share of encoding the queries, twice that per query and spread over
// the waves.  Below a few waves per SIMD it is the chain of one wave that takes the time.  Parts of a group find the rows in
// the L2 of their XCD where the number of tiles is a multiple of the eight XCDs (workgroups go round them in launch order), and
// in memory elsewhere.  The select kernel loads the histograms of kHistBatch tiles at once and pays for each further batch.
//
// Measured (us a layer, 32 query heads, d = 128; tile / parts of the group, chosen *; the median spreads by 0.1):
//                                        2048/1 2048/2 2048/4 4096/1 4096/2 4096/4
//   step,  1 sequence of 16384, group of 4 12.9   11.8   11.4*  14.1   12.4   11.7
//          1 of 20000                      13.1   12.1*  13.7   14.4   12.6   12.6
//          1 of 24576                      13.1   12.2*  13.0   14.2   12.5   13.1
//          1 of 32768                      13.5   12.5   12.8   14.2   12.5   11.8*
//          1 of 32771                      14.3   15.1   16.3   14.9   13.4*  15.7
//          1 of 65540                      20.0   19.6          17.8*  20.1   22.4
//          1 of 100000                     21.9   23.4          19.2*  22.0   28.1
//          2 of 20011                      14.2   15.2   16.6   15.4   14.0*  16.4
//          4 of 60000                      29.3                 27.7*  35.1
//          16 of 17408                     35.2*                35.5
//          16 ragged, up to 32768          40.6                 40.1*
//          1 of 32768, group of 1          15.7*                15.6
//          4 of 32768, group of 1          39.6                 38.4*
//                                        1024/1 1024/2 1024/4 2048/1 2048/2 2048/4 4096/1 4096/2 4096/4
//   top-k, 1 of 4000, group of 4            7.7    7.1    6.7*   8.0    7.5    7.1    9.3    8.1    8.0
//          2 of 20011                      12.2   12.0          10.5   11.1   12.8   11.0   10.2*  12.7
//          16 of 3000                      11.2   11.3          10.5*  11.1   14.4   10.9   11.7   13.7
//   distances, 4 of 8000, group of 2        4.7    4.4           4.9    5.4           5.4    5.4
// The step has no tiles of 1024 tokens: short contexts, where they would pay (1 of 4000: 13.0, 11.9 and 11.5), run as one launch
// (one_launch_waves), and so do the shorter ones of the calls of top-k.
// With three-bit codes the sixteen-wave workgroups of the step spill registers from d = 160 on (1 sequence of 32771, d = 256, group
// of 1: 54.0, 49.2*, 59.8 with tiles of 1024, 2048 and 4096).  Over 972 shapes (d = 64 to 256, groups of 1 to 8, all code
// formats, paged or not) the step's choice is 0.5 % above the best cut on average, top-k's 1.3 and that of the distances alone 3.0;
// where the step's is furthest off (4 to 11 %) the codes are three-bit, or eight heads share a row and two rounds of parts would pay.
inline double scan_cost(ScanUse use, int metric, int head_dim, int64_t n_wg, int64_t n_tiles, int tile, int group, int parts) {
  const bool step = use == ScanUse::kStep;
  const int wg_waves = tile / 256, heads = group / parts;
  // whole rounds while there are few, the average beyond
  const double rounds = n_wg < 4 * kTargetWorkgroups ? (double)((n_wg + kTargetWorkgroups - 1) / kTargetWorkgroups)
                                                     : (double)n_wg / kTargetWorkgroups;
  const double waves = std::fmax(step ? 2.5 : 1.1, rounds * wg_waves / 4);
  const double head = metric == kMetricL2 || metric == kMetricB3 ? 1.2 : 1.0;
  double per_wave = 1.0 + heads * head;
  if (n_tiles % 8 != 0) per_wave += 0.25 * (parts - 1) / parts;
  if (step) per_wave += 2.0 * heads / wg_waves;
  // small workgroups clear and flush as many histograms for fewer tokens
  if (wg_waves == 4) per_wave *= 1.08;
  if (wg_waves == 16 && !step && group > 1) per_wave *= 0.8;
  if (wg_waves == 16 && metric == kMetricB3 && head_dim >= 160) per_wave *= 1.06;
  // One head per row is bound by memory.  Where tiles of 4096 give every compute unit one workgroup, tiles of 2048 give it two, which
  // keep it a little busier if they do not fall on the same channels: 32 planes of 32768 16.2 / 16.4 (16.8 / 17.2 with other
  // caches), 64 of 16384 17.65 / 17.95, 16 planes of two sequences of 32768 17.7 / 16.3.  With units left over the halves are uneven:
  // 32 planes of 20480, 28672 and 36864 15.0 / 14.5, 16.0 / 15.8, 18.5 / 19.3; 8 of 72228 and 131072 16.4 / 14.8, 18.8 / 17.8.
  if (group == 1 && wg_waves == 16 && n_wg == kTargetWorkgroups) per_wave *= 1.1;
  double cost = waves * per_wave + 0.0125 * wg_waves;  // (the smaller workgroup where nothing else tells them apart)
  if (use != ScanUse::kDistances)
    cost += 4.0 * (double)((n_tiles + kHistBatch - 1) / kHistBatch - 1) + 0.4 * (double)n_tiles / kHistBatch;
  return cost;
}

// Query heads per workgroup if 2^g_shift of them share a group; 0 if they cannot share it evenly.
inline int heads_per_part(int group, int g_shift) {
  return g_shift >= 0 && g_shift <= 3 && group % (1 << g_shift) == 0 ? group >> g_shift : 0;
}

// Sets tile_tokens, g_shift and cost.
inline void choose_cut(Plan* pl, ScanUse use, int group, int64_t planes, int64_t max_seq_len) {
  auto n_tiles_of = [&](int tile) { return (max_seq_len + tile - 1) / tile; };
  const int smallest = use == ScanUse::kStep ? 2048 : 1024;
  for (int tile = 4096; tile >= smallest; tile /= 2) {
    if (tile > smallest && tile >= 2 * max_seq_len) continue;
    // never more tiles than two per compute unit in exchange for smaller ones
    if (tile == 1024 && pl->tile_tokens != 0 && planes * n_tiles_of(2048) >= kTargetWorkgroups) break;
    for (int shift = 0; shift <= 2 && heads_per_part(group, shift) != 0; ++shift) {
      const int64_t n_wg = planes * n_tiles_of(tile) << shift;
      if (shift > 0 && n_wg > kTargetWorkgroups) break;
      const double cost =
          scan_cost(use, pl->metric, pl->head_dim, n_wg, n_tiles_of(tile), tile, group, 1 << shift);
      if (pl->tile_tokens == 0 || cost < pl->cost) {
        pl->cost = cost;
        pl->tile_tokens = tile;
        pl->g_shift = shift;
      }
    }
  }
}

// (The budget does not change the plan: the workspace holds every distance whatever it is.)
inline Plan make_plan(const adamas_config* c, int32_t batch, int64_t max_seq_len, ScanUse use) {
  Plan pl{};
  pl.metric = metric_of(c);
  pl.head_dim = c->head_dim;
  choose_cut(&pl, use, c->num_q_heads / c->num_kv_heads, (int64_t)batch * c->num_kv_heads, max_seq_len);
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
inline Plan make_plan_within(size_t bytes, const adamas_config* c, int32_t batch, int64_t max_seq_len) {
  const Plan chosen = make_plan(c, batch, max_seq_len, ScanUse::kStep);
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

// ---- one launch, a workgroup per head (one_launch.hpp) ----

// LDS of such a workgroup that is asked for at launch: the list of rows (paged caches: and that of positions), then the
// distances (16 bits a token), whose place the waves' attention states take afterwards; and what its kernel declares.
inline int32_t one_launch_list(int64_t max_seq_len, int32_t k) { return (int32_t)(((k < max_seq_len ? k : max_seq_len) + 3) & ~(int64_t)3); }
inline size_t one_launch_lds(int waves, int head_dim, int64_t max_seq_len, int32_t k, bool attn, bool paged) {
  const size_t dist = (size_t)((max_seq_len + 63) & ~(int64_t)63) * 2;
  const size_t states = attn ? (size_t)waves * (2 + head_dim) * 4 : 0;
  return (size_t)one_launch_list(max_seq_len, k) * (paged ? 8 : 4) + (dist > states ? dist : states);
}
inline size_t one_launch_static_lds(int metric, int head_dim) { return (size_t)(max_dist_of(metric, head_dim) + 2) * 8 + 1024; }
constexpr size_t kOneLaunchLds = 64 * 1024;  // what a launch may have of a compute unit's 160 KB without asking for more

// Waves of a SIMD that the registers of one_launch_kernel leave room for.
inline int one_launch_waves_per_simd(bool attn, int metric, int d) {
  const bool three = metric == kMetricB3, one = metric == kMetricB1;
  if (attn) return three && d == 256 ? 3 : d == 160 || (three && d >= 160) ? 4 : (d == 256 && !one) || (three && d == 96) ? 5 : 6;
  if (three) return d == 256 ? 4 : d >= 160 ? 5 : d == 96 ? 6 : 8;
  return (d == 160 || d == 256) && !one ? 7 : 8;
}

// The parts of a call that its time in one launch and in two goes with; terms and weights (us) are a least-squares fit to uniform
// lengths of 9000 calls drawn over d = 64 to 256, all code formats, groups of 1 to 8, 1 to 6000 heads, 200 to 31500
// tokens; two thirds of them lie within 11 % of it.
struct CallSize {
  bool step;
  int metric, head_dim, words;        // of a code row, 32 bits each
  double heads, planes, group, length, k;
  double lines;                       // cache lines that the loads of 64 rows touch: a row's pieces each reach for all of them
  double code_mb, gather_mb;          // from memory, 10^6 bytes
};
inline CallSize call_size(ScanUse use, const adamas_config* c, int32_t batch, int64_t max_seq_len, int32_t k) {
  const int row = c->head_dim / 8 * code_bits(c), piece = row % 16 == 0 ? 16 : row % 8 == 0 ? 8 : 4;
  CallSize s{};
  s.step = use == ScanUse::kStep;
  s.metric = metric_of(c);
  s.head_dim = c->head_dim;
  s.words = row / 4;
  s.heads = (double)batch * c->num_q_heads;
  s.planes = (double)batch * c->num_kv_heads;
  s.group = c->num_q_heads / c->num_kv_heads;
  s.length = (double)max_seq_len;
  s.k = k < max_seq_len ? (double)k : (double)max_seq_len;
  s.lines = row / piece * (64.0 * row / 128);
  s.code_mb = s.planes * s.length * row * 1e-6;
  s.gather_mb = s.step ? s.heads * s.k * 4 * s.head_dim * 1e-6 : 0.0;
  return s;
}
// Whole rounds of work while there are few, the average and the uneven last one beyond.
inline double rounds_of(double x) { return x <= 3.0 ? std::ceil(x) : x + 0.5; }

// One launch: a head has its compute unit's rate for its rows.  The planes of an XCD (every eighth one) share its 32 units; what LDS or
// registers do not let in at once starts when another workgroup ends.
inline double one_launch_us(const CallSize& s, int waves, size_t lds) {
  const double share = rounds_of(std::ceil(s.planes / 8) * s.group / 32);          // workgroups of a compute unit
  const double by_lds = std::floor(160.0 * 1024 / (lds + 512.0));
  const double by_waves = std::floor(one_launch_waves_per_simd(s.step, s.metric, s.head_dim) * 4.0 / waves);
  const double generations = std::fmax(1.0, rounds_of(share / std::fmax(1.0, std::fmin(by_lds, by_waves))));
  const double steps = s.length / 64, metric = s.metric == kMetricB3 ? 1.39 : s.metric == kMetricL2 ? 1.25 : 1.0;
  double us = 3.41 + 0.053 * share * waves + 1.5 * (generations - 1.0) + 0.108 * generations * steps / waves +
              share * steps * (0.000809 * metric * s.words + 0.000254 * s.lines) + 0.14 * s.code_mb;
  if (s.step) us += 1.74 + 0.0555 * s.gather_mb + s.k * s.head_dim * 1e-3 * (0.054 * share + 0.364 * generations / waves);
  return us;
}
// Two: the scan is spread over the chip and its rows shared by the heads of a group, and a second kernel waits for it.
inline double two_launch_us(const CallSize& s, const Plan& pl) {
  const double tiles = s.planes * pl.n_tiles * (1 << pl.g_shift), wide = s.heads * pl.n_segs;
  double us = 5.68 + (s.step ? 0.204 : 0.272) * (s.metric == kMetricB3 ? 1.45 : 1.0) * pl.cost * s.words / 8 +
              0.0000945 * rounds_of(tiles / kTargetWorkgroups) * pl.tile_tokens / 64 * s.lines + 0.143 * s.code_mb +
              0.971 * std::fmax(1.0, wide / 512);
  if (s.metric == kMetricL2) us += 0.597 * s.heads * pl.n_tiles / 256;
  if (s.step) us += 1.5 + 0.126 * s.gather_mb + 0.152 * s.k * s.head_dim * 1e-3 / pl.n_segs + (pl.n_segs > 1 ? 1.27 * wide / 256 : 0.0);
  return us;
}

// Waves of the workgroups if the step, or top-k on query codes, is to run as one launch; 0 for scan and select by themselves (pl).
// A head then has one compute unit's rate for its rows, so what decides is the context against the heads that there are to fill the
// chip, in rows of 32 bytes (half of the time goes with the bytes of a row).  us a layer (chosen *):
//                                                two launches    4      8     16 waves
//   step,  one head of 1024 tokens, k = 64              8.5     6.0    5.8*   6.3
//          32 heads of 1000, k = 128                   11.0     7.2    6.6*   7.3
//          32 of 4000, k = 256                         14.1    11.9    9.7    9.7*
//          32 of 8000, k = 128                         11.9    11.2    9.6    9.6*
//          32 of 12000, k = 128                        11.8    13.6   11.6   11.0*
//          32 of 16384, k = 128                        11.5*   15.8   13.3   12.5
//          32 heads alone in their groups, 16384       13.2*   18.8   15.2   14.0
//          256 ragged, up to 8000, k = 256             23.7    18.1   15.3   15.6*
//          384 of 15503, k = 232                       32.6    29.3   28.0*  31.8
//          512 ragged, up to 16469, k = 40             26.9    22.3   21.5*  23.2
//          512 ragged, up to 24000, k = 128            33.0*   37.6   35.9   39.6
//          1536 ragged, up to 6001, paged, k = 256     59.6    52.5*  53.0   67.6
//          2048 of 2048, k = 128                       43.3    38.9*  39.1   59.3
//   top-k, 32 heads of 8000, k = 512                    7.9     9.5    6.8*   7.1
//          32 of 12000                                  8.4*   12.2    8.3    8.1
//          64 of 12000                                  9.8    12.3    8.4    8.2*
//          64 of 20011                                 11.2*   18.2   13.0   12.5
//          256 of 24000                                20.5    21.0   15.5   14.9*
//          512 of 16000                                23.6    22.7   20.7   19.4*
//          512 of 20011                                30.5*   34.2   32.9   31.5
// Sixteen waves where a head is alone on its compute unit and long (or its list is); four where there are several heads for each,
// which then overlap one's gather with another's scan.
// These borders hold for the method at d = 128.  Elsewhere the loads of a longer row take a compute unit several times as long (rows of 64
// bytes touch four times the lines of 32), more workgroups may be due than LDS or registers let in at once, and groups give two
// launches an edge: there the fit has to agree, within what it is off by (up to sixteen heads the step's borders are right more often).  Of
// 9000 calls drawn over all sizes and formats 321 take over 5 % longer than two launches where the borders alone decide (up to 2.4
// times), 132 (up to 1.4) with the fit, and all together take 0.786 of two launches' time; of 440 drawn near the borders 76 and 20.
inline int one_launch_waves(ScanUse use, const adamas_config* c, int32_t batch, int64_t max_seq_len, int32_t k, bool paged, const Plan& pl) {
  const int64_t heads = (int64_t)batch * c->num_q_heads;
  // (the grid's second extent; the kernel's division of a plane by the KV heads is exact below 2^32)
  const int64_t planes = (int64_t)batch * c->num_kv_heads;
  if (use == ScanUse::kDistances || planes > 8 * 65535 || planes * c->num_kv_heads >= (int64_t)1 << 32) return 0;
  const int metric = metric_of(c);
  // (rows that only divide into pieces of four bytes take a load for each; two launches share them among the heads of a group)
  const int row_bytes = c->head_dim / 8 * code_bits(c);
  const double row = row_bytes / 32.0, length = max_seq_len * std::sqrt(row) * (row_bytes % 16 == 0 ? 1.0 : row_bytes % 8 == 0 ? 1.1 : 2.0) +
                                                k * c->head_dim / 128.0;
  const double few = heads < 256 ? (double)heads : 256.0;
  int waves;
  if (use == ScanUse::kStep) {
    if (length >= (heads <= 256 ? 12000.0 + 40.0 * few : row_bytes % 8 == 0 ? 20000.0 : 12000.0)) return 0;
    waves = heads <= 256 && max_seq_len * row + 20.0 * k * c->head_dim / 128 > 8000.0 ? 16 : heads <= 640 ? 8 : 4;
    if (waves == 16 && row >= 3.0) waves = 8;  // (three-bit codes at d = 256 take more registers than sixteen waves may have)
  } else {
    if (max_seq_len >= (heads > 256 ? 18000.0 : 9000.0 + 70.0 * few)) return 0;
    waves = heads > 640 ? 4 : max_seq_len > 8000 ? 16 : 8;
  }
  const size_t lds = one_launch_lds(waves, c->head_dim, max_seq_len, k, use == ScanUse::kStep, paged) +
                     one_launch_static_lds(metric, c->head_dim);
  if (lds > kOneLaunchLds) return 0;
  if (use == ScanUse::kStep && heads <= 16) return waves;
  // Rows that only divide into pieces of four bytes: beyond 5000 tokens top-k in one launch takes 10 to 18 % longer than its estimate.
  // Of 994 such calls that 1.05 lets run as one, 68 are over 5 % slower than two (by up to 44 %), of those that 0.9 does ten (26 %).
  const double within = use == ScanUse::kStep ? 1.1 : row_bytes % 8 == 0 ? 1.05 : 0.9;
  const CallSize size = call_size(use, c, batch, max_seq_len, k);
  return one_launch_us(size, waves, lds) < two_launch_us(size, pl) * within ? waves : 0;
}

// Stand-alone sparse attention: workgroups per head, and whether they are of sixteen waves (one per head then).
struct SparseCut {
  int parts;
  bool wide;
};

// About 32 rows per workgroup, at most kMaxParts workgroups per head; half as many from half as many heads as
// compute units on.  One workgroup per head, which needs no merge launch, where there are at least as many heads as
// compute units and as rows, up to 512 rows.  Powers of two: with 11 or 6 workgroups per head, 96 and 192 heads of 2048
// rows take 22.9 and 37.8 us instead of 17.4 and 30.3 (d = 128).
// One workgroup per head also below that, for up to 16384 elements of K per list (four rows per wave and step, four steps),
// and one of sixteen waves for twice as many where there are 64 to 256 heads (one per compute unit; two of them per unit lose), for
// lists of up to 1024 rows from 192 heads on and below 2048 rows from 208 on: what the other units save in idle time, a long list
// gains by more workgroups.  us as several with their merge / one of four waves / one of sixteen:
//    k d = 16384:  1 head, d = 128  6.1  5.3* 5.6    64 heads  7.0  6.3* 6.2   192 heads  9.1  7.3* 7.2   192, d = 64  9.8  7.2* 7.4
//    k d = 32768:  32 heads         7.0* 8.6  7.3    64 heads  8.3  8.8  7.5*  192 heads 11.1 10.3  9.2*  192, d = 256 11.4 10.4 9.2*
//    k d = 65536:  64 heads         9.7* 13.9 9.9   128 heads 12.3* 16.3 11.9  192 heads 15.5 17.9 14.2*  256 heads 20.0 20.5 17.5*
//    k d = 131072: 64 heads        12.1* 27.3 16.1  128 heads 17.9* 29.7 19.6  192 heads 24.3 31.0 22.8*  256 heads 31.4 34.8 29.2*
// eight workgroups / one of sixteen waves, at 192, 224 and 256 heads:
//    1400 rows  d = 64 17.6* 18.4, 19.7 19.4*, 22.0 20.8*   d = 128 29.5* 29.7, 34.6 33.0*, 38.4 37.0*   d = 256 53.5* 53.1, 63.4 60.4*, 69.2 67.4*
//    1800       d = 64 19.8* 21.4, 22.5 22.8*, 25.2 24.8*   d = 128 35.7* 36.0, 41.6 40.1*, 46.2 44.8*   d = 256 63.9* 65.2, 77.2 73.7*, 84.0 83.3*
//    2048       d = 64 21.1* 23.3, 24.4* 24.8, 27.3* 27.3   d = 128 38.1* 39.7, 45.3* 44.4, 50.2* 49.5   d = 256 70.8* 72.4, 84.7* 81.7, 88.3* 89.4
//    4096       d = 64 33.7* 40.3, 40.2* 43.4, 44.1* 48.1   d = 128 59.4* 67.6, 71.7* 77.1, 78.7* 88.5   d = 256  114*  129,  140*  148,  152*  170
// us at 1 / 4 / 8 / 16 workgroups of four waves per head, d = 64, 128, 256 (chosen: *):
//    96 heads, 2048 rows   26.1  14.5  12.1  12.5*   51.5  22.1  18.0  17.4*   101.6  35.2  28.0  29.2*
//   128 heads,  512 rows    9.0   8.5   8.2*  9.9    14.5  11.6  11.4* 11.7     25.1  16.7  16.4* 16.7
//   128 heads, 1024 rows   15.2  11.5  11.2* 12.0    27.2  16.5  15.8* 15.3     49.8  25.2  24.1* 24.3
//   192 heads, 2048 rows   27.3  20.9  16.9* 19.2    54.3  33.3  28.8* 30.3    107.2  60.9  55.3* 57.3
//   256 heads,  256 rows    6.5*  8.6  10.2  13.7    10.4* 11.9  12.2  13.6     16.1* 17.1  17.2  18.3
//   256 heads, 4000 rows   54.5  37.4  30.6* 30.0   106.5  73.0  62.9* 60.7    203.0 133.3 111.3* 113.6
//   512 heads,  512 rows   15.5* 17.4  17.8  23.5    24.4* 26.8  26.5  28.4     48.1* 52.7  53.5  54.0
//   512 heads, 1500 rows   36.4  33.8  32.4* 35.2    69.3  69.4  62.2* 63.9    121.5 119.9 114.9* 117.4
//  1024 heads, 2048 rows   84.9  79.0  74.5* 82.2   164.6 155.9 141.0* 146.1   319.1 291.3 270.0* 277.5
inline SparseCut sparse_cut(int64_t n_heads, int32_t k, int head_dim) {
  const int64_t elements = (int64_t)k * head_dim;
  const bool wide = elements > 16384 && n_heads <= kTargetWorkgroups &&
                    (elements <= 32768 ? n_heads >= 64 : k <= 1024 ? n_heads >= 192 : k < 2048 && n_heads >= 208);
  if (wide) return {1, true};
  if (elements <= 16384 && n_heads < kTargetWorkgroups) return {1, false};
  if (n_heads >= kTargetWorkgroups && n_heads >= k && k <= 512) return {1, false};
  const int most = n_heads >= kTargetWorkgroups / 2 ? kMaxParts / 2 : kMaxParts, want = (k + 31) / 32;
  return {want < most ? want : most, false};
}

}  // namespace adamas
