// Manhattan-distance scan over the packed code plane (Algorithm 1, distance
// step, Eq. 6), with the query encode and the cache append of the same
// algorithm fused into its prologue for the decode step.
//
// One workgroup owns one tile of blockDim.x * 4 consecutive tokens of one
// (sequence, KV head) and evaluates all G query heads of that KV head's
// group on it, so every code row is fetched once.  It writes
//   - one distance per (query head, token), staged through LDS so that a lane
//     stores eight consecutive tokens: a byte each (plus one bit per token in a
//     plane of ninth bits) when the metric's distances stay below 512, as Eq. 6
//     does (0..384); uint16 otherwise, and
//   - one histogram of those distances (385 bins for Eq. 6) per (query head, tile),
// both with plain stores: nothing needs zero-initialised memory and the
// result does not depend on the order workgroups run in.
//
// Distance on bit planes.  A row word carries 32 low bits and 32 high bits of
// 32 codes.  With x = query ^ key per plane and g = q_hi ^ q_lo (query only):
//   |a - b| = x_lo + 2 * (x_hi & ~(x_lo & g))
// (x_hi = 0: the codes differ by x_lo; x_hi = 1, x_lo = 0: by 2; both set:
// by 3 when the query code is 0 or 3 (g = 0), by 1 when it is 1 or 2), so a
// 32-coefficient word costs two xor, one and, one and-not and two popcounts.
// The squared-difference variant (Section 4.4) needs one more and + popcount:
//   (a - b)^2 = x_lo + 4 * u + 4 * (u & x_lo),  u = x_hi & ~(x_lo & g).
#pragma once

#include "device_utils.hpp"
#include "encode.hpp"

namespace adamas {

constexpr int kScanTokPerThread = 4;
// LDS histogram copies, picked by lane, to thin out same-address atomics: two
// unless the histograms of the group would then take more than 48 KiB.  The
// tile histogram in memory packs two 16-bit bins per word (a tile has at most
// 4096 tokens).  In LDS a group of up to two query heads keeps that format
// (the scan is then bound by memory and the smaller histogram is flushed
// sooner); larger groups are bound by their instructions and use a 32-bit word
// per bin, whose address is the distance itself and whose increment is a
// constant (measured: 0.2 us slower for a group of one, 0.1 to 0.2 us faster
// for a group of four).
constexpr bool hist_wide_bins(int group) { return group > 2; }
constexpr int hist_replicas(int group, int bins) {
  return group * bins * (hist_wide_bins(group) ? 8 : 4) > 48 * 1024 ? 1 : 2;
}

struct ScanParams {
  const uint8_t* codes;      // [Hkv][pool][32]
  uint8_t* codes_w;          // same buffer, written on append (fused only)
  const uint16_t* q;         // bf16 [B][Hq][128]      (fused)
  const uint8_t* qcodes;     // [B][Hq][32]            (not fused)
  const uint16_t* k_new;     // bf16 [B][Hkv][128] or null
  const uint16_t* v_new;
  uint16_t* K;               // pools, written on append
  uint16_t* V;
  const int64_t* seq_start;  // [B]
  const int32_t* seq_len;    // [B]
  void* dist;                // [B*Hq][dist_stride] bytes or uint16 (Dist<>::kDistBytes); may be null
  uint64_t* dist_high;       // ninth bits, [B*Hq][dist_stride / 64] (Dist<>::kHighPlane only)
  int64_t dist_stride;       // tokens per row, a multiple of 128
  uint16_t* dist_user;       // optional second copy, [B*Hq][dist_user_stride]
  int64_t dist_user_stride;
  uint32_t* tilehist;        // [B*Hq][n_tiles][Dist<>::kPairs] words of two 16-bit bins; may be null
  uint32_t* arrivals;        // per-head counter at [head * arrivals_stride], zeroed here; may be null
  int64_t arrivals_stride;
  int64_t pool_tokens, max_seq_len;
  int32_t Hq, Hkv, n_tiles;
  int32_t g_shift;           // 2^g_shift workgroups per (tile, KV head), each takes G of the group's G << g_shift query heads
  // Paged cache (PAGED kernels only): token t of sequence b lives in pool row
  // page_table[b * max_pages + (t >> page_shift)] << page_shift | (t & page mask).
  const int32_t* page_table;
  int32_t max_pages, page_shift;
  Thresholds thr_q, thr_k;
  // Profiling builds only: one record of phase stamps per workgroup (see PhaseTrace).
  uint64_t* trace;
  int64_t trace_records;
};

// Phase stamps of scan_kernel, in the order they are taken.
enum ScanPhase {
  kScanStart = 0,    // first instruction
  kScanLengthKnown,  // past the early barrier: sequence length and start have arrived
  kScanQueryReady,   // the query planes are published in LDS
  kScanRowsDone,     // every row of the tile has arrived and its distances are in LDS
  kScanDistStored,   // distance stores acknowledged
  kScanEnd           // histogram flushed and acknowledged
};

// (The compiler's own lane write and no inline assembly: a vector instruction that writes a scalar register needs two wait states before
// another one reads it, which the compiler keeps between instructions that it knows.)
extern "C" __device__ uint32_t write_lane(uint32_t x, uint32_t lane, uint32_t v) __asm("llvm.amdgcn.writelane.i32");
// v with lane I's value replaced by the wave-uniform x, whether that lane is active or not: only where the wave branched as a whole, by
// a scalar condition.  (A branch by lanes may be run through with none of them active, and v's register hold another path's value.)
template <int I>
__device__ __forceinline__ uint32_t set_lane(uint32_t v, uint32_t x) {
  return write_lane(x, I, v);
}

// An encoded vector from its wave (every lane holds all of it, w[p][g]: plane p of word g) to LDS, a word per lane: twelve lane
// writes and one store, where a store per plane and lane took a quarter of a microsecond of the chain in front of the distances.
// A query as the distances read it: plane p of word g at [W * p + g]; two-bit codes also keep lo ^ hi at [2 W + g].
template <int BITS, int W>
__device__ __forceinline__ void publish_query(const uint32_t (&w)[BITS][W], uint32_t* to, int lane) {
  constexpr int QP = BITS == 2 ? 3 : BITS;
  uint32_t word = 0;
  static_for<QP * W>([&](auto i_) {
    constexpr int i = decltype(i_)::value, pl = i / W, g = i % W;
    word = set_lane<i>(word, pl < BITS ? w[pl < BITS ? pl : 0][g] : w[0][g] ^ w[BITS - 1][g]);
  });
  if (lane < QP * W) to[lane] = word;
}
// A key as a row of the cache.
template <int BITS, int W>
__device__ __forceinline__ void publish_row(const uint32_t (&w)[BITS][W], uint32_t* to, int lane) {
  uint32_t word = 0;
  static_for<BITS * W>([&](auto i_) {
    constexpr int i = decltype(i_)::value;
    word = set_lane<i>(word, w[i % BITS][i / BITS]);
  });
  if (lane < BITS * W) to[lane] = word;
}

// The distance of a key row (row[BITS * wd + pl]: plane pl of word wd) to the query with planes q(j, wd); for two-bit codes
// plane 2 is lo ^ hi.
template <int METRIC, int D, typename Q>
__device__ __forceinline__ uint32_t row_distance(const uint32_t (&row)[Dist<METRIC, D>::kBits * (D / 32)], Q q) {
  constexpr int BITS = Dist<METRIC, D>::kBits, W = D / 32;
  if constexpr (BITS == 2) {
    uint32_t c1 = 0, c2 = 0;
#pragma unroll
    for (int wd = 0; wd < W; ++wd) {
      // Every instruction below takes one query plane: with two of them in one
      // instruction (the compiler's choice when it may merge them) a plane held
      // in a scalar register must first be copied.  Hence the opaque values.
      uint32_t xl = row[2 * wd] ^ q(0, wd);
      asm("" : "+v"(xl));
      uint32_t both = xl & q(2, wd);
      asm("" : "+v"(both));
      uint32_t u = (row[2 * wd + 1] ^ q(1, wd)) & ~both;
      // (and opaque running sums: the count instruction adds to them, a regrouped sum takes additions of its own)
      c1 += __popc(xl);
      // Squared differences: one sum for both counts, and u made once.  With a third sum and the and from its parts the groups of four,
      // five and seven took 65 and 66 registers at d = 128, and a compute unit held one workgroup of sixteen waves instead of two
      // (16 sequences of 32768 tokens, groups of four: 68.9 us a layer, 62.3 now).
      if constexpr (METRIC == kMetricL2) asm("" : "+v"(u));
      c2 += __popc(u);
      asm("" : "+v"(c1), "+v"(c2));
      if constexpr (METRIC == kMetricL2) c2 += __popc(u & xl);
    }
    return METRIC == kMetricL1 ? c1 + 2u * c2 : c1 + 4u * c2;
  } else if constexpr (BITS == 1) {
    uint32_t c = 0;
#pragma unroll
    for (int wd = 0; wd < W; ++wd) c += __popc(row[wd] ^ q(0, wd));
    return c;
  } else {
    // |a - b| of 3-bit codes on bit planes (a query, b key): subtract with
    // borrow, then negate where the borrow out (a < b) is set.
    uint32_t c0 = 0, c1 = 0, c2 = 0;
#pragma unroll
    for (int wd = 0; wd < W; ++wd) {
      const uint32_t a0 = q(0, wd), a1 = q(1, wd), a2 = q(2, wd);
      const uint32_t b0 = row[3 * wd], b1 = row[3 * wd + 1], b2 = row[3 * wd + 2];
      const uint32_t d0 = a0 ^ b0, br1 = ~a0 & b0;
      const uint32_t x1 = a1 ^ b1, d1 = x1 ^ br1, br2 = (~a1 & b1) | (~x1 & br1);
      const uint32_t x2 = a2 ^ b2, d2 = x2 ^ br2, sg = (~a2 & b2) | (~x2 & br2);
      const uint32_t e1 = d1 ^ sg, cy1 = ~d0 & sg;
      const uint32_t r1 = e1 ^ cy1, cy2 = e1 & cy1;
      const uint32_t r2 = d2 ^ sg ^ cy2;
      c0 += __popc(d0);
      c1 += __popc(r1);
      c2 += __popc(r2);
    }
    return c0 + 2u * c1 + 4u * c2;
  }
}

// Waves per SIMD that the registers of a workgroup have to leave room for, where the compiler takes a few more than that by
// itself.  Fused scans of three-bit codes: at d = 256 130 vector registers, with which a compute unit holds one workgroup of eight
// waves instead of two (16 sequences of 17000 tokens, groups of four: 121.6 us a layer, 102.8 with two); at d = 64, groups of two, 85
// scalar ones, of which eight waves may have 80 (scan of 24 ragged sequences of 24000 tokens 24.5 us, 21.6 with them).  (Groups of
// one and eight at d = 256 need more than a few.)  The scan of one-bit query codes at d = 192, groups of eight: 65, one workgroup of
// sixteen waves instead of two (top-k of 24 sequences of 32000 tokens, 64 heads: 65.2 us, 57.3 with two).
template <int G, bool FUSED, int WAVES, int METRIC, int D>
constexpr int kScanWavesPerSimd = FUSED && METRIC == kMetricB3 && D == 64 && G == 2 && WAVES == 16          ? 8
                                  : FUSED && METRIC == kMetricB3 && D == 256 && G > 1 && G < 8 && WAVES == 8 ? 4
                                  : !FUSED && METRIC == kMetricB1 && D == 192 && G == 8 && WAVES == 16       ? 8
                                                                                                             : WAVES / 4;
// WAVES = wavefronts per workgroup (8 or 16, without the encode also 4): the tile is WAVES * 256 tokens.
// D = head dimension: W = D / 32 words per code row.
template <int G, bool FUSED, int WAVES, int METRIC, bool PAGED, int D>
__global__ __launch_bounds__(WAVES * kWave)
__attribute__((amdgpu_waves_per_eu(kScanWavesPerSimd<G, FUSED, WAVES, METRIC, D>)))
void scan_kernel(const ScanParams p) {
  static_assert(FUSED || !PAGED, "the paged layout is served by the fused step only");
  using Fmt = Dist<METRIC, D>;
  constexpr int kNumBins = Fmt::kBins;
  constexpr int BITS = Fmt::kBits, kRowBytes = Fmt::kRowBytes, W = Fmt::kWords;
  constexpr int kRowWords = W * BITS;  // 32-bit words per code row
  constexpr int kHistReplicas = hist_replicas(G, kNumBins);
  constexpr int E = HeadDim<D>::kEncElems;  // elements per lane when a wave encodes one vector
  constexpr int kPairs = Fmt::kPairs;  // 32-bit words of a histogram: two 16-bit bins each
  constexpr bool kWideBins = hist_wide_bins(G);
  constexpr int kHistWords = kWideBins ? 2 * kPairs : kPairs;  // LDS words of one histogram copy
  // [G][kHistReplicas][kHistWords], rounded up to whole 16-byte pieces
  constexpr int kHistTotal = (G * kHistReplicas * kHistWords + 3) & ~3;
  __shared__ __align__(16) uint32_t s_hist[kHistTotal];
  // per query head: plane p of word wd at [W * p + wd]; 2-bit codes also keep lo^hi at [2W + wd]
  __shared__ uint32_t s_q[G][3 * W];
  __shared__ uint32_t s_new[kRowWords];  // code row of the appended key, as stored
  __shared__ uint32_t s_ready;      // query / new-key code rows published so far
  // The heads of a group are served in passes, the planes of a pass's heads together or one after the other (see below).
  constexpr int QP = BITS == 2 ? 3 : BITS;
  constexpr bool kAllTogether = G * QP * W <= 24;
  constexpr int kPassHeads = kAllTogether ? G : (24 / (QP * W) > 0 ? 24 / (QP * W) : 1);
  constexpr int kScanRowWords = kScanTokPerThread * kRowWords, kHeadWords = QP * W + kScanRowWords;
  constexpr bool kScalarPlanes = !kAllTogether && (kHeadWords > 96 || (!FUSED && kHeadWords <= 68 && (BITS == 3 || kHeadWords >= 60)));
  constexpr int kTogether =
      kAllTogether ? G : kScalarPlanes || WAVES == 4 || kPassHeads * QP * W + kScanRowWords <= (BITS == 3 ? 44 : 48) ? kPassHeads : 1;
  // per wave: its 256 distances to each query head of a pass, in token order
  __shared__ __align__(16) uint16_t s_dt[WAVES][kPassHeads][kScanTokPerThread * kWave];

  // blockIdx.y = KV head << g_shift | part: the G query heads of this workgroup are
  // part `gsub` of the KV head's group of G << g_shift (the parts re-read the rows).
  PhaseTrace trace;
  trace.stamp(kScanStart);
  // requested first of all: the row loads cannot be addressed without them
  SeqInfo seq = SeqInfo::request<PAGED, true>(p.seq_len, p.seq_start, (int)blockIdx.z);
  __builtin_amdgcn_sched_barrier(0);
  const int tile_id = blockIdx.x, kvh = blockIdx.y >> p.g_shift, gsub = blockIdx.y & ((1 << p.g_shift) - 1);
  const int b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int nthreads = WAVES * kWave;
  constexpr int tile_tokens = nthreads * kScanTokPerThread;
  const int t0 = tile_id * tile_tokens;
  const int head0 = b * p.Hq + (int)blockIdx.y * G;

  // First of all the encoding waves request their vectors (G queries and, if
  // the call appends, the new key): their addresses need nothing from memory,
  // so these loads travel together with the scalar loads of the sequence
  // length and start below.  Only the encoding waves load: inside a compute
  // unit requests are served in order across waves, so a needless load here
  // would sit in front of other waves' rows.
  constexpr int kEncRounds = (G + 1 + WAVES - 1) / WAVES;  // G queries + 1 new key over the waves
  // 16 bits each until they are used, loaded one by one (wavefront-scope atomic loads, which are plain loads here): widened
  // or split on arrival (D = 64, 192), an encoding wave waited for them before it requested any row, and some of
  // them were requested behind the rows (D = 96, 160).
  uint16_t enc[kEncRounds][E];
#pragma unroll
  for (int r = 0; r < kEncRounds; ++r) {
    const int v = wave + r * WAVES;
#pragma unroll
    for (int e = 0; e < E; ++e) enc[r][e] = 0;
    if (FUSED && (v < G || (v == G && p.k_new != nullptr))) {
      const uint16_t* src = v < G ? p.q + (int64_t)(head0 + v) * D
                                  : p.k_new + ((int64_t)b * p.Hkv + kvh) * D;
#pragma unroll
      for (int e = 0; e < E; ++e)  // (lanes beyond the encoding ones read along; their values are not used)
        enc[r][e] = __hip_atomic_load(src + HeadDim<D>::enc_index(min(lane, HeadDim<D>::kEncLanes - 1), e),
                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
  }

  // Paged cache: the page of each of the wave's four 64-token steps (a step
  // never straddles a page: pages are multiples of 64 tokens).  Scalar loads,
  // on their way together with the length.
  int32_t pte[kScanTokPerThread];
  if constexpr (PAGED) {
    const int uw = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
    for (int i = 0; i < kScanTokPerThread; ++i) {
      const int pg = min((t0 + (uw * kScanTokPerThread + i) * kWave) >> p.page_shift, p.max_pages - 1);
      pte[i] = scalar_load(p.page_table + (int64_t)b * p.max_pages + pg);
    }
  }
  loads_issued_before_here();
  const int L = PAGED ? seq.paged_length(p.max_seq_len, (int64_t)p.max_pages << p.page_shift)
                      : seq.length(p.max_seq_len, p.pool_tokens);
  const int64_t start = seq.start;

  // The only workgroup barrier before the scan sits here, where every wave has
  // just started (and while the loads above are still on their way).  Later on
  // the waves must not wait for each other: a compute unit serves memory
  // requests in order, so late waves get their rows late, and a barrier after
  // the row loads would hold the early waves back with them.
  for (int i = tid; i < kHistTotal / 4; i += nthreads)
    reinterpret_cast<uint4*>(s_hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) s_ready = 0u;
  __syncthreads();

  // The select kernel counts its finished segments per head from zero (tile 0
  // exists for every sequence, empty ones included).
  if (p.arrivals != nullptr && tile_id == 0 && tid < G)
    p.arrivals[(int64_t)(head0 + tid) * p.arrivals_stride] = 0u;
  if (t0 >= L) return;  // whole workgroup
#ifdef ADAMAS_PHASE_TRACE   // (no wait here: the encode vectors are still on their way)
  if (threadIdx.x == 0) trace.t[kScanLengthKnown] = wall_clock64();
#endif

  // Order of the memory operations matters: loads return in issue order, so a
  // wave that waits for one load also waits for everything it issued before.
  // The code rows are requested next and consumed one token at a time as they
  // arrive; the encode runs while they travel.
  const bool appending = FUSED && p.k_new != nullptr && (L - 1) / tile_tokens == tile_id;
  const int n_enc = FUSED ? G + (appending ? 1 : 0) : 0;
  uint32_t qraw[BITS];  // not fused: thread (head, word) of wave 0 fetches its planes
#pragma unroll
  for (int pl = 0; pl < BITS; ++pl) qraw[pl] = 0;
  if (!FUSED && wave == 0) {
    const int i = min(tid, G * W - 1);
    const uint32_t* qc =
        reinterpret_cast<const uint32_t*>(p.qcodes + (int64_t)(head0 + i / W) * kRowBytes);
#pragma unroll
    for (int pl = 0; pl < BITS; ++pl) qraw[pl] = qc[BITS * (i % W) + pl];
  }

  const uint8_t* plane = p.codes + ((int64_t)kvh * p.pool_tokens + start) * kRowBytes;
  constexpr int kPiece = Fmt::kPiece, C = kRowBytes / kPiece;  // a row is fetched in C pieces
  uint32_t rr[kScanTokPerThread][kRowWords];
#pragma unroll
  for (int i = 0; i < kScanTokPerThread; ++i) {
    // Unconditional: a lane past the end re-reads the last row (masked at use).
    // A branch here would make the compiler wait for all loads at once.
    // A wave-uniform base and a 32-bit offset per lane (a sequence's rows span less than 2^27 bytes).
    const int t = min(t0 + (wave * kScanTokPerThread + i) * kWave + lane, L - 1);
    const uint8_t* base = plane;
    uint32_t in_base = (uint32_t)t;
    if constexpr (PAGED) {
      // a page number outside the pool is clamped into it; a lane past the end reads some row of the page
      const int64_t pg = min(max((int64_t)pte[i], (int64_t)0), (p.pool_tokens >> p.page_shift) - 1);
      base += (pg << p.page_shift) * kRowBytes;
      in_base = (uint32_t)t & ((1u << p.page_shift) - 1u);
    }
    const uint8_t* row = base + in_base * (uint32_t)kRowBytes;
#pragma unroll
    for (int c = 0; c < C; ++c) load_piece<kPiece>(row + c * kPiece, &rr[i][c * (kPiece / 4)]);
  }

  // Nothing above may be consumed before the row loads have been issued.
  if (FUSED) {
#pragma unroll
    for (int r = 0; r < kEncRounds; ++r) {
#pragma unroll
      for (int e = 0; e < E; ++e) asm volatile("" : "+v"(enc[r][e]));
    }
  } else {
#pragma unroll
    for (int pl = 0; pl < BITS; ++pl) asm volatile("" : "+v"(qraw[pl]));
  }

  if (FUSED) {
#pragma unroll
    for (int r = 0; r < kEncRounds; ++r) {
      const int v = __builtin_amdgcn_readfirstlane(wave) + r * WAVES;  // (scalar: see set_lane)
      if (v < n_enc) {
        uint32_t w[BITS][W];
        uint32_t raw[E];
#pragma unroll
        for (int e = 0; e < E; ++e) raw[e] = enc[r][e];
        encode_values_wave<BITS, D>(raw, v < G ? p.thr_q : p.thr_k, w);
        if (v < G) publish_query<BITS, W>(w, s_q[v], lane);
        else publish_row<BITS, W>(w, s_new, lane);
        if (lane == 0)
          __hip_atomic_fetch_add(&s_ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  } else if (wave == 0) {
    if (tid < G * W) {
      const int g = tid / W, wd = tid % W;
#pragma unroll
      for (int pl = 0; pl < BITS; ++pl) s_q[g][W * pl + wd] = qraw[pl];
      if (BITS == 2) s_q[g][2 * W + wd] = qraw[0] ^ qraw[BITS - 1];
    }
    if (lane == 0)
      __hip_atomic_fetch_add(&s_ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // Wait for the publishing waves only.  They never wait for anybody, so this
  // ends; the spin bound is a last resort that turns a logic error into wrong
  // distances instead of a hung GPU.
  {
    const uint32_t n_ready = FUSED ? (uint32_t)n_enc : 1u;
    for (int spin = 0; spin < (1 << 22); ++spin) {
      if (__hip_atomic_load(&s_ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= n_ready)
        break;
      __builtin_amdgcn_s_sleep(2);
    }
  }

  trace.stamp(kScanQueryReady);
  // The query planes are wave-uniform, but live in vector registers: an instruction with a scalar operand takes twice the issue
  // time of one without as soon as a SIMD has a second wave (exclusive or, and, three-input logic: 4.2 and 2.4 clocks), and with 24
  // words of planes in scalar registers a wave takes more than 80, of which a compute unit holds 28 waves instead of
  // 32, one workgroup of sixteen instead of two (16 ragged sequences 41.5 -> 45.4 us a layer).  Up to 24 words
  // (the method's group of one or two) at once; larger groups the heads of a pass at once where their planes and the rows leave a wave
  // within 64 registers, else one head after the other over the rows, which stay in registers.  (d = 96, groups of four: one by one
  // 27.4 us for 24 ragged sequences of 24000 tokens, two by two 25.8; d = 64, groups of eight 26.9 and 25.1.)
  // Workgroups of four waves are those of calls that leave compute units idle, where registers to spare cost nothing and a wait for the
  // planes of every head does: all heads of a pass at once (distances of 38 ragged sequences of 841 tokens, one bit, d = 256, groups of
  // eight 7.4 us one by one, 6.8; of 19 of 872, squared differences at d = 128, groups of six 7.4 and 6.7).
  // Scalar registers hold them where they do not fit next to the rows, or cost a workgroup: three-bit codes at d = 256 (24 ragged
  // sequences of 10540 tokens, groups of six 33.9 us a layer, 44.1 in vector registers), and without the encode, which takes most, three-bit codes up to
  // d = 128 and two-bit ones at 192 (top-k of 8 sequences of 24000 tokens, three bits at d = 128, groups of three 31.8 us in vector
  // registers, 30.5; d = 192, groups of two 27.0 and 26.3).
  // qp[g][j][wd]: plane j of word wd; for 2-bit codes j = 2 is lo ^ hi.
  uint32_t* hist_lane = s_hist + (lane & (kHistReplicas - 1)) * kHistWords;
  auto distance = [](const uint32_t (&row)[kRowWords], auto q) { return row_distance<METRIC, D>(row, q); };

  uint32_t one = 1;  // (opaque: otherwise written anew for every use)
  asm("" : "+v"(one));
  // Three-bit codes from d = 160 on spill in workgroups of sixteen waves: the tokens' numbers are made again at their use, not kept (d = 160,
  // groups of three, 24 ragged sequences of 24000 tokens: 85.7 -> 81.4 us; of six 123.2 -> 115.4).  So are those of the one-bit instance
  // that would spill a register otherwise (kScanWavesPerSimd).
  int of_wave = lane;
  if constexpr (WAVES == 16 && (FUSED ? BITS == 3 && D >= 160 : BITS == 1 && D == 192 && G == 8)) asm("" : "+v"(of_wave));
#pragma unroll
  for (int g0 = 0; g0 < G; g0 += kPassHeads) {
#pragma unroll
    for (int g1 = g0; g1 < g0 + kPassHeads && g1 < G; g1 += kTogether) {
      uint32_t qp[kTogether][QP][W];
#pragma unroll
      for (int g = 0; g < kTogether && g1 + g < G; ++g) {
#pragma unroll
        for (int j = 0; j < QP; ++j) {
#pragma unroll
          for (int wd = 0; wd < W; ++wd) {
            qp[g][j][wd] = s_q[g1 + g][W * j + wd];
            if constexpr (kScalarPlanes) qp[g][j][wd] = __builtin_amdgcn_readfirstlane(qp[g][j][wd]);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < kScanTokPerThread; ++i) {
        // keep the tokens in load order, so that each waits only for its own rows
        if (g1 == 0) __builtin_amdgcn_sched_barrier(0);
        const int t = t0 + (wave * kScanTokPerThread + i) * kWave + of_wave;
        // The appended token's row is not in memory yet.  It takes the place of the loaded one once, before
        // the first head (a copy of the row for every pass costs 64 moves per wave with a group of four).
        if (g1 == 0 && appending) {
          if (t == L - 1) {
#pragma unroll
            for (int wq = 0; wq < kRowWords; ++wq) rr[i][wq] = s_new[wq];
          }
        }
        // Groups whose query planes fit the registers together (up to two heads at d = 96 and 128, four at 64, one from 160 on; three
        // times as many with one-bit codes) mask their atomics alone (0.1 us of 12.9 for 32 planes of 9235 ragged tokens),
        // others the whole step.
        constexpr bool kMaskEach = kTogether == G;
        if (kMaskEach || t < L) {
#pragma unroll
          for (int g = 0; g < kTogether && g1 + g < G; ++g) {
            const uint32_t d = distance(rr[i], [&](int j, int wd) { return qp[g][j][wd]; });
            s_dt[wave][g1 + g - g0][i * kWave + lane] = (uint16_t)d;
            if constexpr (kWideBins) {
              if (!kMaskEach || t < L) atomicAdd(hist_lane + (g1 + g) * (kHistReplicas * kHistWords) + d, one);
            } else {
              // two 16-bit bins per word: 1 for an even distance, 0x10000 for an odd one
              // (opaque halves: otherwise the compiler turns them into a compare and a select)
              uint32_t pair = d >> 1, odd16 = (d & 1u) << 4;
              asm("" : "+v"(pair), "+v"(odd16));
              if (!kMaskEach || t < L) atomicAdd(hist_lane + (g1 + g) * (kHistReplicas * kHistWords) + pair, 1u << odd16);
            }
          }
        }
      }
    }
    if (g0 + kPassHeads >= G) trace.stamp(kScanRowsDone);
    // The distances of the pass leave through LDS: a lane computed tokens 64 apart, but stores eight consecutive ones.
    // Byte planes: the low bytes of its eight are picked with two byte permutes, the ninth bits with two permutes and two dot
    // products (weights 1, 2, 4 ... 128).  For 64 tokens of a head that is less than one instruction; a ballot and
    // two lane writes per 64 tokens took three of 27.  (Words of ninth bits computed only where a distance above 255 occurs,
    // by a second walk over the rows: 51.8 instead of 44.3 us a layer for 16 ragged sequences; such distances are common
    // where a few channels of the keys are large.)  With the copies of the rows, the masks and the flush below
    // this loop went from about 30 to 23 vector instructions per 64 tokens and head: 16.1 -> 15.3 us a layer for one sequence
    // of 32771 tokens and G = 4, 34.9 -> 33.9 for four of 60001 and G = 8, 45.4 -> 44.3 for 16 ragged ones and G = 4.
    // The region is private to the wave, so no barrier is needed.  A row of the planes holds a multiple of
    // 128 tokens, so a lane whose first token exists may store all eight.
    constexpr int kLanes = kScanTokPerThread * kWave / 8;  // lanes per head
#pragma unroll
    for (int c = 0; c < (kPassHeads * kLanes + kWave - 1) / kWave; ++c) {
      const int at = c * kWave + lane, g = kPassHeads == 1 ? g0 : g0 + at / kLanes;
      const int tt = t0 + wave * (kScanTokPerThread * kWave) + 8 * (at % kLanes);
      if (p.dist != nullptr && at < kPassHeads * kLanes && g < G && tt < L) {
        uint32_t v[4];
        __builtin_memcpy(v, __builtin_assume_aligned(&s_dt[wave][0][0] + 8 * at, 16), 16);
        const int64_t to = (int64_t)(head0 + g) * p.dist_stride + tt;
        if constexpr (Fmt::kByteDist) {
          uint2 low;
          low.x = __builtin_amdgcn_perm(v[1], v[0], 0x06040200u);
          low.y = __builtin_amdgcn_perm(v[3], v[2], 0x06040200u);
          *reinterpret_cast<uint2*>(static_cast<uint8_t*>(p.dist) + to) = low;
        } else {
          *reinterpret_cast<uint4*>(static_cast<uint16_t*>(p.dist) + to) = make_uint4(v[0], v[1], v[2], v[3]);
        }
        if constexpr (Fmt::kHighPlane) {
          uint32_t high = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(v[1], v[0], 0x07050301u), 0x08040201u, 0u, false);
          high = __builtin_amdgcn_udot4(__builtin_amdgcn_perm(v[3], v[2], 0x07050301u), 0x80402010u, high, false);
          reinterpret_cast<uint8_t*>(p.dist_high)[to >> 3] = (uint8_t)high;
        }
      }
    }
    if (p.dist_user != nullptr) {  // the caller's own array of distances
#pragma unroll 1
      for (int g = g0; g < g0 + kPassHeads && g < G; ++g) {
#pragma unroll
        for (int i = 0; i < kScanTokPerThread; ++i) {
          const int t = t0 + (wave * kScanTokPerThread + i) * kWave + lane;
          if (t < L) p.dist_user[(int64_t)(head0 + g) * p.dist_user_stride + t] = s_dt[wave][g - g0][i * kWave + lane];
        }
      }
    }
  }  // passes over the heads of the group

  trace.stamp(kScanDistStored);
  // Algorithm 1, cache update: the new token's K, V and code row enter the cache.  The
  // scan above already used the new code row (from LDS); the stores come last
  // so that no other memory operation sits between the row loads and their use.
  if (appending && wave == 0 && gsub == 0) {
    const int64_t src = ((int64_t)b * p.Hkv + kvh) * D;
    int64_t row = (int64_t)kvh * p.pool_tokens + start + (L - 1);
    if constexpr (PAGED) {
      const int64_t pg = min(max((int64_t)p.page_table[(int64_t)b * p.max_pages + ((L - 1) >> p.page_shift)],
                                 (int64_t)0), (p.pool_tokens >> p.page_shift) - 1);
      row = (int64_t)kvh * p.pool_tokens + (pg << p.page_shift) + ((L - 1) & ((1 << p.page_shift) - 1));
    }
    if (lane < kRowWords) reinterpret_cast<uint32_t*>(p.codes_w + row * kRowBytes)[lane] = s_new[lane];
#pragma unroll
    for (int c = lane; c < D / 2; c += kWave) {  // D bf16 values = D / 2 dwords per row
      reinterpret_cast<uint32_t*>(p.K + row * D)[c] = reinterpret_cast<const uint32_t*>(p.k_new + src)[c];
      reinterpret_cast<uint32_t*>(p.V + row * D)[c] = reinterpret_cast<const uint32_t*>(p.v_new + src)[c];
    }
  }
  if (p.tilehist != nullptr) {
    __syncthreads();
    // 64 words of one head at a time, so that everything but the lane is the same for a wave
    constexpr int kRows = (kPairs + kWave - 1) / kWave;
    for (int u = __builtin_amdgcn_readfirstlane(wave); u < G * kRows; u += WAVES) {
      const int g = u / kRows, pr = u % kRows * kWave + lane;
      if (pr < kPairs) {
        const uint32_t* h = s_hist + g * (kHistReplicas * kHistWords);
        uint32_t v = 0;
#pragma unroll
        for (int r = 0; r < kHistReplicas; ++r) {
          // (a last odd bin that no distance reaches stays zero)
          if constexpr (kWideBins) v += h[r * kHistWords + 2 * pr] + (h[r * kHistWords + 2 * pr + 1] << 16);
          else v += h[r * kHistWords + pr];
        }
        p.tilehist[((int64_t)(head0 + g) * p.n_tiles + tile_id) * kPairs + pr] = v;
      }
    }
  }
  trace.stamp(kScanEnd);
  trace.flush(p.trace, p.trace_records);
}

}  // namespace adamas
