// The decode step (or top-k on query codes) of one query head in one workgroup, one launch: for contexts that a
// compute unit scans by itself in less time than handing distances and histograms to a second kernel takes.
//
// The steps of Algorithm 1 are those of scan_kernel and select_kernel, with the same results: encode, distances (Eq. 6), the
// threshold distance from the histogram, positions in ascending order with ties to the lowest, attention over the rows.
// What differs is that distances and histogram never leave LDS, no workgroup waits for or hands anything to
// another, and nothing is merged: no scratch memory, no kernel boundary, no round trip for what the scan left.
// The price: every query head of a group reads the code rows by itself (they come from the XCD's L2: the heads
// of a KV head sit 8 workgroups apart, which is the same XCD), and a head has one compute unit's rate.
#pragma once

#include "scan.hpp"
#include "select_attn.hpp"

namespace adamas {

struct OneLaunchParams {
  const uint8_t* codes;      // [Hkv][pool][row bytes]; the appended rows are written to it (FUSED)
  uint8_t* codes_w;
  const uint16_t* q;         // bf16 [B][Hq][D]       (FUSED)
  const uint8_t* qcodes;     // [B][Hq][row bytes]    (not FUSED)
  const uint16_t* k_new;     // bf16 [B][Hkv][D] or null
  const uint16_t* v_new;
  uint16_t* K;               // pools
  uint16_t* V;
  const int64_t* seq_start;  // [B]
  const int32_t* seq_len;    // [B]
  uint16_t* dist_user;       // optional, [B*Hq][max_seq_len] (not FUSED)
  int32_t* idx_out;          // [B*Hq][k] or null
  float* out;                // [B*Hq][D] (FUSED)
  int64_t pool_tokens, max_seq_len;
  int32_t Hq, Hkv, k, group;
  int32_t planes;            // B * Hkv
  uint32_t kv_magic;         // magic_of(Hkv): plane -> sequence
  int32_t list;              // words of the list of positions in LDS (one_launch_list)
  const int32_t* page_table; // PAGED
  int32_t max_pages, page_shift;
  Thresholds thr_q, thr_k;
  double scale_log2e;
};

// Sums over the waves before this one, and over all, of one packed count each.  All lanes active.
template <int WAVES>
__device__ __forceinline__ uint2 waves_before(const uint32_t* s_counts, int wave) {
  static_assert(WAVES <= 16, "one row of lanes");
  const int lane = threadIdx.x & 63;
  uint32_t v = lane < WAVES ? s_counts[lane] : 0u;
  v += dpp_u32<kDppRowShr + 1>(v);
  v += dpp_u32<kDppRowShr + 2>(v);
  v += dpp_u32<kDppRowShr + 4>(v);
  v += dpp_u32<kDppRowShr + 8>(v);
  const uint32_t before = wave == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)v, wave - 1);
  return make_uint2(before, (uint32_t)__builtin_amdgcn_readlane((int)v, WAVES - 1));
}

// One load of BYTES (16, 8 or 4) through a buffer descriptor.
template <int BYTES, typename R>
__device__ __forceinline__ void load_piece_buffer(R rsrc, uint32_t offset, uint32_t* w) {
  if constexpr (BYTES == 16) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, offset, 0, 0);
    w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
  } else if constexpr (BYTES == 8) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, offset, 0, 0);
    w[0] = v[0]; w[1] = v[1];
  } else {
    w[0] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, offset, 0, 0);
  }
}

// Grid (8 * group, planes / 8 rounded up): blockIdx.x = 8 * head of the group + plane % 8.
template <int WAVES, bool FUSED, int METRIC, bool PAGED, int D>
__global__ __launch_bounds__(WAVES * kWave) void one_launch_kernel(const OneLaunchParams p) {
  static_assert(FUSED || !PAGED, "only the step has the paged layout");
  static_assert(WAVES * kWave >= D, "one thread per output dimension");
  using Fmt = Dist<METRIC, D>;
  constexpr int THREADS = WAVES * kWave;
  constexpr int BITS = Fmt::kBits, kRowBytes = Fmt::kRowBytes, W = Fmt::kWords, kRowWords = W * BITS;
  constexpr int kBins = Fmt::kBins, E = HeadDim<D>::kEncElems;
  constexpr int QP = BITS == 2 ? 3 : BITS;
  constexpr int kReplicas = 2;  // of the histogram, picked by lane
  constexpr int kHistBins = kBins + 1;  // the last one takes the lanes past the end
  constexpr int kHistWords = (kReplicas * kHistBins + 3) & ~3;
  // Code rows in flight per lane.  Two of the longer ones: three-bit codes at d = 128 32.4 -> 31.3 us for 40 ragged sequences of 3000
  // tokens, d = 256 33.8 -> 32.9 for 24, and with three-bit codes there four rows spill registers (87 us instead of 30 for 8 x 6000).
  constexpr int U = kRowWords >= 12 ? 2 : 4;
  __shared__ __align__(16) uint32_t s_hist[kHistWords];
  __shared__ uint32_t s_q[3 * W];
  __shared__ uint32_t s_new[kRowWords];
  __shared__ uint32_t s_ready;
  __shared__ uint32_t s_wave[WAVES];
  __shared__ uint32_t s_pass[2][WAVES];
  __shared__ int32_t s_found[2];
  extern __shared__ __align__(16) unsigned char s_dynamic[];
  int32_t* s_sel = reinterpret_cast<int32_t*>(s_dynamic);     // rows to gather, in the order of positions
  int32_t* s_pos = s_sel + (PAGED ? p.list : 0);         // positions
  uint16_t* s_dist = reinterpret_cast<uint16_t*>(s_pos + p.list);

  const int plane = (int)blockIdx.y * 8 + ((int)blockIdx.x & 7), g = (int)blockIdx.x >> 3;
  if (plane >= p.planes) return;
  // (the multiplication is a vector instruction)
  const int b = __builtin_amdgcn_readfirstlane(kv_head_of(plane, p.kv_magic)), kvh = plane - b * p.Hkv;
  SeqInfo seq = SeqInfo::request<PAGED, true>(p.seq_len, p.seq_start, b);
  __builtin_amdgcn_sched_barrier(0);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t head = (int64_t)b * p.Hq + kvh * p.group + g;

  // The query (wave 0) and the new key (wave 1), requested while the length travels.
  uint16_t enc[E];
#pragma unroll
  for (int e = 0; e < E; ++e) enc[e] = 0;
  if (FUSED && (wave == 0 || (wave == 1 && p.k_new != nullptr))) {
    const uint16_t* src = wave == 0 ? p.q + head * D : p.k_new + ((int64_t)b * p.Hkv + kvh) * D;
#pragma unroll
    for (int e = 0; e < E; ++e)
      enc[e] = __hip_atomic_load(src + HeadDim<D>::enc_index(min(lane, HeadDim<D>::kEncLanes - 1), e),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
  // and its row, to be stored into the cache
  constexpr int kNewWords = (D / 2 + kWave - 1) / kWave;
  uint32_t new_k[kNewWords], new_v[kNewWords];
#pragma unroll
  for (int c = 0; c < kNewWords; ++c) new_k[c] = new_v[c] = 0u;
  if (FUSED && wave == 1 && p.k_new != nullptr) {
    const int64_t src = ((int64_t)b * p.Hkv + kvh) * D;
#pragma unroll
    for (int c = 0; c < kNewWords; ++c) {
      const int at = min(c * kWave + lane, D / 2 - 1);
      new_k[c] = reinterpret_cast<const uint32_t*>(p.k_new + src)[at];
      new_v[c] = reinterpret_cast<const uint32_t*>(p.v_new + src)[at];
    }
  }
  uint32_t qraw[BITS];
#pragma unroll
  for (int pl = 0; pl < BITS; ++pl) qraw[pl] = 0;
  if (!FUSED && wave == 0) {
    const uint32_t* qc = reinterpret_cast<const uint32_t*>(p.qcodes + head * kRowBytes);
    const int i = min(lane, W - 1);
#pragma unroll
    for (int pl = 0; pl < BITS; ++pl) qraw[pl] = qc[BITS * i + pl];
  }
  uint4 qv = make_uint4(0, 0, 0, 0);
  if constexpr (FUSED) qv = load_query_piece<D>(p.q + head * D);

  // 64 tokens a step; wave w takes steps w, w + WAVES, ...
  const int32_t* pages = PAGED ? p.page_table + (int64_t)b * p.max_pages : nullptr;
  auto page_of = [&](int step) { return scalar_load(pages + min((step * kWave) >> p.page_shift, p.max_pages - 1)); };
  int32_t pte[U];
#pragma unroll
  for (int i = 0; i < U; ++i) pte[i] = PAGED ? page_of(wave + i * WAVES) : 0;
  loads_issued_before_here();
  const int L = PAGED ? seq.paged_length(p.max_seq_len, (int64_t)p.max_pages << p.page_shift)
                      : seq.length(p.max_seq_len, p.pool_tokens);
  const int64_t start = seq.start;
  const int kk = min(p.k, L);
  int32_t* idx_row = p.idx_out != nullptr ? p.idx_out + head * p.k : nullptr;

  for (int i = tid; i < kHistWords / 4; i += THREADS) reinterpret_cast<uint4*>(s_hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) s_ready = 0u;
  __syncthreads();
  if (L == 0) {
    if (FUSED && tid < D) p.out[head * D + tid] = 0.f;
    if (idx_row != nullptr)
      for (int i = tid; i < p.k; i += THREADS) idx_row[i] = -1;
    return;
  }

  const uint8_t* rows = p.codes + ((int64_t)kvh * p.pool_tokens + start) * kRowBytes;
  constexpr int kPiece = Fmt::kPiece, C = kRowBytes / kPiece;
  const int64_t last_page = PAGED ? (p.pool_tokens >> p.page_shift) - 1 : 0;
  // Buffer loads: everything but the lane's constant offset is scalar, and lanes past the end read zeros and touch no memory.
  const uint32_t lane_bytes = lane * kRowBytes;
  auto request = [&](int step, int32_t page, uint32_t (&r)[kRowWords]) {
    const int t = step * kWave;
    int64_t row = t;
    if constexpr (PAGED) {
      const int64_t pg = min(max((int64_t)page, (int64_t)0), last_page);
      row = (pg << p.page_shift) + (t & ((1 << p.page_shift) - 1));
    }
    // (said to be uniform: a descriptor that the compiler keeps in vector registers makes a loop of every load)
    const uint64_t at = (uint64_t)(rows + row * kRowBytes);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)at), hi = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));
    int left = max(L - t, 0);
    asm("" : "+s"(left));  // (otherwise the two limits become one vector instruction)
    const int bytes = min(left, kWave) * kRowBytes;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)hi << 32 | lo), (short)0, bytes, 0x00020000);
#pragma unroll
    for (int c = 0; c < C; ++c) load_piece_buffer<kPiece>(rsrc, lane_bytes + c * kPiece, &r[c * (kPiece / 4)]);
  };
  const int n_steps = (L + kWave - 1) / kWave;
  uint32_t rr[U][kRowWords];
#pragma unroll
  for (int i = 0; i < U; ++i) request(wave + i * WAVES, pte[i], rr[i]);

  // Nothing above may be consumed before the rows have been requested.
#pragma unroll
  for (int e = 0; e < E; ++e) asm volatile("" : "+v"(enc[e]));
#pragma unroll
  for (int pl = 0; pl < BITS; ++pl) asm volatile("" : "+v"(qraw[pl]));
#pragma unroll
  for (int c = 0; c < kNewWords; ++c) asm volatile("" : "+v"(new_k[c]), "+v"(new_v[c]));

  const bool appending = FUSED && p.k_new != nullptr;
  const int n_enc = appending ? 2 : 1;
  if (FUSED ? wave < n_enc : wave == 0) {
    uint32_t w[BITS][W];
    if constexpr (FUSED) {
      uint32_t raw[E];
#pragma unroll
      for (int e = 0; e < E; ++e) raw[e] = enc[e];
      encode_values_wave<BITS, D>(raw, wave == 0 ? p.thr_q : p.thr_k, w);
    } else {
#pragma unroll
      for (int pl = 0; pl < BITS; ++pl) w[pl][0] = qraw[pl];  // lane wd holds word wd
    }
    if constexpr (FUSED) {
      if (wave == 0) publish_query<BITS, W>(w, s_q, lane);
      else publish_row<BITS, W>(w, s_new, lane);
    } else {
#pragma unroll
      for (int pl = 0; pl < BITS; ++pl) {
        if (lane < W) s_q[W * pl + lane] = w[pl][0];
      }
      if (BITS == 2 && lane < W) s_q[2 * W + lane] = w[0][0] ^ w[BITS - 1][0];
    }
    if (lane == 0) __hip_atomic_fetch_add(&s_ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // (the publishing waves wait for nobody; the bound turns a logic error into wrong distances, not a hang)
  for (int spin = 0; spin < (1 << 22); ++spin) {
    if (__hip_atomic_load(&s_ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= (uint32_t)n_enc) break;
    __builtin_amdgcn_s_sleep(2);
  }

  // Algorithm 1, cache update.  Every head of the group writes the same bytes of K, V and code row: a workgroup then reads back
  // what it wrote itself, whichever XCD the others run on, and needs to wait for none of them.
  if (appending && wave == 1) {
    int64_t row = (int64_t)kvh * p.pool_tokens + start + (L - 1);
    if constexpr (PAGED) {
      const int64_t pg = min(max((int64_t)page_of((L - 1) / kWave), (int64_t)0), last_page);
      row = (int64_t)kvh * p.pool_tokens + (pg << p.page_shift) + ((L - 1) & ((1 << p.page_shift) - 1));
    }
    if (lane < kRowWords) reinterpret_cast<uint32_t*>(p.codes_w + row * kRowBytes)[lane] = s_new[lane];
#pragma unroll
    for (int c = 0; c < kNewWords; ++c) {
      const int at = c * kWave + lane;
      if (at < D / 2) {
        reinterpret_cast<uint32_t*>(p.K + row * D)[at] = new_k[c];
        reinterpret_cast<uint32_t*>(p.V + row * D)[at] = new_v[c];
      }
    }
  }

  uint32_t qp[QP][W];
#pragma unroll
  for (int j = 0; j < QP; ++j) {
#pragma unroll
    for (int wd = 0; wd < W; ++wd) qp[j][wd] = s_q[W * j + wd];
  }
  uint32_t* hist_lane = s_hist + (lane & (kReplicas - 1)) * kHistBins;
  uint16_t* dist_lane = s_dist + lane;
  uint32_t one = 1;
  asm("" : "+v"(one));
  uint32_t new_row[kRowWords];
  auto consume = [&](int step, uint32_t (&r)[kRowWords], auto last_) {
    const int t = step * kWave + lane;
    if constexpr (decltype(last_)::value) {
      if (step >= n_steps) return;
      if (appending && step == n_steps - 1) {  // the appended token's row is not read from memory
#pragma unroll
        for (int wq = 0; wq < kRowWords; ++wq) r[wq] = t == L - 1 ? new_row[wq] : r[wq];
      }
    }
    uint32_t d = row_distance<METRIC, D>(r, [&](int j, int wd) { return qp[j][wd]; });
    if constexpr (decltype(last_)::value) d = t < L ? d : (uint32_t)kBins;
    dist_lane[step * kWave] = (uint16_t)d;
    atomicAdd(hist_lane + d, one);
    if constexpr (!FUSED) {
      if (p.dist_user != nullptr && t < L) p.dist_user[head * p.max_seq_len + t] = (uint16_t)d;
    }
  };
  // Only the last batch of a wave has steps with lanes, or all of it, past the end.
  int s0 = wave;
  for (; s0 + U * WAVES < n_steps; s0 += U * WAVES) {
    if constexpr (PAGED) {
#pragma unroll
      for (int i = 0; i < U; ++i) pte[i] = page_of(s0 + (U + i) * WAVES);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      __builtin_amdgcn_sched_barrier(0);  // in the order of the requests
      consume(s0 + i * WAVES, rr[i], std::false_type{});
      request(s0 + (U + i) * WAVES, pte[i], rr[i]);
    }
  }
  // (read here: at its use the wait would be for the histogram's additions as well; nothing was written there without an append)
#pragma unroll
  for (int wq = 0; wq < kRowWords; ++wq) new_row[wq] = s_new[wq];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    __builtin_amdgcn_sched_barrier(0);
    consume(s0 + i * WAVES, rr[i], std::true_type{});
  }
  __syncthreads();

  // Sixteen tokens a thread, fewer for short contexts: every wave has some.  They share a page.
  const int quads = L <= 4 * THREADS ? 1 : L <= 8 * THREADS ? 2 : 4, per_thread = 4 * quads, pass = THREADS * per_thread;
  int32_t page = 0;
  if constexpr (PAGED) page = pages[min((tid * per_thread) >> p.page_shift, p.max_pages - 1)];

  // Threshold distance T: the bin in which the cumulative count reaches kk; #{D < T}.
  constexpr int PB = (kBins + THREADS - 1) / THREADS;                 // consecutive bins of a thread
  constexpr int kBinWaves = ((kBins + PB - 1) / PB + kWave - 1) / kWave;
  uint32_t bin[PB], sum = 0;
#pragma unroll
  for (int j = 0; j < PB; ++j) {
    const int at = tid * PB + j;
    bin[j] = 0;
    if (at < kBins) {
#pragma unroll
      for (int r = 0; r < kReplicas; ++r) bin[j] += s_hist[r * kHistBins + at];
    }
    sum += bin[j];
  }
  const uint32_t incl = wave_incl_scan_u32(sum);
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  if (wave < kBinWaves) {
    uint32_t run = incl - sum + waves_before<kBinWaves>(s_wave, wave).x;
    if (run < (uint32_t)kk && run + sum >= (uint32_t)kk) {
#pragma unroll
      for (int j = 0; j < PB; ++j) {
        if (run < (uint32_t)kk && run + bin[j] >= (uint32_t)kk) {
          s_found[0] = tid * PB + j;
          s_found[1] = (int32_t)run;
        }
        run += bin[j];
      }
    }
  }
  __syncthreads();
  const uint32_t T = (uint32_t)s_found[0], r_eq = (uint32_t)(kk - s_found[1]);
  const uint32_t y_lt = T * 0x00010001u, y_le = y_lt + 0x00010001u;

  // Positions, in ascending order: a thread's candidates come after those of the threads before it, ties as long as there are some
  // to take.
  uint32_t run_lt = 0, run_eq = 0;
#pragma unroll 1
  for (int t0 = 0, n = 0; t0 < L; t0 += pass, ++n) {
    const int t = t0 + tid * per_thread;
    uint32_t lt16 = 0, eq16 = 0;
    if (t < L) {
      auto flags = [&](auto quads_) {
        constexpr int Q = decltype(quads_)::value;
        uint32_t dw[2 * Q], lt = 0, le = 0;
#pragma unroll
        for (int i = 0; i < (Q + 1) / 2; ++i)
          load_piece<(Q == 1 ? 8 : 16)>(reinterpret_cast<const uint8_t*>(s_dist + t + 8 * i), &dw[4 * i]);
        // bits 15 and 31 of a difference: tokens 2 w and 2 w + 1, below T or not above it
#pragma unroll
        for (int w = 0; w < 2 * Q; ++w) {
          lt = (lt >> 2) | (pk_sub_u16(dw[w], y_lt) & 0x80008000u);
          le = (le >> 2) | (pk_sub_u16(dw[w], y_le) & 0x80008000u);
        }
        lt16 = (((lt & 0xffffu) >> 1) | (lt >> 16)) >> (16 - 4 * Q);
        eq16 = ((((le & 0xffffu) >> 1) | (le >> 16)) >> (16 - 4 * Q)) & ~lt16;
      };
      if (quads == 1) flags(std::integral_constant<int, 1>{});
      else if (quads == 2) flags(std::integral_constant<int, 2>{});
      else flags(std::integral_constant<int, 4>{});
    }
    const uint32_t cnt = (uint32_t)__popc(lt16) | ((uint32_t)__popc(eq16) << 16), in_wave = wave_incl_scan_u32(cnt);
    if (lane == 63) s_pass[n & 1][wave] = in_wave;
    __syncthreads();
    const uint2 waves = waves_before<WAVES>(s_pass[n & 1], wave);
    const uint32_t ex = waves.x + in_wave - cnt;
    const uint32_t eq = run_eq + (ex >> 16);
    uint32_t pos = run_lt + (ex & 0xffffu) + min(eq, r_eq);
    run_lt += waves.y & 0xffffu;
    run_eq += waves.y >> 16;
    int32_t row = t;
    if constexpr (PAGED) {
      row = (int32_t)((min(max((int64_t)page, (int64_t)0), last_page) << p.page_shift) + (t & ((1 << p.page_shift) - 1)));
      page = pages[min((t + pass) >> p.page_shift, p.max_pages - 1)];
    }
    // the thread's last ties may not be taken
    const uint32_t ties = r_eq - min(eq, r_eq);
    while ((uint32_t)__popc(eq16) > ties) eq16 &= ~(0x80000000u >> __builtin_clz(eq16));
    uint32_t take = lt16 | eq16;
    while (take != 0u) {
      const int j = __builtin_ctz(take);
      take &= take - 1u;
      s_pos[pos] = t + j;
      if constexpr (PAGED) s_sel[pos] = row + j;
      ++pos;
    }
  }
  __syncthreads();
  // (before the gather, which waits for it: while the rows travel, or at the end, cost 0.1 us of 6.5)
  if (idx_row != nullptr)
    for (int i = tid; i < p.k; i += THREADS) idx_row[i] = i < kk ? s_pos[i] : -1;
  if constexpr (FUSED) {
    const int64_t row0 = ((int64_t)kvh * p.pool_tokens + start) * D;
    float M, lsum, o;
    PhaseTrace trace;
    attention_rows<THREADS, D>(s_sel, kk, PAGED ? (int)p.pool_tokens : L, qv, p.K + row0, p.V + row0, p.scale_log2e,
                               *reinterpret_cast<AttnShared<THREADS, D>*>(s_dist), M, lsum, o, trace, [] {});
    if (tid < D) p.out[head * D + tid] = lsum > 0.f ? o / lsum : 0.f;
  }
}

}  // namespace adamas
