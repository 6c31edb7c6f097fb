// Instantiates every kernel of ONE (head dimension, metric) pair and exports
// their launchers as a KernelSet.  Compiled once per pair with
//   -DADAMAS_INST_D=<64|96|128|160|192|256> -DADAMAS_INST_METRIC=<0..3>
// (see kernel_set.hpp and build.py).
#include "kernel_set.hpp"

#if !defined(ADAMAS_INST_D) || !defined(ADAMAS_INST_METRIC)
#error "compile with -DADAMAS_INST_D=... -DADAMAS_INST_METRIC=..."
#endif

namespace adamas {
namespace {

constexpr int D = ADAMAS_INST_D;
constexpr int METRIC = ADAMAS_INST_METRIC;
constexpr int BITS = Dist<METRIC, D>::kBits;
constexpr int kSelThreads = 256;

template <int G, bool FUSED, bool PAGED>
bool launch_scan_tile(int tile_tokens, dim3 grid, hipStream_t st, const ScanParams& sp) {
  switch (tile_tokens) {
    case 1024:  // (choose_cut: not for the step)
      if constexpr (FUSED) {
        return false;
      } else {
        hipLaunchKernelGGL((scan_kernel<G, false, 4, METRIC, PAGED, D>), grid, dim3(256), 0, st, sp);
        return true;
      }
    case 2048: hipLaunchKernelGGL((scan_kernel<G, FUSED, 8, METRIC, PAGED, D>), grid, dim3(512), 0, st, sp); return true;
    case 4096: hipLaunchKernelGGL((scan_kernel<G, FUSED, 16, METRIC, PAGED, D>), grid, dim3(1024), 0, st, sp); return true;
    default: return false;
  }
}

template <int G>
bool launch_scan_g(bool fused, int tile_tokens, dim3 grid, hipStream_t st, const ScanParams& sp) {
  if (!fused) return launch_scan_tile<G, false, false>(tile_tokens, grid, st, sp);
  if (sp.page_table != nullptr) return launch_scan_tile<G, true, true>(tile_tokens, grid, st, sp);
  return launch_scan_tile<G, true, false>(tile_tokens, grid, st, sp);
}

// (a kernel of more heads than the caller's grid is cut for would read and write heads beyond the tensors)
bool launch_scan(bool fused, int G, int tile_tokens, dim3 grid, hipStream_t st, const ScanParams& sp) {
  switch (G) {
    case 1: return launch_scan_g<1>(fused, tile_tokens, grid, st, sp);
    case 2: return launch_scan_g<2>(fused, tile_tokens, grid, st, sp);
    case 3: return launch_scan_g<3>(fused, tile_tokens, grid, st, sp);
    case 4: return launch_scan_g<4>(fused, tile_tokens, grid, st, sp);
    case 5: return launch_scan_g<5>(fused, tile_tokens, grid, st, sp);
    case 6: return launch_scan_g<6>(fused, tile_tokens, grid, st, sp);
    case 7: return launch_scan_g<7>(fused, tile_tokens, grid, st, sp);
    case 8: return launch_scan_g<8>(fused, tile_tokens, grid, st, sp);
    default: return false;
  }
}

template <int CHUNK, int TILES>
void launch_select_as(bool attn, bool paged, dim3 grid, hipStream_t st, const SelectParams& sl) {
  if (!attn)
    hipLaunchKernelGGL((select_kernel<kSelThreads, false, METRIC, false, D, CHUNK, TILES>), grid, dim3(kSelThreads), 0, st, sl);
  else if (paged)
    hipLaunchKernelGGL((select_kernel<kSelThreads, true, METRIC, true, D, CHUNK, TILES>), grid, dim3(kSelThreads), 0, st, sl);
  else
    hipLaunchKernelGGL((select_kernel<kSelThreads, true, METRIC, false, D, CHUNK, TILES>), grid, dim3(kSelThreads), 0, st, sl);
}

// The histograms that a call loads together: as many as its longest sequence has tiles, rounded up to four (see select_kernel).
void launch_select(bool attn, bool paged, dim3 grid, hipStream_t st, const SelectParams& sl) {
  // segments of more than two passes (4096 tokens each) share one barrier among up to eight passes;
  // only planes of byte distances have that form
  if (Dist<METRIC, D>::kByteDist && sl.seg_len > 2 * 4096) {
    if (sl.n_tiles <= 8) launch_select_as<8, 8>(attn, paged, grid, st, sl);
    else launch_select_as<8, kHistBatch>(attn, paged, grid, st, sl);
  } else if (sl.n_tiles <= 4) {
    launch_select_as<1, 4>(attn, paged, grid, st, sl);
  } else if (sl.n_tiles <= 8) {
    launch_select_as<1, 8>(attn, paged, grid, st, sl);
  } else if (sl.n_tiles <= 12) {
    launch_select_as<1, 12>(attn, paged, grid, st, sl);
  } else {
    launch_select_as<1, kHistBatch>(attn, paged, grid, st, sl);
  }
}

template <int WAVES, bool FUSED, bool PAGED>
bool launch_one_as(hipStream_t st, const OneLaunchParams& op) {
  const dim3 grid(8 * op.group, (op.planes + 7) / 8);
  hipLaunchKernelGGL((one_launch_kernel<WAVES, FUSED, METRIC, PAGED, D>), grid, dim3(WAVES * kWave),
                     one_launch_lds(WAVES, D, op.max_seq_len, op.k, FUSED, PAGED), st, op);
  return true;
}

template <int WAVES>
bool launch_one_waves(bool fused, hipStream_t st, const OneLaunchParams& op) {
  if (!fused) return launch_one_as<WAVES, false, false>(st, op);
  // (the step with three-bit codes at d = 256 takes more registers than sixteen waves may have: the rule never asks for it)
  if constexpr (WAVES == 16 && METRIC == kMetricB3 && D == 256) {
    return false;
  } else {
    if (op.page_table != nullptr) return launch_one_as<WAVES, true, true>(st, op);
    return launch_one_as<WAVES, true, false>(st, op);
  }
}

bool launch_one(bool fused, int waves, hipStream_t st, const OneLaunchParams& op) {
  switch (waves) {
    case 4: return launch_one_waves<4>(fused, st, op);
    case 8: return launch_one_waves<8>(fused, st, op);
    case 16: return launch_one_waves<16>(fused, st, op);
    default: return false;
  }
}

// The launchers below are templates so that a set that does not export them
// does not instantiate their kernels either.
// Whether a bulk encode with the transform goes to encode_rows_matrix_kernel.  Lane groups / matrix cores, us, for
// 8000, 40000, 160000 and 640000 vectors of two-bit codes with symmetric thresholds:
//   D =  64   3.1 / 2.8   3.8 / 3.5   6.5 / 6.6   18.8 / 16.8
//   D =  96   4.0 / 5.1   6.0 / 6.9  13.1 / 12.7  45.5 / 33.3   (operands to LDS first: 1 us)
//   D = 128   3.5 / 3.5   5.5 / 5.1  11.6 / 10.8  37.2 / 35.6   and 56.9 / 58.3 for 1 Mi
//   D = 160   6.6 / 10.2 10.7 / 13.0 27.4 / 28.7  90.7 / 71.9
//   D = 192   5.2 / 7.2  11.1 / 10.6 33.3 / 23.4 114.4 / 64.5
//   D = 256   4.9 / 6.0   8.9 / 9.0  24.3 / 21.8  86.0 / 71.2
// At the limits below, one-bit codes and unsymmetric thresholds (other caches, so not comparable with the rows above):
//   one bit      D =  64  32768: 4.5 / 4.3   96 196608: 17.6 / 14.5  160 393216: 55.2 / 43.8  192 65536: 14.8 / 12.2  256 196608: 29.2 / 26.5
//   unsymmetric  D =  64 393216: 17.8 / 18.4 96 196608: 19.9 / 17.8  160 393216: 69.3 / 57.6  192 65536: 17.6 / 15.6  256 196608: 39.4 / 36.1
// Three-bit codes (seven masks) and codes without the transform are slower there.
template <int BITS_>
constexpr bool has_matrix_encode() { return BITS_ <= 2 && D != 128; }
inline bool matrix_encode_pays(const Thresholds& thr, int64_t n_vec) {
  if (!thr.transform) return false;
  if (D == 64) return BITS == 1 || thr.symmetric;
  return n_vec >= (D == 192 ? 64 : D == 160 ? 384 : 192) * 1024;
}

// Workgroups of its grid.  Where they put operands in LDS first, as many as run at once: later ones would start a round of
// their own and build the operands again.  Per compute unit, from the kernels' registers (94 to 216): D = 96 five
// (unsymmetric two-bit codes four), 160 three (two), 192 four (one-bit codes three, unsymmetric two).  us for 1 Mi vectors with 512 /
// 768 / 1024 / 1280 / 2560 workgroups, chosen *:
//   D =  96  symmetric 62.1 54.6 54.0  52.8* 53.4   one bit  58.2 49.9  47.1  47.6* 48.5   unsymmetric  64.7  57.4  57.2* 62.1  58.9
//   D = 160           115.1 106.8* 124.2 116.3 115.9        103.9 91.4* 109.8 99.2 101.4                123.1* 150.4 127.7 141.6 143.3
//   D = 192           109.3 101.7 103.1* 109.7 101.2         98.9 90.2* 103.6 95.8  95.1                118.0* 143.9 121.5 131.0 127.9
// Without operands in LDS smaller shares even out better (D = 256, symmetric: 126.5 / 129.1 / 139.5 / 134.9 / 125.9, 5120 119.0).
template <int BITS_, bool SYMMETRIC>
constexpr int64_t most_matrix_workgroups() {
  if (!EncShape<D>::kLds) return 5120;
  constexpr bool kUnsymmetric = BITS_ == 2 && !SYMMETRIC;
  return 256 * (D == 96 ? (kUnsymmetric ? 4 : 5) : D == 160 ? (kUnsymmetric ? 2 : 3) : kUnsymmetric ? 2 : BITS_ == 1 ? 3 : 4);
}

template <int BITS_>
void launch_encode_rows(hipStream_t st, const uint16_t* src, uint8_t* dst, int64_t head_stride_rows,
                        int64_t row_begin, int64_t n_rows, int64_t n_vec, const Thresholds& thr) {
  Divisor32 by_rows{};  // mul = 0: the kernel divides in 64 bits
  if (n_vec < ((int64_t)1 << 32) && n_rows >= 1) by_rows = Divisor32::of((uint32_t)n_rows);
  if constexpr (has_matrix_encode<BITS_>()) {
    if (matrix_encode_pays(thr, n_vec)) {
      // 64 vectors per workgroup and step
      const int64_t want = (n_vec + 63) / 64;
      auto launch = [&](auto symmetric) {
        constexpr int64_t kMost = most_matrix_workgroups<BITS_, decltype(symmetric)::value>();
        const int grid = (int)(want < kMost ? want : kMost);
        const int64_t step_heads = (int64_t)grid * 64 / n_rows, step_rows = (int64_t)grid * 64 % n_rows;
        hipLaunchKernelGGL((encode_rows_matrix_kernel<BITS_, D, decltype(symmetric)::value>), dim3(grid), dim3(256), 0,
                           st, src, dst, head_stride_rows, row_begin, n_rows, n_vec, thr, by_rows, step_heads, step_rows);
      };
      if constexpr (BITS_ == 1) launch(std::false_type{});
      else if constexpr (D == 64) launch(std::true_type{});  // (unsymmetric thresholds do not come here)
      else if (thr.symmetric) launch(std::true_type{});
      else launch(std::false_type{});
      return;
    }
  }
  // vectors per 256-thread workgroup and pass: D / 32 lanes per vector, or D / m lanes for D = 2^n * m (m = 12, 20)
  const int64_t per_wg = 256 / (HeadDim<D>::kPow2 ? D / 32 : D / HeadDim<D>::kBase);
  const int64_t want = (n_vec + per_wg - 1) / per_wg;
  const int grid = (int)(want < 16384 ? want : 16384);
  hipLaunchKernelGGL((encode_rows_kernel<BITS_, D>), dim3(grid), dim3(256), 0, st, src, dst,
                     head_stride_rows, row_begin, n_rows, n_vec, thr, by_rows);
}

template <int D_>
void launch_sparse_attn(bool wide, dim3 grid, hipStream_t st, const AttnParams& ap) {
  if (wide) hipLaunchKernelGGL((sparse_attn_kernel<kAttnThreadsWide, D_>), grid, dim3(kAttnThreadsWide), 0, st, ap);
  else hipLaunchKernelGGL((sparse_attn_kernel<kAttnThreads, D_>), grid, dim3(kAttnThreads), 0, st, ap);
}

template <int D_>
void launch_merge(dim3 grid, hipStream_t st, const MergeParams& mp) {
  hipLaunchKernelGGL(merge_kernel<D_>, grid, dim3(D_), 0, st, mp);
}

template <int G, int D_>
void launch_full_g(dim3 grid, hipStream_t st, const FullAttnParams& fp) {
  hipLaunchKernelGGL((full_attn_kernel<G, D_>), grid, dim3(kFullThreads), 0, st, fp);
}

template <int D_>
void launch_full(int G, dim3 grid, hipStream_t st, const FullAttnParams& fp) {
  switch (G) {
    case 1: launch_full_g<1, D_>(grid, st, fp); break;
    case 2: launch_full_g<2, D_>(grid, st, fp); break;
    case 3: launch_full_g<3, D_>(grid, st, fp); break;
    case 4: launch_full_g<4, D_>(grid, st, fp); break;
    case 5: launch_full_g<5, D_>(grid, st, fp); break;
    case 6: launch_full_g<6, D_>(grid, st, fp); break;
    case 7: launch_full_g<7, D_>(grid, st, fp); break;
    default: launch_full_g<8, D_>(grid, st, fp); break;
  }
}

template <int D_>
void launch_merge_parts(dim3 grid, hipStream_t st, const float* partial, float* out, int Hq,
                        int n_parts) {
  hipLaunchKernelGGL(merge_parts_kernel<D_>, grid, dim3(kMergeThreads), 0, st, partial, out, Hq, n_parts);
}

template <int M>
KernelSet make_set() {
  KernelSet ks{};
  ks.scan = launch_scan;
  ks.select = launch_select;
  ks.one_launch = launch_one;
  if constexpr (M != kMetricL2) ks.encode_rows = launch_encode_rows<BITS>;
  if constexpr (M == kMetricL1) {
    ks.sparse_attn = launch_sparse_attn<D>;
    ks.merge = launch_merge<D>;
    ks.full_attn = launch_full<D>;
    ks.merge_parts = launch_merge_parts<D>;
  }
  return ks;
}

}  // namespace

template <>
const KernelSet& kernel_set<ADAMAS_INST_D, ADAMAS_INST_METRIC>() {
  static const KernelSet ks = make_set<ADAMAS_INST_METRIC>();
  return ks;
}

}  // namespace adamas
