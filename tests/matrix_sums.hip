// Sums of the matrix instruction that the bulk encode relies on, for a test of the bound on their rounding.
#include "device_utils.hpp"

// A[n][16][32], B[n][32][16] (bf16 bits) -> D[n][16][16]; one wave per tile.
__global__ __launch_bounds__(64) void matrix_sums_kernel(const uint16_t* A, const uint16_t* B, float* D) {
  const int64_t tile = blockIdx.x;
  const int n = threadIdx.x % 16, g = threadIdx.x / 16;
  uint32_t a[4], b[4];
  for (int j = 0; j < 4; ++j) {
    const uint16_t* row = A + tile * 512 + n * 32 + 8 * g + 2 * j;
    const uint16_t* col = B + tile * 512 + (8 * g + 2 * j) * 16 + n;
    a[j] = row[0] | (uint32_t)row[1] << 16;
    b[j] = col[0] | (uint32_t)col[16] << 16;
  }
  const adamas::f32x4 c = adamas::mfma_16x16x32(a, b, adamas::f32x4{0.f, 0.f, 0.f, 0.f});
  for (int i = 0; i < 4; ++i) D[tile * 256 + (4 * g + i) * 16 + n] = c[i];
}

extern "C" int matrix_sums(const void* A, const void* B, void* D, int tiles, void* stream) {
  if (tiles < 1) return 1;
  hipLaunchKernelGGL(matrix_sums_kernel, dim3(tiles), dim3(64), 0, (hipStream_t)stream, static_cast<const uint16_t*>(A),
                     static_cast<const uint16_t*>(B), static_cast<float*>(D));
  return (int)hipGetLastError();
}
