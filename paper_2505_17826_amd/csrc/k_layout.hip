// Small layout kernels: hidden-row compaction and zero fills.
#include "rft_internal.h"

namespace rft {

// ------------------------------------------------------- layout helpers ----
// Hc[k, :] = H[rows[k], :] for the valid rows k < count (bf16, 16-byte copies):
// the compacted hidden states every GEMM of the bf16 path reads.
__global__ void __launch_bounds__(256) k_gather_rows16(const uint16_t* __restrict__ H, int64_t d,
                                                       const int32_t* __restrict__ rows,
                                                       const int32_t* __restrict__ cnt,
                                                       int64_t cap, uint16_t* __restrict__ Hc) {
  int64_t n = cnt[0];
  n = n < 0 ? 0 : (n > cap ? cap : n);
  const int64_t d8 = d >> 3;
  for (int64_t k = blockIdx.x; k < n; k += gridDim.x) {
    const uint4* src = (const uint4*)(H + (int64_t)rows[k] * d);
    uint4* dst = (uint4*)(Hc + k * d);
    for (int64_t j = threadIdx.x; j < d8; j += 256) dst[j] = src[j];
  }
}

// Zero the rows of out[T, width] whose mask is 0, and those rows' entries of up
// to three per-token vectors.
__global__ void __launch_bounds__(256) k_zero_masked_rows(const uint8_t* __restrict__ mask,
                                                          int64_t T, int64_t width,
                                                          float* __restrict__ out, float* v0,
                                                          float* v1, float* v2) {
  for (int64_t t = blockIdx.x; t < T; t += gridDim.x) {
    if (mask[t]) continue;
    for (int64_t j = threadIdx.x; j < width; j += 256) out[t * width + j] = 0.f;
    if (threadIdx.x == 0) {
      if (v0) v0[t] = 0.f;
      if (v1) v1[t] = 0.f;
      if (v2) v2[t] = 0.f;
    }
  }
}

__global__ void __launch_bounds__(256) k_fill_zero(float* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    out[i] = 0.f;
}

hipError_t launch_fill_zero(float* out, int64_t n, hipStream_t s) {
  if (n > 0) {
    int64_t b = (n + 255) / 256;
    k_fill_zero<<<(unsigned)(b < 8192 ? b : 8192), 256, 0, s>>>(out, n);
  }
  return hipGetLastError();
}

hipError_t launch_gather_rows16(const uint16_t* H, int64_t d, const int32_t* rows,
                                const int32_t* cnt, int64_t cap, uint16_t* Hc, hipStream_t s) {
  if (cap > 0) k_gather_rows16<<<(unsigned)(cap < 16384 ? cap : 16384), 256, 0, s>>>(H, d, rows, cnt, cap, Hc);
  return hipGetLastError();
}

hipError_t launch_zero_masked_rows(const uint8_t* mask, int64_t T, int64_t width, float* out,
                                   hipStream_t s, float* v0, float* v1, float* v2) {
  if (T > 0)
    k_zero_masked_rows<<<(unsigned)(T < 4096 ? T : 4096), 256, 0, s>>>(mask, T, width, out, v0, v1, v2);
  return hipGetLastError();
}

}  // namespace rft
