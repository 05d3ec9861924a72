// Device code of the token bookkeeping shared by its own kernels and by the
// kernel that runs it for a handful of rows.
#pragma once

#include "rft_internal.h"

namespace rft {
namespace {

__device__ int block_sum_int(int v, int* red) {
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  v = wave_sum_i(v);
  if (lane == 0) red[w] = v;
  __syncthreads();
  int t = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += red[i];
  __syncthreads();
  return t;
}

// Sums of three ints over the block (red3: three per wave), valid in thread 0.
__device__ void block_sum3(int& a, int& b, int& c, int (*red3)[3]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  a = wave_sum_i(a);
  b = wave_sum_i(b);
  c = wave_sum_i(c);
  if (lane == 0) red3[w][0] = a, red3[w][1] = b, red3[w][2] = c;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) {
      a += red3[i][0];
      b += red3[i][1];
      c += red3[i][2];
    }
}

// Exclusive scan of one int per thread over the block; *total gets the sum.
__device__ int block_excl_scan(int v, int* red, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) red[w] = x;
  __syncthreads();
  int before = 0, all = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
    before += i < w ? red[i] : 0;
    all += red[i];
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// Flags of the rows t0 .. t0 + 7 that enter the objective (bit j: row t0 + j).
__device__ __forceinline__ uint32_t mask8(const uint8_t* __restrict__ mask, int64_t t0, int64_t T) {
  uint32_t f = 0;
  if (t0 + 8 <= T && ((uintptr_t)(mask + t0) & 7) == 0) {
    const uint64_t w = *(const uint64_t*)(mask + t0);
#pragma unroll
    for (int j = 0; j < 8; ++j) f |= ((w >> (8 * j)) & 0xff) ? 1u << j : 0u;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (t0 + j < T && mask[t0 + j]) f |= 1u << j;
  }
  return f;
}

// The rows and rollout of the flagged rows t0 .. t0 + 7 from compacted index
// off on; ss is seq_start (LDS or global).  The rollout of a row is the largest
// i in [0, n_seq) with ss[i] <= t, searched for the first row and walked from
// there, or searched again where more than four rollouts lie between two rows
// (empty ones: walking 30000 of them took 2.2 ms; always in bounds).
template <typename P>
__device__ __forceinline__ void place8(uint32_t f, int64_t t0, int64_t T, P ss, int n_seq, int off,
                                       int32_t* __restrict__ rows, int32_t* __restrict__ row_seq,
                                       int32_t* __restrict__ kidx) {
  int lo = 0;
  auto search = [&](int64_t t) {
    int hi = n_seq - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if ((int64_t)ss[mid] <= t) lo = mid; else hi = mid - 1;
    }
  };
  if (f) search(t0);
  int64_t next = lo + 1 < n_seq ? (int64_t)ss[lo + 1] : T;  // first row of the next rollout
  int kx[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int64_t t = t0 + j;
    kx[j] = -1;
    if (f >> j & 1) {
      for (int w = 0; next <= t; ++w) {
        if (w < 4) ++lo; else search(t);
        next = lo + 1 < n_seq ? (int64_t)ss[lo + 1] : T;
      }
      rows[off] = (int32_t)t;
      row_seq[off] = lo;
      kx[j] = off++;
    }
  }
  // kidx and t0 are multiples of 16 bytes and of 8 rows
  if (t0 + 8 <= T) {
    *(int4*)(kidx + t0) = make_int4(kx[0], kx[1], kx[2], kx[3]);
    *(int4*)(kidx + t0 + 4) = make_int4(kx[4], kx[5], kx[6], kx[7]);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (t0 + j < T) kidx[t0 + j] = kx[j];
  }
}

// Small batches: everything in one workgroup (prefix counts of the mask and the
// rollouts' starts in LDS).  A call on few rows is a chain of launches of a few
// microseconds each; the four that every path took were 15 us of the 67 of a
// loss call on 128 rows, this one is 4.  Larger batches take two launches: 24 ->
// 11 us at 262144 rows.
constexpr int kSmallSeq = (int)kFewSeq;
template <int NTH>
__device__ __forceinline__ void tokmeta_small(const rft_tokens& tok, const TokMeta& m) {
  constexpr int kSmallT = 8 * NTH;
  __shared__ int pre[kSmallT + 1];
  __shared__ int ss[kSmallSeq + 1];
  __shared__ int red[16];
  const int T = (int)tok.T, n_seq = (int)tok.n_seq, tid = threadIdx.x;
  for (int i = tid; i <= n_seq; i += NTH) ss[i] = tok.seq_start[i];
  const int t0 = tid * 8;
  const uint32_t f = t0 < T ? mask8(tok.mask, t0, T) : 0u;
  int N;
  const int off = block_excl_scan(__builtin_popcount(f), red, &N);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (t0 + j <= T) pre[t0 + j] = off + __builtin_popcount(f & ((1u << j) - 1));
  if (tid == NTH - 1 && T == kSmallT) pre[T] = N;
  __syncthreads();
  int s = 0, ne = 0, se = 0;
  for (int i = tid; i < n_seq; i += NTH) {
    int a = ss[i], b = ss[i + 1];
    a = a < 0 ? 0 : (a > T ? T : a);
    b = b < a ? a : (b > T ? T : b);
    const int n = pre[b] - pre[a];
    m.n_i[i] = n;
    s += n > 0 ? 1 : 0;
    if (tok.is_expert && tok.is_expert[i]) {
      ne += n;
      se += n > 0 ? 1 : 0;
    }
  }
  __shared__ int red3[16][3];
  block_sum3(s, ne, se, red3);
  if (tid == 0) {
    m.meta[0] = N;
    m.meta[1] = s;
    m.meta[2] = ne;
    m.meta[3] = se;
    m.meta[kMetaCounter] = 0;
  }
  if (t0 < T) place8(f, t0, T, (const int*)ss, n_seq, off, m.rows, m.row_seq, m.kidx);
}

}  // namespace
}  // namespace rft
