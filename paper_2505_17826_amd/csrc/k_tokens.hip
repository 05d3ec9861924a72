// Token bookkeeping: compaction of the masked rows (the "unpadding" a
// training engine does before the model, Sec. 2.1.2) and per-rollout counts of
// the tokens that enter the objective (action mask, Sec. 2.2 / Sec. 3.1.2).
// Integer work, bit-exact and deterministic: block counts and scatter (small
// batches in one workgroup).
#include "rft_internal.h"
#include "tokens_device.h"

namespace rft {

namespace {

constexpr int kThreads = 256;
constexpr int kPerThread = kK0Rows / kThreads;  // 8 consecutive rows per thread
static_assert(kPerThread == 8, "mask8 reads eight rows");

template <int NTH>
__global__ void __launch_bounds__(NTH) k_tokmeta_small(const rft_tokens tok, TokMeta m) {
  tokmeta_small<NTH>(tok, m);
}

// Valid rows of [a, b): four mask bytes at a time between its 4-byte boundaries.
__device__ __forceinline__ int count_range(const uint8_t* __restrict__ mask, int64_t a, int64_t b) {
  const int64_t m0 = (int64_t)((uintptr_t)mask & 3);
  int64_t a4 = ((a + m0 + 3) & ~(int64_t)3) - m0, b4 = ((b + m0) & ~(int64_t)3) - m0;
  if (a4 > b) a4 = b;
  if (b4 < a4) b4 = a4;
  int c = 0;
  for (int64_t t = a4 + (int64_t)threadIdx.x * 4; t < b4; t += kThreads * 4) {
    const uint32_t w = *(const uint32_t*)(mask + t);
    c += __builtin_popcount((((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u);
  }
  if (a + threadIdx.x < a4) c += mask[a + threadIdx.x] ? 1 : 0;
  if (b4 + threadIdx.x < b) c += mask[b4 + threadIdx.x] ? 1 : 0;
  return c;
}

// Blocks [0, nblk): valid rows of each block of kK0Rows rows; the next n_seq
// blocks: valid rows of each rollout.
__global__ void __launch_bounds__(kThreads) k_count(const uint8_t* __restrict__ mask,
                                                    const int32_t* __restrict__ ss, int64_t T,
                                                    int64_t nblk, int64_t n_seq,
                                                    int32_t* __restrict__ blk,
                                                    int32_t* __restrict__ n_i,
                                                    int32_t* __restrict__ meta) {
  __shared__ int red[4];
  const int64_t b = block_index();
  if (b >= nblk + n_seq) return;
  int64_t lo, hi;
  if (b < nblk) {
    lo = b * kK0Rows;
    hi = lo + kK0Rows < T ? lo + kK0Rows : T;
  } else {
    lo = ss[b - nblk], hi = ss[b - nblk + 1];
    lo = lo < 0 ? 0 : (lo > T ? T : lo);
    hi = hi < lo ? lo : (hi > T ? T : hi);
  }
  const int c = block_sum_int(count_range(mask, lo, hi), red);
  if (threadIdx.x == 0) {
    if (b < nblk) blk[b] = c; else n_i[b - nblk] = c;
    if (b == 0) meta[kMetaCounter] = 0;
  }
}

// S, expert tokens and expert rollouts with tokens (all threads of one block).
__device__ void seq_totals(const int32_t* __restrict__ n_i, int64_t n_seq,
                           const uint8_t* __restrict__ is_expert, int N,
                           int32_t* __restrict__ meta) {
  int s = 0, ne = 0, se = 0;
  for (int64_t i = threadIdx.x; i < n_seq; i += kThreads) {
    s += n_i[i] > 0 ? 1 : 0;
    if (is_expert && is_expert[i]) {
      ne += n_i[i];
      se += n_i[i] > 0 ? 1 : 0;
    }
  }
  __shared__ int red3[16][3];
  block_sum3(s, ne, se, red3);
  if (threadIdx.x == 0) {
    meta[0] = N;
    meta[1] = s;
    meta[2] = ne;
    meta[3] = se;
  }
}

// One block: block counts -> exclusive offsets (in place), N and S (batches of
// more than kSelfBlocks blocks; in smaller ones each block of k_scatter adds the
// counts before it itself, one launch less).
constexpr int64_t kSelfBlocks = 1024;
__global__ void __launch_bounds__(kThreads) k_scan(int32_t* __restrict__ blk, int nblk,
                                                   const int32_t* __restrict__ n_i, int64_t n_seq,
                                                   const uint8_t* __restrict__ is_expert,
                                                   int32_t* __restrict__ meta) {
  __shared__ int red[4];
  int carry = 0;
  for (int b0 = 0; b0 < nblk; b0 += kThreads) {
    int b = b0 + threadIdx.x, total;
    int ex = block_excl_scan(b < nblk ? blk[b] : 0, red, &total);
    if (b < nblk) blk[b] = carry + ex;
    carry += total;
  }
  seq_totals(n_i, n_seq, is_expert, carry, meta);
}

// The rollouts' starts go to LDS where they fit: the search for a row's rollout
// is a chain of dependent reads.
template <bool SCANNED>
__global__ void __launch_bounds__(kThreads) k_scatter(const rft_tokens tok, TokMeta m, int nblk) {
  __shared__ int red[4];
  __shared__ int ss[kSmallSeq + 1];
  const int n_seq = (int)tok.n_seq;
  const bool inlds = n_seq <= kSmallSeq;
  if (inlds)
    for (int i = threadIdx.x; i <= n_seq; i += kThreads) ss[i] = tok.seq_start[i];
  const int64_t t0 = (int64_t)blockIdx.x * kK0Rows + (int64_t)threadIdx.x * kPerThread;
  const uint32_t f = t0 < tok.T ? mask8(tok.mask, t0, tok.T) : 0u;
  int base;
  if (SCANNED) {
    base = m.blk[blockIdx.x];
  } else {
    int v = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kThreads) v += m.blk[b];
    base = block_sum_int(v, red);
    if ((int)blockIdx.x == nblk - 1)  // base + its own count = N
      seq_totals(m.n_i, tok.n_seq, tok.is_expert, base + m.blk[blockIdx.x], m.meta);
  }
  int total;
  const int off = base + block_excl_scan(__builtin_popcount(f), red, &total);
  __syncthreads();
  if (inlds) place8(f, t0, tok.T, (const int*)ss, n_seq, off, m.rows, m.row_seq, m.kidx);
  else place8(f, t0, tok.T, tok.seq_start, n_seq, off, m.rows, m.row_seq, m.kidx);
}

}  // namespace

TokMeta carve_tokmeta(Carver& c, int64_t T, int64_t n_seq) {
  TokMeta m;
  int64_t nblk = (T + kK0Rows - 1) / kK0Rows;
  m.rows = c.take<int32_t>(T > 0 ? T : 1);
  m.row_seq = c.take<int32_t>(T > 0 ? T : 1);
  m.kidx = c.take<int32_t>(T > 0 ? T : 1);
  m.n_i = c.take<int32_t>(n_seq > 0 ? n_seq : 1);
  m.blk = c.take<int32_t>(nblk > 0 ? nblk : 1);
  m.meta = c.take<int32_t>(kMetaCounter + 1);
  return m;
}

hipError_t launch_tokmeta(const rft_tokens& tok, const TokMeta& m, hipStream_t s) {
  const int64_t T = tok.T, n_seq = tok.n_seq;
  if (T <= 8192 && n_seq <= kSmallSeq) {
    if (T <= 2048) k_tokmeta_small<256><<<1, 256, 0, s>>>(tok, m);
    else k_tokmeta_small<1024><<<1, 1024, 0, s>>>(tok, m);
    return hipGetLastError();
  }
  const int64_t nblk = (T + kK0Rows - 1) / kK0Rows;
  if (nblk + n_seq > 0)
    k_count<<<grid_xy(nblk + n_seq), kThreads, 0, s>>>(tok.mask, tok.seq_start, T, nblk, n_seq,
                                                       m.blk, m.n_i, m.meta);
  if (nblk == 0 || nblk > kSelfBlocks)
    k_scan<<<1, kThreads, 0, s>>>(m.blk, (int)nblk, m.n_i, n_seq, tok.is_expert, m.meta);
  if (nblk > kSelfBlocks)
    k_scatter<true><<<(unsigned)nblk, kThreads, 0, s>>>(tok, m, (int)nblk);
  else if (nblk > 0)
    k_scatter<false><<<(unsigned)nblk, kThreads, 0, s>>>(tok, m, (int)nblk);
  return hipGetLastError();
}

}  // namespace rft
