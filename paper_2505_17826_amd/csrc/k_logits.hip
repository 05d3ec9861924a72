// Loss-only path from given fp32 logits [T, V]: one workgroup per row.
//   pass 1: stream the row (16-byte loads) keeping per-thread online
//           (max, sum exp, sum exp*z), reduce over the workgroup in a fixed
//           order;
//   row terms: lse, entropy, logp = z_y - lse, the PPO-clip/KL loss terms
//           and c_t = d loss / d logp;
//   pass 2: d_logits = c_t (onehot - p) + e_t p (z - mu_t) (p the softmax,
//           e_t the entropy-bonus coefficient, mu_t = lse - entropy) with
//           non-temporal stores.
// The fused kernel keeps the row on chip between the passes (registers, then
// LDS) so that a row of up to about 600 KB is read from HBM once; shorter rows
// take variants with fewer registers and less LDS, several workgroups per CU,
// so that one's loads run under another's stores.
// A row is cut at the 16-byte boundaries of its logits (RowView): up to three
// elements before the first, whole chunks of four, up to three after the last;
// V and the base need no alignment.  Every kernel that forms statistics gives
// each thread the same chunks of the row in the same order, and an element of
// d_logits depends on the row's statistics and its own logit only, so the
// statistics-only, d_logits-only and fused kernels agree bit for bit.
#include <algorithm>

#include "rft_internal.h"
#include "tokens_device.h"

namespace rft {
namespace lg {

constexpr int NT = 512;
constexpr int UNROLL = 4;

// d_logits need not share the logits' alignment
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// One row of V logits: h elements up to the first 16-byte boundary, n4 chunks
// of four from there, tail elements after them.  Thread t < h + tail also
// takes the single element extra(t).
struct RowView {
  const float* z4;  // first chunk
  int64_t n4;
  int h, tail;
  __device__ __forceinline__ RowView(const float* z, int64_t V) {
    const int a = (int)(((16 - ((uintptr_t)z & 15)) & 15) >> 2);
    h = (int)(a < V ? a : V);
    n4 = (V - h) >> 2;
    tail = (int)((V - h) & 3);
    z4 = z + h;
  }
  // row at a 16-byte boundary with V a multiple of 4
  __device__ __forceinline__ RowView(const float* z, int64_t V, bool) : z4(z), n4(V >> 2), h(0), tail(0) {}
  __device__ __forceinline__ bool has_extra(int t) const { return t < h + tail; }
  __device__ __forceinline__ int64_t extra(int t) const { return t < h ? t : 4 * n4 + t; }
};


// Online (max, sum exp, sum exp * z) over a thread's logits.  Every exponent
// argument is <= 0 (hardware exp2; results below 2^-126 flush to 0).  Logits
// of -inf (masked entries) add nothing: while the running max is still below
// kLowest the exponents are taken against 0, and z is clamped to the finite range
// in the product exp * z (0 * z stays 0).  The same holds for entries masked by
// the type's lowest value, whose product with log2(e) would overflow.
constexpr float kLowest = -2e38f;  // 2e38 log2(e) is finite
__device__ __forceinline__ float zfin(float z) { return fmaxf(z, -FLT_MAX); }

__device__ __forceinline__ void acc4(RowStats& r, float4 q) {
  float mq = fmaxf(fmaxf(q.x, q.y), fmaxf(q.z, q.w));
  if (mq > r.m) {  // rescale to the new running max
    float sc = __builtin_amdgcn_exp2f((r.m - mq) * kLog2e);
    r.s *= sc;
    r.u *= sc;
    r.m = mq;
  }
  float mk = r.m < kLowest ? 0.f : r.m * kLog2e;
  float e0 = __builtin_amdgcn_exp2f(fmaf(q.x, kLog2e, -mk));
  float e1 = __builtin_amdgcn_exp2f(fmaf(q.y, kLog2e, -mk));
  float e2 = __builtin_amdgcn_exp2f(fmaf(q.z, kLog2e, -mk));
  float e3 = __builtin_amdgcn_exp2f(fmaf(q.w, kLog2e, -mk));
  r.s += (e0 + e1) + (e2 + e3);
  r.u += (e0 * zfin(q.x) + e1 * zfin(q.y)) + (e2 * zfin(q.z) + e3 * zfin(q.w));
}

__device__ __forceinline__ void acc1(RowStats& r, float z) {
  if (z > r.m) {
    float sc = __builtin_amdgcn_exp2f((r.m - z) * kLog2e);
    r.s *= sc;
    r.u *= sc;
    r.m = z;
  }
  float e = __builtin_amdgcn_exp2f(fmaf(z, kLog2e, r.m < kLowest ? 0.f : -r.m * kLog2e));
  r.s += e;
  r.u += e * zfin(z);
}

// Workgroup reduction of the per-thread online partials, in a fixed order: a
// binary tree over the waves (lane i of the first wave holds wave i's partial;
// lane 0 ends with the pairs of tree_merge, in its order), so that a row cut
// into 2, 4 or 8 parts of whole waves (k_logits_part) ends with the same bits.
// Six registers: with all the waves' partials in one thread the one-workgroup
// kernel, which holds 224 registers of the row here, spilled four.
template <int NTH = NT>
__device__ RowStats block_stats(RowStats r, RowStats* sh) {
  constexpr int NW = NTH / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float M = wave_max_f(r.m);
  float sc = (r.s > 0.f) ? __builtin_amdgcn_exp2f((r.m - M) * kLog2e) : 0.f;
  float s = wave_sum_f(r.s * sc), u = wave_sum_f(r.u * sc);
  if (lane == 0) sh[w] = RowStats{M, s, u};
  __syncthreads();
  if (threadIdx.x < NW) {
    RowStats v = sh[threadIdx.x];
#pragma unroll
    for (int o = 1; o < NW; o <<= 1) {
      const float m2 = __shfl_xor(v.m, o, 64), s2 = __shfl_xor(v.s, o, 64);
      const float u2 = __shfl_xor(v.u, o, 64);
      lse_merge(v.m, v.s, v.u, m2, s2, u2);
    }
    if (threadIdx.x == 0) sh[NW] = v;
  }
  __syncthreads();
  RowStats out = sh[NW];
  __syncthreads();
  return out;
}

__device__ RowStats row_pass1(const float* __restrict__ z, int64_t V, RowStats* sh) {
  RowStats r = {-INFINITY, 0.f, 0.f};
  const RowView rv(z, V);
  const float4* z4 = (const float4*)rv.z4;
  int64_t j = threadIdx.x;
  for (; j + (UNROLL - 1) * NT < rv.n4; j += UNROLL * NT) {
    float4 q[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) q[u] = z4[j + u * NT];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) acc4(r, q[u]);
  }
  for (; j < rv.n4; j += NT) acc4(r, z4[j]);
  if (rv.has_extra(threadIdx.x)) acc1(r, z[rv.extra(threadIdx.x)]);
  return block_stats(r, sh);
}

// d_logits of four logits, those of the chunk whose first element is j4 (from
// the row's first chunk); ENT adds the entropy-bonus term e p (z - mu).
template <bool ENT>
__device__ __forceinline__ floatx4 dlogit4(floatx4 q, float lk, float c, float e, float mu,
                                           int64_t j, int yc) {
  const int hot = (yc >> 2) == j ? (yc & 3) : -1;
  floatx4 d;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float p = __builtin_amdgcn_exp2f(fmaf(q[i], kLog2e, -lk));
    d[i] = ENT ? dlogit(c, e, mu, p, q[i], hot == i) : c * ((hot == i ? 1.f : 0.f) - p);
  }
  return d;
}
template <bool ENT>
__device__ __forceinline__ float dlogit1(float z, float lk, float c, float e, float mu, bool hot) {
  const float p = __builtin_amdgcn_exp2f(fmaf(z, kLog2e, -lk));
  return ENT ? dlogit(c, e, mu, p, z, hot) : c * ((hot ? 1.f : 0.f) - p);
}

// d_logits of one row: c (onehot - p) + e p (z - mu), 16-byte stores, by ST
// threads; vt: the thread's place among them.  UN chunks' loads in flight at a
// time; with one wavefront per row also of a lane's last few chunks.
template <bool ENT, int UN, int ST = NT>
__device__ void row_pass2(const float* __restrict__ z, int64_t V, float lse, float c, float e,
                          float mu, int y, float* __restrict__ out, int vt) {
  const float lk = lse * kLog2e;
  const RowView rv(z, V);
  const floatx4* z4 = (const floatx4*)rv.z4;
  float* const o4 = out + rv.h;
  const int yc = y - rv.h;
  int64_t j = vt;
  for (; j + (UN - 1) * ST < rv.n4; j += UN * ST) {
    floatx4 q[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) q[u] = z4[j + u * ST];
#pragma unroll
    for (int u = 0; u < UN; ++u)
      __builtin_nontemporal_store((f4u)dlogit4<ENT>(q[u], lk, c, e, mu, j + u * ST, yc),
                                  (f4u*)(o4 + 4 * (j + u * ST)));
  }
  if constexpr (UN > 1 && ST == 64) {
    if (j < rv.n4) {
      floatx4 q[UN - 1];
#pragma unroll
      for (int u = 0; u < UN - 1; ++u) q[u] = z4[min(j + u * ST, rv.n4 - 1)];
#pragma unroll
      for (int u = 0; u < UN - 1; ++u)
        if (j + u * ST < rv.n4)
          __builtin_nontemporal_store((f4u)dlogit4<ENT>(q[u], lk, c, e, mu, j + u * ST, yc),
                                      (f4u*)(o4 + 4 * (j + u * ST)));
    }
  } else {
    for (; j < rv.n4; j += ST)
      __builtin_nontemporal_store((f4u)dlogit4<ENT>(z4[j], lk, c, e, mu, j, yc), (f4u*)(o4 + 4 * j));
  }
  if (rv.has_extra(vt)) {
    const int64_t i = rv.extra(vt);
    out[i] = dlogit1<ENT>(z[i], lk, c, e, mu, i == y);
  }
}

// Zero a row of d_logits, 16-byte stores at its own boundaries (NTS: non-temporal).
template <int ST = NT, bool NTS = true>
__device__ void zero_row(float* __restrict__ out, int64_t V, int vt) {
  const RowView rv(out, V);
  const floatx4 zz = {0.f, 0.f, 0.f, 0.f};
  for (int64_t j = vt; j < rv.n4; j += ST) {
    floatx4* const o = (floatx4*)rv.z4 + j;
    if (NTS) __builtin_nontemporal_store(zz, o);
    else *o = zz;
  }
  if (rv.has_extra(vt)) out[rv.extra(vt)] = 0.f;
}

// ---- statistics only (rft_token_logprobs_from_logits)
__global__ void __launch_bounds__(NT) k_logits_stats(const float* __restrict__ logits, int64_t T,
                                                      int64_t V, const uint8_t* __restrict__ mask,
                                                      const int32_t* __restrict__ ids,
                                                      float* __restrict__ logp,
                                                      float* __restrict__ ent,
                                                      float* __restrict__ lse,
                                                      float* __restrict__ gathered) {
  __shared__ RowStats sh[NT / 64 + 1];
  int64_t t = blockIdx.x;
  if (!mask[t]) {
    if (threadIdx.x == 0) {
      logp[t] = 0.f;
      if (ent) ent[t] = 0.f;
      lse[t] = 0.f;
      if (gathered) gathered[t] = 0.f;
    }
    return;
  }
  const float* z = logits + t * V;
  RowStats r = row_pass1(z, V, sh);
  if (threadIdx.x == 0) {
    float L = r.m + logf(r.s);
    int y = ids[t];
    bool ok = y >= 0 && (int64_t)y < V;
    float zy = ok ? z[y] : __int_as_float(0x7fc00000);
    lse[t] = L;
    if (ent) ent[t] = L - r.u / r.s;
    logp[t] = zy - L;
    if (gathered) gathered[t] = zy;
  }
}

// ---- d_logits only (rft_ppo_clip_loss_bwd_logits).  Row t by ST threads, this one
// the vt-th.
template <bool ENT, int UN, int ST>
__device__ __forceinline__ void bwd_row(const float* __restrict__ logits, int64_t V, int64_t t,
                                        int vt, const uint8_t* __restrict__ mask,
                                        const int32_t* __restrict__ ids,
                                        const float* __restrict__ lse,
                                        const float* __restrict__ grad,
                                        const float* __restrict__ egrad,
                                        const float* __restrict__ ent, float* __restrict__ dl) {
  float* out = dl + t * V;
  if (!mask[t]) {
    zero_row<ST>(out, V, vt);
    return;
  }
  int y = ids[t];
  const float L = lse[t];
  const float e = ENT ? egrad[t] : 0.f, mu = ENT ? L - ent[t] : 0.f;
  row_pass2<ENT, UN, ST>(logits + t * V, V, L, grad[t], e, mu,
                         (y >= 0 && (int64_t)y < V) ? y : -1, out, vt);
}

// 2^lp workgroups per row, of NT / 2^lp threads each
template <bool ENT, int UN>
__global__ void __launch_bounds__(NT) k_logits_bwd(const float* __restrict__ logits, int64_t V,
                                                    const uint8_t* __restrict__ mask,
                                                    const int32_t* __restrict__ ids,
                                                    const float* __restrict__ lse,
                                                    const float* __restrict__ grad,
                                                    const float* __restrict__ egrad,
                                                    const float* __restrict__ ent,
                                                    float* __restrict__ dl, int lp) {
  const int64_t t = blockIdx.x >> lp;
  const int vt = (int)(blockIdx.x & ((1u << lp) - 1)) * (NT >> lp) + threadIdx.x;
  bwd_row<ENT, UN, NT>(logits, V, t, vt, mask, ids, lse, grad, egrad, ent, dl);
}

// Short rows: one wavefront per row, four rows per workgroup.  What bounds them is
// the chain of a row's loads (mask, its scalars, its logits), so the rows in
// flight count.  One wavefront against 512 threads per row: 96311 rows of 25 logits
// 21.4 / 90 us, 49502 of 316 22.6 / 52, 20000 of 1001 29.2 / 30.7; from there on
// the 512 threads are as fast or faster (8000 rows of 2047 25.1 / 22.3).
constexpr int kShortRow = 1024, kShortT = 256;
template <bool ENT, int UN>
__global__ void __launch_bounds__(kShortT) k_logits_bwd_short(
    const float* __restrict__ logits, int64_t T, int64_t V, const uint8_t* __restrict__ mask,
    const int32_t* __restrict__ ids, const float* __restrict__ lse, const float* __restrict__ grad,
    const float* __restrict__ egrad, const float* __restrict__ ent, float* __restrict__ dl) {
  const int64_t t = (int64_t)blockIdx.x * (kShortT / 64) +
                    __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (t < T)
    bwd_row<ENT, UN, 64>(logits, V, t, threadIdx.x & 63, mask, ids, lse, grad, egrad, ent, dl);
}

// ---- a handful of long rows: one workgroup per row leaves CUs idle, and a CU
// reads a row at its own rate (about 40 us for 600 KB read and written), so a
// row is cut into P = 2, 4 or 8 parts of 8 / P waves: this kernel (and the token
// bookkeeping in one workgroup more), the row terms of all rows in one workgroup
// (launch_few_terms), then k_logits_bwd with P
// workgroups per row, which finds the logits in the last-level cache.  Whole
// call at V = 151936: 128 rows 47 -> 42 us, 64 rows 48 -> 34, 16 rows 46 -> 26.
template <int P>
__global__ void __launch_bounds__(NT / P) k_logits_part(const float* __restrict__ logits, int64_t V,
                                                         const rft_tokens tok, TokMeta m,
                                                         RowStats* __restrict__ part) {
  __shared__ RowStats sh[NT / P / 64 + 1];
  const int64_t t = blockIdx.x / P;
  if (t == tok.T) {  // one workgroup more for the token bookkeeping
    tokmeta_small<NT / P>(tok, m);
    return;
  }
  if (!tok.mask[t]) return;
  const int vt = (int)(blockIdx.x % P) * (NT / P) + threadIdx.x;
  const float* z = logits + t * V;
  RowStats r = {-INFINITY, 0.f, 0.f};
  const RowView rv(z, V);
  const float4* z4 = (const float4*)rv.z4;
  constexpr int UN = 16;
  int64_t j = vt;
  for (; j + (UN - 1) * NT < rv.n4; j += UN * NT) {
    float4 q[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) q[u] = z4[j + u * NT];
#pragma unroll
    for (int u = 0; u < UN; ++u) acc4(r, q[u]);
  }
  float4 q[UN];
#pragma unroll
  for (int u = 0; u < UN; ++u)
    if (j + u * NT < rv.n4) q[u] = z4[j + u * NT];
#pragma unroll
  for (int u = 0; u < UN; ++u)
    if (j + u * NT < rv.n4) acc4(r, q[u]);
  if (rv.has_extra(vt)) acc1(r, z[rv.extra(vt)]);
  r = block_stats<NT / P>(r, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = r;
}

// ---- fused: statistics, loss terms and d_logits (rft_ppo_clip_fused_logits),
// reading the row twice: rows beyond a buffer descriptor (V > 2^28)
__global__ void __launch_bounds__(NT) k_logits_fused(
    const float* __restrict__ logits, int64_t T, int64_t V, const uint8_t* __restrict__ mask,
    const int32_t* __restrict__ ids, const int32_t* __restrict__ kidx,
    const int32_t* __restrict__ row_seq, const int32_t* __restrict__ n_i,
    const int32_t* __restrict__ meta, const float* __restrict__ old, const float* __restrict__ ref,
    const float* __restrict__ adv, LossConst cst, float* __restrict__ logp,
    float* __restrict__ ent, float* __restrict__ lse_out, float* __restrict__ grad_out,
    float* __restrict__ dl, LossPartial* __restrict__ parts) {
  __shared__ RowStats sh[NT / 64 + 1];
  __shared__ float row_c, row_e, row_mu;
  int64_t t = blockIdx.x;
  float* out = dl + t * V;
  int k = kidx[t];
  if (k < 0) {
    zero_row(out, V, threadIdx.x);
    if (threadIdx.x == 0) {
      logp[t] = 0.f;
      if (ent) ent[t] = 0.f;
      if (lse_out) lse_out[t] = 0.f;
      if (grad_out) grad_out[t] = 0.f;
      parts[t] = RFT_ZERO_PARTIAL;
    }
    return;
  }
  const float* z = logits + t * V;
  RowStats r = row_pass1(z, V, sh);
  if (threadIdx.x == 0) {
    float L = r.m + logf(r.s);
    float H = L - r.u / r.s;
    int y = ids[t];
    bool ok = y >= 0 && (int64_t)y < V;
    float lp = ok ? z[y] - L : __int_as_float(0x7fc00000);
    logp[t] = lp;
    if (ent) ent[t] = H;
    if (lse_out) lse_out[t] = L;
    LossPartial p = RFT_ZERO_PARTIAL;
    float c = 0.f, e = 0.f;
    if (!ok) {
      p.bad = 1;
    } else {
      int i = row_seq[k];
      float rf = ref ? ref[t] : lp;
      const bool ex = cst.is_expert && cst.is_expert[i];
      c = row_loss(lp, old[t], rf, adv[i], n_i[i], ex, meta, (double)H, cst, p, &e);
    }
    if (grad_out) grad_out[t] = c;
    parts[t] = p;
    row_c = c;
    row_e = e;
    row_mu = L - H;
    sh[NT / 64].m = L;
  }
  __syncthreads();
  float c = row_c, L = sh[NT / 64].m;
  int y = ids[t];
  row_pass2<true, 8>(z, V, L, c, row_e, row_mu, (y >= 0 && (int64_t)y < V) ? y : -1, out, threadIdx.x);
}

// ---- fused, with the row kept on chip: the first REG*NTC float4 of the row
// stay in registers and the next LCAP float4 in LDS between the two passes;
// only the remainder is read twice.
typedef int v4i __attribute__((ext_vector_type(4)));
constexpr int NTC = NT;

__device__ __forceinline__ void acc4v(RowStats& r, floatx4 q) {
  acc4(r, make_float4(q[0], q[1], q[2], q[3]));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* p, int64_t bytes) {
  uint64_t a = (uint64_t)p;
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  int nr = __builtin_amdgcn_readfirstlane((int)bytes);
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), 0, nr, 0x00020000);
}

// REGS float4 per thread in registers, LCH in LDS, WPS waves per SIMD (WPS / 2
// workgroups per CU).  AL: every row of the logits and of d_logits starts at a
// 16-byte boundary and V is a multiple of 4 (the general form costs the
// one-workgroup variant 2.6%: 1848 us against 1800 for 8192 x 151936).
template <bool ENT, int REGS, int LCH, int WPS, bool AL>
__global__ void __launch_bounds__(NTC, WPS) k_logits_fused_cached(
    const float* __restrict__ logits, int64_t T, int64_t V, const uint8_t* __restrict__ mask,
    const int32_t* __restrict__ ids, const int32_t* __restrict__ kidx,
    const int32_t* __restrict__ row_seq, const int32_t* __restrict__ n_i,
    const int32_t* __restrict__ meta, const float* __restrict__ old, const float* __restrict__ ref,
    const float* __restrict__ adv, LossConst cst, float* __restrict__ logp,
    float* __restrict__ ent, float* __restrict__ lse_out, float* __restrict__ grad_out,
    float* __restrict__ dl, LossPartial* __restrict__ parts) {
  constexpr int LCAP = LCH * NTC;
  extern __shared__ floatx4 row_lds[];  // LCAP float4
  __shared__ RowStats sh[NTC / 64 + 1];
  __shared__ float row_c, row_e, row_mu;
  const int tid = threadIdx.x;
  const int64_t t = blockIdx.x;
  float* out = dl + t * V;
  const int k = kidx[t];
  // descriptors over the row's whole chunks (at most 1 GiB, checked by the
  // launcher)
  const float* const zrow = logits + t * V;
  const RowView rv = AL ? RowView(zrow, V, true) : RowView(zrow, V);
  const int64_t n4 = rv.n4;
  const __amdgpu_buffer_rsrc_t rin = row_rsrc(rv.z4, n4 * 16);
  const __amdgpu_buffer_rsrc_t rout = row_rsrc(out + rv.h, n4 * 16);
  const uint32_t vo = (uint32_t)tid * 16u;
  constexpr uint32_t SU = (uint32_t)NTC * 16u;  // bytes between a thread's chunks
  if (k < 0) {
    // Where two or three workgroups share a CU, masked rows are cleared by ordinary
    // stores: 17622 rows of 27176 logits, 90% masked, 530 -> 461 us (one workgroup
    // per CU took 490), 10% masked 742 -> 709; 4000 of 50001 236 -> 201 and 324 ->
    // 312.  With four (60000 rows of 4000: 410 -> 422) and with one (8192 of 151936,
    // half masked: 1409 -> 1448) the non-temporal ones are faster.
    constexpr bool NTS = LCH == 0 || WPS == 2;
    if (AL) {
      const floatx4 zz = {0.f, 0.f, 0.f, 0.f};
      for (int64_t j = tid, o = vo; j < n4; j += NTC, o += SU)
        __builtin_amdgcn_raw_buffer_store_b128((v4i)zz, rout, (uint32_t)o, 0, NTS ? 2 : 0);
    } else {
      zero_row<NT, NTS>(out, V, threadIdx.x);
    }
    if (tid == 0) {
      logp[t] = 0.f;
      if (ent) ent[t] = 0.f;
      if (lse_out) lse_out[t] = 0.f;
      if (grad_out) grad_out[t] = 0.f;
      parts[t] = RFT_ZERO_PARTIAL;
    }
    return;
  }
  // The row's scalars for the loss terms (uniform over the workgroup: scalar
  // loads), issued now so that they have arrived when pass 1 ends.
  const int y0 = ids[t];
  const bool ok = y0 >= 0 && (int64_t)y0 < V;
  const float zy = ok ? zrow[y0] : 0.f;
  const int i_seq = row_seq[k];
  const float old_t = old[t], ref_t = ref ? ref[t] : 0.f, adv_i = adv[i_seq];
  const int n_seq_i = n_i[i_seq];
  const int32_t meta4[4] = {meta[0], meta[1], meta[2], meta[3]};

  // pass 1.  The LDS part of the row goes straight from HBM into LDS
  // (buffer_load ... lds, all of a lane's chunks in flight at once: lane l of
  // wave w fills slot s = c NTC + 64 w + l with chunk j_lds + s, the slot the
  // same thread reads back), then the register part, then the rest; chunks
  // past the row read as 0 and are left out of the statistics.
  const int64_t j_lds = (int64_t)REGS * NTC, j_rest = j_lds + LCAP;
  {
    const int w = tid >> 6;
#pragma unroll
    for (int c = 0; c < LCAP / NTC; ++c) {
      const int64_t j = j_lds + (int64_t)c * NTC + tid;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rin, (__attribute__((address_space(3))) void*)(row_lds + c * NTC + w * 64), 16,
          j < n4 ? (uint32_t)(j * 16) : 0x80000000u, 0, 0, 2);
    }
  }
  const int u_full = (int)min((int64_t)REGS, n4 / NTC);  // chunks complete for every thread
  // a lane whose chunk lies past the row takes a vector offset of 2^31, out of
  // range for the descriptor whether or not the scalar offset is counted
  const int nv = (int)min((int64_t)REGS, (n4 - tid + NTC - 1) / NTC);  // this lane's chunks
  floatx4 regs[REGS];
#pragma unroll
  for (int u = 0; u < REGS; ++u)
    regs[u] = (floatx4)__builtin_amdgcn_raw_buffer_load_b128(rin, u < nv ? vo : 0x80000000u,
                                                             (uint32_t)u * SU, 2);
  RowStats r = {-INFINITY, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < REGS; ++u) {
    if (u < u_full || (u == u_full && tid + (int64_t)u * NTC < n4)) acc4v(r, regs[u]);
  }
  // the direct-to-LDS loads have landed: this wave's loads are all back
  // (vmcnt 0), then the barrier (each thread reads back only its own slots)
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __syncthreads();
  for (int64_t j = j_lds + tid, s_ = tid; j < n4 && s_ < LCAP; j += NTC, s_ += NTC)
    acc4v(r, row_lds[s_]);
  for (int64_t j = j_rest + tid; j < n4; j += NTC)
    acc4v(r, (floatx4)__builtin_amdgcn_raw_buffer_load_b128(rin, (uint32_t)(j * 16), 0, 0));
  const bool ex1 = rv.has_extra(tid);
  const float zx = ex1 ? zrow[rv.extra(tid)] : 0.f;
  if (ex1) acc1(r, zx);
  r = block_stats<NTC>(r, sh);
  if (tid == 0) {
    float L = r.m + logf(r.s);
    float H = L - r.u / r.s;
    float lp = ok ? zy - L : __int_as_float(0x7fc00000);
    logp[t] = lp;
    if (ent) ent[t] = H;
    if (lse_out) lse_out[t] = L;
    LossPartial p = RFT_ZERO_PARTIAL;
    float c = 0.f, e = 0.f;
    if (!ok) {
      p.bad = 1;
    } else {
      float rf = ref ? ref_t : lp;
      const bool ex = cst.is_expert && cst.is_expert[i_seq];  // MIX only
      LossConst cc = cst;
      if (!ENT) cc.ent_coef = 0.f;  // the launcher picks ENT = (ent_coef > 0)
      c = row_loss(lp, old_t, rf, adv_i, n_seq_i, ex, meta4, (double)H, cc, p, &e);
    }
    if (grad_out) grad_out[t] = c;
    parts[t] = p;
    row_c = c;
    row_e = e;
    row_mu = L - H;
    sh[NTC / 64].m = L;
  }
  __syncthreads();
  const float c = row_c, lk = sh[NTC / 64].m * kLog2e, e = row_e, mu = row_mu;
  const int y = (ok ? y0 : -1) - rv.h;  // from the row's first chunk
  // pass 2: same three regions; stores past the row are dropped by the descriptor
  uint32_t vo2 = vo;
  int nv2 = nv;
  asm volatile("" : "+v"(vo2), "+v"(nv2));  // recomputed here, not held through pass 1
#pragma unroll
  for (int u = 0; u < REGS; ++u)
    __builtin_amdgcn_raw_buffer_store_b128(
        (v4i)dlogit4<ENT>(regs[u], lk, c, e, mu, tid + (int64_t)u * NTC, y), rout,
        u < nv2 ? vo2 + (uint32_t)u * SU : 0x80000000u, 0, 2);
  for (int64_t j = j_lds + tid, s_ = tid; j < n4 && s_ < LCAP; j += NTC, s_ += NTC)
    __builtin_amdgcn_raw_buffer_store_b128((v4i)dlogit4<ENT>(row_lds[s_], lk, c, e, mu, j, y), rout,
                                           (uint32_t)(j * 16), 0, 2);
  for (int64_t j = j_rest + tid; j < n4; j += NTC)
    __builtin_amdgcn_raw_buffer_store_b128(
        (v4i)dlogit4<ENT>((floatx4)__builtin_amdgcn_raw_buffer_load_b128(rin, (uint32_t)(j * 16), 0, 0),
                     lk, c, e, mu, j, y),
        rout, (uint32_t)(j * 16), 0, 2);
  if (rv.has_extra(tid)) {
    const int64_t i = rv.extra(tid);
    out[i] = dlogit1<ENT>(zrow[i], lk, c, e, mu, i - rv.h == y);
  }
}

}  // namespace lg

// Rows per launch: one workgroup of 512 threads per row, and a launch holds fewer
// than 2^32 work-items in x.  (The row's index from y as well, in one launch,
// cost the one-workgroup variant 2.4%.)
constexpr int64_t kLaunchRows = (int64_t)1 << 22;
template <class T>
static T* from(T* p, int64_t i) {
  return p ? p + i : nullptr;
}

hipError_t launch_logits_stats(const float* logits, const rft_tokens& tok, int64_t V, float* logp,
                               float* ent, float* lse, float* gathered, hipStream_t s) {
  for (int64_t t0 = 0; t0 < tok.T; t0 += kLaunchRows) {
    const int64_t n = std::min(tok.T - t0, kLaunchRows);
    lg::k_logits_stats<<<(unsigned)n, lg::NT, 0, s>>>(logits + t0 * V, n, V, tok.mask + t0,
                                                      tok.token_ids + t0, logp + t0, from(ent, t0),
                                                      lse + t0, from(gathered, t0));
  }
  return hipGetLastError();
}

// log2 of the parts a row is cut into: as many as the CUs hold beside the other
// rows (at most the eight waves of a row), if a part saves at least 32768 logits'
// time (8 us) for the launch that it costs; 0 = one workgroup per row.
static hipError_t row_parts(int64_t T, int64_t V, int* lp) {
  int ncu = 0;
  hipError_t e = cu_count(&ncu);
  if (e != hipSuccess) return e;
  *lp = 0;
  for (int k = 1; k <= 3; ++k)
    if ((T << k) <= ncu && V - (V >> k) >= 32768) *lp = k;
  return hipSuccess;
}

hipError_t launch_logits_bwd(const float* logits, const rft_tokens& tok, int64_t V,
                             const float* lse, const float* grad, const float* egrad,
                             const float* ent, float* dl, hipStream_t s) {
  if (tok.T <= 0) return hipSuccess;
  int lp = 0;
  hipError_t e = row_parts(tok.T, V, &lp);
  if (e != hipSuccess) return e;
  const bool en = egrad != nullptr;
  if (V <= lg::kShortRow) {
    auto k = V <= 256 ? (en ? lg::k_logits_bwd_short<true, 1> : lg::k_logits_bwd_short<false, 1>)
                      : (en ? lg::k_logits_bwd_short<true, 4> : lg::k_logits_bwd_short<false, 4>);
    for (int64_t t0 = 0; t0 < tok.T; t0 += kLaunchRows) {
      const int64_t n = std::min(tok.T - t0, kLaunchRows);
      k<<<(unsigned)((n + 3) / 4), lg::kShortT, 0, s>>>(logits + t0 * V, n, V, tok.mask + t0,
                                                        tok.token_ids + t0, lse + t0, grad + t0,
                                                        from(egrad, t0), from(ent, t0), dl + t0 * V);
    }
    return hipGetLastError();
  }
  // eight chunks in flight per thread where the rows leave CUs to spare, and for
  // rows of two to four such batches; otherwise one, whose few registers let every
  // wave slot fill.  One against eight: 600 rows of 151936 139 / 145 us, 8192 of them
  // 1945 / 2015, 60000 of 4000 303 / 327; 4096 of 32000 205 / 202, 4000 of 60000 378 /
  // 372.
  const bool eight = lp > 0 || (V > 16384 && V <= 65536);
  auto k = eight ? (en ? lg::k_logits_bwd<true, 8> : lg::k_logits_bwd<false, 8>)
                 : (en ? lg::k_logits_bwd<true, 1> : lg::k_logits_bwd<false, 1>);
  for (int64_t t0 = 0; t0 < tok.T; t0 += kLaunchRows) {
    const int64_t n = std::min(tok.T - t0, kLaunchRows);
    k<<<(unsigned)(n << lp), lg::NT >> lp, 0, s>>>(logits + t0 * V, V, tok.mask + t0,
                                                   tok.token_ids + t0, lse + t0, grad + t0,
                                                   from(egrad, t0), from(ent, t0), dl + t0 * V, lp);
  }
  return hipGetLastError();
}

// The on-chip variant for rows of V logits: the one with the most workgroups
// per CU that holds the row (REGS + LCH chunks of four for each of 512
// threads).  Two or more workgroups per CU overlap one row's loads with
// another's stores, which one cannot: it has read its whole row before it
// writes any of it.
template <bool ENT, int REGS, int LCH, int WPS, bool AL, class... A>
static hipError_t fused_cached(int64_t T, hipStream_t s, A... args) {
  auto k = lg::k_logits_fused_cached<ENT, REGS, LCH, WPS, AL>;
  constexpr int lds = LCH * lg::NTC * 16;
  if (lds > 0) {
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  k<<<(unsigned)T, lg::NTC, lds, s>>>(args...);
  return hipGetLastError();
}
template <bool ENT, bool AL, class... A>
static hipError_t fused_any(int64_t V, int64_t T, hipStream_t s, A... args) {
  constexpr int64_t kChunk = 4 * lg::NTC;  // logits per chunk of every thread
  if (V <= 6 * kChunk) return fused_cached<ENT, 6, 0, 8, AL>(T, s, args...);
  if (V <= 17 * kChunk) return fused_cached<ENT, 11, 6, 6, AL>(T, s, args...);
  if (V <= 31 * kChunk) return fused_cached<ENT, 22, 9, 4, AL>(T, s, args...);
  // 152 KiB of LDS: rows of up to 153600 logits stay on chip (149504 with the
  // entropy bonus, whose term needs two chunks' registers); longer rows read
  // their rest twice
  return fused_cached<ENT, ENT ? 54 : 56, 19, 2, AL>(T, s, args...);
}

hipError_t launch_logits_fused(const float* logits, const rft_tokens& tok, const TokMeta& m,
                               int64_t V, const float* old, const float* ref, const float* adv,
                               const LossConst& c, float* logp, float* ent, float* lse,
                               float* grad, float* dl, LossPartial* parts, LossPartial* parts2,
                               rft_ppo_stats* st, hipStream_t s) {
  hipError_t e = hipSuccess;
  int lp = 0;
  if (tok.T > 0 && (e = row_parts(tok.T, V, &lp)) != hipSuccess) return e;
  // the parts (12 bytes each) take the room of the T row partials and of the
  // one after them (workspaces are whole multiples of 256 bytes)
  while (lp > 0 && (tok.T << lp) * (int64_t)sizeof(RowStats) > (char*)parts2 - (char*)parts + 256) --lp;
  // few rows: k_logits_part does the bookkeeping (T <= 8 threads of a part)
  const bool few = lp > 0 && tok.n_seq <= kFewSeq && tok.T <= 8 * (lg::NT >> lp);
  if (!few && (e = launch_tokmeta(tok, m, s)) != hipSuccess) return e;
  if (few) {
    RowStats* const part = (RowStats*)parts;
    const unsigned nb = (unsigned)(tok.T << lp) + 1;
    if (lp == 3) lg::k_logits_part<8><<<nb, lg::NT / 8, 0, s>>>(logits, V, tok, m, part);
    else if (lp == 2) lg::k_logits_part<4><<<nb, lg::NT / 4, 0, s>>>(logits, V, tok, m, part);
    else lg::k_logits_part<2><<<nb, lg::NT / 2, 0, s>>>(logits, V, tok, m, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_few_terms(logits, tok, m, V, 1 << lp, old, ref, adv, c, logp, ent, lse, grad,
                              parts, st, s)) != hipSuccess)
      return e;
    const float* const terms = (const float*)parts;
    const bool bonus = c.ent_coef > 0.f;
    return launch_logits_bwd(logits, tok, V, terms, terms + tok.T, bonus ? terms + 2 * tok.T : nullptr,
                             bonus ? terms + 3 * tok.T : nullptr, dl, s);
  }
  const bool al = V % 4 == 0 && (((uintptr_t)logits | (uintptr_t)dl) & 15) == 0;
  for (int64_t t0 = 0; t0 < tok.T && e == hipSuccess; t0 += kLaunchRows) {
    const int64_t n = std::min(tok.T - t0, kLaunchRows);
    auto go = [&](auto k) {
      return k(logits + t0 * V, n, V, tok.mask + t0, tok.token_ids + t0, m.kidx + t0, m.row_seq,
               m.n_i, m.meta, old + t0, from(ref, t0), adv, c, logp + t0, from(ent, t0),
               from(lse, t0), from(grad, t0), dl + t0 * V, parts + t0);
    };
    if (V > ((int64_t)1 << 28)) {  // buffer descriptors span one row: 32-bit byte offsets
      e = go([&](auto... a) {
        lg::k_logits_fused<<<(unsigned)n, lg::NT, 0, s>>>(a...);
        return hipGetLastError();
      });
    } else if (c.ent_coef > 0.f) {
      e = al ? go([&](auto... a) { return fused_any<true, true>(V, n, s, a...); })
             : go([&](auto... a) { return fused_any<true, false>(V, n, s, a...); });
    } else {
      e = al ? go([&](auto... a) { return fused_any<false, true>(V, n, s, a...); })
             : go([&](auto... a) { return fused_any<false, false>(V, n, s, a...); });
    }
  }
  if (e != hipSuccess) return e;
  return launch_loss_reduce(parts, tok.T, parts2, m.meta, st, s);
}

}  // namespace rft
