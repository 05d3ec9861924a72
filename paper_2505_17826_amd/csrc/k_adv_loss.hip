// GRPO group advantages, the per-token PPO-clip/KL loss and the SFT loss with
// their fixed-order fp64 reduction, and the merge of the per-tile
// log-sum-exp partials into per-token log-prob / entropy / lse.
#include "rft_internal.h"

namespace rft {

// ---------------------------------------------------------- advantages ----
// GRPO (Sec. 3.2, Listing 4, advantage_fn "grpo"): one wavefront per group;
// mean and sample (or population) std by wavefront shuffles, computed in fp64.
__global__ void __launch_bounds__(256) k_group_adv(const float* __restrict__ r, int64_t n_groups,
                                                   int G, float eps, int unbiased,
                                                   float* __restrict__ adv) {
  int lane = threadIdx.x & 63;
  int64_t g = block_index() * 4 + (threadIdx.x >> 6);
  if (g >= n_groups) return;
  const float* rg = r + g * G;
  double s = 0.0;
  float mn = INFINITY, mx = -INFINITY;
  for (int j = lane; j < G; j += 64) {
    float v = rg[j];
    s += (double)v;
    mn = fminf(mn, v);
    mx = fmaxf(mx, v);
  }
  s = wave_sum_d(s);
  mn = wave_min_f(mn);
  mx = wave_max_f(mx);
  double mu = s / (double)G;
  double q = 0.0;
  for (int j = lane; j < G; j += 64) {
    double dv = (double)rg[j] - mu;
    q += dv * dv;
  }
  q = wave_sum_d(q);
  bool degenerate = (G < 2) || (mn == mx);
  double sd = degenerate ? 0.0 : sqrt(q / (double)(unbiased ? G - 1 : G));
  for (int j = lane; j < G; j += 64)
    adv[g * G + j] = degenerate ? 0.f : (float)(((double)rg[j] - mu) / (sd + (double)eps));
}

hipError_t launch_group_adv(const float* r, int64_t n_groups, int G, float eps, int unbiased,
                            float* adv, hipStream_t s) {
  if (n_groups > 0)
    k_group_adv<<<grid_xy((n_groups + 3) / 4), 256, 0, s>>>(r, n_groups, G, eps, unbiased, adv);
  return hipGetLastError();
}

// ------------------------------------------- advantages over group ids ----
// Explicit, variable-size groups (modes as rft_adv_mode), in work linear in
// the number of rollouts:
//   k_adv_count    count each group's rollouts (integer atomics: exact), and
//                  give 0 to rollouts whose id is outside [0, n_groups);
//   k_adv_scan_*   exclusive scan of the counts: group g's members go to
//                  mem[off[g] .. off[g + 1]);
//   k_adv_scatter  place each rollout index in its group's range (the order
//                  inside a range depends on the atomics);
//   k_adv_member_groups  one workgroup per group: sort the member indices
//                  (bitonic, in LDS), so the members are in index order
//                  whatever the scatter did, then fp64 sums over them in a
//                  fixed order and the advantages.  A group with more members
//                  than the LDS sort holds scans every id instead (members
//                  in index order as well), which only such large groups pay.
// Results are deterministic run to run.
template <typename Tv>
__device__ Tv block_sum256(Tv v, Tv* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}

__device__ float block_min256(float v, float* sh) {
  v = wave_min_f(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return fminf(fminf(sh[0], sh[1]), fminf(sh[2], sh[3]));
}

__device__ float block_max256(float v, float* sh) {
  v = wave_max_f(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

constexpr int kAdvScanBlock = 1024;  // counts per block of the scan (4 per thread)
constexpr int kAdvSortSmall = 256;   // members the small-group kernel sorts (1 KiB of LDS)
constexpr int kAdvSortCap = 16384;   // members the large-group kernel sorts (64 KiB)

__global__ void __launch_bounds__(256) k_adv_zero2(int32_t* __restrict__ a, int32_t* __restrict__ b,
                                                   int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) {
    a[i] = 0;
    b[i] = 0;
  }
}

__global__ void __launch_bounds__(256) k_adv_count(const int32_t* __restrict__ gid, int64_t n,
                                                   int64_t n_groups, int32_t* __restrict__ cnt,
                                                   float* __restrict__ adv) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int g = gid[i];
  if (g < 0 || (int64_t)g >= n_groups) adv[i] = 0.f;
  else atomicAdd(cnt + g, 1);
}

// Per block of kAdvScanBlock counts: the block's total.
__global__ void __launch_bounds__(256) k_adv_scan_totals(const int32_t* __restrict__ cnt,
                                                         int64_t ng, int32_t* __restrict__ tot) {
  __shared__ int shi[4];
  const int64_t b0 = (int64_t)blockIdx.x * kAdvScanBlock;
  int v = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t g = b0 + threadIdx.x * 4 + k;
    v += g < ng ? cnt[g] : 0;
  }
  v = block_sum256(v, shi);
  if (threadIdx.x == 0) tot[blockIdx.x] = v;
}

// Exclusive scan of one int per thread over the 256 threads of a block.
__device__ int block_excl_scan256(int v, int* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {
    const int add = threadIdx.x >= (unsigned)o ? sh[threadIdx.x - o] : 0;
    __syncthreads();
    sh[threadIdx.x] += add;
    __syncthreads();
  }
  const int incl = sh[threadIdx.x];
  __syncthreads();
  return incl - v;
}

// One block: exclusive scan of the block totals, in place.
__global__ void __launch_bounds__(256) k_adv_scan_top(int32_t* __restrict__ tot, int64_t nb) {
  __shared__ int sh[256];
  int carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += 256) {
    const int64_t b = b0 + threadIdx.x;
    const int v = b < nb ? tot[b] : 0;
    const int ex = block_excl_scan256(v, sh);
    if (b < nb) tot[b] = carry + ex;
    // the block's total: the last thread's exclusive value plus its own
    if (threadIdx.x == 255) sh[0] = ex + v;
    __syncthreads();
    carry += sh[0];
    __syncthreads();
  }
}

// off[g] = exclusive prefix of the counts; off[ng] = the total.
__global__ void __launch_bounds__(256) k_adv_scan_apply(const int32_t* __restrict__ cnt,
                                                        int64_t ng, const int32_t* __restrict__ tot,
                                                        int32_t* __restrict__ off) {
  __shared__ int sh[256];
  const int64_t b0 = (int64_t)blockIdx.x * kAdvScanBlock;
  int c[4], v = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t g = b0 + threadIdx.x * 4 + k;
    c[k] = g < ng ? cnt[g] : 0;
    v += c[k];
  }
  int run = tot[blockIdx.x] + block_excl_scan256(v, sh);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t g = b0 + threadIdx.x * 4 + k;
    if (g < ng) off[g] = run;
    run += c[k];
    if (g == ng - 1) off[ng] = run;
  }
}

__global__ void __launch_bounds__(256) k_adv_scatter(const int32_t* __restrict__ gid, int64_t n,
                                                     int64_t n_groups,
                                                     const int32_t* __restrict__ off,
                                                     int32_t* __restrict__ cur,
                                                     int32_t* __restrict__ mem) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int g = gid[i];
  if (g < 0 || (int64_t)g >= n_groups) return;
  mem[off[g] + atomicAdd(cur + g, 1)] = (int32_t)i;
}

// Advantage of reward v in a group with sum s, mean mu, std sd and G members.
__device__ __forceinline__ float adv_value(int mode, bool degenerate, double v, double s,
                                           double mu, double sd, double G, float eps) {
  if (degenerate) return 0.f;
  double a;
  if (mode == RFT_ADV_GRPO) a = (v - mu) / (sd + (double)eps);
  else if (mode == RFT_ADV_MEAN_CENTER) a = v - mu;
  else a = v - (s - v) / (G - 1.0);
  return (float)a;
}

// Few rollouts (at most kAdvFew): one launch instead of eight.  Every thread takes
// one rollout and walks all ids and rewards (in LDS) twice, adding its own group's
// in index order; the walk is kAdvFew long, past which the bucketed path is the
// faster one.  Whole call, walk against buckets: 128 rollouts 10 / 29 us, 256 14 / 29,
// 512 26 / 29, 640 32 / 29, 1024 48 / 29.
constexpr int kAdvFew = 512;
__global__ void __launch_bounds__(256) k_adv_few(const float* __restrict__ r,
                                                 const int32_t* __restrict__ gid, int n,
                                                 int64_t n_groups, int mode, float eps,
                                                 int unbiased, float* __restrict__ adv) {
  __shared__ __align__(16) int sg[kAdvFew];  // read four at a time
  __shared__ __align__(16) float sr[kAdvFew];
  const int n4 = (n + 3) & ~3;
  for (int j = threadIdx.x; j < n4; j += 256) {
    const int g = j < n ? gid[j] : -1;
    sg[j] = g >= 0 && (int64_t)g < n_groups ? g : -1;
    sr[j] = j < n ? r[j] : 0.f;
  }
  __syncthreads();
  const int i = (int)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int g = sg[i];
  if (g < 0) {
    adv[i] = 0.f;
    return;
  }
  double s = 0.0, q = 0.0;
  float mn = INFINITY, mx = -INFINITY;
  int G = 0;
  for (int j = 0; j < n4; j += 4) {
    const int4 gj = *(const int4*)(sg + j);
    const float4 vj = *(const float4*)(sr + j);
    auto take = [&](int gg, float v) {  // selects: a branch per element costs more
      const bool in = gg == g;
      s += in ? (double)v : 0.0;
      mn = in ? fminf(mn, v) : mn;
      mx = in ? fmaxf(mx, v) : mx;
      G += in ? 1 : 0;
    };
    take(gj.x, vj.x);
    take(gj.y, vj.y);
    take(gj.z, vj.z);
    take(gj.w, vj.w);
  }
  const double Gd = (double)G, mu = s / Gd;
  const bool degenerate = G < 2 || (mode == RFT_ADV_GRPO && mn == mx);
  double sd = 0.0;
  if (mode == RFT_ADV_GRPO && !degenerate) {
    for (int j = 0; j < n4; j += 4) {
      const int4 gj = *(const int4*)(sg + j);
      const float4 vj = *(const float4*)(sr + j);
      auto take = [&](int gg, float v) {
        const double dv = gg == g ? (double)v - mu : 0.0;
        q += dv * dv;
      };
      take(gj.x, vj.x);
      take(gj.y, vj.y);
      take(gj.z, vj.z);
      take(gj.w, vj.w);
    }
    sd = sqrt(q / (unbiased ? Gd - 1.0 : Gd));
  }
  adv[i] = adv_value(mode, degenerate, (double)sr[i], s, mu, sd, Gd, eps);
}

// Groups with LO < G <= CAP members sort them in LDS; with CAP = kAdvSortCap
// the kernel also takes the groups beyond it (by scanning the ids).  Two
// instantiations split the groups so that the many small ones run with little
// LDS per workgroup.
template <int LO, int CAP>
__global__ void __launch_bounds__(256) k_adv_member_groups(
    const float* __restrict__ r, const int32_t* __restrict__ gid, int64_t n, int64_t n_groups,
    const int32_t* __restrict__ off, const int32_t* __restrict__ mem, int mode, float eps,
    int unbiased, float* __restrict__ adv) {
  __shared__ int32_t key[CAP];
  __shared__ double shd[4];
  __shared__ float shf[4];
  if (block_index() >= n_groups) return;
  const int g = (int)block_index();
  const int64_t a0 = off[g];
  const int G = off[g + 1] - (int32_t)a0;
  if (G <= LO || (CAP < kAdvSortCap && G > CAP)) return;
  const int tid = threadIdx.x;
  double s = 0.0, q = 0.0;
  float mn = INFINITY, mx = -INFINITY;
  if (G <= CAP) {
    int P = 1;
    while (P < G) P <<= 1;
    for (int k = tid; k < P; k += 256) key[k] = k < G ? mem[a0 + k] : 0x7fffffff;
    __syncthreads();
    // bitonic sort of key[0, P) ascending
    for (int size = 2; size <= P; size <<= 1) {
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int k = tid; k < P / 2; k += 256) {
          const int lo = 2 * k - (k & (stride - 1));
          const int hi = lo + stride;
          const bool up = (lo & size) == 0;
          const int x = key[lo], y = key[hi];
          if ((x > y) == up) {
            key[lo] = y;
            key[hi] = x;
          }
        }
        __syncthreads();
      }
    }
    for (int k = tid; k < G; k += 256) {
      const float v = r[key[k]];
      s += (double)v;
      mn = fminf(mn, v);
      mx = fmaxf(mx, v);
    }
  } else {
    for (int64_t i = tid; i < n; i += 256) {
      if (gid[i] != g) continue;
      const float v = r[i];
      s += (double)v;
      mn = fminf(mn, v);
      mx = fmaxf(mx, v);
    }
  }
  s = block_sum256(s, shd);
  mn = block_min256(mn, shf);
  mx = block_max256(mx, shf);
  const double Gd = (double)G, mu = s / Gd;
  const bool degenerate = G < 2 || (mode == RFT_ADV_GRPO && mn == mx);
  double sd = 0.0;
  if (mode == RFT_ADV_GRPO && !degenerate) {
    if (G <= CAP) {
      for (int k = tid; k < G; k += 256) {
        const double dv = (double)r[key[k]] - mu;
        q += dv * dv;
      }
    } else {
      for (int64_t i = tid; i < n; i += 256) {
        if (gid[i] != g) continue;
        const double dv = (double)r[i] - mu;
        q += dv * dv;
      }
    }
    q = block_sum256(q, shd);
    sd = sqrt(q / (unbiased ? Gd - 1.0 : Gd));
  }
  if (G <= CAP) {
    for (int k = tid; k < G; k += 256) {
      const int i = key[k];
      adv[i] = adv_value(mode, degenerate, (double)r[i], s, mu, sd, Gd, eps);
    }
  } else {
    for (int64_t i = tid; i < n; i += 256)
      if (gid[i] == g) adv[i] = adv_value(mode, degenerate, (double)r[i], s, mu, sd, Gd, eps);
  }
}

AdvIdsWs carve_adv_ids(Carver& c, int64_t n, int64_t n_groups) {
  AdvIdsWs w;
  const int64_t ng = n_groups > 0 ? n_groups : 1;
  w.cnt = c.take<int32_t>((size_t)ng);
  w.cur = c.take<int32_t>((size_t)ng);
  w.off = c.take<int32_t>((size_t)ng + 1);
  w.tot = c.take<int32_t>((size_t)((ng + kAdvScanBlock - 1) / kAdvScanBlock));
  w.mem = c.take<int32_t>((size_t)(n > 0 ? n : 1));
  return w;
}

hipError_t launch_group_adv_ids(const float* r, const int32_t* gid, int64_t n, int64_t n_groups,
                                int mode, float eps, int unbiased, float* adv, const AdvIdsWs& w,
                                hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n <= kAdvFew) {
    k_adv_few<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(r, gid, (int)n, n_groups, mode, eps,
                                                          unbiased, adv);
    return hipGetLastError();
  }
  const unsigned nbn = (unsigned)((n + 255) / 256);
  if (n_groups > 0)
    k_adv_zero2<<<(unsigned)((n_groups + 255) / 256), 256, 0, s>>>(w.cnt, w.cur, n_groups);
  k_adv_count<<<nbn, 256, 0, s>>>(gid, n, n_groups, w.cnt, adv);
  if (n_groups == 0) return hipGetLastError();
  const int64_t nbs = (n_groups + kAdvScanBlock - 1) / kAdvScanBlock;
  k_adv_scan_totals<<<(unsigned)nbs, 256, 0, s>>>(w.cnt, n_groups, w.tot);
  k_adv_scan_top<<<1, 256, 0, s>>>(w.tot, nbs);
  k_adv_scan_apply<<<(unsigned)nbs, 256, 0, s>>>(w.cnt, n_groups, w.tot, w.off);
  k_adv_scatter<<<nbn, 256, 0, s>>>(gid, n, n_groups, w.off, w.cur, w.mem);
  k_adv_member_groups<0, kAdvSortSmall><<<grid_xy(n_groups), 256, 0, s>>>(
      r, gid, n, n_groups, w.off, w.mem, mode, eps, unbiased, adv);
  k_adv_member_groups<kAdvSortSmall, kAdvSortCap><<<grid_xy(n_groups), 256, 0, s>>>(
      r, gid, n, n_groups, w.off, w.mem, mode, eps, unbiased, adv);
  return hipGetLastError();
}

// -------------------------------------------------------- loss reduction ----
// The loss kernels run at most kLossBlocks blocks of kLossThreads threads, up to
// kLossRows rows of a thread in flight at a time.  What bounds a loss call is
// the chain of dependent steps (compaction index, rollout, its counts, the fp64
// terms, the sums), not its bytes: few waves, since each pays for the eleven
// sums, and few blocks, since each one's arrival at the final sum costs an L2
// write-back (1024 blocks took 31 us).
constexpr int kLossThreads = 256, kLossBlocks = 256, kLossRows = 4;
static int loss_blocks(int64_t T) {
  const int64_t nb = (T + kLossThreads - 1) / kLossThreads;
  return (int)(nb < 1 ? 1 : (nb > kLossBlocks ? kLossBlocks : nb));
}

// The fields of a partial as eight doubles and three integers.
constexpr int kFields = 11, kDoubles = 8;
static_assert(sizeof(LossPartial) == kFields * 8 && sizeof(long long) == 8, "fields of 8 bytes");

__device__ __forceinline__ void add_partial(LossPartial& p, const LossPartial& q) {
  p.loss += q.loss; p.pg += q.pg; p.klw += q.klw; p.kl += q.kl;
  p.ent += q.ent; p.ratio += q.ratio; p.sft += q.sft; p.entw += q.entw;
  p.clipped += q.clipped; p.bad += q.bad; p.expert += q.expert;
}

// Sum over the block in a fixed order: thread f < kFields returns field f's bits.
__device__ __forceinline__ long long block_total(LossPartial p, LossPartial* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, f = threadIdx.x;
  p.loss = wave_sum_d(p.loss);
  p.pg = wave_sum_d(p.pg);
  p.klw = wave_sum_d(p.klw);
  p.kl = wave_sum_d(p.kl);
  p.ent = wave_sum_d(p.ent);
  p.ratio = wave_sum_d(p.ratio);
  p.sft = wave_sum_d(p.sft);
  p.entw = wave_sum_d(p.entw);
  p.clipped = wave_sum_i((int)p.clipped);  // counts of at most T <= 2^30 rows
  p.bad = wave_sum_i((int)p.bad);
  p.expert = wave_sum_i((int)p.expert);
  __syncthreads();  // sh may still be read from a previous sum
  if (lane == 0) sh[w] = p;
  __syncthreads();
  long long bits = 0;
  if (f < kDoubles) {
    double d = 0.0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) d += ((const double*)(sh + i))[f];
    bits = __double_as_longlong(d);
  } else if (f < kFields) {
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) bits += ((const long long*)(sh + i))[f];
  }
  return bits;
}

__device__ void write_stats(const LossPartial& t, const int32_t* meta, rft_ppo_stats* st,
                            int sft_only) {
  const int N = meta[0], S = meta[1], Ne = meta[2], Ng = N - Ne;
  const double inv = N > 0 ? 1.0 / (double)N : 0.0;
  const double invg = Ng > 0 ? 1.0 / (double)Ng : 0.0;
  st->loss = N > 0 ? t.loss : 0.0;
  st->pg_loss = N > 0 ? t.pg : 0.0;
  st->kl_loss = N > 0 ? t.klw : 0.0;
  st->kl_mean = t.kl * invg;
  st->entropy_mean = t.ent * inv;
  st->ratio_mean = t.ratio * invg;
  st->clipfrac = (double)t.clipped * invg;
  st->n_valid = N;
  st->n_seq_valid = S;
  st->n_clipped = t.clipped;
  st->n_bad_ids = t.bad;
  st->sft_loss = sft_only ? (N > 0 ? t.loss : 0.0) : (Ne > 0 ? t.sft / (double)Ne : 0.0);
  st->n_expert = Ne;
  st->entropy_loss = N > 0 ? t.entw : 0.0;
}

// The stats from every block's partial (all threads of every block call this
// last).  Each block's sum goes to parts[blockIdx.x]; the last block to arrive
// (an atomic count, which launch_tokmeta has set to 0; the fences make every
// block's sum visible to it) adds them in index order, so the result does not
// depend on which block that is.  One launch of a single workgroup less (8-9 us).
__device__ void reduce_stats(const LossPartial& p, LossPartial* parts, int32_t* meta,
                             rft_ppo_stats* st, int sft_only) {
  __shared__ LossPartial sh[kLossThreads / 64];
  __shared__ LossPartial tot;
  __shared__ int last;
  const int f = threadIdx.x;
  long long bits = block_total(p, sh);
  if (gridDim.x > 1) {
    if (f < kFields) {
      ((long long*)(parts + blockIdx.x))[f] = bits;
      __threadfence();
    }
    if (f == 0) last = atomicAdd(meta + kMetaCounter, 1) == (int)gridDim.x - 1 ? 1 : 0;
    __syncthreads();
    if (!last) return;
    __threadfence();
    LossPartial q = RFT_ZERO_PARTIAL;
    if (f < (int)gridDim.x) q = parts[f];
    bits = block_total(q, sh);
  }
  if (f < kFields) ((long long*)&tot)[f] = bits;
  __syncthreads();
  if (f == 0) write_stats(tot, meta, st, sft_only);
}

// Per-token loss over rows [0, T).
__global__ void __launch_bounds__(kLossThreads) k_loss_fwd(
    const int32_t* __restrict__ ids, const int32_t* __restrict__ kidx,
    const int32_t* __restrict__ row_seq, const int32_t* __restrict__ n_i, int32_t* meta,
    int64_t T, const float* __restrict__ logp,
    const float* __restrict__ old, const float* __restrict__ ref, const float* __restrict__ adv,
    const float* __restrict__ ent, LossConst c, float* __restrict__ grad,
    float* __restrict__ egrad, LossPartial* parts, rft_ppo_stats* __restrict__ st) {
  LossPartial p = RFT_ZERO_PARTIAL;
  const int64_t step = (int64_t)gridDim.x * kLossThreads;
  for (int64_t t0 = (int64_t)blockIdx.x * kLossThreads + threadIdx.x; t0 < T; t0 += kLossRows * step) {
    int k[kLossRows], i[kLossRows], y[kLossRows], n[kLossRows];
    float lp[kLossRows], od[kLossRows], rf[kLossRows], A[kLossRows], en[kLossRows];
    bool ex[kLossRows];
#pragma unroll
    for (int u = 0; u < kLossRows; ++u) {
      const int64_t t = t0 + u * step;
      k[u] = t < T ? kidx[t] : -1;
    }
#pragma unroll
    for (int u = 0; u < kLossRows; ++u) {
      const int64_t t = k[u] < 0 ? t0 : t0 + u * step;
      i[u] = k[u] < 0 ? 0 : row_seq[k[u]];
      y[u] = ids[t];
      lp[u] = logp[t];
      od[u] = old[t];
      rf[u] = ref ? ref[t] : lp[u];
      en[u] = ent ? ent[t] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kLossRows; ++u) {
      n[u] = n_i[i[u]];
      A[u] = adv[i[u]];
      ex[u] = c.is_expert && c.is_expert[i[u]];
    }
#pragma unroll
    for (int u = 0; u < kLossRows; ++u) {
      const int64_t t = t0 + u * step;
      if (t >= T) break;
      float gout = 0.f, eout = 0.f;
      if (k[u] >= 0) {
        if (y[u] < 0 || (int64_t)y[u] >= c.V) {
          p.bad += 1;
        } else {
          LossPartial q = RFT_ZERO_PARTIAL;
          gout = row_loss(lp[u], od[u], rf[u], A[u], n[u], ex[u], meta, (double)en[u], c, q, &eout);
          add_partial(p, q);
        }
      }
      grad[t] = gout;
      if (egrad) egrad[t] = eout;
    }
  }
  reduce_stats(p, parts, meta, st, 0);
}

// Sum of per-row partials.
__global__ void __launch_bounds__(kLossThreads) k_loss_reduce(const LossPartial* __restrict__ parts,
                                                              int64_t n, LossPartial* out,
                                                              int32_t* meta,
                                                              rft_ppo_stats* __restrict__ st) {
  LossPartial p = RFT_ZERO_PARTIAL;
  for (int64_t i = (int64_t)blockIdx.x * kLossThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kLossThreads)
    add_partial(p, parts[i]);
  reduce_stats(p, out, meta, st, 0);
}

hipError_t launch_loss_reduce(const LossPartial* parts, int64_t n, LossPartial* tmp, int32_t* meta,
                              rft_ppo_stats* stats, hipStream_t s) {
  k_loss_reduce<<<loss_blocks(n), kLossThreads, 0, s>>>(parts, n, tmp, meta, stats);
  return hipGetLastError();
}

// A handful of rows (at most kLossThreads) whose statistics are in P parts each:
// the merge, the row terms and the loss statistics in one workgroup.  Every part is read before the terms (lse, c, e, entropy, [T] each)
// take its place.
template <int P>
__global__ void __launch_bounds__(kLossThreads) k_few_terms(
    const float* __restrict__ logits, const rft_tokens tok, TokMeta m, int64_t V,
    const float* __restrict__ old, const float* __restrict__ ref, const float* __restrict__ adv,
    LossConst c, float* __restrict__ logp, float* __restrict__ ent, float* __restrict__ lse,
    float* __restrict__ grad, float* scratch, rft_ppo_stats* __restrict__ st) {
  const int t = threadIdx.x, T = (int)tok.T;
  const bool on = t < T && tok.mask[t];
  RowStats v[P];
#pragma unroll
  for (int i = 0; i < P; ++i)
    v[i] = on ? ((const RowStats*)scratch)[t * P + i] : RowStats{0.f, 1.f, 0.f};
  int y = on ? tok.token_ids[t] : -1;
  const int i = on ? m.row_seq[m.kidx[t]] : 0;
  const float A = on ? adv[i] : 0.f;
  const int n = on ? m.n_i[i] : 0;
  const bool ok = y >= 0 && (int64_t)y < V;
  const float zy = ok ? logits[(int64_t)t * V + y] : 0.f;
  const float od = on ? old[t] : 0.f, rf0 = on && ref ? ref[t] : 0.f;
  __syncthreads();  // every part is read
  LossPartial p = RFT_ZERO_PARTIAL;
  if (t < T) {
    float L = 0.f, H = 0.f, lp = 0.f, g = 0.f, e = 0.f;
    if (on) {
      tree_merge(v);
      L = v[0].m + logf(v[0].s);
      H = L - v[0].u / v[0].s;
      lp = ok ? zy - L : __int_as_float(0x7fc00000);
      if (!ok) {
        p.bad = 1;
      } else {
        const bool ex = c.is_expert && c.is_expert[i];
        g = row_loss(lp, od, ref ? rf0 : lp, A, n, ex, m.meta, (double)H, c, p, &e);
      }
    }
    logp[t] = lp;
    if (ent) ent[t] = H;
    if (lse) lse[t] = L;
    if (grad) grad[t] = g;
    scratch[t] = L;
    scratch[T + t] = g;
    scratch[2 * T + t] = e;
    scratch[3 * T + t] = H;
  }
  reduce_stats(p, nullptr, m.meta, st, 0);
}

hipError_t launch_few_terms(const float* logits, const rft_tokens& tok, const TokMeta& m, int64_t V,
                            int P, const float* old, const float* ref, const float* adv,
                            const LossConst& c, float* logp, float* ent, float* lse, float* grad,
                            void* scratch, rft_ppo_stats* st, hipStream_t s) {
  if (tok.T > kLossThreads) return hipErrorInvalidValue;
  auto k = P == 8 ? k_few_terms<8> : P == 4 ? k_few_terms<4> : k_few_terms<2>;
  k<<<1, kLossThreads, 0, s>>>(logits, tok, m, V, old, ref, adv, c, logp, ent, lse, grad,
                               (float*)scratch, st);
  return hipGetLastError();
}

// SFT loss of the train-only mode: sum_t w_t (-logp_t) over the valid rows
// whose id is in range, w_t the aggregation weight; grad = -w_t.
__global__ void __launch_bounds__(kLossThreads) k_sft_fwd(
    const int32_t* __restrict__ ids, const int32_t* __restrict__ kidx,
    const int32_t* __restrict__ row_seq, const int32_t* __restrict__ n_i, int32_t* meta, int64_t T,
    int64_t V, const float* __restrict__ logp, int agg, double denom, float* __restrict__ grad,
    LossPartial* parts, rft_ppo_stats* __restrict__ st) {
  LossPartial p = RFT_ZERO_PARTIAL;
  for (int64_t t = (int64_t)blockIdx.x * kLossThreads + threadIdx.x; t < T;
       t += (int64_t)gridDim.x * kLossThreads) {
    const int k = kidx[t];
    float g = 0.f;
    if (k >= 0) {
      const int y = ids[t];
      if (y < 0 || (int64_t)y >= V) {
        p.bad += 1;
      } else {
        const double w = agg_weight(agg, denom, n_i[row_seq[k]], meta[0], meta[1]);
        p.loss += w * -(double)logp[t];
        g = (float)-w;
      }
    }
    grad[t] = g;
  }
  reduce_stats(p, parts, meta, st, 1);
}

hipError_t launch_sft_fwd(const rft_tokens& tok, const TokMeta& m, int64_t V, const float* logp,
                          int agg, double denom, float* grad, LossPartial* parts,
                          rft_ppo_stats* st, hipStream_t s) {
  k_sft_fwd<<<loss_blocks(tok.T), kLossThreads, 0, s>>>(tok.token_ids, m.kidx, m.row_seq, m.n_i,
                                                        m.meta, tok.T, V, logp, agg, denom, grad,
                                                        parts, st);
  return hipGetLastError();
}

hipError_t launch_loss_fwd(const rft_tokens& tok, const TokMeta& m, const float* logp,
                           const float* old, const float* ref, const float* adv, const float* ent,
                           const LossConst& c, float* grad, float* egrad, LossPartial* parts,
                           rft_ppo_stats* st, hipStream_t s) {
  k_loss_fwd<<<loss_blocks(tok.T), kLossThreads, 0, s>>>(tok.token_ids, m.kidx, m.row_seq, m.n_i,
                                                         m.meta, tok.T, logp, old, ref, adv, ent, c,
                                                         grad, egrad, parts, st);
  return hipGetLastError();
}

// -------------------------------------------------------- lse partials ----
// Merge the per-vocabulary-tile partials (m, s, u) of each valid row into
// lse, entropy = lse - u/s and logp = z_y - lse; masked rows get 0.
// parts are [ntiles][ld] with the compacted row index as the inner index.
__global__ void __launch_bounds__(kMergeThreads) k_merge_rows(
    const int32_t* __restrict__ kidx, const int32_t* __restrict__ ids, int64_t T, int64_t V,
    const float* __restrict__ pm, const float* __restrict__ ps, const float* __restrict__ pu,
    int ntiles, int64_t ld, const float* __restrict__ zy, float* __restrict__ logp,
    float* __restrict__ ent, float* __restrict__ lse) {
  __shared__ RowStats sh[kMergeThreads];
  const int64_t t = block_index() * kMergeRows + threadIdx.x % kMergeRows;
  const int k = t < T ? kidx[t] : -1;
  const RowStats r = merge_tiles(pm + (k < 0 ? 0 : k), ps + (k < 0 ? 0 : k), pu + (k < 0 ? 0 : k), ld,
                               ntiles, k >= 0, sh);
  if (threadIdx.x >= kMergeRows || t >= T) return;
  if (k < 0) {
    logp[t] = 0.f;
    if (ent) ent[t] = 0.f;
    lse[t] = 0.f;
    return;
  }
  float L = r.m + logf(r.s);
  lse[t] = L;
  if (ent) ent[t] = L - r.u / r.s;
  int y = ids[t];
  logp[t] = (y >= 0 && (int64_t)y < V) ? zy[k] - L : __int_as_float(0x7fc00000);
}

hipError_t launch_merge_rows(const rft_tokens& tok, const TokMeta& m, int64_t V, const float* pm,
                             const float* ps, const float* pu, int ntiles, int64_t ld,
                             const float* zy, float* logp, float* ent, float* lse, hipStream_t s) {
  const int64_t nb = (tok.T + kMergeRows - 1) / kMergeRows;
  if (nb > 0)
    k_merge_rows<<<grid_xy(nb), kMergeThreads, 0, s>>>(m.kidx, tok.token_ids, tok.T, V, pm, ps, pu,
                                                       ntiles, ld, zy, logp, ent, lse);
  return hipGetLastError();
}

}  // namespace rft
