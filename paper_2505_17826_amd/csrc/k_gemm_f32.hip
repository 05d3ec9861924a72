// fp32 GEMM core of the policy head (hidden and weight given in fp32) on the
// fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32 products, fp32
// accumulation, 256 flops per clock and CU):
//   C[m, n] = sum_k A(m, k) B(n, k)
// Each operand is either K-contiguous (element (r, k) = p[row(r) ld + k], the
// rows optionally through a map) or row-contiguous (element (r, k) =
// p[row(k) ld + r], the K rows optionally through a map), so the forward and
// the recompute (H rows by the map, W), dH (dZ, W as stored) and dW (dZ and the
// H rows as stored) run without transposed copies.
//
// What bounds it: the matrix pipe.  A 128 x 128 tile takes 4096 matrix clocks
// per SIMD and K step of 32 and reads 16 KiB of fragments per wave in that
// time, so LDS and L2 stay far below their rates; what is left is to keep
// enough independent work per SIMD.  256 threads, four waves: 2 x 2 waves of 64 x 64 (128 x 128
// tile, 16 accumulator tiles per wave) or 4 x 1 waves of 16 x 64 (64 x 64 tile)
// where the larger tile would leave CUs idle (tile128).  K steps of 32 go
// through registers into one of two LDS stages (the next step's loads are in
// flight during the products; one barrier per step), and the fragments of
// four K are read while the previous four's products run.  Measured (one pass
// of forward, recompute, dH and dW; 1527 of 2048 rows valid, d = 1024, V =
// 32000): 13.7-14.6 ms with the 64 x 64 vector-FMA tiles this replaces, 3.5-3.8 ms
// now on the same cards; the products run at 95-110 TFLOP/s, the matrix pipe 60-68%
// busy at 2.2-2.4 GHz
// (rocBLAS's largest fp32 product on the same card: 153).  Eight waves of 32 x 64
// per tile and a wave priority by workgroup changed nothing.
//
// The epilogues take the library's exponential: the hardware exp2 of the rounded
// x log2(e) would save 1% of a step (3.32 against 3.35 ms, 2048 rows, d = 1024, V =
// 32000) but is off by up to 15 half-ulps at x = -15, all with one sign.
//
// LDS stage: element (r, k) of an operand tile at k BT + (r ^ swz(k)).  Fragment
// reads (16 rows at four consecutive k), the four-byte writes of a
// K-contiguous operand (8 rows at eight k of the same k % 4) and the 16-byte
// writes of a row-contiguous one each touch every bank once.
#include <algorithm>

#include "rft_internal.h"

namespace rft {
namespace f3 {

constexpr int BK = 32, NT = 256;
enum { EPI_STATS = 0, EPI_DZ = 1, EPI_STORE = 2 };

// unaligned 16-byte access (fp32 rows need only 4-byte alignment)
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

struct Operand {
  const float* p;
  int64_t ld;
  const int32_t* map;  // row map (rows of a K-contiguous operand, K rows otherwise) or nullptr
  int64_t moff;        // first entry of the map
};

struct Args {
  Operand A, B;
  int M, N, K;
  int NB;  // rows of B that exist (read only for n < NB; 0 = N)
  const int32_t* cnt; int64_t cnt_off, cnt_cap; int m_from_cnt, k_from_cnt;
  const int32_t* rows; int64_t rows_off;
  const int32_t* ids; const float* lse; const float* cgrad;
  const float* egrad; const float* ent;  // EPI_DZ entropy bonus (egrad nullptr = none)
  float* pm; float* ps; float* pu; int64_t ldp; float* zy;
  float* dz; int64_t ldz; int64_t Vvalid;
  float* C; int64_t ldc; int accumulate; int c_scatter;
  // EPI_STORE over splits of K: slice s = blockIdx.y covers K [s kper, s kper +
  // kper) and stores its sum to part + s part_ld (rows of N, compact); 0 = no split.
  // SEQ: one workgroup walks the slices and adds their sums itself (part unused)
  int kper; float* part; int64_t part_ld;
};

__device__ __forceinline__ int swz(int k) { return 16 * ((k + (k >> 2)) & 3) ^ 8 * ((k >> 4) & 1); }

// Tile loader of a K-contiguous operand: lane l of wave w holds K chunk l / 8
// (four values) of rows 8 w + l % 8 + 32 it.  Rows past the end read the last
// row (they reach only rows or columns of C that are not stored).
template <int BT>
struct LoadK {
  static constexpr int NI = BT / 32;
  const float* q[NI];
  int row, kc;
  __device__ __forceinline__ void start(const Operand& o, int r0, int R, int k0, int) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    row = w * 8 + (lane & 7);
    kc = lane >> 3;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int r = min(r0 + row + it * 32, R - 1);
      q[it] = o.p + (o.map ? (int64_t)o.map[o.moff + r] : (int64_t)r) * o.ld + k0 + kc * 4;
    }
  }
  // whole K step inside K
  __device__ __forceinline__ bool whole(int k0, int K) const { return k0 + BK <= K; }
  __device__ __forceinline__ void load(const Operand&, int, int, floatx4 (&v)[NI]) {
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      v[it] = (floatx4)(*(const f4u*)q[it]);
      q[it] += BK;
    }
  }
  __device__ __forceinline__ void load_edge(const Operand&, int k0, int K, floatx4 (&v)[NI]) {
#pragma unroll
    for (int it = 0; it < NI; ++it) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[it][e] = k0 + kc * 4 + e < K ? q[it][e] : 0.f;
      q[it] += BK;
    }
  }
  __device__ __forceinline__ void put(float* s, const floatx4 (&v)[NI]) const {
#pragma unroll
    for (int it = 0; it < NI; ++it)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = kc * 4 + e;
        s[k * BT + ((row + it * 32) ^ swz(k))] = v[it][e];
      }
  }
};

// Tile loader of a row-contiguous operand: thread t holds four consecutive
// rows of K row t / (BT / 4) + it (1024 / BT).  The map entries are read one
// step ahead of the rows they name.
template <int BT>
struct LoadR {
  static constexpr int NI = BT / 32, PER = 1024 / BT;
  int64_t src[NI];
  int r4, kr, rbase, Rn;
  __device__ __forceinline__ void idx(const Operand& o, int k0, int K) {
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int k = min(k0 + kr + it * PER, K - 1);
      src[it] = o.map ? (int64_t)o.map[o.moff + k] : (int64_t)k;
    }
  }
  __device__ __forceinline__ void start(const Operand& o, int r0, int R, int k0, int K) {
    r4 = (threadIdx.x % (BT / 4)) * 4;
    kr = threadIdx.x / (BT / 4);
    rbase = r0 + r4;
    Rn = R;
    idx(o, k0, K);
  }
  // whole K step inside K and whole tile inside the rows
  __device__ __forceinline__ bool whole(int k0, int K) const {
    return k0 + BK <= K && rbase - r4 + BT <= Rn;
  }
  __device__ __forceinline__ void load(const Operand& o, int k0, int K, floatx4 (&v)[NI]) {
#pragma unroll
    for (int it = 0; it < NI; ++it)
      v[it] = (floatx4)(*(const f4u*)(o.p + src[it] * o.ld + rbase));
    idx(o, k0 + BK, K);
  }
  __device__ __forceinline__ void load_edge(const Operand& o, int k0, int K, floatx4 (&v)[NI]) {
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const bool kv = k0 + kr + it * PER < K;
      const float* q = o.p + src[it] * o.ld + rbase;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[it][e] = kv && rbase + e < Rn ? q[e] : 0.f;
    }
    idx(o, k0 + BK, K);
  }
  __device__ __forceinline__ void put(float* s, const floatx4 (&v)[NI]) const {
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int k = kr + it * PER;
      *(floatx4*)(s + k * BT + (r4 ^ swz(k))) = v[it];
    }
  }
};

template <int BT, bool KC> struct Load : LoadK<BT> {};
template <int BT> struct Load<BT, false> : LoadR<BT> {};

// MIA = 4: 128 x 128 tile; MIA = 1: 64 x 64.  AKC / BKC: operand K-contiguous.
// SEQ: the slices of K in turn, each from zero, their sums added in order: the
// bits of the split launch and k_sum_slices, with no room for partial sums
// (64 x 64 tile only: a second set of a 128 x 128 tile's sums does not fit).
template <int EPI, int MIA, bool AKC, bool BKC, bool SEQ = false>
__global__ void __launch_bounds__(NT, 2) k_gemm_f32(const Args g) {
  static_assert(!SEQ || MIA == 1, "see above");
  constexpr int BT = MIA == 4 ? 128 : 64;
  constexpr int WN = BT / 64;  // waves along N, 64 columns each
  constexpr int NR = MIA * 4;  // rows per lane
  // steps whose loads are in flight: the small tile's products (1024 clocks per
  // step) are shorter than a load
  constexpr int PF = MIA == 4 ? 1 : 2;
  __shared__ __attribute__((aligned(16))) float lds[2][2][BK * BT];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (w / WN) * (MIA * 16), wn = (w % WN) * 64;
  const int r16 = lane & 15, q4 = lane >> 4;
  int M = g.M, K = g.K;
  if (g.cnt) {
    int64_t c = (int64_t)g.cnt[0] - g.cnt_off;
    c = c < 0 ? 0 : (c > g.cnt_cap ? g.cnt_cap : c);
    if (g.m_from_cnt) M = (int)c;
    if (g.k_from_cnt) K = (int)c;
  }
  const int N = g.N, NB = g.NB > 0 ? g.NB : N;
  if (EPI == EPI_STORE && g.k_from_cnt && K == 0 && g.accumulate) return;
  // Workgroup b runs on XCD b % 8; each XCD takes a contiguous run of tiles,
  // the dimension with fewer tiles first, so that the larger operand's panel
  // is read by one XCD.
  const int nTm = (M + BT - 1) / BT, nTn = (N + BT - 1) / BT;
  const int64_t tiles = (int64_t)nTm * nTn, per = (tiles + 7) / 8;
  const int64_t b = (int64_t)blockIdx.z * gridDim.x + blockIdx.x;
  const int64_t t = (b & 7) * per + (b >> 3);
  if ((b >> 3) >= per || t >= tiles) return;
  const bool mfast = nTm <= nTn;
  const int mt = (int)(mfast ? t % nTm : t / nTn), nt = (int)(mfast ? t / nTm : t % nTn);
  const int m0 = mt * BT, n0 = nt * BT;
  int k0 = 0, k1 = K;
  const bool split = EPI == EPI_STORE && !SEQ && g.kper > 0;
  if (split) {
    k0 = (int)blockIdx.y * g.kper;
    k1 = k0 + g.kper < K ? k0 + g.kper : K;
  }

  floatx4 acc[MIA][4];
#pragma unroll
  for (int i = 0; i < MIA; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
  floatx4 tot[SEQ ? MIA : 1][SEQ ? 4 : 1];  // SEQ: the sum of the slices before this one
  if constexpr (SEQ) {
#pragma unroll
    for (int i = 0; i < MIA; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) tot[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
  }
  int kend = SEQ ? g.kper : 0;  // end of the slice (whole K steps)
  Load<BT, AKC> la;
  Load<BT, BKC> lb;
  if (k0 < k1) {
    la.start(g.A, m0, M, k0, k1);
    lb.start(g.B, n0, NB, k0, k1);
  }
  floatx4 va[PF][Load<BT, AKC>::NI], vb[PF][Load<BT, BKC>::NI];
  auto fetch = [&](int k, int p) {
    if (la.whole(k, k1)) la.load(g.A, k, k1, va[p]); else la.load_edge(g.A, k, k1, va[p]);
    if (lb.whole(k, k1)) lb.load(g.B, k, k1, vb[p]); else lb.load_edge(g.B, k, k1, vb[p]);
  };
#pragma unroll
  for (int p = 0; p < PF; ++p)
    if (k0 + p * BK < k1) fetch(k0 + p * BK, p);
  for (int kb = k0; kb < k1; kb += PF * BK) {
#pragma unroll
   for (int p = 0; p < PF; ++p) {
    const int k = kb + p * BK;
    if (k >= k1) break;
    if constexpr (SEQ) {
      if (k == kend) {
        kend += g.kper;
#pragma unroll
        for (int i = 0; i < MIA; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            tot[i][j] += acc[i][j];
            acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
          }
      }
    }
    const int st = PF == 1 ? ((k - k0) / BK) & 1 : p & 1;
    la.put(lds[st][0], va[p]);
    lb.put(lds[st][1], vb[p]);
    // this step's stage is complete; the other one is free once every wave is
    // past its products, i.e. at the next step's barrier
    __syncthreads();
    if (k + PF * BK < k1) fetch(k + PF * BK, p);
    const float* As = lds[st][0];
    const float* Bs = lds[st][1];
    // the fragments of four K are read while the previous four's products run
    float a[2][MIA], b[2][4];
    auto frag = [&](int kg, float (&fa)[MIA], float (&fb)[4]) {
      const int kk = kg * 4 + q4;
      const int x = 16 * ((q4 + kg) & 3) ^ 8 * (kg >> 2);  // swz(kk)
#pragma unroll
      for (int i = 0; i < MIA; ++i) fa[i] = As[kk * BT + ((wm + i * 16 + r16) ^ x)];
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[j] = Bs[kk * BT + ((wn + j * 16 + r16) ^ x)];
    };
    frag(0, a[0], b[0]);
#pragma unroll
    for (int kg = 0; kg < BK / 4; ++kg) {
      if (kg + 1 < BK / 4) frag(kg + 1, a[(kg + 1) & 1], b[(kg + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MIA; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kg & 1][i], b[kg & 1][j], acc[i][j],
                                                           0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
   }
  }

  if constexpr (SEQ) {
#pragma unroll
    for (int i = 0; i < MIA; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = tot[i][j] + acc[i][j];
  }

  // lane (r16, q4) holds rows m0 + wm + 16 i + 4 q4 + q, columns n0 + wn + 16 j + r16
  if constexpr (EPI == EPI_STATS) {
    // partials of this wave's 64 columns: one entry per row and 64-column group
    float mx[NR], sm[NR], um[NR];
#pragma unroll
    for (int e = 0; e < NR; ++e) {
      mx[e] = -INFINITY;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (n0 + wn + j * 16 + r16 < N) mx[e] = fmaxf(mx[e], acc[e >> 2][j][e & 3]);
    }
    row16_max_n(mx);
#pragma unroll
    for (int e = 0; e < NR; ++e) {
      const int m = m0 + wm + (e >> 2) * 16 + q4 * 4 + (e & 3);
      const int y = m < M ? g.ids[g.rows[g.rows_off + m]] : -1;
      sm[e] = um[e] = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = n0 + wn + j * 16 + r16;
        const float z = acc[e >> 2][j][e & 3];
        if (n < N) {
          const float p = expf(z - mx[e]);
          sm[e] += p;
          um[e] += p * z;
          if (n == y) g.zy[g.rows_off + m] = z;
        }
      }
    }
    row16_sum_n(sm);
    row16_sum_n(um);
    // lane r16 owns row e = r16 of its group
    float om = mx[0], os = sm[0], ou = um[0];
#pragma unroll
    for (int e = 1; e < NR; ++e) {
      om = r16 == e ? mx[e] : om;
      os = r16 == e ? sm[e] : os;
      ou = r16 == e ? um[e] : ou;
    }
    const int m = m0 + wm + (r16 >> 2) * 16 + q4 * 4 + (r16 & 3);
    if (r16 < NR && m < M && n0 + wn < N) {
      const int64_t o = (int64_t)((n0 + wn) >> 6) * g.ldp + g.rows_off + m;
      g.pm[o] = om;
      g.ps[o] = os;
      g.pu[o] = ou;
    }
  } else {
#pragma unroll
    for (int e = 0; e < NR; ++e) {
      const int m = m0 + wm + (e >> 2) * 16 + q4 * 4 + (e & 3);
      if (m >= M) continue;
      if constexpr (EPI == EPI_DZ) {
        const int tk = g.rows[g.rows_off + m];
        const int y = g.ids[tk];
        const float L = g.lse[tk], c = g.cgrad[tk];
        const float eg = g.egrad ? g.egrad[tk] : 0.f, mu = g.egrad ? L - g.ent[tk] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int n = n0 + wn + j * 16 + r16;
          const float z = acc[e >> 2][j][e & 3];
          if (n < N)
            g.dz[(int64_t)m * g.ldz + n] =
                n < g.Vvalid ? dlogit(c, eg, mu, expf(z - L), z, n == y) : 0.f;
        }
      } else {
        float* dst = split
                         ? g.part + (int64_t)blockIdx.y * g.part_ld + (int64_t)m * N
                         : g.C + (int64_t)(g.c_scatter ? g.rows[g.rows_off + m] : m) * g.ldc;
        const bool add = g.accumulate && !split;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int n = n0 + wn + j * 16 + r16;
          if (n < N) dst[n] = add ? acc[e >> 2][j][e & 3] + dst[n] : acc[e >> 2][j][e & 3];
        }
      }
    }
  }
}

// Sum of the K slices' partial results in slice order, scattered to token
// rows: C[rows[rows_off + m], n] = sum_s part[s part_ld + m N + n].
__global__ void __launch_bounds__(256) k_sum_slices(const float* __restrict__ part, int S,
                                                    int64_t part_ld, int64_t N,
                                                    const int32_t* __restrict__ cnt,
                                                    int64_t cnt_off, int64_t cap,
                                                    const int32_t* __restrict__ rows,
                                                    int64_t rows_off, float* __restrict__ C,
                                                    int64_t ldc) {
  int64_t M = (int64_t)cnt[0] - cnt_off;
  M = M < 0 ? 0 : (M > cap ? cap : M);
  for (int64_t m = blockIdx.x; m < M; m += gridDim.x) {
    float* const dst = C + (int64_t)rows[rows_off + m] * ldc;
    const float* const src = part + m * N;
    for (int64_t n = threadIdx.x; n < N; n += 256) {
      float v = 0.f;
      for (int s = 0; s < S; ++s) v += src[s * part_ld + n];
      dst[n] = v;
    }
  }
}

// Whether the 128 x 128 tile takes less time than the 64 x 64 one: tiles run
// in rounds over the CUs, a quarter of the work per 64 x 64 tile at ~15% less
// per clock (twice the operand traffic and barriers per product).
static bool tile128(int64_t M, int64_t N, int64_t splits, int64_t ncu) {
  const int64_t big = (M + 127) / 128 * ((N + 127) / 128) * splits;
  const int64_t small = (M + 63) / 64 * ((N + 63) / 64) * splits;
  return (big + ncu - 1) / ncu * 400 <= (small + ncu - 1) / ncu * 115;
}

template <int EPI, bool AKC, bool BKC, bool SEQ = false>
static hipError_t launch(const Args& a, int64_t Mcap, int64_t N, int splits, hipStream_t s) {
  int ncu = 0;
  hipError_t e = cu_count(&ncu);
  if (e != hipSuccess) return e;
  const bool big = !SEQ && tile128(Mcap, N, splits, ncu);
  const int64_t bt = big ? 128 : 64;
  const int64_t tiles = (Mcap + bt - 1) / bt * ((N + bt - 1) / bt);
  // at most 2^20 workgroups in x (a launch holds fewer than 2^32 work-items there)
  const int64_t nb = (tiles + 7) / 8 * 8, bx = nb < (1 << 20) ? nb : (1 << 20);
  const dim3 grid((unsigned)bx, (unsigned)splits, (unsigned)((nb + bx - 1) / bx));
  if (big) k_gemm_f32<EPI, 4, AKC, BKC><<<grid, NT, 0, s>>>(a);
  else k_gemm_f32<EPI, 1, AKC, BKC, SEQ><<<grid, NT, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace f3

hipError_t f32_fwd_stats(const float* H, int64_t d, const float* W, int64_t V, const int32_t* rows,
                         const int32_t* ids, const int32_t* cnt, int64_t cap, float* pm, float* ps,
                         float* pu, int64_t ldp, float* zy, hipStream_t s) {
  if (cap <= 0) return hipSuccess;
  f3::Args a = {};
  a.A = {H, d, rows, 0};
  a.B = {W, d, nullptr, 0};
  a.M = (int)cap; a.N = (int)V; a.K = (int)d;
  a.cnt = cnt; a.cnt_off = 0; a.cnt_cap = cap; a.m_from_cnt = 1;
  a.rows = rows; a.rows_off = 0; a.ids = ids;
  a.pm = pm; a.ps = ps; a.pu = pu; a.ldp = ldp; a.zy = zy;
  return f3::launch<f3::EPI_STATS, true, true>(a, cap, V, 1, s);
}

// dZ (fp32) of compacted rows [c0, c0 + Tc) into dz [Tc, Vpad]; columns >= V are 0.
hipError_t f32_dz(const float* H, int64_t d, const float* W, int64_t V, int64_t Vpad,
                  const int32_t* rows, const int32_t* ids, const float* lse, const float* cgrad,
                  const float* egrad, const float* ent, const int32_t* cnt, int64_t c0,
                  int64_t Tc, float* dz, hipStream_t s) {
  f3::Args a = {};
  a.A = {H, d, rows, c0};
  a.B = {W, d, nullptr, 0};
  a.M = (int)Tc; a.N = (int)Vpad; a.K = (int)d;
  a.NB = (int)V;  // W has V rows; columns V..Vpad-1 are written as 0
  a.cnt = cnt; a.cnt_off = c0; a.cnt_cap = Tc; a.m_from_cnt = 1;
  a.rows = rows; a.rows_off = c0; a.ids = ids; a.lse = lse; a.cgrad = cgrad;
  a.egrad = egrad; a.ent = ent;
  a.dz = dz; a.ldz = Vpad; a.Vvalid = V;
  return f3::launch<f3::EPI_DZ, true, true>(a, Tc, Vpad, 1, s);
}

// dH[rows[c0 + m], :] = dZ[m, :] . W for the chunk's rows.  With few rows the
// tiles of [Tc, d] leave CUs idle while K = V is long, so K is split into
// slices whose partial sums go to `part` and are added in slice order: enough
// slices for about eight tiles
// per CU (the valid rows are fewer than Tc, and the last round is then a small
// part), each of at least 128 K (a step of 32 K costs about 1 us while nothing
// else runs, the sum's launch 4 us) and at most 64 (the sum reads them all:
// 390 slices of 64 rows, d = 128, V = 50000 took 177 us for the backward, 64
// take 85), their sums no larger than d_weight.  1 = no split.
static int64_t dh_slices(int64_t Tc, int64_t d, int64_t V, int64_t ncu) {
  const int64_t tiles = (Tc + 127) / 128 * ((d + 127) / 128);
  if (tiles >= ncu) return 1;
  const int64_t S = std::min<int64_t>((8 * ncu + tiles - 1) / tiles, std::min<int64_t>(V / 128, 64));
  return std::max<int64_t>(1, std::min<int64_t>(S, V / Tc));
}

// fp32 values that the partial sums of chunks of Tc rows take (a workspace is
// sized without a device: for the 256 CUs of the card; fewer take fewer slices).
int64_t f32_dh_part_elems(int64_t Tc, int64_t d, int64_t V) {
  const int64_t S = dh_slices(Tc, d, V, 256);
  return S > 1 ? S * Tc * d : 0;
}

// part: room for f32_dh_part_elems(Tc, d, V) values, or nullptr: the workgroups
// then walk the same slices one after the other, on as few CUs as there are
// tiles, and the sums are the same bit for bit.
hipError_t f32_dh(const float* dz, int64_t Vpad, const float* W, int64_t V, int64_t d, int64_t Tc,
                  const int32_t* cnt, int64_t c0, const int32_t* rows, float* dH, float* part,
                  hipStream_t s) {
  if (Tc <= 0) return hipSuccess;
  int ncu = 0;
  hipError_t e = cu_count(&ncu);
  if (e != hipSuccess) return e;
  f3::Args a = {};
  a.A = {dz, Vpad, nullptr, 0};
  a.B = {W, d, nullptr, 0};
  a.M = (int)Tc; a.N = (int)d; a.K = (int)V;
  a.cnt = cnt; a.cnt_off = c0; a.cnt_cap = Tc; a.m_from_cnt = 1;
  a.C = dH; a.ldc = d; a.rows = rows; a.rows_off = c0; a.c_scatter = 1;
  int64_t S = dh_slices(Tc, d, V, std::min(ncu, 256));
  if (S < 2) return f3::launch<f3::EPI_STORE, true, false>(a, Tc, d, 1, s);
  const int64_t kper = ((V + S - 1) / S + f3::BK - 1) / f3::BK * f3::BK;
  S = (V + kper - 1) / kper;
  a.kper = (int)kper;
  if (!part) return f3::launch<f3::EPI_STORE, true, false, true>(a, Tc, d, 1, s);
  a.part = part;
  a.part_ld = Tc * d;
  if ((e = f3::launch<f3::EPI_STORE, true, false>(a, Tc, d, (int)S, s)) != hipSuccess) return e;
  f3::k_sum_slices<<<(unsigned)(Tc < 16384 ? Tc : 16384), 256, 0, s>>>(
      part, (int)S, a.part_ld, d, cnt, c0, Tc, rows, c0, dH, d);
  return hipGetLastError();
}

// dW[v, :] (+)= sum over the chunk's rows of dZ[t, v] H[rows[c0 + t], :].
hipError_t f32_dw(const float* dz, int64_t Vpad, const float* H, int64_t d, int64_t V, int64_t Tc,
                  const int32_t* cnt, int64_t c0, const int32_t* rows, float* dW, int accumulate,
                  hipStream_t s) {
  if (Tc <= 0) return hipSuccess;
  f3::Args a = {};
  a.A = {dz, Vpad, nullptr, 0};
  a.B = {H, d, rows, c0};
  a.M = (int)V; a.N = (int)d; a.K = (int)Tc;
  a.cnt = cnt; a.cnt_off = c0; a.cnt_cap = Tc; a.k_from_cnt = 1;
  a.C = dW; a.ldc = d; a.accumulate = accumulate;
  return f3::launch<f3::EPI_STORE, false, false>(a, V, d, 1, s);
}

}  // namespace rft
