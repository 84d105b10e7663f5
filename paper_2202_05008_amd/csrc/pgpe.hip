// PGPE ask / tell for gfx950 (Section 4, "Devising New Algorithms": ask generates a
// population of parameters, tell reports the evaluation results back for the state update;
// PGPE is the algorithm named in Section 5; Section 2, "Modern ML Optimizers": the gradient
// estimate is handed to an Adam-class optimizer).
//
// Design: the perturbations are never stored.  ask streams mu and sigma once and writes the
// population; tell regenerates every normal from the counter-based generator, reduces the
// rank-weighted sums in registers / LDS in a fixed order and applies the optimizer in the
// same kernel, so mu, sigma and the moments are read and written exactly once.
#include "kernels.h"
#include "mlp_f32_body.h"
#include "philox.h"
#include "bf16.h"

#include <math.h>
#include <string.h>
#include <new>

struct pgpe_state {
  pgpe_config cfg;
  float* mu;
  float* sigma;
  float* m;
  float* v;
  float* aux;
  void* work;
  uint32_t t;
  bool device_t;  // the generation index also lives on the device and the kernels read it there
  bool pending;
  uint64_t seed;
  int32_t pop;
  bool tickets_ready;  // the words of the one-launch generation have been cleared
};

namespace evo {

// ---- workspace layout ------------------------------------------------------------------
constexpr int kNormBlocks = 256;  // partial sums of a squared norm over P (ClipUp)

struct Workspace {
  float2* pairs;   // [pop_max / 2] pair weights (w, u)
  float* norm;     // [2][kNormBlocks] partial sums of |g|^2 and |vel|^2
  uint32_t* gen;   // generation index t on the device (used once pgpe_device_generation has been called)
};

static inline size_t ws_arrays_bytes(int pop_max) {
  return ((static_cast<size_t>(pop_max) * 2 + 2 * kNormBlocks) * 4 + 255) & ~size_t(255);
}
constexpr int kSmallSumWords = 2 * 4096;  // the loss sums of the one-launch generation, two words each
constexpr unsigned kGradNormParts = 8192;        // workgroups of tell whose partial sums ClipUp takes
constexpr unsigned kGradNormBytes = 4 + 3 * 8;   // of each: see TellArgs::norm_part
static inline size_t ws_bytes(int pop_max) { return ws_arrays_bytes(pop_max) + 256 + kGradNormBytes * kGradNormParts; }

static inline Workspace ws_carve(void* base, int pop_max) {
  Workspace w;
  w.pairs = static_cast<float2*>(base);
  w.norm = static_cast<float*>(base) + 2 * static_cast<size_t>(pop_max);
  w.gen = reinterpret_cast<uint32_t*>(static_cast<char*>(base) + ws_arrays_bytes(pop_max));
  return w;
}

// ---- ask -------------------------------------------------------------------------------
// Four consecutive parameters of mu and sigma (both 16-byte aligned); zeros beyond P.
__device__ __forceinline__ void load_quad(const float* __restrict__ mu, const float* __restrict__ sigma, int col, int P,
                                          float mu4[4], float sg4[4]) {
  if (col + 3 < P) {
    const float4 a = *reinterpret_cast<const float4*>(mu + col);
    const float4 b = *reinterpret_cast<const float4*>(sigma + col);
    mu4[0] = a.x, mu4[1] = a.y, mu4[2] = a.z, mu4[3] = a.w;
    sg4[0] = b.x, sg4[1] = b.y, sg4[2] = b.z, sg4[3] = b.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mu4[i] = col + i < P ? mu[col + i] : 0.f;
      sg4[i] = col + i < P ? sigma[col + i] : 0.f;
    }
  }
}

// Rows start on any parameter, so with P no multiple of 4 most of them are not 16-byte aligned.  A 16-byte store needs
// only the alignment of its elements here, and a wave's stores cover whole cache lines but for two: one store per lane
// and row whatever P is.  (P = 300007, 250 members: four 4-byte stores per lane and row 103 us, this way 65 us.)
template <bool STREAM>
__device__ __forceinline__ void store_row4(float* row, int col, int P, const float v[4]) {
  if (col + 3 < P) {
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    const f32x4u x = {v[0], v[1], v[2], v[3]};
    if (STREAM) __builtin_nontemporal_store(x, reinterpret_cast<f32x4u*>(row + col));
    else *reinterpret_cast<f32x4u*>(row + col) = x;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (col + i < P) row[col + i] = v[i];
  }
}

// STREAM: the population is larger than the memory-side cache: streaming stores in the order of the workgroup numbers,
// which is how memory takes them best (6.5 TB/s where rows are whole cache lines).  A smaller population stays in the
// caches for the evaluation, which reads it next: ordinary stores; and because a line at the border of two workgroups
// is written by both, workgroups whose numbers are 8 apart, which run on the same die and share its L2, take
// neighbouring pieces of a row, eight of them (kAskRun; longer runs leave dies of a small grid without any).  P = 45130, 500 members (90 MB): streaming in order 20.3 us, this 15.0 us.  P = 145674, 1024 members
// (600 MB): 127 us streaming, 110 us like this, but the evaluation behind it then pays for the write-back (the
// generation takes the same); P = 300007, 250 members (300 MB): 65 and 61 us, the generation 174 and 182 us.
constexpr unsigned kAskRun = 8;
template <bool STREAM>
__device__ __forceinline__ void ask_block(unsigned xblocks, unsigned& xb, unsigned& k) {
  if (STREAM) {  // grid (xblocks, N): the same order as one row of workgroup numbers, which has room for 128 GiB only
    k = blockIdx.y, xb = blockIdx.x;
    return;
  }
  const unsigned die = blockIdx.x & 7u, i = blockIdx.x >> 3;
  const unsigned b = (8 * (i / kAskRun) + die) * kAskRun + i % kAskRun;
  k = b / xblocks, xb = b - k * xblocks;
}

// fp32 population: one thread owns four consecutive parameters (one Philox counter) of one pair; the two mirrored rows
// share one draw.
template <bool STREAM>
__global__ __launch_bounds__(256) void ask_kernel(const float* __restrict__ mu, const float* __restrict__ sigma,
                                                  float* __restrict__ params, int P, int nquads, unsigned xblocks,
                                                  unsigned N, uint32_t gen_host,
                                                  const uint32_t* __restrict__ gen_dev, uint32_t key0, uint32_t key1) {
  const uint32_t gen = gen_dev ? *gen_dev : gen_host;  // uniform: the device copy when the state keeps one
  unsigned xb, k;
  ask_block<STREAM>(xblocks, xb, k);
  const int q = xb * 256 + threadIdx.x;
  if (q >= nquads || k >= N) return;
  const int col = q * 4;
  float mu4[4], sg4[4];
  load_quad(mu, sigma, col, P, mu4, sg4);
  float z[4], plus[4], minus[4];
  philox_normal4(static_cast<uint32_t>(q), static_cast<uint32_t>(k), gen, EVO_TAG_NOISE, key0, key1, z);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // both members from the exact product: each is rounded once, so they mirror about mu
    plus[i] = fmaf(sg4[i], z[i], mu4[i]);
    minus[i] = fmaf(-sg4[i], z[i], mu4[i]);
  }
  float* row = params + static_cast<size_t>(2 * k) * P;
  store_row4<STREAM>(row, col, P, plus);
  store_row4<STREAM>(row + P, col, P, minus);
}

// bfloat16 population: one thread owns eight consecutive parameters (two Philox counters) of one pair, so that each
// row takes one 16-byte streaming store per thread (on any 2-byte address, as above).  WHOLE: P is a multiple of 8, so
// no thread's parameters end early (the test for it costs 6 % where the draw is what bounds: 86544 x 4096 members).
template <bool WHOLE, bool STREAM>
__global__ __launch_bounds__(256) void ask_bf16_kernel(const float* __restrict__ mu, const float* __restrict__ sigma,
                                                       uint16_t* __restrict__ params, int P, int noct, unsigned xblocks,
                                                       unsigned N, uint32_t gen_host,
                                                       const uint32_t* __restrict__ gen_dev, uint32_t key0, uint32_t key1) {
  const uint32_t gen = gen_dev ? *gen_dev : gen_host;
  unsigned xb, k;
  ask_block<STREAM>(xblocks, xb, k);
  const int o = xb * 256 + threadIdx.x;
  if (o >= noct || k >= N) return;
  const int col = o * 8;
  float mu8[8], sg8[8];
  if (WHOLE || col + 7 < P) {  // (one branch around all four loads: two would put their waits one after the other)
    const float4 ma = *reinterpret_cast<const float4*>(mu + col), mb = *reinterpret_cast<const float4*>(mu + col + 4);
    const float4 sa = *reinterpret_cast<const float4*>(sigma + col), sb = *reinterpret_cast<const float4*>(sigma + col + 4);
    mu8[0] = ma.x, mu8[1] = ma.y, mu8[2] = ma.z, mu8[3] = ma.w, mu8[4] = mb.x, mu8[5] = mb.y, mu8[6] = mb.z, mu8[7] = mb.w;
    sg8[0] = sa.x, sg8[1] = sa.y, sg8[2] = sa.z, sg8[3] = sa.w, sg8[4] = sb.x, sg8[5] = sb.y, sg8[6] = sb.z, sg8[7] = sb.w;
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      mu8[i] = mu[min(col + i, P - 1)];
      sg8[i] = sigma[min(col + i, P - 1)];
    }
  }
  float z[8];
  philox_normal4(static_cast<uint32_t>(2 * o), static_cast<uint32_t>(k), gen, EVO_TAG_NOISE, key0, key1, z);
  philox_normal4(static_cast<uint32_t>(2 * o + 1), static_cast<uint32_t>(k), gen, EVO_TAG_NOISE, key0, key1, z + 4);
  typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));
  u32x4u plus, minus;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    plus[i] = pack_bf16x2(fmaf(sg8[2 * i], z[2 * i], mu8[2 * i]), fmaf(sg8[2 * i + 1], z[2 * i + 1], mu8[2 * i + 1]));
    minus[i] = pack_bf16x2(fmaf(-sg8[2 * i], z[2 * i], mu8[2 * i]), fmaf(-sg8[2 * i + 1], z[2 * i + 1], mu8[2 * i + 1]));
  }
  uint16_t* row = params + static_cast<size_t>(2 * k) * P;
  if (WHOLE || col + 7 < P) {
    if (STREAM) {
      __builtin_nontemporal_store(plus, reinterpret_cast<u32x4u*>(row + col));
      __builtin_nontemporal_store(minus, reinterpret_cast<u32x4u*>(row + P + col));
    } else {
      *reinterpret_cast<u32x4u*>(row + col) = plus;
      *reinterpret_cast<u32x4u*>(row + P + col) = minus;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (col + i >= P) break;
      row[col + i] = static_cast<uint16_t>(plus[i >> 1] >> (16 * (i & 1)));
      row[P + col + i] = static_cast<uint16_t>(minus[i >> 1] >> (16 * (i & 1)));
    }
  }
}

// ---- ask fused with the sphere fitness: the population is never written --------------------------
// Thread = kFusedQuads parameter quads x kFusedPairs pairs: mu, sigma and x_star are loaded once
// per quad, each draw serves both members of its pair, and theta is formed exactly as ask_kernel
// stores it (one fused multiply-add, rounded once) before x_star is subtracted.  A workgroup
// leaves one partial sum per member in part[member][blockIdx.x]; sphere_finish_kernel adds a
// member's partial sums in a fixed order.
constexpr int kFusedQuads = 4;
constexpr int kFusedPairs = 4;

__global__ __launch_bounds__(256) void ask_sphere_kernel(const float* __restrict__ mu, const float* __restrict__ sigma,
                                                         const float* __restrict__ x_star, float* __restrict__ part,
                                                         int P, int nquads, int N, int xblocks, uint32_t gen_host,
                                                         const uint32_t* __restrict__ gen_dev, uint32_t key0,
                                                         uint32_t key1) {
  const uint32_t gen = gen_dev ? *gen_dev : gen_host;
  __shared__ float red[4][2 * kFusedPairs];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k0 = blockIdx.y * kFusedPairs;
  float acc[kFusedPairs][2];
#pragma unroll
  for (int ki = 0; ki < kFusedPairs; ++ki) acc[ki][0] = acc[ki][1] = 0.f;
  for (int qi = 0; qi < kFusedQuads; ++qi) {
    const int q = (blockIdx.x * kFusedQuads + qi) * 256 + tid;
    if (q >= nquads) break;
    const int col = q * 4;
    float mu4[4], sg4[4], xs4[4];
    load_quad(mu, sigma, col, P, mu4, sg4);  // columns beyond P contribute (0 - 0)^2
    if (col + 3 < P) {
      const float4 c = *reinterpret_cast<const float4*>(x_star + col);
      xs4[0] = c.x, xs4[1] = c.y, xs4[2] = c.z, xs4[3] = c.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) xs4[i] = col + i < P ? x_star[col + i] : 0.f;
    }
#pragma unroll
    for (int ki = 0; ki < kFusedPairs; ++ki) {
      if (k0 + ki >= N) break;  // uniform over the workgroup
      float z[4];
      philox_normal4(static_cast<uint32_t>(q), static_cast<uint32_t>(k0 + ki), gen, EVO_TAG_NOISE, key0, key1, z);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float dp = fmaf(sg4[i], z[i], mu4[i]) - xs4[i];
        const float dm = fmaf(-sg4[i], z[i], mu4[i]) - xs4[i];
        acc[ki][0] = fmaf(dp, dp, acc[ki][0]);
        acc[ki][1] = fmaf(dm, dm, acc[ki][1]);
      }
    }
  }
#pragma unroll
  for (int ki = 0; ki < kFusedPairs; ++ki)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      float v = acc[ki][s];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (lane == 0) red[wave][2 * ki + s] = v;
    }
  __syncthreads();
  if (tid < 2 * kFusedPairs && k0 + (tid >> 1) < N) {
    const float total = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
    part[static_cast<size_t>(2 * k0 + tid) * xblocks + blockIdx.x] = total;
  }
}

// fitness[m] = -(sum of the member's xblocks partial sums): one wavefront per member, lane l adds
// partial sums l, l + 64, ... in order, then a fixed butterfly over the lanes.
__global__ __launch_bounds__(256) void sphere_finish_kernel(const float* __restrict__ part, int xblocks, int pop,
                                                            float* __restrict__ fitness) {
  const int lane = threadIdx.x & 63;
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (m >= pop) return;
  const float* row = part + static_cast<size_t>(m) * xblocks;
  float v = 0.f;
  for (int i = lane; i < xblocks; i += 64) v += row[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if (lane == 0) fitness[m] = -v;
}

static inline int fused_xblocks(int P) { return ((P + 3) / 4 + 256 * kFusedQuads - 1) / (256 * kFusedQuads); }

// ---- centered ranks and pair weights ------------------------------------------------------
// fp32 bits -> u32 that orders like the float: -0 counts as +0, NaN sorts lowest.
__device__ __forceinline__ uint32_t orderable(float f) {
  uint32_t b = __float_as_uint(f);
  if ((b & 0x7FFFFFFFu) > 0x7F800000u) return 0u;
  if (b == 0x80000000u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Centered ranks by counting: the rank of member m is the number of 64-bit keys
// (orderable fitness << 32 | member index) below its own.  Keys are unique, so the ranks are
// exactly those of a stable sort, and the count needs no sort at all.  The orderable words of the whole population are
// staged in LDS (at most 16 KB, padded with words above every key).
//
// tell only needs the pair weights w = (c+ - c-) / 2 and u = (c+ + c-) / 2 - b.  Centered ranks come in pairs of opposite
// sign, so their mean b is exactly zero and a pair's weights follow from its two ranks alone.
__device__ __forceinline__ void stage_orderable(const float* fitness, int pop, int padded, uint32_t* ord, int threads) {
  for (int i = threadIdx.x; i < padded; i += threads) ord[i] = i < pop ? orderable(fitness[i]) : 0xFFFFFFFFu;
}
__device__ __forceinline__ float centered_rank(uint32_t rank, int pop) {
  // one correctly rounded divide of two exactly representable integers
  return static_cast<float>(2 * static_cast<int>(rank) - (pop - 1)) / static_cast<float>(2 * (pop - 1));
}
__device__ __forceinline__ float2 pair_weights(float cp, float cm, double b) {
  const double p = cp, m = cm;
  return make_float2(static_cast<float>(0.5 * (p - m)), static_cast<float>(0.5 * (p + m) - b));
}
// Sum over the 64 lanes (register lane moves only), valid in every lane.
__device__ __forceinline__ uint32_t wave_count(uint32_t v) {
  int x = static_cast<int>(v);
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(x, 63));
}

// One wavefront per pair: a lane compares four keys per 16-byte LDS read against both members, and one sum over the
// wave of the two packed counts gives both ranks.  (Sixteen lanes per member and 4-byte reads, 256 threads, 14.4 us at
// 4096 members; this way, and with the pair weights formed here instead of by every workgroup of tell, tell takes 121 -> 98
// us at P = 86544 and 20.5 -> 14.0 us at P = 22152, 1000 members.)  THREADS: 1024 above 1024 members, so that a workgroup's staging serves sixteen pairs.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void rank_kernel(const float* __restrict__ fitness, int pop,
                                                       uint32_t* __restrict__ rank_out, float* __restrict__ shaped_out,
                                                       float2* __restrict__ pairs_out) {
  __shared__ __attribute__((aligned(16))) uint32_t ord[EVO_POP_MAX];
  const int padded = (pop + 255) & ~255;
  stage_orderable(fitness, pop, padded, ord, THREADS);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x * (THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (2 * k >= pop) return;
  const int m0 = 2 * k, m1 = min(2 * k + 1, pop - 1);
  const uint64_t key0 = (static_cast<uint64_t>(ord[m0]) << 32) | static_cast<uint32_t>(m0);
  const uint64_t key1 = (static_cast<uint64_t>(ord[m1]) << 32) | static_cast<uint32_t>(m1);
  uint32_t count0 = 0, count1 = 0;
  for (int j = 4 * lane; j < padded; j += 256) {
    const uint4 o = *reinterpret_cast<const uint4*>(ord + j);
    const uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t key = (static_cast<uint64_t>(w[i]) << 32) | static_cast<uint32_t>(j + i);
      count0 += key < key0 ? 1u : 0u;
      count1 += key < key1 ? 1u : 0u;
    }
  }
  const uint32_t counts = wave_count(count0 | (count1 << 16));
  if (lane == 0) {
    const uint32_t r0 = counts & 0xffffu, r1 = counts >> 16;
    const float c0 = centered_rank(r0, pop), c1 = centered_rank(r1, pop);
    if (rank_out) {
      rank_out[m0] = r0;
      if (m0 + 1 < pop) rank_out[m0 + 1] = r1;
    }
    if (shaped_out) {
      shaped_out[m0] = c0;
      if (m0 + 1 < pop) shaped_out[m0 + 1] = c1;
    }
    if (pairs_out) pairs_out[k] = pair_weights(c0, c1, 0.0);
  }
}

// Total of n values in fp64 with a fixed tree, by 256 threads, in every thread; red: 256 doubles of LDS.
__device__ __forceinline__ double total256(const float* c, int n, double* red) {
  const int tid = threadIdx.x;
  double acc = 0.0;
  for (int i = tid; i < n; i += 256) acc += static_cast<double>(c[i]);
  red[tid] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  return red[0];
}

// Pair weights of the raw fitness (no shaping): one workgroup.
__global__ __launch_bounds__(256) void raw_pairs_kernel(const float* __restrict__ fitness, int pop,
                                                        float2* __restrict__ pairs_out) {
  __shared__ double red[256];
  const double b = total256(fitness, pop, red) / static_cast<double>(pop);
  for (int k = threadIdx.x; k < pop / 2; k += 256) pairs_out[k] = pair_weights(fitness[2 * k], fitness[2 * k + 1], b);
}

// The pair weights of a small population inside a workgroup of 256: four threads per member (128 members: two, more: one),
// which share the count of the keys below its own.  fitness: memory or LDS; ord: (pop rounded up to 4) words of LDS,
// 16-byte aligned; c: pop floats of LDS; red: 256 doubles of LDS; pairs: pop / 2 float2 of LDS.  Ends with a barrier.
__device__ __forceinline__ void small_pairs(const float* fitness, int pop, int shaping, uint32_t* ord, float* c, double* red,
                                            float2* pairs) {
  const int tid = threadIdx.x, padded = (pop + 3) & ~3;
  if (shaping) {
    stage_orderable(fitness, pop, padded, ord, 256);
    __syncthreads();
    const int share = pop <= 64 ? 2 : pop <= 128 ? 1 : 0, sharers = 1 << share;  // (log2 of the) threads per member
    for (int m0 = 0; m0 < pop; m0 += 256 >> share) {
      const int m = m0 + (tid >> share);
      const uint64_t key_m = (static_cast<uint64_t>(ord[min(m, pop - 1)]) << 32) | static_cast<uint32_t>(m);
      uint32_t count = 0;
#pragma unroll 2
      for (int j = 4 * (tid & (sharers - 1)); j < padded; j += 4 * sharers) {
        const uint4 o = *reinterpret_cast<const uint4*>(ord + j);
        const uint32_t w[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
          count += ((static_cast<uint64_t>(w[i]) << 32) | static_cast<uint32_t>(j + i)) < key_m ? 1u : 0u;
      }
      int sum = static_cast<int>(count);
      if (share >= 1) sum += __builtin_amdgcn_update_dpp(0, sum, 0xb1, 0xf, 0xf, false);  // quad_perm 1,0,3,2
      if (share >= 2) sum += __builtin_amdgcn_update_dpp(0, sum, 0x4e, 0xf, 0xf, false);  // quad_perm 2,3,0,1
      if (m < pop && (tid & (sharers - 1)) == 0) c[m] = centered_rank(static_cast<uint32_t>(sum), pop);
    }
    __syncthreads();
    for (int k = tid; k < pop / 2; k += 256) pairs[k] = pair_weights(c[2 * k], c[2 * k + 1], 0.0);
  } else {
    const double b = total256(fitness, pop, red) / static_cast<double>(pop);
    for (int k = tid; k < pop / 2; k += 256) pairs[k] = pair_weights(fitness[2 * k], fitness[2 * k + 1], b);
  }
  __syncthreads();
}

// wave_sum's moves and order in fp64 (as shuffles through LDS 0.3 us a sum).
template <typename MOVE>
__device__ __forceinline__ double moved(double v, MOVE move) {
  return __hiloint2double(move(__double2hiint(v)), move(__double2loint(v)));
}
__device__ __forceinline__ double wave_sum(double v) {
  const unsigned lo = __double2loint(v), hi = __double2hiint(v);
  const auto l32 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h32 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  v = __hiloint2double(h32[0], l32[0]) + __hiloint2double(h32[1], l32[1]);
  const unsigned lo16 = __double2loint(v), hi16 = __double2hiint(v);
  const auto l = __builtin_amdgcn_permlane16_swap(lo16, lo16, false, false), h = __builtin_amdgcn_permlane16_swap(hi16, hi16, false, false);
  v = __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
  v += moved(v, [](int x) { return __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false); });  // row_ror:8
  v += moved(v, [](int x) { return __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, false); });  // row_ror:4
  v += moved(v, [](int x) { return __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, false); });   // quad_perm 2,3,0,1
  v += moved(v, [](int x) { return __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, false); });   // quad_perm 1,0,3,2
  return v;
}

// Sum of the 256 per-thread values of a workgroup, fixed order; valid in every thread.  scratch: 4 floats of LDS.
__device__ __forceinline__ float block_sum256(float v, float* scratch) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = v;
  __syncthreads();
  return (scratch[0] + scratch[1]) + (scratch[2] + scratch[3]);
}

// ---- tell --------------------------------------------------------------------------------
struct TellArgs {
  float* mu;
  float* sigma;
  float* m;
  float* v;
  float* ms;  // sigma moments (rule 1) or null
  float* vs;
  float* gmu_out;  // gradient-only mode
  float* gsg_out;
  const float2* pairs;   // pair weights (w, u)[N] in memory, or null: formed in the kernel from `fitness`
  const float* fitness;
  int shaping;
  const float* theta;   // stored population [2N][P] (STORED form) or null
  int P, nquads, N, KS;
  uint32_t gen, key0, key1;
  const uint32_t* gen_dev;  // when set: t is read here and the bias corrections are formed in the kernel
  float* norm_part;        // ClipUp: [kGradNormParts] partial sums of g_mu^2, one per workgroup, or null; see norm_sums
  float inv_n, lr_mu, lr_sigma, max_change, beta1, beta2, eps, bc1, bc2, momentum;
};

__device__ __forceinline__ float adam_step(float x, float g, float& m, float& v, float lr, const TellArgs& a) {
  m = a.beta1 * m + (1.0f - a.beta1) * g;
  v = a.beta2 * v + (1.0f - a.beta2) * g * g;
  const float m_hat = m * a.bc1;
  const float v_hat = v * a.bc2;
  return x + lr * m_hat / (sqrtf(v_hat) + a.eps);
}

// Behind them: [3][kGradNormParts] the same in fp64, of vel^2 and of vel g_mu.
__host__ __device__ inline double* norm_sums(float* norm_part) { return reinterpret_cast<double*>(norm_part + kGradNormParts); }

// Thread (q, ks): parameter quad q, pairs ks, ks+KS, ks+2KS, ...  The KS partial sums of a
// quad are added in increasing ks by one thread, so the result does not depend on timing.
// OPT: what happens to mu.  SRULE: sigma rule 0 (clipped ascent) or 1 (Adam); unused with OPT_GRAD.
// STORED: the perturbation eps = theta[2k] - mu is read back from the population that ask wrote
// (sums of w eps and u (eps^2 - sigma^2)) instead of being regenerated (sums of w z and u (z^2 - 1)).
enum { OPT_ADAM = 0, OPT_CLIPUP_GRAD = 1, OPT_MOMENTUM = 2, OPT_GRAD = 3 };
// PAIRS: where the pair weights lie (memory or LDS).  part: 256 * 8 floats of LDS.
template <int OPT, int SRULE, bool STORED, typename PAIRS>
__device__ __forceinline__ void tell_block(TellArgs a, int block, PAIRS pairs, float* part) {
  const int tid = threadIdx.x;
  if (a.gen_dev) {  // generation index on the device: the same double-precision bias corrections the host forms
    a.gen = *a.gen_dev;
    const double t = static_cast<double>(a.gen);
    a.bc1 = static_cast<float>(1.0 / (1.0 - pow(static_cast<double>(a.beta1), t)));
    a.bc2 = static_cast<float>(1.0 / (1.0 - pow(static_cast<double>(a.beta2), t)));
  }
  const int QPB = 256 / a.KS;
  const int ql = tid % QPB;
  const int ks = tid / QPB;
  const int q = block * QPB + ql;
  float A[4] = {0.f, 0.f, 0.f, 0.f}, B[4] = {0.f, 0.f, 0.f, 0.f};
  if (q < a.nquads && !STORED) {
    auto sum = [&](int k0) {
      for (int k = k0; k < a.N; k += a.KS) {
        float z[4];
        philox_normal4(static_cast<uint32_t>(q), static_cast<uint32_t>(k), a.gen, EVO_TAG_NOISE, a.key0, a.key1, z);
        const float2 wu = pairs[k];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          A[i] = fmaf(wu.x, z[i], A[i]);
          B[i] = fmaf(wu.y, fmaf(z[i], z[i], -1.0f), B[i]);
        }
      }
    };
    // slices of whole waves: the pair is the same for all lanes, its weights and the first round's product are scalar
    if (QPB >= 64) sum(__builtin_amdgcn_readfirstlane(ks));
    else sum(ks);
  }
  if (q < a.nquads && STORED) {
    const int col = q * 4;
    float mu4[4], nv4[4];             // centre and -sigma^2
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = min(col + i, a.P - 1);
      const float sg = a.sigma[c];
      mu4[i] = a.mu[c];
      nv4[i] = -sg * sg;
    }
    const bool whole = col + 3 < a.P;  // rows start on any parameter's address: 16-byte loads need no more
#pragma unroll 8
    for (int k = ks; k < a.N; k += a.KS) {
      const float* row = a.theta + static_cast<size_t>(2 * k) * a.P;
      float th[4];
      if (whole) {
        typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
        const f32x4u t = __builtin_nontemporal_load(reinterpret_cast<const f32x4u*>(row + col));
        th[0] = t[0], th[1] = t[1], th[2] = t[2], th[3] = t[3];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) th[i] = row[min(col + i, a.P - 1)];
      }
      const float2 wu = pairs[k];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = th[i] - mu4[i];
        A[i] = fmaf(wu.x, e, A[i]);
        B[i] = fmaf(wu.y, fmaf(e, e, nv4[i]), B[i]);
      }
    }
  }
  // The KS partial sums of a parameter are added in increasing ks, each parameter by one thread, which then also makes its
  // update: neighbouring threads have neighbouring parameters, whatever KS.
  {
    float* mine = part + tid * 8;
    *reinterpret_cast<float4*>(mine) = make_float4(A[0], A[1], A[2], A[3]);
    *reinterpret_cast<float4*>(mine + 4) = make_float4(B[0], B[1], B[2], B[3]);
  }
  __syncthreads();
  float sq = 0.f;
  double gg = 0.0, vv = 0.0, vg = 0.0;
  for (int p = tid; p < 4 * QPB; p += 256) {
    const int c = block * QPB * 4 + p;
    if (c >= a.P) break;
    const float* sums = part + (p >> 2) * 8 + (p & 3);
    float sa = sums[0], sb = sums[4];
#pragma unroll 8
    for (int s = 1; s < a.KS; ++s) {
      sa += sums[s * QPB * 8];
      sb += sums[s * QPB * 8 + 4];
    }
    const float sg = a.sigma[c];
    const float g_mu = STORED ? sa * a.inv_n : sg * sa * a.inv_n;
    const float g_sg = STORED ? (sg > 0.f ? sb / sg * a.inv_n : 0.f) : sg * sb * a.inv_n;
    if (OPT == OPT_GRAD) {
      a.gmu_out[c] = g_mu;
      a.gsg_out[c] = g_sg;
      continue;
    }
    if (OPT == OPT_ADAM) {
      float m = a.m[c], v = a.v[c];
      a.mu[c] = adam_step(a.mu[c], g_mu, m, v, a.lr_mu, a);
      a.m[c] = m;
      a.v[c] = v;
    } else if (OPT == OPT_MOMENTUM) {
      const float vel = a.momentum * a.m[c] + a.lr_mu * g_mu;
      a.m[c] = vel;
      a.mu[c] += vel;
    } else {
      a.v[c] = g_mu;  // ClipUp needs |g_mu| over all of P first: the gradient waits in v
      if (a.norm_part) {
        const double vel = a.m[c], g = g_mu;
        sq = fmaf(g_mu, g_mu, sq), gg = fma(g, g, gg), vv = fma(vel, vel, vv), vg = fma(vel, g, vg);
      }
    }
    if (SRULE == 0) {
      const float lim = a.max_change * sg;
      a.sigma[c] = sg + fminf(fmaxf(a.lr_sigma * g_sg, -lim), lim);
    } else {
      float ms = a.ms[c], vs = a.vs[c];
      a.sigma[c] = fmaxf(adam_step(sg, g_sg, ms, vs, a.lr_sigma, a), 1e-8f);
      a.ms[c] = ms;
      a.vs[c] = vs;
    }
  }
  if (OPT == OPT_CLIPUP_GRAD && a.norm_part) {
    __syncthreads();  // the partial sums have been read
    double* all = reinterpret_cast<double*>(part);  // [3][256]: a wave adds up one of the three
    all[tid] = gg, all[256 + tid] = vv, all[512 + tid] = vg;
    const float t = block_sum256(sq, part + 2 * 3 * 256);  // (with the barrier that the three need)
    if (tid == 0) a.norm_part[block] = t;
    const int wave = tid >> 6, lane = tid & 63;
    if (wave < 3) {
      const double* x = all + 256 * wave + lane;
      const double sum = wave_sum((x[0] + x[64]) + (x[128] + x[192]));
      if (lane == 0) norm_sums(a.norm_part)[wave * kGradNormParts + block] = sum;
    }
  }
}

// SMALL: the pair weights of at most kSmallPairs members are formed by every workgroup itself instead of by a launch of
// rank_kernel (P = 676, 64 members: 10.2 -> 7.4 us for tell, P = 100003, 64 members: 16 -> 10 us).  With 256 members the
// thousands of instructions per workgroup cost more than the launch (P = 300007: 28 -> 42 us), and so they do with
// many workgroups (kSmallWork).
constexpr int kSmallPairs = 128;
constexpr long kSmallWork = 128 * 2048;  // members x workgroups
template <int OPT, int SRULE, bool STORED, bool SMALL>
__global__ __launch_bounds__(256) void tell_kernel(TellArgs a) {
  __shared__ __attribute__((aligned(16))) float part[256 * 8];
  if (SMALL) {
    __shared__ __attribute__((aligned(16))) uint32_t ord[kSmallPairs];
    __shared__ float2 pairs[kSmallPairs / 2];
    small_pairs(a.fitness, 2 * a.N, a.shaping, ord, part, reinterpret_cast<double*>(part), pairs);
    tell_block<OPT, SRULE, STORED>(a, blockIdx.x, static_cast<const float2*>(pairs), part);
  } else {
    tell_block<OPT, SRULE, STORED>(a, blockIdx.x, a.pairs, part);
  }
}

// ---- one whole generation in one launch (small problems) ----------------------------------------------------
// ask -> forward + loss -> fitness -> ranks -> tell for problems whose launches are bound by their latency
// (Section 2's loop of ask, evaluate, tell at cfg1's size).  Workgroup (tile, member): draws the member's parameters
// into LDS exactly as ask_kernel would store them, runs mlp_f32_body on its tile of samples and hands the tile's
// loss sum over.  The first n_tell workgroups then wait for every tile's sum (every other workgroup exits, so those
// that wait cannot keep anyone from arriving; the wait is bounded), form every member's fitness and utility in LDS
// with the arithmetic of finalize_kernel and rank_kernel and run tell_block for their block of parameters: the
// same bits as the calls one by one give.  mu and sigma are first written after every workgroup has read them.
//
// The hand-over has no fence and no counter that anyone waits for: on this chip a release at device scope writes a die's
// cache back (measured: 5 us from the end of the forward to the counted arrival, 13 us until 512 arrivals had been seen).
// The sums themselves are the flags: a workgroup stores its sum and the number of the launch in one 8-byte device-scope
// store, and the waiting workgroups poll the words with device-scope loads until all carry this launch's number.  The
// number lives on the device and the last waiting workgroup to finish advances it, so no launch ever meets its own
// number in an older sum, whatever happened to the state or the population in between and however often a recorded
// launch is replayed.  (Words that a generation cleared for the next one, in two arrays by the parity of t, were such older
// sums after a reset, an import, a generation by the separate calls or a larger population than the one before.)
struct GenSmallArgs {
  MlpArgs mlp;       // params and partial unused: the parameters are drawn here, the sums go through `sums`
  TellArgs tell;     // pairs and fitness unused: the pair weights are formed here
  float* fitness;    // [pop] out
  float scale;       // fitness = scale * sum of the member's loss sums
  uint64_t* sums;    // [kSmallMaxTiles] (launch number, bits of the loss sum) of (member, tile)
  uint32_t* launches;  // launches so far
  uint32_t* done;    // waiting workgroups that have finished (the last one clears it and advances launches and gen_rw)
  uint32_t* gen_rw;  // the device copy of t, or null
  int pop, shaping, n_tell, total;
};
constexpr int kSmallMaxTiles = 4096;       // (member, tile) pairs of one launch
constexpr int kSmallSpinLimit = 1 << 21;   // polls of about a microsecond: a sum that has not come by then never will
typedef __attribute__((address_space(3))) const float* lds_cfloat_ptr;

template <int LOSS, int OPT, int SRULE>
__global__ __launch_bounds__(256) void generation_small_kernel(GenSmallArgs g) {
  extern __shared__ __attribute__((aligned(16))) float gs_smem[];
  __shared__ int missing;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int member = blockIdx.y, tile = blockIdx.x;
  const int wg = member * gridDim.x + tile;
  const int P = g.tell.P, nquads = g.tell.nquads;
  const uint32_t gen = g.tell.gen_dev ? *g.tell.gen_dev : g.tell.gen;
  const uint32_t launch = *g.launches + 1u;  // this launch's number
  if (tid == 0) missing = 0;
  // ---- ask: this member's row, as ask_kernel forms it ----
  {
    const float sign = (member & 1) ? -1.0f : 1.0f;
    for (int q = tid; q < nquads; q += 256) {
      const int col = q * 4;
      float mu4[4], sg4[4];
      load_quad(g.tell.mu, g.tell.sigma, col, P, mu4, sg4);
      float z[4];
      philox_normal4(static_cast<uint32_t>(q), static_cast<uint32_t>(member >> 1), gen, EVO_TAG_NOISE, g.tell.key0,
                     g.tell.key1, z);
#pragma unroll
      for (int i = 0; i < 4; ++i) gs_smem[col + i] = fmaf(sign * sg4[i], z[i], mu4[i]);
    }
  }
  __syncthreads();
  // ---- forward and loss of this tile; thread 0 holds the tile's sum and hands it over ----
  float* mlp_lds = gs_smem + 4 * nquads;
  const float tile_loss = mlp_f32_body<LOSS>(g.mlp, (lds_cfloat_ptr)gs_smem, member, tile, mlp_lds);
  if (tid == 0)
    __hip_atomic_store(g.sums + wg, (static_cast<uint64_t>(launch) << 32) | __float_as_uint(tile_loss), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  if (wg >= g.n_tell) return;
  __syncthreads();  // the tile's LDS is free
  // ---- every tile's sum, polled into LDS ----
  float* tell_smem = gs_smem;                  // 256 * 8 floats
  const int pop4 = (g.pop + 3) & ~3;
  uint32_t* ord_s = reinterpret_cast<uint32_t*>(tell_smem + 256 * 8);
  float* fit_s = reinterpret_cast<float*>(ord_s + pop4);
  float* shaped_s = fit_s + pop4;
  float2* pairs_s = reinterpret_cast<float2*>(shaped_s + pop4);
  float* part_s = reinterpret_cast<float*>(pairs_s) + pop4;
  for (int i = tid; i < g.total; i += 256) {
    uint64_t word = __hip_atomic_load(g.sums + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int polls = 0; static_cast<uint32_t>(word >> 32) != launch && polls < kSmallSpinLimit; ++polls) {
      __builtin_amdgcn_s_sleep(2);
      word = __hip_atomic_load(g.sums + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (static_cast<uint32_t>(word >> 32) != launch) missing = 1;
    part_s[i] = __uint_as_float(static_cast<uint32_t>(word));
  }
  // the last of the waiting workgroups to finish advances the launch's number, and t where it lives on the device
  auto finish = [&]() {
    if (tid != 0 || atomicAdd(g.done, 1u) != static_cast<uint32_t>(g.n_tell - 1)) return;
    *g.done = 0u;
    *g.launches = launch;
    if (g.gen_rw) *g.gen_rw += 1u;
  };
  __syncthreads();
  if (missing) {  // never seen; the fitness says so rather than a silent wrong update
    if (wg == 0 && tid == 0) g.fitness[0] = __builtin_nanf("");
    finish();
    return;
  }
  // ---- fitness, orderable words and utilities of every member, in LDS ----
  // finalize_kernel's sum per member: lane j takes tiles j, j + 64, ..., then the fixed butterfly over the 64 lanes.
  // With at most 16 tiles the butterfly's first two levels add the zeros of lanes 16..63 (x + 0 = x, and a sum of
  // per-sample losses is never -0), so four members share a wave, sixteen lanes each, and take the last four levels.
  const int tiles = g.mlp.tiles;
  if (tiles <= 16) {
    const int sub = lane >> 4, j = lane & 15;
    for (int m0 = 4 * wave; m0 < g.pop; m0 += 16) {
      const int m = m0 + sub;
      float acc = (m < g.pop && j < tiles) ? part_s[m * tiles + j] : 0.f;
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
      if (j == 0 && m < g.pop) {
        const float f = g.scale * acc;
        fit_s[m] = f;
        if (wg == 0) g.fitness[m] = f;
      }
    }
  } else {
    for (int m = wave; m < g.pop; m += 4) {
      float acc = 0.f;
      for (int j = lane; j < tiles; j += 64) acc += part_s[m * tiles + j];
      acc = wave_sum(acc);
      if (lane == 0) {
        const float f = g.scale * acc;
        fit_s[m] = f;
        if (wg == 0) g.fitness[m] = f;
      }
    }
  }
  __syncthreads();
  small_pairs(fit_s, g.pop, g.shaping, ord_s, shaped_s, reinterpret_cast<double*>(tell_smem), pairs_s);
  // ---- tell for this workgroup's block of parameters ----
  tell_block<OPT, SRULE, false>(g.tell, wg, static_cast<const float2*>(pairs_s), tell_smem);
  finish();
}

// ---- ClipUp: two norms over P, each as partial sums in a fixed order ------------------------------------------
// The sums come per workgroup of tell (at most kGradNormParts of them) and one launch does the rest; with more workgroups |g|^2 per workgroup of sqnorm_kernel and |vel|^2 per workgroup of the velocity kernel, in two launches.
// Their totals: total256, the same bits in every thread of every workgroup (one thread adding 256 partial sums in turn
// made each of the two kernels that need a total 7..10 us long).
// part[b] = sum of x[i]^2 over the elements of workgroup b (grid-stride, kNormBlocks workgroups).
__global__ __launch_bounds__(256) void sqnorm_kernel(const float* __restrict__ x, int P, float* __restrict__ part) {
  __shared__ float scratch[4];
  float acc = 0.f;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < P; i += kNormBlocks * 256) acc = fmaf(x[i], x[i], acc);
  const float t = block_sum256(acc, scratch);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// vel = momentum vel + step g / |g| (g waits in `g`, |g|^2 in n_g partial sums); partial sums of vel^2 to part_v.
__global__ __launch_bounds__(256) void clipup_velocity_kernel(float* __restrict__ vel, const float* __restrict__ g,
                                                              int P, float momentum, float step,
                                                              const float* __restrict__ part_g, int n_g,
                                                              float* __restrict__ part_v) {
  __shared__ float scratch[4];
  __shared__ double red[256];
  const double n2 = total256(part_g, n_g, red);
  const float scale = n2 > 0.0 ? static_cast<float>(static_cast<double>(step) / sqrt(n2)) : 0.f;
  float acc = 0.f;
  auto one = [&](float& v, float gi) {
    v = fmaf(scale, gi, momentum * v);
    acc = fmaf(v, v, acc);
  };
  const int first = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
#pragma unroll 4
  for (int i = first; i < P / 4; i += stride) {
    const float4 gi = reinterpret_cast<const float4*>(g)[i];
    float4 v = reinterpret_cast<float4*>(vel)[i];
    one(v.x, gi.x), one(v.y, gi.y), one(v.z, gi.z), one(v.w, gi.w);
    reinterpret_cast<float4*>(vel)[i] = v;
  }
  if (first < (P & 3)) one(vel[(P & ~3) + first], g[(P & ~3) + first]);
  const float t = block_sum256(acc, scratch);
  if (threadIdx.x == 0) part_v[blockIdx.x] = t;
}

// Both in one launch, where tell has left the sums of g^2, vel^2 and vel g: the norm of the new velocity
//   |momentum vel + s g|^2 = momentum^2 vel^2 + 2 momentum s vel g + s^2 g^2,  s = step / |g|,
// is known before any of it is formed.  The three sums are fp64 from the elements on: s comes from a sum of fp32 squares
// (their overflow takes the normalised gradient to 0), which for elements around 1e-21 holds a few units of the last
// place, and |s g| is then tens of percent off step; and a velocity from outside may cancel against the gradient.
// (Length of a clipped velocity against max_speed, 144 steps of 500..300007 parameters: 2.3e-8 rms, at most 4.3e-8; where
// the new velocity's elements are added up in fp32 2.5e-8 and 5.6e-8.)  Bound by latency: the sums, their total, then
// three loads and two stores per quad.  Alone, the two launches and this one: 6.0 + 4.6 and 5.5 us at P = 45530, 6.7 + 5.3
// and 6.7 us at 300007, for at most 0.3 us more in tell.
__global__ __launch_bounds__(256) void clipup_step_kernel(float* __restrict__ mu, float* __restrict__ vel,
                                                          const float* __restrict__ g, int P, float momentum, float step,
                                                          float max_speed, const float* __restrict__ part,
                                                          const double* __restrict__ sums, int n) {
  __shared__ double red[4][256];
  const int tid = threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int i = tid; i < n; i += 256) {
    acc[3] += static_cast<double>(part[i]);
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[k] += sums[k * kGradNormParts + i];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) red[k][tid] = acc[k];
  __syncthreads();
  {  // a wave adds up one of the four, in a tree of halves
    double* x = red[tid >> 6];
    const int lane = tid & 63;
    const double sum = wave_sum((x[lane] + x[lane + 128]) + (x[lane + 64] + x[lane + 192]));
    if (lane == 0) x[0] = sum;
  }
  __syncthreads();
  const double gg = red[0][0], vv = red[1][0], vg = red[2][0], n2 = red[3][0];
  const float scale = n2 > 0.0 ? static_cast<float>(static_cast<double>(step) / sqrt(n2)) : 0.f;
  const double m = momentum, sc = scale;
  // a gradient whose squares overflow (scale 0) or whose elements are all 0 leaves momentum vel alone
  const double speed = sqrt(fmax(m * m * vv + (scale != 0.f ? 2.0 * m * sc * vg + sc * sc * gg : 0.0), 0.0));
  const float clip = speed > static_cast<double>(max_speed) ? static_cast<float>(static_cast<double>(max_speed) / speed) : 1.0f;
  auto one = [&](float& v, float gi, float& x) {
    v = fmaf(scale, gi, momentum * v) * clip;
    x += v;
  };
  const int first = blockIdx.x * 256 + tid, stride = gridDim.x * 256;
#pragma unroll 4
  for (int i = first; i < P / 4; i += stride) {
    const float4 gi = reinterpret_cast<const float4*>(g)[i];
    float4 v = reinterpret_cast<float4*>(vel)[i], x = reinterpret_cast<float4*>(mu)[i];
    one(v.x, gi.x, x.x), one(v.y, gi.y, x.y), one(v.z, gi.z, x.z), one(v.w, gi.w, x.w);
    reinterpret_cast<float4*>(vel)[i] = v;
    reinterpret_cast<float4*>(mu)[i] = x;
  }
  if (first < (P & 3)) one(vel[(P & ~3) + first], g[(P & ~3) + first], mu[(P & ~3) + first]);
}

// Clip the velocity to max_speed and move mu.
__global__ __launch_bounds__(256) void clipup_apply_kernel(float* __restrict__ mu, float* __restrict__ vel, int P,
                                                           float max_speed, const float* __restrict__ part_v, int n_v) {
  __shared__ double red[256];
  const double speed = sqrt(total256(part_v, n_v, red));
  const float clip = speed > static_cast<double>(max_speed) ? static_cast<float>(static_cast<double>(max_speed) / speed) : 1.0f;
  const int first = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
#pragma unroll 4
  for (int i = first; i < P / 4; i += stride) {
    float4 v = reinterpret_cast<float4*>(vel)[i], x = reinterpret_cast<float4*>(mu)[i];
    v.x *= clip, v.y *= clip, v.z *= clip, v.w *= clip;
    x.x += v.x, x.y += v.y, x.z += v.z, x.w += v.w;
    reinterpret_cast<float4*>(vel)[i] = v;
    reinterpret_cast<float4*>(mu)[i] = x;
  }
  if (first < (P & 3)) {
    const int i = (P & ~3) + first;
    vel[i] *= clip;
    mu[i] += vel[i];
  }
}

// rows copies of the centre: params[r][i] = mu[i] (fp32) or its bfloat16 rounding.
template <typename OutT>
__global__ __launch_bounds__(256) void center_kernel(const float* __restrict__ mu, OutT* __restrict__ params, int P,
                                                     int rows) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= P) return;
  const float v = mu[i];
  for (int r = 0; r < rows; ++r) {
    if (sizeof(OutT) == 4) reinterpret_cast<float*>(params)[static_cast<size_t>(r) * P + i] = v;
    else reinterpret_cast<uint16_t*>(params)[static_cast<size_t>(r) * P + i] = to_bf16(v);
  }
}

// t <- value (set != 0) or t <- t + 1, by one thread, in stream order after the kernels that read t.
__global__ void generation_kernel(uint32_t* __restrict__ gen, uint32_t value, int set) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *gen = set ? value : *gen + 1u;
}

__global__ __launch_bounds__(256) void fill_kernel(float* __restrict__ p, size_t n, float value) {
  const size_t stride = static_cast<size_t>(gridDim.x) * 256;
  for (size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x; i < n; i += stride) p[i] = value;
}

static int fill(float* p, size_t n, float value, hipStream_t s) {
  if (n == 0) return EVO_OK;
  const unsigned blocks = static_cast<unsigned>(n / 256 + 1 < 4096 ? n / 256 + 1 : 4096);
  hipLaunchKernelGGL(fill_kernel, dim3(blocks), dim3(256), 0, s, p, n, value);
  return check_launch("fill_kernel");
}

__global__ __launch_bounds__(256) void philox_words_kernel(uint32_t gen, uint32_t pair, uint32_t block0,
                                                           uint32_t nblocks, uint32_t tag, uint32_t key0,
                                                           uint32_t key1, uint32_t* __restrict__ words,
                                                           float* __restrict__ normals) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= nblocks) return;
  if (words) {
    const u32x4 w = philox4x32_10(block0 + i, pair, gen, tag, key0, key1);
    reinterpret_cast<uint4*>(words)[i] = make_uint4(w.x, w.y, w.z, w.w);
  }
  if (normals) {
    float z[4];
    philox_normal4(block0 + i, pair, gen, tag, key0, key1, z);
    reinterpret_cast<float4*>(normals)[i] = make_float4(z[0], z[1], z[2], z[3]);
  }
}

static int launch_rank(const float* fitness, int pop, uint32_t* rank, float* shaped, float2* pairs, hipStream_t s) {
  if (pop > 1024)
    hipLaunchKernelGGL(rank_kernel<1024>, dim3((pop + 31) / 32), dim3(1024), 0, s, fitness, pop, rank, shaped, pairs);
  else
    hipLaunchKernelGGL(rank_kernel<256>, dim3((pop + 7) / 8), dim3(256), 0, s, fitness, pop, rank, shaped, pairs);
  return check_launch("rank_kernel");
}

static int check_cfg(const pgpe_config* c) {
  EVO_REQUIRE(c != nullptr, EVO_ERR_ARG, "pgpe_config is null");
  EVO_REQUIRE(c->P >= 1, EVO_ERR_ARG, "P must be >= 1 (got %d)", c->P);
  EVO_REQUIRE(c->pop_max >= 2 && c->pop_max <= EVO_POP_MAX && (c->pop_max & 1) == 0, EVO_ERR_ARG,
              "pop_max must be even and in [2, %d] (got %d)", EVO_POP_MAX, c->pop_max);
  EVO_REQUIRE(c->sigma_rule == 0 || c->sigma_rule == 1, EVO_ERR_ARG, "sigma_rule must be 0 or 1");
  EVO_REQUIRE(c->shaping == 0 || c->shaping == 1, EVO_ERR_ARG, "shaping must be 0 or 1");
  EVO_REQUIRE(c->beta1 >= 0.f && c->beta1 < 1.f && c->beta2 >= 0.f && c->beta2 < 1.f, EVO_ERR_ARG,
              "Adam betas must lie in [0,1)");
  EVO_REQUIRE(c->optimizer == EVO_OPT_ADAM || c->optimizer == EVO_OPT_CLIPUP || c->optimizer == EVO_OPT_MOMENTUM,
              EVO_ERR_ARG, "optimizer must be EVO_OPT_ADAM, EVO_OPT_CLIPUP or EVO_OPT_MOMENTUM (got %d)", c->optimizer);
  if (c->optimizer != EVO_OPT_ADAM)
    EVO_REQUIRE(c->momentum >= 0.f && c->momentum < 1.f, EVO_ERR_ARG, "momentum must lie in [0,1)");
  if (c->optimizer == EVO_OPT_CLIPUP) EVO_REQUIRE(c->max_speed > 0.f, EVO_ERR_ARG, "max_speed must be positive");
  return EVO_OK;
}

extern "C" float pgpe_clipup_default_max_speed(float lr_mu) { return 2.0f * lr_mu; }

extern "C" int pgpe_config_defaults(pgpe_config* cfg, int32_t P, int32_t pop_max) {
  EVO_REQUIRE(cfg != nullptr, EVO_ERR_ARG, "pgpe_config_defaults: cfg is null");
  cfg->P = P, cfg->pop_max = pop_max;
  cfg->sigma_init = 0.1f, cfg->lr_mu = 0.01f, cfg->lr_sigma = 0.1f, cfg->sigma_max_change = 0.2f;
  cfg->beta1 = 0.9f, cfg->beta2 = 0.999f, cfg->eps = 1e-8f;
  cfg->sigma_rule = 0, cfg->shaping = 1, cfg->optimizer = EVO_OPT_ADAM;
  cfg->momentum = 0.9f, cfg->max_speed = pgpe_clipup_default_max_speed(cfg->lr_mu);
  return EVO_OK;
}

static int check_ask_pop(const pgpe_state* st, int32_t pop, const char* who) {
  EVO_REQUIRE(pop >= 2 && (pop & 1) == 0 && pop <= st->cfg.pop_max, EVO_ERR_ARG,
              "%s: pop must be even and in [2, pop_max=%d] (got %d)", who, st->cfg.pop_max, pop);
  return EVO_OK;
}

// The device copy of t, or null while the state keeps t on the host only.
static const uint32_t* device_generation(const pgpe_state* st) {
  return st->device_t ? ws_carve(st->work, st->cfg.pop_max).gen : nullptr;
}

// What the calls that fuse ask into an evaluation (other source files) need of a state.
int pgpe_view(const pgpe_state* st, PgpeView* out) {
  EVO_REQUIRE(st != nullptr && out != nullptr, EVO_ERR_ARG, "pgpe state is null");
  out->mu = st->mu, out->sigma = st->sigma, out->P = st->cfg.P, out->t = st->t;
  out->gen_dev = device_generation(st);
  return EVO_OK;
}
int pgpe_check_ask(const pgpe_state* st, int32_t pop, const char* who) { return check_ask_pop(st, pop, who); }
void pgpe_note_ask(pgpe_state* st, uint64_t seed, int32_t pop) {
  st->pending = true;
  st->seed = seed;
  st->pop = pop;
}

// Host t -> device copy, in stream order.
static int write_device_generation(pgpe_state* st, hipStream_t s) {
  hipLaunchKernelGGL(generation_kernel, dim3(1), dim3(64), 0, s, ws_carve(st->work, st->cfg.pop_max).gen, st->t, 1);
  return check_launch("generation_kernel");
}

// Device copy -> host t; waits for the stream.
static int read_device_generation(pgpe_state* st, hipStream_t s) {
  uint32_t t = 0;
  hipError_t e = hipMemcpyAsync(&t, ws_carve(st->work, st->cfg.pop_max).gen, sizeof(t), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "reading the generation index back failed: %s", hipGetErrorString(e));
  st->t = t;
  return EVO_OK;
}

// After a tell: t <- t + 1, on the host and (in stream order) on the device.
static int advance_generation(pgpe_state* st, hipStream_t s) {
  st->pending = false;
  st->t += 1;
  if (!st->device_t) return EVO_OK;
  hipLaunchKernelGGL(generation_kernel, dim3(1), dim3(64), 0, s, ws_carve(st->work, st->cfg.pop_max).gen, 0u, 0);
  return check_launch("generation_kernel");
}

// The arguments of the tell kernels for the pending ask (theta: stored population or null) and the number of
// workgroups.
static TellArgs tell_args(const pgpe_state* st, const float* fitness, float* gmu, float* gsg, const float* theta,
                          unsigned* blocks_out) {
  const pgpe_config& c = st->cfg;
  const int N = st->pop / 2, P = c.P;
  Workspace ws = ws_carve(st->work, c.pop_max);
  TellArgs a;
  a.mu = st->mu, a.sigma = st->sigma, a.m = st->m, a.v = st->v;
  a.ms = st->aux, a.vs = st->aux ? st->aux + P : nullptr;
  a.gmu_out = gmu, a.gsg_out = gsg;
  a.pairs = ws.pairs, a.fitness = fitness, a.shaping = c.shaping;
  a.theta = theta;
  a.P = P, a.nquads = (P + 3) / 4, a.N = N;
  // split the pair loop KS ways until about 2^19 threads (eight waves per SIMD) are in flight:
  // measured, that is where the time stops falling, and beyond 64 slices the LDS reduction of
  // the partial sums costs more than it gains
  int KS = 1;
  const long threads_wanted = theta ? 262144 : 524288;
  while (KS < 64 && KS * 2 <= N && static_cast<long>(a.nquads) * KS < threads_wanted) KS *= 2;
  a.KS = KS;
  a.gen = st->t, a.key0 = static_cast<uint32_t>(st->seed), a.key1 = static_cast<uint32_t>(st->seed >> 32);
  a.gen_dev = st->device_t ? ws.gen : nullptr;
  a.inv_n = 1.0f / static_cast<float>(N);
  a.lr_mu = c.lr_mu, a.lr_sigma = c.lr_sigma, a.max_change = c.sigma_max_change;
  a.beta1 = c.beta1, a.beta2 = c.beta2, a.eps = c.eps, a.momentum = c.momentum;
  a.bc1 = static_cast<float>(1.0 / (1.0 - pow(static_cast<double>(c.beta1), static_cast<double>(st->t))));
  a.bc2 = static_cast<float>(1.0 / (1.0 - pow(static_cast<double>(c.beta2), static_cast<double>(st->t))));
  const int QPB = 256 / KS;
  *blocks_out = static_cast<unsigned>((a.nquads + QPB - 1) / QPB);
  // the words of the one-launch generation, which ClipUp never runs as, take the partial sums
  a.norm_part = c.optimizer == EVO_OPT_CLIPUP && *blocks_out <= kGradNormParts ? reinterpret_cast<float*>(ws.gen + 64) : nullptr;
  return a;
}

// Shared by pgpe_tell, pgpe_tell_stored and the gradient hook (theta: stored population or null).
static int run_tell(pgpe_state* st, const float* fitness, float* gmu, float* gsg, const float* theta,
                    hipStream_t s) {
  const pgpe_config& c = st->cfg;
  const int pop = st->pop, P = c.P;
  Workspace ws = ws_carve(st->work, c.pop_max);
  unsigned blocks;
  const TellArgs a = tell_args(st, fitness, gmu, gsg, theta, &blocks);
  const bool small = pop <= kSmallPairs && static_cast<long>(pop) * blocks <= kSmallWork;
  int rc = EVO_OK;
  if (!small) {
    if (c.shaping) {
      rc = launch_rank(fitness, pop, nullptr, nullptr, ws.pairs, s);
    } else {
      hipLaunchKernelGGL(raw_pairs_kernel, dim3(1), dim3(256), 0, s, fitness, pop, ws.pairs);
      rc = check_launch("raw_pairs_kernel");
    }
    if (rc) return rc;
  }
#define EVO_TELL_FORM(OPTV, SRV, STOREDV)                                                                            \
  do {                                                                                                               \
    if (small) hipLaunchKernelGGL((tell_kernel<OPTV, SRV, STOREDV, true>), dim3(blocks), dim3(256), 0, s, a);        \
    else hipLaunchKernelGGL((tell_kernel<OPTV, SRV, STOREDV, false>), dim3(blocks), dim3(256), 0, s, a);             \
  } while (0)
#define EVO_TELL(OPTV, SRV)                          \
  do {                                               \
    if (theta) EVO_TELL_FORM(OPTV, SRV, true);       \
    else EVO_TELL_FORM(OPTV, SRV, false);            \
  } while (0)
  if (gmu) {
    EVO_TELL(OPT_GRAD, 0);
  } else if (c.optimizer == EVO_OPT_ADAM) {
    if (c.sigma_rule == 0) EVO_TELL(OPT_ADAM, 0);
    else EVO_TELL(OPT_ADAM, 1);
  } else if (c.optimizer == EVO_OPT_MOMENTUM) {
    if (c.sigma_rule == 0) EVO_TELL(OPT_MOMENTUM, 0);
    else EVO_TELL(OPT_MOMENTUM, 1);
  } else {
    if (c.sigma_rule == 0) EVO_TELL(OPT_CLIPUP_GRAD, 0);
    else EVO_TELL(OPT_CLIPUP_GRAD, 1);
  }
#undef EVO_TELL
#undef EVO_TELL_FORM
  rc = check_launch("tell_kernel");
  if (rc || gmu || c.optimizer != EVO_OPT_CLIPUP) return rc;
  // ClipUp: |g|, velocity and its norm, clip and move; the gradient waits in v
  const int grid = (P + 1023) / 1024 < kNormBlocks ? (P + 1023) / 1024 : kNormBlocks;  // four parameters per thread
  if (a.norm_part) {
    hipLaunchKernelGGL(clipup_step_kernel, dim3(grid), dim3(256), 0, s, st->mu, st->m, st->v, P, c.momentum, c.lr_mu, c.max_speed,
                       a.norm_part, norm_sums(a.norm_part), static_cast<int>(blocks));
    return check_launch("clipup_step_kernel");
  }
  hipLaunchKernelGGL(sqnorm_kernel, dim3(kNormBlocks), dim3(256), 0, s, st->v, P, ws.norm);
  hipLaunchKernelGGL(clipup_velocity_kernel, dim3(grid), dim3(256), 0, s, st->m, st->v, P, c.momentum, c.lr_mu, ws.norm,
                     kNormBlocks, ws.norm + kNormBlocks);
  hipLaunchKernelGGL(clipup_apply_kernel, dim3(grid), dim3(256), 0, s, st->mu, st->m, P, c.max_speed,
                     ws.norm + kNormBlocks, grid);
  return check_launch("clipup kernels");
}

// One generation in one launch (see generation_small_kernel).  The caller has validated the task; this checks what
// the kernel itself needs and leaves the state as pgpe_ask followed by pgpe_tell would.
int pgpe_generation_small(pgpe_state* st, uint64_t seed, int32_t pop, const MlpShape& sh, const float* obs,
                          int64_t obs_stride, int B, int loss, const void* target, float scale, float* fitness,
                          hipStream_t s) {
  EVO_REQUIRE(st != nullptr, EVO_ERR_ARG, "pgpe_generation: state is null");
  int rc = check_ask_pop(st, pop, "pgpe_generation");
  if (rc) return rc;
  const pgpe_config& c = st->cfg;
  EVO_REQUIRE(sh.P == c.P, EVO_ERR_ARG, "pgpe_generation: the policy has %d parameters, the state %d", sh.P, c.P);
  EVO_REQUIRE(c.optimizer != EVO_OPT_CLIPUP, EVO_ERR_UNSUPPORTED,
              "pgpe_generation: ClipUp needs norms over all parameters between its steps (use ask, rollout, tell)");
  EVO_REQUIRE(c.P <= 8192 && sh.max_width <= 256, EVO_ERR_UNSUPPORTED,
              "pgpe_generation: at most 8192 parameters and widths up to 256 (got P = %d, width %d)", c.P, sh.max_width);
  // every waiting workgroup ranks the whole population by itself: beyond a few hundred members that tail is
  // longer than the launches it saves
  EVO_REQUIRE(pop <= 512, EVO_ERR_UNSUPPORTED, "pgpe_generation: at most 512 members (got %d)", pop);
  const uint64_t seed_before = st->seed;
  const int32_t pop_before = st->pop;
  st->seed = seed, st->pop = pop;  // what tell_args reads
  GenSmallArgs g;
  unsigned n_tell;
  g.tell = tell_args(st, nullptr, nullptr, nullptr, nullptr, &n_tell);
  g.mlp.sh = sh, g.mlp.params = nullptr, g.mlp.obs = obs, g.mlp.obs_stride = obs_stride, g.mlp.B = B;
  g.mlp.out = nullptr, g.mlp.target = target, g.mlp.partial = nullptr, g.mlp.fitness = nullptr;
  g.mlp.tiles = (B + kMlpTile - 1) / kMlpTile, g.mlp.ldw = sh.max_width, g.mlp.pop = pop;
  const long total = static_cast<long>(pop) * g.mlp.tiles;
  const size_t lds_a = sizeof(float) * (4 * static_cast<size_t>(g.tell.nquads) + 2 * static_cast<size_t>(g.mlp.ldw) * kMlpTile);
  const size_t lds_c = sizeof(float) * (256 * 8 + 4 * static_cast<size_t>((pop + 3) & ~3) + static_cast<size_t>(total));
  const size_t lds = lds_a > lds_c ? lds_a : lds_c;
  if (!(n_tell <= 128 && static_cast<long>(n_tell) <= total && total <= kSmallMaxTiles && lds <= 160 * 1024 - 64)) {
    st->seed = seed_before, st->pop = pop_before;
    EVO_REQUIRE(false, EVO_ERR_UNSUPPORTED,
                "pgpe_generation: %u update workgroups for %ld evaluation workgroups, %zu bytes of LDS: not a small problem",
                n_tell, total, lds);
  }
  static_assert(kSmallSumWords == 2 * kSmallMaxTiles && 4 * kSmallSumWords <= kGradNormBytes * kGradNormParts, "two words per sum, in the room");
  Workspace ws = ws_carve(st->work, c.pop_max);
  g.done = ws.gen + 16, g.launches = ws.gen + 32;  // inside the 256 bytes kept for the generation word
  g.sums = reinterpret_cast<uint64_t*>(ws.gen + 64);  // behind them
  if (!st->tickets_ready) {  // once per state: no launch so far, nothing has arrived, nobody has finished
    rc = fill(reinterpret_cast<float*>(g.done), 64 - 16 + kSmallSumWords, 0.f, s);
    if (rc) return rc;
    st->tickets_ready = true;
  }
  g.fitness = fitness, g.scale = scale;
  g.gen_rw = st->device_t ? ws.gen : nullptr;
  g.pop = pop, g.shaping = c.shaping, g.n_tell = static_cast<int>(n_tell), g.total = static_cast<int>(total);
  const dim3 grid(g.mlp.tiles, pop);
#define EVO_GEN(LOSSV, OPTV, SRV)                                                                               \
  do {                                                                                                          \
    auto kern = generation_small_kernel<LOSSV, OPTV, SRV>;                                                      \
    if (lds > 64 * 1024) {                                                                                      \
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                                   \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));    \
      if (e != hipSuccess) (void)hipGetLastError();                                                             \
      EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(e));        \
    }                                                                                                           \
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, s, g);                                                       \
  } while (0)
#define EVO_GEN_OPT(LOSSV)                                                                 \
  do {                                                                                     \
    if (c.optimizer == EVO_OPT_ADAM) {                                                     \
      if (c.sigma_rule == 0) EVO_GEN(LOSSV, OPT_ADAM, 0);                                  \
      else EVO_GEN(LOSSV, OPT_ADAM, 1);                                                    \
    } else {                                                                               \
      if (c.sigma_rule == 0) EVO_GEN(LOSSV, OPT_MOMENTUM, 0);                              \
      else EVO_GEN(LOSSV, OPT_MOMENTUM, 1);                                                \
    }                                                                                      \
  } while (0)
  if (loss == LOSS_CE) EVO_GEN_OPT(LOSS_CE);
  else EVO_GEN_OPT(LOSS_MSE);
#undef EVO_GEN_OPT
#undef EVO_GEN
  rc = check_launch("generation_small_kernel");
  if (rc) return rc;
  st->pending = false;  // asked and told
  st->t += 1;           // the device copy, if any, was advanced by the kernel
  return EVO_OK;
}

}  // namespace evo

using namespace evo;

extern "C" size_t pgpe_workspace_bytes(const pgpe_config* cfg) {
  if (check_cfg(cfg) != EVO_OK) return 0;
  return ws_bytes(cfg->pop_max);
}

extern "C" int pgpe_create(pgpe_state** out, const pgpe_config* cfg, float* mu_dev, float* sigma_dev,
                           float* m_dev, float* v_dev, float* aux_dev, void* work_dev) {
  EVO_REQUIRE(out != nullptr, EVO_ERR_ARG, "pgpe_create: out is null");
  *out = nullptr;
  int rc = check_cfg(cfg);
  if (rc) return rc;
  EVO_REQUIRE(mu_dev && sigma_dev && m_dev && v_dev && work_dev, EVO_ERR_ARG,
              "pgpe_create: mu, sigma, m, v and work must be non-null");
  EVO_REQUIRE(cfg->sigma_rule == 0 || aux_dev != nullptr, EVO_ERR_ARG,
              "pgpe_create: sigma_rule 1 needs aux_dev[2P]");
  EVO_REQUIRE(aligned16(mu_dev) && aligned16(sigma_dev) && aligned16(m_dev) && aligned16(v_dev) &&
                  aligned16(work_dev) && aligned16(aux_dev),
              EVO_ERR_ARG, "pgpe_create: device pointers must be 16-byte aligned");
  pgpe_state* st = new (std::nothrow) pgpe_state;
  EVO_REQUIRE(st != nullptr, EVO_ERR_ARG, "pgpe_create: out of host memory");
  st->cfg = *cfg;
  st->mu = mu_dev, st->sigma = sigma_dev, st->m = m_dev, st->v = v_dev, st->aux = aux_dev, st->work = work_dev;
  st->t = 1, st->device_t = false, st->pending = false, st->seed = 0, st->pop = 0, st->tickets_ready = false;
  *out = st;
  return EVO_OK;
}

extern "C" int pgpe_destroy(pgpe_state* st) {
  delete st;
  return EVO_OK;
}

extern "C" int pgpe_reset(pgpe_state* st, void* stream) {
  EVO_REQUIRE(st != nullptr, EVO_ERR_ARG, "pgpe_reset: state is null");
  hipStream_t s = as_stream(stream);
  const size_t P = static_cast<size_t>(st->cfg.P);
  int rc = fill(st->sigma, P, st->cfg.sigma_init, s);
  if (!rc) rc = fill(st->m, P, 0.f, s);
  if (!rc) rc = fill(st->v, P, 0.f, s);
  if (!rc && st->aux) rc = fill(st->aux, 2 * P, 0.f, s);
  st->t = 1;
  st->pending = false;
  if (!rc && st->device_t) rc = write_device_generation(st, s);
  return rc;
}

extern "C" int pgpe_device_generation(pgpe_state* st, const uint32_t** gen_dev_out, void* stream) {
  EVO_REQUIRE(st != nullptr, EVO_ERR_ARG, "pgpe_device_generation: state is null");
  EVO_REQUIRE(!st->pending, EVO_ERR_STATE, "pgpe_device_generation: an ask is pending (call it between tell and ask)");
  st->device_t = true;
  if (gen_dev_out) *gen_dev_out = ws_carve(st->work, st->cfg.pop_max).gen;
  return write_device_generation(st, as_stream(stream));
}

extern "C" int pgpe_sync_generation(pgpe_state* st, void* stream) {
  EVO_REQUIRE(st != nullptr, EVO_ERR_ARG, "pgpe_sync_generation: state is null");
  if (!st->device_t) return EVO_OK;
  return read_device_generation(st, as_stream(stream));
}

extern "C" int pgpe_center(const pgpe_state* st, int32_t rows, void* params_dev, int32_t dtype, void* stream) {
  EVO_REQUIRE(st != nullptr && params_dev != nullptr, EVO_ERR_ARG, "pgpe_center: null argument");
  EVO_REQUIRE(rows >= 1 && rows <= EVO_POP_MAX, EVO_ERR_ARG, "pgpe_center: rows must be in [1, %d] (got %d)",
              EVO_POP_MAX, rows);
  EVO_REQUIRE(dtype == EVO_F32 || dtype == EVO_BF16, EVO_ERR_ARG, "pgpe_center: bad dtype %d", dtype);
  const int P = st->cfg.P;
  const dim3 grid(static_cast<unsigned>((P + 255) / 256));
  if (dtype == EVO_F32)
    hipLaunchKernelGGL(center_kernel<float>, grid, dim3(256), 0, as_stream(stream), st->mu,
                       static_cast<float*>(params_dev), P, rows);
  else
    hipLaunchKernelGGL(center_kernel<uint16_t>, grid, dim3(256), 0, as_stream(stream), st->mu,
                       static_cast<uint16_t*>(params_dev), P, rows);
  return check_launch("center_kernel");
}

// ---- checkpoint: header + the state arrays, in host memory ---------------------------------------
namespace {
struct StateHeader {
  char magic[8];  // "EVOPGPE1"
  uint32_t header_bytes;
  uint32_t t;
  pgpe_config cfg;
};
const char kStateMagic[8] = {'E', 'V', 'O', 'P', 'G', 'P', 'E', '1'};

size_t state_bytes(const pgpe_config& c) {
  const size_t arrays = c.sigma_rule == 1 ? 6 : 4;  // mu, sigma, m, v (+ the two sigma moments)
  return sizeof(StateHeader) + arrays * static_cast<size_t>(c.P) * sizeof(float);
}

int copy_checked(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t s, const char* who) {
  hipError_t e = hipMemcpyAsync(dst, src, n, kind, s);
  if (e != hipSuccess) {
    set_error("%s: copy failed: %s", who, hipGetErrorString(e));
    return EVO_ERR_HIP;
  }
  return EVO_OK;
}
}  // namespace

extern "C" size_t pgpe_state_bytes(const pgpe_state* st) { return st ? state_bytes(st->cfg) : 0; }

extern "C" int pgpe_state_export(const pgpe_state* st, void* host_buf, size_t bytes, void* stream) {
  EVO_REQUIRE(st != nullptr && host_buf != nullptr, EVO_ERR_ARG, "pgpe_state_export: null argument");
  EVO_REQUIRE(bytes >= state_bytes(st->cfg), EVO_ERR_ARG, "pgpe_state_export: buffer of %zu bytes, %zu needed", bytes,
              state_bytes(st->cfg));
  EVO_REQUIRE(!st->pending, EVO_ERR_STATE, "pgpe_state_export: an ask is pending (export between tell and ask)");
  uint32_t t_now = st->t;
  if (st->device_t) {  // replays of a captured generation advance only the device copy
    hipError_t e = hipMemcpyAsync(&t_now, device_generation(st), sizeof(t_now), hipMemcpyDeviceToHost, as_stream(stream));
    if (e == hipSuccess) e = hipStreamSynchronize(as_stream(stream));
    EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "pgpe_state_export: %s", hipGetErrorString(e));
  }
  StateHeader h;
  memcpy(h.magic, kStateMagic, 8);
  h.header_bytes = sizeof(StateHeader);
  h.t = t_now;
  h.cfg = st->cfg;
  memcpy(host_buf, &h, sizeof(h));
  hipStream_t s = as_stream(stream);
  char* out = static_cast<char*>(host_buf) + sizeof(StateHeader);
  const size_t row = static_cast<size_t>(st->cfg.P) * sizeof(float);
  const float* arrays[6] = {st->mu, st->sigma, st->m, st->v, st->aux, st->aux ? st->aux + st->cfg.P : nullptr};
  const int n = st->cfg.sigma_rule == 1 ? 6 : 4;
  for (int i = 0; i < n; ++i)
    if (int rc = copy_checked(out + i * row, arrays[i], row, hipMemcpyDeviceToHost, s, "pgpe_state_export")) return rc;
  hipError_t e = hipStreamSynchronize(s);
  EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "pgpe_state_export: %s", hipGetErrorString(e));
  return EVO_OK;
}

extern "C" int pgpe_state_import(pgpe_state* st, const void* host_buf, size_t bytes, void* stream) {
  EVO_REQUIRE(st != nullptr && host_buf != nullptr, EVO_ERR_ARG, "pgpe_state_import: null argument");
  EVO_REQUIRE(bytes >= sizeof(StateHeader), EVO_ERR_ARG, "pgpe_state_import: buffer shorter than the header");
  StateHeader h;
  memcpy(&h, host_buf, sizeof(h));
  EVO_REQUIRE(memcmp(h.magic, kStateMagic, 8) == 0 && h.header_bytes == sizeof(StateHeader), EVO_ERR_ARG,
              "pgpe_state_import: not a state written by pgpe_state_export of this library version");
  EVO_REQUIRE(h.cfg.P == st->cfg.P && h.cfg.sigma_rule == st->cfg.sigma_rule, EVO_ERR_ARG,
              "pgpe_state_import: state has P = %d, sigma_rule = %d; the handle has P = %d, sigma_rule = %d", h.cfg.P,
              h.cfg.sigma_rule, st->cfg.P, st->cfg.sigma_rule);
  EVO_REQUIRE(h.t >= 1 && bytes >= state_bytes(st->cfg), EVO_ERR_ARG, "pgpe_state_import: truncated state");
  hipStream_t s = as_stream(stream);
  const char* in = static_cast<const char*>(host_buf) + sizeof(StateHeader);
  const size_t row = static_cast<size_t>(st->cfg.P) * sizeof(float);
  float* arrays[6] = {st->mu, st->sigma, st->m, st->v, st->aux, st->aux ? st->aux + st->cfg.P : nullptr};
  const int n = st->cfg.sigma_rule == 1 ? 6 : 4;
  for (int i = 0; i < n; ++i)
    if (int rc = copy_checked(arrays[i], in + i * row, row, hipMemcpyHostToDevice, s, "pgpe_state_import")) return rc;
  hipError_t e = hipStreamSynchronize(s);  // the host buffer may be released on return
  EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "pgpe_state_import: %s", hipGetErrorString(e));
  st->t = h.t;
  st->pending = false;
  return st->device_t ? write_device_generation(st, s) : EVO_OK;
}

extern "C" int pgpe_get_generation(const pgpe_state* st, uint32_t* t_out) {
  EVO_REQUIRE(st && t_out, EVO_ERR_ARG, "pgpe_get_generation: null argument");
  *t_out = st->t;
  return EVO_OK;
}

extern "C" int pgpe_set_generation(pgpe_state* st, uint32_t t) {
  EVO_REQUIRE(st != nullptr && t >= 1, EVO_ERR_ARG, "pgpe_set_generation: state null or t < 1");
  EVO_REQUIRE(!st->device_t, EVO_ERR_STATE,
              "pgpe_set_generation: the state keeps t on the device; use pgpe_state_import or pgpe_reset");
  st->t = t;
  st->pending = false;
  return EVO_OK;
}

extern "C" int pgpe_ask(pgpe_state* st, uint64_t seed, int32_t pop, void* params_dev, int32_t dtype,
                        void* stream) {
  EVO_REQUIRE(st != nullptr && params_dev != nullptr, EVO_ERR_ARG, "pgpe_ask: null argument");
  if (int rc = check_ask_pop(st, pop, "pgpe_ask")) return rc;
  EVO_REQUIRE(dtype == EVO_F32 || dtype == EVO_BF16, EVO_ERR_ARG, "pgpe_ask: bad dtype %d", dtype);
  EVO_REQUIRE(aligned16(params_dev), EVO_ERR_ARG, "pgpe_ask: params_dev must be 16-byte aligned");
  const int P = st->cfg.P, N = pop / 2;
  const size_t size = dtype == EVO_F32 ? 4 : 2;
  // one thread per 16 bytes of a row and pair, x fastest (see ask_block)
  const int pieces = dtype == EVO_F32 ? (P + 3) / 4 : (P + 7) / 8;
  const unsigned xblocks = static_cast<unsigned>((pieces + 255) / 256);
  const bool stream_stores = size * pop * P > (size_t(256) << 20);
  const size_t blocks = static_cast<size_t>(xblocks) * N;
  const size_t run = 8 * kAskRun;
  const dim3 grid = stream_stores ? dim3(xblocks, static_cast<unsigned>(N))
                                  : dim3(static_cast<unsigned>((blocks + run - 1) / run * run));
  hipStream_t s = as_stream(stream);
  const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
  const uint32_t* gen_dev = device_generation(st);
#define EVO_ASK(KERNEL, T)                                                                                            \
  hipLaunchKernelGGL((KERNEL), grid, dim3(256), 0, s, st->mu, st->sigma, static_cast<T*>(params_dev), P, pieces, xblocks, \
                     static_cast<unsigned>(N), st->t, gen_dev, k0, k1)
  if (dtype == EVO_F32) {
    if (stream_stores) EVO_ASK(ask_kernel<true>, float);
    else EVO_ASK(ask_kernel<false>, float);
  } else if ((P & 7) == 0) {
    if (stream_stores) EVO_ASK((ask_bf16_kernel<true, true>), uint16_t);
    else EVO_ASK((ask_bf16_kernel<true, false>), uint16_t);
  } else {
    if (stream_stores) EVO_ASK((ask_bf16_kernel<false, true>), uint16_t);
    else EVO_ASK((ask_bf16_kernel<false, false>), uint16_t);
  }
#undef EVO_ASK
  int rc = check_launch("ask_kernel");
  if (rc) return rc;
  st->pending = true;
  st->seed = seed;
  st->pop = pop;
  return EVO_OK;
}

extern "C" size_t pgpe_ask_sphere_workspace_bytes(const pgpe_config* cfg) {
  if (check_cfg(cfg) != EVO_OK) return 0;
  return (static_cast<size_t>(cfg->pop_max) * fused_xblocks(cfg->P) * sizeof(float) + 255) & ~size_t(255);
}

extern "C" int pgpe_ask_sphere(pgpe_state* st, uint64_t seed, int32_t pop, const float* x_star_dev,
                               float* fitness_dev, void* work_dev, void* stream) {
  EVO_REQUIRE(st && x_star_dev && fitness_dev && work_dev, EVO_ERR_ARG, "pgpe_ask_sphere: null argument");
  int rc = check_ask_pop(st, pop, "pgpe_ask_sphere");
  if (rc) return rc;
  EVO_REQUIRE(aligned16(x_star_dev) && aligned16(work_dev), EVO_ERR_ARG,
              "pgpe_ask_sphere: x_star_dev and work_dev must be 16-byte aligned");
  const int P = st->cfg.P, N = pop / 2, nquads = (P + 3) / 4, xblocks = fused_xblocks(P);
  hipStream_t s = as_stream(stream);
  float* part = static_cast<float*>(work_dev);
  const dim3 grid(static_cast<unsigned>(xblocks), static_cast<unsigned>((N + kFusedPairs - 1) / kFusedPairs));
  hipLaunchKernelGGL(ask_sphere_kernel, grid, dim3(256), 0, s, st->mu, st->sigma, x_star_dev, part, P, nquads, N,
                     xblocks, st->t, device_generation(st), static_cast<uint32_t>(seed),
                     static_cast<uint32_t>(seed >> 32));
  rc = check_launch("ask_sphere_kernel");
  if (rc) return rc;
  hipLaunchKernelGGL(sphere_finish_kernel, dim3(static_cast<unsigned>((pop + 3) / 4)), dim3(256), 0, s, part, xblocks,
                     pop, fitness_dev);
  rc = check_launch("sphere_finish_kernel");
  if (rc) return rc;
  st->pending = true;
  st->seed = seed;
  st->pop = pop;
  return EVO_OK;
}

extern "C" int pgpe_tell(pgpe_state* st, const float* fitness_dev, void* stream) {
  EVO_REQUIRE(st != nullptr && fitness_dev != nullptr, EVO_ERR_ARG, "pgpe_tell: null argument");
  EVO_REQUIRE(st->pending, EVO_ERR_STATE, "pgpe_tell: no pending ask");
  int rc = run_tell(st, fitness_dev, nullptr, nullptr, nullptr, as_stream(stream));
  if (rc) return rc;
  return advance_generation(st, as_stream(stream));
}

extern "C" int pgpe_tell_stored(pgpe_state* st, const float* fitness_dev, const float* params_dev, void* stream) {
  EVO_REQUIRE(st && fitness_dev && params_dev, EVO_ERR_ARG, "pgpe_tell_stored: null argument");
  EVO_REQUIRE(aligned16(params_dev), EVO_ERR_ARG, "pgpe_tell_stored: params_dev must be 16-byte aligned");
  EVO_REQUIRE(st->pending, EVO_ERR_STATE, "pgpe_tell_stored: no pending ask");
  int rc = run_tell(st, fitness_dev, nullptr, nullptr, params_dev, as_stream(stream));
  if (rc) return rc;
  return advance_generation(st, as_stream(stream));
}

extern "C" int evo_pgpe_gradients(pgpe_state* st, const float* fitness_dev, float* gmu_dev, float* gsigma_dev,
                                  const float* params_dev, void* stream) {
  EVO_REQUIRE(st && fitness_dev && gmu_dev && gsigma_dev, EVO_ERR_ARG, "evo_pgpe_gradients: null argument");
  EVO_REQUIRE(st->pending, EVO_ERR_STATE, "evo_pgpe_gradients: no pending ask");
  return run_tell(st, fitness_dev, gmu_dev, gsigma_dev, params_dev, as_stream(stream));
}

extern "C" int evo_centered_rank(const float* fitness_dev, int32_t pop, uint32_t* rank_dev, float* shaped_dev,
                                 void* stream) {
  EVO_REQUIRE(fitness_dev && rank_dev && shaped_dev, EVO_ERR_ARG, "evo_centered_rank: null argument");
  EVO_REQUIRE(pop >= 2 && pop <= EVO_POP_MAX, EVO_ERR_ARG, "evo_centered_rank: pop must be in [2, %d] (got %d)",
              EVO_POP_MAX, pop);
  return launch_rank(fitness_dev, pop, rank_dev, shaped_dev, nullptr, as_stream(stream));
}

static int philox_hook(uint64_t seed, uint32_t gen, uint32_t pair, uint32_t block0, uint32_t nblocks, uint32_t tag,
                       uint32_t* words, float* normals, void* stream) {
  EVO_REQUIRE(words || normals, EVO_ERR_ARG, "philox hook: output pointer is null");
  EVO_REQUIRE(aligned16(words) && aligned16(normals), EVO_ERR_ARG, "philox hook: output must be 16-byte aligned");
  if (nblocks == 0) return EVO_OK;
  hipLaunchKernelGGL(philox_words_kernel, dim3((nblocks + 255) / 256), dim3(256), 0, as_stream(stream), gen, pair,
                     block0, nblocks, tag, static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32), words,
                     normals);
  return check_launch("philox_words_kernel");
}

extern "C" int evo_philox_u32(uint64_t seed, uint32_t gen, uint32_t pair, uint32_t block0, uint32_t nblocks,
                              uint32_t tag, uint32_t* out_dev, void* stream) {
  return philox_hook(seed, gen, pair, block0, nblocks, tag, out_dev, nullptr, stream);
}

extern "C" int evo_philox_normal(uint64_t seed, uint32_t gen, uint32_t pair, uint32_t block0, uint32_t nblocks,
                                 uint32_t tag, float* out_dev, void* stream) {
  return philox_hook(seed, gen, pair, block0, nblocks, tag, nullptr, out_dev, stream);
}
