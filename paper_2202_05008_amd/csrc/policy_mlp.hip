// Population-batched fp32 MLP forward: every member has its own weights, observations are
// shared or per member (Section 2, "Global Policy"; Section 4, "Exploring Novel Policy
// Architectures": get_actions passes a batch through one model whose parameters are data).
// The loss epilogue makes a supervised single-step task (Section 3, "Supervised Learning
// Tasks") one kernel: logits never leave the chip.
//
// Mapping: workgroup = (member, tile of 64 samples).  Lane = sample, so an activation
// h[k][sample] is one conflict-free LDS read; the four waves take different groups of
// output neurons, whose weights W[k][o..] are contiguous and wave-uniform (LDS broadcasts; networks of
// more than kStagedParams parameters: scalar loads).
//
// Four kernels, chosen by mlp_form below: any fan-in of 64 or more runs on the matrix cores with fp32 operands as two-term
// scaled fp16 splits (mlp_f32_mfma_kernel or, the same bits, mlp_f32_short_kernel for wide layers and few workgroups;
// split16.h: three v_mfma_f32_16x16x32_f16 per product, fp32 accumulation);
// narrower networks on the fp32 matrix instruction (mlp_f32_units_kernel) or, small ones, on the vector ALU
// (mlp_f32_kernel).  The last two give the same bits, which are also those of the one-launch generation.
#include "kernels.h"
#include "mlp_f32_body.h"
#include "split16.h"

#include <algorithm>
#include <type_traits>

namespace evo {

typedef __attribute__((address_space(3))) const float* lds_cfloat_ptr;

// STAGED: the member's parameters pass through LDS, behind the activations; else they are read where they lie.
template <int LOSS, bool STAGED, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void mlp_f32_kernel(MlpArgs a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const float* theta = a.params + static_cast<size_t>(blockIdx.y) * a.sh.P;
  if (STAGED) {
    float* theta_lds = lds + 2 * a.ldw * kMlpTile;
    mlp_f32_body<LOSS, WAVES>(a, (lds_cfloat_ptr)theta_lds, blockIdx.y, blockIdx.x, lds, theta_lds, theta);
  } else {
    mlp_f32_body<LOSS, WAVES>(a, theta, blockIdx.y, blockIdx.x, lds);
  }
}

// Two tiles, all samples of a member, in one workgroup of two teams, which adds the two sums up as finalize_kernel would: no
// launch of that kernel.
template <int LOSS>
__global__ __launch_bounds__(512) void mlp_f32_pair_kernel(MlpArgs a, float* __restrict__ fitness) {
  extern __shared__ __attribute__((aligned(16))) float lds[];  // (and no other shared array: the parameters start on 16 bytes)
  const int team = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), tid = threadIdx.x & 255, member = blockIdx.x;
  float* theta_lds = lds + 4 * a.ldw * kMlpTile;
  float* sums = theta_lds + a.sh.P + 8;
  const float* theta = a.params + static_cast<size_t>(member) * a.sh.P;
  const float loss = mlp_f32_body<LOSS>(a, (lds_cfloat_ptr)theta_lds, member, team, lds + 2 * team * a.ldw * kMlpTile, theta_lds,
                                        team == 0 ? theta : nullptr, tid);
  if (tid == 0) sums[team] = loss;
  __syncthreads();
  if (threadIdx.x == 0) fitness[member] = a.scale * (sums[0] + sums[1]);
}

// ---- the matrix-core form ------------------------------------------------------------------------------
// Workgroup = (member, tile of 128 or 64 samples), eight waves (two per SIMD).  A wave owns sixteen samples from the
// observations to the loss: a layer is computed transposed on 16 x 16 tiles (rows = neurons: A operand, the member's
// weights; columns = samples: B operand), so a lane ends up with four consecutive neurons of one sample, and since the
// order in which a contraction runs over k is free, those four and the four of the next tile ARE the lane's eight k of
// the next layer's B operand (k = 32 s + 16 (e >> 2) + 4 q + (e & 3) for lane group q, element e).  Activations never
// leave the registers, and a layer needs no exchange between waves.
//
// The weights pass through LDS in chunks of sixteen units (eight in networks of widths up to 128; a unit = one neuron tile
// x 32 k), already split into two fp16 terms and in operand order, so that every wave's read is one conflict-free 16-byte access per lane.  The eight waves
// stage together and run ahead of their own products, across layers: while chunk i is consumed, chunk i + 1 is split
// and stored, the neurons' largest magnitudes of chunk i + 2 are published, and chunk i + 3 is on its way from memory.
// One barrier per chunk.  Out-of-range rows and columns are zeros by the buffer's own bounds check.
// Scales (powers of two, so that every finite fp32 value fits fp16's range): the weights of a NEURON from their largest
// magnitude; the activations of a SAMPLE from the largest magnitude among its outputs of the layer (in-lane maxima and
// two lane exchanges).  Both factors ride in the multiply-add that adds the bias.
// Bound by the issue of vector instructions and their latency at two waves per SIMD (staging, activations, the outputs'
// splits; vector pipe 45 %, matrix pipe 15 %, LDS 19 % busy).  Against the form it replaced, which kept activations in LDS, gathered every
// wave's own weights and split them for 64 samples at a time: 100-200-120-10, 500 members of 300 samples 235 -> 163 us;
// 64-256-256-16, 1024 of 512 926 -> 570 us; 128-128-128-8, 1000 of 200 258 -> 99 us; its error against 64 bits fell from
// 2.8e-7 to 2.1e-7 (64-256-256-16) with the cross terms in a chain of their own.
typedef float floatx4m __attribute__((ext_vector_type(4)));
constexpr int kMfmaMaxWidth = 256;             // fan-in and fan-out of a layer
constexpr int kMfmaWaves = 8;
constexpr int kMfmaUnitB = 2 * 64 * 16;        // two terms x 64 lanes x 16 bytes

// What follows the last layer on sixteen samples of a wave: lanes j, j + 16, j + 32, j + 48 have sample b's outputs,
// out(t, i) = neuron 16 t + 4 q + i.  Writes them, or returns the loss sum of the wave's live samples in every lane.
template <int NTM, int LOSS, int UNROLL = NTM, typename OUT>
__device__ __forceinline__ float mlp_finish(const MlpArgs& a, int member, int b, bool live, int A, int q, OUT out) {
  if (LOSS == LOSS_NONE) {
    if (!live) return 0.f;
    float* dst = a.out + (static_cast<size_t>(member) * a.B + b) * A;
    const bool wide = (A & 3) == 0 && (reinterpret_cast<uintptr_t>(a.out) & 15u) == 0;
#pragma unroll UNROLL
    for (int t = 0; t < NTM; ++t) {
      if (16 * t >= A) break;
      const int o = 16 * t + 4 * q;
      if (wide) {
        if (o < A) *reinterpret_cast<float4*>(dst + o) = make_float4(out(t, 0), out(t, 1), out(t, 2), out(t, 3));
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (o + i < A) dst[o + i] = out(t, i);
      }
    }
    return 0.f;
  }
  float loss = 0.f;
  {
    if (LOSS == LOSS_CE) {
      const int y = live ? min(max(static_cast<const int32_t*>(a.target)[b], 0), A - 1) : 0;  // labels outside [0, A) are clamped
      float mx = -__builtin_inff(), se = 0.f, hit = 0.f;
#pragma unroll UNROLL
      for (int t = 0; t < NTM; ++t) {
        if (16 * t >= A) break;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (16 * t + 4 * q + i < A) mx = fmaxf(mx, out(t, i));
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
#pragma unroll UNROLL
      for (int t = 0; t < NTM; ++t) {
        if (16 * t >= A) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int o = 16 * t + 4 * q + i;
          if (o < A) se += expf(out(t, i) - mx);
          if (o == y) hit = out(t, i);
        }
      }
      se += __shfl_xor(se, 16, 64);
      se += __shfl_xor(se, 32, 64);
      hit += __shfl_xor(hit, 16, 64);
      hit += __shfl_xor(hit, 32, 64);
      loss = live && q == 0 ? (mx + logf(se)) - hit : 0.f;
    } else {
      // the targets of eight tiles are on their way together (fetched and used one tile after the other they took 5 of the
      // 29 us of 256-256 on 64 samples)
      constexpr int kAhead = NTM < 8 ? NTM : 8;
      const int first = __builtin_amdgcn_readfirstlane(b), j = b - first;
      const float* tg = static_cast<const float*>(a.target) + (static_cast<size_t>(member) * a.B + first) * A;
      const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(tg), 0, 4 * max(0, min(a.B - first, 16)) * A, 0x00020000);
      const bool wide = (A & 3) == 0 && (reinterpret_cast<uintptr_t>(a.target) & 15u) == 0;
#pragma unroll UNROLL
      for (int t0 = 0; t0 < NTM; t0 += kAhead) {
        if (16 * t0 >= A) break;
        float y[kAhead][4];
#pragma unroll
        for (int t = 0; t < kAhead; ++t) {
          if (16 * (t0 + t) >= A) break;
          const int o = 16 * (t0 + t) + 4 * q;
          if (wide) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(rows, o < A ? 4u * (j * A + o) : 0x40000000u, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) y[t][i] = __uint_as_float(v[i]);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              y[t][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, o + i < A ? 4u * (j * A + o + i) : 0x40000000u, 0, 0));
          }
        }
#pragma unroll
        for (int t = 0; t < kAhead; ++t) {
          if (16 * (t0 + t) >= A) break;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (live && 16 * (t0 + t) + 4 * q + i < A) {
              const float d = out(t0 + t, i) - y[t][i];
              loss = fmaf(d, d, loss);
            }
          }
        }
      }
    }
  }
  return wave_sum(loss);
}

// One layer as the staging sees it (wave-uniform).
struct MfmaCursor {
  int l, tile;        // layer, first neuron tile of the chunk
  int off;            // the layer's first parameter
  int lg;             // log2 of the units per neuron tile (k steps rounded up to a power of two)
};

// KSM: k steps of the widest fan-in; the tiles of a layer's outputs are 2 KSM at most.
template <int KSM, int LOSS>
__global__ __launch_bounds__(64 * kMfmaWaves, KSM <= 4 ? 4 : 2) void mlp_f32_mfma_kernel(MlpArgs a, int wg_tiles) {
  constexpr int kUnits = KSM <= 4 ? 8 : 16;     // units per chunk
  constexpr int kChunkB = kUnits * kMfmaUnitB;
  __shared__ __attribute__((aligned(16))) unsigned char buf_s[2 * kChunkB + 2 * kMfmaUnitB];  // (+ reads one step ahead)
  __shared__ uint32_t max_s[3][kUnits * 16];    // [tile of the chunk][neuron]: largest magnitude (bits of |w|)
  __shared__ __attribute__((aligned(16))) float uw_s[2][kUnits][16];    // [tile of the chunk][neuron]: 1 / scale
  __shared__ __attribute__((aligned(16))) float bias_s[2][kUnits][16];
  __shared__ float red_s[kMfmaWaves];
  constexpr int NTM = 2 * KSM;
  constexpr int UR = kUnits / kMfmaWaves;   // units a wave stages per chunk
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, q = lane >> 4;
  // Workgroup -> (member, tile): consecutive workgroup numbers go to the eight dies in turn, each with a cache
  // of its own, so a member's tiles, which read the same weights, take numbers that are 8 apart.
  const int wgs = (a.tiles + wg_tiles - 1) / wg_tiles;
  const int die = blockIdx.x & 7, turn = blockIdx.x >> 3;
  const int member = 8 * (turn / wgs) + die, b0 = (turn % wgs) * wg_tiles * kMlpTile;
  if (member >= a.pop) return;
  const float* theta = a.params + static_cast<size_t>(member) * a.sh.P;
  const float* obs = a.obs + static_cast<size_t>(member) * a.obs_stride;
  const int n_layers = a.sh.n_layers;
  const int b = b0 + 16 * wave + j;                                        // this lane's sample
  const bool works = wave < 4 * wg_tiles && b0 + 16 * wave < a.B;          // the wave has samples at all
  const bool live = works && b < a.B;

  // ---- staging --------------------------------------------------------------------------------------------
  // tiles of layer l: an even number, so that its outputs fill the next fan-in up to a multiple of 32
  auto tiles_of = [&](int l) { return ((a.sh.dims[l + 1] + 31) & ~31) >> 4; };
  auto lg_of = [&](int l) {
    const int K = a.sh.dims[l];
    return K <= 32 ? 0 : K <= 64 ? 1 : K <= 128 ? 2 : 3;
  };
  float rl[UR][8], rs[UR][8], bl[UR], bs[UR];    // raw weights on their way / waiting to be split
  int lg_l, lg_s;                                // log2 units per tile of those chunks
  MfmaCursor cur = {0, 0, 0, lg_of(0)};
  auto load_chunk = [&](float (&raw)[UR][8], float (&bias)[UR], int& lg) {
    lg = cur.lg;
    // behind the last layer the buffer is empty: zeros without an access
    const bool more = cur.l < n_layers;
    const int K = more ? a.sh.dims[cur.l] : 0, N = more ? a.sh.dims[cur.l + 1] : 0;
    const auto w = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(theta + cur.off), 0, 4 * K * N, 0x00020000);
    const auto wb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(theta + cur.off + K * N), 0, 4 * N, 0x00020000);
#pragma unroll
    for (int r = 0; r < UR; ++r) {
      const int u = wave + kMfmaWaves * r, st = u & ((1 << cur.lg) - 1);
      const int n = 16 * (cur.tile + (u >> cur.lg)) + j;
      const unsigned at = n < N ? 4u * static_cast<unsigned>((32 * st + 4 * q) * N + n) : 0x40000000u;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        raw[r][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(w, at + 4u * N * (16 * (e >> 2) + (e & 3)), 0, 0));
      bias[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wb, 4u * n, 0, 0));
    }
    cur.tile += kUnits >> cur.lg;
    if (more && cur.tile >= tiles_of(cur.l)) {
      cur.off += K * N + N;
      cur.tile = 0;
      ++cur.l;
      if (cur.l < n_layers) cur.lg = lg_of(cur.l);
    }
  };
  auto publish_maxima = [&](int third) {
#pragma unroll
    for (int r = 0; r < UR; ++r) {
      float m = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(rs[r][e]));
      atomicMax(&max_s[third][16 * ((wave + kMfmaWaves * r) >> lg_s) + j], __float_as_uint(m));
    }
  };
  auto take_arrived = [&]() {
#pragma unroll
    for (int r = 0; r < UR; ++r) {
#pragma unroll
      for (int e = 0; e < 8; ++e) rs[r][e] = rl[r][e];
      bs[r] = bl[r];
    }
    lg_s = lg_l;
  };
  auto split_chunk = [&](int slot, int third) {
#pragma unroll
    for (int r = 0; r < UR; ++r) {
      const int u = wave + kMfmaWaves * r, first = u >> lg_s << lg_s;
      const float m = __uint_as_float(max_s[third][16 * (u >> lg_s) + j]);
      const float s_w = split_pow2_scale(m);
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = rs[r][e] * s_w;
      f16x8 lead, resid;
      split2_x8_true<false>(x, lead, resid);
      unsigned char* dst = buf_s + slot * kChunkB + u * kMfmaUnitB + 16 * lane;
      *reinterpret_cast<f16x8*>(dst) = lead;
      *reinterpret_cast<f16x8*>(dst + kMfmaUnitB / 2) = resid;
      if (u == first && q == 0) {
        uw_s[slot][u >> lg_s][j] = pow2_reciprocal(s_w);
        bias_s[slot][u >> lg_s][j] = bs[r];
      }
    }
  };
  load_chunk(rs, bs, lg_s);
  load_chunk(rl, bl, lg_l);
  for (int i = tid; i < 3 * kUnits * 16; i += 64 * kMfmaWaves) max_s[0][i] = 0u;

  // ---- observations: laid out as a layer's outputs are, held[tile][i] = feature 16 tile + 4 q + i of the sample -----
  float held[NTM][4];
  {
    const int D = a.sh.dims[0];
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(obs + static_cast<size_t>(b0) * D), 0,
                                                        4 * min(a.B - b0, kMlpTile * wg_tiles) * D, 0x00020000);
    const unsigned row = live ? 4u * (b - b0) * D : 0x40000000u;
    if ((D & 3) == 0 && (reinterpret_cast<uintptr_t>(obs) & 15u) == 0) {  // then every row starts on 16 bytes
#pragma unroll
      for (int t = 0; t < NTM; ++t) {
        const int d = 16 * t + 4 * q;
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rows, d < D ? row + 4u * d : 0x40000000u, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) held[t][i] = __uint_as_float(v[i]);
      }
    } else {
#pragma unroll
      for (int t = 0; t < NTM; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = 16 * t + 4 * q + i;
          held[t][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, d < D ? row + 4u * d : 0x40000000u, 0, 0));
        }
    }
  }

  __syncthreads();
  publish_maxima(0);
  __syncthreads();
  split_chunk(0, 0);
  take_arrived();
  publish_maxima(1);
  load_chunk(rl, bl, lg_l);

  // The two waves of a SIMD take a chunk's two kinds of work in opposite order, so that one's matrix instructions run
  // beside the other's vector instructions: four waves stage right behind the barrier, the others ahead of the next
  // one (with 64 samples: the four that have none, beside the other four's products).
  const bool early = (wave < 4) == (wg_tiles == 2);
  bool pending = false;
  int slot = 1;       // buffer of the chunk that is consumed
  int third = 2;      // that chunk's number modulo 3: its place among the maxima
  auto stage = [&]() {
    const int next = third == 2 ? 0 : third + 1, after = next == 2 ? 0 : next + 1;
    if (tid < kUnits * 16) max_s[third][tid] = 0u;   // for the chunk after the next two (last read before the barrier)
    split_chunk(slot ^ 1, next);
    take_arrived();
    publish_maxima(after);
    load_chunk(rl, bl, lg_l);
  };
  auto next_chunk = [&]() {
    slot ^= 1;
    third = third == 2 ? 0 : third + 1;
    __syncthreads();  // chunk i is in LDS, chunk i - 1 is done with, the maxima of chunk i + 1 are out
  };
  for (int l = 0; l < n_layers; ++l) {
    const int K = a.sh.dims[l], act = a.sh.act[l];
    const int KS = (K + 31) >> 5, NT = tiles_of(l), lg = lg_of(l), in_chunk = (kUnits >> lg) - 1;
    // ---- the layer's input: the sample's scale from its largest magnitude, two fp16 terms ----
    f16x8 xb[2][KSM];
    float u_s;
    {
      float m = 0.f;
#pragma unroll
      for (int t = 0; t < NTM; ++t)
        if (t < 2 * KS) m = fmaxf(fmaxf(m, fmaxf(fabsf(held[t][0]), fabsf(held[t][1]))), fmaxf(fabsf(held[t][2]), fabsf(held[t][3])));
      m = fmaxf(m, __shfl_xor(m, 16, 64));
      m = fmaxf(m, __shfl_xor(m, 32, 64));
      const float sc = split_pow2_scale(m);
      u_s = pow2_reciprocal(sc);
#pragma unroll
      for (int st = 0; st < KSM; ++st) {
        if (st < KS) {
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = sc * held[2 * st + (e >> 2)][e & 3];
          split2_x8_true<false>(x, xb[0][st], xb[1][st]);
        }
      }
    }
    // ---- its neurons, two tiles at a time ----
#pragma unroll
    for (int t = 0; t < NTM; t += 2) {
      if (t >= NT) break;
      const bool boundary = (t & in_chunk) == 0;
      if (early && boundary) next_chunk();
      if (early ? boundary : pending) {
        stage();
        pending = false;
      }
      if (!early && boundary) {
        next_chunk();
        pending = true;
      }
      if (!works) continue;
      // leading products and cross terms apart: two chains per tile, and the large sum is rounded once per step
      floatx4m acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, cross[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
      const int at = t & in_chunk;
      const unsigned char* src0 = buf_s + slot * kChunkB + (at << lg) * kMfmaUnitB + 16 * lane;
      const unsigned char* src1 = src0 + (kMfmaUnitB << lg);
      f16x8 w[2][2][2];  // [step parity][tile][term]
      auto fetch = [&](int st) {
#pragma unroll
        for (int term = 0; term < 2; ++term) {
          w[st & 1][0][term] = *reinterpret_cast<const f16x8*>(src0 + st * kMfmaUnitB + term * (kMfmaUnitB / 2));
          w[st & 1][1][term] = *reinterpret_cast<const f16x8*>(src1 + st * kMfmaUnitB + term * (kMfmaUnitB / 2));
        }
      };
      __builtin_amdgcn_s_setprio(1);
      fetch(0);
      float4 u4[2], b4[2];
      auto factors = [&]() {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          u4[k] = *reinterpret_cast<const float4*>(&uw_s[slot][at + k][4 * q]);
          b4[k] = *reinterpret_cast<const float4*>(&bias_s[slot][at + k][4 * q]);
        }
      };
      if (KSM > 4) factors();  // ahead of the products where there are registers for that
#pragma unroll
      for (int st = 0; st < KSM; ++st) {
        if (st >= KS) break;
        if (st + 1 < KSM) fetch(st + 1);  // (behind the last step: read and not used)
#pragma unroll
        for (int k = 0; k < 2; ++k) cross[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[st & 1][k][0], xb[1][st], cross[k], 0, 0, 0);
#pragma unroll
        for (int k = 0; k < 2; ++k) acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[st & 1][k][0], xb[0][st], acc[k], 0, 0, 0);
#pragma unroll
        for (int k = 0; k < 2; ++k) cross[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[st & 1][k][1], xb[0][st], cross[k], 0, 0, 0);
      }
      __builtin_amdgcn_s_setprio(0);
      if (KSM <= 4) factors();
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        held[t + k][0] = fmaf(acc[k][0] + cross[k][0], u_s * u4[k].x, b4[k].x);
        held[t + k][1] = fmaf(acc[k][1] + cross[k][1], u_s * u4[k].y, b4[k].y);
        held[t + k][2] = fmaf(acc[k][2] + cross[k][2], u_s * u4[k].z, b4[k].z);
        held[t + k][3] = fmaf(acc[k][3] + cross[k][3], u_s * u4[k].w, b4[k].w);
      }
      // the activation of the tiles' eight values per lane, switched once and not per value
      auto apply = [&](auto f) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int i = 0; i < 4; ++i) held[t + k][i] = f(held[t + k][i]);
      };
      if (act == EVO_ACT_TANH) apply([](float x) { return tanh_fast_accurate(x); });
      else if (act == EVO_ACT_RELU) apply([](float x) { return fmaxf(x, 0.f); });
    }
  }

  const float loss = works ? mlp_finish<NTM, LOSS>(a, member, b, live, a.sh.dims[n_layers], q, [&](int t, int i) { return held[t][i]; }) : 0.f;
  if (LOSS == LOSS_NONE) return;
  if (lane == 0) red_s[wave] = loss;
  __syncthreads();
  auto sum64 = [&](int tile) { return (red_s[4 * tile] + red_s[4 * tile + 1]) + (red_s[4 * tile + 2] + red_s[4 * tile + 3]); };
  if (a.fitness) {  // one or two sums: finalize_kernel's butterfly adds nothing but zeros to them
    if (tid == 0) a.fitness[member] = a.scale * (a.tiles == 2 ? sum64(0) + sum64(1) : sum64(0));
  } else if (tid < wg_tiles && b0 / kMlpTile + tid < a.tiles) {  // one partial sum per 64 samples
    a.partial[static_cast<size_t>(member) * a.tiles + b0 / kMlpTile + tid] = sum64(tid);
  }
}

// ---- the split form for few workgroups ------------------------------------------------------------------------
// The same sums, bit for bit, shared out the other way round: a wave takes neurons instead of samples.  With few
// workgroups, or samples for half of a workgroup's waves only, the form above is a chain through every neuron tile per
// wave, one chunk of weights waiting for the other; here the waves work on a layer's tiles side by side, each reading its
// own neurons' weights.  It pays from layers of 192 to 192 on, whose eight waves all have tiles, and where no fan-in is
// ragged (clamped addresses and zeroes per weight then cost more than the other form's bounds checks).  In us, that form
// and this one: 64-256-256-16 128 members of 64 samples 31.7 and 28.9, one member of 2000 33.6 and 29.3, 4096 of 64 529 and
// 518; 256-256-16 one of 300 24.2 and 20.6; 64-192-192-16 1000 of 64 101 and 92; against it 240-240-16 200 of 64 25.2 and
// 27.6, 200-200-200-20 4096 of 64 609 and 649, 256-40-10 one of 300 12.0 and 13.4.
// Workgroup = (member, tile of 64 samples), eight waves (two per SIMD).  A layer is computed transposed: rows of a
// 16 x 16 tile are neurons (A operand: the member's weights, fetched one tile ahead of their use and split once per neuron
// tile), columns are samples (B operand: the layer's input, kept in LDS as two fp16 terms [term][sample][k], the eight k of
// a lane group side by side: one 16-byte read per term and 32 k).  A lane then ends up with four consecutive neurons of one
// sample: bias, activation, and one 8-byte LDS store per term hand them to the next layer.  Wave w takes neuron tiles
// w, w + 8, ...; its outputs wait in registers until every wave has finished reading the layer's input, which they then
// overwrite.  Scales as above: the weights of a neuron, the activations of a sample (in-lane maxima, two lane exchanges,
// one LDS word per wave and sample).
constexpr int kMfmaKSteps = kMfmaMaxWidth / 32;
constexpr int kMfmaSlots = kMfmaMaxWidth / 16 / kMfmaWaves;  // neuron tiles per wave
// Place of a layer's input k among a sample's: lane group q of a step has k = 16 h + 4 q + e (h = 0, 1, e = 0..3).
__device__ __forceinline__ int short_place(int k) { return (k & ~31) + 8 * ((k >> 2) & 3) + 4 * ((k >> 4) & 1) + (k & 3); }

template <int LOSS>
__global__ __launch_bounds__(64 * kMfmaWaves, 2) void mlp_f32_short_kernel(MlpArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  constexpr int TB = kMlpTile;
  static_assert(TB == 64, "four column tiles of 16 samples");
  const int kRowB = (a.ldw + 8) * 2;       // bytes of one sample's row of one term (a.ldw: widest padded fan-in)
  const int kTermB = TB * kRowB;
  __shared__ float red_s[4];
  unsigned char* at = lds_raw;                                    // [2][64][ldw + 8] fp16
  float* smax = reinterpret_cast<float*>(lds_raw + 2 * kTermB);   // [8][64] per wave: largest |output| of a sample
  float* us_s = smax + kMfmaWaves * TB;                                    // [64] 1 / scale of the staged observations
  float* fin = reinterpret_cast<float*>(lds_raw);                 // [A][64] network output (after the last layer)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, q = lane >> 4;
  // Workgroup -> (member, tile): consecutive workgroup numbers go to the eight dies in turn, each with a cache
  // of its own, so a member's tiles, which read the same weights, take numbers that are 8 apart.
  const int die = blockIdx.x & 7, turn = blockIdx.x >> 3;
  const int member = 8 * (turn / a.tiles) + die, tile = turn % a.tiles, b0 = tile * TB;
  if (member >= a.pop) return;
  const float* theta = a.params + static_cast<size_t>(member) * a.sh.P;
  const float* obs = a.obs + static_cast<size_t>(member) * a.obs_stride;

  // ---- observations -> two fp16 terms per value, scaled per sample (eight threads per sample) --------------
  {
    const int D = a.sh.dims[0], KP = (D + 31) & ~31;
    const int smp = tid >> 3, part = tid & 7;
    const bool live = b0 + smp < a.B;
    const float* row = obs + static_cast<size_t>(b0 + smp) * D;
    float sc;
    if ((D & 3) == 0 && (reinterpret_cast<uintptr_t>(obs) & 15u) == 0) {  // then every row starts on 16 bytes
      // every 16-byte load of the thread's share of the row is in flight at once: one trip to memory
      float4 v[kMfmaMaxWidth / 32];
      float m = 0.f;
#pragma unroll
      for (int c = 0; c < kMfmaMaxWidth / 32; ++c) {
        const int d = 4 * (part + 8 * c);
        v[c] = (live && d < D) ? *reinterpret_cast<const float4*>(row + d) : make_float4(0.f, 0.f, 0.f, 0.f);
        m = fmaxf(fmaxf(m, fmaxf(fabsf(v[c].x), fabsf(v[c].y))), fmaxf(fabsf(v[c].z), fabsf(v[c].w)));
      }
      m = fmaxf(m, __shfl_xor(m, 1, 64));
      m = fmaxf(m, __shfl_xor(m, 2, 64));
      m = fmaxf(m, __shfl_xor(m, 4, 64));
      sc = split_pow2_scale(m);
#pragma unroll
      for (int c = 0; c < kMfmaMaxWidth / 32; ++c) {
        const int d = 4 * (part + 8 * c);
        if (d < KP) {
          uint2 lead, resid;
          split2_pair_true(sc * v[c].x, sc * v[c].y, lead.x, resid.x);
          split2_pair_true(sc * v[c].z, sc * v[c].w, lead.y, resid.y);
          *reinterpret_cast<uint2*>(at + smp * kRowB + short_place(d) * 2) = lead;
          *reinterpret_cast<uint2*>(at + kTermB + smp * kRowB + short_place(d) * 2) = resid;
        }
      }
    } else {
      float m = 0.f;
      for (int d = part; d < D; d += 8) m = fmaxf(m, live ? fabsf(row[d]) : 0.f);
      m = fmaxf(m, __shfl_xor(m, 1, 64));
      m = fmaxf(m, __shfl_xor(m, 2, 64));
      m = fmaxf(m, __shfl_xor(m, 4, 64));
      sc = split_pow2_scale(m);
      for (int d = 2 * part; d < KP; d += 16) {
        const float x0 = (live && d < D) ? sc * row[d] : 0.f, x1 = (live && d + 1 < D) ? sc * row[d + 1] : 0.f;
        uint32_t lead, resid;
        split2_pair_true(x0, x1, lead, resid);
        *reinterpret_cast<uint32_t*>(at + smp * kRowB + short_place(d) * 2) = lead;
        *reinterpret_cast<uint32_t*>(at + kTermB + smp * kRowB + short_place(d) * 2) = resid;
      }
    }
    if (part == 0) us_s[smp] = pow2_reciprocal(sc);
  }
  __syncthreads();
  float u_s[4];  // 1 / scale of the stored input of sample 16 ct + j
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) u_s[ct] = us_s[16 * ct + j];

  // A neuron tile's weights as A operands, A[row j][k = 32 s + 16 (e >> 2) + 4 q + (e & 3)] = W[k][16 nt + j], and its four biases
  // per lane, are fetched one tile ahead: all 64 loads of the next tile are in flight while the matrix
  // instructions of this one run.
  float raw[kMfmaKSteps][8], bias4[4];
  const int n_layers = a.sh.n_layers;
  auto tiles_of = [&](int l) {  // neuron tiles of layer l: its outputs fill the next fan-in up to a multiple of 32
    const int N = a.sh.dims[l + 1];
    return l == n_layers - 1 ? (N + 15) >> 4 : ((N + 31) & ~31) >> 4;
  };
  // Fetches this wave's first tile at or after (layer l, slot).  Loads go to clamped addresses, so that none is
  // predicated or waited for here; what lies beyond the layer's fan-in or fan-out is zeroed where the tile is used.
  auto fetch_from = [&](int l, int slot, const float* W) {
    while (l < n_layers && !(slot < kMfmaSlots && wave + kMfmaWaves * slot < tiles_of(l))) {
      W += a.sh.dims[l] * a.sh.dims[l + 1] + a.sh.dims[l + 1];
      ++l, slot = 0;
    }
    if (l >= n_layers) return;
    const int K = a.sh.dims[l], N = a.sh.dims[l + 1], nt = wave + kMfmaWaves * slot;
    const int KS = (K + 31) >> 5;
    // address = a wave-uniform row pointer + an unsigned per-lane offset (no per-load vector arithmetic); only
    // a ragged last step clamps its rows per lane
    const unsigned lane_off = 4u * static_cast<unsigned>(4 * q * N + min(16 * nt + j, N - 1));  // bytes
#pragma unroll
    for (int st = 0; st < kMfmaKSteps; ++st) {
      if (st < KS) {
        if (32 * st + 32 <= K) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            raw[st][e] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(W + (32 * st + 16 * (e >> 2) + (e & 3)) * N) + lane_off);
        } else {
          const unsigned col = static_cast<unsigned>(min(16 * nt + j, N - 1));
#pragma unroll
          for (int e = 0; e < 8; ++e) raw[st][e] = W[static_cast<unsigned>(min(32 * st + 16 * (e >> 2) + 4 * q + (e & 3), K - 1) * N) + col];
        }
      }
    }
    const float* bias = W + K * N;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = 16 * nt + 4 * q + i;
      bias4[i] = bias[min(o, N - 1)];
    }
  };
  fetch_from(0, 0, theta);

  int off = 0;
  for (int l = 0; l < n_layers; ++l) {
    const int K = a.sh.dims[l], N = a.sh.dims[l + 1], act = a.sh.act[l];
    const bool last = l == n_layers - 1;
    const int KS = (K + 31) >> 5;
    const int NT = tiles_of(l);
    const float* W = theta + off;
    float held[kMfmaSlots][4][4];  // [slot][sample tile][neuron 4 q + i]: this wave's outputs of the layer
    float m_s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int slot = 0; slot < kMfmaSlots; ++slot) {
      const int nt = wave + kMfmaWaves * slot;
      if (nt >= NT) continue;
      // ---- zeros beyond a ragged fan-in or fan-out, scale from the neuron's largest magnitude, split ----
      if ((K & 31) != 0 || 16 * nt + 16 > N) {
        const bool ok = 16 * nt + j < N;
#pragma unroll
        for (int st = 0; st < kMfmaKSteps; ++st) {
          if (st < KS) {
#pragma unroll
            for (int e = 0; e < 8; ++e) raw[st][e] = (ok && 32 * st + 16 * (e >> 2) + 4 * q + (e & 3) < K) ? raw[st][e] : 0.f;
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) bias4[i] = 16 * nt + 4 * q + i < N ? bias4[i] : 0.f;
      }
      float w_max = 0.f;
#pragma unroll
      for (int st = 0; st < kMfmaKSteps; ++st) {
        if (st < KS) {
#pragma unroll
          for (int e = 0; e < 8; ++e) w_max = fmaxf(w_max, fabsf(raw[st][e]));
        }
      }
      w_max = fmaxf(w_max, __shfl_xor(w_max, 16, 64));
      w_max = fmaxf(w_max, __shfl_xor(w_max, 32, 64));
      const float s_w = split_pow2_scale(w_max);
      float u_w[4];  // 1 / scale of the neurons 4 q + i
#pragma unroll
      for (int i = 0; i < 4; ++i) u_w[i] = __shfl(pow2_reciprocal(s_w), 4 * q + i, 64);
      f16x8 wa[2][kMfmaKSteps];
#pragma unroll
      for (int st = 0; st < kMfmaKSteps; ++st) {
        if (st < KS) {
#pragma unroll
          for (int e = 0; e < 8; ++e) raw[st][e] *= s_w;
          split2_x8_true<false>(raw[st], wa[0][st], wa[1][st]);
        }
      }
      float b4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) b4[i] = bias4[i];
      // ---- this wave's next tile: the layer's second one, else the first of a later layer ----
      fetch_from(l, slot + 1, W);
      // ---- four sample tiles ----
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        floatx4m acc = {0.f, 0.f, 0.f, 0.f}, cross = {0.f, 0.f, 0.f, 0.f};
        const unsigned char* src = at + (16 * ct + j) * kRowB + 16 * q;
#pragma unroll
        for (int st = 0; st < kMfmaKSteps; ++st) {
          if (st < KS) {
            const f16x8 x0 = *reinterpret_cast<const f16x8*>(src + 64 * st);
            const f16x8 x1 = *reinterpret_cast<const f16x8*>(src + kTermB + 64 * st);
            cross = __builtin_amdgcn_mfma_f32_16x16x32_f16(wa[0][st], x1, cross, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(wa[0][st], x0, acc, 0, 0, 0);
            cross = __builtin_amdgcn_mfma_f32_16x16x32_f16(wa[1][st], x0, cross, 0, 0, 0);
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) held[slot][ct][i] = fmaf(acc[i] + cross[i], u_s[ct] * u_w[i], b4[i]);
      }
      // the activation of the tile's sixteen values per lane, switched once and not per value
      auto apply = [&](auto f) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v = f(held[slot][ct][i]);
            held[slot][ct][i] = v;
            m_s[ct] = fmaxf(m_s[ct], fabsf(v));
          }
      };
      if (act == EVO_ACT_TANH) apply([](float x) { return tanh_fast_accurate(x); });
      else if (act == EVO_ACT_RELU) apply([](float x) { return fmaxf(x, 0.f); });
      else apply([](float x) { return x; });
    }
    if (last) {
      __syncthreads();  // every wave has read the layer's input: the buffer takes the network's output
#pragma unroll
      for (int slot = 0; slot < kMfmaSlots; ++slot) {
        const int nt = wave + kMfmaWaves * slot;
        if (nt >= NT) continue;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int o = 16 * nt + 4 * q + i;
            if (o < N) fin[o * TB + 16 * ct + j] = held[slot][ct][i];
          }
      }
      __syncthreads();
      break;
    }
    // ---- per-sample scale of this layer's outputs: the largest magnitude over all neurons ----
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      float m = m_s[ct];
      m = fmaxf(m, __shfl_xor(m, 16, 64));
      m = fmaxf(m, __shfl_xor(m, 32, 64));
      if (q == 0) smax[wave * TB + 16 * ct + j] = m;
    }
    __syncthreads();  // every wave has read the layer's input, and the maxima are out
    float s_new[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      const int smp = 16 * ct + j;
      float m = smax[smp];
#pragma unroll
      for (int w = 1; w < kMfmaWaves; ++w) m = fmaxf(m, smax[w * TB + smp]);
      s_new[ct] = split_pow2_scale(m);
      u_s[ct] = pow2_reciprocal(s_new[ct]);
    }
#pragma unroll
    for (int slot = 0; slot < kMfmaSlots; ++slot) {
      const int nt = wave + kMfmaWaves * slot;
      if (nt >= NT) continue;
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        uint2 lead, resid;
        split2_pair_true(s_new[ct] * held[slot][ct][0], s_new[ct] * held[slot][ct][1], lead.x, resid.x);
        split2_pair_true(s_new[ct] * held[slot][ct][2], s_new[ct] * held[slot][ct][3], lead.y, resid.y);
        unsigned char* dst = at + (16 * ct + j) * kRowB + short_place(16 * nt + 4 * q) * 2;
        *reinterpret_cast<uint2*>(dst) = lead;
        *reinterpret_cast<uint2*>(dst + kTermB) = resid;
      }
    }
    __syncthreads();
    off += K * N + N;
  }

  // ---- the network output [A][sample] -> memory, or its loss: sixteen samples per wave, as the form above has them ----
  const int A = a.sh.dims[n_layers];
  if (LOSS == LOSS_NONE) {
    float* dst = a.out + (static_cast<size_t>(member) * a.B + b0) * A;
    const int rows = min(TB, a.B - b0);
    for (int i = tid; i < rows * A; i += 64 * kMfmaWaves) {
      const int ss = i / A, o = i - ss * A;
      dst[i] = fin[o * TB + ss];
    }
    return;
  }
  if (wave < 4) {
    const int b = b0 + 16 * wave + j;
    const float loss = mlp_finish<kMfmaMaxWidth / 16, LOSS, 1>(
        a, member, b, b < a.B, A, q, [&](int t, int i) { return fin[(16 * t + 4 * q + i) * TB + 16 * wave + j]; });
    if (lane == 0) red_s[wave] = loss;
  }
  __syncthreads();
  const float sum = (red_s[0] + red_s[1]) + (red_s[2] + red_s[3]);
  if (tid == 0 && a.fitness) a.fitness[member] = a.scale * sum;
  else if (tid == 0) a.partial[static_cast<size_t>(member) * a.tiles + tile] = sum;
}

// ---- the fp32 matrix form ------------------------------------------------------------------------------
// Networks of widths up to 64 run on v_mfma_f32_16x16x4_f32: fp32 operands as they are, so there is
// nothing to split or scale.  The instruction adds its four products one after the other, each as one fused
// multiply-add, so a sum that starts from the bias and runs over k in its order has the bits of the vector form, and the
// outputs and losses of the two forms are the same bit for bit.
// Workgroup = (member, up to 1024 samples), eight waves; the member's weights go to LDS once, in operand order, and then
// every wave takes tiles of sixteen samples through the whole network by itself.  A layer is computed transposed (rows =
// neurons, columns = samples); row 4 q + i of a tile is neuron 16 t + 4 i + q, so that a lane (group q) ends up with those
// four of one sample, and a product over the four k 16 t + 4 i + (0..3) takes exactly the lane's value i of tile t as its
// B operand -- a layer's outputs are the next one's operands where they are.  A unit is a 16 x 16 block of weights, one
// 16-byte LDS read per lane for four products; two neuron tiles at a time are two chains of sums.
// Bound by the fp32 matrix instruction (32 cycles for 2 kFLOP) plus the activations, which it does not overlap with.
// get_actions, vector form and here: 20-50-60-5 tanh, 1000 members of 300 samples 226 and 68 us; 60-40-8 ReLU, 1000 of
// 500 245 and 54 us; 63-64-64, 1000 of 300 222 and 64 us.
constexpr int kF32UnitB = 64 * 16;
constexpr int kF32MaxGroup = 16;        // pieces of 64 samples per workgroup
constexpr int kF32MaxWidth = 64;

__host__ __device__ inline int f32_units(const MlpShape& sh) {
  int n = 0;
  for (int l = 0; l < sh.n_layers; ++l) n += ((sh.dims[l] + 15) >> 4) * ((sh.dims[l + 1] + 15) >> 4);
  return n;
}
__host__ __device__ inline int f32_out_tiles(const MlpShape& sh) {
  int n = 0;
  for (int l = 0; l < sh.n_layers; ++l) n += (sh.dims[l + 1] + 15) >> 4;
  return n;
}
// weights, one unit that is read ahead and not used, biases, one loss per sample
inline size_t f32_lds_bytes(const MlpShape& sh, int group) {
  return static_cast<size_t>(f32_units(sh) + 1) * kF32UnitB + (f32_out_tiles(sh) * 16 + group * kMlpTile) * sizeof(float);
}

// v[i] of lane group q <-> v[q] of lane group i (groups of sixteen lanes).
__device__ __forceinline__ void transpose_groups(float (&v)[4]) {
  uint32_t u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) u[i] = __float_as_uint(v[i]);
  const auto a = __builtin_amdgcn_permlane32_swap(u[0], u[2], false, false), b = __builtin_amdgcn_permlane32_swap(u[1], u[3], false, false);
  const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false), d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  v[0] = __uint_as_float(c[0]), v[1] = __uint_as_float(c[1]), v[2] = __uint_as_float(d[0]), v[3] = __uint_as_float(d[1]);
}
// The values of the four lane groups, in every group.
__device__ __forceinline__ void gather_groups(float v, float (&all)[4]) {
  const uint32_t u = __float_as_uint(v);
  const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);            // groups (0 1 0 1), (2 3 2 3)
  const auto a = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false), b = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
  all[0] = __uint_as_float(a[0]), all[1] = __uint_as_float(a[1]), all[2] = __uint_as_float(b[0]), all[3] = __uint_as_float(b[1]);
}

// Loss of the lane's sample from its outputs, v[t][i] = neuron 16 t + 4 i + q, with the vector form's arithmetic (sums over
// the outputs in their order); the same in all four groups.
template <int NTM, int LOSS>
__device__ __forceinline__ float f32_sample_loss(const MlpArgs& a, int member, int b, bool live, int A, int q, const float (&v)[NTM][4]) {
  float sum = 0.f, mx = -__builtin_inff(), hit = 0.f;
  const int y = LOSS == LOSS_CE && live ? min(max(static_cast<const int32_t*>(a.target)[b], 0), A - 1) : 0;  // labels outside [0, A) are clamped
  if (LOSS == LOSS_CE) {
#pragma unroll
    for (int t = 0; t < NTM; ++t) {
      if (16 * t >= A) break;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = 16 * t + 4 * i + q;
        if (o < A) mx = fmaxf(mx, v[t][i]);
        if (o == y) hit = v[t][i];
      }
    }
    float all[4];
    gather_groups(mx, all);
    mx = fmaxf(fmaxf(all[0], all[1]), fmaxf(all[2], all[3]));
    gather_groups(hit, all);
    hit = (all[0] + all[1]) + (all[2] + all[3]);    // three of them are zero
  }
  const float* tg = static_cast<const float*>(a.target) + (LOSS == LOSS_MSE && live ? (static_cast<size_t>(member) * a.B + b) * A : 0);
#pragma unroll
  for (int t = 0; t < NTM; ++t) {
    if (16 * t >= A) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (16 * t + 4 * i >= A) break;
      const int o = 16 * t + 4 * i + q;
      float all[4];
      if (LOSS == LOSS_CE) {
        gather_groups(o < A ? expf(v[t][i] - mx) : 0.f, all);
        sum = (((sum + all[0]) + all[1]) + all[2]) + all[3];
      } else {
        gather_groups(o < A && live ? v[t][i] - tg[o] : 0.f, all);
        sum = fmaf(all[3], all[3], fmaf(all[2], all[2], fmaf(all[1], all[1], fmaf(all[0], all[0], sum))));
      }
    }
  }
  if (LOSS == LOSS_CE) sum = (mx + logf(sum)) - hit;
  return live ? sum : 0.f;
}

template <int LOSS>
__global__ __launch_bounds__(512, 4) void mlp_f32_units_kernel(MlpArgs a, int group, bool spread) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  constexpr int NTM = kF32MaxWidth / 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, q = lane >> 4;
  // consecutive workgroup numbers go to the eight dies in turn: the groups of one member, which read the same weights, 8
  // apart; fewer than 64 members (spread) have all dies work on each (20-50-60-5, one member of 100000 samples: 169 us on
  // one die, 35 us on all)
  const int by = spread ? 1 : 8;
  const int member = by * blockIdx.y + blockIdx.x % by, first = blockIdx.x / by * group;     // (in pieces of 64 samples)
  if (member >= a.pop) return;
  const int n_layers = a.sh.n_layers, units = f32_units(a.sh);
  float* bias_s = reinterpret_cast<float*>(lds_raw + static_cast<size_t>(units + 1) * kF32UnitB);
  float* loss_s = bias_s + 16 * f32_out_tiles(a.sh);
  const float* theta = a.params + static_cast<size_t>(member) * a.sh.P;
  const float* obs = a.obs + static_cast<size_t>(member) * a.obs_stride;

  // ---- the member's weights into LDS; rows and columns beyond a layer are zeros by the buffer's bounds check ----
  {
    int off = 0, unit0 = 0, tile0 = 0;
    for (int l = 0; l < n_layers; ++l) {
      const int K = a.sh.dims[l], N = a.sh.dims[l + 1], KT = (K + 15) >> 4, NT = (N + 15) >> 4;
      const auto w = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(theta + off), 0, 4 * K * N, 0x00020000);
      const auto wb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(theta + off + K * N), 0, 4 * N, 0x00020000);
      // this wave's units, four at a time: sixteen loads in flight
      for (int u0 = wave; u0 < KT * NT; u0 += 4 * 8) {
        float v[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int u = u0 + 8 * r, nt = u / KT, kt = u - nt * KT, n = 16 * nt + 4 * (j & 3) + (j >> 2);
          const unsigned at = n < N ? 4u * static_cast<unsigned>((16 * kt + q) * N + n) : 0x40000000u;
#pragma unroll
          for (int i = 0; i < 4; ++i) v[r][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(w, at + 16u * N * i, 0, 0));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int u = u0 + 8 * r;
          if (u < KT * NT)
            *reinterpret_cast<float4*>(lds_raw + static_cast<size_t>(unit0 + u) * kF32UnitB + 16 * lane) =
                make_float4(v[r][0], v[r][1], v[r][2], v[r][3]);
        }
      }
      if (tid < 16 * NT) {
        const unsigned n = (tid & ~15) + 4 * (tid & 3) + ((tid >> 2) & 3);
        bias_s[16 * tile0 + tid] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wb, 4u * n, 0, 0));
      }
      off += K * N + N;
      unit0 += KT * NT;
      tile0 += NT;
    }
  }
  const int D = a.sh.dims[0], A = a.sh.dims[n_layers];
  const bool wide_obs = (D & 3) == 0 && (reinterpret_cast<uintptr_t>(obs) & 15u) == 0;  // then every row starts on 16 bytes
  const int pieces = min(group, a.tiles - first), s_end = min(a.B, (first + pieces) * kMlpTile);
  float x[NTM][4], ahead[NTM][4];
  // sixteen samples from b0 on, laid out as a layer's outputs are (16-byte loads: once they are transposed); zeros beyond
  // the observation and the batch
  auto observe = [&](int b0) {
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(obs + static_cast<size_t>(b0) * D), 0,
                                                        4 * min(s_end - b0, 16) * D, 0x00020000);
#pragma unroll
    for (int t = 0; t < NTM; ++t) {
      if (16 * t >= D) break;
      const int d = 16 * t + 4 * q;
      if (wide_obs) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rows, d < D ? 4u * (j * D + d) : 0x40000000u, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) ahead[t][i] = __uint_as_float(v[i]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int f = 16 * t + 4 * i + q;
          ahead[t][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, f < D ? 4u * (j * D + f) : 0x40000000u, 0, 0));
        }
      }
    }
  };
  int b0 = first * kMlpTile + 16 * wave;
  if (b0 < s_end) observe(b0);
  __syncthreads();
  for (; b0 < s_end; b0 += 16 * 8) {
#pragma unroll
    for (int t = 0; t < NTM; ++t) {
      if (wide_obs && 16 * t < D) transpose_groups(ahead[t]);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[t][i] = ahead[t][i];
    }
    if (b0 + 16 * 8 < s_end) observe(b0 + 16 * 8);  // the wave's next sixteen are on their way meanwhile
    const unsigned char* src = lds_raw + 16 * lane;
    const float* bias = bias_s + 4 * q;
    for (int l = 0; l < n_layers; ++l) {
      const int K = a.sh.dims[l], N = a.sh.dims[l + 1], act = a.sh.act[l], KT = (K + 15) >> 4, NT = (N + 15) >> 4;
      float y[NTM][4];
      auto finish = [&](int t, const floatx4m& acc) {
        if (act == EVO_ACT_TANH) {
#pragma unroll
          for (int i = 0; i < 4; ++i) y[t][i] = tanh_fast_accurate(acc[i]);
        } else if (act == EVO_ACT_RELU) {
#pragma unroll
          for (int i = 0; i < 4; ++i) y[t][i] = fmaxf(acc[i], 0.f);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) y[t][i] = acc[i];
        }
        if (16 * t + 16 > N) {  // neurons that do not exist must not hand a NaN on (zero weights x an infinite input)
#pragma unroll
          for (int i = 0; i < 4; ++i) y[t][i] = 16 * t + 4 * i + q < N ? y[t][i] : 0.f;
        }
      };
#pragma unroll
      for (int t = 0; t < NTM; t += 2) {
        if (t >= NT) continue;
        const bool two = t + 1 < NT;
        const unsigned char* src1 = two ? src + KT * kF32UnitB : src;
        const float4 b4 = *reinterpret_cast<const float4*>(bias), c4 = *reinterpret_cast<const float4*>(bias + (two ? 16 : 0));
        floatx4m acc = {b4.x, b4.y, b4.z, b4.w}, acc1 = {c4.x, c4.y, c4.z, c4.w};
        float4 w = *reinterpret_cast<const float4*>(src), w1 = *reinterpret_cast<const float4*>(src1);
#pragma unroll
        for (int kt = 0; kt < NTM; ++kt) {
          if (kt < KT) {
            const float4 v = w, v1 = w1;
            src += kF32UnitB, src1 += kF32UnitB;
            w = *reinterpret_cast<const float4*>(src), w1 = *reinterpret_cast<const float4*>(src1);  // one unit ahead
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v.x, x[kt][0], acc, 0, 0, 0);
            if (two) acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(v1.x, x[kt][0], acc1, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v.y, x[kt][1], acc, 0, 0, 0);
            if (two) acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(v1.y, x[kt][1], acc1, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v.z, x[kt][2], acc, 0, 0, 0);
            if (two) acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(v1.z, x[kt][2], acc1, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v.w, x[kt][3], acc, 0, 0, 0);
            if (two) acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(v1.w, x[kt][3], acc1, 0, 0, 0);
          }
        }
        finish(t, acc);
        if (two) finish(t + 1, acc1);
        src = two ? src1 : src;
        bias += two ? 32 : 16;
      }
#pragma unroll
      for (int t = 0; t < NTM; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (t < NT) x[t][i] = y[t][i];
    }
    const int b = b0 + j;
    if (LOSS == LOSS_NONE) {
#pragma unroll
      for (int t = 0; t < NTM; ++t) {
        if (16 * t >= A) break;
        transpose_groups(x[t]);
      }
      mlp_finish<NTM, LOSS>(a, member, b, b < s_end, A, q, [&](int t, int i) { return x[t][i]; });
    } else {
      const float loss = f32_sample_loss<NTM, LOSS>(a, member, b, b < s_end, A, q, x);
      if (q == 0) loss_s[b - first * kMlpTile] = loss;
    }
  }
  if (LOSS == LOSS_NONE) return;
  __syncthreads();
  for (int piece = wave; piece < pieces; piece += 8) {   // one partial sum per 64 samples, added as the vector form does
    const int at = piece * kMlpTile + lane;
    const float loss = wave_sum(first * kMlpTile + at < s_end ? loss_s[at] : 0.f);
    if (lane == 0) {
      if (a.fitness) bias_s[piece] = loss;  // (the biases are done with)
      else a.partial[static_cast<size_t>(member) * a.tiles + first + piece] = loss;
    }
  }
  if (a.fitness) {
    __syncthreads();
    if (wave == 0) {
      const float loss = member_loss(bias_s, a.tiles);
      if (lane == 0) a.fitness[member] = a.scale * loss;
    }
  }
}

// Any fan-in of 64 or more: the split form.  (It is fast on narrow networks as well, but its operands' 22 bits show there:
// 8-16-3 1.2e-7 from 64-bit results where fp32 operands give 0.8e-7; from sums over 64 terms on the accumulation outweighs
// them.)  All narrower: the fp32 matrix form where it is the faster one, else the vector form, which gives the same bits.
// A matrix tile costs the same whether the layer fills it or not, and a wave carries sixteen samples instead of 64, so
// small layers are the vector form's.  get_actions, vector and matrix form in us (300 sizes of 25 networks measured; the
// rule costs at most a tenth where it misses the faster form by the vector form's measure):
//   products per sample >= 1100: 32-32-4 (1152), 514 members of 300 samples 27 and 21, 64 of 512 11.7 and 7.8;
//     below, 8-24-24-4 (864) 1000 of 128 17.4 and 19.5, 8-16-3 4096 of 16 13.7 and 29
//   one piece of samples each, many members (half of a workgroup's waves have no samples) >= 1900: 16-32-32-4 (1664)
//     2048 of 64 29 and 33 with the loss; >= 2800 from 700 members on where hidden widths are multiples of four (four
//     weights per LDS read in the vector form): 40-40-8 (1920) 1000 of 50 11.8 and 14.8, 2048 of 64 20 and 26,
//     36-36-36-4 (2736) 1000 of 50 16 and 21, 4096 of 16 50 and 74 with the loss
//   a width of 48 or more (the vector form keeps 512 bytes of LDS per width, few workgroups fit): 8-64-2 1000 of 128 66
//     and 18, 60-5 514 of 64 10.3 and 7.4
//   enough samples that set-up and latency drop out: 16-32-4 2048 of 500 (6.6e8 products) 100 and 61, 600 of 1024 (3.9e8)
//     47 and 52 with the loss
// The vector form: parameters through LDS up to 16 KB of them (more would leave room for fewer workgroups).  A tiny network
// (fewer than 16 inputs, outputs of w <= 16) on 600 + 15 w^2 workgroups and more by one wave each: no waves without a neuron
// and barriers among none, but more LDS per wave and longer chains.  us with four waves and one: 3-4, 1000 of 300 samples 7.3
// and 5.8, 16 of 512 3.0 and 3.4; 1-7, 518 of 858 13.5 and 8.0; 4-8-4, 2318 of 668 with a loss 47 and 32; 1-28, 1530 of 244
// 20.8 and 26.9; 1-15, 582 of 114 5.0 and 5.7.  Over 5551 networks of one to three layers on 512 to 16384 workgroups the
// rule costs 1.1 % against the better of the two.
constexpr int kStagedParams = 4096;
enum MlpForm { FORM_VECTOR, FORM_SPLIT, FORM_F32 };
static MlpForm mlp_form(const MlpShape& sh, int pop, int B) {
  int products = 0;
  // the vector form reads four weights at a time (44-44-9, 4096 of 16 without a loss: 44 us and 40)
  bool quads = sh.n_layers > 1 && (sh.max_width <= 40 || B > 16);
  for (int l = 0; l < sh.n_layers; ++l) {
    if (sh.dims[l] >= 64) return FORM_SPLIT;
    products += sh.dims[l] * sh.dims[l + 1];
    quads &= sh.dims[l + 1] % 4 == 0 || l + 1 == sh.n_layers;
  }
  if (sh.max_width > kF32MaxWidth) return FORM_VECTOR;
  const bool single = B <= kMlpTile && pop > (quads ? 700 : 1024);
  return sh.max_width >= 48 || products >= (single ? (quads ? 2800 : 1900) : 1100) || 1.0 * products * pop * B >= 6e8 ? FORM_F32 : FORM_VECTOR;
}

int launch_mlp_f32(const MlpShape& sh, const float* params, const float* obs, int64_t obs_stride, int pop, int B,
                   float* out, int loss, const void* target, float* partial, float* fitness, float scale, bool* finished,
                   hipStream_t s) {
  EVO_REQUIRE(sh.max_width <= 256, EVO_ERR_UNSUPPORTED, "fp32 MLP: layer widths above 256 are not supported (%d)",
              sh.max_width);
  MlpArgs a;
  a.sh = sh, a.params = params, a.obs = obs, a.obs_stride = obs_stride, a.B = B;
  a.out = out, a.target = target, a.partial = partial;
  a.tiles = (B + kMlpTile - 1) / kMlpTile;
  a.pop = pop;
  a.fitness = nullptr, a.scale = scale;
  // a workgroup has all samples of its member: it writes the fitness itself
  auto whole_member = [&](bool yes) {
    if (loss == LOSS_NONE || !yes) return;
    a.fitness = fitness;
    *finished = true;
  };
  const dim3 grid(a.tiles, pop);
  const MlpForm form = mlp_form(sh, pop, B);
  if (form == FORM_F32) {
    // as large a group of samples per workgroup as leaves two workgroups per compute unit
    const int64_t per = static_cast<int64_t>(pop) * a.tiles / 512;
    const int group = static_cast<int>(std::min<int64_t>(std::max<int64_t>(per, 2), std::min(a.tiles, kF32MaxGroup)));
    const int wgs = (a.tiles + group - 1) / group;
    const size_t lds = f32_lds_bytes(sh, group);
    const bool spread = pop < 64;
    whole_member(wgs == 1);
    auto launch_units = [&](auto kern) -> int {
      if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) (void)hipGetLastError();
        EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(e));
      }
      // (in two dimensions: one has room for fewer than 2^32 threads, 8.6e9 samples of all members)
      hipLaunchKernelGGL(kern, spread ? dim3(wgs, pop) : dim3(8 * wgs, (pop + 7) / 8), dim3(512), lds, s, a, group, spread);
      return check_launch("mlp_f32_units_kernel");
    };
    if (loss == LOSS_NONE) return launch_units(mlp_f32_units_kernel<LOSS_NONE>);
    if (loss == LOSS_CE) return launch_units(mlp_f32_units_kernel<LOSS_CE>);
    return launch_units(mlp_f32_units_kernel<LOSS_MSE>);
  }
  if (form == FORM_SPLIT) {
    bool wide = false, whole = true;
    for (int l = 0; l < sh.n_layers; ++l) {
      wide |= sh.dims[l] >= 192 && sh.dims[l + 1] >= 192;
      wide |= sh.dims[l + 1] == 256 && a.tiles == 1 && pop > 256;  // (64-256-16, 1000 members of 64: 64 there and 59 here)
      whole &= sh.dims[l] % 32 == 0;
    }
    // (a single layer: 256-256, one member of 300, classification 26 us there and 30 here, squared error 24 and 21.5;
    // outputs of 255, whose rows start off 16 bytes, one member of 2000 31 and 25.5)
    const bool single = loss == LOSS_MSE || (loss == LOSS_NONE && sh.dims[sh.n_layers] % 4 != 0);
    if (wide && whole && (sh.n_layers > 1 || single) && (a.tiles == 1 || static_cast<int64_t>(pop) * a.tiles <= 256)) {
      int kp = 32;      // widest fan-in, padded to the matrix instruction's 32
      for (int l = 0; l < sh.n_layers; ++l) kp = max(kp, (sh.dims[l] + 31) & ~31);
      a.ldw = kp;
      whole_member(a.tiles == 1);
      // two fp16 terms of a layer's input and the maxima, or the network's output in their place
      const size_t input = static_cast<size_t>(2) * kMlpTile * (kp + 8) * 2 + (kMfmaWaves + 1) * kMlpTile * sizeof(float);
      const size_t lds = std::max(input, sh.dims[sh.n_layers] * kMlpTile * sizeof(float));
      auto launch_short = [&](auto kern) -> int {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) (void)hipGetLastError();
        EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(e));
        hipLaunchKernelGGL(kern, dim3(8 * ((pop + 7) / 8) * a.tiles), dim3(64 * kMfmaWaves), lds, s, a);
        return check_launch("mlp_f32_short_kernel");
      };
      if (loss == LOSS_NONE) return launch_short(mlp_f32_short_kernel<LOSS_NONE>);
      if (loss == LOSS_CE) return launch_short(mlp_f32_short_kernel<LOSS_CE>);
      return launch_short(mlp_f32_short_kernel<LOSS_MSE>);
    }
    const int wg_tiles = static_cast<int64_t>(pop) * ((a.tiles + 1) / 2) >= 256 ? 2 : 1;
    const int wgs = (a.tiles + wg_tiles - 1) / wg_tiles;
    whole_member(wgs == 1);
    auto launch_mfma = [&](auto kern) -> int {
      hipLaunchKernelGGL(kern, dim3(8 * ((pop + 7) / 8) * wgs), dim3(64 * kMfmaWaves), 0, s, a, wg_tiles);
      return check_launch("mlp_f32_mfma_kernel");
    };
    auto by_width = [&](auto loss_c) -> int {
      constexpr int L = decltype(loss_c)::value;
      return sh.max_width <= 128 ? launch_mfma(mlp_f32_mfma_kernel<4, L>) : launch_mfma(mlp_f32_mfma_kernel<8, L>);
    };
    if (loss == LOSS_NONE) return by_width(std::integral_constant<int, LOSS_NONE>());
    if (loss == LOSS_CE) return by_width(std::integral_constant<int, LOSS_CE>());
    return by_width(std::integral_constant<int, LOSS_MSE>());
  }
  a.ldw = sh.max_width;
  const bool staged = sh.P <= kStagedParams;
  whole_member(a.tiles == 1);
  // two tiles in one workgroup while the chip is not full (us with finalize_kernel / this way: 16-32-4, 64 members of 100
  // 7.6 / 6.7, 512 of 128 9.8 / 8.6, but 1000 of 128 13.4 / 14.4; four tiles gain nothing, more lose)
  const size_t pair_lds = sizeof(float) * (4 * a.ldw * kMlpTile + sh.P + 8 + 2);
  if (loss != LOSS_NONE && staged && a.tiles == 2 && pop <= 512 && pair_lds <= 64 * 1024) {
    a.partial = nullptr, *finished = true;
    auto launch_pair = [&](auto kern) -> int {
      hipLaunchKernelGGL(kern, dim3(pop), dim3(512), pair_lds, s, a, fitness);
      return check_launch("mlp_f32_pair_kernel");
    };
    return loss == LOSS_CE ? launch_pair(mlp_f32_pair_kernel<LOSS_CE>) : launch_pair(mlp_f32_pair_kernel<LOSS_MSE>);
  }
  const size_t shmem = sizeof(float) * (2 * a.ldw * kMlpTile + (staged ? sh.P + 8 : 0));
  auto launch = [&](auto kern, int threads) -> int {
    if (shmem > 64 * 1024) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(shmem));
      EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(e));
    }
    hipLaunchKernelGGL(kern, grid, dim3(threads), shmem, s, a);
    return check_launch("mlp_f32_kernel");
  };
  auto by_size = [&](auto loss_c) -> int {
    constexpr int L = decltype(loss_c)::value;
    if (!staged) return launch(mlp_f32_kernel<L, false, 4>, 256);
    int widest = 0;  // of the layers' outputs
    for (int l = 1; l <= sh.n_layers; ++l) widest = std::max(widest, sh.dims[l]);
    const bool lone = sh.dims[0] < 16 && widest <= 16 && static_cast<int64_t>(pop) * a.tiles >= 600 + 15 * widest * widest;
    return lone ? launch(mlp_f32_kernel<L, true, 1>, 64) : launch(mlp_f32_kernel<L, true, 4>, 256);
  };
  if (loss == LOSS_NONE) return by_size(std::integral_constant<int, LOSS_NONE>());
  if (loss == LOSS_CE) return by_size(std::integral_constant<int, LOSS_CE>());
  return by_size(std::integral_constant<int, LOSS_MSE>());
}

// One wavefront per member: lanes read the partial sums coalesced (lane, lane + 64, ...) and the
// 64 lane totals are combined by a fixed butterfly, so the result does not depend on timing.
__global__ __launch_bounds__(64) void finalize_kernel(const float* __restrict__ partial, int pop, int n,
                                                      float scale, float* __restrict__ fitness) {
  const int m = blockIdx.x, lane = threadIdx.x;
  float acc = 0.f;
  for (int j = lane; j < n; j += 64) acc += partial[static_cast<size_t>(m) * n + j];
  acc = wave_sum(acc);
  if (lane == 0) fitness[m] = scale * acc;
}

int launch_finalize(const float* partial, int pop, int n, float scale, float* fitness, hipStream_t s) {
  hipLaunchKernelGGL(finalize_kernel, dim3(pop), dim3(64), 0, s, partial, pop, n, scale, fitness);
  return check_launch("finalize_kernel");
}

// ---- sphere --------------------------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

// Workgroup (chunk, member) streams one contiguous piece of the member's row with 16-byte loads;
// x fastest, so consecutive workgroups read consecutive pieces of one row.  Per-thread order and
// the tree are fixed; the per-chunk sums are added in chunk order by finalize_kernel.
constexpr int kSphereChunk = 4096;  // parameters per workgroup (16 KB of fp32)

// Aligned rows (fp32, P a multiple of 4): thread t takes the quads t, t + 256, ... of its piece straight from memory.
// Any other row starts on any element: the piece is read with 16-byte loads on element addresses, all of them in flight,
// and passes through LDS so that thread t still sums the elements t, t + 256, ... in order.  (Read element by element:
// 250 fp32 rows of 300007 91 us, now 63; 4096 bfloat16 rows of 86544 373 us, now 231.)
template <typename T, bool ALIGNED>
__global__ __launch_bounds__(256) void sphere_kernel(const T* __restrict__ params,
                                                     const float* __restrict__ x_star, int P, int chunks,
                                                     float* __restrict__ partial) {
  __shared__ float red[4];
  __shared__ __attribute__((aligned(16))) float piece_s[ALIGNED ? 4 : kSphereChunk];
  const int tid = threadIdx.x;
  const T* row = params + static_cast<size_t>(blockIdx.y) * P;
  const int begin = blockIdx.x * kSphereChunk, end = min(P, begin + kSphereChunk);
  float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f, acc3 = 0.f;
  if (ALIGNED) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4* r4 = reinterpret_cast<const f32x4*>(row);
    const float4* x4 = reinterpret_cast<const float4*>(x_star);
    for (int i = begin / 4 + tid; i < end / 4; i += 256) {
      const f32x4 p = __builtin_nontemporal_load(r4 + i);  // read once: keep it out of the caches
      const float4 x = x4[i];
      const float d0 = p.x - x.x, d1 = p.y - x.y, d2 = p.z - x.z, d3 = p.w - x.w;
      acc0 = fmaf(d0, d0, acc0);
      acc1 = fmaf(d1, d1, acc1);
      acc2 = fmaf(d2, d2, acc2);
      acc3 = fmaf(d3, d3, acc3);
    }
  } else {
    constexpr int E = 16 / sizeof(T), R = kSphereChunk / (256 * E);  // elements per load, loads per thread
    typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));
    u32x4u v[R];
    const int last = end - E;  // (lanes beyond the piece's last whole load read that one; it lies in the row, P >= E)
    if (P >= E) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        v[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4u*>(row + min(begin + E * (tid + 256 * r), last)));
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = begin + E * (tid + 256 * r);
      if (i + E <= end) {
        float* dst = piece_s + (i - begin);
        if (sizeof(T) == 4) {
          *reinterpret_cast<u32x4u*>(dst) = v[r];
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            *reinterpret_cast<float2*>(dst + 2 * k) = make_float2(__uint_as_float(v[r][k] << 16), __uint_as_float(v[r][k] & 0xffff0000u));
        }
      } else {
        for (int k = i; k < end; ++k)
          piece_s[k - begin] = sizeof(T) == 4 ? reinterpret_cast<const float*>(row)[k]
                                              : bf16_to_f32(reinterpret_cast<const uint16_t*>(row)[k]);
      }
    }
    __syncthreads();
    for (int i = begin + tid; i < end; i += 256) {
      const float d = piece_s[i - begin] - x_star[i];
      acc0 = fmaf(d, d, acc0);
    }
  }
  float acc = wave_sum((acc0 + acc1) + (acc2 + acc3));
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) partial[static_cast<size_t>(blockIdx.y) * chunks + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

int sphere_chunks(int P) { return (P + kSphereChunk - 1) / kSphereChunk; }

int launch_sphere(const void* params, int dtype, const float* x_star, int pop, int P, float* partial, float* fitness,
                  hipStream_t s) {
  const int chunks = sphere_chunks(P);
  const dim3 grid(chunks, pop);
  const float* f32 = static_cast<const float*>(params);
  if (dtype != EVO_F32)
    hipLaunchKernelGGL((sphere_kernel<uint16_t, false>), grid, dim3(256), 0, s, static_cast<const uint16_t*>(params),
                       x_star, P, chunks, partial);
  else if ((P & 3) == 0)
    hipLaunchKernelGGL((sphere_kernel<float, true>), grid, dim3(256), 0, s, f32, x_star, P, chunks, partial);
  else
    hipLaunchKernelGGL((sphere_kernel<float, false>), grid, dim3(256), 0, s, f32, x_star, P, chunks, partial);
  int rc = check_launch("sphere_kernel");
  if (rc) return rc;
  return launch_finalize(partial, pop, chunks, -1.0f, fitness, s);
}

}  // namespace evo
