// The fp32 MLP forward of one (member, tile of 64 samples) on the vector ALU, as a device function: the kernel of
// policy_mlp.hip runs it with the member's weights in memory, the one-launch generation of pgpe.hip with weights
// that it has just drawn into LDS.  Same instructions in the same order either way, so the two give the same bits.
#pragma once
#include "kernels.h"

#include <type_traits>

namespace evo {

struct MlpArgs {
  MlpShape sh;
  const float* params;
  const float* obs;
  int64_t obs_stride;
  int B;
  float* out;
  const void* target;
  float* partial;
  int tiles;
  int ldw;  // LDS row capacity (max width)
  int pop;
  float* fitness;  // where the workgroup that has all of a member's samples puts scale * loss sum, or null: partial
  float scale;
};

// tanh without branches: 1 - 2 / (e^{2|x|} + 1) through the hardware's exp2 and reciprocal (absolute error about
// 1e-7, so 5e-7 relative from |x| = 0.25 on) and, below 0.25, the odd series up to x^9 (next term 9e-3 x^11: 2e-9
// relative); saturates to 1 for large |x| (e^{2|x|} = inf), propagates NaN.
__device__ __forceinline__ float tanh_fast_accurate(float x) {
  const float ax = fabsf(x);
  const float big = fmaf(-2.0f, __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(2.885390081777927f * ax) + 1.0f), 1.0f);
  const float x2 = ax * ax;
  float p = fmaf(x2, 62.0f / 2835.0f, -17.0f / 315.0f);
  p = fmaf(x2, p, 2.0f / 15.0f);
  p = fmaf(x2, p, -1.0f / 3.0f);
  p = fmaf(x2 * ax, p, ax);
  return copysignf(ax < 0.25f ? p : big, x);
}

__device__ __forceinline__ float activate(float x, int act) {
  if (act == EVO_ACT_TANH) return tanh_fast_accurate(x);
  if (act == EVO_ACT_RELU) return fmaxf(x, 0.f);
  return x;
}

// Sum over the 64 lanes of a wave in a fixed butterfly order, distances 32 to 1 (every lane gets the result).  Register
// to register: swaps of halves and rows, then rotations of a row (the lanes 8 and 4 places on hold what the lanes at these
// distances hold, as the values repeat by then), then quad permutations.  (Through LDS, as shuffles, 0.3 us per sum.)
__device__ __forceinline__ float wave_sum(float v) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));  // row_ror:8
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));  // row_ror:4
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4e, 0xf, 0xf, false));   // quad_perm 2,3,0,1
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xb1, 0xf, 0xf, false));   // quad_perm 1,0,3,2
  return v;
}

// What finalize_kernel makes of a member's partial sums (at most 64 of them, in LDS), by one wave; valid in every lane.
__device__ __forceinline__ float member_loss(const float* sums, int tiles) {
  const int lane = threadIdx.x & 63;
  return wave_sum(lane < tiles ? 0.f + sums[lane] : 0.f);
}

// Neurons o0 .. o0 + G - 1 of a layer for the wave's 64 samples (bias, then the inputs in order).  Those behind the last one
// are not stored; their weights are what follows in LDS (at most 7 floats behind the parameters), or, in memory, the
// last neuron's.
// QUADS: rows start on 16 bytes, so four weights take one LDS read.
template <int G, bool QUADS, typename WPtr>
__device__ __forceinline__ void mlp_f32_neurons(const float* hin, float* hout, WPtr W, WPtr bias, int n_in, int n_out, int o0,
                                                int s, int act) {
  constexpr bool kInLds = !std::is_same<WPtr, const float*>::value;
  float acc[G];
  if constexpr (QUADS) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const f4* quads;
#pragma unroll
    for (int j = 0; j < G; j += 4) {
      const f4 b = *(quads)(bias + o0 + j);
      acc[j] = b[0], acc[j + 1] = b[1], acc[j + 2] = b[2], acc[j + 3] = b[3];
    }
#pragma unroll 4
    for (int k = 0; k < n_in; ++k) {
      const float hk = hin[k * kMlpTile + s];
      f4 w[G / 4];
#pragma unroll
      for (int j = 0; j < G / 4; ++j) w[j] = *(quads)(W + k * n_out + o0 + 4 * j);
#pragma unroll
      for (int j = 0; j < G; ++j) acc[j] = fmaf(hk, w[j >> 2][j & 3], acc[j]);
    }
  } else if (kInLds || o0 + G <= n_out) {
#pragma unroll
    for (int j = 0; j < G; ++j) acc[j] = bias[o0 + j];
    // unrolled so that the weight and activation reads of several k are issued before the first is waited for
#pragma unroll 4
    for (int k = 0; k < n_in; ++k) {
      const float hk = hin[k * kMlpTile + s];
      const WPtr wr = W + k * n_out + o0;
#pragma unroll
      for (int j = 0; j < G; ++j) acc[j] = fmaf(hk, wr[j], acc[j]);
    }
  } else {
    int at[G];
#pragma unroll
    for (int j = 0; j < G; ++j) at[j] = min(o0 + j, n_out - 1), acc[j] = bias[at[j]];
#pragma unroll 4
    for (int k = 0; k < n_in; ++k) {
      const float hk = hin[k * kMlpTile + s];
      const WPtr wr = W + k * n_out;
#pragma unroll
      for (int j = 0; j < G; ++j) acc[j] = fmaf(hk, wr[at[j]], acc[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < G; ++j)
    if (o0 + j < n_out) hout[(o0 + j) * kMlpTile + s] = activate(acc[j], act);
}

// WPtr: pointer to the member's flat parameters (global memory: const float*; LDS: an address-space-3 pointer).
// staged: null, or where in memory the parameters lie that theta is to be filled with first (theta in LDS then).
// tid: the thread among the 64 WAVES that work on this tile (a workgroup may hold two such teams on tiles of their own, of
// which the first stages the parameters).
// lds: 2 * a.ldw * 64 floats.  Every thread of the 64 WAVES returns; nothing is left in flight.  With a loss, thread 0
// returns the tile's loss sum, which is also stored to a.partial, or as the fitness of a member of one tile, where that is
// not null.
// A small network is a chain of latencies: parameters and observations are requested together, once; the four waves
// share every layer's neurons in groups as large as leaves all four something to do (an output layer of four neurons: one
// per wave).  Against four neurons per wave at a time with their weights fetched four inputs ahead from memory, get_actions
// from a recorded graph: 16-32-4, 64 members of 512 samples 8.4 -> 6.1 us, 1000 of 300 27 -> 22.8; 20-30-10, 64 of 512 11.0
// -> 7.1; 8-24-24-4, 1000 of 128 17.4 -> 13.6.  Unrolled by four inputs: by eight, 74 registers, 20-30-10 takes 9.1.
template <int LOSS, int WAVES = 4, typename WPtr>
__device__ __forceinline__ float mlp_f32_body(const MlpArgs& a, WPtr theta, int member, int tile, float* lds,
                                              float* theta_lds = nullptr, const float* staged = nullptr,
                                              int tid = threadIdx.x) {
  constexpr int TB = kMlpTile, THREADS = 64 * WAVES;
  float* hin = lds;
  float* hout = lds + a.ldw * TB;
  const int s = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b0 = tile * TB;
  const int b = b0 + s;
  const bool live = b < a.B;
  const float* obs = a.obs + static_cast<size_t>(member) * a.obs_stride;
  const int D = a.sh.dims[0], P = a.sh.P;
  float ahead[4];  // the first parameters, on their way with the observations
  if (staged) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (THREADS * r < P) ahead[r] = staged[min(tid + THREADS * r, P - 1)];
  }
  // the observation tile transposed: hin[d][sample]; lane = sample, the waves take features in turn
  {
    const float* row = obs + static_cast<size_t>(min(b, a.B - 1)) * D;
    if ((D & 3) == 0 && (reinterpret_cast<uintptr_t>(obs) & 15u) == 0) {
#pragma unroll 4
      for (int d = 4 * wave; d < D; d += 4 * WAVES) {
        const float4 v = *reinterpret_cast<const float4*>(row + d);
        hin[d * TB + s] = live ? v.x : 0.f, hin[(d + 1) * TB + s] = live ? v.y : 0.f;
        hin[(d + 2) * TB + s] = live ? v.z : 0.f, hin[(d + 3) * TB + s] = live ? v.w : 0.f;
      }
    } else {
#pragma unroll 4
      for (int d = wave; d < D; d += WAVES) hin[d * TB + s] = live ? row[d] : 0.f;
    }
  }
  if (staged) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (tid + THREADS * r < P) theta_lds[tid + THREADS * r] = ahead[r];
#pragma unroll 4
    for (int i = tid + 4 * THREADS; i < P; i += THREADS) theta_lds[i] = staged[i];
  }
  __syncthreads();
  int off = 0;
  for (int l = 0; l < a.sh.n_layers; ++l) {
    const int n_in = a.sh.dims[l], n_out = a.sh.dims[l + 1], act = a.sh.act[l];
    const WPtr W = theta + off;
    const WPtr bias = W + n_in * n_out;
    constexpr bool kQuads = !std::is_same<WPtr, const float*>::value && WAVES > 1;
    const bool quads = kQuads && ((off | n_out) & 3) == 0;  // (theta itself starts on 16 bytes)
    if (WAVES == 1) {
      if (n_out > 4)
        for (int o0 = 0; o0 < n_out; o0 += 8) mlp_f32_neurons<8, false>(hin, hout, W, bias, n_in, n_out, o0, s, act);
      else
        mlp_f32_neurons<4, false>(hin, hout, W, bias, n_in, n_out, 0, s, act);
    } else if (n_out > 16) {
      if (quads)
        for (int o0 = 8 * wave; o0 < n_out; o0 += 32) mlp_f32_neurons<8, kQuads>(hin, hout, W, bias, n_in, n_out, o0, s, act);
      else
        for (int o0 = 8 * wave; o0 < n_out; o0 += 32) mlp_f32_neurons<8, false>(hin, hout, W, bias, n_in, n_out, o0, s, act);
    } else if (n_out > 8) {
      if (4 * wave < n_out) {
        if (quads) mlp_f32_neurons<4, kQuads>(hin, hout, W, bias, n_in, n_out, 4 * wave, s, act);
        else mlp_f32_neurons<4, false>(hin, hout, W, bias, n_in, n_out, 4 * wave, s, act);
      }
    } else if (n_out > 4) {
      if (2 * wave < n_out) mlp_f32_neurons<2, false>(hin, hout, W, bias, n_in, n_out, 2 * wave, s, act);
    } else if (wave < n_out) {
      mlp_f32_neurons<1, false>(hin, hout, W, bias, n_in, n_out, wave, s, act);
    }
    __syncthreads();
    float* t = hin;
    hin = hout;
    hout = t;
    off += n_in * n_out + n_out;
  }
  // hin now holds the network output [A][sample]
  const int A = a.sh.dims[a.sh.n_layers];
  if (LOSS == LOSS_NONE) {
    float* dst = a.out + (static_cast<size_t>(member) * a.B + b0) * A;
    const int rows = min(TB, a.B - b0);
    for (int i = tid; i < rows * A; i += THREADS) {
      const int ss = i / A, o = i - ss * A;
      dst[i] = hin[o * TB + ss];
    }
    return 0.f;
  }
  if (wave != 0) return 0.f;
  float loss = 0.f;
  if (live) {
    if (LOSS == LOSS_CE) {
      const int y = min(max(static_cast<const int32_t*>(a.target)[b], 0), A - 1);  // labels outside [0, A) are clamped
      float mx = hin[s];
#pragma unroll 4
      for (int o = 1; o < A; ++o) mx = fmaxf(mx, hin[o * TB + s]);
      float se = 0.f;
#pragma unroll 4
      for (int o = 0; o < A; ++o) se += expf(hin[o * TB + s] - mx);
      loss = (mx + logf(se)) - hin[y * TB + s];
    } else {
      const float* tg = static_cast<const float*>(a.target) + (static_cast<size_t>(member) * a.B + b) * A;
#pragma unroll 4
      for (int o = 0; o < A; ++o) {
        const float d = hin[o * TB + s] - tg[o];
        loss = fmaf(d, d, loss);
      }
    }
  }
  loss = wave_sum(loss);
  if (s == 0) {
    if (a.fitness) a.fitness[member] = a.scale * loss;
    else if (a.partial) a.partial[static_cast<size_t>(member) * a.tiles + tile] = loss;
  }
  return loss;
}

}  // namespace evo
