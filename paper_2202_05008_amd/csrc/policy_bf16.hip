// Population-batched MLP forward with bfloat16 weights on the matrix cores: every member
// has its own weight matrices and its own (or a shared) batch of observations (Section 2,
// "Global Policy"; Section 4, "Exploring Novel Policy Architectures").
//
// One workgroup per member.  A layer is out[B][N] = act(in[B][K] W[K][N] + b) with
// v_mfma_f32_32x32x16_bf16: activations live in LDS as bf16 rows (A operand: 8 consecutive
// k per lane, one 16-byte read), the weights stream from HBM exactly once (B operand),
// accumulation, bias and activation are fp32, and only the fitness (or the final outputs)
// is written back.  Arithmetic intensity is B flop per weight byte, so at small B the
// kernel is bound by the weight stream, not by the matrix cores.
//
// Register layouts of v_mfma_f32_32x32x16_bf16 (lane = 32 g + c):
//   A[row c][k = 8 g + i], B[k = 8 g + i][col c], i = 0..7 (eight bf16 per lane)
//   D[row 8 b + 4 g + i][col c] in register 4 b + i, b = 0..3, i = 0..3
#include <type_traits>

#include "bf16.h"
#include "kernels.h"
#include "mlp_f32_body.h"
#include "philox.h"

namespace evo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kBf16Threads = 256;
constexpr int kBf16Waves = kBf16Threads / 64;
constexpr int kMaxRows = 64;    // B <= 64: two 32-row tiles
constexpr int kMaxWidth = 256;  // widest layer
constexpr int kRowPad = 8;      // bf16 elements of padding per LDS row (16 bytes: keeps 16-byte alignment)

struct Bf16Args {
  MlpShape sh;
  const uint16_t* params;
  const float* obs;
  int64_t obs_stride;
  int B;
  float* out;
  const float* target;
  float* fitness;
  int loss;
  int window_params, rag_at, rag_rows, bias_at;  // generic kernel: see there
};

union Pack8 {
  uint16_t h[8];
  uint4 v;
  bf16x8 b;
};

// ---- streaming kernel for three-layer networks D0 -> H -> H -> A with H = 256 -----------------
// The weights are the dominant HBM stream (2 P bytes per member, used once).  Eight waves per
// member, wave w owning output columns 32 w .. 32 w + 31 of both hidden layers, so every wave
// streams its own slice of W1 and W2 (and waves 0..3 all of W3) with 16-byte loads.  A matrix
// B operand needs eight consecutive k at one column while memory is contiguous along the
// columns: the slice goes through a small wave-private LDS tile and comes back transposed with
// ds_read_b64_tr_b16.  Within each group of 16 lanes that instruction returns to lane l,
// element j, the 16-bit element (l & 3) of the 8 bytes addressed by lane (l >> 2) + 4 j; with
// lane r pointing at row (r >> 2), columns 4 (r & 3) .. +3 of the tile, lane l receives rows
// 0..3 of column l: four consecutive k for its own column.
typedef float floatx4v __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;

__device__ __forceinline__ bf16x8 join_bf16(short4v lo, short4v hi) {
  union {
    short4v h[2];
    bf16x8 b;
  } u;
  u.h[0] = lo;
  u.h[1] = hi;
  return u.b;
}

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& v) {
  Pack8 p;
  p.v = v;
  return p.b;
}

__device__ __forceinline__ float act_f(float v, int act) {
  if (act == EVO_ACT_TANH) return tanhf(v);
  // max(v, 0) on the bit pattern as a signed integer: every negative float (and -0) is a negative integer, the
  // others order like themselves; one instruction where the floating-point maximum of a matrix result needs a
  // canonicalising move first, and a NaN stays a NaN
  if (act == EVO_ACT_RELU) return __int_as_float(max(__float_as_int(v), 0));
  return v;
}

// ---- any other network of widths up to 256, at most 64 observations per member -------------------------
// What bounds it is the weight stream (2 P bytes per member, used once) and, at a few tens of kilobytes per member,
// the latency in front of it.  A member's parameters are one contiguous vector, W1 rows, b1, W2 rows, ..., and the
// workgroup takes them as that: up to 48 KB at a time (a window: usually the whole member) are requested in one go,
// sixteen bytes a lane, and left in LDS as rows; a longer vector comes in several windows, the next one in flight under
// the products of this one.  The biases, which the sums start from, are fetched ahead of the first window into LDS of
// their own.  Operands are read back transposed (ds_read_b64_tr_b16: four consecutive k of a column per lane); a tile is
// an immediate of the read.
// The activations never leave the registers.  Products are transposed (rows = neurons, columns = the wave's sixteen
// observations); with v_mfma_f32_16x16x32_bf16 lane (j, q) of a product ends with neurons 16 t + 4 q + i of
// observation j.  The next layer takes them as k = 32 s + 8 q + e of lane group q, for which two lane swaps per packed
// pair bring the eight values of a group together (no LDS, no barrier between layers).  The instruction adds its four
// lane groups' eight products one group after the other, so with each group's k in their own order the sums are, bit for
// bit, those of the 32x32x16 products over the same k from the same start, which the streaming and resident kernels
// use; the order inside a group does not matter, and odd groups take their two halves in turn so that the sixteen
// 32-byte row pieces of a transposed read (rows 8 q + (0..3) and 8 q + (4..7)) meet all banks with a row stride of an
// odd multiple of 32 bytes.
// Measured (get_actions, 48-144-96-12 tanh, 50 observations per member, against a kernel that gathered W element by element
// with nothing in flight and kept activations in LDS, whose bits these are): 1024 members 141 -> 40 us, 256 members
// 32 -> 17 us; 64-256-256-32 ReLU of 64, 1024 members 207 -> 59 us (3.5 TB/s); 48-96-12 ReLU, 1024 members 59 -> 11 us.
// Bound by instruction issue: LDS holds two members per CU, i.e. two waves per SIMD.  9 us of the 40 are
// tanhf against one by the hardware exponential and reciprocal (1e-6 relative), which rounded some activations
// to the other bfloat16.  Tried: 32 observations per wave (accumulators and inputs of both groups do not fit beside the
// window, 50 us), the reads one group of tiles ahead of the products (no change), three workgroups per CU with fewer
// registers (spills; LDS allows two).
__host__ __device__ constexpr int gen_pieces(int NT) { return NT == 4 ? 6 : 12; }  // 16 bytes each, per thread and window
__host__ __device__ constexpr int gen_window(int NT) { return gen_pieces(NT) * kBf16Threads * 8; }  // elements

// Bytes from row to row of a layer of N outputs in LDS.
__host__ __device__ __forceinline__ int gen_stride(int N) { return 32 * (((N + 15) >> 4) | 1); }
// Rows of a layer's W in LDS: a layer that ends with half a step gets sixteen rows of zeros, so that no step is special.
__host__ __device__ __forceinline__ int gen_rows(int K) { return (K + 31) & ~31; }
// Floats from observation to observation of the errors in LDS: up to 128 outputs, and eight more so that the rows 4 apart
// that a read takes at once meet different banks.
__host__ __device__ __forceinline__ int gen_error_stride(int A) { return (A > 96 ? 128 : (A + 31) & ~31) + 8; }
// Elements of theta from row k0 of a layer (offset off) to the end of that step of 32 rows; the bias row belongs to
// the last step.
__host__ __device__ __forceinline__ int gen_step_end(int off, int k0, int K, int N) {
  return k0 + 32 < K ? off + (k0 + 32) * N : off + K * N + N;
}

template <int NT>  // neuron tiles of the widest layer
__global__ __launch_bounds__(kBf16Threads, NT >= 12 ? 2 : NT == 8 ? 3 : 4) void mlp_bf16_generic_kernel(Bf16Args a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char window_s[];
  __shared__ float red[kBf16Waves];
  constexpr int NS = NT / 2;                   // steps of 32 k of the widest layer
  constexpr int kGenPieces = gen_pieces(NT), kGenWindow = gen_window(NT);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, q = lane >> 4;
  const int member = blockIdx.x, B = a.B, n_layers = a.sh.n_layers, P = a.sh.P;
  const int b = 16 * wave + j;                 // this lane's observation
  const bool busy = 16 * wave < B;                  // waves beyond the batch only help to fetch weights
  const uint16_t* theta = a.params + static_cast<size_t>(member) * P;

  // ---- the weight stream ---------------------------------------------------------------------------------
  typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));  // rows start on 2 bytes when P is odd
  u32x4v piece[kGenPieces];
  const int Pw = a.window_params;              // a multiple of 8: theta without a ragged last layer
  auto fetch = [&](int begin) {                // (lanes beyond the end fetch its last piece again: no load is predicated)
    const char* src = reinterpret_cast<const char*>(theta + begin);
    const uint32_t last = static_cast<uint32_t>(2 * (Pw - begin) - 16);
#pragma unroll
    for (int i = 0; i < kGenPieces; ++i)
      piece[i] = *reinterpret_cast<const u32x4u*>(src + min(16u * static_cast<uint32_t>(tid + kBf16Threads * i), last));
  };
  auto zero_rows = [&](int at, int stride) {   // sixteen rows
    for (int i = tid; i < stride; i += kBf16Threads) *reinterpret_cast<uint4*>(window_s + at + 16 * i) = make_uint4(0u, 0u, 0u, 0u);
  };
  // The fetched elements [begin, end), which begin with row k0 of layer l (offset off), -> LDS rows, that row first
  // (the biases among them are in LDS already).
  auto store = [&](int begin, int end, int l, int k0, int off) {
    int base = 0;                              // LDS address of the window's first row of the layer
    while (l < n_layers && off + k0 * a.sh.dims[l + 1] < end) {
      const int K = a.sh.dims[l], N = a.sh.dims[l + 1], stride = gen_stride(N), w = N >> 3;
      const int p0 = (off + k0 * N - begin) >> 3, p1 = (min(off + K * N + N, end) - begin) >> 3;
      // piece p0 + x of the window is piece x of the layer's rows here: row r, column c; the thread's next one is
      // kBf16Threads further
      const int i0 = p0 / kBf16Threads, i1 = (p1 + kBf16Threads - 1) / kBf16Threads;  // its slots: i0 <= i < i1
      const int dr = kBf16Threads / w, dc = kBf16Threads - dr * w;
      int x = tid + kBf16Threads * i0 - p0;    // (negative: belongs to the layer before); below 2^13: the quotient is exact
      const int r = static_cast<int>(floorf((static_cast<float>(x) + 0.5f) * __builtin_amdgcn_rcpf(static_cast<float>(w))));
      int c = x - r * w;
      int dst = base + r * stride + 16 * c;
      const int n_x = min(p1 - p0, (K - k0) * w);
#pragma unroll
      for (int i = 0; i < kGenPieces; ++i) {
        if (i < i0 || i >= i1) continue;       // uniform
        if (x >= 0 && x < n_x) *reinterpret_cast<u32x4v*>(window_s + dst) = piece[i];
        x += kBf16Threads, c += dc;
        const bool wrap = c >= w;
        c -= wrap ? w : 0;
        dst += dr * stride + 16 * dc + (wrap ? stride - 16 * w : 0);
      }
      if ((K & 31) != 0 && off + K * N < end) zero_rows(base + (K - k0) * stride, stride);
      base += (gen_rows(K) - k0) * stride;
      off += K * N + N, k0 = 0, ++l;
    }
  };
  // A last layer whose width is no multiple of 8 comes into LDS of its own behind the window: where that is little all of it
  // element by element, requested at the start; else by rows, 16 bytes at a time on whatever address and the last up to
  // seven elements of a row one by one, all rows (rag_rows = K) or 32 of them.  (256-250, one member: 22 -> 13.5 us against
  // element by element.)
  constexpr int kRagged = 8;                   // elements per thread that are requested ahead
  const int rag_K = a.sh.dims[n_layers - 1], rag_N = a.sh.dims[n_layers];
  const bool ragged = a.rag_rows > 0;
  const float rag_inv = 1.0f / static_cast<float>(rag_N);
  int rag_k0 = 0;                              // first row in LDS
  auto rag_put = [&](int e, uint16_t v) {      // (e below 2^11: exact, as above)
    const int r = static_cast<int>((static_cast<float>(e) + 0.5f) * rag_inv), c = e - r * rag_N;
    *reinterpret_cast<uint16_t*>(window_s + a.rag_at + r * gen_stride(rag_N) + 2 * c) = v;
  };
  auto rag_fetch = [&](int k0, int rows) {     // (more than 2^11 elements: eight columns and more)
    for (int r = tid >> 3; r < rows; r += kBf16Threads / 8) {
      const uint16_t* src = theta + Pw + (k0 + r) * rag_N;
      unsigned char* dst = window_s + a.rag_at + r * gen_stride(rag_N);
      u32x4v v[kMaxWidth / 64];
#pragma unroll
      for (int i = 0; i < kMaxWidth / 64; ++i)  // (lanes beyond the row's last whole piece fetch its last eight elements)
        v[i] = *reinterpret_cast<const u32x4u*>(src + min(8 * (tid & 7) + 64 * i, rag_N - 8));
#pragma unroll
      for (int i = 0; i < kMaxWidth / 64; ++i) {
        const int c = 8 * (tid & 7) + 64 * i;
        if (c + 8 <= rag_N) {
          *reinterpret_cast<u32x4v*>(dst + 2 * c) = v[i];
        } else if (c < rag_N) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (rag_N - 8 + e >= c)
              *reinterpret_cast<uint16_t*>(dst + 2 * (rag_N - 8 + e)) = static_cast<uint16_t>(v[i][e >> 1] >> (16 * (e & 1)));
        }
      }
    }
  };
  const bool rag_ahead = ragged && a.rag_rows >= rag_K && rag_K * rag_N <= kRagged * kBf16Threads;
  uint16_t rag[kRagged];
  // the biases, one element per thread and layer, in the order of the layers (every offset but the last one's end is a
  // multiple of 16 elements)
  uint16_t* const bias_s = reinterpret_cast<uint16_t*>(window_s + a.bias_at);
  uint16_t bias[EVO_MAX_LAYERS];
  {
    int at = 0;
#pragma unroll
    for (int i = 0; i < EVO_MAX_LAYERS; ++i) {
      if (i >= n_layers) break;
      at += a.sh.dims[i] * a.sh.dims[i + 1];
      bias[i] = theta[at + min(tid, a.sh.dims[i + 1] - 1)];
      at += a.sh.dims[i + 1];
    }
  }
  if (Pw > 0) fetch(0);
  if (rag_ahead) {
#pragma unroll
    for (int i = 0; i < kRagged; ++i) rag[i] = theta[min(Pw + tid + kBf16Threads * i, P - 1)];
  }

  // ---- this lane's observation: eight values per step, straight into operand order (widths are multiples of 16) ----
  const int half = 4 * (q & 1);                // the half of its group's eight k that a lane takes first
  bf16x8 in[NS];
  {
    const int D = a.sh.dims[0];
    const bool live = b < B;
    const float* row = a.obs + static_cast<size_t>(member) * a.obs_stride + static_cast<size_t>(live ? b : 0) * D;
    // no load is predicated: what lies beyond the batch or the width is fetched from a row's start and set to zero
    float4 lo[NS], hi[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const float* src = row + (32 * s + 8 * q < D ? 32 * s + 8 * q : 0);
      lo[s] = *reinterpret_cast<const float4*>(src + half);
      hi[s] = *reinterpret_cast<const float4*>(src + (half ^ 4));
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const uint32_t m = live && 32 * s + 8 * q < D ? ~0u : 0u;
      in[s] = as_bf16x8(make_uint4(pack_bf16x2(lo[s].x, lo[s].y) & m, pack_bf16x2(lo[s].z, lo[s].w) & m,
                                   pack_bf16x2(hi[s].x, hi[s].y) & m, pack_bf16x2(hi[s].z, hi[s].w) & m));
    }
  }
  {
    int at = 0;
#pragma unroll
    for (int i = 0; i < EVO_MAX_LAYERS; ++i) {
      if (i >= n_layers) break;
      if (tid < a.sh.dims[i + 1]) bias_s[at + tid] = bias[i];
      at += a.sh.dims[i + 1];
    }
  }
  if (rag_ahead) {
#pragma unroll
    for (int i = 0; i < kRagged; ++i) {
      const int e = tid + kBf16Threads * i;
      if (e < rag_K * rag_N) rag_put(e, rag[i]);
    }
    if ((rag_K & 31) != 0) zero_rows(a.rag_at + rag_K * gen_stride(rag_N), gen_stride(rag_N));
  }
  __syncthreads();                             // (the first window is still on its way)

  floatx4v acc[NT];
  auto start_sums = [&](int at) {              // `at`: the layer's first bias; what lies beyond its width is dropped later
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const uint2 v = *reinterpret_cast<const uint2*>(bias_s + at + 4 * q + 16 * t);
      acc[t] = floatx4v{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                        __uint_as_float(v.y & 0xffff0000u)};
    }
  };
  start_sums(0);
  int biases = 0;                              // of the layers before this one
  int l = 0, k0 = 0, off = 0;                  // the layer, its offset in theta, the step's first row
  int K = a.sh.dims[0], N = a.sh.dims[1], stride = gen_stride(N);
  // One step: rows k0 .. k0 + 31 of the layer, which lie in LDS from `at` on, against in[0].  Every tile of the class is
  // computed, without a branch between them (guards around groups of tiles made the compiler copy all accumulators at
  // every join, four times the step's own instructions); what lies beyond the layer's width is dropped later.
  auto step = [&](int at) {
    const bf16x8 x = in[0];
#pragma unroll
    for (int s = 0; s + 1 < NS; ++s) in[s] = in[s + 1];
    const unsigned char* src = window_s + at + (8 * q + half + (j >> 2)) * stride + 8 * (j & 3);
    const unsigned char* src_hi = src + (half ? -4 : 4) * stride;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(src + 32 * t));
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(src_hi + 32 * t));
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(join_bf16(lo, hi), x, acc[t], 0, 0, 0);
    }
  };
  // A hidden layer is complete: its activations become the next one's input.
  auto next_layer = [&]() {
    const int act = a.sh.act[l];
    auto hand_on = [&](auto f) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (32 * s >= N) break;                // the next layer's steps end here
        const floatx4v x = acc[2 * s], y = 32 * s + 16 < N ? acc[2 * s + 1] : floatx4v{0.f, 0.f, 0.f, 0.f};
        uint32_t first[2], second[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          // lane groups (x0 x1 x2 x3), (y0 y1 y2 y3) -> (x0 x2 y0 y2), (x1 x3 y1 y3): k 8 q + 0..3 and 8 q + 4..7
          const auto far = __builtin_amdgcn_permlane32_swap(pack_bf16x2(f(x[2 * h]), f(x[2 * h + 1])),
                                                            pack_bf16x2(f(y[2 * h]), f(y[2 * h + 1])), false, false);
          const auto near = __builtin_amdgcn_permlane16_swap(far[0], far[1], false, false);
          first[h] = half ? near[1] : near[0], second[h] = half ? near[0] : near[1];
        }
        in[s] = as_bf16x8(make_uint4(first[0], first[1], second[0], second[1]));
      }
    };
    if (busy) {
      if (act == EVO_ACT_TANH) hand_on([](float v) { return tanhf(v); });
      else if (act == EVO_ACT_RELU) hand_on([](float v) { return fmaxf(v, 0.f); });
      else hand_on([](float v) { return v; });
    }
    off += K * N + N, biases += N;
    ++l, k0 = 0, K = N, N = a.sh.dims[l + 1], stride = gen_stride(N);
    start_sums(biases);
  };
  const int n_windowed = n_layers - (ragged ? 1 : 0);  // layers that come through the windows
  for (int begin = 0; begin < Pw;) {
    int w_end = min(begin + kGenWindow, Pw);
    if (w_end < Pw) {                          // the window ends with the last step that fits
      int fl = l, fk = k0, fo = off;
      for (;;) {
        const int fK = a.sh.dims[fl], fN = a.sh.dims[fl + 1], fe = gen_step_end(fo, fk, fK, fN);
        if (fe > w_end) break;
        fk += 32;
        if (fk >= fK) fo = fe, fk = 0, ++fl;
      }
      w_end = fo + fk * a.sh.dims[fl + 1];
    }
    if (begin > 0) {                           // (the first window was requested at the start)
      fetch(begin);
      __syncthreads();                         // every wave has read the last window
    }
    store(begin, w_end, l, k0, off);
    __syncthreads();
    begin = w_end;
    int at = 0;
#pragma unroll 1
    for (;;) {
      if (busy) step(at);
      at += 32 * stride;
      k0 += 32;
      if (k0 >= K) {
        if (l + 1 == n_layers) break;
        next_layer();
        if (l == n_windowed) break;
      }
      if (off + k0 * N >= w_end) break;
    }
  }
  if (ragged) {
#pragma unroll 1
    for (; k0 < K; k0 += 32) {
      if (!rag_ahead && (k0 == 0 || a.rag_rows < K)) {
        __syncthreads();                       // every wave has read the rows before
        rag_k0 = k0;
        const int rows = a.rag_rows >= K ? K : min(32, K - k0);
        rag_fetch(k0, rows);
        if ((rows & 31) != 0) zero_rows(a.rag_at + rows * stride, stride);
        __syncthreads();
      }
      if (busy) step(a.rag_at + (k0 - rag_k0) * stride);
    }
  }
  // ---- outputs or their squared error ------------------------------------------------------------------
  const int A = a.sh.dims[n_layers], act = a.sh.act[n_layers - 1];
  const bool live = b < B;
  const bool quad = (A & 3) == 0;              // a lane's four outputs are 16 aligned bytes
  const size_t out_at = (static_cast<size_t>(member) * B + (live ? b : 0)) * A + 4 * q;
  auto outputs = [&](int t, float (&v)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      v[i] = act == EVO_ACT_TANH ? tanhf(acc[t][i]) : act == EVO_ACT_RELU ? fmaxf(acc[t][i], 0.f) : acc[t][i];
  };
  if (a.loss == LOSS_NONE) {
    if (!live) return;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (16 * t >= A) break;
      float v[4];
      outputs(t, v);
      float* dst = a.out + out_at + 16 * t;
      const int n = 16 * t + 4 * q;
      if (quad) {
        if (n < A) *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < A) dst[i] = v[i];
      }
    }
    return;
  }
  // The squared errors are added as 32 x 32 tiles of the outputs hold them (rows = observations: lane 32 g + c has
  // column c and rows 8 r + 4 g + i), the tiles of 32 outputs one per wave in turn: the errors pass through LDS, eight
  // neuron tiles at a time.
  float loss_acc = 0.f;
  const int stride_e = gen_error_stride(A);
  float* const err_s = reinterpret_cast<float*>(window_s);
  const int c = lane & 31, g = lane >> 5;
#pragma unroll
  for (int t0 = 0; t0 < NT; t0 += 8) {
    if (16 * t0 >= A) break;
    __syncthreads();                           // every wave has read its weights, or the errors before
#pragma unroll
    for (int t = t0; t < t0 + 8 && t < NT; ++t) {
      if (32 * (t >> 1) >= A) break;           // whole tiles of 32 outputs, zeros beyond the last one
      float v[4], y[4];
      outputs(t, v);
      const float* tg = a.target + out_at + 16 * t;
      const int n = 16 * t + 4 * q;
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = v[i];
      if (quad) {
        if (live && n < A) {
          const float4 w = *reinterpret_cast<const float4*>(tg);
          y[0] = w.x, y[1] = w.y, y[2] = w.z, y[3] = w.w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (live && n + i < A) y[i] = tg[i];
      }
      *reinterpret_cast<float4*>(err_s + b * stride_e + 16 * (t - t0) + 4 * q) =
          make_float4(live && n < A ? v[0] - y[0] : 0.f, live && n + 1 < A ? v[1] - y[1] : 0.f,
                      live && n + 2 < A ? v[2] - y[2] : 0.f, live && n + 3 < A ? v[3] - y[3] : 0.f);
    }
    __syncthreads();
    if (16 * t0 + 32 * wave < A) {
#pragma unroll
      for (int r = 0; r < 32; ++r) {
        const float d = err_s[(8 * (r >> 2) + 4 * g + (r & 3)) * stride_e + 32 * wave + c];
        loss_acc = fmaf(d, d, loss_acc);
      }
    }
  }
  loss_acc = wave_sum(loss_acc);
  if (lane == 0) red[wave] = loss_acc;
  __syncthreads();
  if (tid == 0) a.fitness[member] = -(((red[0] + red[1]) + red[2]) + red[3]) / (static_cast<float>(B) * static_cast<float>(A));
}

// The weight stream of one wave is a fixed sequence of B operands ("units", 1 KB each): D0/16 of
// layer 1, 16 of layer 2 and (waves 0..3) 8 of layer 3.  kDepth units are kept in flight in a
// register ring (one 16-byte load per lane and unit); the loads do not depend on activations, so
// the stream runs ahead across the layer boundaries and the workgroup barriers.
constexpr int kDepth = 12;
constexpr int kStageLd = 40;   // row stride (elements) of the 16 x 32 staging tile of layers 1, 2
constexpr int kStageLd3 = 24;  // row stride of the 32 x 16 staging tile of layer 3
constexpr int kStageElems = 32 * kStageLd3;  // 768 elements >= 16 * kStageLd

// At most 64 observations per member (one tile); more go to the register-resident kernel below.
// RELU: the hidden activations are ReLU and the output is linear (the shape's usual policy), which
// removes the per-value activation switch from the epilogues.
template <int D0, int H, int A, bool RELU>
__global__ __launch_bounds__(512, 4) void mlp_bf16_stream_kernel(Bf16Args a) {
  static_assert(H == 256 && D0 % 32 == 0 && A == 16, "shape of the streaming kernel");
  constexpr int LD0 = D0 + kRowPad, LDH = H + kRowPad;
  constexpr int U1 = D0 / 16, U2 = H / 16, U3 = H / 32, UT = U1 + U2 + U3;
  __shared__ __attribute__((aligned(16))) uint16_t x_s[64 * LD0];
  __shared__ __attribute__((aligned(16))) uint16_t h_s[64 * LDH];
  __shared__ __attribute__((aligned(16))) uint16_t stage_s[8 * kStageElems];
  __shared__ float red[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, g = lane >> 5;
  const int c16 = lane & 15, g4 = lane >> 4;
  uint16_t* stage = stage_s + wave * kStageElems;
  const int member = blockIdx.x, B = a.B;
  const uint16_t* theta = a.params + static_cast<size_t>(member) * a.sh.P;
  const uint16_t* W1 = theta;
  const uint16_t* B1 = W1 + D0 * H;
  const uint16_t* W2 = B1 + H;
  const uint16_t* B2 = W2 + H * H;
  const uint16_t* W3 = B2 + H;
  const uint16_t* B3 = W3 + H * A;
  const bool tail = wave < 4;  // waves that also run layer 3

  u32x4v ring[kDepth];
  // unit u -> its 16-byte load (compile-time u after unrolling).  Layers 1, 2: tile of 16 rows x
  // 32 columns, lane = (row lane >> 2, 8 columns from 8 (lane & 3)); layer 3: 32 rows x 16 columns,
  // lane = (row lane >> 1, 8 columns from 8 (lane & 1)).
  const uint16_t* p12 = theta + static_cast<size_t>(lane >> 2) * H + 32 * wave + 8 * (lane & 3);
  const uint16_t* p3 = W3 + (lane >> 1) * A + 8 * (lane & 1);
  auto issue = [&](int u) {
    u32x4v& r = ring[u % kDepth];
    if (u < U1) r = *reinterpret_cast<const u32x4v*>(p12 + static_cast<size_t>(16 * u) * H);
    else if (u < U1 + U2) r = *reinterpret_cast<const u32x4v*>(p12 + (W2 - theta) + static_cast<size_t>(16 * (u - U1)) * H);
    else if (u < UT && tail) r = *reinterpret_cast<const u32x4v*>(p3 + 32 * (u - U1 - U2) * A);
  };
  // registers of unit u -> staging tile -> transposed B operand of this lane
  auto operand12 = [&](int u) -> bf16x8 {
    *reinterpret_cast<u32x4v*>(stage + (lane >> 2) * kStageLd + 8 * (lane & 3)) = ring[u % kDepth];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint16_t* q = stage + (8 * g + (c16 >> 2)) * kStageLd + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q + 4 * kStageLd));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return join_bf16(lo, hi);
  };
  auto operand3 = [&](int u) -> bf16x8 {
    *reinterpret_cast<u32x4v*>(stage + (lane >> 1) * kStageLd3 + 8 * (lane & 1)) = ring[u % kDepth];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint16_t* q = stage + (8 * g4 + (c16 >> 2)) * kStageLd3 + 4 * (lane & 3);
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q + 4 * kStageLd3));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return join_bf16(lo, hi);
  };
  // rows = observations 8 rr + 4 g + i, columns = the wave's neurons 32 wave + c; the two column biases are
  // fetched here, ahead of the tile (a load at the point of use would sit between two layers)
  const float bias_col[2] = {from_bf16(B1[32 * wave + c]), from_bf16(B2[32 * wave + c])};
  auto bias_rows = [&](int layer, floatx16 (&acc)[2]) {
    const float b = bias_col[layer];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mt][r] = b;
  };
  auto store_rows = [&](const floatx16 (&acc)[2], int act) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = mt * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
        h_s[row * LDH + 32 * wave + c] = to_bf16(act_f(acc[mt][r], act));
      }
  };
  const float bias3 = from_bf16(B3[c16]);  // layer 3: column = output c16
  float loss_acc = 0.f;
  // the observation loads go first so that waiting for them does not drain the weight stream
  constexpr int kObsPieces = 64 * D0 / 4 / 512;
  float4 ov[kObsPieces];
  {
    const float* obs = a.obs + static_cast<size_t>(member) * a.obs_stride;
#pragma unroll
    for (int j = 0; j < kObsPieces; ++j) {
      const int i = tid + 512 * j, r = i / (D0 / 4), d4 = i - r * (D0 / 4);
      ov[j] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (r < B) ov[j] = reinterpret_cast<const float4*>(obs + static_cast<size_t>(r) * D0)[d4];
    }
  }
#pragma unroll
  for (int u = 0; u < kDepth; ++u) issue(u);

  // ---- observations -> bf16 rows (rows beyond B are zero) ---------------------------------------
#pragma unroll
  for (int j = 0; j < kObsPieces; ++j) {
    const int i = tid + 512 * j, r = i / (D0 / 4), d4 = i - r * (D0 / 4);
    uint2 pk;
    pk.x = pack_bf16x2(ov[j].x, ov[j].y);
    pk.y = pack_bf16x2(ov[j].z, ov[j].w);
    *reinterpret_cast<uint2*>(x_s + r * LD0 + 4 * d4) = pk;
  }
  // targets of this lane's four output rows (layer 3 tile of wave < 4): output c16 of observations 16 wave + 4 g4 + i
  float tgt[4] = {0.f, 0.f, 0.f, 0.f};
  if (tail && a.loss != LOSS_NONE) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * wave + 4 * g4 + i;
      if (row < B) tgt[i] = a.target[(static_cast<size_t>(member) * B + row) * A + c16];
    }
  }
  __syncthreads();

  // ---- layer 1 ----------------------------------------------------------------------------------
  floatx16 acc[2];
  bias_rows(0, acc);
#pragma unroll
  for (int u = 0; u < U1; ++u) {
    const bf16x8 bv = operand12(u);
    issue(u + kDepth);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      const uint4 av = *reinterpret_cast<const uint4*>(x_s + (mt * 32 + c) * LD0 + 16 * u + 8 * g);
      acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(av), bv, acc[mt], 0, 0, 0);
    }
  }
  store_rows(acc, RELU ? EVO_ACT_RELU : a.sh.act[0]);
  __syncthreads();

  // ---- layer 2 ----------------------------------------------------------------------------------
  bias_rows(1, acc);
#pragma unroll
  for (int u = U1; u < U1 + U2; ++u) {
    const bf16x8 bv = operand12(u);
    issue(u + kDepth);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      const uint4 av = *reinterpret_cast<const uint4*>(h_s + (mt * 32 + c) * LDH + 16 * (u - U1) + 8 * g);
      acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(av), bv, acc[mt], 0, 0, 0);
    }
  }
  __syncthreads();  // every wave has read h1: the buffer can take h2
  store_rows(acc, RELU ? EVO_ACT_RELU : a.sh.act[1]);
  __syncthreads();

  // ---- layer 3: four waves, one 16-row tile each (16x16x32 tiles: lane = 16 g4 + c16) -------------
  if (tail) {
    floatx4v o = {bias3, bias3, bias3, bias3};
#pragma unroll
    for (int u = U1 + U2; u < UT; ++u) {
      const bf16x8 bv = operand3(u);
      issue(u + kDepth);
      const uint4 av = *reinterpret_cast<const uint4*>(h_s + (16 * wave + c16) * LDH + 32 * (u - U1 - U2) + 8 * g4);
      o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(av), bv, o, 0, 0, 0);
    }
    const int act = RELU ? EVO_ACT_NONE : a.sh.act[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * wave + 4 * g4 + i;
      const float v = act_f(o[i], act);
      if (row < B) {
        if (a.loss == LOSS_NONE) {
          a.out[(static_cast<size_t>(member) * B + row) * A + c16] = v;
        } else {
          const float d = v - tgt[i];
          loss_acc = fmaf(d, d, loss_acc);
        }
      }
    }
  }
  if (a.loss == LOSS_NONE) return;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) loss_acc += __shfl_xor(loss_acc, o, 64);
  if (lane == 0 && tail) red[wave] = loss_acc;
  __syncthreads();
  if (tid == 0) a.fitness[member] = -(red[0] + red[1] + red[2] + red[3]) / (static_cast<float>(B) * A);
}

// ---- ask fused into the forward: one workgroup per antithetic pair, the population never written -------
// The streaming kernel above is bound by the weight stream that ask wrote a moment earlier (cfg4: 709 MB
// written and read straight back).  Here the two members of a pair are evaluated together and their weights
// are never in memory: where the streaming kernel loads the 16 bytes of unit u that belong to a lane (eight
// consecutive parameters), this kernel draws them -- mu and sigma of those eight parameters (fp32, shared by
// every pair, so they come from the L2), the two Philox blocks of the pair's noise, theta+ and theta- formed
// and rounded exactly as pgpe_ask stores them -- and hands each member's 16 bytes to the same staging tile and
// transposed read.  One draw serves both members; the matrix products, epilogues and the loss follow the
// streaming kernel instruction for instruction, so the fitness is bit for bit that of ask followed by rollout.
// The kernel is bound by the noise generation (the cost of ask alone); the forward rides along.
// The small output layer's operands are drawn once per workgroup (wave w draws rows 32 w .. 32 w + 31) and left
// in LDS in operand form for the four waves that run layer 3.
struct PairArgs {
  MlpShape sh;
  const float* mu;
  const float* sigma;
  uint32_t key0, key1, gen;
  const uint32_t* gen_dev;
  const float* obs;
  int64_t obs_stride;
  int B;
  float* out;
  const float* target;
  float* fitness;
  int loss;
};

// theta+ and theta- of parameter i as pgpe_ask stores them in bfloat16, widened again.
__device__ __forceinline__ void theta_pair_at(const PairArgs& a, uint32_t pair, uint32_t gen, int i, float& plus,
                                              float& minus) {
  float z[4];
  philox_normal4(static_cast<uint32_t>(i >> 2), pair, gen, EVO_TAG_NOISE, a.key0, a.key1, z);
  const int e = i & 3;
  const float zz = e == 0 ? z[0] : (e == 1 ? z[1] : (e == 2 ? z[2] : z[3]));
  const float m = a.mu[i], sg = a.sigma[i];
  plus = from_bf16(to_bf16(fmaf(sg, zz, m)));
  minus = from_bf16(to_bf16(fmaf(-sg, zz, m)));
}

template <int D0, int H, int A>
constexpr size_t pair_lds_bytes() {
  return (2 * 64 * (D0 + kRowPad) + 2 * 64 * (H + kRowPad) + 8 * kStageElems) * sizeof(uint16_t) +
         2 * (H / 32) * 64 * 16;
}

template <int D0, int H, int A, bool RELU>
__global__ __launch_bounds__(512) void mlp_bf16_pair_kernel(PairArgs a) {
  static_assert(H == 256 && D0 % 32 == 0 && A == 16, "shape of the pair kernel");
  constexpr int LD0 = D0 + kRowPad, LDH = H + kRowPad;
  constexpr int U1 = D0 / 16, U2 = H / 16, U3 = H / 32;
  constexpr int oB1 = D0 * H, oW2 = oB1 + H, oB2 = oW2 + H * H, oW3 = oB2 + H, oB3 = oW3 + H * A;
  static_assert(U3 == 8, "one output-layer unit per wave");
  extern __shared__ __attribute__((aligned(16))) uint16_t pair_lds[];
  uint16_t* x_s = pair_lds;                         // [2][64][LD0]
  uint16_t* h_s = x_s + 2 * 64 * LD0;               // [2][64][LDH]
  uint16_t* stage_s = h_s + 2 * 64 * LDH;           // [8][kStageElems]
  u32x4v* w3_s = reinterpret_cast<u32x4v*>(stage_s + 8 * kStageElems);  // [2][U3][64] output-layer operands
  __shared__ float red[2][4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, g = lane >> 5;
  const int c16 = lane & 15, g4 = lane >> 4;
  uint16_t* stage = stage_s + wave * kStageElems;
  const uint32_t pair = blockIdx.x;
  const uint32_t gen = a.gen_dev ? *a.gen_dev : a.gen;
  const int B = a.B;
  const bool tail = wave < 4;  // waves that also run layer 3

  // ---- the draw of unit u: mu and sigma of the lane's eight parameters, fetched kAhead units early ------
  constexpr int kAhead = 2;
  float4 ms[kAhead][4];
  const int lane12 = (lane >> 2) * H + 32 * wave + 8 * (lane & 3);  // this lane's eight parameters inside a unit
  auto unit_index = [&](int u) -> int {
    if (u < U1) return 16 * u * H + lane12;
    return oW2 + 16 * (u - U1) * H + lane12;
  };
  auto fetch = [&](int u) {
    if (u >= U1 + U2) return;
    const int i = unit_index(u);
    float4* r = ms[u % kAhead];
    r[0] = *reinterpret_cast<const float4*>(a.mu + i);
    r[1] = *reinterpret_cast<const float4*>(a.mu + i + 4);
    r[2] = *reinterpret_cast<const float4*>(a.sigma + i);
    r[3] = *reinterpret_cast<const float4*>(a.sigma + i + 4);
  };
  // eight parameters from index i (a multiple of 8): both members' 16 bytes, as pgpe_ask stores them
  auto draw8 = [&](int i, const float4 (&r)[4], u32x4v& plus, u32x4v& minus) {
    const float mu8[8] = {r[0].x, r[0].y, r[0].z, r[0].w, r[1].x, r[1].y, r[1].z, r[1].w};
    const float sg8[8] = {r[2].x, r[2].y, r[2].z, r[2].w, r[3].x, r[3].y, r[3].z, r[3].w};
    float z[8];
    philox_normal4(static_cast<uint32_t>(i >> 2), pair, gen, EVO_TAG_NOISE, a.key0, a.key1, z);
    philox_normal4(static_cast<uint32_t>(i >> 2) + 1u, pair, gen, EVO_TAG_NOISE, a.key0, a.key1, z + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      plus[e] = pack_bf16x2(fmaf(sg8[2 * e], z[2 * e], mu8[2 * e]), fmaf(sg8[2 * e + 1], z[2 * e + 1], mu8[2 * e + 1]));
      minus[e] = pack_bf16x2(fmaf(-sg8[2 * e], z[2 * e], mu8[2 * e]), fmaf(-sg8[2 * e + 1], z[2 * e + 1], mu8[2 * e + 1]));
    }
  };
  // 16 bytes of a lane -> staging tile -> transposed B operand of this lane (layers 1, 2: 16 rows x 32 columns)
  auto operand12 = [&](const u32x4v& v) -> bf16x8 {
    *reinterpret_cast<u32x4v*>(stage + (lane >> 2) * kStageLd + 8 * (lane & 3)) = v;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint16_t* q = stage + (8 * g + (c16 >> 2)) * kStageLd + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q + 4 * kStageLd));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return join_bf16(lo, hi);
  };
  // layer 3: 32 rows x 16 columns
  auto operand3 = [&](const u32x4v& v) -> bf16x8 {
    *reinterpret_cast<u32x4v*>(stage + (lane >> 1) * kStageLd3 + 8 * (lane & 1)) = v;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint16_t* q = stage + (8 * g4 + (c16 >> 2)) * kStageLd3 + 4 * (lane & 3);
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q + 4 * kStageLd3));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return join_bf16(lo, hi);
  };

  // ---- observations and targets of both members (requested first: they come from HBM) --------------------
  constexpr int kObsPieces = 64 * D0 / 4 / 512;
  float4 ov[2][kObsPieces];
#pragma unroll
  for (int mem = 0; mem < 2; ++mem) {
    const float* obs = a.obs + static_cast<size_t>(2 * pair + mem) * a.obs_stride;
#pragma unroll
    for (int j = 0; j < kObsPieces; ++j) {
      const int i = tid + 512 * j, r = i / (D0 / 4), d4 = i - r * (D0 / 4);
      ov[mem][j] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (r < B) ov[mem][j] = reinterpret_cast<const float4*>(obs + static_cast<size_t>(r) * D0)[d4];
    }
  }
  fetch(0);
  fetch(1);
  float tgt[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  if (tail && a.loss != LOSS_NONE) {
#pragma unroll
    for (int mem = 0; mem < 2; ++mem)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * wave + 4 * g4 + i;
        if (row < B) tgt[mem][i] = a.target[(static_cast<size_t>(2 * pair + mem) * B + row) * A + c16];
      }
  }
  // ---- output layer: wave w draws rows 32 w .. 32 w + 31 of W3 and leaves both members' operands in LDS ----
  {
    const int i = oW3 + (32 * wave + (lane >> 1)) * A + 8 * (lane & 1);
    float4 r[4];
    r[0] = *reinterpret_cast<const float4*>(a.mu + i);
    r[1] = *reinterpret_cast<const float4*>(a.mu + i + 4);
    r[2] = *reinterpret_cast<const float4*>(a.sigma + i);
    r[3] = *reinterpret_cast<const float4*>(a.sigma + i + 4);
    u32x4v plus, minus;
    draw8(i, r, plus, minus);
    w3_s[(0 * U3 + wave) * 64 + lane] = __builtin_bit_cast(u32x4v, operand3(plus));
    w3_s[(1 * U3 + wave) * 64 + lane] = __builtin_bit_cast(u32x4v, operand3(minus));
  }
  // biases of this lane's columns (layers 1, 2) and output (layer 3), both members
  float bias_col[2][2], bias3[2];
  theta_pair_at(a, pair, gen, oB1 + 32 * wave + c, bias_col[0][0], bias_col[1][0]);
  theta_pair_at(a, pair, gen, oB2 + 32 * wave + c, bias_col[0][1], bias_col[1][1]);
  theta_pair_at(a, pair, gen, oB3 + c16, bias3[0], bias3[1]);

  // ---- observations -> bf16 rows (rows beyond B are zero) ---------------------------------------
#pragma unroll
  for (int mem = 0; mem < 2; ++mem)
#pragma unroll
    for (int j = 0; j < kObsPieces; ++j) {
      const int i = tid + 512 * j, r = i / (D0 / 4), d4 = i - r * (D0 / 4);
      uint2 pk;
      pk.x = pack_bf16x2(ov[mem][j].x, ov[mem][j].y);
      pk.y = pack_bf16x2(ov[mem][j].z, ov[mem][j].w);
      *reinterpret_cast<uint2*>(x_s + mem * 64 * LD0 + r * LD0 + 4 * d4) = pk;
    }
  __syncthreads();

  floatx16 acc[2][2];  // [member][row tile]
  auto bias_rows = [&](int layer) {
#pragma unroll
    for (int mem = 0; mem < 2; ++mem)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mem][mt][r] = bias_col[mem][layer];
  };
  auto store_rows = [&](int act) {
#pragma unroll
    for (int mem = 0; mem < 2; ++mem)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = mt * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
          h_s[mem * 64 * LDH + row * LDH + 32 * wave + c] = to_bf16(act_f(acc[mem][mt][r], act));
        }
  };
  // one unit of layer 1 or 2: draw, then both members' products
  auto unit = [&](int u, const uint16_t* in, int ld, int k0) {
    u32x4v pm[2];
    draw8(unit_index(u), ms[u % kAhead], pm[0], pm[1]);
    fetch(u + kAhead);
#pragma unroll
    for (int mem = 0; mem < 2; ++mem) {
      const bf16x8 bv = operand12(pm[mem]);
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const uint4 av = *reinterpret_cast<const uint4*>(in + mem * 64 * ld + (mt * 32 + c) * ld + k0 + 8 * g);
        acc[mem][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(av), bv, acc[mem][mt], 0, 0, 0);
      }
    }
  };

  // ---- layer 1 ----------------------------------------------------------------------------------
  bias_rows(0);
#pragma unroll
  for (int u = 0; u < U1; ++u) unit(u, x_s, LD0, 16 * u);
  store_rows(RELU ? EVO_ACT_RELU : a.sh.act[0]);
  __syncthreads();

  // ---- layer 2 ----------------------------------------------------------------------------------
  bias_rows(1);
#pragma unroll
  for (int u = U1; u < U1 + U2; ++u) unit(u, h_s, LDH, 16 * (u - U1));
  __syncthreads();  // every wave has read h1: the buffer can take h2
  store_rows(RELU ? EVO_ACT_RELU : a.sh.act[1]);
  __syncthreads();

  // ---- layer 3: four waves, one 16-row tile each per member ------------------------------------------
  float loss_acc[2] = {0.f, 0.f};
  if (tail) {
#pragma unroll
    for (int mem = 0; mem < 2; ++mem) {
      floatx4v o = {bias3[mem], bias3[mem], bias3[mem], bias3[mem]};
#pragma unroll
      for (int u = 0; u < U3; ++u) {
        const bf16x8 bv = __builtin_bit_cast(bf16x8, w3_s[(mem * U3 + u) * 64 + lane]);
        const uint4 av = *reinterpret_cast<const uint4*>(h_s + mem * 64 * LDH + (16 * wave + c16) * LDH + 32 * u + 8 * g4);
        o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(av), bv, o, 0, 0, 0);
      }
      const int act = RELU ? EVO_ACT_NONE : a.sh.act[2];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * wave + 4 * g4 + i;
        const float v = act_f(o[i], act);
        if (row < B) {
          if (a.loss == LOSS_NONE) {
            a.out[(static_cast<size_t>(2 * pair + mem) * B + row) * A + c16] = v;
          } else {
            const float d = v - tgt[mem][i];
            loss_acc[mem] = fmaf(d, d, loss_acc[mem]);
          }
        }
      }
    }
  }
  if (a.loss == LOSS_NONE) return;
#pragma unroll
  for (int mem = 0; mem < 2; ++mem) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) loss_acc[mem] += __shfl_xor(loss_acc[mem], o, 64);
    if (lane == 0 && tail) red[mem][wave] = loss_acc[mem];
  }
  __syncthreads();
  if (tid < 2)
    a.fitness[2 * pair + tid] = -(red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3]) / (static_cast<float>(B) * A);
}

// Two floats rounded to bf16 (one conversion instruction) and max(x, 0) taken on both halves at once.
typedef short short2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t relu_pack_bf16x2(float lo, float hi) {
  const bf16x2_t r = __builtin_convertvector(float2v{lo, hi}, bf16x2_t);
  const short2v h = __builtin_elementwise_max(__builtin_bit_cast(short2v, r), short2v{0, 0});
  return __builtin_bit_cast(uint32_t, h);
}

// ---- register-resident kernel for more than 64 observations per member -----------------------------
// With hundreds of observations per member the weights are a small part of the traffic and the layer
// products are real matrix work.  Four waves per member; wave w owns neurons 64 w .. 64 w + 63 of both
// hidden layers, i.e. two 32-neuron tiles, and builds every matrix operand of its weights once (a
// prologue: 16-byte loads, the wave-private staging tile and the transposed read of the streaming
// kernel), 48 operands = 192 registers per lane, the member's 173 KB across the workgroup.  The tile
// loop over 64 observations then runs with no weight traffic at all.  Products are transposed (rows =
// neurons, columns = 32 observations): one 16-byte LDS read of activations feeds two matrix
// instructions (the wave's two neuron tiles), which halves the LDS traffic per instruction against
// one tile per wave -- with one tile per wave the 1 KB operand per instruction is exactly the CU's
// LDS bandwidth when all four SIMDs issue back to back.  The observations of the next tile are
// requested before the current tile's layers run.
template <int D0, int H, int A, int MT, bool RELU>
__global__ __launch_bounds__(256) void mlp_bf16_resident_kernel(Bf16Args a) {
  constexpr int kRows = 32 * MT;  // observations per pass of the tile loop
  static_assert(H == 256 && D0 % 32 == 0 && A == 16 && (MT == 2 || MT == 4), "shape of the resident kernel");
  constexpr int LD0 = D0 + kRowPad, LDH = H + kRowPad;
  constexpr int U1 = D0 / 16, U2 = H / 16, U3 = H / 32;
  extern __shared__ __attribute__((aligned(16))) uint16_t resident_lds[];  // resident_lds_bytes(MT)
  uint16_t* x_s = resident_lds;                  // [kRows][LD0]
  uint16_t* h_s = x_s + kRows * LD0;             // [kRows][LDH]
  __shared__ float red[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, g = lane >> 5;
  const int c16 = lane & 15, g4 = lane >> 4;
  const int member = blockIdx.x, B = a.B;
  const uint16_t* theta = a.params + static_cast<size_t>(member) * a.sh.P;
  const uint16_t* W1 = theta;
  const uint16_t* B1 = W1 + D0 * H;
  const uint16_t* W2 = B1 + H;
  const uint16_t* B2 = W2 + H * H;
  const uint16_t* W3 = B2 + H;
  const uint16_t* B3 = W3 + H * A;

  // observations of a tile: 64 x D0 floats, 16-byte pieces, kObsPieces per thread
  constexpr int kObsPieces = kRows * D0 / 4 / 256;
  const float* obs_member = a.obs + static_cast<size_t>(member) * a.obs_stride;
  float4 ov[kObsPieces];
  auto load_obs = [&](int row0) {
#pragma unroll
    for (int j = 0; j < kObsPieces; ++j) {
      const int i = tid + 256 * j, r = i / (D0 / 4), d4 = i - r * (D0 / 4);
      ov[j] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (row0 + r < B) ov[j] = reinterpret_cast<const float4*>(obs_member + static_cast<size_t>(row0 + r) * D0)[d4];
    }
  };
  load_obs(0);

  // ---- prologue: this wave's matrix operands ---------------------------------------------------------
  // 16-byte loads of W (contiguous along the columns), a wave-private staging tile in LDS, and the
  // transposed read that hands every lane eight consecutive k of its column.  Four tiles per round trip
  // through LDS; the staging tiles borrow the wave's quarter of the (still unused) hidden-activation buffer.
  constexpr int kBatch = 4;
  uint16_t* stage = h_s + wave * (kRows * LDH / 4);
  static_assert(kBatch * kStageElems <= kRows * LDH / 4, "staging tiles fit into a quarter of the activation buffer");
  auto fence_wave = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // 16 rows x 32 columns of W1 / W2 per tile
  auto transposed12 = [&](const u32x4v* raw, bf16x8* out) {
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      *reinterpret_cast<u32x4v*>(stage + j * kStageElems + (lane >> 2) * kStageLd + 8 * (lane & 3)) = raw[j];
    fence_wave();
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const uint16_t* q = stage + j * kStageElems + (8 * g + (c16 >> 2)) * kStageLd + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q));
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q + 4 * kStageLd));
      out[j] = join_bf16(lo, hi);
    }
    fence_wave();
  };
  // 32 rows x 16 columns of W3 per tile
  auto transposed3 = [&](const u32x4v* raw, bf16x8* out) {
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      *reinterpret_cast<u32x4v*>(stage + j * kStageElems + (lane >> 1) * kStageLd3 + 8 * (lane & 1)) = raw[j];
    fence_wave();
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const uint16_t* q = stage + j * kStageElems + (8 * g4 + (c16 >> 2)) * kStageLd3 + 4 * (lane & 3);
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q));
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(q + 4 * kStageLd3));
      out[j] = join_bf16(lo, hi);
    }
    fence_wave();
  };
  static_assert(U1 % kBatch == 0 && U2 % kBatch == 0 && U3 % kBatch == 0, "operands come in rounds of four");
  bf16x8 w1[2][U1], w2[2][U2], w3[U3];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const uint16_t* p12 = theta + static_cast<size_t>(lane >> 2) * H + 32 * (2 * wave + t) + 8 * (lane & 3);
    u32x4v raw[U1 + U2];
#pragma unroll
    for (int u = 0; u < U1; ++u) raw[u] = *reinterpret_cast<const u32x4v*>(p12 + static_cast<size_t>(16 * u) * H);
#pragma unroll
    for (int u = 0; u < U2; ++u)
      raw[U1 + u] = *reinterpret_cast<const u32x4v*>(p12 + (W2 - theta) + static_cast<size_t>(16 * u) * H);
#pragma unroll
    for (int u = 0; u < U1; u += kBatch) transposed12(raw + u, w1[t] + u);
#pragma unroll
    for (int u = 0; u < U2; u += kBatch) transposed12(raw + U1 + u, w2[t] + u);
  }
  {
    const uint16_t* p3 = W3 + (lane >> 1) * A + 8 * (lane & 1);
    u32x4v raw[U3];
#pragma unroll
    for (int u = 0; u < U3; ++u) raw[u] = *reinterpret_cast<const u32x4v*>(p3 + 32 * u * A);
#pragma unroll
    for (int u = 0; u < U3; u += kBatch) transposed3(raw + u, w3 + u);
  }
  // The hidden layers' biases enter as one more product: a weight operand whose k = 0 column is the bias
  // of the lane's neuron (everything else zero) times an activation operand whose k = 0 row is one.  The
  // accumulators then start from that product with a zero addend: no bias registers, no initial copies.
  bf16x8 wb1[2], wb2[2], ones;
  {
    Pack8 p;
    p.v = make_uint4(0u, 0u, 0u, 0u);
    if (g == 0) p.h[0] = 0x3F80;  // bf16 1.0
    ones = p.b;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      p.v = make_uint4(0u, 0u, 0u, 0u);
      if (g == 0) p.h[0] = B1[64 * wave + 32 * t + c];
      wb1[t] = p.b;
      p.v = make_uint4(0u, 0u, 0u, 0u);
      if (g == 0) p.h[0] = B2[64 * wave + 32 * t + c];
      wb2[t] = p.b;
    }
  }
  float bias3[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) bias3[i] = from_bf16(B3[4 * g4 + i]);

  // activation, two bf16 per word, four consecutive neurons of one observation per 8-byte store.
  // RELU: rounding keeps the sign, so max(x, 0) is taken after the rounding, on both halves of a word at
  // once as a signed 16-bit maximum (a negative bf16 is a negative int16).
  auto store_rows = [&](const floatx16& acc, int t, int mt, int act) {
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      uint2 pk;
      if (RELU) {
        pk.x = relu_pack_bf16x2(acc[4 * rr], acc[4 * rr + 1]);
        pk.y = relu_pack_bf16x2(acc[4 * rr + 2], acc[4 * rr + 3]);
      } else {
        pk.x = pack_bf16x2(act_f(acc[4 * rr], act), act_f(acc[4 * rr + 1], act));
        pk.y = pack_bf16x2(act_f(acc[4 * rr + 2], act), act_f(acc[4 * rr + 3], act));
      }
      *reinterpret_cast<uint2*>(h_s + (mt * 32 + c) * LDH + 64 * wave + 32 * t + 8 * rr + 4 * g) = pk;
    }
  };
  // One layer's products: step s = (k-slice s / 2, observation tile s % 2) reads one activation operand and
  // feeds the wave's two neuron tiles.  The reads run kAhead steps ahead of the matrix instructions; the
  // scheduling fences keep that order (left alone, the compiler issues each read right before its use).
  constexpr int kAhead = 3;
  auto layer_products = [&](floatx16 (&acc)[2][MT], const uint16_t* in, int ld, const bf16x8 (&wb)[2], auto wt,
                            auto steps_c) {
    constexpr int kSteps = decltype(steps_c)::value;
    const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      acc[0][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[0], ones, zero, 0, 0, 0);
      acc[1][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[1], ones, zero, 0, 0, 0);
    }
    uint4 av[kSteps];
    auto read = [&](int s) { av[s] = *reinterpret_cast<const uint4*>(in + ((s % MT) * 32 + c) * ld + 16 * (s / MT) + 8 * g); };
#pragma unroll
    for (int s = 0; s < kAhead && s < kSteps; ++s) read(s);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      if (s + kAhead < kSteps) read(s + kAhead);
      __builtin_amdgcn_sched_barrier(0);
      acc[0][s % MT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wt(0, s / MT), as_bf16x8(av[s]), acc[0][s % MT], 0, 0, 0);
      acc[1][s % MT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wt(1, s / MT), as_bf16x8(av[s]), acc[1][s % MT], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  float loss_acc = 0.f;
#pragma unroll 1
  for (int row0 = 0; row0 < B; row0 += kRows) {
    // ---- observations -> bf16 rows (rows beyond B are zero); the next tile's are requested at once ----
#pragma unroll
    for (int j = 0; j < kObsPieces; ++j) {
      const int i = tid + 256 * j, r = i / (D0 / 4), d4 = i - r * (D0 / 4);
      uint2 pk;
      pk.x = pack_bf16x2(ov[j].x, ov[j].y);
      pk.y = pack_bf16x2(ov[j].z, ov[j].w);
      *reinterpret_cast<uint2*>(x_s + r * LD0 + 4 * d4) = pk;
    }
    if (row0 + kRows < B) load_obs(row0 + kRows);
    // layer 3: a wave takes MT / 2 groups of 16 observations; lane = observation c16 of a group, outputs 4 g4 ..
    constexpr int kGroups = MT / 2;
    float4 tgt[kGroups];
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
      const int row = row0 + 16 * (kGroups * wave + gi) + c16;
      tgt[gi] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (a.loss != LOSS_NONE && row < B)
        tgt[gi] = *reinterpret_cast<const float4*>(a.target + (static_cast<size_t>(member) * B + row) * A + 4 * g4);
    }
    __syncthreads();  // x_s is complete; every wave has left layer 3 of the previous tile

    // ---- layer 1 ------------------------------------------------------------------------------------
    floatx16 acc[2][MT];
    layer_products(acc, x_s, LD0, wb1, [&](int t, int u) { return w1[t][u]; }, std::integral_constant<int, MT * U1>{});
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) store_rows(acc[t][mt], t, mt, RELU ? EVO_ACT_RELU : a.sh.act[0]);
    __syncthreads();

    // ---- layer 2 ------------------------------------------------------------------------------------
    layer_products(acc, h_s, LDH, wb2, [&](int t, int u) { return w2[t][u]; }, std::integral_constant<int, MT * U2>{});
    __syncthreads();  // every wave has read h1: the buffer can take h2
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) store_rows(acc[t][mt], t, mt, RELU ? EVO_ACT_RELU : a.sh.act[1]);
    __syncthreads();

    // ---- layer 3: 16x16x32 tiles (lane = 16 g4 + c16), MT / 2 groups of 16 observations per wave ----------
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
      const int local = 16 * (kGroups * wave + gi) + c16, row = row0 + local;
      floatx4v o = {bias3[0], bias3[1], bias3[2], bias3[3]};
#pragma unroll
      for (int u = 0; u < U3; ++u) {
        const uint4 av = *reinterpret_cast<const uint4*>(h_s + local * LDH + 32 * u + 8 * g4);
        o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w3[u], as_bf16x8(av), o, 0, 0, 0);
      }
      if (row < B) {
        const int act = RELU ? EVO_ACT_NONE : a.sh.act[2];
        const float v0 = act_f(o[0], act), v1 = act_f(o[1], act), v2 = act_f(o[2], act), v3 = act_f(o[3], act);
        if (a.loss == LOSS_NONE) {
          *reinterpret_cast<float4*>(a.out + (static_cast<size_t>(member) * B + row) * A + 4 * g4) = make_float4(v0, v1, v2, v3);
        } else {
          const float d0 = v0 - tgt[gi].x, d1 = v1 - tgt[gi].y, d2 = v2 - tgt[gi].z, d3 = v3 - tgt[gi].w;
          loss_acc = fmaf(d0, d0, loss_acc);
          loss_acc = fmaf(d1, d1, loss_acc);
          loss_acc = fmaf(d2, d2, loss_acc);
          loss_acc = fmaf(d3, d3, loss_acc);
        }
      }
    }
  }
  if (a.loss == LOSS_NONE) return;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) loss_acc += __shfl_xor(loss_acc, o, 64);
  if (lane == 0) red[wave] = loss_acc;
  __syncthreads();
  if (tid == 0) a.fitness[member] = -(red[0] + red[1] + red[2] + red[3]) / (static_cast<float>(B) * A);
}

template <int D0, int H, int MT>
constexpr size_t resident_lds_bytes() {
  return static_cast<size_t>(32 * MT) * (D0 + kRowPad + H + kRowPad) * sizeof(uint16_t);
}

constexpr int kStreamMaxRows = 4096;  // observations per member of the streaming kernel (tiles of 64)

static bool stream_shape(const MlpShape& sh, int B) {
  return sh.n_layers == 3 && sh.dims[0] == 64 && sh.dims[1] == 256 && sh.dims[2] == 256 && sh.dims[3] == 16 &&
         B <= kStreamMaxRows;
}

int mlp_bf16_supported(const MlpShape& sh, int B) {
  if (B >= 1 && stream_shape(sh, B)) return EVO_OK;  // the streaming kernel walks over tiles of 64 rows
  EVO_REQUIRE(B >= 1 && B <= kMaxRows, EVO_ERR_UNSUPPORTED, "bf16 MLP: B must be in [1, %d] (got %d)", kMaxRows, B);
  EVO_REQUIRE(sh.max_width <= kMaxWidth, EVO_ERR_UNSUPPORTED, "bf16 MLP: widths above %d are not supported (%d)",
              kMaxWidth, sh.max_width);
  for (int l = 0; l < sh.n_layers; ++l)
    EVO_REQUIRE(sh.dims[l] % 16 == 0, EVO_ERR_UNSUPPORTED,
                "bf16 MLP: every layer input width must be a multiple of 16 (dims[%d] = %d)", l, sh.dims[l]);
  return EVO_OK;
}

int launch_mlp_bf16(const MlpShape& sh, const uint16_t* params, const float* obs, int64_t obs_stride, int pop, int B,
                    float* out, int loss, const void* target, float* fitness, hipStream_t s) {
  EVO_REQUIRE(loss != LOSS_CE, EVO_ERR_UNSUPPORTED, "bf16 MLP: the classification loss is not implemented");
  Bf16Args a;
  a.sh = sh, a.params = params, a.obs = obs, a.obs_stride = obs_stride, a.B = B;
  a.out = out, a.target = static_cast<const float*>(target), a.fitness = fitness, a.loss = loss;
  if (stream_shape(sh, B)) {
    const bool relu = sh.act[0] == EVO_ACT_RELU && sh.act[1] == EVO_ACT_RELU && sh.act[2] == EVO_ACT_NONE;
    if (B <= 64) {
      if (relu)
        hipLaunchKernelGGL((mlp_bf16_stream_kernel<64, 256, 16, true>), dim3(pop), dim3(512), 0, s, a);
      else
        hipLaunchKernelGGL((mlp_bf16_stream_kernel<64, 256, 16, false>), dim3(pop), dim3(512), 0, s, a);
    } else {
      constexpr int MT = 2;  // 64 observations per pass (128 measured slower: 2.17 vs 1.64 ms at B = 2048)
      constexpr size_t lds = resident_lds_bytes<64, 256, MT>();
      const void* fn = relu ? reinterpret_cast<const void*>(&mlp_bf16_resident_kernel<64, 256, 16, MT, true>)
                            : reinterpret_cast<const void*>(&mlp_bf16_resident_kernel<64, 256, 16, MT, false>);
      hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
      EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(e));
      if (relu)
        hipLaunchKernelGGL((mlp_bf16_resident_kernel<64, 256, 16, MT, true>), dim3(pop), dim3(256), lds, s, a);
      else
        hipLaunchKernelGGL((mlp_bf16_resident_kernel<64, 256, 16, MT, false>), dim3(pop), dim3(256), lds, s, a);
      return check_launch("mlp_bf16_resident_kernel");
    }
    return check_launch("mlp_bf16_stream_kernel");
  }
  // registers follow the widest layer, in classes of 64
  // LDS: the largest window as rows, behind it a ragged last layer (or 32 rows of it), the biases, and what a read beyond
  // the last of them takes; the errors of the outputs later take its place
  const int A = sh.dims[sh.n_layers], K_last = sh.dims[sh.n_layers - 1];
  const bool ragged = (A & 7) != 0;
  a.window_params = ragged ? sh.P - (K_last + 1) * A : sh.P;
  const int nt_class = (sh.max_width + 63) / 64 * 4, window = gen_window(nt_class);
  size_t lds = 0, rows_bytes = 0;
  int w_end = window, off = 0;
  for (int l = 0; l < sh.n_layers - (ragged ? 1 : 0); ++l) {
    const int K = sh.dims[l], N = sh.dims[l + 1];
    for (int k0 = 0; k0 < K; k0 += 32) {
      const int end = gen_step_end(off, k0, K, N);
      if (end > w_end) w_end = off + k0 * N + window, rows_bytes = 0;  // this step opens a window
      rows_bytes += static_cast<size_t>(32) * gen_stride(N);
      lds = rows_bytes > lds ? rows_bytes : lds;
    }
    off += K * N + N;
  }
  a.rag_at = static_cast<int>(lds);
  a.rag_rows = 0;
  if (ragged) {
    a.rag_rows = gen_rows(K_last) * gen_stride(A) <= 24 * 1024 ? K_last : 32;
    lds += static_cast<size_t>(a.rag_rows >= K_last ? gen_rows(K_last) : 32) * gen_stride(A);
  }
  a.bias_at = static_cast<int>(lds);
  for (int l = 0; l < sh.n_layers; ++l) lds += sizeof(uint16_t) * sh.dims[l + 1];
  lds = ((lds + 15) & ~size_t(15)) + 32 * nt_class;
  const size_t errors = loss == LOSS_NONE ? 0 : sizeof(float) * kMaxRows * gen_error_stride(A);
  lds = lds > errors ? lds : errors;
  auto launch = [&](auto kern) -> int {
    if (lds > 64 * 1024) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                         static_cast<int>(lds));
      if (e != hipSuccess) (void)hipGetLastError();
      EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(e));
    }
    hipLaunchKernelGGL(kern, dim3(pop), dim3(kBf16Threads), lds, s, a);
    return check_launch("mlp_bf16_generic_kernel");
  };
  if (nt_class == 4) return launch(mlp_bf16_generic_kernel<4>);
  if (nt_class == 8) return launch(mlp_bf16_generic_kernel<8>);
  if (nt_class == 12) return launch(mlp_bf16_generic_kernel<12>);
  return launch(mlp_bf16_generic_kernel<16>);
}

int mlp_bf16_pair_supported(const MlpShape& sh, int B) {
  EVO_REQUIRE(stream_shape(sh, B) && B <= 64, EVO_ERR_UNSUPPORTED,
              "ask fused with the forward: the policy must be the bfloat16 MLP 64-256-256-16 with at most 64 "
              "observations per member");
  return EVO_OK;
}

int launch_mlp_bf16_pair(const MlpShape& sh, const float* mu, const float* sigma, uint64_t seed, uint32_t gen,
                         const uint32_t* gen_dev, const float* obs, int64_t obs_stride, int pop, int B, float* out,
                         int loss, const void* target, float* fitness, hipStream_t s) {
  EVO_REQUIRE(loss != LOSS_CE, EVO_ERR_UNSUPPORTED, "bf16 MLP: the classification loss is not implemented");
  PairArgs a;
  a.sh = sh, a.mu = mu, a.sigma = sigma;
  a.key0 = static_cast<uint32_t>(seed), a.key1 = static_cast<uint32_t>(seed >> 32), a.gen = gen, a.gen_dev = gen_dev;
  a.obs = obs, a.obs_stride = obs_stride, a.B = B;
  a.out = out, a.target = static_cast<const float*>(target), a.fitness = fitness, a.loss = loss;
  const bool relu = sh.act[0] == EVO_ACT_RELU && sh.act[1] == EVO_ACT_RELU && sh.act[2] == EVO_ACT_NONE;
  constexpr size_t lds = pair_lds_bytes<64, 256, 16>();
  static_assert(lds + 64 <= 160 * 1024, "LDS budget of a CU");
  const void* fn = relu ? reinterpret_cast<const void*>(&mlp_bf16_pair_kernel<64, 256, 16, true>)
                        : reinterpret_cast<const void*>(&mlp_bf16_pair_kernel<64, 256, 16, false>);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) (void)hipGetLastError();
  EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "hipFuncSetAttribute failed: %s", hipGetErrorString(e));
  if (relu)
    hipLaunchKernelGGL((mlp_bf16_pair_kernel<64, 256, 16, true>), dim3(pop / 2), dim3(512), lds, s, a);
  else
    hipLaunchKernelGGL((mlp_bf16_pair_kernel<64, 256, 16, false>), dim3(pop / 2), dim3(512), lds, s, a);
  return check_launch("mlp_bf16_pair_kernel");
}

}  // namespace evo
