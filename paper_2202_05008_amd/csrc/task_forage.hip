// The shared-world task: the whole population lives as agents of one world (Section 3, WaterWorld
// paragraph: every member is spawned in the same task roll-out and measured there).  The paper
// gives the scheme, not the rules; the world is this library's own definition, stated in
// include/evo.h (unit square, food and poison items that reappear elsewhere once eaten, sensing of
// the nearest food, poison and other agent, point-mass motion with drag and walls).
//
// Agents of one world see each other's positions of the current step, so a step is a dependency
// between all workgroups of a world.  Two forms, the same trajectories bit for bit: the whole episode in
// one launch whose workgroups hand positions over to each other (world_resident_kernel below), and one
// launch per step, positions double-buffered in the task's workspace (world_step_kernel: into recorded
// graphs, for worlds that do not fit the chip, and for the single-step hook).
// A step's launch is a few microseconds of work spread as widely as its parallelism allows:
//   workgroup = 8 agents x 4 worlds, two waves per world (main and helper; the four main waves read
//   the same policy weights);
//   eight lanes per agent: they split the nearest-neighbour scans (each judges two candidates per
//   16-byte LDS read, then a three-stage reduction on (distance, index) by lane moves) and the hidden
//   units of the policy (each an eighth of a layer; the layer's activations go round by lane shuffles);
//   the helper wave stages half of the positions, places the items and keeps their book, scans the item
//   lists and the upper half of the agents, leaves its results in LDS and exits; the main wave scans the
//   lower half, merges, runs the policy, moves its agents and tests the touches.
// Everything that decides an integer -- who is nearest, who touches an item -- is computed in
// binary32 with each operation rounded on its own (no fused multiply-add), as the task defines it.
#include <algorithm>

#include "kernels.h"

#include <atomic>
#include <cfloat>
#include <cmath>
#include <mutex>
#include "philox.h"

namespace evo {

constexpr uint32_t kTagAgent = EVO_TAG_WORLD_AGENT;  // Philox streams of the start positions and of the items
constexpr uint32_t kTagItem = EVO_TAG_WORLD_ITEM;
constexpr int kObs = 8;
constexpr int kLanesPerAgent = 8;
constexpr int kAgentsPerBlock = 64 / kLanesPerAgent;  // a wave; the workgroup's waves are worlds
constexpr int kWorldsPerBlock = 4;
constexpr int kStepThreads = 2 * 64 * kWorldsPerBlock;  // per world a main wave and a helper wave

__host__ __device__ constexpr int pad_to(int n, int m) { return (n + m - 1) / m * m; }

struct WorldConst {
  float dt, thrust, drag, vmax, r2;
  int n_food, n_items;
};

struct StepArgs {
  const float* params;  // [pop][P]; unused when actions_in is set
  int P, pop, worlds;
  int act[3];
  WorldConst c;
  uint32_t key0, key1, gen;
  const uint32_t* gen_dev;
  const float2* pos_in;      // [worlds][pop]
  float2* pos_out;           // [worlds][pop]
  const float2* vel_in;      // [worlds][pop]
  float2* vel_out;           // [worlds][pop] (may alias vel_in: an agent's velocity is its own)
  int32_t* reward;           // [worlds][pop]: += this step's reward (accumulate) or = (otherwise)
  int accumulate;
  const uint32_t* counts_in;   // [worlds][n_items]: times each item was eaten before the previous step
  const uint32_t* hits_prev;   // [worlds][n_items] or null: eaten in the previous step
  uint32_t* counts_out;        // [worlds][n_items] or null: counts_in + hits_prev, for the next step
  uint32_t* hits_cur;          // [worlds][n_items]: set to 1 for every item touched in this step (zero on entry)
  uint32_t* hits_clear;        // [worlds][n_items] or null: zeroed for the step after the next
  const float2* actions_in;    // test hook: [worlds][pop] actions instead of the policy's
  float* obs_out;              // test hook: [worlds][pop][8]
};

// Value of the partner lane in the butterfly stages that cover an agent's eight (or sixteen) lanes, as
// data-parallel-primitive moves (register to register, no trip through LDS): stage 0 swaps
// neighbours, stage 1 swaps pairs (both quad permutations), stage 2 mirrors the eight lanes, which
// pairs each lane of one quad with a lane of the other, stage 3 mirrors a row of sixteen lanes.
template <int STAGE>
__device__ __forceinline__ int partner_bits(int x) {
  // quad_perm 1,0,3,2 / quad_perm 2,3,0,1 / row_half_mirror / row_mirror
  constexpr int ctrl = STAGE == 0 ? 0xB1 : STAGE == 1 ? 0x4E : STAGE == 2 ? 0x141 : 0x140;
  // every lane has a partner in these patterns, so the value for lanes without one is never used
  return __builtin_amdgcn_update_dpp(0, x, ctrl, 0xF, 0xF, true);
}
template <int STAGE>
__device__ __forceinline__ float partner(float x) {
  return __int_as_float(partner_bits<STAGE>(__float_as_int(x)));
}
// Value of the lane N places away in the rotation of a row of sixteen lanes (the lanes of one agent when it has
// sixteen), again register to register.  Which way the hardware rotates does not matter to the callers: they
// apply the same move to the lane number to learn whose value they receive.
template <int N>
__device__ __forceinline__ int rotated_bits(int x) {
  static_assert(N >= 1 && N <= 15, "a rotation inside a row");
  return __builtin_amdgcn_update_dpp(0, x, 0x120 + N, 0xF, 0xF, true);  // row_ror:N
}
template <int N>
__device__ __forceinline__ float rotated(float x) {
  return __int_as_float(rotated_bits<N>(__float_as_int(x)));
}

// Sum over an agent's LPA lanes (8 or 16), left in every one of them.
template <int LPA = kLanesPerAgent>
__device__ __forceinline__ float agent_sum(float x) {
  static_assert(LPA == 8 || LPA == 16, "the butterfly covers eight or sixteen lanes");
  x += partner<0>(x);
  x += partner<1>(x);
  x += partner<2>(x);
  if (LPA == 16) x += partner<3>(x);
  return x;
}
template <int LPA = kLanesPerAgent>
__device__ __forceinline__ int agent_sum(int x) {
  x += partner_bits<0>(x);
  x += partner_bits<1>(x);
  x += partner_bits<2>(x);
  if (LPA == 16) x += partner_bits<3>(x);
  return x;
}

// The task's distance: products and sum rounded one by one.
__device__ __forceinline__ float dist2(float dx, float dy) {
#pragma clang fp contract(off)
  const float xx = dx * dx;
  const float yy = dy * dy;
  return xx + yy;
}

// Nearest candidate so far: distance and index (the offset is read back from the index at the end).
struct Nearest {
  float d2;
  int idx;
};

// Candidates arrive in increasing index within a lane: strict "<" keeps the lowest index.
template <bool CHECK>
__device__ __forceinline__ void nearest_offer(Nearest& n, float2 p, float ox, float oy, int idx, int self) {
  const float d2 = dist2(ox - p.x, oy - p.y);
  bool take = d2 < n.d2;
  if (CHECK) take = take && idx != self;
  n.d2 = take ? d2 : n.d2;
  n.idx = take ? idx : n.idx;
}

// 64 candidates: four chunks of 2 per lane and 8 lanes.
__device__ __forceinline__ void load_scan64(float4 (&c)[4], const float2* s, int base, int q) {
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = *reinterpret_cast<const float4*>(s + base + k * 2 * kLanesPerAgent + 2 * q);
}

template <bool CHECK>
__device__ __forceinline__ void nearest_scan64(Nearest& n, float2 p, const float4 (&c)[4], int base, int q, int self) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int i = base + k * 2 * kLanesPerAgent + 2 * q;
    nearest_offer<CHECK>(n, p, c[k].x, c[k].y, i, self);
    nearest_offer<CHECK>(n, p, c[k].z, c[k].w, i + 1, self);
  }
}

// One chunk of candidates, two per lane of the agent (the item lists are short).
__device__ __forceinline__ void nearest_scan16(Nearest& n, float2 p, const float2* s, int base, int q) {
  const float4 c = *reinterpret_cast<const float4*>(s + base + 2 * q);
  nearest_offer<false>(n, p, c.x, c.y, base + 2 * q, -1);
  nearest_offer<false>(n, p, c.z, c.w, base + 2 * q + 1, -1);
}

// Smallest value over an agent's lanes, in every one of them.
template <int LPA = kLanesPerAgent>
__device__ __forceinline__ uint32_t agent_min(uint32_t x) {
  x = min(x, static_cast<uint32_t>(partner_bits<0>(x)));
  x = min(x, static_cast<uint32_t>(partner_bits<1>(x)));
  x = min(x, static_cast<uint32_t>(partner_bits<2>(x)));
  if (LPA == 16) x = min(x, static_cast<uint32_t>(partner_bits<3>(x)));
  return x;
}

// Merge over the lanes of an agent (smallest distance, then the lowest index that has it) and read the offset back.  A
// distance is a sum of squares or the initial infinity, and non-negative floats order like their bit patterns.  (Pairs of
// distance and index through every stage take twice the instructions: 1024 members alone, 500 steps 640 -> 604 us.)
template <int LPA = kLanesPerAgent>
__device__ __forceinline__ float2 nearest_finish(Nearest n, float2 p, const float2* s, int limit) {
  const uint32_t d = __float_as_uint(n.d2), m = agent_min<LPA>(d);
  const int idx = static_cast<int>(agent_min<LPA>(d == m ? static_cast<uint32_t>(n.idx) : 0x7fffffffu));
  if (idx >= limit) return make_float2(0.f, 0.f);  // nothing comparable (non-finite positions)
  const float2 o = s[idx];
  return make_float2(o.x - p.x, o.y - p.y);
}

__device__ __forceinline__ float tanh_hw(float x) {
  const float e = __builtin_amdgcn_exp2f(2.885390081777927f * x);  // e^{2x}
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}

__device__ __forceinline__ float activate(float x, int act) {
  if (act == EVO_ACT_TANH) return tanh_hw(x);
  if (act == EVO_ACT_RELU) return fmaxf(x, 0.f);
  return x;
}

// A lane's slice of the policy's weights (columns c0 .. c0 + HQ - 1 of every layer, rows c0 .. of the
// last one), loaded at the start of the kernel so that the round trip to L2 runs under the scans.
template <int H, int LPA = kLanesPerAgent>
struct PolicySlice {
  static constexpr int HQ = H / LPA;
  static_assert(HQ >= 2 && HQ % 2 == 0, "a lane's columns are loaded two at a time");
  static constexpr int kRows2 = H <= 32 ? H : 8;   // rows of W2 held here; the rest is read when it is used
  // With sixteen lanes per agent and the whole of W2 held here, the rows sit in the order in which the hidden
  // activations reach the lane by rotations of its row: w2[n HQ + v] is the row of activation v of the lane whose
  // value rotation n delivers (n = 0: the lane's own), so layer 2 needs no gather at all.
  static constexpr bool kRotated = LPA == 16 && kRows2 == H;
  float w1[kObs][HQ], b1[HQ], w2[kRows2][HQ], b2[HQ], w3[HQ][2], b3[2];
  const float* rest;  // &W2[kRows2][c0]
};

// Rows of W2 in rotation order (see PolicySlice): rotation N delivers the value of lane `from`.
template <int H, int LPA, int N>
__device__ __forceinline__ void rotated_rows(const float* __restrict__ W2, int q, int c0, PolicySlice<H, LPA>& s) {
  constexpr int HQ = PolicySlice<H, LPA>::HQ;
  if constexpr (N < 16) {
    int from = q;
    if constexpr (N > 0) from = rotated_bits<N>(q);
#pragma unroll
    for (int v = 0; v < HQ; ++v)
#pragma unroll
      for (int u = 0; u < HQ; u += 2) {
        const float2 w = *reinterpret_cast<const float2*>(W2 + (from * HQ + v) * H + c0 + u);
        s.w2[N * HQ + v][u] = w.x, s.w2[N * HQ + v][u + 1] = w.y;
      }
    rotated_rows<H, LPA, N + 1>(W2, q, c0, s);
  }
}
// Layer 2 on activations that arrive by rotation: part[u] += h[from][v] W2[from HQ + v][c0 + u] for every lane of
// the agent in turn.
template <int H, int LPA, int N>
__device__ __forceinline__ void rotated_layer(const PolicySlice<H, LPA>& s, const float (&mine)[H / LPA],
                                              float (&part)[H / LPA]) {
  constexpr int HQ = H / LPA;
  if constexpr (N < 16) {
#pragma unroll
    for (int v = 0; v < HQ; ++v) {
#pragma unroll
      for (int u = 0; u < HQ; ++u) {
        if constexpr (N == 0) {
          part[u] = fmaf(mine[v], s.w2[v][u], part[u]);
        } else {
          // the rotation rides in the multiply-add itself (the compiler keeps it as a move of its own).  A lane
          // move may not read a register in the two instructions after it is written: the first of these
          // statements brings its own wait, the others read registers written long before
          if constexpr (N == 1)
            asm("s_nop 1\n\tv_fmac_f32_dpp %0, %1, %2 row_ror:%3 row_mask:0xf bank_mask:0xf bound_ctrl:0"
                : "+v"(part[u])
                : "v"(mine[v]), "v"(s.w2[N * HQ + v][u]), "n"(N));
          else
            asm("v_fmac_f32_dpp %0, %1, %2 row_ror:%3 row_mask:0xf bank_mask:0xf bound_ctrl:0"
                : "+v"(part[u])
                : "v"(mine[v]), "v"(s.w2[N * HQ + v][u]), "n"(N));
        }
      }
    }
    rotated_layer<H, LPA, N + 1>(s, mine, part);
  }
}

template <int H, int LPA>
__device__ __forceinline__ void policy_load(const float* __restrict__ th, int q, PolicySlice<H, LPA>& s) {
  constexpr int HQ = PolicySlice<H, LPA>::HQ;
  const int c0 = q * HQ;
  const float* W1 = th;
  const float* b1 = W1 + kObs * H;
  const float* W2 = b1 + H;
  const float* b2 = W2 + H * H;
  const float* W3 = b2 + H;
  const float* b3 = W3 + H * 2;
  auto row = [&](const float* src, float (&dst)[HQ]) {
#pragma unroll
    for (int u = 0; u < HQ; u += 2) {
      const float2 w = *reinterpret_cast<const float2*>(src + c0 + u);
      dst[u] = w.x, dst[u + 1] = w.y;
    }
  };
#pragma unroll
  for (int i = 0; i < kObs; ++i) row(W1 + i * H, s.w1[i]);
  row(b1, s.b1);
  if constexpr (PolicySlice<H, LPA>::kRotated) {
    rotated_rows<H, LPA, 0>(W2, q, c0, s);
  } else {
#pragma unroll
    for (int i = 0; i < PolicySlice<H, LPA>::kRows2; ++i) row(W2 + i * H, s.w2[i]);
  }
  s.rest = W2 + PolicySlice<H, LPA>::kRows2 * H + c0;
  row(b2, s.b2);
#pragma unroll
  for (int u = 0; u < HQ; ++u) {
    const float2 w = *reinterpret_cast<const float2*>(W3 + (c0 + u) * 2);
    s.w3[u][0] = w.x, s.w3[u][1] = w.y;
  }
  s.b3[0] = b3[0], s.b3[1] = b3[1];
}

// All H activations of a layer to every lane of the agent.
template <int H, int LPA>
__device__ __forceinline__ void gather_agent(const float (&mine)[H / LPA], int lane, float (&full)[H]) {
  constexpr int HQ = H / LPA;
#pragma unroll
  for (int s = 0; s < LPA; ++s)
#pragma unroll
    for (int u = 0; u < HQ; ++u) full[s * HQ + u] = __shfl(mine[u], (lane & ~(LPA - 1)) | s);
}

// The policy of dims (8, H, H, 2) for one agent; every lane of the agent returns both outputs.
// TANH: all three activations are tanh (the usual policy), known when the kernel is built: no switch per value.
template <int H, int LPA, bool TANH = false>
__device__ __forceinline__ float2 policy_forward(const PolicySlice<H, LPA>& s, const int (&act_rt)[3], int lane,
                                                 const float (&obs)[kObs]) {
  const int act[3] = {TANH ? EVO_ACT_TANH : act_rt[0], TANH ? EVO_ACT_TANH : act_rt[1],
                      TANH ? EVO_ACT_TANH : act_rt[2]};
  constexpr int HQ = PolicySlice<H, LPA>::HQ;
  float part[HQ], full[H];
#pragma unroll
  for (int u = 0; u < HQ; ++u) part[u] = s.b1[u];
#pragma unroll
  for (int i = 0; i < kObs; ++i)
#pragma unroll
    for (int u = 0; u < HQ; ++u) part[u] = fmaf(obs[i], s.w1[i][u], part[u]);
#pragma unroll
  for (int u = 0; u < HQ; ++u) part[u] = activate(part[u], act[0]);
  if constexpr (PolicySlice<H, LPA>::kRotated) {
    float h1[HQ];
#pragma unroll
    for (int u = 0; u < HQ; ++u) h1[u] = part[u], part[u] = s.b2[u];
    rotated_layer<H, LPA, 0>(s, h1, part);
  } else {
    gather_agent<H, LPA>(part, lane, full);
#pragma unroll
    for (int u = 0; u < HQ; ++u) part[u] = s.b2[u];
#pragma unroll
    for (int i = 0; i < PolicySlice<H, LPA>::kRows2; ++i)
#pragma unroll
      for (int u = 0; u < HQ; ++u) part[u] = fmaf(full[i], s.w2[i][u], part[u]);
#pragma unroll 16
    for (int i = PolicySlice<H, LPA>::kRows2; i < H; ++i)
#pragma unroll
      for (int u = 0; u < HQ; u += 2) {
        const float2 w = *reinterpret_cast<const float2*>(s.rest + (i - PolicySlice<H, LPA>::kRows2) * H + u);
        part[u] = fmaf(full[i], w.x, part[u]);
        part[u + 1] = fmaf(full[i], w.y, part[u + 1]);
      }
  }
#pragma unroll
  for (int u = 0; u < HQ; ++u) part[u] = activate(part[u], act[1]);
  float o0 = 0.f, o1 = 0.f;
#pragma unroll
  for (int u = 0; u < HQ; ++u) {
    o0 = fmaf(part[u], s.w3[u][0], o0);
    o1 = fmaf(part[u], s.w3[u][1], o1);
  }
  o0 = agent_sum<LPA>(o0), o1 = agent_sum<LPA>(o1);
  return make_float2(activate(o0 + s.b3[0], act[2]), activate(o1 + s.b3[1], act[2]));
}

// One axis of the motion: new velocity and position, each operation rounded on its own.
__device__ __forceinline__ void move_axis(const WorldConst& c, float a, float& p, float& v) {
#pragma clang fp contract(off)
  a = fminf(fmaxf(a, -1.f), 1.f);
  const float dv = c.drag * v;
  const float da = c.thrust * a;
  float nv = dv + da;
  nv = fminf(fmaxf(nv, -c.vmax), c.vmax);
  const float step = c.dt * nv;
  float np = p + step;
  if (np < 0.f) np = 0.f, nv = 0.f;
  if (np > 1.f) np = 1.f, nv = 0.f;
  p = np, v = nv;
}

// Touches of one list of items (16 slots per chunk); returns how many this lane found.
__device__ __forceinline__ int touch_scan(const WorldConst& c, float2 p, const float2* s, int padded, int q,
                                          uint32_t* hits) {
  int found = 0;
  for (int base = 0; base < padded; base += 2 * kLanesPerAgent) {
    const float4 it = *reinterpret_cast<const float4*>(s + base + 2 * q);
    if (dist2(it.x - p.x, it.y - p.y) <= c.r2) ++found, atomicOr(hits + base + 2 * q, 1u);
    if (dist2(it.z - p.x, it.w - p.y) <= c.r2) ++found, atomicOr(hits + base + 2 * q + 1, 1u);
  }
  return found;
}

// Per lane of a helper wave, for the main wave of the same world: its part of the agent scan and the
// two item offsets, as six words (structure of arrays: word w of lane l at [w][l]).
constexpr int kExchangeWords = 6;

template <int H, bool TANH>
__device__ __forceinline__ void world_step_block(StepArgs a, int block_x, int block_y, float4* lds4) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = wave & (kWorldsPerBlock - 1);  // which of the workgroup's worlds
  const bool helper = wave >= kWorldsPerBlock;    // waves 4..7 assist waves 0..3
  const int q = lane & (kLanesPerAgent - 1);
  const int agent0 = block_x * kAgentsPerBlock;
  const int agent = agent0 + lane / kLanesPerAgent;
  const int world = block_y * kWorldsPerBlock + slot;
  const bool world_live = world < a.worlds;
  const bool live = world_live && agent < a.pop;
  const int n_food = a.c.n_food, n_items = a.c.n_items;
  const int pop_pad = pad_to(a.pop, 64), food_pad = pad_to(n_food, 16), poison_pad = pad_to(n_items - n_food, 16);
  const int region = pop_pad + food_pad + poison_pad;
  // a world's region: every agent, the food, the poison; unused slots lie infinitely far away
  float2* s_pos = reinterpret_cast<float2*>(lds4) + slot * region;
  float2* s_food = s_pos + pop_pad;
  float2* s_poison = s_food + food_pad;
  float* s_xch = reinterpret_cast<float*>(reinterpret_cast<float2*>(lds4) + kWorldsPerBlock * region) +
                 slot * kExchangeWords * 64;
  if (a.gen_dev) a.gen = *a.gen_dev;
  const float inf = __builtin_inff();

  PolicySlice<H> weights;
  if (world_live) {
    const float2* pin = a.pos_in + static_cast<size_t>(world) * a.pop;
    const int role = helper ? 1 : 0;
    float2 t[8];  // the two waves of a world stage alternate runs of 64 positions: eight loads in flight each
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int j = (2 * k + role) * 64 + lane;
      t[k] = pin[min(j, a.pop - 1)];  // in bounds; slots past the last agent are replaced when they are stored
    }
    // main wave: the policy's weights, requested behind the positions; their round trip to L2 runs under
    // everything up to the forward pass
    if (!helper && live && !a.actions_in) policy_load<H>(a.params + static_cast<size_t>(agent) * a.P, q, weights);
    if (helper) {  // the items and their book
      for (int sl = lane; sl < food_pad + poison_pad; sl += 64) {
        const bool is_food = sl < food_pad;
        const int i = is_food ? sl : n_food + sl - food_pad;
        float2 where = make_float2(inf, inf);
        if (i < (is_food ? n_food : n_items)) {
          const size_t o = static_cast<size_t>(world) * n_items + i;
          uint32_t cnt = a.counts_in[o];
          if (a.hits_prev) cnt += a.hits_prev[o];
          if (block_x == 0) {  // one workgroup per world keeps the item book
            if (a.counts_out) a.counts_out[o] = cnt;
            if (a.hits_clear) a.hits_clear[o] = 0u;
          }
          const u32x4 w = philox4x32_10(256u * cnt + static_cast<uint32_t>(i), static_cast<uint32_t>(world), a.gen,
                                        kTagItem, a.key0, a.key1);
          where = make_float2(unit_open(w.x), unit_open(w.y));
        }
        s_food[sl] = where;  // the poison list follows the food list
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int j = (2 * k + role) * 64 + lane;
      if (j < pop_pad) s_pos[j] = j < a.pop ? t[k] : make_float2(inf, inf);  // the first use of the loaded values
    }
    for (int j = 1024 + role * 64 + lane; j < pop_pad; j += 128) s_pos[j] = j < a.pop ? pin[j] : make_float2(inf, inf);
  }
  __syncthreads();

  // The agent scan is shared: the main wave takes the first blocks of 64 candidates, the helper the rest
  // and the two item lists (about two blocks' worth of work).
  const int blocks = pop_pad / 64;
  const int main_blocks = min(blocks, (blocks + 3) / 2);
  const size_t me = static_cast<size_t>(world) * a.pop + min(agent, a.pop - 1);
  float2 p = make_float2(0.f, 0.f), v = p;
  Nearest other{inf, 0x7fffffff};
  float2 f = p, g = p;
  if (live) {
    p = s_pos[agent];
    const int own_block = agent0 & ~63;  // the only 64 candidates that hold agents of this wave
    // two sets of 64 candidates take turns: one is on its way from LDS while the other is judged
    auto judge = [&](const float4 (&c)[4], int base) {
      if (base == own_block)
        nearest_scan64<true>(other, p, c, base, q, agent);
      else
        nearest_scan64<false>(other, p, c, base, q, agent);
    };
    const int first = helper ? main_blocks * 64 : 0, last = helper ? pop_pad : main_blocks * 64;
    float4 ping[4], pong[4];
    if (first < last) load_scan64(ping, s_pos, first, q);
    for (int base = first; base < last; base += 128) {
      const bool second = base + 64 < last;
      if (second) load_scan64(pong, s_pos, base + 64, q);
      judge(ping, base);
      if (base + 128 < last) load_scan64(ping, s_pos, base + 128, q);
      if (second) judge(pong, base + 64);
    }
    if (helper) {
      Nearest food{inf, 0x7fffffff}, poison{inf, 0x7fffffff};
      for (int base = 0; base < food_pad; base += 16) nearest_scan16(food, p, s_food, base, q);
      for (int base = 0; base < poison_pad; base += 16) nearest_scan16(poison, p, s_poison, base, q);
      f = nearest_finish(food, p, s_food, food_pad);
      g = nearest_finish(poison, p, s_poison, poison_pad);
      s_xch[0 * 64 + lane] = other.d2;
      s_xch[1 * 64 + lane] = __int_as_float(other.idx);
      s_xch[2 * 64 + lane] = f.x, s_xch[3 * 64 + lane] = f.y;
      s_xch[4 * 64 + lane] = g.x, s_xch[5 * 64 + lane] = g.y;
    } else {
      v = a.vel_in[me];
    }
  }
  __syncthreads();
  if (helper || !live) return;  // no barrier below this line

  {  // the helper's candidates all have higher indices: they win only when strictly nearer
    const float hd = s_xch[0 * 64 + lane];
    const int hi = __float_as_int(s_xch[1 * 64 + lane]);
    const bool take = hd < other.d2;
    other.d2 = take ? hd : other.d2;
    other.idx = take ? hi : other.idx;
    f = make_float2(s_xch[2 * 64 + lane], s_xch[3 * 64 + lane]);
    g = make_float2(s_xch[4 * 64 + lane], s_xch[5 * 64 + lane]);
  }
  const float2 o = nearest_finish(other, p, s_pos, pop_pad);

  const float obs[kObs] = {v.x, v.y, f.x, f.y, g.x, g.y, o.x, o.y};
  if (a.obs_out && q == 0) {
    float4* dst = reinterpret_cast<float4*>(a.obs_out + me * kObs);
    dst[0] = make_float4(obs[0], obs[1], obs[2], obs[3]);
    dst[1] = make_float4(obs[4], obs[5], obs[6], obs[7]);
  }
  float2 action;
  if (a.actions_in)
    action = a.actions_in[me];
  else
    action = policy_forward<H, kLanesPerAgent, TANH>(weights, a.act, lane, obs);

  move_axis(a.c, action.x, p.x, v.x);
  move_axis(a.c, action.y, p.y, v.y);

  uint32_t* hits = a.hits_cur + static_cast<size_t>(world) * n_items;
  int reward = touch_scan(a.c, p, s_food, food_pad, q, hits) - touch_scan(a.c, p, s_poison, poison_pad, q, hits + n_food);
  reward = agent_sum(reward);
  if (q == 0) {
    a.pos_out[me] = p;
    a.vel_out[me] = v;
    a.reward[me] = a.accumulate ? a.reward[me] + reward : reward;
  }
}

template <int H, bool TANH>
__global__ __launch_bounds__(kStepThreads) void world_step_kernel(StepArgs a) {
  extern __shared__ float4 lds4[];
  world_step_block<H, TANH>(a, blockIdx.x, blockIdx.y, lds4);
}

// ---- the whole episode of shared worlds in one launch -----------------------------------------------------
// A launch per step takes 9.1 us (1024 agents, 8 worlds, H = 32), of which the gap, the reloading of the weights and the
// staging of four worlds are two thirds; this kernel's step takes 3.4 us, and 2.7 us where a world is small.  The agents
// stay where they are: a workgroup owns agents of ONE world for all steps, weights, state
// and reward in registers, and what a step has to hand over goes through memory as its own flag: an agent's position is
// one 8-byte word, x and y with the step's number modulo four in the two top bits of x (a coordinate lies in [0, 1], so
// they are free), and the items that a workgroup's agents touch are words of 32 items under the step's number.  Every workgroup
// polls the words of its world until all carry the number.  A word handed over and seen by everyone takes 1.6 us on this
// chip, the same whether a world's workgroups share a die or not (a plain load misses the news in the vector cache; atomics
// on the die's cache 3.3 us; invalidating the vector cache before a plain load 30 us).
//
// Waves: eight main waves own the agents: scan of the other agents, policy, motion, touches.  Beside their scan the item
// waves move the touched items (each of them in a copy of its own, so they need no order among themselves; where an item
// goes next is drawn ahead) and find the agents' nearest items, eight lanes per agent.
// Lanes of a main wave: the agent scan takes all 64 for the wave's agents together (a candidate is read from LDS once for
// four agents, and only the distance is tracked: 5.5 vector instructions per candidate instead of 8; the index is looked
// up afterwards among the candidates of the lane that holds the minimum).  Policy: sixteen lanes per agent for H <= 32;
// for H = 64 a wave per agent, since sixteen lanes would need 303 registers each for the weights.
// The order of every sum is world_step_kernel's, so the trajectories are its trajectories bit for bit.
// What a step consists of (cycles of a main wave at 1024 agents, 8600 in all when it was measured and a step took 3.6 us):
// waiting for the positions 2000 + 900 (the
// slowest workgroup), scan 2100 (at the issue rate of two main waves and an item wave per SIMD), look-up 500, waiting for
// the items 900, policy 950, motion and touches 1300 (a dependent chain at one instruction per 6 to 7 cycles).  With the
// items and touches in the main waves and one helper wave a step took 9600.
//
// A wait needs the other workgroups of the world on the chip.  The host launches no more workgroups than compute units
// and one such launch at a time; where other work holds the chip all the same, a wait ends after wait_ticks, the
// flag of the world's place in its launch is raised, everybody leaves, and world_rerun_kernel plays the world again from
// its start, on whatever part of the chip it gets.  The flag stays up for the episode's later launches: who waits at that
// place then leaves at the first look at it, and the place's worlds are played again, the finished ones for the same result.
// (A check of the launch before at each start took 10 % of the step, by other scalar registers for the loop; so did the
// place's number in place of the world's at H = 32, while H = 16 gained as much.)
constexpr int kMainWaves = 8;           // main waves per workgroup
constexpr int kMaxResident = 256;       // workgroups of a launch; the room in the workspace is for these
constexpr uint32_t kFar = 0x7F800000u;  // infinity's bits
constexpr int resident_lanes(int H) { return H <= 32 ? 16 : 64; }                           // of a main wave, per agent
constexpr int resident_agents(int H) { return kMainWaves * 64 / resident_lanes(H); }        // per workgroup
constexpr int item_waves(int H) { return resident_agents(H) / kAgentsPerBlock; }            // per workgroup
constexpr int resident_threads(int H) { return 64 * (kMainWaves + item_waves(H)); }

struct ResidentArgs {
  const float* params;  // [pop][P]
  int P, pop, worlds, steps;
  int act[3];
  WorldConst c;
  uint32_t key0, key1, gen;
  const uint32_t* gen_dev;
  int per_lane;          // candidates per lane of the agent scan (even)
  uint32_t lane_magic;   // ceil(2^32 / per_lane): j / per_lane is the high word of j times this for the j here
  unsigned long long* even;  // [worlds][pop] tagged positions of even and of odd steps
  unsigned long long* odd;
  unsigned long long* hand;  // [2][worlds of the launch][groups][chunks] tagged touches
  uint32_t tag0;             // the tag of step t's touches is tag0 + t (a number of no launch before)
  int world0, per_launch;    // the launch's first world and the most worlds it has
  int groups;                // workgroups of a world
  uint32_t* flag;            // of a world's place in the launch, at the world's number: a wait has ended without its word
  unsigned long long wait_ticks;  // of the 100 MHz clock
  // CHECK: from these steps on the main waves of the first fail_groups workgroups of a world wait for positions that nobody
  // hands over, and their item waves for such touches
  int fail_main, fail_items, fail_groups;
  int32_t* reward;       // [worlds][pop]
  float2* pos_out;       // [worlds][pop] state after the last step
  float2* vel_out;       // [worlds][pop]
  uint32_t* counts_out;  // [worlds][n_items] or null: the book after the last step
};

// A lane's columns c0 .. c0 + HQ - 1 of the layers, rows in their natural order.
template <int H, int LPA>
struct ResidentSlice {
  static constexpr int HQ = H / LPA;
  float w1[kObs][HQ], b1[HQ], w2[H][HQ], b2[HQ], w3[HQ][2], b3[2];
};
template <int H, int LPA>
__device__ __forceinline__ void resident_load(const float* __restrict__ th, int q, ResidentSlice<H, LPA>& s) {
  constexpr int HQ = ResidentSlice<H, LPA>::HQ;
  const int c0 = q * HQ;
  const float* W1 = th;
  const float* b1 = W1 + kObs * H;
  const float* W2 = b1 + H;
  const float* b2 = W2 + H * H;
  const float* W3 = b2 + H;
  const float* b3 = W3 + H * 2;
#pragma unroll
  for (int u = 0; u < HQ; ++u) {
#pragma unroll
    for (int i = 0; i < kObs; ++i) s.w1[i][u] = W1[i * H + c0 + u];
#pragma unroll
    for (int i = 0; i < H; ++i) s.w2[i][u] = W2[i * H + c0 + u];
    s.b1[u] = b1[c0 + u], s.b2[u] = b2[c0 + u];
    s.w3[u][0] = W3[(c0 + u) * 2], s.w3[u][1] = W3[(c0 + u) * 2 + 1];
  }
  s.b3[0] = b3[0], s.b3[1] = b3[1];
}

// Layer 2, sixteen lanes per agent: activation I of the agent, broadcast over its row inside the multiply-add.  A lane
// move may not read a register in the two instructions after it is written: the statements that read a register first
// (I < HQ) bring their own wait, and each chain runs through one of them per register before any other.
template <int H, int I>
__device__ __forceinline__ void row_layer(const ResidentSlice<H, 16>& s, const float (&mine)[H / 16],
                                          float (&part)[H / 16]) {
  constexpr int HQ = H / 16;
  if constexpr (I < H) {
#pragma unroll
    for (int u = 0; u < HQ; ++u) {
      if constexpr (I < HQ)
        asm("s_nop 1\n\tv_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
            : "+v"(part[u])
            : "v"(mine[I % HQ]), "v"(s.w2[I][u]), "n"(I / HQ));
      else
        asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
            : "+v"(part[u])
            : "v"(mine[I % HQ]), "v"(s.w2[I][u]), "n"(I / HQ));
    }
    row_layer<H, I + 1>(s, mine, part);
  }
}

template <int CTRL>
__device__ __forceinline__ float lane_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// The policy of dims (8, H, H, 2); every lane of the agent returns both outputs.  The sums are policy_forward's with
// eight lanes per agent: layers 1 and 2 from the bias over the inputs in order, layer 3 as eight chains of H / 8 neurons
// added in a tree of neighbours.
template <int H, int LPA, bool TANH>
__device__ __forceinline__ float2 resident_forward(const ResidentSlice<H, LPA>& s, const int (&act_rt)[3], int lane,
                                                   const float (&obs)[kObs]) {
  constexpr int HQ = ResidentSlice<H, LPA>::HQ;
  const int act[3] = {TANH ? EVO_ACT_TANH : act_rt[0], TANH ? EVO_ACT_TANH : act_rt[1],
                      TANH ? EVO_ACT_TANH : act_rt[2]};
  float h1[HQ], part[HQ];
#pragma unroll
  for (int u = 0; u < HQ; ++u) {
    h1[u] = s.b1[u];
#pragma unroll
    for (int i = 0; i < kObs; ++i) h1[u] = fmaf(obs[i], s.w1[i][u], h1[u]);
    h1[u] = activate(h1[u], act[0]);
    part[u] = s.b2[u];
  }
  if constexpr (LPA == 16) {
    row_layer<H, 0>(s, h1, part);
  } else {
#pragma unroll
    for (int i = 0; i < H; ++i) part[0] = fmaf(lane_value(h1[0], i), s.w2[i][0], part[0]);
  }
#pragma unroll
  for (int u = 0; u < HQ; ++u) part[u] = activate(part[u], act[1]);
  float o[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float x = 0.f;
    if constexpr (LPA == 16) {  // a chain starts in the even lane of a pair and ends in the odd one
#pragma unroll
      for (int u = 0; u < HQ; ++u) x = fmaf(part[u], s.w3[u][j], x);
      x = lane_move<0xA0>(x);  // quad_perm 0,0,2,2
#pragma unroll
      for (int u = 0; u < HQ; ++u) x = fmaf(part[u], s.w3[u][j], x);
      x = lane_move<0xF5>(x);  // quad_perm 1,1,3,3
      x += partner<1>(x);
      x += partner<2>(x);
      x += partner<3>(x);
    } else {  // a chain of eight lanes; its last lane holds the value
      static_assert(LPA == 16 || H == 64, "a wave per agent: one neuron per lane, eight per chain");
      x = part[0] * s.w3[0][j];
      const float first = x;
#pragma unroll
      for (int k = 1; k < 8; ++k) {
        const float before = lane_move<0x111>(x);  // row_shr:1
        x = (lane & 7) == 0 ? first : fmaf(part[0], s.w3[0][j], before);
      }
      float p[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) p[k] = lane_value(x, 8 * k + 7);
      x = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    }
    o[j] = activate(x + s.b3[j], act[2]);
  }
  return make_float2(o[0], o[1]);
}

// A wave-uniform value in a vector register (the scan's multiply-adds run at half rate on a scalar operand).
__device__ __forceinline__ float in_vector(float uniform) {
  float v;
  asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(uniform));
  return v;
}

// 100 MHz, the same on the whole chip.
__device__ __forceinline__ unsigned long long now_ticks() { return wall_clock64(); }

// What a wait does every 64 looks: has the world been given up, or has this wait taken too long?
__device__ __forceinline__ bool give_up(uint32_t* flag, unsigned long long wait_ticks, unsigned long long& since) {
  const unsigned long long now = now_ticks();
  if (since == 0) since = now;
  if (now - since >= wait_ticks) __hip_atomic_store(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
}
__device__ __forceinline__ unsigned long long peek(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void hand_over(unsigned long long* p, unsigned long long w) {
  __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kChunk = 32;     // slots of the item lists: two for each lane of a row of sixteen
constexpr int kMaxChunks = 9;  // 256 items in two lists of whole chunks

// Number of the lowest set bit; 0xFFFFFFFF of none.
__device__ __forceinline__ uint32_t first_bit(uint32_t x) { return static_cast<uint32_t>(__builtin_ffs(x)) - 1u; }
// Where in LDS.
__device__ __forceinline__ uint32_t lds_address(const uint32_t* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) uint32_t*)p));
}
// The nearest food and the nearest poison, as offsets; eight lanes per agent.  Smallest distance first, then the lowest
// index that has it.  Both lists (of `food` and `poison` chunks) go together; the shorter one's last chunk is judged again.
__device__ __forceinline__ float4 nearest_items(float2 p, const float2* list, int food, int poison, int q) {
  Nearest n[2] = {{__builtin_inff(), 0x7fffffff}, {__builtin_inff(), 0x7fffffff}};
#pragma unroll 1
  for (int c = 0; c < max(food, poison); ++c) {
    const int base[2] = {min(c, food - 1) * kChunk, (food + min(c, poison - 1)) * kChunk};
    float4 x[2], y[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      x[j] = *reinterpret_cast<const float4*>(list + base[j] + 2 * q);
      y[j] = *reinterpret_cast<const float4*>(list + base[j] + 16 + 2 * q);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      nearest_offer<false>(n[j], p, x[j].x, x[j].y, base[j] + 2 * q, -1);
      nearest_offer<false>(n[j], p, x[j].z, x[j].w, base[j] + 2 * q + 1, -1);
      nearest_offer<false>(n[j], p, y[j].x, y[j].y, base[j] + 16 + 2 * q, -1);
      nearest_offer<false>(n[j], p, y[j].z, y[j].w, base[j] + 16 + 2 * q + 1, -1);
    }
  }
  uint32_t at[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t d = __float_as_uint(n[j].d2), m = agent_min(d);
    at[j] = agent_min(d == m ? static_cast<uint32_t>(n[j].idx) : 0x7fffffffu);
    at[j] = min(at[j], static_cast<uint32_t>((food + poison) * kChunk - 1));  // (every list has an item at a finite place)
  }
  const float2 f = list[at[0]], g = list[at[1]];
  return make_float4(f.x - p.x, f.y - p.y, g.x - p.x, g.y - p.y);
}

// CHECK: a build of its own in which waits can be made to fail at a stated step (the two comparisons per step cost the
// kernel proper 3 % in scalar registers that it has to put aside).
template <int H, bool TANH, bool CHECK>
__global__ __launch_bounds__(resident_threads(H)) void world_resident_kernel(const ResidentArgs a) {
  constexpr int LPA = resident_lanes(H), APW = 64 / LPA, kAgents = resident_agents(H), kItemWaves = item_waves(H);
  extern __shared__ float4 lds4[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int place = blockIdx.x / a.groups, group = blockIdx.x - place * a.groups, world = a.world0 + place;
  const int n_food = a.c.n_food, n_items = a.c.n_items;
  const int food_pad = pad_to(n_food, kChunk), slots = food_pad + pad_to(n_items - n_food, kChunk);
  const int chunks = slots / kChunk;
  // candidates: lane l judges agents l G .. l G + G - 1, which start at an odd number of 16-byte words from each other,
  // so that sixteen lanes' 16-byte reads meet every bank once
  const int G = a.per_lane, S = (G >> 1) & 1 ? G : G + 2;
  const int region = 64 * S;
  const int lists = kItemWaves * slots;
  float4* s_near = lds4;                                             // [agents] offsets of the nearest food and poison
  float2* s_own = reinterpret_cast<float2*>(s_near + kAgents);       // [agents] positions of the workgroup's agents
  float2* s_pos = s_own + kAgents;                                   // the world's agents
  float2* s_item = s_pos + region;                                   // [item waves][slots] where the items are
  float2* s_next = s_item + lists;                                   // [item waves][slots] and where they go when eaten
  uint32_t* s_count = reinterpret_cast<uint32_t*>(s_next + lists);   // [item waves][slots] times eaten
  uint32_t* s_all = s_count + lists;                                 // [item waves][chunks] touched by anyone
  uint32_t* s_hit = s_all + kItemWaves * kMaxChunks;                 // [chunks] touched by this workgroup
  uint32_t* s_done = s_hit + kMaxChunks;                             // main waves whose touches are in s_hit
  uint32_t* s_stop = s_done + 1;
  const uint32_t gen = a.gen_dev ? *a.gen_dev : a.gen;
  const float inf = __builtin_inff();
  auto place_agent = [&](int j) {
    const u32x4 w = philox4x32_10(static_cast<uint32_t>(j), static_cast<uint32_t>(world), gen, kTagAgent, a.key0, a.key1);
    return make_float2(unit_open(w.x), unit_open(w.y));
  };
  // everybody's start; the slots of no agent lie infinitely far away
#pragma unroll 1
  for (int i = tid; i < region; i += resident_threads(H)) {
    const int l = i / S, k = i - l * S, j = l * G + k;
    s_pos[i] = k < G && j < a.pop ? place_agent(j) : make_float2(inf, inf);
  }
  if (tid < kAgents) s_own[tid] = place_agent(min(group * kAgents + tid, a.pop - 1));
  if (tid < kItemWaves * kMaxChunks + kMaxChunks + 2) s_all[tid] = 0u;  // s_all, s_hit, s_done and s_stop
  __syncthreads();

  auto item_of = [&](int slot) {  // item index of a slot, or -1
    const bool is_food = slot < food_pad;
    const int i = is_food ? slot : n_food + slot - food_pad;
    return i < (is_food ? n_food : n_items) ? i : -1;
  };
  auto place_item = [&](int i, uint32_t c) {
    const u32x4 w = philox4x32_10(256u * c + static_cast<uint32_t>(i), static_cast<uint32_t>(world), gen, kTagItem,
                                  a.key0, a.key1);
    return make_float2(unit_open(w.x), unit_open(w.y));
  };
#pragma unroll 1
  for (int j = tid; j < lists; j += resident_threads(H)) {
    const int i = item_of(j % slots);
    s_item[j] = i >= 0 ? place_item(i, 0u) : make_float2(inf, inf);
    s_next[j] = i >= 0 ? place_item(i, 1u) : make_float2(inf, inf);
    s_count[j] = 0u;
  }
  __syncthreads();
  const int words = a.groups * chunks;  // a world's touches of a step
  unsigned long long* hand = a.hand + static_cast<size_t>(place) * words;
  const size_t half = static_cast<size_t>(a.per_launch) * words;

  if (wave >= kMainWaves) {  // ---- item waves; the two barriers of a step are those of the main waves below
    const int iw = wave - kMainWaves, q = lane & (kLanesPerAgent - 1);
    const int mine = iw * kAgentsPerBlock + lane / kLanesPerAgent;
    float2* food = s_item + iw * slots;
    float2* next = s_next + iw * slots;
    uint32_t* count = s_count + iw * slots;
    uint32_t* all = s_all + iw * kMaxChunks;
    auto settle = [] {  // LDS keeps a wave's order; this keeps the compiler's
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto touched = [&](int slot) {  // slot 2 q of a chunk in bit q of its word, slot 2 q + 1 in bit 16 + q
      return ((all[slot / kChunk] >> ((slot & 1) * 16 + ((slot & (kChunk - 1)) >> 1))) & 1u) != 0u;
    };
    const int fail_items = CHECK && group < a.fail_groups ? a.fail_items : 0x7fffffff;
    // what anybody touched moves on (false: given up)
    auto collect = [&](int step) -> bool {
      const unsigned long long* in = hand + (step & 1) * half;
      const uint32_t tag = CHECK && step >= fail_items ? ~0u : a.tag0 + static_cast<uint32_t>(step);  // (~0: nobody's)
      bool stop = false;
#pragma unroll 1
      for (int i = lane; i < words; i += 128) {  // two words at a time
        const int j = i + 64 < words ? i + 64 : i;
        unsigned long long w0, w1, since = 0;
        for (uint32_t looks = 0;;) {
          w0 = peek(in + i), w1 = peek(in + j);
          if (static_cast<uint32_t>(w0 >> 32) == tag && static_cast<uint32_t>(w1 >> 32) == tag) break;
          if ((looks++ & 63) == 63) {
            if (give_up(a.flag + world, a.wait_ticks, since)) {
              stop = true;
              break;
            }
          }
        }
        if (static_cast<uint32_t>(w0)) atomicOr(all + i % chunks, static_cast<uint32_t>(w0));
        if (j != i && static_cast<uint32_t>(w1)) atomicOr(all + j % chunks, static_cast<uint32_t>(w1));
      }
      settle();
#pragma unroll 1
      for (int slot = lane; slot < slots; slot += 64)  // (slots of no item are never touched)
        if (touched(slot)) food[slot] = next[slot];
      settle();
      return __builtin_amdgcn_ballot_w64(stop) == 0;
    };
    // off the step's critical path: where the moved ones would go next
    auto refill = [&] {
#pragma unroll 1
      for (int slot = lane; slot < slots; slot += 64)
        if (touched(slot)) {
          const uint32_t n = ++count[slot];
          next[slot] = place_item(item_of(slot), n + 1u);
        }
      settle();
      if (lane < chunks) all[lane] = 0u;
      settle();
    };
    bool go_on = true;
#pragma unroll 1
    for (int t = 0; t < a.steps; ++t) {
      if (t > 1) refill();
      if (!go_on) *s_stop = 1u;
      __syncthreads();
      if (*s_stop) return;
      if (t > 0) go_on = collect(t);
      const float2 p = s_own[mine];
      const float4 both = nearest_items(p, food, food_pad / kChunk, chunks - food_pad / kChunk, q);
      if (q == 0) s_near[mine] = both;
      __syncthreads();
    }
    if (a.counts_out && group == 0 && iw == 0) {
      if (a.steps > 1) refill();
      collect(a.steps);
      refill();
      for (int slot = lane; slot < slots; slot += 64) {
        const int i = item_of(slot);
        if (i >= 0) a.counts_out[static_cast<size_t>(world) * n_items + i] = count[slot];
      }
    }
    return;
  }

  // ---- main waves
  const int row = lane >> 4, q = lane & 15;
  const int slot0 = wave * APW + (LPA == 16 ? row : 0);  // the agent's place in the workgroup
  const bool live = group * kAgents + slot0 < a.pop;
  const int agent = min(group * kAgents + slot0, a.pop - 1);  // lanes without an agent follow the last one and hand nothing over
  const bool speaks = live && (LPA == 16 ? q : lane) == 0;
  const size_t me = static_cast<size_t>(world) * a.pop + agent;
  ResidentSlice<H, LPA> weights;
  resident_load<H, LPA>(a.params + static_cast<size_t>(agent) * a.P, LPA == 16 ? q : lane, weights);
  auto pos_slot = [&](int j) { return j + static_cast<int>(__umulhi(j, a.lane_magic)) * (S - G); };  // agent j's place
  const int own_lane = agent / G;  // whose candidates the agent itself is among
  int own_lanes[APW];              // the same of all the wave's agents
#pragma unroll
  for (int i = 0; i < APW; ++i) own_lanes[i] = __builtin_amdgcn_readlane(own_lane, 16 * i);
  float2 p = s_own[slot0], v = make_float2(0.f, 0.f);
  int reward = 0;
  constexpr int kStride = LPA == 16 ? 2 : 4;  // chunks judged for touches at a time
  const uint64_t live_lanes = __builtin_amdgcn_ballot_w64(live);
  const int fail_main = CHECK && group < a.fail_groups ? a.fail_main : 0x7fffffff;

#pragma unroll 1
  for (int t = 0; t < a.steps; ++t) {
    if (t > 0) {
      const unsigned long long* in = (t & 1 ? a.odd : a.even) + static_cast<size_t>(world) * a.pop;
      const uint32_t want = CHECK && t >= fail_main ? 4u : static_cast<uint32_t>(t) & 3u;  // (4: nobody's)
      bool stop = false;
#pragma unroll 1
      for (int j = tid; j < a.pop; j += 2 * 64 * kMainWaves) {  // two words at a time
        const int k = j + 64 * kMainWaves;
        const bool two = k < a.pop;
        const int k1 = two ? k : j;
        unsigned long long w0, w1, since = 0;
        for (uint32_t looks = 0;;) {
          w0 = peek(in + j), w1 = peek(in + k1);
          if ((static_cast<uint32_t>(w0) >> 30) == want && (static_cast<uint32_t>(w1) >> 30) == want) break;
          if ((looks++ & 63) == 63) {
            if (give_up(a.flag + world, a.wait_ticks, since)) {
              stop = true;
              break;
            }
          }
        }
        s_pos[pos_slot(j)] = make_float2(__uint_as_float(static_cast<uint32_t>(w0) & 0x3FFFFFFFu),
                                         __uint_as_float(static_cast<uint32_t>(w0 >> 32)));
        if (two)
          s_pos[pos_slot(k)] = make_float2(__uint_as_float(static_cast<uint32_t>(w1) & 0x3FFFFFFFu),
                                           __uint_as_float(static_cast<uint32_t>(w1 >> 32)));
      }
      if (stop) *s_stop = 1u;
    }
    __syncthreads();     // the positions of step t
    if (*s_stop) return;  // set before this barrier or after the last one only: all leave together

    // the nearest other agent of the wave's agents
    float px[APW], py[APW];
    uint32_t best[APW];
#pragma unroll
    for (int i = 0; i < APW; ++i) {
      px[i] = in_vector(lane_value(p.x, 16 * i)), py[i] = in_vector(lane_value(p.y, 16 * i));
      best[i] = kFar;
    }
    const float4* cand = reinterpret_cast<const float4*>(s_pos + lane * S);
    auto judge = [&](const float4& c) {
#pragma unroll
      for (int i = 0; i < APW; ++i) {
        const uint32_t d0 = __float_as_uint(dist2(c.x - px[i], c.y - py[i]));
        const uint32_t d1 = __float_as_uint(dist2(c.z - px[i], c.w - py[i]));
        best[i] = min(min(best[i], d0), d1);  // squares' sums order like their bits
      }
    };
    const int units = G >> 1;
    int u = 0;
#pragma unroll 1
    for (; u + 4 <= units; u += 4) {
      float4 c[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) c[n] = cand[u + n];
#pragma unroll
      for (int n = 0; n < 4; ++n) judge(c[n]);
    }
#pragma unroll 1
    for (; u < units; ++u) judge(cand[u]);
    // every agent met itself there: the lane that holds it drops out for it, and the agent's row judges that lane's
    // other candidates in its place
    uint32_t beside = kFar;
#pragma unroll 1
    for (int base = 0; base < G; base += 16) {
      const int k = base + q;
      const float2 c = s_pos[own_lane * S + min(k, G - 1)];
      const uint32_t d = __float_as_uint(dist2(c.x - p.x, c.y - p.y));
      beside = min(beside, ((k < G) & (own_lane * G + k != agent)) ? d : kFar);
    }
#pragma unroll
    for (int i = 0; i < APW; ++i) best[i] = lane == own_lanes[i] ? kFar : best[i];
    // minimum over the lanes, agent i's in row i (a wave per agent: in every lane)
    uint32_t m;
    if constexpr (APW == 4) {
      const auto x = __builtin_amdgcn_permlane32_swap(best[0], best[2], false, false);
      const auto y = __builtin_amdgcn_permlane32_swap(best[1], best[3], false, false);
      const auto z = __builtin_amdgcn_permlane16_swap(min(x[0], x[1]), min(y[0], y[1]), false, false);
      m = min(z[0], z[1]);
    } else {
      const auto x = __builtin_amdgcn_permlane32_swap(best[0], best[0], false, false);
      m = min(x[0], x[1]);
      const auto z = __builtin_amdgcn_permlane16_swap(m, m, false, false);
      m = min(z[0], z[1]);
    }
    m = min(m, beside);
    m = min(m, static_cast<uint32_t>(partner_bits<0>(m)));
    m = min(m, static_cast<uint32_t>(partner_bits<1>(m)));
    m = min(m, static_cast<uint32_t>(partner_bits<2>(m)));
    m = min(m, static_cast<uint32_t>(partner_bits<3>(m)));
    // lowest lane that holds it, then the lowest of that lane's candidates at this distance: the lowest index
    uint32_t held_lo = 0, held_hi = 0;
#pragma unroll
    for (int i = 0; i < APW; ++i) {
      const uint64_t held = __builtin_amdgcn_ballot_w64(best[i] == static_cast<uint32_t>(__builtin_amdgcn_readlane(m, 16 * i)));
      held_lo = APW == 1 || row == i ? static_cast<uint32_t>(held) : held_lo;
      held_hi = APW == 1 || row == i ? static_cast<uint32_t>(held >> 32) : held_hi;
    }
    const uint64_t near_by = __builtin_amdgcn_ballot_w64(beside == m);
    uint32_t holder = min(first_bit(held_lo), first_bit(held_hi) | 32u);
    holder = (static_cast<uint32_t>(near_by >> (16 * row)) & 0xFFFFu) != 0u ? min(holder, static_cast<uint32_t>(own_lane)) : holder;
    const float2* theirs = s_pos + holder * S;
    const int self = agent - static_cast<int>(holder) * G;  // the agent's own place among them, if any
    auto find = [&](int base) {  // (bit number of nothing: -1)
      const int k = base + q;
      const float2 c = theirs[min(k, G - 1)];
      const bool same = (k < G) & (k != self) & (__float_as_uint(dist2(c.x - p.x, c.y - p.y)) == m);
      return first_bit(static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(same) >> (16 * row)) & 0xFFFFu);
    };
    uint32_t slot = find(0);
#pragma unroll 1
    for (int base = 16; base < G; base += 16) {
      const uint32_t later = find(base);
      slot = static_cast<int>(slot) < 0 && static_cast<int>(later) >= 0 ? base + later : slot;
    }
    const float2 near = theirs[min(slot, static_cast<uint32_t>(G - 1))];
    __syncthreads();  // the nearest items

    const float4 item = s_near[slot0];
    // the first chunks that the agent may touch, on their way during the policy
    float4 ahead[LPA == 16 ? 2 : 1];
#pragma unroll
    for (int c = 0; c < (LPA == 16 ? 2 : 1); ++c)
      ahead[c] = *reinterpret_cast<const float4*>(s_item + min(LPA == 16 ? c : row, chunks - 1) * kChunk + 2 * q);
    const float obs[kObs] = {v.x, v.y, item.x, item.y, item.z, item.w, near.x - p.x, near.y - p.y};
    const float2 action = resident_forward<H, LPA, TANH>(weights, a.act, lane, obs);
    move_axis(a.c, action.x, p.x, v.x);
    move_axis(a.c, action.y, p.y, v.y);
    if ((LPA == 16 ? q : lane) == 0) s_own[slot0] = p;
    if (speaks && t + 1 < a.steps)
      hand_over((t & 1 ? a.even : a.odd) + me,
                (static_cast<unsigned long long>(__float_as_uint(p.y)) << 32) | __float_as_uint(p.x) |
                    (static_cast<uint32_t>(t + 1) & 3u) << 30);
    // what the moved agents touch: the main waves' words meet in LDS, and the last of them tells the world
    auto judge_items = [&](const float4& it, int chunk, uint64_t& even, uint64_t& odd) {
      const float limit = chunk < chunks ? a.c.r2 : -1.f;  // (a chunk past the last one: nothing)
      const bool hit0 = dist2(it.x - p.x, it.y - p.y) <= limit, hit1 = dist2(it.z - p.x, it.w - p.y) <= limit;
      const int found = static_cast<int>(hit0) + static_cast<int>(hit1);
      reward += chunk * kChunk < food_pad ? found : -found;
      even = __builtin_amdgcn_ballot_w64(hit0) & live_lanes, odd = __builtin_amdgcn_ballot_w64(hit1) & live_lanes;
    };
#pragma unroll 1
    for (int c = 0; c < chunks; c += kStride) {
      uint32_t word;
      if constexpr (LPA == 16) {  // two chunks, each judged by all rows: their words to lanes 0 and 1
        uint64_t even[2], odd[2];
        uint32_t w[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (c > 0) ahead[j] = *reinterpret_cast<const float4*>(s_item + min(c + j, chunks - 1) * kChunk + 2 * q);
          judge_items(ahead[j], c + j, even[j], odd[j]);
          uint32_t e = static_cast<uint32_t>(even[j] | even[j] >> 32), o = static_cast<uint32_t>(odd[j] | odd[j] >> 32);
          e |= e >> 16, o |= o >> 16;
          w[j] = (e & 0xFFFFu) | o << 16;
        }
        word = lane == 0 ? w[0] : w[1];
      } else {  // four chunks, a row each: their words to lanes 0 .. 3
        uint64_t even, odd;
        if (c > 0) ahead[0] = *reinterpret_cast<const float4*>(s_item + min(c + row, chunks - 1) * kChunk + 2 * q);
        judge_items(ahead[0], c + row, even, odd);
        word = (static_cast<uint32_t>(even >> (16 * (lane & 3))) & 0xFFFFu) | static_cast<uint32_t>(odd >> (16 * (lane & 3))) << 16;
      }
      if (lane < kStride && c + lane < chunks) atomicOr(s_hit + c + lane, word);
    }
    // A wave's LDS operations are carried out in order: who counts last finds every wave's touches in what it reads next.
    // (A fence here would also wait for the position's store, 800 cycles.)
    if (lane < kMaxChunks) {
      uint32_t before, bits;
      asm volatile("ds_add_rtn_u32 %0, %2, %3\n\tds_read_b32 %1, %4\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(before), "=&v"(bits)
                   : "v"(lds_address(s_done)), "v"(lane == 0 ? 1u : 0u), "v"(lds_address(s_hit + lane))
                   : "memory");
      if (__builtin_amdgcn_readfirstlane(before) == kMainWaves - 1) {
        if (lane < chunks) {
          const uint32_t tag = a.tag0 + static_cast<uint32_t>(t) + 1u;
          hand_over(hand + ((t + 1) & 1) * half + group * chunks + lane, (static_cast<unsigned long long>(tag) << 32) | bits);
          s_hit[lane] = 0u;
        }
        if (lane == 0) *s_done = 0u;
      }
    }
  }
  reward = agent_sum<16>(reward);
  if constexpr (LPA == 64) {
    reward += __shfl_xor(reward, 16);
    reward += __shfl_xor(reward, 32);
  }
  if (speaks) {
    a.reward[me] = reward;
    a.pos_out[me] = p;
    a.vel_out[me] = v;
  }
}

// Plays the worlds again that world_resident_kernel gave up, with world_step_block (a world of its four that was not given
// up gets the same result once more).  Nothing to do otherwise.
// The chip may be held by other work here, so nothing may depend on how many of the workgroups run.  The crew of four
// worlds takes tickets from a counter: phase 0 sets the worlds up, phase t + 1 is step t, the last one the item book,
// each a ticket per workgroup of the step's grid.  A ticket's holder waits until every ticket of the phases before is
// done.  Those are held by workgroups that run (a ticket is taken by running), and the holder of the lowest one that is
// not done waits for nobody: every wait ends, with one workgroup on the chip as well as with all.
// 1024 agents x 8 worlds x 500 steps, H = 32, every wait given up: 17 ms (by one workgroup per four
// worlds 455 ms, with the fences in every wave 40 ms); 1024 x 64 x 50 11 ms, 4800 x 1 x 20 2.5 ms.
struct RerunArgs {
  const uint32_t* flag;  // [per_launch]
  int per_launch;        // worlds of one launch
  uint32_t* tickets;     // per four worlds: taken, done (zero at the start)
  int crew;              // workgroups of four worlds
  int steps;
  float2* pos[2];
  uint32_t* book;        // counts[2] and hits[3]: 5 x [worlds][n_items]
  uint32_t* counts_out;  // [worlds][n_items] or null
};

template <int H, bool TANH>
__global__ __launch_bounds__(kStepThreads) void world_rerun_kernel(StepArgs a, RerunArgs r) {
  extern __shared__ float4 lds4[];
  const int tid = threadIdx.x, four = blockIdx.x / r.crew;
  const int world0 = four * kWorldsPerBlock, world1 = min(world0 + kWorldsPerBlock, a.worlds);
  uint32_t any = 0;
  for (int w = world0; w < world1; ++w) any |= r.flag[w % r.per_launch];
  if (!any) return;
  if (a.gen_dev) a.gen = *a.gen_dev;
  const size_t nb = static_cast<size_t>(a.worlds) * a.c.n_items;
  const uint32_t blocks = (a.pop + kAgentsPerBlock - 1) / kAgentsPerBlock;
  const uint32_t total = blocks * (r.steps + (r.counts_out ? 2u : 1u));  // (below 2^30: 2^20 steps of 613 workgroups)
  uint32_t* taken = r.tickets + 2 * four;
  uint32_t* done = taken + 1;
  uint32_t* s_ticket = reinterpret_cast<uint32_t*>(lds4);  // (in the staging area, before a step uses it)
  // One thread's part of a round stands in one place: with its count at the round's end and its ticket at the next one's
  // start, the compiler let the other 63 lanes of its wave go round without it, past the barriers.
#pragma unroll 1
  for (uint32_t finished = 0;; finished = 1u) {
    if (tid == 0) {
      __threadfence();  // (release) what every wave wrote, which has arrived at the die's cache
      if (finished) atomicAdd(done, 1u);
      const uint32_t mine = atomicAdd(taken, 1u);
      const uint32_t before = mine / blocks * blocks;
      while (mine < total && __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < before)
        __builtin_amdgcn_s_sleep(4);
      __threadfence();  // (acquire) what the phases before wrote, on whatever die; this compute unit's cache is every wave's
      *s_ticket = mine;
    }
    __syncthreads();
    const uint32_t ticket = __builtin_amdgcn_readfirstlane(*s_ticket);
    __syncthreads();  // the staging area is free
    if (ticket >= total) return;
    const int phase = static_cast<int>(ticket / blocks), block = static_cast<int>(ticket % blocks);
    const int first = block * kStepThreads + tid, stride = static_cast<int>(blocks) * kStepThreads;
    if (phase == 0) {
      for (int i = world0 * a.pop + first; i < world1 * a.pop; i += stride) {
        const u32x4 w = philox4x32_10(static_cast<uint32_t>(i % a.pop), static_cast<uint32_t>(i / a.pop), a.gen, kTagAgent, a.key0, a.key1);
        r.pos[0][i] = make_float2(unit_open(w.x), unit_open(w.y));
        a.vel_out[i] = make_float2(0.f, 0.f);
        a.reward[i] = 0;
      }
      for (int k = 0; k < 5; ++k)
        for (int i = world0 * a.c.n_items + first; i < world1 * a.c.n_items; i += stride) r.book[k * nb + i] = 0u;
    } else if (phase <= r.steps) {
      const int t = phase - 1;
      a.pos_in = r.pos[t & 1], a.pos_out = r.pos[(t + 1) & 1];
      a.counts_in = r.book + (t & 1) * nb, a.counts_out = r.book + ((t + 1) & 1) * nb;
      a.hits_prev = t > 0 ? r.book + (2 + (t + 2) % 3) * nb : nullptr;
      a.hits_cur = r.book + (2 + t % 3) * nb, a.hits_clear = r.book + (2 + (t + 1) % 3) * nb;
      world_step_block<H, TANH>(a, block, four, lds4);
    } else {
      for (int i = world0 * a.c.n_items + first; i < world1 * a.c.n_items; i += stride)
        r.counts_out[i] = r.book[(r.steps & 1) * nb + i] + r.book[(2 + (r.steps - 1) % 3) * nb + i];
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
  }
}

// ---- single-agent form: every member alone in its own copy of each world ---------------------------------
// Nothing couples the members, so the whole episode runs in one launch (the fused roll-out of the control
// tasks): wave = 64 / LPA members x LPA lanes in one world (sixteen lanes where the hidden width allows it:
// twice the waves and half the length of a member's dependent chain), the policy's weights in registers for
// all steps, each member's item lists and item book in LDS.  A touched item is moved at once by the lane
// that found it (every slot is judged by exactly one lane per step, after the step's sensing), which is
// "from the next step on".  All members start at agent 0's place among the same items.
struct SoloArgs {
  const float* params;  // [pop][P]
  int P, pop, worlds, steps;
  int act[3];
  WorldConst c;
  uint32_t key0, key1, gen;
  const uint32_t* gen_dev;
  int32_t* reward;       // [worlds][pop]: the episode's summed reward
  float2* pos_out;       // [worlds][pop] or null: state after the last step
  float2* vel_out;       // [worlds][pop] or null
  uint32_t* counts_out;  // [worlds][pop][n_items] or null: times each item was eaten
};

template <int H, int LPA, bool TANH>
__global__ __launch_bounds__(64 * kWorldsPerBlock) void world_solo_kernel(SoloArgs a) {
  constexpr int kMembers = 64 / LPA;  // members per wave
  extern __shared__ float4 lds4[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = lane & (LPA - 1), la = lane / LPA;
  const int agent = blockIdx.x * kMembers + la;
  const int world = blockIdx.y * kWorldsPerBlock + wave;
  const bool live = world < a.worlds && agent < a.pop;
  const int n_food = a.c.n_food, n_items = a.c.n_items;
  const int food_pad = pad_to(n_food, 2 * LPA), poison_pad = pad_to(n_items - n_food, 2 * LPA);
  const int slots = food_pad + poison_pad;
  // per wave: [members][slots] positions, then [members][slots] counts
  float2* s_item = reinterpret_cast<float2*>(lds4) + wave * kMembers * slots;
  uint32_t* s_count = reinterpret_cast<uint32_t*>(reinterpret_cast<float2*>(lds4) + kWorldsPerBlock * kMembers * slots) +
                      wave * kMembers * slots;
  if (a.gen_dev) a.gen = *a.gen_dev;
  const float inf = __builtin_inff();
  auto item_of = [&](int slot) {  // item index of a slot of the two padded lists, or -1
    const bool is_food = slot < food_pad;
    const int i = is_food ? slot : n_food + slot - food_pad;
    return i < (is_food ? n_food : n_items) ? i : -1;
  };
  auto place = [&](int i, uint32_t cnt) {
    const u32x4 w = philox4x32_10(256u * cnt + static_cast<uint32_t>(i), static_cast<uint32_t>(world), a.gen, kTagItem,
                                  a.key0, a.key1);
    return make_float2(unit_open(w.x), unit_open(w.y));
  };

  PolicySlice<H, LPA> weights;
  if (live) policy_load<H, LPA>(a.params + static_cast<size_t>(agent) * a.P, q, weights);
  if (world < a.worlds) {  // the same fresh items for every member of the wave
    for (int slot = lane; slot < slots; slot += 64) {
      const int i = item_of(slot);
      const float2 where = i >= 0 ? place(i, 0u) : make_float2(inf, inf);
      for (int m = 0; m < kMembers; ++m) s_item[m * slots + slot] = where, s_count[m * slots + slot] = 0u;
    }
  }
  __syncthreads();
  if (!live) return;  // no barrier below this line; the lanes of a member stay together

  float2* my_food = s_item + la * slots;
  float2* my_poison = my_food + food_pad;
  uint32_t* my_count = s_count + la * slots;
  float2 p, v = make_float2(0.f, 0.f);
  {
    const u32x4 w = philox4x32_10(0u, static_cast<uint32_t>(world), a.gen, kTagAgent, a.key0, a.key1);
    p = make_float2(unit_open(w.x), unit_open(w.y));
  }
  int reward = 0;
#pragma unroll 1
  for (int step = 0; step < a.steps; ++step) {
    Nearest food{inf, 0x7fffffff}, poison{inf, 0x7fffffff};
    for (int base = 0; base < food_pad; base += 2 * LPA) nearest_scan16(food, p, my_food, base, q);
    for (int base = 0; base < poison_pad; base += 2 * LPA) nearest_scan16(poison, p, my_poison, base, q);
    const float2 f = nearest_finish<LPA>(food, p, my_food, food_pad);
    const float2 g = nearest_finish<LPA>(poison, p, my_poison, poison_pad);
    const float obs[kObs] = {v.x, v.y, f.x, f.y, g.x, g.y, 0.f, 0.f};  // nobody else is there
    const float2 action = policy_forward<H, LPA, TANH>(weights, a.act, lane, obs);
    move_axis(a.c, action.x, p.x, v.x);
    move_axis(a.c, action.y, p.y, v.y);
    // touches: the lane that judges a slot also moves the item it finds eaten
    for (int base = 0; base < slots; base += 2 * LPA) {
      const float4 it = *reinterpret_cast<const float4*>(my_food + base + 2 * q);
      const bool hit0 = dist2(it.x - p.x, it.y - p.y) <= a.c.r2, hit1 = dist2(it.z - p.x, it.w - p.y) <= a.c.r2;
      if (hit0 || hit1) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if (k == 0 ? hit0 : hit1) {
            const int slot = base + 2 * q + k, i = item_of(slot);
            reward += slot < food_pad ? 1 : -1;
            const uint32_t cnt = my_count[slot] + 1u;
            my_count[slot] = cnt;
            my_food[slot] = place(i, cnt);
          }
        }
      }
    }
    // the next step's sensing reads what this step's touches wrote (same wave: LDS keeps program order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  reward = agent_sum<LPA>(reward);
  const size_t me = static_cast<size_t>(world) * a.pop + agent;
  if (q == 0) {
    a.reward[me] = reward;
    if (a.pos_out) a.pos_out[me] = p;
    if (a.vel_out) a.vel_out[me] = v;
  }
  if (a.counts_out)
    for (int slot = q; slot < slots; slot += LPA) {
      const int i = item_of(slot);
      if (i >= 0) a.counts_out[me * n_items + i] = my_count[slot];
    }
}

struct ResetArgs {
  int pop, worlds, n_items;
  uint32_t key0, key1, gen;
  const uint32_t* gen_dev;
  float2* pos;       // [worlds][pop]
  float2* vel;       // [worlds][pop]
  int32_t* reward;   // [worlds][pop]
  uint32_t* book;    // counts[2] and hits[3]: 5 x [worlds][n_items], all zero at the start
  // of the launch with waits, or null: positions of odd steps (a step number no reader waits for first), touches and flags
  unsigned long long* odd;
  unsigned long long* hand;
  uint32_t* flag;  // and the second run's tickets behind them
  int n_hand, n_flag;
};

__global__ __launch_bounds__(256) void world_reset_kernel(ResetArgs a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (a.gen_dev) a.gen = *a.gen_dev;
  if (i < a.worlds * a.pop) {
    const uint32_t world = i / a.pop, agent = i % a.pop;
    const u32x4 w = philox4x32_10(agent, world, a.gen, kTagAgent, a.key0, a.key1);
    a.pos[i] = make_float2(unit_open(w.x), unit_open(w.y));
    a.vel[i] = make_float2(0.f, 0.f);
    a.reward[i] = 0;
    if (a.odd) a.odd[i] = ~0ull;
  }
  if (i < 5 * a.worlds * a.n_items) a.book[i] = 0u;
  if (i < a.n_hand) a.hand[i] = 0ull;
  if (i < a.n_flag) a.flag[i] = 0u;
}

// fitness[a] = mean over the worlds of the summed reward (an exact integer sum, one division).
__global__ __launch_bounds__(256) void world_finish_kernel(const int32_t* reward, int pop, int worlds, float* fitness) {
  const int agent = blockIdx.x * 256 + threadIdx.x;
  if (agent >= pop) return;
  int sum = 0;
  for (int r = 0; r < worlds; ++r) sum += reward[static_cast<size_t>(r) * pop + agent];
  fitness[agent] = static_cast<float>(sum) / static_cast<float>(worlds);
}

__global__ __launch_bounds__(256) void world_fill_kernel(uint32_t* dst, int n, uint32_t value) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = value;
}

// How each world was played (ForageForm::told), from the flags of the launch with waits.
__global__ __launch_bounds__(256) void world_told_kernel(const uint32_t* flag, int per_launch, int worlds, uint32_t* told) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < worlds) told[i] = 1u + flag[i % per_launch];
}

// counts_out = counts + hits (the book after the last step), for the state hook.
__global__ __launch_bounds__(256) void world_counts_kernel(const uint32_t* counts, const uint32_t* hits, int n,
                                                           uint32_t* out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] = counts[i] + hits[i];
}

struct Layout {
  size_t pos[2], vel, reward, book, hand, flag, bytes;  // byte offsets into the workspace, and what it takes
  bool room;                                            // hand and flag are there
};

static int item_chunks(int n_food, int n_items) {
  return (pad_to(n_food, kChunk) + pad_to(n_items - n_food, kChunk)) / kChunk;
}
// The most chunks that n_items take, whatever the split into food and poison.
static int most_chunks(int n_items) { return (n_items - 2) / kChunk + 2; }
// world_resident_kernel: workgroups of a world, and the words in which a world's touches of a step are handed over.
static int resident_groups(int pop, int H) { return (pop - 1) / resident_agents(H) + 1; }
static size_t touch_words(int pop, int H, int chunks) {
  return static_cast<size_t>(resident_groups(pop, H)) * chunks;
}
// Worlds of one launch of it.
static int resident_worlds(int pop, int worlds, int H) { return std::min(worlds, kMaxResident / resident_groups(pop, H)); }

// Is the episode in launches of per_launch worlds faster than a launch per step?  Each of them costs a fixed time of its
// own, and each of its steps about 3 us however few agents the workgroups have; a step's launch takes as many rounds of 256
// workgroups (8 agents x 4 worlds) as it has.  So a launch per step is better for a few steps, for many worlds of a few
// agents, and, as a workgroup of the one launch has only 8 agents there, for many workgroups at H = 64.
// Microseconds per step, a launch per step / this way, 24 + 24 items:
//   H = 32: 64 x 8 worlds 7.0 / 2.9, 1024 x 1 7.3 / 3.7, 1024 x 8 9.1 / 3.4, 4800 x 1 51 / 8.7, 64 x 512 24 / 12, 1024 x 64 60 / 29,
//           8 x 512 6.9 / 5.6, 8 x 1024 6.9 / 10.8, 8 x 4096 24 / 43, 16 x 4096 47 / 43, 32 x 4096 92 / 45
//   H = 16: 8 x 4096 13 / 40, 32 x 4096 46 / 40, 256 x 1024 89 / 89
//   H = 64: 64 x 8 13.4 / 3.4, 1024 x 2 11.6 / 4.0, 600 x 6 15.3 / 8.4, 1024 x 8 17.0 / 16.6, 8 x 4096 51 / 48, 512 x 64 55 / 65, 1024 x 64 120 / 135
// and whole calls: H = 32, 1024 x 8, 1 step 13.4 / 20.1, 2 steps 22.2 / 23.0, 4 steps 40 / 30; 8 x 1, 4 steps 23.3 / 25.6.
// Over 360 sizes of 2 to 4800 agents in 1 to 4096 worlds and 1 to 120 steps the estimates below choose the slower form by
// 2 % and more eleven times, by 6 % at most.
static bool one_launch_pays(int H, int pop, int worlds, int steps, int per_launch) {
  struct Cost {
    float launch, round, world, agent;  // us of a step's launch: fixed, and of a round: fixed, per world (of four), per agent of a world
    float step, step_agent;             // us of a step of the one launch: fixed, per agent
  };
  const Cost c = H == 16   ? Cost{3.7f, 0.73f, 0.48f, 0.0007f, 2.55f, 0.0009f}
                 : H == 32 ? Cost{1.6f, 2.7f, 0.75f, 0.0015f, 2.75f, 0.0008f}
                           : Cost{3.2f, 1.65f, 2.57f, 0.0025f, 3.05f, 0.0021f};
  const int64_t blocks = static_cast<int64_t>((pop + kAgentsPerBlock - 1) / kAgentsPerBlock) * ((worlds + kWorldsPerBlock - 1) / kWorldsPerBlock);
  // (H = 16: two workgroups fit a compute unit)
  const float rounds = H == 16 ? std::max(1.f, static_cast<float>(blocks) / 256.f) : static_cast<float>((blocks + 255) / 256);
  const float staged = static_cast<float>(pop) + 1.2f * static_cast<float>(std::max(0, pop - 1024));  // fewer workgroups fit
  const float per_step = c.launch + rounds * (c.round + c.world * static_cast<float>(std::min(worlds, kWorldsPerBlock)) + c.agent * staged);
  const float scanned = static_cast<float>(H == 64 ? std::min(pop, 512) + 0.35f * static_cast<float>(std::max(0, pop - 512)) : pop);
  const float launches = static_cast<float>((worlds + per_launch - 1) / per_launch);
  return static_cast<float>(steps) * (1.05f * per_step - launches * (c.step + c.step_agent * scanned)) > 8.f + 3.5f * launches;
}

// A flag per world of a launch (at most all worlds), and the second run's two tickets per four worlds.
static size_t flag_words(int worlds) {
  return static_cast<size_t>(worlds) + 2 * static_cast<size_t>((worlds + kWorldsPerBlock - 1) / kWorldsPerBlock);
}

static Layout carve(int pop, int worlds, int n_items) {
  const size_t agents = static_cast<size_t>(pop) * worlds;
  auto up = [](size_t n) { return (n + 255) & ~size_t(255); };
  Layout l;
  size_t o = 0;
  l.pos[0] = o, o += up(agents * sizeof(float2));
  l.pos[1] = o, o += up(agents * sizeof(float2));
  l.vel = o, o += up(agents * sizeof(float2));
  l.reward = o, o += up(agents * sizeof(int32_t));
  l.book = o, o += up(5 * static_cast<size_t>(worlds) * n_items * sizeof(uint32_t));
  // room for the launch with waits (at most 53 KB), unless it would be what makes the workspace too large for the
  // built-in scratch.  A workspace made for the largest problem has to serve the smaller ones, so no size may shrink as
  // pop, worlds or items grow: the room is for the most workgroups that a launch could have at any hidden width, not for
  // those of this call (whole worlds in kMaxResident workgroups: 1024 agents take more of them than 1026), and what
  // loses its room asks for the whole built-in scratch.
  const size_t groups = std::min(static_cast<size_t>(kMaxResident), static_cast<size_t>(resident_groups(pop, 64)) * worlds);
  l.hand = o, l.flag = o + up(2 * groups * most_chunks(n_items) * sizeof(unsigned long long));
  l.bytes = l.flag + up(flag_words(worlds) * sizeof(uint32_t));
  l.room = o > EVO_STATIC_SCRATCH_BYTES || l.bytes <= EVO_STATIC_SCRATCH_BYTES;
  if (!l.room) l.bytes = EVO_STATIC_SCRATCH_BYTES;
  return l;
}

constexpr size_t kMaxLdsBytes = 160 * 1024;  // per workgroup on this chip

static size_t step_lds_bytes(int pop, int n_food, int n_items) {
  return static_cast<size_t>(kWorldsPerBlock) *
         ((pad_to(pop, 64) + pad_to(n_food, 16) + pad_to(n_items - n_food, 16)) * sizeof(float2) +
          kExchangeWords * 64 * sizeof(float));
}

static int fill_const(const float* cp, WorldConst* c) {
  c->dt = cp[0], c->thrust = cp[1], c->drag = cp[2], c->vmax = cp[3];
  // the squared touch radius, rounded once; never infinite, or the empty slots of the item lists, which lie infinitely
  // far away, would count as touched
  c->r2 = std::fmin(cp[4] * cp[4], FLT_MAX);
  c->n_food = static_cast<int>(cp[5]);
  c->n_items = c->n_food + static_cast<int>(cp[6]);
  EVO_REQUIRE(cp[5] == static_cast<float>(c->n_food) && cp[6] == static_cast<float>(c->n_items - c->n_food),
              EVO_ERR_ARG, "forage: cp[5] (food items) and cp[6] (poison items) must be whole numbers");
  EVO_REQUIRE(c->n_food >= 1 && c->n_items > c->n_food && c->n_items <= 256, EVO_ERR_ARG,
              "forage: needs at least one food and one poison item and at most 256 items (got %d + %d)", c->n_food,
              c->n_items - c->n_food);
  EVO_REQUIRE(cp[0] > 0.f && cp[1] >= 0.f && cp[2] >= 0.f && cp[2] <= 1.f && cp[3] > 0.f && cp[4] > 0.f, EVO_ERR_ARG,
              "forage: needs dt > 0, thrust >= 0, drag in [0,1], vmax > 0, radius > 0");
  return EVO_OK;
}

template <int H, bool TANH>
static int launch_step_built(const StepArgs& a, hipStream_t s) {
  const dim3 grid((a.pop + kAgentsPerBlock - 1) / kAgentsPerBlock, (a.worlds + kWorldsPerBlock - 1) / kWorldsPerBlock);
  // more than 64 KB of dynamic LDS has to be asked for, once per kernel and device
  static std::atomic<bool> raised[64];  // zero-initialised; a second setter does the same harmless call
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e == hipSuccess && device >= 0 && device < 64 && !raised[device].load()) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&world_step_kernel<H, TANH>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kMaxLdsBytes));
    raised[device].store(e == hipSuccess);
  }
  EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "forage: raising the LDS limit of the step kernel failed: %s",
              hipGetErrorString(e));
  hipLaunchKernelGGL((world_step_kernel<H, TANH>), grid, dim3(kStepThreads),
                     step_lds_bytes(a.pop, a.c.n_food, a.c.n_items), s, a);
  return check_launch("world_step_kernel");
}
template <int H>
static int launch_step(const StepArgs& a, hipStream_t s) {
  const bool all_tanh = a.act[0] == EVO_ACT_TANH && a.act[1] == EVO_ACT_TANH && a.act[2] == EVO_ACT_TANH;
  return all_tanh ? launch_step_built<H, true>(a, s) : launch_step_built<H, false>(a, s);
}

static int launch_step_for(int H, const StepArgs& a, hipStream_t s) {
  switch (H) {
    case 16: return launch_step<16>(a, s);
    case 32: return launch_step<32>(a, s);
    case 64: return launch_step<64>(a, s);
  }
  return fail(EVO_ERR_UNSUPPORTED, "forage: the hidden width must be 16, 32 or 64");
}

int forage_supported(const MlpShape& sh, int pop, int worlds, const float* cp) {
  WorldConst c;
  int rc = fill_const(cp, &c);
  if (rc) return rc;
  EVO_REQUIRE(sh.n_layers == 3 && sh.dims[0] == kObs && sh.dims[3] == 2 && sh.dims[1] == sh.dims[2] &&
                  (sh.dims[1] == 16 || sh.dims[1] == 32 || sh.dims[1] == 64),
              EVO_ERR_UNSUPPORTED, "forage: the policy must be an MLP of dims {8, H, H, 2} with H = 16, 32 or 64");
  EVO_REQUIRE(pop >= 2, EVO_ERR_ARG, "forage: a world needs at least two agents (got pop = %d)", pop);
  EVO_REQUIRE(worlds >= 1 && worlds <= 4096, EVO_ERR_ARG, "forage: n_rollouts (worlds) must be in [1, 4096]");
  const size_t lds = step_lds_bytes(pop, c.n_food, c.n_items);
  EVO_REQUIRE(lds <= kMaxLdsBytes, EVO_ERR_UNSUPPORTED,
              "forage: too many agents per world: staging the positions of four worlds takes %zu bytes of LDS, %zu fit",
              lds, kMaxLdsBytes);
  return EVO_OK;
}

size_t forage_workspace_bytes(int pop, int worlds, const float* cp) {
  WorldConst c;
  if (fill_const(cp, &c) || pop < 1 || worlds < 1) return 0;
  return carve(pop, worlds, c.n_items).bytes;
}

// ---- the whole episode in one launch: host side ----
// A wait for workgroups that are not on the chip lasts about as long as playing the worlds again does (1 ms, and 20 us a
// step), so that at worst an episode takes twice that; the longest wait between workgroups that run is some 10 us.
constexpr uint64_t kWaitTicks = 100000, kWaitTicksPerStep = 2000;  // of 10 ns
// Launches with waits follow one another: two at a time could each hold a part of the chip and wait for the rest of it.
struct ResidentTurn {
  std::mutex m;
  hipEvent_t done = nullptr;
  bool used = false;
};

template <int H>
static int launch_resident_acts(const ResidentArgs& a, int worlds, size_t lds, hipStream_t s) {
  const bool all_tanh = a.act[0] == EVO_ACT_TANH && a.act[1] == EVO_ACT_TANH && a.act[2] == EVO_ACT_TANH;
  const dim3 grid(worlds * a.groups), threads(resident_threads(H));
  if (a.fail_groups > 0) hipLaunchKernelGGL((world_resident_kernel<H, false, true>), grid, threads, lds, s, a);
  else if (all_tanh) hipLaunchKernelGGL((world_resident_kernel<H, true, false>), grid, threads, lds, s, a);
  else hipLaunchKernelGGL((world_resident_kernel<H, false, false>), grid, threads, lds, s, a);
  return check_launch("world_resident_kernel");
}
static int launch_resident(int H, const ResidentArgs& a, int worlds, size_t lds, hipStream_t s) {
  switch (H) {
    case 16: return launch_resident_acts<16>(a, worlds, lds, s);
    case 32: return launch_resident_acts<32>(a, worlds, lds, s);
    default: return launch_resident_acts<64>(a, worlds, lds, s);
  }
}

template <int H>
static int launch_rerun_acts(const StepArgs& a, const RerunArgs& r, size_t lds, hipStream_t s) {
  const bool all_tanh = a.act[0] == EVO_ACT_TANH && a.act[1] == EVO_ACT_TANH && a.act[2] == EVO_ACT_TANH;
  const void* kernel = all_tanh ? reinterpret_cast<const void*>(&world_rerun_kernel<H, true>)
                                : reinterpret_cast<const void*>(&world_rerun_kernel<H, false>);
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kMaxLdsBytes));
    EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "forage: raising the LDS limit of the second run failed: %s", hipGetErrorString(e));
  }
  const dim3 grid((a.worlds + kWorldsPerBlock - 1) / kWorldsPerBlock * r.crew);
  if (all_tanh) hipLaunchKernelGGL((world_rerun_kernel<H, true>), grid, dim3(kStepThreads), lds, s, a, r);
  else hipLaunchKernelGGL((world_rerun_kernel<H, false>), grid, dim3(kStepThreads), lds, s, a, r);
  return check_launch("world_rerun_kernel");
}
static int launch_rerun(int H, const StepArgs& a, const RerunArgs& r, size_t lds, hipStream_t s) {
  switch (H) {
    case 16: return launch_rerun_acts<16>(a, r, lds, s);
    case 32: return launch_rerun_acts<32>(a, r, lds, s);
    default: return launch_rerun_acts<64>(a, r, lds, s);
  }
}

// May this call take the launch with waits?  Not into a recorded graph (its replays would not take their turn), and
// only with a compute unit per workgroup.  The turn of the device, or null.  A caller that may not create anything takes the
// launch without an event as long as there is none; another stream's launch that it meets then costs both a second run.
static ResidentTurn* resident_turn(int workgroups, bool create, hipStream_t s) {
  static ResidentTurn turns[64];
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &capture) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  int device = 0, cus = 0;
  if (capture != hipStreamCaptureStatusNone || hipGetDevice(&device) != hipSuccess || device < 0 || device >= 64 ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || workgroups > cus)
    return nullptr;
  ResidentTurn* turn = &turns[device];
  std::lock_guard<std::mutex> lock(turn->m);
  if (create && !turn->done && hipEventCreateWithFlags(&turn->done, hipEventDisableTiming) != hipSuccess) {
    turn->done = nullptr;
    (void)hipGetLastError();
    return nullptr;
  }
  return turn;
}

int launch_forage(const MlpShape& sh, const float* params, int pop, int worlds, int steps, const float* cp,
                  uint64_t seed, uint32_t gen, const uint32_t* gen_dev, void* work, float* fitness, float* pos_out,
                  float* vel_out, int32_t* reward_out, uint32_t* counts_out, const ForageForm& form, hipStream_t s) {
  WorldConst c;
  int rc = fill_const(cp, &c);
  if (rc) return rc;
  const Layout l = carve(pop, worlds, c.n_items);
  char* base = static_cast<char*>(work);
  float2* pos[2] = {reinterpret_cast<float2*>(base + l.pos[0]), reinterpret_cast<float2*>(base + l.pos[1])};
  float2* vel = reinterpret_cast<float2*>(base + l.vel);
  int32_t* reward = reinterpret_cast<int32_t*>(base + l.reward);
  uint32_t* book = reinterpret_cast<uint32_t*>(base + l.book);
  const size_t nb = static_cast<size_t>(worlds) * c.n_items;  // one page of the item book
  uint32_t* counts[2] = {book, book + nb};
  uint32_t* hits[3] = {book + 2 * nb, book + 3 * nb, book + 4 * nb};

  // The whole episode in one launch for as many worlds as the chip holds at once, one such launch after the other: where a
  // world has at most 256 workgroups (any that is supported; at H = 64 pop <= 2048), where that is faster, and with constants
  // that keep every position a number in [0, 1] (the tags of the handed-over positions need it).
  const int H = sh.dims[1], groups = resident_groups(pop, H), per_launch = resident_worlds(pop, worlds, H);
  const bool tame = std::isfinite(cp[0]) && std::isfinite(cp[1]) && std::isfinite(cp[2]) && std::isfinite(cp[3]);
  ResidentTurn* turn = nullptr;
  if (form.force != 2 && tame && l.room && per_launch > 0 &&
      (form.force == 1 || one_launch_pays(H, pop, worlds, steps, per_launch)) &&
      static_cast<uint64_t>((worlds + per_launch - 1) / per_launch) * (static_cast<uint64_t>(steps) + 1) < (1ull << 32))
    turn = resident_turn(groups * per_launch, form.create, s);

  ResetArgs ra;
  ra.pop = pop, ra.worlds = worlds, ra.n_items = c.n_items;
  ra.key0 = static_cast<uint32_t>(seed), ra.key1 = static_cast<uint32_t>(seed >> 32), ra.gen = gen, ra.gen_dev = gen_dev;
  ra.pos = pos[0], ra.vel = vel, ra.reward = reward, ra.book = book;
  ra.odd = nullptr, ra.hand = nullptr, ra.flag = nullptr, ra.n_hand = 0, ra.n_flag = 0;
  const int chunks = item_chunks(c.n_food, c.n_items);
  if (turn) {
    ra.odd = reinterpret_cast<unsigned long long*>(pos[1]);
    ra.hand = reinterpret_cast<unsigned long long*>(base + l.hand), ra.n_hand = static_cast<int>(2 * touch_words(pop, H, chunks) * per_launch);
    ra.flag = reinterpret_cast<uint32_t*>(base + l.flag), ra.n_flag = static_cast<int>(flag_words(worlds));
  }
  const int n_reset = static_cast<int>(std::max({static_cast<size_t>(worlds) * pop, 5 * nb, static_cast<size_t>(ra.n_hand), static_cast<size_t>(ra.n_flag)}));
  hipLaunchKernelGGL(world_reset_kernel, dim3((n_reset + 255) / 256), dim3(256), 0, s, ra);
  rc = check_launch("world_reset_kernel");
  if (rc) return rc;

  StepArgs a;
  a.params = params, a.P = sh.P, a.pop = pop, a.worlds = worlds;
  a.act[0] = sh.act[0], a.act[1] = sh.act[1], a.act[2] = sh.act[2];
  a.c = c;
  a.key0 = ra.key0, a.key1 = ra.key1, a.gen = gen, a.gen_dev = gen_dev;
  a.vel_in = vel, a.vel_out = vel, a.reward = reward, a.accumulate = 1;
  a.actions_in = nullptr, a.obs_out = nullptr;
  if (turn) {
    ResidentArgs b;
    b.params = params, b.P = sh.P, b.pop = pop, b.worlds = worlds, b.steps = steps;
    b.act[0] = sh.act[0], b.act[1] = sh.act[1], b.act[2] = sh.act[2];
    b.c = c, b.key0 = a.key0, b.key1 = a.key1, b.gen = gen, b.gen_dev = gen_dev;
    b.per_lane = pad_to((pop + 63) / 64, 2);
    b.lane_magic = static_cast<uint32_t>(((1ull << 32) + b.per_lane - 1) / b.per_lane);
    b.even = reinterpret_cast<unsigned long long*>(pos[0]), b.odd = reinterpret_cast<unsigned long long*>(pos[1]);
    b.hand = ra.hand, b.groups = groups, b.wait_ticks = form.wait_ticks == kForageWait ? kWaitTicks + kWaitTicksPerStep * static_cast<uint64_t>(steps) : form.wait_ticks;
    b.fail_main = form.fail_main, b.fail_items = form.fail_items, b.fail_groups = form.fail_groups;
    b.reward = reward, b.pos_out = pos[steps & 1], b.vel_out = vel, b.counts_out = counts_out;
    const int stride = (b.per_lane >> 1) & 1 ? b.per_lane : b.per_lane + 2;
    const size_t slots = static_cast<size_t>(chunks) * kChunk;
    const size_t lds = resident_agents(H) * (sizeof(float4) + sizeof(float2)) +
                       (64 * static_cast<size_t>(stride) + 2 * item_waves(H) * slots) * sizeof(float2) +
                       (item_waves(H) * (slots + kMaxChunks) + kMaxChunks + 2) * sizeof(uint32_t);
    {
      std::lock_guard<std::mutex> lock(turn->m);
      hipError_t e = turn->used ? hipStreamWaitEvent(s, turn->done, 0) : hipSuccess;
      EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "forage: waiting for the launch before failed: %s", hipGetErrorString(e));
      b.per_launch = per_launch;
      for (int w = 0; w < worlds; w += per_launch) {
        b.world0 = w, b.flag = ra.flag - w, b.tag0 = static_cast<uint32_t>(w / per_launch) * (static_cast<uint32_t>(steps) + 1u);
        rc = launch_resident(H, b, std::min(per_launch, worlds - w), lds, s);
        if (rc) return rc;
      }
      if (turn->done) {
        e = hipEventRecord(turn->done, s);
        EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "forage: recording the launch failed: %s", hipGetErrorString(e));
        turn->used = true;
      }
    }
    RerunArgs r;
    const int fours = (worlds + kWorldsPerBlock - 1) / kWorldsPerBlock, blocks = (pop + kAgentsPerBlock - 1) / kAgentsPerBlock;
    r.tickets = ra.flag + worlds, r.crew = std::max(1, std::min(blocks, kMaxResident / fours));
    r.flag = ra.flag, r.per_launch = per_launch, r.steps = steps, r.pos[0] = pos[0], r.pos[1] = pos[1], r.book = book, r.counts_out = counts_out;
    rc = launch_rerun(H, a, r, step_lds_bytes(pop, c.n_food, c.n_items), s);
    if (rc) return rc;
  }
  for (int t = 0; t < (turn ? 0 : steps); ++t) {
    a.pos_in = pos[t & 1], a.pos_out = pos[(t + 1) & 1];
    a.counts_in = counts[t & 1], a.counts_out = counts[(t + 1) & 1];
    a.hits_prev = t > 0 ? hits[(t + 2) % 3] : nullptr;  // the page written by step t - 1
    a.hits_cur = hits[t % 3], a.hits_clear = hits[(t + 1) % 3];
    rc = launch_step_for(sh.dims[1], a, s);
    if (rc) return rc;
  }
  if (form.told) {
    if (turn) hipLaunchKernelGGL(world_told_kernel, dim3((worlds + 255) / 256), dim3(256), 0, s, ra.flag, per_launch, worlds, form.told);
    else hipLaunchKernelGGL(world_fill_kernel, dim3((worlds + 255) / 256), dim3(256), 0, s, form.told, worlds, 0u);
    rc = check_launch("world_told_kernel");
    if (rc) return rc;
  }
  if (fitness) {
    hipLaunchKernelGGL(world_finish_kernel, dim3((pop + 255) / 256), dim3(256), 0, s, reward, pop, worlds, fitness);
    rc = check_launch("world_finish_kernel");
    if (rc) return rc;
  }
  // state after the last step, for the test hook
  const size_t agents = static_cast<size_t>(worlds) * pop;
  hipError_t e = hipSuccess;
  if (pos_out) e = hipMemcpyAsync(pos_out, pos[steps & 1], agents * sizeof(float2), hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess && vel_out) e = hipMemcpyAsync(vel_out, vel, agents * sizeof(float2), hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess && reward_out)
    e = hipMemcpyAsync(reward_out, reward, agents * sizeof(int32_t), hipMemcpyDeviceToDevice, s);
  EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "forage: copying the final state failed: %s", hipGetErrorString(e));
  if (counts_out && !turn) {
    // step steps - 1 read counts[(steps - 1) & 1] + hits of step steps - 2 into counts[steps & 1]; its own hits are
    // in hits[(steps - 1) % 3]
    hipLaunchKernelGGL(world_counts_kernel, dim3((static_cast<int>(nb) + 255) / 256), dim3(256), 0, s,
                       counts[steps & 1], hits[(steps - 1) % 3], static_cast<int>(nb), counts_out);
    rc = check_launch("world_counts_kernel");
    if (rc) return rc;
  }
  return EVO_OK;
}

// Lanes per member of the episode kernel: sixteen where a lane then still owns two columns of a layer.
constexpr int solo_lanes(int H) { return H >= 32 ? 16 : 8; }

static size_t solo_lds_bytes(int n_food, int n_items, int lanes) {
  const size_t slots = pad_to(n_food, 2 * lanes) + pad_to(n_items - n_food, 2 * lanes);
  return static_cast<size_t>(kWorldsPerBlock) * (64 / lanes) * slots * (sizeof(float2) + sizeof(uint32_t));
}

template <int H, bool TANH>
static int launch_solo_built(const SoloArgs& a, hipStream_t s) {
  constexpr int LPA = solo_lanes(H);
  const size_t lds = solo_lds_bytes(a.c.n_food, a.c.n_items, LPA);
  static std::atomic<bool> raised[64];  // zero-initialised; a second setter does the same harmless call
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e == hipSuccess && device >= 0 && device < 64 && !raised[device].load()) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&world_solo_kernel<H, LPA, TANH>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kMaxLdsBytes));
    raised[device].store(e == hipSuccess);
  }
  EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "forage: raising the LDS limit of the episode kernel failed: %s",
              hipGetErrorString(e));
  constexpr int members = 64 / LPA;
  const dim3 grid((a.pop + members - 1) / members, (a.worlds + kWorldsPerBlock - 1) / kWorldsPerBlock);
  hipLaunchKernelGGL((world_solo_kernel<H, LPA, TANH>), grid, dim3(64 * kWorldsPerBlock), lds, s, a);
  return check_launch("world_solo_kernel");
}
template <int H>
static int launch_solo(const SoloArgs& a, hipStream_t s) {
  const bool all_tanh = a.act[0] == EVO_ACT_TANH && a.act[1] == EVO_ACT_TANH && a.act[2] == EVO_ACT_TANH;
  return all_tanh ? launch_solo_built<H, true>(a, s) : launch_solo_built<H, false>(a, s);
}

int forage_solo_supported(const MlpShape& sh, int pop, int worlds, const float* cp) {
  WorldConst c;
  int rc = fill_const(cp, &c);
  if (rc) return rc;
  EVO_REQUIRE(sh.n_layers == 3 && sh.dims[0] == kObs && sh.dims[3] == 2 && sh.dims[1] == sh.dims[2] &&
                  (sh.dims[1] == 16 || sh.dims[1] == 32 || sh.dims[1] == 64),
              EVO_ERR_UNSUPPORTED, "forage: the policy must be an MLP of dims {8, H, H, 2} with H = 16, 32 or 64");
  EVO_REQUIRE(pop >= 1, EVO_ERR_ARG, "forage: pop must be positive (got %d)", pop);
  EVO_REQUIRE(worlds >= 1 && worlds <= 4096, EVO_ERR_ARG, "forage: n_rollouts (worlds) must be in [1, 4096]");
  EVO_REQUIRE(solo_lds_bytes(c.n_food, c.n_items, solo_lanes(sh.dims[1])) <= kMaxLdsBytes, EVO_ERR_UNSUPPORTED,
              "forage: too many items");
  return EVO_OK;
}

size_t forage_solo_workspace_bytes(int pop, int worlds) {
  if (pop < 1 || worlds < 1) return 0;
  return (static_cast<size_t>(pop) * worlds * sizeof(int32_t) + 255) & ~size_t(255);
}

int launch_forage_solo(const MlpShape& sh, const float* params, int pop, int worlds, int steps, const float* cp,
                       uint64_t seed, uint32_t gen, const uint32_t* gen_dev, void* work, float* fitness, float* pos_out,
                       float* vel_out, int32_t* reward_out, uint32_t* counts_out, hipStream_t s) {
  SoloArgs a;
  int rc = fill_const(cp, &a.c);
  if (rc) return rc;
  a.params = params, a.P = sh.P, a.pop = pop, a.worlds = worlds, a.steps = steps;
  a.act[0] = sh.act[0], a.act[1] = sh.act[1], a.act[2] = sh.act[2];
  a.key0 = static_cast<uint32_t>(seed), a.key1 = static_cast<uint32_t>(seed >> 32), a.gen = gen, a.gen_dev = gen_dev;
  a.reward = static_cast<int32_t*>(work);
  a.pos_out = reinterpret_cast<float2*>(pos_out), a.vel_out = reinterpret_cast<float2*>(vel_out);
  a.counts_out = counts_out;
  switch (sh.dims[1]) {
    case 16: rc = launch_solo<16>(a, s); break;
    case 32: rc = launch_solo<32>(a, s); break;
    case 64: rc = launch_solo<64>(a, s); break;
    default: return fail(EVO_ERR_UNSUPPORTED, "forage: the hidden width must be 16, 32 or 64");
  }
  if (rc) return rc;
  if (fitness) {
    hipLaunchKernelGGL(world_finish_kernel, dim3((pop + 255) / 256), dim3(256), 0, s, a.reward, pop, worlds, fitness);
    rc = check_launch("world_finish_kernel");
    if (rc) return rc;
  }
  if (reward_out) {
    hipError_t e = hipMemcpyAsync(reward_out, a.reward, static_cast<size_t>(worlds) * pop * sizeof(int32_t),
                                  hipMemcpyDeviceToDevice, s);
    EVO_REQUIRE(e == hipSuccess, EVO_ERR_HIP, "forage: copying the rewards failed: %s", hipGetErrorString(e));
  }
  return EVO_OK;
}

int launch_forage_step(int pop, int worlds, const float* cp, uint64_t seed, uint32_t gen, const float* pos,
                       const float* vel, const uint32_t* counts, const float* actions, float* obs_out, float* pos_out,
                       float* vel_out, int32_t* reward_out, uint32_t* hit_out, hipStream_t s) {
  WorldConst c;
  int rc = fill_const(cp, &c);
  if (rc) return rc;
  const int nb = worlds * c.n_items;
  hipLaunchKernelGGL(world_fill_kernel, dim3((nb + 255) / 256), dim3(256), 0, s, hit_out, nb, 0u);
  rc = check_launch("world_fill_kernel");
  if (rc) return rc;
  StepArgs a;
  a.params = nullptr, a.P = 0, a.pop = pop, a.worlds = worlds;
  a.act[0] = a.act[1] = a.act[2] = EVO_ACT_NONE;
  a.c = c;
  a.key0 = static_cast<uint32_t>(seed), a.key1 = static_cast<uint32_t>(seed >> 32), a.gen = gen, a.gen_dev = nullptr;
  a.pos_in = reinterpret_cast<const float2*>(pos), a.pos_out = reinterpret_cast<float2*>(pos_out);
  a.vel_in = reinterpret_cast<const float2*>(vel), a.vel_out = reinterpret_cast<float2*>(vel_out);
  a.reward = reward_out, a.accumulate = 0;
  a.counts_in = counts, a.hits_prev = nullptr, a.counts_out = nullptr, a.hits_cur = hit_out, a.hits_clear = nullptr;
  a.actions_in = reinterpret_cast<const float2*>(actions), a.obs_out = obs_out;
  return launch_step<16>(a, s);  // the policy is bypassed: any width
}

}  // namespace evo
