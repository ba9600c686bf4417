// wdc.hip — continuous Tag: the C ABI of include/wdc.h and its kernels (gfx950).
//
// One thread per agent.  Envs of at most 32 agents: a workgroup of `bd` threads holds floor(bd / N) envs; the
// moved positions and velocities of the workgroup's envs are staged in LDS, where the runner-side tag test
// and the brute-force K-nearest search read them (env_kernel, rollout_kernel).  Larger envs have a
// workgroup each, sort their agents by strip and column and search windows of that list (block_kernel).
// Every float32 operation that feeds a comparison is written as its own statement and the file is
// compiled without contraction, so that the state is reproducible to the bit (arXiv 2108.13976, Sec. 5.1,
// continuous variant; the numbers are this build's reading, stated in wdc.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "../../include/wdc.h"
#include "wd_dev_common.h"
#include "wd_dev_rows.h"
#include "wd_dev_strips.h"
#include "wdc_dev_strips.h"

namespace wdc {

constexpr int kMaxThreads = 1024;      // one thread per agent, so also the largest env
constexpr int kMaxK = 8;
constexpr uint32_t kStreamActionC = 2;  // random streams of this variant (0 and 1 are the discrete variant's)
constexpr uint32_t kStreamInitC = 3;
enum Mode : int { kSample = 1, kStep = 2, kResetDone = 4, kResetAll = 8 };

struct Params {
  int32_t E, N, N_tag, H, T, K, D;
  int32_t envs_per_wg, threads;
  uint32_t env_offset, seed_lo, seed_hi;
  wd::FastDiv div_N;
  float L, inv_L, inv_T, accel, vmax_tagger, vmax_runner, tag_r2, tag_reward, tag_penalty;
  float *x, *y, *v;
  int32_t* h;
  float *x0, *y0;
  int32_t* h0;
  int32_t* live;
  int32_t* action;
  float* reward;
  float* obs;
  int32_t *t, *done, *n_live_runners, *tags_step;
  const float2* table;  // (cx, cy) per heading
};

// What block_kernel needs beyond that: the geometry of an env's list, the tag check's form and reach, and
// the LDS map in byte offsets (see plan_block).  Apart from Params, which every launch of the other
// kernels carries.
struct BlockPlan {
  int32_t kt;            // neighbours searched for (2, 4, 6 or 8, at least K); 0: block_kernel does not serve this
  int32_t threads, strip_rmax, tag_by_tagger;
  float strip_scale, tag_reach;
  int32_t off_misc, off_tag, off_near, off_list, off_ids, off_table, off_found, off_stage, lds;
};

namespace {

using wd::dev::philox_block;
using wd::dev::sample_action;

// start state of every agent (once per reset of all envs)
__global__ __launch_bounds__(256) void init_kernel(const Params p) {
  const int64_t a = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (a >= int64_t(p.E) * p.N) return;
  const uint32_t e = uint32_t(a / p.N), i = uint32_t(a - int64_t(e) * p.N);
  const wd::dev::Block4 r = philox_block(p.env_offset + e, i, 0u, kStreamInitC, p.seed_lo, p.seed_hi);
  const float u0 = static_cast<float>(r.w[0] >> 8) * (1.0f / 16777216.0f);
  const float u1 = static_cast<float>(r.w[1] >> 8) * (1.0f / 16777216.0f);
  p.x0[a] = u0 * p.L;
  p.y0[a] = u1 * p.L;
  p.h0[a] = int32_t(__umulhi(r.w[2], uint32_t(p.H)));
}

// heading index brought into [0, H): also keeps a caller's stray value from indexing outside the table
__device__ __forceinline__ int wrap_heading(int h, int H) {
  const int r = h % H;
  return r < 0 ? r + H : r;
}

__device__ __forceinline__ float squared_distance(float xa, float ya, float xb, float yb) {
  const float dx = xa - xb;
  const float dy = ya - yb;
  const float dx2 = dx * dx;
  const float dy2 = dy * dy;
  return dx2 + dy2;
}

// One live agent turns, changes speed, moves and meets the walls.
__device__ __forceinline__ void advance_agent(const Params& p, bool tagger, int lvl_acc, int lvl_turn, float& x, float& y,
                                              float& v, int& h, float2& dir) {
  h = wrap_heading(h + (lvl_turn - 2), p.H);
  dir = p.table[h];
  const float vmax = tagger ? p.vmax_tagger : p.vmax_runner;
  const float dv = static_cast<float>(lvl_acc - 2) * p.accel;
  v = v + dv;
  if (v < 0.0f) v = 0.0f;
  if (v > vmax) v = vmax;
  const float step_x = v * dir.x;
  const float step_y = v * dir.y;
  x = x + step_x;
  y = y + step_y;
  bool clamped = false;
  if (x < 0.0f) { x = 0.0f; clamped = true; }
  if (x > p.L) { x = p.L; clamped = true; }
  if (y < 0.0f) { y = 0.0f; clamped = true; }
  if (y > p.L) { y = p.L; clamped = true; }
  if (clamped) v = 0.0f;
}

// An agent's ten probabilities (five per action category) as five 8-byte pieces.
struct Probs10 {
  float2 q[5];
};
__device__ __forceinline__ Probs10 load_probs(const float* __restrict__ probs, int64_t a) {
  const float2* pr = reinterpret_cast<const float2*>(probs + a * 10);
  Probs10 r;
#pragma unroll
  for (int k = 0; k < 5; ++k) r.q[k] = pr[k];
  return r;
}

// The two levels of an agent's action from its ten probabilities and one random block.
__device__ __forceinline__ int2 draw_levels(const Params& p, const Probs10& pr, int e, int i, uint32_t g_lo,
                                            uint32_t g_hi) {
  const wd::dev::Block4 r = philox_block(p.env_offset + uint32_t(e), uint32_t(i), g_lo, kStreamActionC | (g_hi << 8),
                                         p.seed_lo, p.seed_hi);
  const int lvl_acc = sample_action(pr.q[0].x, pr.q[0].y, pr.q[1].x, pr.q[1].y, r.w[0]);   // probabilities 0..3 of category 0
  const int lvl_turn = sample_action(pr.q[2].y, pr.q[3].x, pr.q[3].y, pr.q[4].x, r.w[1]);  // 5..8 = 0..3 of category 1
  return make_int2(lvl_acc, lvl_turn);
}

// The nearest tagger of a runner at (x, y) by (d2, index): true if it is in range.
__device__ __forceinline__ bool tagger_in_range(const Params& p, const float* s_x, const float* s_y, int first, float x,
                                                float y, int* tagger_out) {
  int best_t = 0;
  float best_d2 = squared_distance(x, y, s_x[first], s_y[first]);
  for (int t = 1; t < p.N_tag; ++t) {
    const float d2 = squared_distance(x, y, s_x[first + t], s_y[first + t]);
    if (d2 < best_d2) {
      best_d2 = d2;
      best_t = t;
    }
  }
  *tagger_out = best_t;
  return best_d2 <= p.tag_r2;
}

// The observation row of agent i of the env whose agents sit in LDS slots first .. first + N - 1.
template <int KT>
__device__ __forceinline__ void write_row(const Params& p, float* row, const float* s_x, const float* s_y,
                                          const float* s_vx, const float* s_vy, const int32_t* s_live, int first, int i,
                                          float x, float y, float v, float2 dir, bool tagger, int live, int t_out) {
  const int K = p.K;
  uint64_t keys[KT];
#pragma unroll
  for (int k = 0; k < KT; ++k) keys[k] = ~0ull;
  if (live == 1 && K > 0) {
    for (int j = 0; j < p.N; ++j) {
      if (j == i || s_live[first + j] != 1) continue;
      const float d2 = squared_distance(s_x[first + j], s_y[first + j], x, y);
      uint64_t key = (uint64_t(__float_as_uint(d2)) << 32) | uint32_t(j);  // d2 >= +0: its bits order like its value
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        if (k < K && key < keys[k]) {
          const uint64_t tmp = keys[k];
          keys[k] = key;
          key = tmp;
        }
      }
    }
  }
  float2* row2 = reinterpret_cast<float2*>(row);  // D is even and the buffer 256-byte aligned: 8-byte pieces
  row2[0] = make_float2(x * p.inv_L, y * p.inv_L);
  row2[1] = make_float2(v, dir.x);
  row2[2] = make_float2(dir.y, tagger ? 1.0f : 0.0f);
  row2[3] = make_float2(live == 1 ? 1.0f : 0.0f, static_cast<float>(t_out) * p.inv_T);
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    if (k < K) {
      float2 s0 = make_float2(0.0f, 0.0f), s1 = s0, s2 = s0;
      if (keys[k] != ~0ull) {
        const int j = int(uint32_t(keys[k]));
        const float dx = s_x[first + j] - x;
        const float dy = s_y[first + j] - y;
        s0 = make_float2(dx * p.inv_L, dy * p.inv_L);
        s1 = make_float2(s_vx[first + j], s_vy[first + j]);
        s2 = make_float2(j < p.N_tag ? 1.0f : 0.0f, 1.0f);
      }
      row2[4 + 3 * k] = s0;
      row2[5 + 3 * k] = s1;
      row2[6 + 3 * k] = s2;
    }
  }
}

// KT: length of the register list of nearest keys (4 or 8, at least K)
template <int KT>
__global__ __launch_bounds__(kMaxThreads) void env_kernel(const Params p, const int mode, const float* __restrict__ probs,
                                                           const uint32_t g_lo, const uint32_t g_hi) {
  // per local agent slot: moved position, velocity components, live flag, credits (taggers)
  // (dynamic LDS: 26 bytes per thread of the workgroup, see lds_bytes)
  extern __shared__ __align__(16) unsigned char smem[];
  float* const s_x = reinterpret_cast<float*>(smem);
  float* const s_y = s_x + p.threads;
  float* const s_vx = s_y + p.threads;
  float* const s_vy = s_vx + p.threads;
  int32_t* const s_live = reinterpret_cast<int32_t*>(s_vy + p.threads);
  int32_t* const s_credits = s_live + p.threads;
  int32_t* const s_tags = s_credits + p.threads;  // per env of the workgroup: at most threads / 2
  const int tid = threadIdx.x;
  const int el = int(wd::dev::fastdiv(uint32_t(tid), p.div_N));  // env of the workgroup
  const int i = tid - el * p.N;                                  // agent
  const int e = blockIdx.x * p.envs_per_wg + el;
  const bool valid = el < p.envs_per_wg && e < p.E;
  const int first = el * p.N;  // slot of the env's agent 0
  const int64_t a = int64_t(valid ? e : 0) * p.N + i;
  const bool tagger = i < p.N_tag;

  // ---- sampler: two draws per agent from one random block ------------------------------------
  int lvl_acc = 2, lvl_turn = 2;
  if (mode & kSample) {
    if (valid) {
      const int2 lv = draw_levels(p, load_probs(probs, a), e, i, g_lo, g_hi);
      lvl_acc = lv.x;
      lvl_turn = lv.y;
      *reinterpret_cast<int2*>(p.action + 2 * a) = lv;
    }
    if (mode == kSample) return;
  } else if ((mode & kStep) && valid) {
    const int2 act = *reinterpret_cast<const int2*>(p.action + 2 * a);
    lvl_acc = act.x;
    lvl_turn = act.y;
  }

  int done_in = 0, t_in = 0, nlr_in = 0;
  if (valid) {
    done_in = p.done[e];
    t_in = p.t[e];
    nlr_in = p.n_live_runners[e];
  }
  const bool step_act = (mode & kStep) && valid && !done_in;
  bool new_rows = false;
  int t_out = t_in;
  bool done_now = done_in != 0;
  float x = 0.0f, y = 0.0f, v = 0.0f;
  int h = 0, live = 0;
  float2 dir = make_float2(1.0f, 0.0f);

  if (mode & kStep) {
    if (step_act) {
      x = p.x[a];
      y = p.y[a];
      v = p.v[a];
      h = p.h[a];
      live = p.live[a];
      if (live == 1) {
        advance_agent(p, tagger, lvl_acc, lvl_turn, x, y, v, h, dir);
        p.x[a] = x;
        p.y[a] = y;
        p.v[a] = v;
        p.h[a] = h;
      } else {
        dir = p.table[wrap_heading(h, p.H)];
      }
      s_x[tid] = x;
      s_y[tid] = y;
      s_vx[tid] = v * dir.x;
      s_vy[tid] = v * dir.y;
      s_live[tid] = live;
      s_credits[tid] = 0;
      if (i == 0) s_tags[el] = 0;
    }
    __syncthreads();
    // ---- tag test from the runner's side: nearest tagger by (d2, index) ------------------------
    bool tagged_now = false;
    if (step_act && !tagger && live == 1 && p.tag_r2 >= 0.0f) {
      int best_t;
      if (tagger_in_range(p, s_x, s_y, first, x, y, &best_t)) {
        tagged_now = true;
        live = 0;
        s_live[tid] = 0;  // (the loops above read taggers only, and taggers stay live)
        p.live[a] = 0;
        atomicAdd(&s_credits[first + best_t], 1);
        atomicAdd(&s_tags[el], 1);
      }
    }
    __syncthreads();
    // ---- rewards, clock, end of episode ---------------------------------------------------------
    if (step_act) {
      float rew = 0.0f;
      if (tagger)
        rew = static_cast<float>(s_credits[tid]) * p.tag_reward;
      else if (tagged_now)
        rew = p.tag_penalty;
      p.reward[a] = rew;
      const int tags = s_tags[el];
      const int nlr = nlr_in - tags;
      t_out = t_in + 1;
      done_now = nlr == 0 || t_out >= p.T;
      if (i == 0) {
        p.t[e] = t_out;
        p.n_live_runners[e] = nlr;
        p.tags_step[e] = tags;
        p.done[e] = done_now ? 1 : 0;
      }
      new_rows = true;
    }
  }

  // ---- reset: envs that are done (or all) go back to their start state ---------------------------
  if (mode & (kResetDone | kResetAll)) {
    if (valid && ((mode & kResetAll) || done_now)) {
      x = p.x0[a];
      y = p.y0[a];
      h = wrap_heading(p.h0[a], p.H);
      v = 0.0f;
      live = 1;
      dir = p.table[h];
      p.x[a] = x;
      p.y[a] = y;
      p.h[a] = h;
      p.v[a] = v;
      p.live[a] = 1;
      t_out = 0;
      if (i == 0) {
        p.t[e] = 0;
        p.n_live_runners[e] = p.N - p.N_tag;
        p.tags_step[e] = 0;
        p.done[e] = 0;
      }
      s_x[tid] = x;
      s_y[tid] = y;
      s_vx[tid] = v * dir.x;
      s_vy[tid] = v * dir.y;
      s_live[tid] = 1;
      new_rows = true;
    }
  }
  __syncthreads();

  // ---- observation rows ---------------------------------------------------------------------------
  if (!new_rows) return;
  write_row<KT>(p, p.obs + a * p.D, s_x, s_y, s_vx, s_vy, s_live, first, i, x, y, v, dir, tagger, live, t_out);
}

// Several roll-out iterations in one launch (envs never interact, and an env's agents share a
// workgroup, so no synchronisation beyond the workgroup is needed).  Between the iterations an
// agent's state stays in its thread's registers and the env's clock, live count and done flag in
// every one of its threads; iteration s draws with step g0 + s from ring entry (ring_pos + s) mod
// ring_len and writes action, reward and rows to slice s of the roll-out arrays (to the in-place
// arrays where a roll-out array is not given, and always in the last iteration); the done flags
// recorded are those before the reset.  The state arrays are written once, at the end.
struct Roll {
  int32_t steps, ring_len, ring_pos, pad;
  int32_t* action;
  float* reward;
  int32_t* done;
  float* obs;
  const float* ring;
  uint64_t g0;
};

template <int KT>
__global__ __launch_bounds__(kMaxThreads) void rollout_kernel(const Params p, const Roll roll) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* const s_x = reinterpret_cast<float*>(smem);
  float* const s_y = s_x + p.threads;
  float* const s_vx = s_y + p.threads;
  float* const s_vy = s_vx + p.threads;
  int32_t* const s_live = reinterpret_cast<int32_t*>(s_vy + p.threads);
  int32_t* const s_credits = s_live + p.threads;
  int32_t* const s_tags = s_credits + p.threads;
  const int tid = threadIdx.x;
  const int el = int(wd::dev::fastdiv(uint32_t(tid), p.div_N));
  const int i = tid - el * p.N;
  const int e = blockIdx.x * p.envs_per_wg + el;
  const bool valid = el < p.envs_per_wg && e < p.E;
  const int first = el * p.N;
  const int64_t a = int64_t(valid ? e : 0) * p.N + i;
  const bool tagger = i < p.N_tag;
  const int64_t EN = int64_t(p.E) * p.N;

  float x = 0.0f, y = 0.0f, v = 0.0f;
  int h = 0, live = 0, t = 0, nlr = 0, tags_last = 0;
  bool done = false;
  if (valid) {
    x = p.x[a];
    y = p.y[a];
    v = p.v[a];
    h = wrap_heading(p.h[a], p.H);
    live = p.live[a];
    t = p.t[e];
    nlr = p.n_live_runners[e];
    tags_last = p.tags_step[e];
    done = p.done[e] != 0;
  }
  float2 dir = p.table[h];
  // (an env that enters done: the first iteration does not step it; the last slice is copied from the in-place arrays)
  if (done && roll.reward && roll.steps > 1) roll.reward[a] = p.reward[a];

  for (int s = 0; s < roll.steps; ++s) {
    const bool last = s + 1 == roll.steps;
    const uint64_t g = roll.g0 + uint64_t(s);
    const float* probs = roll.ring + int64_t((roll.ring_pos + s) % roll.ring_len) * EN * 10;
    int32_t* const action_out = (roll.action && !last) ? roll.action + int64_t(s) * 2 * EN : p.action;
    float* const reward_out = (roll.reward && !last) ? roll.reward + int64_t(s) * EN : p.reward;
    float* const obs_out = (roll.obs && !last) ? roll.obs + int64_t(s) * EN * p.D : p.obs;
    int2 lv = make_int2(2, 2);
    if (valid) {
      lv = draw_levels(p, load_probs(probs, a), e, i, uint32_t(g), uint32_t(g >> 32));
      *reinterpret_cast<int2*>(action_out + 2 * a) = lv;
    }
    const bool step_act = valid && !done;
    bool new_rows = false;
    if (step_act) {
      if (live == 1) advance_agent(p, tagger, lv.x, lv.y, x, y, v, h, dir);
      s_x[tid] = x;
      s_y[tid] = y;
      s_vx[tid] = v * dir.x;
      s_vy[tid] = v * dir.y;
      s_live[tid] = live;
      s_credits[tid] = 0;
      if (i == 0) s_tags[el] = 0;
    }
    __syncthreads();
    bool tagged_now = false;
    if (step_act && !tagger && live == 1 && p.tag_r2 >= 0.0f) {
      int best_t;
      if (tagger_in_range(p, s_x, s_y, first, x, y, &best_t)) {
        tagged_now = true;
        live = 0;
        s_live[tid] = 0;
        atomicAdd(&s_credits[first + best_t], 1);
        atomicAdd(&s_tags[el], 1);
      }
    }
    __syncthreads();
    if (step_act) {
      float rew = 0.0f;
      if (tagger)
        rew = static_cast<float>(s_credits[tid]) * p.tag_reward;
      else if (tagged_now)
        rew = p.tag_penalty;
      reward_out[a] = rew;
      tags_last = s_tags[el];
      nlr -= tags_last;
      t += 1;
      done = nlr == 0 || t >= p.T;
      new_rows = true;
    }
    if (roll.done && valid && i == 0) roll.done[int64_t(s) * p.E + e] = done ? 1 : 0;  // the flag before the reset
    if (valid && done) {  // back to the start state
      x = p.x0[a];
      y = p.y0[a];
      h = wrap_heading(p.h0[a], p.H);
      v = 0.0f;
      live = 1;
      dir = p.table[h];
      t = 0;
      nlr = p.N - p.N_tag;
      tags_last = 0;
      done = false;
      s_x[tid] = x;
      s_y[tid] = y;
      s_vx[tid] = v * dir.x;
      s_vy[tid] = v * dir.y;
      s_live[tid] = 1;
      new_rows = true;
    }
    __syncthreads();
    if (new_rows)
      write_row<KT>(p, obs_out + a * p.D, s_x, s_y, s_vx, s_vy, s_live, first, i, x, y, v, dir, tagger, live, t);
    __syncthreads();  // the rows are read out of LDS before the next iteration overwrites it
  }
  if (valid) {
    p.x[a] = x;
    p.y[a] = y;
    p.v[a] = v;
    p.h[a] = h;
    p.live[a] = live;
    if (i == 0) {
      p.t[e] = t;
      p.n_live_runners[e] = nlr;
      p.tags_step[e] = tags_last;
      p.done[e] = done ? 1 : 0;
    }
  }
}


// ----------------------------------------------------------------------------------
// Envs of more than 32 agents: one workgroup per env, one thread per agent, any mode, one or more
// iterations per launch.  The agents in play are sorted by strip and column every iteration
// (wdc_dev_strips.h); the search runs in list order over fixed windows, and the few agents that
// these do not settle are served by sixteen lanes each.  Between the iterations of a launch an
// agent's state stays in its thread's registers.
//
// Bound: comparing all pairs was bound by the vector ALUs; now a launch is the latency of one workgroup's
// chain (about 23 000 cycles at 105 agents: 7 800 for the first loads and draws, 5 200 the list, 2 100 the tag
// check, 4 700 the search, 4 000 the rows) between a burst of loads and a burst of row stores.  2000 envs x 105
// agents, K = 4: 33.8 -> 18.0 us per iteration (46 MB: 2.5 TB/s); 250 x 820, four recorded iterations per launch:
// 1007 -> 70.4 us (184 MB).  Five waves per SIMD: at 64 registers (eight) the windows spill, 26 us instead of 18.8.
// ----------------------------------------------------------------------------------
constexpr int kScanAll = 64;      // lists up to this length (the most that six bits number) are compared whole: 11
                                  // instructions an entry against about 500 for the 38 window slots and their bounds
                                  // (K = 4), and hardly ever a second try.  us per iteration with 44 / 64: 500 x 64
                                  // 12.6 / 11.2, in three clusters 20.4 / 11.1; 2000 x 48, K = 8 16.9 / 16.3, 25.6 / 15.8
constexpr int kCrowdCost = 250;   // what a queued agent of a crowd costs a wave, in the instructions that a lane spends on
                                  // 1 / (8 + 4 KT) list entries
constexpr int kGroupLanes = 16, kGroups = wd::kWaveSize / kGroupLanes;  // lanes that serve a queued agent together
enum Misc : int { kTags = 0, kQueued = 1, kStray = 2, kOpen = 3, kWaveTotals = 4, kMiscWords = 20 };
constexpr float kOpenLimit = -1.0f;  // in limit[]: this queued agent is to be compared with the whole list

struct BlockLds {
  float4* me;         // [threads] x, y and the velocity components after the move
  int32_t* misc;
  uint64_t* tag_key;  // [threads] per runner: smallest (d2, tagger) in range
  int32_t* credits;   // [threads]
  uint16_t* nearest;  // [threads][KT] (from here on over tag_key and credits)
  float* limit;       // [threads] per queued agent: no neighbour of it is farther than this (squared)
  uint16_t* queue;    // [threads] list slots of the agents that the windows did not settle
  float2* list;       // positions by strip and column, pads on either side
  uint16_t* ids;
  uint16_t* table;    // bin starts
  uint64_t* found;    // [waves][kGroups][kGroupLanes] keys collected for queued agents
  float* stage;       // [waves][kStageRows][stage_stride(KT)], over the list
  __device__ __forceinline__ BlockLds(unsigned char* smem, const BlockPlan& b, int kt) {
    const int nt = b.threads, pad = list_pad(kt);
    me = reinterpret_cast<float4*>(smem);
    misc = reinterpret_cast<int32_t*>(smem + b.off_misc);
    tag_key = reinterpret_cast<uint64_t*>(smem + b.off_tag);
    credits = reinterpret_cast<int32_t*>(smem + b.off_tag + 8 * nt);
    limit = reinterpret_cast<float*>(smem + b.off_near);
    queue = reinterpret_cast<uint16_t*>(smem + b.off_near + 4 * nt);
    nearest = queue + nt;
    list = reinterpret_cast<float2*>(smem + b.off_list) + pad;
    ids = reinterpret_cast<uint16_t*>(smem + b.off_ids);
    table = reinterpret_cast<uint16_t*>(smem + b.off_table);
    found = reinterpret_cast<uint64_t*>(smem + b.off_found);
    stage = reinterpret_cast<float*>(smem + b.off_stage);
  }
};

// Sorts the agents in play into the list (a counting sort over the bins); returns their number, and
// this thread's slot.  Every thread of the workgroup calls.  The counters in misc start at zero again.
template <int KT>
__device__ __forceinline__ int build_list(float world, int threads, const BlockLds& L, const Strips& g, int tid, bool in_play,
                                          float x, float y, int& slot) {
  uint32_t* const tw = reinterpret_cast<uint32_t*>(L.table);
  const int words = (g.R * kColumns + 2) >> 1;
  for (int j = tid; j < words; j += threads) tw[j] = 0u;
  if (tid < kWaveTotals) L.misc[tid] = 0;
  __syncthreads();
  const int bin = strip_at(y, g) * kColumns + column_at(x, g);
  if (in_play) {
    wd::dev::strip_count(tw, bin);
    if (!(x >= 0.0f && x <= world && y >= 0.0f && y <= world)) L.misc[kStray] = 1;  // (a caller's start state)
  }
  __syncthreads();
  const int chunk = (words + threads - 1) / threads;
  const int j0 = min(tid * chunk, words), j1 = min(j0 + chunk, words);
  int part = 0;
  for (int j = j0; j < j1; ++j) part += int(tw[j] & 0xFFFFu) + int(tw[j] >> 16);
  int incl = part;
  const int lane = tid & (wd::kWaveSize - 1), wave = tid >> 6;
#pragma unroll
  for (int d = 1; d < wd::kWaveSize; d <<= 1) {
    const int up = __shfl_up(incl, d);
    if (lane >= d) incl += up;
  }
  if (lane == wd::kWaveSize - 1) L.misc[kWaveTotals + wave] = incl;
  __syncthreads();
  int run = incl - part, n = 0;
  for (int w = 0; w < threads / wd::kWaveSize; ++w) {
    const int wt = L.misc[kWaveTotals + w];
    if (w < wave) run += wt;
    n += wt;
  }
  for (int j = j0; j < j1; ++j) {
    const uint32_t c = tw[j];
    const uint32_t lo = uint32_t(run);
    run += int(c & 0xFFFFu);
    tw[j] = lo | (uint32_t(run) << 16);
    run += int(c >> 16);
  }
  __syncthreads();
  if (in_play) {
    slot = int(wd::dev::strip_take_slot(tw, bin));
    L.list[slot] = make_float2(x, y);
    L.ids[slot] = uint16_t(tid);
  }
  constexpr int pad = list_pad(KT);
  static_assert(2 * pad <= wd::kWaveSize, "one wave writes the pads");
  if (tid < 2 * pad) L.list[tid < pad ? -1 - tid : n + (tid - pad)] = make_float2(0.0f, kGone);
  __syncthreads();
  return n;
}

// Runners within reach of tagger `tagger` at (x, y) get the smallest (d2, tagger) key.
__device__ __forceinline__ void reach_of_tagger(const Params& p, float reach, const BlockLds& L, const Strips& g, int tagger,
                                                float x, float y) {
  const int c0 = column_at(x - reach, g), c1 = column_at(x + reach, g);
  const int r0 = strip_at(y - reach, g), r1 = strip_at(y + reach, g);
  for (int r = r0; r <= r1; ++r) {
    const int end = L.table[r * kColumns + c1 + 1];
    for (int q = L.table[r * kColumns + c0]; q < end; ++q) {
      const int j = L.ids[q];
      if (j < p.N_tag) continue;
      const float2 at = L.list[q];
      const float d2 = squared_distance(at.x, at.y, x, y);
      if (d2 <= p.tag_r2)
        atomicMin(reinterpret_cast<unsigned long long*>(&L.tag_key[j]),
                  (static_cast<unsigned long long>(__float_as_uint(d2)) << 32) | static_cast<unsigned long long>(tagger));
    }
  }
}

// The KT nearest of the agent in list slot q, into nearest[]; false if the windows do not settle them
// (`limit` then bounds the squared distance of the KT-th from above, as far as that is known).
template <int KT>
__device__ __forceinline__ bool search_windows(const BlockLds& L, const Strips& g, int q, int n, float* limit) {
  const float2 me = L.list[q];
  uint32_t keys[KT + 1];
  int below = 0, above = 0;
  float reach2 = kFarF * kFarF;
  const bool whole = n <= kScanAll;  // uniform
  if (whole)
    near_all<KT>(keys, me, q, n, L.list);
  else
    reach2 = near_windows<KT>(keys, me, q, n, g, L.list, L.table, below, above);
  const uint32_t kth = keys[KT - 1];
  // above the exact squared distance of the KT-th: the dropped bits filled up, and some
  const float kth_most = __uint_as_float((kth | kNumberMask) + 2u * kNumberMask);
  *limit = kth < kGoneKey ? kth_most : kFarF * kFarF;
  const bool complete = kth < kGoneKey ? kth_most < reach2 : reach2 >= kFarF * kFarF;
  if (!complete || undecided(kth, keys[KT])) return false;
  uint64_t exact[KT];
  bool close = false;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const int number = int(keys[k] & kNumberMask);
    const int s = keys[k] < kGoneKey ? (whole ? number : slot_of_number<KT>(number, q, below, above)) : q;
    exact[k] = keys[k] < kGoneKey ? uint64_t(L.ids[s]) : uint64_t(kNobody);
    if (k > 0) close |= undecided(keys[k - 1], keys[k]);
  }
  if (close) {  // hardly ever: the order of two neighbours takes their exact squared distances
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      if (exact[k] == kNobody) {
        exact[k] = ~0ull;
        continue;
      }
      const float4 o = L.me[uint32_t(exact[k])];
      exact[k] |= uint64_t(__float_as_uint(squared_distance(o.x, o.y, me.x, me.y))) << 32;
    }
#pragma unroll
    for (int a = 0; a < KT - 1; ++a)
#pragma unroll
      for (int b = 0; b < KT - 1 - a; ++b) {
        const uint64_t lo = exact[b] < exact[b + 1] ? exact[b] : exact[b + 1];
        const uint64_t hi = exact[b] < exact[b + 1] ? exact[b + 1] : exact[b];
        exact[b] = lo;
        exact[b + 1] = hi;
      }
  }
  uint32_t* const out = reinterpret_cast<uint32_t*>(L.nearest + uint32_t(L.ids[q]) * KT);
#pragma unroll
  for (int k = 0; k < KT / 2; ++k) out[k] = (uint32_t(exact[2 * k]) & 0xFFFFu) | (uint32_t(exact[2 * k + 1]) << 16);
  return true;
}

// The exact key of list entry s for the agent at `me` in slot q; ~0: not a candidate.
__device__ __forceinline__ uint64_t exact_key(const BlockLds& L, int s, int q, float2 me) {
  const uint32_t id = L.ids[s];
  const float2 at = L.list[s];
  const uint64_t key = (uint64_t(__float_as_uint(squared_distance(at.x, at.y, me.x, me.y))) << 32) | id;
  return (s == q || (id & kGoneId)) ? ~0ull : key;
}

// One agent by a whole wave: the KT smallest keys of the list, one after the other.
template <int KT>
__device__ __forceinline__ void search_by_wave(const BlockLds& L, int q, int n, int lane) {
  const float2 me = L.list[q];
  const uint32_t i = L.ids[q];
  uint64_t last = 0;
  for (int k = 0; k < KT; ++k) {
    uint64_t best = ~0ull;
    if (k == 0 || last != ~0ull)
      for (int s = lane; s < n; s += wd::kWaveSize) {
        const uint64_t key = exact_key(L, s, q, me);
        if ((k == 0 || key > last) && key < best) best = key;
      }
    last = wave_min(best);
    if (lane == 0) L.nearest[i * KT + k] = last == ~0ull ? kNobody : uint16_t(last);
  }
}

// One agent by its lane: every entry of the list.
template <int KT>
__device__ __forceinline__ void search_by_lane(const BlockLds& L, int q, int n) {
  const float2 me = L.list[q];
  uint64_t keys[KT];
#pragma unroll
  for (int k = 0; k < KT; ++k) keys[k] = ~0ull;
  for (int s0 = 0; s0 < n; s0 += 4) {
    uint64_t key[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) key[j] = exact_key(L, min(s0 + j, n - 1), q, me);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (s0 + j >= n) key[j] = ~0ull;
      if (key[j] < keys[KT - 1]) {
#pragma unroll
        for (int k = 0; k < KT; ++k) {
          const uint64_t lo = key[j] < keys[k] ? key[j] : keys[k];
          key[j] = key[j] < keys[k] ? keys[k] : key[j];
          keys[k] = lo;
        }
      }
    }
  }
  uint32_t* const out = reinterpret_cast<uint32_t*>(L.nearest + uint32_t(L.ids[q]) * KT);
#pragma unroll
  for (int k = 0; k < KT / 2; ++k) out[k] = (uint32_t(keys[2 * k]) & 0xFFFFu) | (uint32_t(keys[2 * k + 1]) << 16);  // (~0: kNobody)
}

// The queued agents, four to a wave, sixteen lanes each.  No neighbour of such an agent is farther than its
// limit, so only the bins that this radius touches are read, a strip at a time; the entries within the limit
// are collected with their exact keys, and an entry's rank among them is its place.  An agent without a
// limit, or with more entries in it than there is room for (agents crowded at one distance), is marked open.
template <int KT>
__device__ __forceinline__ void search_queue(const BlockLds& L, const Strips& g, int n, int queued, int lane, int wave,
                                             int waves) {
  const int sub = lane & (kGroupLanes - 1), group = lane / kGroupLanes;
  uint64_t* const found = L.found + wave * wd::kWaveSize + group * kGroupLanes;
  for (int w0 = wave * kGroups; w0 < queued; w0 += waves * kGroups) {
    const int w = w0 + group;
    bool open = false;
    if (w < queued) {
      const int q = L.queue[w];
      const float limit = L.limit[w];
      const float2 me = L.list[q];
      const uint32_t i = L.ids[q];
      open = !(limit < kFarF);
      if (!open) {
        const float reach = sqrtf(limit) * 1.00001f + g.eps;
        const int c0 = column_at(me.x - reach, g), c1 = column_at(me.x + reach, g);
        const int r0 = strip_at(me.y - reach, g), r1 = strip_at(me.y + reach, g);
        int count = 0;
        for (int r = r0; r <= r1; ++r) {
          const int end = L.table[r * kColumns + c1 + 1];
          for (int s0 = L.table[r * kColumns + c0]; s0 < end; s0 += kGroupLanes) {
            const int s = s0 + sub;
            const uint64_t key = s < end ? exact_key(L, s, q, me) : ~0ull;
            const bool in = key != ~0ull && __uint_as_float(uint32_t(key >> 32)) <= limit;
            const uint32_t votes = uint32_t(__ballot(in) >> (group * kGroupLanes)) & ((1u << kGroupLanes) - 1u);
            const int at = count + __popc(votes & ((1u << sub) - 1u));
            if (in && at < kGroupLanes) found[at] = key;
            count += __popc(votes);
          }
        }
        open = count > kGroupLanes;
        if (!open) {
          wd::dev::wave_sync_lds();
          const uint64_t mine = sub < count ? found[sub] : ~0ull;
          int rank = 0;
          for (int j = 0; j < count; ++j) rank += found[j] < mine ? 1 : 0;
          if (sub < count && rank < KT) L.nearest[i * KT + rank] = uint16_t(mine);
          if (sub >= count && sub < KT) L.nearest[i * KT + sub] = kNobody;
        }
      }
    }
    if (open && sub == 0) {
      L.limit[w] = kOpenLimit;
      atomicAdd(&L.misc[kOpen], 1);
    }
    wd::dev::wave_sync_lds();  // `found` is read before the next agents overwrite it
  }
}

// The agents marked open: a few of them by a whole wave each; many (a crowd, whose distances the windows cannot tell
// apart) by a lane each, which costs as much as comparing all pairs, but once for all of them.  With everybody on one spot
// every one of them had a wave, one after the other: 2000 x 105 177 us per iteration -> 34.8 (comparing all pairs: 44.0),
// 250 x 820, K = 8 1143 -> 402 (484); in three clusters 2000 x 105, K = 8 69.4 -> 45.9 (41.6), 250 x 820, K = 8 420 -> 237 (345).
template <int KT>
__device__ __forceinline__ void search_open(const BlockLds& L, int n, int queued, int open, int tid, int waves) {
  // (instructions of a wave: KT passes over the list and reductions for an agent, or the list once for 64)
  if (open * KT * (2 * n / 5 + 90) <= waves * n * (20 + 4 * KT)) {
    for (int w = __builtin_amdgcn_readfirstlane(tid >> 6); w < queued; w += waves)
      if (L.limit[w] == kOpenLimit) search_by_wave<KT>(L, L.queue[w], n, tid & (wd::kWaveSize - 1));
  } else if (tid < queued && L.limit[tid] == kOpenLimit) {
    search_by_lane<KT>(L, L.queue[tid], n);
  }
}

// A wave stores its 64 agents' rows.  With K == KT a row is a whole number of 16-byte pieces: 32 rows at a
// time go to LDS, a row per lane, and leave in pieces that are contiguous across the wave.  Other K
// (odd ones): each lane stores its own row.
constexpr int kStageRows = 32;
constexpr int stage_stride(int kt) {  // floats between staged rows: an odd number of 16-byte pieces, which meets the banks evenly
  return (8 + 6 * kt) % 8 == 0 ? 8 + 6 * kt + 4 : 8 + 6 * kt;
}
template <int KT>
__device__ __forceinline__ void store_rows(const Params& p, const BlockLds& L, float* const rows0, float* const rows1,
                                           int tid, float x, float y, float v, float2 dir, bool tagger, int live, int t) {
  constexpr int DT = 8 + 6 * KT;
  const int lane = tid & (wd::kWaveSize - 1), wave = tid >> 6, K = p.K;
  float row[DT];
  row[0] = x * p.inv_L;
  row[1] = y * p.inv_L;
  row[2] = v;
  row[3] = dir.x;
  row[4] = dir.y;
  row[5] = tagger ? 1.0f : 0.0f;
  row[6] = live == 1 ? 1.0f : 0.0f;
  row[7] = static_cast<float>(t) * p.inv_T;
  // no branch: an empty slot looks up the agent itself and is masked
  uint32_t pair[KT / 2];
#pragma unroll
  for (int k = 0; k < KT / 2; ++k) pair[k] = reinterpret_cast<const uint32_t*>(L.nearest + tid * KT)[k];
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const uint32_t j = (k & 1) ? pair[k >> 1] >> 16 : pair[k >> 1] & 0xFFFFu;
    const bool none = live != 1 || j == kNobody;
    const float4 o = L.me[none ? tid : int(j)];
    const float dx = o.x - x;
    const float dy = o.y - y;
    row[8 + 6 * k] = none ? 0.0f : dx * p.inv_L;
    row[9 + 6 * k] = none ? 0.0f : dy * p.inv_L;
    row[10 + 6 * k] = none ? 0.0f : o.z;
    row[11 + 6 * k] = none ? 0.0f : o.w;
    row[12 + 6 * k] = (!none && int(j) < p.N_tag) ? 1.0f : 0.0f;
    row[13 + 6 * k] = none ? 0.0f : 1.0f;
  }
  if (K == KT && ((reinterpret_cast<uintptr_t>(rows0) | reinterpret_cast<uintptr_t>(rows1)) & 15) == 0) {
    constexpr int S = stage_stride(KT), kPerRow = DT / 4, kPieces = kStageRows * kPerRow;
    constexpr int kRounds = (kPieces + wd::kWaveSize - 1) / wd::kWaveSize;
    float* const stage = L.stage + wave * (kStageRows * S);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if ((lane >> 5) == h) {
        float4* const dst = reinterpret_cast<float4*>(stage + (lane & 31) * S);
#pragma unroll
        for (int c = 0; c < kPerRow; ++c) dst[c] = make_float4(row[4 * c], row[4 * c + 1], row[4 * c + 2], row[4 * c + 3]);
      }
      wd::dev::wave_sync_lds();
      float4 q[kRounds];
#pragma unroll
      for (int it = 0; it < kRounds; ++it) {
        const int w = min(lane + it * wd::kWaveSize, kPieces - 1);
        q[it] = *reinterpret_cast<const float4*>(stage + (w / kPerRow) * S + 4 * (w % kPerRow));
      }
      const int first = wave * wd::kWaveSize + h * kStageRows;
      const int limit = min(p.N - first, kStageRows) * kPerRow - lane;  // pieces of these rows from this lane on
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        float* const rows = d ? rows1 : rows0;
        if (rows) {
          float4* const out = reinterpret_cast<float4*>(rows + int64_t(first) * DT) + lane;
#pragma unroll
          for (int it = 0; it < kRounds; ++it)
            if (it * wd::kWaveSize < limit) out[it * wd::kWaveSize] = q[it];
        }
      }
      wd::dev::wave_sync_lds();
    }
  } else if (tid < p.N) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      float* const rows = d ? rows1 : rows0;
      if (rows) {
        float2* const out = reinterpret_cast<float2*>(rows + int64_t(tid) * p.D);  // D is even, the arrays 8-byte aligned
#pragma unroll
        for (int c = 0; c < DT / 2; ++c)
          if (c < 4 + 3 * K) out[c] = make_float2(row[2 * c], row[2 * c + 1]);
      }
    }
  }
}

struct BlockArgs {  // the one kernel argument
  Params p;
  BlockPlan b;
  Roll roll;
  int32_t mode;
};

// The arguments are read through a pointer into the kernel-argument segment that is opaque to the
// optimiser from phase to phase: each phase then loads the fields it uses, instead of holding all of
// them in scalar registers over the loop (which spilled 180 of them).
typedef const __attribute__((address_space(4))) BlockArgs* KernargBlock;
#define WDC_NEW_PHASE() asm volatile("" : "+s"(ka))
#define p (((const BlockArgs*)ka)->p)
#define roll (((const BlockArgs*)ka)->roll)
#define plan (((const BlockArgs*)ka)->b)

template <int KT>
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(KT <= 4 ? 5 : 4, 8))) void block_kernel(
    const BlockArgs args) {
  extern __shared__ __align__(16) unsigned char smem[];
  KernargBlock ka = (KernargBlock)__builtin_amdgcn_kernarg_segment_ptr();  // args is at offset 0
  const int mode = ka->mode, steps = roll.steps;
  int tid = threadIdx.x;
  const int e = blockIdx.x, N = p.N;
  const bool valid = tid < N, tagger = tid < p.N_tag;
  const int64_t EN = int64_t(p.E) * N, a = int64_t(e) * N + (valid ? tid : 0);
  const bool stepping = (mode & kStep) != 0;
  int t = 0, nlr = 0, tags_last = 0;
  bool done = true;
  float x = 0.0f, y = 0.0f, v = 0.0f;
  int h = 0, live = 0;
  Probs10 next = {};  // those of the iteration to come: requested one iteration ahead
  if ((mode & kSample) && valid) next = load_probs(roll.ring + int64_t(roll.ring_pos % roll.ring_len) * EN * 10, a);
  if (!(mode & kResetAll)) {
    if (valid) {
      x = p.x[a];
      y = p.y[a];
      v = p.v[a];
      h = p.h[a];
      live = p.live[a];
    }
    done = p.done[e] != 0;
    t = p.t[e];
    nlr = p.n_live_runners[e];
    tags_last = p.tags_step[e];
    if ((mode == kStep && done) || (mode == kResetDone && !done)) return;  // this env keeps its state and rows
    if (done && roll.reward && valid) roll.reward[a] = p.reward[a];  // (an env that enters done: the first iteration does not step it)
  }
  float2 dir = make_float2(1.0f, 0.0f);
  if (live != 1) dir = p.table[wrap_heading(h, p.H)];  // (an agent in play looks its direction up when it moves)
  for (int s = 0; s < steps; ++s) {
    const bool last = s + 1 == steps;
    WDC_NEW_PHASE();
    asm volatile("" : "+v"(tid));  // likewise: what a thread derives from its number is derived in every iteration
    const BlockLds L(smem, plan, KT);
    const int lane = tid & (wd::kWaveSize - 1), wave = tid >> 6;
    int2 lv = make_int2(2, 2);
    if (mode & kSample) {
      const uint64_t g = roll.g0 + uint64_t(s);
      if (valid) {
        lv = draw_levels(p, next, e, tid, uint32_t(g), uint32_t(g >> 32));
        if (!last) next = load_probs(roll.ring + int64_t((roll.ring_pos + s + 1) % roll.ring_len) * EN * 10, a);
        if (last) *reinterpret_cast<int2*>(p.action + 2 * a) = lv;
        if (roll.action) *reinterpret_cast<int2*>(roll.action + int64_t(s) * 2 * EN + 2 * a) = lv;
      }
    } else if (stepping && valid) {
      lv = *reinterpret_cast<const int2*>(p.action + 2 * a);
    }
    int n = 0, slot = 0;
    Strips g = make_strips(p.L, plan.strip_scale, plan.strip_rmax, nlr + p.N_tag);
    if (stepping && !done) {
      if (valid && live == 1) advance_agent(p, tagger, lv.x, lv.y, x, y, v, h, dir);
      L.me[tid] = make_float4(x, y, v * dir.x, v * dir.y);
      L.tag_key[tid] = ~0ull;
      L.credits[tid] = 0;
      const bool in_play = valid && live == 1;
      n = build_list<KT>(p.L, plan.threads, L, g, tid, in_play, x, y, slot);
      WDC_NEW_PHASE();
      // ---- tag test: nearest tagger by (d2, index) ----------------------------------------------
      bool tagged_now = false;
      if (p.tag_r2 >= 0.0f) {
        const bool runner = in_play && !tagger;
        int tagged_by = 0;
        if (plan.tag_by_tagger) {
          if (tagger) reach_of_tagger(p, plan.tag_reach, L, g, tid, x, y);
          __syncthreads();
          if (runner) {
            const uint64_t key = L.tag_key[tid];
            tagged_now = key != ~0ull;
            tagged_by = int(uint32_t(key));
          }
        } else if (runner) {
          float best = 0.0f;
          for (int k = 0; k < p.N_tag; ++k) {
            const float4 o = L.me[k];
            const float d2 = squared_distance(x, y, o.x, o.y);
            if (k == 0 || d2 < best) {
              best = d2;
              tagged_by = k;
            }
          }
          tagged_now = best <= p.tag_r2;
        }
        if (tagged_now) {
          live = 0;
          L.list[slot].y = kGone;
          L.ids[slot] = uint16_t(tid) | kGoneId;
          atomicAdd(&L.credits[tagged_by], 1);
          atomicAdd(&L.misc[kTags], 1);
        }
        __syncthreads();
      }
      WDC_NEW_PHASE();
      // ---- rewards, clock, end of episode ---------------------------------------------------------
      if (valid) {
        const float rew = tagger ? static_cast<float>(L.credits[tid]) * p.tag_reward : tagged_now ? p.tag_penalty : 0.0f;
        if (last) p.reward[a] = rew;
        if (roll.reward) roll.reward[int64_t(s) * EN + a] = rew;
      }
      tags_last = L.misc[kTags];
      nlr -= tags_last;
      t += 1;
      done = nlr == 0 || t >= p.T;
    }
    if (roll.done && tid == 0) roll.done[int64_t(s) * p.E + e] = done ? 1 : 0;  // the flag before the reset
    if ((mode & (kResetDone | kResetAll)) && done) {  // back to the start state
      if (valid) {
        x = p.x0[a];
        y = p.y0[a];
        h = wrap_heading(p.h0[a], p.H);
        live = 1;
      }
      v = 0.0f;
      dir = p.table[h];
      t = 0;
      nlr = N - p.N_tag;
      tags_last = 0;
      done = false;
      g = make_strips(p.L, plan.strip_scale, plan.strip_rmax, N);
      __syncthreads();  // the step's tables have been read
      L.me[tid] = make_float4(x, y, v * dir.x, v * dir.y);
      n = build_list<KT>(p.L, plan.threads, L, g, tid, valid, x, y, slot);
    }
    __syncthreads();  // credits have been read: the neighbour lists may overlay them
    WDC_NEW_PHASE();
    // ---- the nearest agents in play, in list order --------------------------------------------------
    const bool stray = L.misc[kStray] != 0;  // an agent off the world: every list is searched whole
    if (tid < n && !(L.ids[tid] & kGoneId)) {
      float limit = __uint_as_float(0x7F800000u);
      if (stray || !search_windows<KT>(L, g, tid, n, &limit)) {
        const int at = atomicAdd(&L.misc[kQueued], 1);
        L.queue[at] = uint16_t(tid);
        L.limit[at] = limit;
      }
    }
    __syncthreads();
    const int queued = L.misc[kQueued];
    const int waves = plan.threads / wd::kWaveSize;
    // a crowd: a lane each is faster than groups of sixteen lanes one after the other (uniform)
    const bool all_open = 2 * queued > n && queued * kCrowdCost > n * waves * (8 + 4 * KT);
    if (!all_open) search_queue<KT>(L, g, n, queued, lane, wave, waves);
    __syncthreads();
    const int open = all_open ? 0 : L.misc[kOpen];
    if (all_open) {
      if (tid < queued) search_by_lane<KT>(L, L.queue[tid], n);
      __syncthreads();
    } else if (open != 0) {
      search_open<KT>(L, n, queued, open, tid, waves);
      __syncthreads();
    }
    WDC_NEW_PHASE();
    store_rows<KT>(p, L, last ? p.obs + int64_t(e) * N * p.D : nullptr,
                   roll.obs ? roll.obs + (int64_t(s) * EN + int64_t(e) * N) * p.D : nullptr, tid, x, y, v, dir, tagger,
                   live, t);
    __syncthreads();  // the rows are out before the next iteration overwrites the tables
  }
  if (valid) {
    p.x[a] = x;
    p.y[a] = y;
    p.v[a] = v;
    p.h[a] = h;
    p.live[a] = live;
    if (tid == 0) {
      p.t[e] = t;
      p.n_live_runners[e] = nlr;
      p.tags_step[e] = tags_last;
      p.done[e] = done ? 1 : 0;
    }
  }
}

#undef p
#undef roll
#undef plan
#undef WDC_NEW_PHASE

}  // namespace
}  // namespace wdc

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
struct wdc_handle {
  wdc_config cfg;
  wdc_buffers bufs;
  wdc::Params params;
  wdc::BlockPlan block;
  hipStream_t stream;
  uint64_t g;
  bool started;
  void* table;
  std::string last_error;
};

namespace {

int check_config(const wdc_config* c) {
  if (!c) return WD_E_NULL;
  if (c->struct_size != sizeof(wdc_config)) return WD_E_CONFIG;
  if (c->num_envs < 1 || c->env_offset < 0) return WD_E_CONFIG;
  if (c->num_agents < 2 || c->num_agents > wdc::kMaxThreads) return WD_E_CONFIG;
  if (c->num_taggers < 1 || c->num_taggers > c->num_agents - 1) return WD_E_CONFIG;
  if (c->num_headings < 4 || c->num_headings > 4096 || c->num_headings % 4 != 0) return WD_E_CONFIG;
  if (c->episode_length < 1) return WD_E_CONFIG;
  if (c->obs_k < 0 || c->obs_k > wdc::kMaxK || c->obs_k > c->num_agents - 1) return WD_E_CONFIG;
  if (!(c->world_size > 0.0f) || std::isinf(c->world_size)) return WD_E_CONFIG;
  const float fields[] = {c->accel, c->max_speed_tagger, c->max_speed_runner, c->tag_r2, c->tag_reward, c->tag_penalty};
  for (float f : fields)
    if (!(f == f) || std::isinf(f)) return WD_E_CONFIG;
  if (c->accel < 0.0f || c->max_speed_tagger < 0.0f || c->max_speed_runner < 0.0f) return WD_E_CONFIG;
  if (int64_t(c->num_envs) * c->num_agents > int64_t(INT32_MAX) / 2) return WD_E_CONFIG;
  return WD_OK;
}

// The heading table: the first octant from double-precision cos / sin rounded to float32, the
// rest by reflection about the diagonal and by quarter turns; zeros are +0.
std::vector<float2> heading_table(int H) {
  std::vector<float2> t(H);
  const int quarter = H / 4;
  const double pi = 3.14159265358979323846;
  for (int h = 0; h < H; ++h) {
    const int turns = h / quarter;
    int r = h % quarter;
    const bool reflect = 2 * r > quarter;
    if (reflect) r = quarter - r;
    const double angle = 2.0 * pi * double(r) / double(H);
    float c = float(std::cos(angle)), s = float(std::sin(angle));
    if (2 * r == quarter) s = c;
    if (reflect) std::swap(c, s);
    for (int k = 0; k < turns; ++k) {  // a quarter turn to the left
      const float old_c = c;
      c = -s;
      s = old_c;
    }
    t[h] = make_float2(c + 0.0f, s + 0.0f);  // (-0) + 0 = +0
  }
  return t;
}

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

int fail_hip(wdc_handle* h, hipError_t err, const char* what) {
  h->last_error = std::string(what) + ": " + hipGetErrorString(err);
  return WD_E_HIP;
}

// four float and two int arrays of one element per thread, one int per env of the workgroup
size_t lds_bytes(const wdc::Params& p) { return size_t(p.threads) * 24 + size_t(p.threads / 2) * 4; }

constexpr int kBlockAbove = 32;  // agents per env

// One workgroup per env (block_kernel) serves envs of more than 32 agents: geometry of the list, form of the
// tag check, LDS map.  Smaller envs share a workgroup, and comparing all pairs is the shorter chain; without
// neighbours there is nothing to search; and outside a world of ordinary size the search's bounds (squares
// of distances as float32) have no room.  Measured, us per iteration, all pairs -> block_kernel (K = 4):
// 300 x 20 8.1 -> 9.7, 4000 x 20 12.6 -> 14.6; 10 x 33 9.6 -> 8.9, 4000 x 33 16.4 -> 16.0 (four recorded iterations of
// 300 x 33 40.4 -> 29.5); 2000 x 48 16.1 -> 14.8, K = 8 22.5 -> 17.5; 10 x 64 13.8 -> 10.1, 4000 x 64 26.5 -> 20.1.
void plan_block(const wdc::Params& p, wdc::BlockPlan* b) {
  *b = wdc::BlockPlan{};
  if (p.N <= kBlockAbove || p.K < 1 || p.L < 1e-3f || p.L > 1e6f) return;
  b->threads = (p.N + 63) / 64 * 64;
  b->kt = p.K <= 2 ? 2 : p.K <= 4 ? 4 : p.K <= 6 ? 6 : 8;
  const int nt = b->threads, waves = nt / wd::kWaveSize, pad = wdc::list_pad(b->kt);
  // strips about 1.5 expected K-th-neighbour distances tall: L / R = 1.5 L sqrt(K / (pi n))
  b->strip_scale = float(std::sqrt(3.14159265358979 / double(b->kt)) / 1.5);
  b->strip_rmax = int(double(b->strip_scale) * std::sqrt(double(p.N)) + 0.5) + 1;
  const double reach = p.tag_r2 > 0.0f ? std::sqrt(double(p.tag_r2)) : 0.0, L = p.L;
  b->tag_reach = float(std::min(reach, 4.0 * L) * 1.00001 + 4e-6 * L);
  // The tag check is one lane's chain either way: a runner's over all taggers (8 instructions each), or a
  // tagger's over the bins its reach touches (30 instructions per strip, 12 per agent in them).
  const double box = std::min(1.0, 2.0 * reach / L);
  const double by_tagger = 30.0 * (box * b->strip_rmax + 1.0) + 12.0 * box * box * p.N;
  b->tag_by_tagger = 8.0 * p.N_tag > by_tagger ? 1 : 0;
  int at = 0;
  auto take = [&at](int bytes) {
    const int here = at;
    at = (at + bytes + 15) / 16 * 16;
    return here;
  };
  take(16 * nt);
  b->off_misc = take(4 * wdc::kMiscWords);
  b->off_tag = b->off_near = take(std::max(12 * nt, (6 + 2 * b->kt) * nt));
  b->off_list = b->off_stage = take(8 * (nt + 2 * pad));
  b->off_ids = take(2 * nt);
  b->off_table = take(2 * (b->strip_rmax * wdc::kColumns + 2));
  b->off_found = take(8 * nt);
  b->lds = std::max(at, b->off_stage + 4 * wdc::kStageRows * wdc::stage_stride(b->kt) * waves);
}

template <int KT>
hipError_t launch_block_variant(const wdc_handle* h, const wdc::Roll& roll, int mode) {
  const wdc::BlockPlan& b = h->block;
  hipLaunchKernelGGL(wdc::block_kernel<KT>, dim3(h->params.E), dim3(b.threads), size_t(b.lds), h->stream,
                     wdc::BlockArgs{h->params, b, roll, mode});
  return hipGetLastError();
}

int launch_block(wdc_handle* h, const wdc::Roll& roll, int mode) {
  hipError_t err;
  switch (h->block.kt) {
    case 2: err = launch_block_variant<2>(h, roll, mode); break;
    case 4: err = launch_block_variant<4>(h, roll, mode); break;
    case 6: err = launch_block_variant<6>(h, roll, mode); break;
    default: err = launch_block_variant<8>(h, roll, mode); break;
  }
  return err == hipSuccess ? WD_OK : fail_hip(h, err, "block_kernel launch");
}

// More than the 64 KB of LDS that a launch may ask for by default: granted once per kernel function.
hipError_t grant_block_lds(const wdc::BlockPlan& b) {
  if (b.lds <= 64 * 1024) return hipSuccess;
  const void* kernel = b.kt == 2   ? reinterpret_cast<const void*>(wdc::block_kernel<2>)
                       : b.kt == 4 ? reinterpret_cast<const void*>(wdc::block_kernel<4>)
                       : b.kt == 6 ? reinterpret_cast<const void*>(wdc::block_kernel<6>)
                                   : reinterpret_cast<const void*>(wdc::block_kernel<8>);
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

int launch(wdc_handle* h, int mode, const float* probs) {
  const wdc::Params& p = h->params;
  if (h->block.kt && mode != wdc::kSample) {
    wdc::Roll one = {};
    one.steps = 1;
    one.ring_len = 1;
    one.ring = probs;
    one.g0 = h->g;
    return launch_block(h, one, mode);
  }
  const int groups = (p.E + p.envs_per_wg - 1) / p.envs_per_wg;
  if (p.K <= 4)
    hipLaunchKernelGGL(wdc::env_kernel<4>, dim3(groups), dim3(p.threads), lds_bytes(p), h->stream, p, mode, probs,
                       uint32_t(h->g), uint32_t(h->g >> 32));
  else
    hipLaunchKernelGGL(wdc::env_kernel<wdc::kMaxK>, dim3(groups), dim3(p.threads), lds_bytes(p), h->stream, p, mode, probs,
                       uint32_t(h->g), uint32_t(h->g >> 32));
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail_hip(h, err, "env_kernel launch");
  return WD_OK;
}

}  // namespace

extern "C" {

int wdc_query_layout(const wdc_config* cfg, wdc_layout* out) {
  if (!cfg || !out) return WD_E_NULL;
  const int rc = check_config(cfg);
  if (rc != WD_OK) return rc;
  const int64_t EN = int64_t(cfg->num_envs) * cfg->num_agents;
  out->obs_dim = 8 + 6 * cfg->obs_k;
  out->agent_elems = EN;
  out->action_elems = 2 * EN;
  out->obs_elems = EN * out->obs_dim;
  out->env_elems = cfg->num_envs;
  out->probs_elems = 10 * EN;
  // 40 probabilities, 20 state read, 20 state written, 8 actions, 4 reward, 4 D row; 24 per env
  out->bytes_per_iteration = EN * (40 + 20 + 20 + 8 + 4 + 4 * int64_t(out->obs_dim)) + 24 * int64_t(cfg->num_envs);
  return WD_OK;
}

int wdc_create(const wdc_config* cfg, const wdc_buffers* bufs, wdc_handle** out) {
  if (!cfg || !bufs || !out) return WD_E_NULL;
  *out = nullptr;
  const int rc = check_config(cfg);
  if (rc != WD_OK) return rc;
  const void* ptrs[] = {bufs->x, bufs->y, bufs->v, bufs->h, bufs->x0, bufs->y0, bufs->h0, bufs->live,
                        bufs->action, bufs->reward, bufs->obs, bufs->t, bufs->done, bufs->n_live_runners,
                        bufs->tags_step};
  for (const void* q : ptrs) {
    if (!q) return WD_E_NULL;
    if (!aligned(q, 256)) return WD_E_ALIGN;
  }
  wdc_handle* h = new (std::nothrow) wdc_handle();
  if (!h) return WD_E_HIP;
  h->cfg = *cfg;
  h->bufs = *bufs;
  h->stream = static_cast<hipStream_t>(cfg->stream);
  h->g = 0;
  h->started = false;
  h->table = nullptr;
  wdc::Params& p = h->params;
  p.E = cfg->num_envs;
  p.N = cfg->num_agents;
  p.N_tag = cfg->num_taggers;
  p.H = cfg->num_headings;
  p.T = cfg->episode_length;
  p.K = cfg->obs_k;
  p.D = 8 + 6 * cfg->obs_k;
  // (envs that fit a wave, in a batch of at most a quarter of a million agents: workgroups of one wave,
  // whose barriers cost nothing and which spread over more compute units)
  p.threads = (p.N <= 64 && int64_t(p.E) * p.N <= 262144) ? 64 : (p.N <= 256 ? 256 : (p.N + 63) / 64 * 64);
  p.envs_per_wg = p.threads / p.N;
  p.env_offset = uint32_t(cfg->env_offset);
  p.seed_lo = uint32_t(cfg->seed);
  p.seed_hi = uint32_t(cfg->seed >> 32);
  p.div_N = wd::make_fastdiv(uint32_t(p.N));
  p.L = cfg->world_size;
  p.inv_L = float(1.0 / double(cfg->world_size));
  p.inv_T = float(1.0 / double(cfg->episode_length));
  p.accel = cfg->accel;
  p.vmax_tagger = cfg->max_speed_tagger;
  p.vmax_runner = cfg->max_speed_runner;
  p.tag_r2 = cfg->tag_r2;
  p.tag_reward = cfg->tag_reward;
  p.tag_penalty = cfg->tag_penalty;
  p.x = bufs->x; p.y = bufs->y; p.v = bufs->v; p.h = bufs->h;
  p.x0 = bufs->x0; p.y0 = bufs->y0; p.h0 = bufs->h0;
  p.live = bufs->live; p.action = bufs->action; p.reward = bufs->reward; p.obs = bufs->obs;
  p.t = bufs->t; p.done = bufs->done; p.n_live_runners = bufs->n_live_runners; p.tags_step = bufs->tags_step;
  plan_block(p, &h->block);
  const std::vector<float2> table = heading_table(p.H);
  hipError_t err = h->block.kt ? grant_block_lds(h->block) : hipSuccess;
  if (err == hipSuccess) err = hipMalloc(&h->table, sizeof(float2) * table.size());
  if (err == hipSuccess) err = hipMemcpy(h->table, table.data(), sizeof(float2) * table.size(), hipMemcpyHostToDevice);
  if (err != hipSuccess) {
    if (h->table) (void)hipFree(h->table);
    delete h;
    return WD_E_HIP;
  }
  p.table = static_cast<const float2*>(h->table);
  *out = h;
  return WD_OK;
}

int wdc_reset(wdc_handle* h, int mode) {
  if (!h) return WD_E_NULL;
  if (mode != WD_RESET_ALL && mode != WD_RESET_DONE) return WD_E_CONFIG;
  if (mode == WD_RESET_DONE) {
    if (!h->started) return WD_E_STATE;
    return launch(h, wdc::kResetDone, nullptr);
  }
  const int64_t agents = int64_t(h->params.E) * h->params.N;
  hipLaunchKernelGGL(wdc::init_kernel, dim3(uint32_t((agents + 255) / 256)), dim3(256), 0, h->stream, h->params);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail_hip(h, err, "init_kernel launch");
  h->g = 0;
  const int rc = launch(h, wdc::kResetAll, nullptr);
  if (rc == WD_OK) h->started = true;
  return rc;
}

int wdc_sample(wdc_handle* h, const float* probs) {
  if (!h || !probs) return WD_E_NULL;
  if (!aligned(probs, 8)) return WD_E_ALIGN;
  if (!h->started) return WD_E_STATE;
  return launch(h, wdc::kSample, probs);
}

int wdc_step(wdc_handle* h) {
  if (!h) return WD_E_NULL;
  if (!h->started) return WD_E_STATE;
  const int rc = launch(h, wdc::kStep, nullptr);
  if (rc == WD_OK) ++h->g;
  return rc;
}

int wdc_iterate(wdc_handle* h, const float* probs) {
  if (!h || !probs) return WD_E_NULL;
  if (!aligned(probs, 8)) return WD_E_ALIGN;
  if (!h->started) return WD_E_STATE;
  const int rc = launch(h, wdc::kSample | wdc::kStep | wdc::kResetDone, probs);
  if (rc == WD_OK) ++h->g;
  return rc;
}

int wdc_rollout(wdc_handle* h, const float* probs_ring, int ring_len, int k, const wdc_rollout_buffers* out) {
  if (!h || !probs_ring) return WD_E_NULL;
  if (ring_len < 1 || k < 1) return WD_E_CONFIG;
  if (!aligned(probs_ring, 8)) return WD_E_ALIGN;
  if (out) {
    const void* ptrs[] = {out->action, out->reward, out->done, out->obs};
    for (const void* q : ptrs)
      if (!aligned(q, 8)) return WD_E_ALIGN;
  }
  if (!h->started) return WD_E_STATE;
  const wdc::Params& p = h->params;
  wdc::Roll roll = {};
  roll.steps = k;
  roll.ring_len = ring_len;
  roll.ring_pos = int32_t(h->g % uint64_t(ring_len));
  roll.ring = probs_ring;
  roll.g0 = h->g;
  if (out) {
    roll.action = out->action;
    roll.reward = out->reward;
    roll.done = out->done;
    roll.obs = out->obs;
  }
  if (h->block.kt) {  // (writes the last iteration to the in-place arrays and to its slices)
    const int rc = launch_block(h, roll, wdc::kSample | wdc::kStep | wdc::kResetDone);
    if (rc == WD_OK) h->g += uint64_t(k);
    return rc;
  }
  const int groups = (p.E + p.envs_per_wg - 1) / p.envs_per_wg;
  if (p.K <= 4)
    hipLaunchKernelGGL(wdc::rollout_kernel<4>, dim3(groups), dim3(p.threads), lds_bytes(p), h->stream, p, roll);
  else
    hipLaunchKernelGGL(wdc::rollout_kernel<wdc::kMaxK>, dim3(groups), dim3(p.threads), lds_bytes(p), h->stream, p, roll);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail_hip(h, err, "rollout_kernel launch");
  if (out) {  // the last iteration wrote the in-place arrays: its slices are copies of them
    const int64_t EN = int64_t(p.E) * p.N, last = int64_t(k - 1);
    if (out->action && err == hipSuccess)
      err = hipMemcpyAsync(out->action + last * 2 * EN, h->bufs.action, size_t(2 * EN) * 4, hipMemcpyDeviceToDevice, h->stream);
    if (out->reward && err == hipSuccess)
      err = hipMemcpyAsync(out->reward + last * EN, h->bufs.reward, size_t(EN) * 4, hipMemcpyDeviceToDevice, h->stream);
    if (out->obs && err == hipSuccess)
      err = hipMemcpyAsync(out->obs + last * EN * p.D, h->bufs.obs, size_t(EN * p.D) * 4, hipMemcpyDeviceToDevice, h->stream);
    if (err != hipSuccess) return fail_hip(h, err, "copy of the last roll-out slice");
  }
  h->g += uint64_t(k);
  return WD_OK;
}

int wdc_get_step(const wdc_handle* h, uint64_t* g) {
  if (!h || !g) return WD_E_NULL;
  *g = h->g;
  return WD_OK;
}

int wdc_set_step(wdc_handle* h, uint64_t g) {
  if (!h) return WD_E_NULL;
  h->g = g;
  return WD_OK;
}

int wdc_destroy(wdc_handle* h) {
  if (!h) return WD_OK;
  if (h->table) (void)hipFree(h->table);
  delete h;
  return WD_OK;
}

const char* wdc_last_error(const wdc_handle* h) { return h ? h->last_error.c_str() : ""; }

}  // extern "C"
