// wd_api.hip — host side of libwd: the C ABI of include/wd.h, configuration checks,
// launch geometry and LDS map, and the calls into the launchers of wd_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>

#include "../../include/wd.h"
#include "wd_internal.h"

struct wd_handle {
  wd_config cfg;
  wd_buffers bufs;
  wd::Params params;
  hipStream_t stream;
  uint64_t g;          // global step: RNG step index
  bool started;        // wd_reset(WD_RESET_ALL) has run
  bool rows_valid;     // bufs.obs holds the rows this library wrote for the current state
  void* scratch;       // device memory of the large-env tables (NULL for the small layout)
  // roll-outs of the large-env layout: a second stream for the observation kernels, a second
  // table image and two events per image (created by the first such roll-out, freed by wd_destroy)
  hipStream_t obs_stream;
  hipEvent_t tables_ready[2], rows_done[2];
  void* second_image;
  bool pipe_ready;
  std::string last_error;
};

namespace {

// LDS of one gfx950 compute unit, less the 256 bytes of static LDS the env kernels carry (the
// workgroup votes of __syncthreads_and / __syncthreads_or): what a launch may ask for dynamically
constexpr int64_t kLdsLimitBytes = 160 * 1024 - 256;
constexpr int kMaxAgents = 32768;
constexpr int kMaxGrid = 32767;
// spread form of the large-env pair: while its observation kernel has a compute unit per workgroup to spare
constexpr int kSpreadMaxWorkgroups = 192;
constexpr int kSpreadMinAgents = 1024;
// envs: one round of waves on the chip (256 compute units x 32 waves)
constexpr int kWaveEnvsMaxBatch = 8192;
// threads that a launch may have at most (one more and their number wraps, without an error)
constexpr int64_t kMaxLaunchThreads = (int64_t(1) << 32) - 1;

int bits_for(uint32_t v) {  // bits needed to hold values 0..v
  int b = 1;
  while ((uint64_t(1) << b) <= v) ++b;
  return b;
}

uint32_t pow2_ceil(uint32_t v) {
  uint32_t r = 1;
  while (r < v) r <<= 1;
  return r;
}

int32_t isqrt64(int64_t v) {
  int64_t r = int64_t(std::sqrt(double(v)));
  while (r * r > v) --r;
  while ((r + 1) * (r + 1) <= v) ++r;
  return int32_t(r);
}

int64_t align16(int64_t v) { return (v + 15) & ~int64_t(15); }

int check_config(const wd_config* c) {
  if (!c) return WD_E_NULL;
  if (c->struct_size != sizeof(wd_config)) return WD_E_CONFIG;
  if (c->num_envs < 1 || c->env_offset < 0) return WD_E_CONFIG;
  if (int64_t(c->num_envs) + int64_t(c->env_offset) > int64_t(INT32_MAX)) return WD_E_CONFIG;
  if (c->num_agents < 2 || c->num_agents > kMaxAgents) return WD_E_CONFIG;
  if (c->num_taggers < 1 || c->num_taggers > c->num_agents - 1) return WD_E_CONFIG;
  if (c->grid_size < 1 || c->grid_size > kMaxGrid) return WD_E_CONFIG;
  if (c->num_actions != wd::kNumActions) return WD_E_CONFIG;
  if (c->episode_length < 1) return WD_E_CONFIG;
  if (c->obs_mode != WD_OBS_PARTIAL && c->obs_mode != WD_OBS_FULL) return WD_E_CONFIG;
  if (c->obs_mode == WD_OBS_PARTIAL && (c->obs_k < 0 || c->obs_k > c->num_agents - 1)) return WD_E_CONFIG;
  if (!(c->tag_reward == c->tag_reward) || !(c->tag_penalty == c->tag_penalty)) return WD_E_CONFIG;  // NaN
  if (int64_t(c->num_envs) * c->num_agents > int64_t(INT32_MAX)) return WD_E_CONFIG;
  return WD_OK;
}

int32_t obs_dim(const wd_config* c) {
  return c->obs_mode == WD_OBS_PARTIAL ? 5 + 4 * c->obs_k : 5 + 4 * c->num_agents;
}

bool aligned256(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255u) == 0; }

// probs is read with aligned 16-byte loads when N % 4 == 0, else with loads that need 4-byte alignment
bool probs_aligned(const wd::Params& p, const void* probs) {
  return (reinterpret_cast<uintptr_t>(probs) & (p.vec4 ? 15u : 3u)) == 0;
}

// LDS map of the strip variant: per team a kept part (positions by index, scalars, strip edges),
// an X part (the padded strip-sorted list and the table of bin starts) that the row staging area
// overlays once the neighbour search is done, and a Y part (slots, tag keys, credits) that the
// retry queue and the neighbour lists overlay once the rewards are out.  The columns are as narrow
// as the table's share of LDS allows without costing the launch a workgroup per CU.
bool plan_strip_layout(const wd_config& c, wd::Params* p) {
  const int N = c.num_agents, G = c.grid_size, K = p->K;
  const int64_t NPAD = p->NPAD;
  const int tpw = p->teams_per_wg;
  // strips about 1.5 expected K-th-neighbour distances tall: G / R = 1.5 G sqrt(K / (pi n))
  const int KS = wd::strip_list_size(K);
  p->strip_scale = float(std::sqrt(3.14159265358979 / double(KS)) / 1.5);
  // the own window overhangs the list by up to its half width, and the window of a neighbouring strip then sits beyond it
  p->pad_l = wd::strip_pad(KS);
  p->pad_r = wd::strip_pad(KS);
  const int64_t slots = NPAD + p->pad_l + p->pad_r;
  const int r_want = std::min<int64_t>(G, int64_t(std::ceil(double(p->strip_scale) * std::sqrt(double(N)))) + 1);
  const int64_t waves = p->wg_size / wd::kWaveSize;
  int srl = 5;  // rows per wave and flush of the staging area: 32, or 16 if an env does not fit otherwise
  const int64_t nbr_bytes = align16((K == 4 && N < 1024) ? 5 * NPAD : 2 * NPAD * K);
  const int64_t retry_bytes = align16(2 * NPAD);
  auto layout = [&](int cshift, bool commit) -> int64_t {
    const int64_t stage = waves * (int64_t(1) << srl) * p->D * 4;
    const int C = ((G - 1) >> cshift) + 1;
    const int64_t entries = int64_t(r_want) * C + 1;
    int64_t off = 0;
    auto take = [&off](int64_t bytes) {
      const int64_t at = off;
      off = align16(off + bytes);
      return int32_t(at);
    };
    const int32_t o_pl = take(4 * NPAD), o_misc = take(128), o_edges = take(2 * (r_want + 2));
    const int64_t keep = off;
    off = 0;
    const int32_t o_sorted = take(4 * slots), o_id = take(2 * slots), o_t = take(2 * (entries + 1));
    const int64_t x_stride = off;
    off = 0;
    const int32_t o_slot = take(2 * NPAD), o_best = take(4 * NPAD), o_credits = take(4ll * c.num_taggers);
    const int64_t y_tables = off;
    const int64_t x_area = x_stride * tpw;
    int64_t x_span, y_stride;
    if (tpw == 1) {
      x_span = x_area;
      y_stride = align16(std::max<int64_t>(std::max<int64_t>(y_tables, retry_bytes + nbr_bytes), stage + nbr_bytes - x_area));
    } else {
      x_span = std::max<int64_t>(x_area, stage);
      y_stride = align16(std::max<int64_t>(y_tables, retry_bytes + nbr_bytes));
    }
    const int64_t total = keep * tpw + x_span + y_stride * tpw;
    if (commit) {
      p->cshift = cshift;
      p->strip_C = C;
      p->strip_rmax = r_want;
      p->off_pl = o_pl;
      p->off_misc = o_misc;
      p->off_edges = o_edges;
      p->keep_stride = int32_t(keep);
      p->off_sorted = o_sorted + 4 * p->pad_l;
      p->off_sorted_id = o_id + 2 * p->pad_l;
      p->off_starts = o_t;
      p->x_stride = int32_t(x_stride);
      p->off_slot = o_slot;
      p->off_best = o_best;
      p->off_credits = o_credits;
      p->off_counts = 0;
      p->off_retry = 0;
      p->compact_nbr = (K == 4 && N < 1024) ? 1 : 0;
      p->stage_rows_log2 = srl;
      p->y_stride = int32_t(y_stride);
      p->off_nbr = int32_t(y_stride - nbr_bytes);
      p->x_base = int32_t(keep * tpw);
      p->y_base = int32_t(p->x_base + x_span);
      p->lds_bytes = int32_t(std::min<int64_t>(total, INT32_MAX));
      p->g_stride_image = p->y_base;
    }
    return total;
  };
  // the share of LDS that keeps as many workgroups on a CU as the coarsest columns would
  int64_t total_min = layout(15, false);
  if (total_min > kLdsLimitBytes) {
    srl = 4;
    total_min = layout(15, false);
  }
  if (total_min > kLdsLimitBytes) return false;
  const int64_t by_threads = std::max<int64_t>(1, 2048 / p->wg_size);
  const int64_t wgs = std::max<int64_t>(1, std::min<int64_t>(by_threads, kLdsLimitBytes / total_min));
  const int64_t budget = kLdsLimitBytes / wgs;
  int cshift = 0;
  while (cshift < 15 && layout(cshift, false) > budget) ++cshift;
  layout(cshift, true);
  return true;
}

// The strip search keeps the positions of its list scaled by 2^h per axis (2 h >= idx_bits), so that the
// squared length of a packed 16-bit difference is the key's distance part where it belongs; an entry out of
// play has y field 0x7FFF.  That needs room in 16 bits: the keys of such entries, at least (32767 - A)^2 with
// A = (G - 1) << h, must lie above every key of a live pair, below 2 A^2 + 2^(2 h).
bool strip_positions_fit(int idx_bits, int G, int* h, uint32_t* dead_key_min) {
  *h = (idx_bits + 1) / 2;
  const int64_t A = int64_t(G - 1) << *h;
  const int64_t dead_min = A < 32767 ? (32767 - A) * (32767 - A) : 0;
  *dead_key_min = uint32_t(dead_min);
  return A < 32767 && 2 * A * A + (int64_t(1) << (2 * *h)) <= dead_min;
}

// Launch geometry and LDS map of the env-per-team kernels.  Returns false if an env does
// not fit one workgroup's LDS.
// (`big_tables_in_lds`: a large env also keeps slots, tag keys and credits in LDS when they fit; `max_log2`:
// the widest workgroup of the small layout)
bool plan_env_kernels(const wd_config& c, wd::Params* p, bool big, bool big_tables_in_lds = false, int max_log2 = 10) {
  const int N = c.num_agents, G = c.grid_size;
  // the variants with K = 1 .. 16, small layout, sort by strip where the scaled positions fit
  p->idx_bits = bits_for(uint32_t(N - 1));
  int strip_h = 0;
  uint32_t strip_dead_key_min = 0;
  const bool strips = !big && c.obs_mode == WD_OBS_PARTIAL && p->K >= 1 && p->K <= wd::kMaxRegisterK2 &&
                      strip_positions_fit(p->idx_bits, G, &strip_h, &strip_dead_key_min);
  p->NG = (N + 3) / 4;
  p->big = big ? 1 : 0;
  int ts_log2 = 3;
  while ((1 << ts_log2) < p->NG && ts_log2 < 8) ++ts_log2;
  // A batch that cannot fill the chip is bound by the latency of one workgroup's chain of
  // phases, not by throughput: give each env more lanes (fewer search rounds per lane) and each
  // workgroup fewer envs (fewer row chunks per wave) while that still shortens the chain.
  while (!big && ts_log2 < 8) {
    const int ts_now = 1 << ts_log2, tpw_now = 256 / ts_now;
    const int64_t waves_if_doubled = int64_t(c.num_envs) * std::max(1, 2 * ts_now / wd::kWaveSize);
    const int64_t rows_per_wg = int64_t(std::min(tpw_now, c.num_envs)) * N;
    // 8192 wave slots on the chip: beyond that, wider teams only add rounds of workgroups
    // (and up to a whole wave per team in any case: the strip search serves the teams of a wave one
    // after the other; a batch of at most one workgroup per CU gets a workgroup per env, whose
    // kernel variant keeps everything that depends on the team in scalar registers:
    // 10 envs x 5 agents 13.1 -> 11.7 us per iteration, 11.6 -> 8.1 inside a roll-out)
    const int min_width = c.num_envs <= 256 ? 256 : wd::kWaveSize;
    if (waves_if_doubled > 8192 || (rows_per_wg <= 64 && N <= ts_now && ts_now >= min_width)) break;
    ++ts_log2;
  }
  p->wg_size = 256;
  // Wider workgroups.  A batch of up to a thousand envs of more than 256 agents is bound by one workgroup's
  // chain of phases, which more lanes shorten; and an env of more than 1024 agents takes more LDS than lets
  // eight 256-thread workgroups share a CU, so that wider ones keep the CU's wave slots filled.
  // Measured, us per iteration, 256 / 512 / 1024 threads.  Strips: K = 4: 10 x 333 18.1 / 17.4 / -,
  // 450 x 333 23.1 / 22.4, 777 x 333 25.3 / 25.4; 10 x 700 19.2 / 17.8 / 18.2, 300 x 1000 26.9 / 24.7 / 26.1,
  // 777 x 1000 34.9 / 33.8; 200 x 1300 - / 25.5 / 24.6, 450 x 1300 - / 31.0 / 31.5; 200 x 2000 - / 30.1 / 28.5,
  // 777 x 2000 - / 67.5 / 69.5; 460 x 2600 - / 93.4 / 49.3, 1500 x 2600 - / 178 / 130; K = 8: 450 x 1000 38.6 / 35.8,
  // 777 x 1000 49.2 / 62.6; K = 12: 200 x 1000 51.7 / 40.7, 500 x 1000 62.3 / 76.6.
  // Bucket rings (larger grids): K = 4: 250 x 300 36.5 / 30.7, 500 x 500 45.2 / 42.7, 1000 x 700 70.5 / 80.4,
  // 460 x 1100 - / 62.0 / 83.8, 460 x 2800 - / 113 / 130; K = 16: 250 x 300 170 / 131, 500 x 500 225 / 295.
  // No list in registers: K = 17: 20 x 300 99.7 / 81.9 (not taken), 200 x 1100 - / 154 / 129, 800 x 1100 - / 284 / 300,
  // 500 x 3000 (K = 20) - / 1897 / 1789; K = 0: 600 x 2600 - / 42.8 / 48.2; full views 20 x 1100 - / 32.0 / 33.0.
  if (!big && N > 256 && ts_log2 <= 8) {
    const bool partial = c.obs_mode == WD_OBS_PARTIAL;
    const int K = p->K;
    if (N > 3072) {
      ts_log2 = 10;
    } else if (N > 1024) {
      ts_log2 = 9;
      if (strips || (partial && K > wd::kMaxRegisterK2)) {
        if (c.num_envs <= 256) ts_log2 = 10;
        // a CU holds three 512-thread workgroups of such an env at most, but two of 1024 threads.  Only where the
        // kernel's registers leave room for more waves than two workgroups of 512 threads have: K = 2 .. 4, not
        // K = 1 and K > 4 (1500 x 2600, 512 / 1024 threads: K = 1 92.2 / 124, K = 6 168 / 188)
        if (N > 2500 && ((K >= 2 && K <= 4) || K > wd::kMaxRegisterK2)) ts_log2 = 10;
      }
      // and of the others where LDS holds one workgroup per CU anyway (1500 x 2600: K = 8 235 / 216, K = 10
      // 346 / 280; bucket rings 460 x 2800, K = 8 283 / 253, K = 10 552 / 509)
      if (N > 2500 && ts_log2 == 9 && max_log2 > 9 && partial && K >= 1) {
        wd::Params narrow = *p;
        if (plan_env_kernels(c, &narrow, false, false, 9) && 2 * int64_t(narrow.lds_bytes) > kLdsLimitBytes) ts_log2 = 10;
      }
    } else if (partial && K >= 1 && K <= wd::kMaxRegisterK2) {
      // (K = 1 and K > 4: half the waves on a CU, for registers; K > 8: fewer still, for staged rows)
      const int envs = K > wd::kMaxRegisterK ? 256 : (!strips || N <= 512 || K > 4 || K < 2) ? 512 : 1024;
      if (c.num_envs <= envs) ts_log2 = 9;
    }
    ts_log2 = std::min(ts_log2, max_log2);
    if (ts_log2 > 8) p->wg_size = 1 << ts_log2;
  }
  if (big) {  // one env per 1024-thread workgroup
    ts_log2 = 10;
    p->wg_size = wd::kBigEnvWorkgroupSize;
  }
  const int ts = 1 << ts_log2;
  p->ts_log2 = ts_log2;
  p->teams_per_wg = p->wg_size / ts;
  p->gpt = (p->NG + ts - 1) / ts;
  p->NPAD = (4 * p->NG + 7) / 8 * 8;
  p->vec4 = (N % 4 == 0) ? 1 : 0;
  uint32_t nb_cap = pow2_ceil(uint32_t(N)) / 2;
  if (nb_cap > 4096u) nb_cap = 4096u;
  if (nb_cap < uint32_t(ts)) nb_cap = uint32_t(ts);
  if (nb_cap < 16u) nb_cap = 16u;
  p->nb_cap = int32_t(nb_cap);
  p->scan_chunk = int32_t(nb_cap) / ts;
  // buckets are 65536 / mul cells wide; the table holds nbx^2 <= nb_cap of them
  uint32_t side = 1;
  while ((side + 1) * (side + 1) <= nb_cap) ++side;
  // largest mul with ((G - 1) * mul >> 16) + 1 <= side
  uint32_t mul_max = 65536u;
  if (G > 1) mul_max = uint32_t(std::min<uint64_t>(65536u, ((uint64_t(side) << 16) - 1) / uint64_t(G - 1)));
  p->bucket_mul_max = mul_max;
  p->bucket_scale = float(65536.0 / double(G));
  // target live agents per bucket: about 5 in an env of a hundred agents, 2.2 from five hundred on
  // (with every agent of the headline shape in play: 80.2 us per iteration at 1.5 .. 2.0, where the
  // size of the bucket table sets the width, 78.2 at 2.2, 78.9 at 2.6, 80.9 at 3.0)
  p->lambda_c = 47.0f;
  p->lambda_min = 2.2f;
  p->lambda_max = 5.0f;
  if (ts >= N) {  // a lane per agent: one search round, so fewer, fuller buckets shorten the chain
    p->lambda_c = 70.0f;
    p->lambda_max = 8.0f;
  }
  if (p->K > 4) {  // more neighbours wanted: the 3x3 block of the first pass has to hold more agents
    const float ks = float(p->K) / 4.0f;
    p->lambda_c *= ks;
    p->lambda_min *= ks;
    p->lambda_max *= ks;
  }
  p->div_N = wd::make_fastdiv(uint32_t(N));
  p->div_NG = wd::make_fastdiv(uint32_t(p->NG));

  // (distance, index) keys and bucket entries: 32 bits when they fit, else 64
  p->xy_bits = bits_for(uint32_t(G - 1));
  const uint64_t d2max = 2ull * uint64_t(G - 1) * uint64_t(G - 1);
  // 32-bit form: live keys stay below 2^31, and a dead mark (x + dead_dx) exists that puts the
  // squared distance of a marked entry from any grid cell into [2^(31-ib), 2^(32-ib))
  bool narrow = false;
  p->dead_dx = 0;
  if (p->idx_bits <= 16) {
    const uint64_t band = 1ull << (31 - p->idx_bits);
    uint64_t lo = uint64_t(std::sqrt(double(band)));
    while (lo * lo < band) ++lo;
    const uint64_t shift = lo + uint64_t(G - 1);
    const uint64_t far = shift + uint64_t(G - 1);
    if (d2max + 1 <= band && far <= 32767 && far * far + uint64_t(G - 1) * uint64_t(G - 1) < 2 * band) {
      narrow = true;
      p->dead_dx = int32_t(shift);
    }
  }
  if (!big && c.obs_mode == WD_OBS_PARTIAL && p->K >= 1 && p->K <= wd::kMaxRegisterK2) {
    narrow = strips;  // (these variants search by strip with 32-bit keys, on larger grids by bucket rings with 64-bit keys)
    if (narrow) {
      p->pos_shift = strip_h;
      p->key_shift = 2 * strip_h;
      p->dead_key_min = strip_dead_key_min;
    }
  }
  // Else, in the large-env layout: keys that need all 32 bits, the dead mark moved into bit 15
  // of the index array.  Else 64-bit keys.
  const bool flagged32 = !narrow && big && p->idx_bits <= 15 && G <= 32767 &&
                         p->idx_bits + bits_for(uint32_t(d2max)) <= 32 &&
                         ((d2max << p->idx_bits) | uint64_t(N - 1)) < 0xFFFFFFFFull;  // all ones = "none"
  if (flagged32) narrow = true;  // the same table layout as the 31-bit form
  p->wide = flagged32 ? 2 : (narrow ? 0 : 1);
  const int key_bytes = narrow ? 4 : 8;
  const bool register_path = c.obs_mode == WD_OBS_PARTIAL && p->K <= wd::kMaxRegisterK2;
  // The variants with 32-bit keys and K = 1 .. 16 (small layout) sort by strip and column
  // instead of by square bucket (wd_dev_strips.h).
  p->strips = strips ? 1 : 0;
  if (p->strips) return plan_strip_layout(c, p);

  int64_t off = 0;
  auto take = [&off](int64_t bytes) {
    const int64_t at = off;
    off = align16(off + bytes);
    return int32_t(at);
  };
  const int64_t NPAD = p->NPAD;
  const int tpw = p->teams_per_wg;
  p->off_pl = take(4 * NPAD);
  p->off_misc = take(128);
  p->off_edges = take(2 * (side + 2));
  p->keep_stride = int32_t(off);
  off = 0;
  p->off_sorted = take((narrow ? 4 : 8) * (NPAD + 4));
  p->off_sorted_id = take(narrow ? 2 * (NPAD + 4) : 0);
  p->off_starts = take(2ll * (nb_cap + 4));
  p->x_stride = int32_t(off);
  off = 0;
  p->big_lds_tables = (big && big_tables_in_lds) ? 1 : 0;
  if (!big || big_tables_in_lds) {
    p->off_slot = take(2 * NPAD);
    p->off_best = take(key_bytes * NPAD);
    p->off_credits = take(4ll * c.num_taggers);
  }
  p->off_counts = take(4ll * nb_cap);
  // slots of the second search pass: over slot[] (not needed any more by then), which the
  // neighbour lists therefore must not overlay; a large env has no slot[] in LDS
  p->off_retry = 0;  // (a large env searches in its observation kernel, which needs no second pass)
  const int64_t retry_bytes = (big || !register_path) ? 0 : align16(2 * NPAD);
  const int64_t y_tables = off;
  // neighbour lists: K 16-bit ids per agent, or 40 bits per agent when K = 4 and ids fit 10 bits
  p->compact_nbr = (!big && narrow && p->K == 4 && N < 1024) ? 1 : 0;
  const int64_t nbr_bytes = (!register_path || big) ? 0 : align16(p->compact_nbr ? 5 * NPAD : 2 * NPAD * p->K);
  // per-env strides of the tables a large env keeps in device memory
  p->g_stride_agents = NPAD;
  p->g_stride_credits = (c.num_taggers + 3) / 4 * 4;
  // observation kernel of a large env: about one search per thread
  p->big_slices = std::max(1, std::min(64, (N + wd::kBigObsWorkgroupSize - 1) / wd::kBigObsWorkgroupSize));
  // The staging area of the rows (32 or 16 rows per wave and flush) overlays the X parts and,
  // in a one-team workgroup, the head of the Y part in front of the neighbour lists.
  const int64_t x_area = int64_t(p->x_stride) * tpw;
  const int64_t waves = p->wg_size / wd::kWaveSize;
  const int64_t stage32 = register_path ? waves * 32 * p->D * 4 : 0;
  const int64_t stage16 = register_path ? waves * 16 * p->D * 4 : 0;
  auto plan_with = [&](int64_t stage, int64_t* x_span, int64_t* y_stride) {
    if (tpw == 1) {
      *x_span = x_area;
      *y_stride = align16(std::max<int64_t>(std::max<int64_t>(y_tables, retry_bytes + nbr_bytes), stage + nbr_bytes - x_area));
    } else {
      *x_span = std::max<int64_t>(x_area, stage);
      *y_stride = align16(std::max<int64_t>(y_tables, retry_bytes + nbr_bytes));
    }
    return p->keep_stride * int64_t(tpw) + *x_span + *y_stride * tpw;
  };
  int64_t xs32, ys32, xs16, ys16;
  const int64_t total32 = plan_with(stage32, &xs32, &ys32);
  const int64_t total16 = plan_with(stage16, &xs16, &ys16);
  // 32 rows: whole 64-row chunks then leave through the path without bounds tests, which is
  // worth more than the workgroup per CU that the larger staging area can cost (measured at 100
  // agents per env: 6 workgroups per CU with 32 rows beat 7 with 16); 16 rows only if 32 do not fit
  const bool use32 = total32 <= kLdsLimitBytes;
  (void)total16;
  p->stage_rows_log2 = use32 ? 5 : 4;
  const int64_t x_span = use32 ? xs32 : xs16;
  p->y_stride = int32_t(use32 ? ys32 : ys16);
  p->off_nbr = int32_t(p->y_stride - nbr_bytes);
  p->x_base = p->keep_stride * tpw;
  p->y_base = int32_t(p->x_base + x_span);
  const int64_t total = int64_t(p->y_base) + int64_t(p->y_stride) * tpw;
  p->lds_bytes = int32_t(std::min<int64_t>(total, INT32_MAX));
  p->g_stride_image = p->y_base;  // kept part + sorted part, a multiple of 16 bytes
  return total <= kLdsLimitBytes;
}

// Spread form of the large-env pair.  The pair's first kernel runs one workgroup per env, so a
// batch of a few envs leaves most of the chip idle through seven phases of one workgroup's
// latency; the spread form gives every 512 agents a workgroup for the move and the tag check
// and lets every slice of the second kernel build the env's tables itself.  It pays while the
// batch has far fewer slices than the chip has compute units.  Measured, us per iteration, one
// workgroup per env -> spread (K = 4, a tenth of the agents taggers): 10 envs x 500 agents
// 21.4 -> 21.5, 10 x 2000 24.8 -> 23.8, 10 x 8192 35.9 -> 29.1, 32 x 2000 25.5 -> 25.2,
// 64 x 2000 27.2 -> 27.8, 64 x 4096 35.7 -> 47.2, 128 x 2000 31.3 -> 41.9.
void plan_spread(const wd_config& c, wd::Params* p) {
  p->big_spread = 0;
  if (!p->big || c.num_taggers > wd::kSpreadMaxTaggers || c.num_agents < kSpreadMinAgents ||
      int64_t(c.num_envs) * p->big_slices > kSpreadMaxWorkgroups)
    return;
  p->big_spread = 1;
  // The second kernel's slices: as many as the chip has compute units for, down to 256 agents each (every
  // slice sorts the whole env, so narrower slices only shorten the search and the row stores:
  // tag_10x8192 with 12 / 16 / 20 / 25 slices per env: 30.6 / 28.6 / 28.2 / 28.0 us per iteration).
  p->big_slices = std::max<int64_t>(p->big_slices, std::min<int64_t>(std::min<int64_t>(64, c.num_agents / 256), 250 / c.num_envs));
  p->spread_slices = (p->NG + wd::kSpreadMoveThreads - 1) / wd::kSpreadMoveThreads;
  // coarse cells of the taggers' table: at least a tag radius wide, so that a runner looks at no
  // more than three per axis, and at most kSpreadTagSide per grid side
  const int64_t width = std::max<int64_t>(std::max<int64_t>(p->tag_rad, 1),
                                          (c.grid_size + wd::kSpreadTagSide - 1) / wd::kSpreadTagSide);
  p->tag_mul = uint32_t(std::max<int64_t>(1, 65536 / width));
  p->tag_nbx = int32_t((uint64_t(c.grid_size - 1) * p->tag_mul) >> 16) + 1;
  p->acc_credits = 0;
  p->acc_tags = int32_t(p->g_stride_credits);
  p->g_stride_acc = (p->acc_tags + 1 + 3) / 4 * 4;
}

// Full observations: whether the rows have a launch of their own (full_rows_kernel, spread over the chip).  It costs about 4
// us (8 where step and reset are called one by one) and pays once the rows are long or many and one workgroup per env
// (or per few envs) does not write them as fast: batches that fill the chip do where every row is written, and the two
// forms differ in which rows are (an agent out of play keeps its row).  Measured, us per iteration, rows written by
// env_kernel -> apart, in mid-training (a fifth to a half of the agents in play) and with every agent in play:
//   agent counts that are multiples of four: 20 x 70 16.7 -> 20.5 (three separate calls 22.1 -> 29.4); 1000 x 64 44.5 -> 24.9
// and 45.3 -> 32.6, 8000 x 64 240 -> 92.7 and 246 -> 190, 16000 x 64 184 -> 187 and 259 -> 370; 100 x 100 54.2 -> 22.2,
// 8000 x 100 373 -> 218 and 427 -> 420, 16000 x 100 366 -> 411 and 568 -> 813; 2000 x 220 252 -> 167 and 356 -> 406;
// 200 x 500 364 -> 66.9 and 370 -> 189, 500 x 500 373 -> 157 and 384 -> 469, 2000 x 1000 2587 -> 1676 and 6085 -> 6162.
//   others (env_kernel deals their slots to all lanes of a team, which serves small batches better): 1000 x 65 20.3 -> 25.9 and
// 22.7 -> 33.6; 200 x 101 24.0 -> 19.6 and 24.6 -> 23.0, 1000 x 101 28.3 -> 34.2 and 46.3 -> 59.5; 500 x 150 37.9 -> 30.0
// and 49.7 -> 57.9, 1000 x 150 44.0 -> 49.9 and 91.0 -> 110; 750 x 243 (15 taggers) 169 -> 121; 500 x 201 56.5 -> 39.4 and 83.5 -> 94.1, 5000 x 201 406 -> 329
// and 681 -> 826; 2000 x 251 227 -> 221 and 516 -> 513; 1000 x 499 410 -> 301 and 1049 -> 908.
//   With the step in crew_env_kernel instead of env_kernel (20 to 60 agents: bucket rings and rows in one launch): 10 x 16 17.4 -> 8.9 and 16.8 -> 9.1,
// 8192 x 16 73.1 -> 28.5 and 65.8 -> 38.8; 6000 x 20 61.8 -> 26.7 and 57.6 -> 35.7; 8192 x 32 125 -> 41.9 and 112 -> 59.6; 100 x 48 30.2 -> 9.6 and 28.4 ->
// 10.0, 6000 x 48 127 -> 46.5 and 115 -> 66.5; 8192 x 60 216 -> 84.8 and 197 -> 160; 50 x 80 49.0 -> 9.9, 500 x 80 46.8 -> 16.2 and 46.1 -> 19.5, 8192 x
// 96 208 -> 198 and 343 -> 336.  Others: 5 x 41 12.4 -> 8.6 and 14.4 -> 9.1, 700 x 46 18.1 -> 15.5 and 19.4 -> 18.6, 700 x 50 18.6 -> 17.5 and 19.9 -> 20.3,
// 900 x 50 19.3 -> 19.2 and 21.0 -> 23.1, 1500 x 43 20.0 -> 21.4 and 21.9 -> 26.4; 500 x 65 19.9 -> 15.7 and 21.5 -> 19.2, 500 x 127 32.8 -> 23.2 and 34.1
// -> 31.6; 1000 x 65 20.7 -> 19.7 and 20.9 -> 23.9, 1000 x 101 29.1 -> 31.3; 700 x 150 41.2 -> 32.7 and 51.5 -> 49.7, 700 x 199 60.8 -> 44.4 and 110 -> 94.8,
// 1000 x 150 63.1 -> 53.1 and 91.0 -> 98.7.
//   Larger grids (the figures above are of grids of up to 110 cells a side), rows of env_kernel -> apart behind env_kernel -> apart behind
// crew_env_kernel, which has keys of 32 bits (up to 1639 cells for 20 agents, 1159 for 64, 820 for 100, 579 for 200): 8000 x 64 on 600 cells 239 -> 102
// -> 89.3 and 246 -> 191 -> 178, 1100 x 64 49.7 -> 29.4 -> 23.4, 1000 x 96 62.2 -> 33.6 -> 27.9; 500 x 48 on 700 cells 30.1 -> 13.9, 6000 x 20 on 600
// 60.7 -> 27.2 and 55.6 -> 37.2, 100 x 43 on 800 13.3 -> 9.4.  Keys of 64 bits: 8000 x 64 on 5000 cells 265 -> 101 and 271 -> 191, 3000 x 80 on 1000 153 ->
// 57.1 and 158 -> 86.2, 1000 x 96 on 4500 61.8 -> 33.4 and 63.6 -> 43.4.
bool full_rows_apart(const wd_config& c, const wd::Params& p) {
  const int N = c.num_agents, E = c.num_envs;
  // (small envs: where crew_env_kernel does the step, which has keys of 32 bits)
  const bool short_step = !p.big && N <= wd::kMaxEnvWorkgroupSize && !p.wide;
  if (N % 4 == 0) {
    const int64_t row_bytes = int64_t(E) * N * obs_dim(&c) * 4;
    return (N >= 100 || (N >= 16 && short_step) || (N >= wd::kWaveSize && row_bytes >= (64 << 20))) && E <= 8192;
  }
  if (N >= 200) return true;
  if (!short_step) return (N >= 128 && E <= 512) || (N >= 100 && E <= 256);
  return N >= 128 ? E <= 700 : N >= 64 ? E <= 500 : N >= 40 && E <= 700;
}

// Envs that run in a wave each, without workgroup barriers: in wave_env_kernel (a lane per agent, everything in
// registers; keys of 32 bits: squared distance << 6 | index) or in small_env_kernel (up to 128 agents, tables in LDS, a
// lane per group of four while it samples and moves).  Measured, us per iteration:
//   env_kernel -> small_env_kernel, K = 4: 10 x 100 14.7 -> 11.7, 3000 x 100 26.8 -> 20.1, 20000 x 100 86.5 -> 70.7,
// 3000 x 128 28.9 -> 22.9; 15000 x 100, K = 8 105.8 -> 78.3; 20000 x 5 24.4 -> 28.0.
//   wave_env_kernel / small_env_kernel, agent counts that are multiples of four: K = 4: 2000 x 64 9.4 / 10.0, 3000 x 64
// 12.5 / 11.4, 8000 x 64 25.3 / 19.9, 4000 x 32 9.7 / 10.6, 4000 x 40 11.6 / 11.4; 9000 x 20 13.1 / 15.3, 9000 x 28
// 15.2 / 16.0, 20000 x 28 33.6 / 28.7; K = 8: 9000 x 20 17.2 / 19.1, 9000 x 28 20.8 / 20.4.
//   Other agent counts, whose groups of four small_env_kernel loads and stores one by one: K = 1: 4000 x 33 9.3 / 10.8,
// 8000 x 63 16.9 / 19.6, 20000 x 50 30.8 / 35.7 (env_kernel 36.1); K = 4: 4000 x 33 10.5 / 12.7, 6000 x 50 17.5 / 16.9,
// 9000 x 25 14.5 / 18.4, 9000 x 41 19.1 / 20.4 (four recorded iterations 86.7 / 72.3), 20000 x 34 39.1 / 38.7 (38.2);
// K = 8: 4000 x 41 15.7 / 15.7, 8000 x 33 21.2 / 22.6, 9000 x 33 23.2 / 24.2 (four recorded 123.9 / 91.6),
// 18000 x 25, K = 5 29.2 / 32.3 (35.3); 20000 x 25 48.1 / 45.2 (42.5).
//   With K > 8 (bucket rings, which strips replaced / strips / wave_env_kernel): K = 12: 9000 x 20 37.2 / 40.6 / 21.2,
// 20000 x 20 64.3 / 71.6 / 54.4, 20000 x 32 93.3 / 87.6 / 85.2, 20000 x 40 88.1 / 76.3 / 101; K = 9: 20000 x 12 28.3 /
// 36.8 / 27.0, 20000 x 32 61.1 / 79.9 / 66.2, 20000 x 34 78.6 / 69.0 / 74.8 (bucket rings were faster yet around
// 20000 x 24 with K = 9 and 10: 45.0 / 47.3 / 50.8 and 46.3 / 71.1 / 56.0).
//   wave_env_kernel / quad_env_kernel, one round of waves.  Single calls: K = 4: 100 x 16 5.3 / 4.5, 8000 x 16 10.7 / 8.9,
// 8000 x 5 9.3 / 8.5, 1200 x 18 6.0 / 5.6, 2500 x 18 6.8 / 7.0, 5000 x 18 8.9 / 9.7, 2500 x 24 7.1 / 7.2, 2500 x 32 7.7 / 7.3,
// 2500 x 33 8.3 / 8.7, 100 x 50 6.0 / 5.3, 1200 x 64 7.8 / 7.5; K = 8: 100 x 60 7.3 / 5.0, 5000 x 20 12.1 / 11.4, 8000 x 15
// 14.3 / 10.6; K = 14: 100 x 60 9.0 / 6.0, 5000 x 30 19.8 / 15.9.  Twenty recorded iterations: K = 4: 10 x 5 32.9 / 21.8,
// 100 x 50 63.3 / 31.7, 1000 x 50 68.2 / 53.3, 1500 x 50 79.8 / 80.3, 8000 x 14 115.8 / 99.1, 4000 x 20 76.2 / 80.8, 8000 x 30
// 228 / 205; K = 8: 100 x 50 81.5 / 37.9, 2000 x 50 145 / 141; K = 16: 100 x 50 112 / 51.3, 8000 x 50 1187 / 749; twelve:
// K = 4: 5000 x 18 54.6 / 63, 5000 x 24 64.8 / 67, 2500 x 33 50.5 / 52, 2500 x 40 58.2 / 55; K = 8: 5000 x 20 86.6 / 88.
void plan_waves(const wd_config& c, wd::Params* p) {
  const int N = c.num_agents, E = c.num_envs, K = p->K;
  p->wave_envs = 0;
  if (p->big || c.obs_mode != WD_OBS_PARTIAL) return;
  if ((int64_t(E) + 3) * wd::kWaveSize > kMaxLaunchThreads) return;  // (beyond 67 million envs; fewer lanes per env then)
  const int64_t agents = int64_t(E) * N;
  const bool one_round = E <= kWaveEnvsMaxBatch, fours = N % 4 == 0;
  if (p->strips && N <= wd::kSmallEnvAgents && K <= wd::kMaxRegisterK) {
    bool small = N > wd::kWaveSize;
    if (!small && fours)  // (a wave then has others to wait with)
      small = one_round ? N >= 32 && agents >= 128000 : N >= 24;
    else if (!small)
      small = one_round ? agents >= 128000 && ((K > 4 && N > 40) || (K > 2 && N >= 48 && E >= 5000))
                        : (K > 4 && N > 32) || (K > 2 && N >= 40);
    if (small) {
      p->wave_envs = wd::kSmallEnvs;
      return;
    }
  }
  if (N > wd::kWaveSize || K > wd::kMaxRegisterK2 || c.grid_size > 4096) return;
  bool wave = one_round;
  if (!wave && p->strips)
    wave = K > wd::kMaxRegisterK ? N <= 32
                                 : N >= 12 && (N < 24 || (!fours && (K <= 3 || (K <= 6 && N <= 32) || E <= 2 * kWaveEnvsMaxBatch)));
  if (wave) p->wave_envs = 1;
  if (wave && one_round) {
    // (`used`: of the lanes, per cent; the waves of an env repeat its move and tag check)
    const int waves = (N + wd::kQuadAgents - 1) / wd::kQuadAgents;
    const int used = 100 * N / (waves * wd::kQuadAgents), total = E * waves;
    p->quad_single = K > 4 || waves == 1 || E <= 2000 || used >= 75;
    p->quad_roll = K > 8 || waves == 1 || (K > 4 ? total <= 8000 || used >= 75 : total <= 5000 || used >= 82);
  }
}

// Words per row of crew_env_kernel's map of the cells that taggers reach; 0: no map, every runner is compared with every tagger.
// The map costs two barriers' worth and a row of marks per cell of the tag's height, a comparison about four instructions per
// tagger, so the map pays from 16 taggers per row of the reach on.  us per iteration in mid-training, without / with it: radius 0, 16 taggers
// 256 x 1000 18.5 / 18.4; radius 1, 777 x 333: 16 taggers 17.8 / 17.8, 32 19.3 / 18.3, 64 20.2 / 18.5; radius 3: 32 taggers 777 x 200 15.3 / 15.6, 64 777 x
// 333 20.3 / 19.2, 100 22.4 / 20.3; radius 5: 64 19.1 / 18.8, 100 22.6 / 20.1; radius 8: 16 17.4 / 18.4, 100 777 x 200 19.1 / 20.6, 256 x 1000 21.4 / 20.8, 500 34.7
// / 32.4.  (Larger grids and longer reaches: the map's 16 KB and two words per mark are where it was made to end.)
int crew_map_words(const wd_config& c, const wd::Params& p) {
  const int words = (c.grid_size + 31) / 32 + 1;  // (a tagger's reach in a row touches two words at most)
  return p.tag_rad <= 8 && words * c.grid_size <= 4096 && c.num_taggers >= 16 * (1 + p.tag_rad) ? words : 0;
}

// Many taggers whose reach holds few agents, without the map: comparing every runner with every tagger costs crew_env_kernel more than its shorter
// chain gains, for env_kernel's taggers look into the bins that they reach, four agents to a lane, and so does the large-env pair.  us per
// iteration, the other kernel / crew_env_kernel, K = 4 and 3 to 11 agents in reach: 192 taggers 250 x 1000 23.4 / 24.7; 250 100 x 1000 21.6 / 24.0, 21.5 / 23.3;
// 500 60 x 1000 20.9 / 29.7, 21.4 / 29.3, 250 x 1000 22.5 / 31.6; 600 10 x 700 20.9 / 24.4; but 200 20 x 512 17.9 / 14.8, 256 x 700 no
// difference, 150 120 x 850 23.0 / 20.4, 500 x 333 23.1 / 17.8.  More in reach: 600 10 x 700 with 7 (three and a half taggers to a lane) 31.5 / 24.6,
// 250 100 x 1000 with 44 53.6 / 24.9, 500 60 x 1000 with 44 42.6 / 30.8.  K = 12 and 16: 192 60 x 1000 39.5 / 38.9 and 45.1 / 46.9; 250 100 x 1000
// 40.0 / 41.9 and 45.1 / 49.9; 500 60 x 1000 37.8 / 45.0 and 43.4 / 51.4.
bool tag_check_elsewhere(const wd_config& c, const wd::Params& p) {
  if (p.tag_r2 < 0 || crew_map_words(c, p)) return false;
  const int64_t N = c.num_agents, N_tag = c.num_taggers, G = c.grid_size, side = 2 * int64_t(p.tag_rad) + 1;
  if (N_tag * N <= (p.K > wd::kMaxRegisterK ? 200000 : 170000)) return false;
  return (4 * N_tag + N - 1) / N * N * side * side <= 24 * G * G;
}

// Envs of 65 to 1024 agents that run in crew_env_kernel: a workgroup per env, a lane per agent.  A shorter chain of phases than
// env_kernel's (or small_env_kernel's, up to 128 agents), for more lanes and instructions per agent: it wins while the chain is what
// bounds a batch.  Measured, us per iteration in mid-training, the other kernel -> crew_env_kernel:
//   K = 4: 20 x 100 11.8 -> 9.1, 1000 x 100 14.2 -> 11.7, 3000 x 100 19.3 -> 17.7 (every agent in play 20.8 -> 21.3), 5000 x 100
// 24.4 -> 24.3 (28.1 -> 29.7), 20000 x 100 68.4 -> 70.3; 800 x 65 12.6 -> 10.5, 4000 x 65 18.8 -> 18.1 (18.1 -> 20.3), four recorded
// iterations of 2000 x 65 39.3 -> 40.9; 4000 x 128 25.7 -> 22.1; 100 x 160 16.2 -> 9.8, 5000 x 160 39.8 -> 32.6, 8000 x 200 62.7 -> 58.6;
// 20 x 333 17.8 -> 11.0, 777 x 333 25.4 -> 17.3, 3500 x 333 56.3 -> 49.2; 2000 x 480 37.7 -> 37.5; 1000 x 512 27.3 -> 25.1, 2000 x 512
// 39.1 -> 39.6; 500 x 700 24.3 -> 22.1, 1000 x 700 31.2 -> 33.7 (two workgroups fit a CU); 500 x 850 28.4 -> 23.1; 256 x 1000 23.1 -> 18.2,
// 500 x 1000 27.1 -> 25.1, 600 x 1000 30.5 -> 32.6, 2000 x 1000 63.7 -> 75.2.
//   K = 8: 500 x 333 28.4 -> 18.5, 2500 x 333 77.5 -> 51.2, 3000 x 100 25.0 -> 22.6, 5000 x 100 32.2 -> 34.9, 256 x 1000 29.4 -> 22.8,
// 500 x 850 37.1 -> 37.1, 500 x 1000 37.6 -> 40.0; K = 1: 100 x 200 14.9 -> 9.6, 500 x 700 20.8 -> 19.7.
//   K = 12: 20 x 100 18.4 -> 19.1, 100 x 100 22.2 -> 19.8, 300 x 65 19.9 -> 20.4 (recorded 66.5 -> 72.3), 2000 x 128 47.7 -> 32.8, 500 x 333
// 39.8 -> 29.7, 3500 x 200 82.3 -> 71.3, 1300 x 512 79.8 -> 64.7, 250 x 1000 40.8 -> 33.4, 560 x 1000 89.4 -> 81.0; K = 16: 20 x 128 22.5 ->
// 23.5, 300 x 128 33.0 -> 28.4, 300 x 100 22.7 -> 27.1, 500 x 333 50.7 -> 36.8, 2000 x 200 84.9 -> 63.7, 400 x 1000 82.1 -> 70.9.
//   Four recorded iterations: K = 4: 100 x 200 57.6 -> 33.1, 1200 x 333 109 -> 75, 2700 x 200 146 -> 95; K = 12: 500 x 333 169 -> 103.
//   Full observations whose rows have a launch of their own (the step alone; bucket rings before): 20 x 100 15.5 -> 9.8, 400 x 150 29.7 ->
// 22.1, 200 x 500 93.9 -> 87.9, 250 x 1000 351 -> 344, 8000 x 64 124 -> 117.
//   What bounds it beyond 768 agents with K > 4 is LDS: one workgroup fits a CU (500 x 1000, K = 8 99 232 bytes).  The limits on agents below
// (500 000 for K > 12, 700 000 for K > 8, 1 200 000 for 129 to 480 agents) are where measuring ended, with the kernel still ahead, and no crossovers.
//   Crowds, the other kernel / this: three clusters per env in mid-training: K = 4 100 x 100 13.1 / 11.9, 1500 x 66 15.2 / 13.6 (every agent in play 12.7 /
// 13.6), 2000 x 200 48.5 / 23.4, 777 x 333 54.3 / 20.4, 256 x 1000 64.3 / 25.7; K = 8 2000 x 128 24.1 / 23.9 (21.9 / 23.5), 4000 x 128 30.8 / 33.4 (30.9 / 37.4), 256 x
// 1000 89.4 / 40.1; K = 12 500 x 1000 173 / 83, K = 16 250 / 106.  Most of them on one cell: K = 4 256 x 1000 467 / 78, K = 16 500 x 1000 571 / 220, but
// 65 to 128 agents, which small_env_kernel compares whole whatever they do: K = 4 2000 x 128 17.4 / 22.1, 1000 x 100 14.4 / 17.9, K = 8 2000 x 128 22.0 / 25.6.
bool crew_serves(const wd_config& c, const wd::Params& p) {
  const int N = c.num_agents, E = c.num_envs, K = p.K;
  if (p.big || N > wd::kMaxEnvWorkgroupSize) return false;
  if (c.obs_mode == WD_OBS_FULL) return p.obs_mode == wd::kObsFullSplit && !p.wide;
  if (!p.strips || N <= wd::kWaveSize) return false;
  if (tag_check_elsewhere(c, p)) return false;
  const int64_t agents = int64_t(E) * N;
  if (K > wd::kMaxRegisterK3) return agents <= 500000 && (N > wd::kSmallEnvAgents || (N >= 112 && E >= 256));
  if (K > wd::kMaxRegisterK) return agents <= 700000 && (N >= 112 || (N >= 96 && E >= 64));
  if (N < 96) return E <= 1500;
  if (N < 112) return E <= 3000;
  if (N <= wd::kSmallEnvAgents) return E <= 4096;
  if (N <= 480) return agents <= 1200000;
  if (K > 4 && N > 768) return E <= 256;
  const int waves = (N + wd::kWaveSize - 1) / wd::kWaveSize;
  return E <= 256 * (32 / waves);  // one round of workgroups
}

void plan_crew(const wd_config& c, wd::Params* p) {
  p->crew_threads = 0;
  if (!crew_serves(c, *p)) return;
  const int N = c.num_agents, threads = (N + wd::kWaveSize - 1) / wd::kWaveSize * wd::kWaveSize;
  p->crew_threads = threads;
  p->wave_envs = 0;
  const bool full = c.obs_mode == WD_OBS_FULL;
  const int KT = full ? 0 : p->K <= 4 ? 4 : p->K <= 8 ? 8 : 16;  // places in the neighbour lists
  if (!full) {
    int shift = 0;  // columns as narrow as four bins per lane allow
    while (p->strip_rmax * (((c.grid_size - 1) >> shift) + 1) > 4 * threads) ++shift;
    p->cshift = shift;
    p->strip_C = ((c.grid_size - 1) >> shift) + 1;
  }
  p->crew_reach_words = crew_map_words(c, *p);
  int64_t off = 0;
  auto take = [&off](int64_t bytes) {
    const int64_t at = off;
    off = align16(off + bytes);
    return int32_t(at);
  };
  take(4 * threads);  // packed positions
  p->crew_misc = take(4 * 40);
  p->crew_taggers = take(4 * (c.num_taggers + 3));
  p->crew_reached = take(4 * p->crew_reach_words * c.grid_size);
  p->crew_credits = take(4 * c.num_taggers);
  if (!full) {
    p->crew_nbr = take(2 * KT * threads);
    p->crew_list = take(4 * (threads + p->pad_l + p->pad_r));  // (the rows are staged over the list and its table)
    p->crew_ids = take(2 * (threads + p->pad_l + p->pad_r));
    p->crew_starts = take(2 * (p->strip_rmax * p->strip_C + 4));
    p->crew_edges = take(2 * (p->strip_rmax + 2));
    p->crew_queue = take(4 * threads);
    off = std::max<int64_t>(off, p->crew_list + int64_t(threads / wd::kWaveSize) * (p->K <= 8 ? 32 : 16) * p->D * 4);
  }
  p->crew_lds = int32_t(off);
}

// (`own_tables`: the handle's, allocated for it.  wd_iterate_static has a fixed array for them and refuses what exceeds
// it, so the set of configurations that need tables there is a rule of its own: see wd.h)
int fill_params(const wd_config& c, const wd_buffers& b, wd::Params* p, bool own_tables) {
  std::memset(p, 0, sizeof(*p));
  p->E = c.num_envs;
  p->N = c.num_agents;
  p->N_tag = c.num_taggers;
  p->G = c.grid_size;
  p->T = c.episode_length;
  const int64_t d2max = 2ll * int64_t(c.grid_size - 1) * int64_t(c.grid_size - 1);
  p->tag_r2 = c.tag_r2 < 0 ? -1 : int32_t(std::min<int64_t>(c.tag_r2, d2max));  // beyond d2max everything is in range
  p->tag_rad = c.tag_r2 < 0 ? 0 : isqrt64(p->tag_r2);
  p->K = c.obs_mode == WD_OBS_PARTIAL ? c.obs_k : 0;
  p->D = obs_dim(&c);
  p->obs_mode = c.obs_mode;
  p->env_offset = uint32_t(c.env_offset);
  p->seed_lo = uint32_t(c.seed);
  p->seed_hi = uint32_t(c.seed >> 32);
  p->tag_reward = c.tag_reward;
  p->tag_penalty = c.tag_penalty;
  p->inv_G = float(1.0 / double(c.grid_size));
  p->inv_T = float(1.0 / double(c.episode_length));
  p->pos_x = b.pos_x;
  p->pos_y = b.pos_y;
  p->pos_x0 = b.pos_x0;
  p->pos_y0 = b.pos_y0;
  p->live = b.live;
  p->action = b.action;
  p->reward = b.reward;
  p->obs = b.obs;
  p->t = b.t;
  p->done = b.done;
  p->n_live_runners = b.n_live_runners;
  p->tags_step = b.tags_step;
  // Two layouts serve an env: one workgroup with every table in LDS, or the large-env pair of
  // kernels (the step, then the neighbour search spread over many workgroups).  The pair costs a second
  // launch and a round trip of the tables through device memory, but puts a whole chip on the search of a
  // few envs, so it wins while the batch is too small to fill the chip with one workgroup per env.
  // Measured, K = 4, us per iteration, one workgroup -> pair.  With the strip search: N = 1000: E = 10 19.0 -> 22.4,
  // 300 24.7 -> 38.0; N = 1300: E = 10 20.5 -> 20.8; N = 2000: E = 10 22.9 -> 21.2, 100 26.9 -> 27.8,
  // 300 35.2 -> 46.0 (K = 8: E = 60 34.9 -> 31.3, 200 38.3 -> 39.1; K = 12:
  // N = 500: E = 60 41.7 -> 43.5; N = 1000: E = 60 39.2 -> 38.4, 200 40.7 -> 45.8; N = 2000: E = 200 63.8 -> 50.5); N = 3000: E = 10 26.9 -> 22.9, 100 32.2 -> 32.5, 300 48.1 -> 68.5.  With bucket rings
  // (64-bit keys): E = 10: N = 500 26 -> 22, N = 2000 64 -> 26, N = 6000 158 -> 36; E = 320:
  // N = 1000 39 -> 45, N = 2000 82 -> 66, N = 4000 133 -> 114; E = 640: N = 2000 92 -> 106.
  const bool pair_serves = c.obs_mode == WD_OBS_PARTIAL && p->K <= wd::kMaxRegisterK2;
  const int64_t pair_up_to = c.num_agents <= 1024 ? 3ll * c.num_agents / 10 : 450;  // envs
  bool prefer_pair = pair_serves && c.num_agents >= 384 && c.num_envs <= pair_up_to;
  // the largest batch that the pair serves faster than strips do
  // (up to 1024 agents crew_env_kernel is faster yet: 100 x 1000, K = 12 39.8 -> 32.1; of what it leaves, pair / env_kernel: K = 12 60 x 1000
  // 39.8 / 40.8, 100 x 1000 40.1 / 41.4; K = 16 60 x 1000 44.9 / 54.4, 100 x 1000 46.0 / 54.6, 150 x 1000 57.4 / 54.8, 100 x 850 47.1 / 55.0,
  // 140 x 850 57.0 / 56.1, 100 x 700 43.7 / 47.1)
  int pair_envs = p->K > wd::kMaxRegisterK ? (c.num_agents - 500) / (p->K > wd::kMaxRegisterK3 ? 2 : 4)
                                           : (c.num_agents - 1300) / (p->K > 4 ? 5 : 18);
  if (c.num_agents <= wd::kMaxEnvWorkgroupSize) pair_envs = tag_check_elsewhere(c, *p) ? std::min(pair_envs, 110000 / c.num_agents) : 0;
  if (prefer_pair && own_tables && c.num_envs > pair_envs) {
    wd::Params small = *p;
    if (plan_env_kernels(c, &small, false) && small.strips) prefer_pair = false;
  }
  const wd::Params filled = *p;
  bool planned = prefer_pair && plan_env_kernels(c, p, true, true);
  if (!planned && prefer_pair) {
    *p = filled;
    planned = plan_env_kernels(c, p, true);
  }
  if (!planned) {
    *p = filled;
    planned = plan_env_kernels(c, p, false);
  }
  // The rows that sixteen waves stage may be what does not fit (K = 15 and 16, about 2600 to 3072 agents).  The pair is
  // faster there than eight waves are (460 x 2600, K = 16: 216 -> 126 us with strips; 460 x 2800 791 -> 216 with bucket
  // rings), but eight waves need no tables.
  if (!planned && !prefer_pair && !own_tables && c.num_agents <= 3072) {
    *p = filled;
    planned = plan_env_kernels(c, p, false, false, 9);
  }
  if (!planned && !prefer_pair) {
    *p = filled;
    planned = plan_env_kernels(c, p, true, true);
    if (!planned) {
      *p = filled;
      planned = plan_env_kernels(c, p, true);
    }
  }
  if (!planned || !wd::env_kernel_available(*p)) return WD_E_UNSUPPORTED;
  if (c.obs_mode == WD_OBS_FULL && full_rows_apart(c, *p)) p->obs_mode = wd::kObsFullSplit;
  plan_spread(c, p);
  plan_waves(c, p);
  plan_crew(c, p);
  const int64_t groups = (int64_t(c.num_envs) + p->teams_per_wg - 1) / p->teams_per_wg;
  if (!p->wave_envs && groups * p->wg_size > kMaxLaunchThreads) return WD_E_UNSUPPORTED;
  return WD_OK;
}

int hip_failed(wd_handle* h, hipError_t err, const char* what) {
  h->last_error = std::string(what) + ": " + hipGetErrorString(err);
  return WD_E_HIP;
}

// Work tables of the large-env layout (slots, tag keys, credits and the table image of every env):
// total bytes, and the pointers into one block of that size.
int64_t place_big_tables(wd::Params* p, int64_t E, unsigned char* base) {
  const int64_t key_bytes = p->wide == 1 ? 8 : 4;
  const int64_t slot_b = align16(2 * p->g_stride_agents * E), best_b = align16(key_bytes * p->g_stride_agents * E);
  const int64_t cred_b = align16(4 * p->g_stride_credits * E), image_b = p->big_spread ? 0 : p->g_stride_image * E;
  // spread form: packed positions, the envs' scalars, the number of each env's current set of accumulators, both sets
  const int64_t pl_b = p->big_spread ? align16(4 * p->g_stride_agents * E) : 0;
  const int64_t env_b = p->big_spread ? 16 * E : 0, set_b = p->big_spread ? align16(4 * E) : 0;
  const int64_t acc_b = p->big_spread ? 2 * 4 * p->g_stride_acc * E : 0;
  if (base) {
    p->g_best = base;
    p->g_credits = reinterpret_cast<int32_t*>(base + best_b);
    p->g_slot = reinterpret_cast<uint16_t*>(base + best_b + cred_b);
    p->g_image = base + best_b + cred_b + slot_b;
    unsigned char* at = p->g_image + image_b;
    p->g_pl = reinterpret_cast<uint32_t*>(at);
    p->g_env = reinterpret_cast<int32_t*>(at + pl_b);
    p->g_acc = reinterpret_cast<uint32_t*>(at + pl_b + env_b + set_b);
  }
  return slot_b + best_b + cred_b + image_b + pl_b + env_b + set_b + acc_b;
}

// What a roll-out of the large-env layout needs to run the observation kernel of one iteration
// beside the step kernel of the next: a stream of default priority, events, a second table image.
int ensure_pipe(wd_handle* h) {
  if (h->pipe_ready) return WD_OK;
  hipError_t err = hipStreamCreateWithFlags(&h->obs_stream, hipStreamNonBlocking);
  if (err != hipSuccess) return hip_failed(h, err, "stream for the observation kernels");
  for (int b = 0; b < 2 && err == hipSuccess; ++b) {
    err = hipEventCreateWithFlags(&h->tables_ready[b], hipEventDisableTiming);
    if (err == hipSuccess) err = hipEventCreateWithFlags(&h->rows_done[b], hipEventDisableTiming);
  }
  if (err == hipSuccess) err = hipMalloc(&h->second_image, size_t(h->params.g_stride_image) * size_t(h->params.E));
  if (err != hipSuccess) return hip_failed(h, err, "events and second table image of a roll-out");
  h->pipe_ready = true;
  return WD_OK;
}

// The work tables of wd_iterate_static: one array per device, held until the process ends.
constexpr size_t kStaticScratchBytes = size_t(WD_STATIC_SCRATCH_BYTES);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, once asked for

}  // namespace

extern "C" {

int wd_query_layout(const wd_config* cfg, wd_layout* out) {
  if (!cfg || !out) return WD_E_NULL;
  const int rc = check_config(cfg);
  if (rc != WD_OK) return rc;
  const int64_t E = cfg->num_envs, N = cfg->num_agents, D = obs_dim(cfg);
  out->obs_dim = int32_t(D);
  out->per_agent_elems = E * N;
  out->obs_elems = E * N * D;
  out->per_env_elems = E;
  out->probs_elems = E * N * wd::kNumActions;
  out->bytes_per_iteration = E * N * (4 * wd::kNumActions + 36 + 4 * D) + 24 * E;
  return WD_OK;
}

int wd_create(const wd_config* cfg, const wd_buffers* bufs, wd_handle** out) {
  if (!cfg || !bufs || !out) return WD_E_NULL;
  *out = nullptr;
  int rc = check_config(cfg);
  if (rc != WD_OK) return rc;
  const void* ptrs[] = {bufs->pos_x, bufs->pos_y, bufs->pos_x0, bufs->pos_y0, bufs->live, bufs->action,
                        bufs->reward, bufs->obs, bufs->t, bufs->done, bufs->n_live_runners, bufs->tags_step};
  for (const void* ptr : ptrs)
    if (!ptr) return WD_E_NULL;
  for (const void* ptr : ptrs)
    if (!aligned256(ptr)) return WD_E_ALIGN;
  wd::Params params;
  rc = fill_params(*cfg, *bufs, &params, true);
  if (rc != WD_OK) return rc;
  wd_handle* h = new (std::nothrow) wd_handle();
  if (!h) return WD_E_NULL;
  h->scratch = nullptr;
  if (params.big) {
    // large envs: slots, tag keys, credits and the table image of every env, in one allocation
    if (hipMalloc(&h->scratch, size_t(place_big_tables(&params, cfg->num_envs, nullptr))) != hipSuccess) {
      (void)hipGetLastError();
      delete h;
      return WD_E_HIP;
    }
    place_big_tables(&params, cfg->num_envs, static_cast<unsigned char*>(h->scratch));
    const size_t clear = size_t(align16(4 * int64_t(cfg->num_envs)) + 2 * 4 * params.g_stride_acc * int64_t(cfg->num_envs));
    if (params.big_spread && hipMemset(wd::spread_sets(params), 0, clear) != hipSuccess) {  // set 0 is the first, both start clear
      (void)hipGetLastError();
      (void)hipFree(h->scratch);
      delete h;
      return WD_E_HIP;
    }
  }
  h->cfg = *cfg;
  h->bufs = *bufs;
  h->params = params;
  h->stream = static_cast<hipStream_t>(cfg->stream);
  h->g = 0;
  h->started = false;
  h->rows_valid = false;
  h->obs_stream = nullptr;
  h->second_image = nullptr;
  h->pipe_ready = false;
  *out = h;
  return WD_OK;
}

int wd_reset(wd_handle* h, int mode) {
  if (!h) return WD_E_NULL;
  if (mode != WD_RESET_ALL && mode != WD_RESET_DONE) return WD_E_CONFIG;
  if (mode == WD_RESET_DONE && !h->started) return WD_E_STATE;
  hipError_t err;
  if (mode == WD_RESET_ALL) {
    err = wd::launch_init_start_positions(h->params, h->stream);
    if (err != hipSuccess) return hip_failed(h, err, "start-position kernel");
    err = wd::launch_env_kernel(h->params, wd::kModeResetAll, nullptr, 0, h->stream);
    if (err != hipSuccess) return hip_failed(h, err, "reset kernel");
    h->g = 0;
    h->started = true;
    h->rows_valid = true;
    return WD_OK;
  }
  err = wd::launch_env_kernel(h->params, wd::kModeResetDone, nullptr, 0, h->stream);
  if (err != hipSuccess) return hip_failed(h, err, "reset kernel");
  return WD_OK;
}

int wd_sample(wd_handle* h, const float* probs) {
  if (!h || !probs) return WD_E_NULL;
  if (!probs_aligned(h->params, probs)) return WD_E_ALIGN;
  if (!h->started) return WD_E_STATE;
  const hipError_t err = wd::launch_sample(h->params, probs, h->g, h->stream);
  if (err != hipSuccess) return hip_failed(h, err, "sample kernel");
  return WD_OK;
}

int wd_step(wd_handle* h) {
  if (!h) return WD_E_NULL;
  if (!h->started) return WD_E_STATE;
  wd::Params q = h->params;
  q.rows_kept = h->rows_valid ? 1 : 0;
  const hipError_t err = wd::launch_env_kernel(q, wd::kModeStep, nullptr, h->g, h->stream);
  if (err != hipSuccess) return hip_failed(h, err, "step kernel");
  h->rows_valid = true;
  h->g += 1;
  return WD_OK;
}

int wd_iterate(wd_handle* h, const float* probs) {
  if (!h || !probs) return WD_E_NULL;
  if (!probs_aligned(h->params, probs)) return WD_E_ALIGN;
  if (!h->started) return WD_E_STATE;
  wd::Params q = h->params;
  q.rows_kept = h->rows_valid ? 1 : 0;
  const hipError_t err = wd::launch_env_kernel(q, wd::kModeIterate, probs, h->g, h->stream);
  if (err != hipSuccess) return hip_failed(h, err, "iterate kernel");
  h->rows_valid = true;
  h->g += 1;
  return WD_OK;
}

int wd_iterate_static(const wd_config* cfg, const wd_buffers* bufs, const float* probs, uint64_t g) {
  if (!cfg || !bufs || !probs) return WD_E_NULL;
  int rc = check_config(cfg);
  if (rc != WD_OK) return rc;
  const void* ptrs[] = {bufs->pos_x, bufs->pos_y, bufs->pos_x0, bufs->pos_y0, bufs->live, bufs->action,
                        bufs->reward, bufs->obs, bufs->t, bufs->done, bufs->n_live_runners, bufs->tags_step};
  for (const void* ptr : ptrs)
    if (!ptr) return WD_E_NULL;
  for (const void* ptr : ptrs)
    if (!aligned256(ptr)) return WD_E_ALIGN;
  wd::Params params;
  rc = fill_params(*cfg, *bufs, &params, false);
  if (rc != WD_OK) return rc;
  if (!probs_aligned(params, probs)) return WD_E_ALIGN;
  params.big_spread = 0;  // (its accumulators have to start clear; the pair with one workgroup per env needs nothing of the kind)
  if (params.big) {
    if (size_t(place_big_tables(&params, cfg->num_envs, nullptr)) > kStaticScratchBytes) return WD_E_SCRATCH;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
      (void)hipGetLastError();
      return WD_E_HIP;
    }
    if (!g_scratch_ptr[dev]) {  // this device's copy of the array, at its own address
      void* ptr = nullptr;
      if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
        (void)hipGetLastError();
        return WD_E_HIP;
      }
      g_scratch_ptr[dev] = ptr;
    }
    // (nothing in the tables has to start at zero: the kernels write every entry before they read it)
    place_big_tables(&params, cfg->num_envs, static_cast<unsigned char*>(g_scratch_ptr[dev]));
  }
  params.rows_kept = 0;  // no handle, so nothing is known about what `obs` holds: every row is written whole
  if (wd::launch_env_kernel(params, wd::kModeIterate, probs, g, static_cast<hipStream_t>(cfg->stream)) != hipSuccess) {
    (void)hipGetLastError();
    return WD_E_HIP;
  }
  return WD_OK;
}

int wd_rollout(wd_handle* h, const float* probs_ring, int ring_len, int k, const wd_rollout_buffers* out) {
  if (!h || !probs_ring) return WD_E_NULL;
  if (ring_len < 1 || k < 1) return WD_E_CONFIG;
  if (!probs_aligned(h->params, probs_ring)) return WD_E_ALIGN;
  if (out) {
    const void* ptrs[] = {out->action, out->reward, out->done, out->obs};
    for (const void* ptr : ptrs)
      if (reinterpret_cast<uintptr_t>(ptr) & 15u) return WD_E_ALIGN;
  }
  if (!h->started) return WD_E_STATE;
  // recorded observations go to slices that hold nothing yet, and the in-place rows that the last
  // iteration then meets date from before the call: every row is written whole
  const int rows_kept = (h->rows_valid && !(out && out->obs)) ? 1 : 0;
  if (!wd::rollout_available(h->params)) {
    // Configurations without a multi-step kernel (large-env layout, full observations,
    // K > 16, K > 8 with 64-bit keys): the same results from one launch of the iteration kernels per iteration,
    // outputs redirected to the slices, the last slice copied from the in-place buffers.
    // In the large-env layout the observation kernel of iteration s runs on a second stream beside
    // the step kernel of iteration s + 1 (which needs the state, not the rows): two table images
    // in turn, an image rewritten only once the observation kernel that read it has finished.
    const bool piped = h->params.big && !h->params.big_spread && k > 1;
    if (piped) {
      const int rc = ensure_pipe(h);
      if (rc != WD_OK) return rc;
    }
    const int64_t EN = int64_t(h->cfg.num_envs) * h->cfg.num_agents, D = h->params.D;
    for (int s = 0; s < k; ++s) {
      wd::Params q = h->params;
      q.rows_kept = rows_kept;
      wd::ObsPipe pipe = {};
      if (piped) {
        const int b = s & 1;
        if (b) q.g_image = static_cast<unsigned char*>(h->second_image);
        if (s >= 2) {
          const hipError_t werr = hipStreamWaitEvent(h->stream, h->rows_done[b], 0);
          if (werr != hipSuccess) return hip_failed(h, werr, "wait for a table image");
        }
        pipe.stream = h->obs_stream;
        pipe.tables_ready = h->tables_ready[b];
        pipe.rows_done = h->rows_done[b];
      }
      if (out && s + 1 < k) {
        if (out->action) q.action = out->action + int64_t(s) * EN;
        if (out->reward) q.reward = out->reward + int64_t(s) * EN;
        if (out->reward && s == 0) q.kept_reward = h->params.reward;
        if (out->obs) q.obs = out->obs + int64_t(s) * EN * D;
      }
      q.done_log = (out && out->done) ? out->done + int64_t(s) * h->cfg.num_envs : nullptr;
      const float* probs = probs_ring + int64_t((h->g + uint64_t(s)) % uint64_t(ring_len)) * EN * wd::kNumActions;
      const hipError_t err = wd::launch_env_kernel(q, wd::kModeIterate, probs, h->g + uint64_t(s), h->stream,
                                                   piped ? &pipe : nullptr);
      if (err != hipSuccess) return hip_failed(h, err, "iteration kernel of a roll-out");
    }
    if (piped) {  // what follows on the caller's stream sees every row
      const hipError_t werr = hipStreamWaitEvent(h->stream, h->rows_done[(k - 1) & 1], 0);
      if (werr != hipSuccess) return hip_failed(h, werr, "wait for the last observation kernel");
    }
    if (out) {
      const int64_t last = int64_t(k - 1) * EN;
      hipError_t err = hipSuccess;
      if (out->action && err == hipSuccess)
        err = hipMemcpyAsync(out->action + last, h->bufs.action, size_t(EN) * 4, hipMemcpyDeviceToDevice, h->stream);
      if (out->reward && err == hipSuccess)
        err = hipMemcpyAsync(out->reward + last, h->bufs.reward, size_t(EN) * 4, hipMemcpyDeviceToDevice, h->stream);
      if (out->obs && err == hipSuccess)
        err = hipMemcpyAsync(out->obs + last * D, h->bufs.obs, size_t(EN * D) * 4, hipMemcpyDeviceToDevice, h->stream);
      if (err != hipSuccess) return hip_failed(h, err, "copy of the last roll-out slice");
    }
    h->rows_valid = true;
    h->g += uint64_t(k);
    return WD_OK;
  }
  wd::Roll roll;
  std::memset(&roll, 0, sizeof(roll));
  roll.steps = k;
  roll.ring_len = ring_len;
  roll.ring_pos = int32_t(h->g % uint64_t(ring_len));
  if (out) {
    roll.action = out->action;
    roll.reward = out->reward;
    roll.done = out->done;
    roll.obs = out->obs;
  }
  wd::Params q = h->params;
  q.rows_kept = rows_kept;
  const hipError_t err = wd::launch_rollout(q, roll, probs_ring, h->g, h->stream);
  if (err != hipSuccess) return hip_failed(h, err, "rollout kernel");
  h->rows_valid = true;
  h->g += uint64_t(k);
  return WD_OK;
}

int wd_get_step(wd_handle* h, uint64_t* g) {
  if (!h || !g) return WD_E_NULL;
  *g = h->g;
  return WD_OK;
}

int wd_set_step(wd_handle* h, uint64_t g) {
  if (!h) return WD_E_NULL;
  h->g = g;
  h->rows_valid = false;  // a resumed run: the caller may have restored the state arrays without the observations
  return WD_OK;
}

int wd_invalidate_obs(wd_handle* h) {
  if (!h) return WD_E_NULL;
  h->rows_valid = false;
  return WD_OK;
}

int wd_destroy(wd_handle* h) {
  if (!h) return WD_E_NULL;
  if (h->scratch) (void)hipFree(h->scratch);
  if (h->pipe_ready) {
    (void)hipStreamSynchronize(h->obs_stream);
    (void)hipFree(h->second_image);
    for (int b = 0; b < 2; ++b) {
      (void)hipEventDestroy(h->tables_ready[b]);
      (void)hipEventDestroy(h->rows_done[b]);
    }
    (void)hipStreamDestroy(h->obs_stream);
  }
  delete h;
  return WD_OK;
}

const char* wd_strerror(int status) {
  switch (status) {
    case WD_OK: return "ok";
    case WD_E_NULL: return "a required pointer is NULL";
    case WD_E_CONFIG: return "configuration field out of range";
    case WD_E_ALIGN: return "device buffer not aligned as required";
    case WD_E_STATE: return "call before the first wd_reset(WD_RESET_ALL)";
    case WD_E_HIP: return "HIP call failed";
    case WD_E_UNSUPPORTED: return "configuration not covered by this build's kernels";
    case WD_E_SCRATCH: return "work tables of this configuration exceed the static scratch array of wd_iterate_static";
    default: return "unknown status";
  }
}

const char* wd_last_error(wd_handle* h) { return h ? h->last_error.c_str() : ""; }

}  // extern "C"
