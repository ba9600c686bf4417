// wdc_dev_strips.h — continuous Tag: the strip-sorted list of an env's agents in play and the K-nearest
// searches over it.  Device-side helpers; included by wdc.hip only.
//
// Comparing every agent with every other (arXiv 2108.13976, Sec. 5.5: full pairwise work makes the
// step O(N^2)) is vector-ALU bound from about a hundred agents on.  Here the agents in play are sorted by
// (strip, column) — strips are horizontal bands of the world about one K-th-neighbour distance tall,
// columns narrow vertical ones, so inside a strip the list is ordered by column — and an agent looks
// at fixed windows of the list around its own slot and around its column in the strips above and below.
// A candidate costs five vector instructions (two subtracts, a multiply, a multiply-add, and the
// packing of its key) and one per kept key.  A key is the bits of the squared distance with the low six
// replaced by the candidate's number inside the windows, so the sorted insertion moves one register
// per key and no index is loaded; what the six bits (and the fused multiply-add's rounding) leave
// undecided is decided afterwards on the exact squared distances.
#ifndef WDC_DEV_STRIPS_H
#define WDC_DEV_STRIPS_H

#include "wd_dev_tables.h"

namespace wdc {
namespace {

constexpr float kGone = 1e18f;               // y of a list entry that is out of play, and of the pads
constexpr uint32_t kGoneKey = 0x7149F2CAu;   // bits of 1e30f: keys from here on belong to nobody in play
constexpr uint16_t kGoneId = 0x8000u;        // mark in the id of a list entry that is out of play
constexpr float kFarF = 1e15f;               // "no bound on this side"
constexpr int kColumns = 64;                 // columns per strip
constexpr uint16_t kNobody = 0xFFFFu;
constexpr uint32_t kNumberMask = 63u;        // the key bits that number a candidate

// Windows for K neighbours: entries on either side of the agent's slot, and on either side of its
// column in the strips below and above; at most 64 in all, for six bits number them.
constexpr int half_own(int k) { return k + 3; }
constexpr int half_adj(int k) { return k + 2; }
constexpr int list_pad(int k) { return half_own(k) + 2 * half_adj(k); }

// Geometry of one env's list.
struct Strips {
  float mul, cmul;  // strip = y * mul, column = x * cmul (truncated, clamped)
  float hgt, cw;    // height of a strip, width of a column
  float eps;        // covers the rounding of every bound below
  int R;
};

__device__ __forceinline__ Strips make_strips(float L, float scale, int rmax, int n_live) {
  Strips g;
  g.R = min(max(int(scale * sqrtf(static_cast<float>(max(n_live, 1))) + 0.5f), 1), rmax);
  g.mul = static_cast<float>(g.R) / L;
  g.cmul = static_cast<float>(kColumns) / L;
  g.hgt = L / static_cast<float>(g.R);
  g.cw = L / static_cast<float>(kColumns);
  g.eps = L * 4e-6f;
  return g;
}
// (monotone in the coordinate, for any value of it: clamped at both ends)
__device__ __forceinline__ int strip_at(float y, const Strips& g) { return min(max(int(y * g.mul), 0), g.R - 1); }
__device__ __forceinline__ int column_at(float x, const Strips& g) { return min(max(int(x * g.cmul), 0), kColumns - 1); }

// Key of a candidate at p for an agent at me; `number` in the low six bits.
__device__ __forceinline__ uint32_t near_key(float2 p, float2 me, uint32_t number) {
  const float dx = p.x - me.x, dy = p.y - me.y;
  return (__float_as_uint(__builtin_fmaf(dy, dy, dx * dx)) & ~kNumberMask) | number;
}

// kN list entries from `w` on, numbered from kNumber on.
template <int KL, int kNumber, int... J>
__device__ __forceinline__ void near_chunk(uint32_t (&keys)[KL], const float2* w, float2 me,
                                           std::integer_sequence<int, J...>) {
  float2 p[sizeof...(J)];
  ((p[J] = w[J]), ...);
  (wd::dev::insert_key<KL>(keys, near_key(p[J], me, uint32_t(kNumber + J))), ...);
}
template <int KL, int N, int kNumber, int kFirst = 0>
__device__ __forceinline__ void near_slots(uint32_t (&keys)[KL], const float2* w, float2 me) {
  constexpr int kN = N - kFirst < 8 ? N - kFirst : 8;  // eight loads in flight
  near_chunk<KL, kNumber + kFirst>(keys, w + kFirst, me, std::make_integer_sequence<int, kN>{});
  if constexpr (kFirst + kN < N) near_slots<KL, N, kNumber, kFirst + kN>(keys, w, me);
}

// Distance below which nothing can lie unseen on one side of a window: `done` = the window reaches the
// end of its strip there.
__device__ __forceinline__ float side_reach(bool done, float dist) { return done ? kFarF : fmaxf(dist, 0.0f); }

// The windows of the agent in slot q.  keys[0 .. KT] receives the KT + 1 smallest keys met, `below` and
// `above` the first slots of the two neighbouring strips' windows; returns the square of a distance
// within which every agent in play has been met (kFarF * kFarF: all of them).
//
// The list is one array, strip after strip, so a window may run past the ends of its strip: that only
// adds candidates, as long as none is met twice; so the window below ends where the own window (or
// strip) begins, and the window above begins where it ends.  With pads of list_pad(KT) entries on
// either side of the list every access is inside them: the own window overhangs the list by at most
// half_own, and a neighbouring strip's window then sits next to it.
template <int KT>
__device__ __forceinline__ float near_windows(uint32_t (&keys)[KT + 1], float2 me, int q, int n, const Strips& g,
                                              const float2* list, const uint16_t* T, int& below, int& above) {
  constexpr int HO = half_own(KT), HA = half_adj(KT);
  static_assert(2 * HO + 4 * HA <= 64, "candidates are numbered in six bits");
  const int r = strip_at(me.y, g), row0 = r * kColumns, bin = row0 + column_at(me.x, g);
#pragma unroll
  for (int k = 0; k <= KT; ++k) keys[k] = ~0u;
  const int s_own = T[row0], e_own = T[row0 + kColumns];
  near_slots<KT + 1, HO, 0>(keys, list + (q - HO), me);
  near_slots<KT + 1, HO, HO>(keys, list + (q + 1), me);
  // an unseen entry to the left is in the window's first column or left of it, to the right likewise
  const auto left_of = [&](int slot) { return me.x - static_cast<float>(column_at(list[slot].x, g) + 1) * g.cw - g.eps; };
  const auto right_of = [&](int slot) { return static_cast<float>(column_at(list[slot].x, g)) * g.cw - me.x - g.eps; };
  const float own = fminf(side_reach(q - HO <= s_own, left_of(q - HO)), side_reach(q + HO >= e_own - 1, right_of(q + HO)));
  float reach2 = own * own;
  const int lo_edge = min(s_own, q - HO), hi_edge = max(e_own, q + HO + 1);
  {
    const bool has = r >= 1;
    const int bb = has ? bin - kColumns : bin;
    const int pc = (int(T[bb]) + int(T[bb + 1]) + 1) >> 1;
    const int a = has ? min(pc - HA, lo_edge - 2 * HA) : n;
    below = a;
    near_slots<KT + 1, 2 * HA, 2 * HO>(keys, list + a, me);
    const int start = T[has ? row0 - kColumns : row0];
    const float b = fminf(side_reach(a <= start, left_of(a)), side_reach(a + 2 * HA >= lo_edge, right_of(a + 2 * HA - 1)));
    const float gap = fmaxf(me.y - static_cast<float>(r) * g.hgt - g.eps, 0.0f);
    if (has) reach2 = fminf(reach2, b * b + gap * gap);
  }
  {
    const bool has = r + 1 < g.R;
    const int bb = has ? bin + kColumns : bin;
    const int pc = (int(T[bb]) + int(T[bb + 1]) + 1) >> 1;
    const int a = has ? max(pc - HA, hi_edge) : n;
    above = a;
    near_slots<KT + 1, 2 * HA, 2 * HO + 2 * HA>(keys, list + a, me);
    const int end = T[has ? row0 + 2 * kColumns : row0 + kColumns];
    const float b = fminf(side_reach(a <= hi_edge, left_of(a)), side_reach(a + 2 * HA >= end, right_of(a + 2 * HA - 1)));
    const float gap = fmaxf(static_cast<float>(r + 1) * g.hgt - me.y - g.eps, 0.0f);
    if (has) reach2 = fminf(reach2, b * b + gap * gap);
  }
  // the strips beyond
  if (r >= 2) {
    const float gap = fmaxf(me.y - static_cast<float>(r - 1) * g.hgt - g.eps, 0.0f);
    reach2 = fminf(reach2, gap * gap);
  }
  if (r + 2 < g.R) {
    const float gap = fmaxf(static_cast<float>(r + 2) * g.hgt - me.y - g.eps, 0.0f);
    reach2 = fminf(reach2, gap * gap);
  }
  return reach2;
}

// Slot of the candidate with this number in the windows.
template <int KT>
__device__ __forceinline__ int slot_of_number(int number, int q, int below, int above) {
  constexpr int HO = half_own(KT), HA = half_adj(KT);
  const int own = number < HO ? q - HO + number : q + 1 + (number - HO);
  const int adj = number < 2 * HO + 2 * HA ? below + (number - 2 * HO) : above + (number - 2 * HO - 2 * HA);
  return number < 2 * HO ? own : adj;
}

// A short list is compared whole: every lane reads the same entries, eight per round; the last round may
// run into the pad behind the list.  An entry's number is its slot.  The agent meets itself too, so one
// key more is kept and its own (distance 0, its slot) is taken out at the end.
template <int KT>
__device__ __forceinline__ void near_all(uint32_t (&keys)[KT + 1], float2 me, int q, int n, const float2* list) {
  uint32_t all[KT + 2];
#pragma unroll
  for (int k = 0; k < KT + 2; ++k) all[k] = ~0u;
  for (int s0 = 0; s0 < n; s0 += 8) {
    float2 p[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = list[s0 + j];
#pragma unroll
    for (int j = 0; j < 8; ++j) wd::dev::insert_key<KT + 2>(all, near_key(p[j], me, uint32_t(s0 + j)));
  }
  bool passed = false;
#pragma unroll
  for (int k = 0; k <= KT; ++k) {
    passed |= all[k] == uint32_t(q);
    keys[k] = passed ? all[k + 1] : all[k];
  }
}

// Two keys whose distance parts are this close may belong to distances in either order (the six bits
// dropped, and one unit in the last place of the fused multiply-add).
__device__ __forceinline__ bool undecided(uint32_t a, uint32_t b) {
  return b < kGoneKey && (b / (kNumberMask + 1u)) - (a / (kNumberMask + 1u)) <= 1u;
}

__device__ __forceinline__ uint64_t wave_min(uint64_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const uint32_t lo = uint32_t(__shfl_xor(int(uint32_t(v)), d)), hi = uint32_t(__shfl_xor(int(uint32_t(v >> 32)), d));
    const uint64_t o = (uint64_t(hi) << 32) | lo;
    v = o < v ? o : v;
  }
  return v;
}

}  // namespace
}  // namespace wdc
#endif  // WDC_DEV_STRIPS_H
