// Routing of a workgroup's tokens (route.hip has the launch and says why it looks like this; plan.hip routes a few tokens in the
// planner's launch).  Not part of the public ABI.
#pragma once
#include "common.h"

#include <type_traits>

#include <float.h>
#include <math.h>

// every float operation in this file is rounded on its own
#pragma clang fp contract(off)

namespace occult {

__device__ __forceinline__ float exp_ref(float z) {
  // z <= 0.  z < -80 -> 0.  n = rint(z*log2e); r = (z - n*ln2_hi) - n*ln2_lo; degree-7 Taylor
  // polynomial by Horner; result scaled by 2^n through the exponent bits.
  const float kLog2e = 1.4426950408889634f;
  const float kLn2Hi = 0.693359375f;
  const float kLn2Lo = -2.12194440054690583e-4f;
  const float zc = fmaxf(z, -80.0f);
  const float n = rintf(zc * kLog2e);
  float r = zc - n * kLn2Hi;
  r = r - n * kLn2Lo;
  float p = 1.0f / 5040.0f;
  p = p * r + 1.0f / 720.0f;
  p = p * r + 1.0f / 120.0f;
  p = p * r + 1.0f / 24.0f;
  p = p * r + 1.0f / 6.0f;
  p = p * r + 0.5f;
  p = p * r + 1.0f;
  p = p * r + 1.0f;
  const float scale = __int_as_float(((int)n + 127) << 23);
  const float out = p * scale;
  return z < -80.0f ? 0.0f : out;
}

// Cross-lane steps on the VALU's data-parallel primitives (no LDS crossbar): four symmetric exchanges leave every lane of
// a row of 16 with the row's result.
// Two row broadcasts carry it on into lane 63 where a token has the whole wavefront.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ int dpp_i(int own, int v) {   // rows outside the mask keep `own`
  return __builtin_amdgcn_update_dpp(own, v, CTRL, ROW_MASK, 0xF, false);
}
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp_f(float own, float v) {
  return __builtin_bit_cast(float, dpp_i<CTRL, ROW_MASK>(__builtin_bit_cast(int, own), __builtin_bit_cast(int, v)));
}
constexpr int kQuadSwap1 = 0xB1;       // quad_perm [1,0,3,2]
constexpr int kQuadSwap2 = 0x4E;       // quad_perm [2,3,0,1]
constexpr int kRowHalfMirror = 0x141;
constexpr int kRowMirror = 0x140;
constexpr int kRowBcast15 = 0x142;     // lane 15 of each row into the next row (rows 1 and 3 take it)
constexpr int kRowBcast31 = 0x143;     // lane 31 into rows 2 and 3

// (value, index) as one 64-bit key whose unsigned order is "larger value first, equal values -> lower index":
// the value's bits made monotone (negative floats inverted, positive ones offset) in the high word, the
// complemented index in the low word.  One 64-bit compare per step instead of three compares.  The key of a finite
// value is never 0, which stands for "taken" and "not there".
typedef unsigned long long key_t64;
__device__ __forceinline__ key_t64 argmax_key(float v, int i) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const unsigned ord = u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
  return ((key_t64)ord << 32) | (unsigned)(~i);
}
__device__ __forceinline__ int key_index(key_t64 key) { return ~(int)(unsigned)key; }
__device__ __forceinline__ float key_value(key_t64 key) {
  const unsigned ord = (unsigned)(key >> 32);
  return __builtin_bit_cast(float, ord ^ ((ord >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ key_t64 key_max_step(key_t64 key) {
  const int klo = (int)(unsigned)key, khi = (int)(unsigned)(key >> 32);
  const int lo = dpp_i<CTRL, ROW_MASK>(klo, klo), hi = dpp_i<CTRL, ROW_MASK>(khi, khi);
  const key_t64 other = ((key_t64)(unsigned)hi << 32) | (unsigned)lo;
  return other > key ? other : key;
}
// largest key of a token's LANES lanes, in every one of them
template <int LANES>
__device__ __forceinline__ key_t64 token_max(key_t64 key) {
  key = key_max_step<kQuadSwap1>(key);
  key = key_max_step<kQuadSwap2>(key);
  key = key_max_step<kRowHalfMirror>(key);
  key = key_max_step<kRowMirror>(key);
  if (LANES == 16) return key;
  key = key_max_step<kRowBcast15, 0xA>(key);
  key = key_max_step<kRowBcast31, 0xC>(key);
  return ((key_t64)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(key >> 32), 63) << 32) |
         (unsigned)__builtin_amdgcn_readlane((int)(unsigned)key, 63);
}
// Sum over a token's experts (or slots) in one order for both lane counts, so that a token's gates do not depend on the
// size of its batch: v[q] holds a lane's share of the columns of residue 16 q + lane % 16 modulo 64 (with 64 lanes: q = 0,
// the columns of residue `lane`).  Each sixteen are added up on their own, then the four sums as (3 + 2) + (1 + 0).
template <int LANES, int N>
__device__ __forceinline__ float token_sum(float (&v)[N]) {
#pragma unroll
  for (int q = 0; q < N; ++q) {
    v[q] += dpp_f<kQuadSwap1>(v[q], v[q]);
    v[q] += dpp_f<kQuadSwap2>(v[q], v[q]);
    v[q] += dpp_f<kRowHalfMirror>(v[q], v[q]);
    v[q] += dpp_f<kRowMirror>(v[q], v[q]);
  }
  if constexpr (LANES == 16) {
    static_assert(N == 1 || N == 2 || N == 4, "sixteen columns per sum");
    if constexpr (N == 4) return (v[3] + v[2]) + (v[1] + v[0]);
    return N == 2 ? v[N - 1] + v[0] : v[0];
  } else {
    static_assert(N == 1, "a lane per column");
    float s = v[0];
    s += dpp_f<kRowBcast15, 0xA>(0.0f, s);
    s += dpp_f<kRowBcast31, 0xC>(0.0f, s);
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s), 63));
  }
}

// LANES = lanes per token, 16 or 64; EPL = experts per lane, E <= LANES * EPL.  Lane r of a token writes slots r and,
// with 16 lanes, r + 16.
template <int LANES, int EPL, bool PRUNE>
__device__ __forceinline__ void route_tokens(   // the tokens of workgroup `block` of 256 threads
    int block, const float* __restrict__ logits, int T, int E, int k, int D, int G,
    const int32_t* __restrict__ expert_pos, int n_d, int prune_mode, int renorm,
    const int32_t* __restrict__ sim_table, int32_t* __restrict__ ids, float* __restrict__ w) {
  __shared__ int s_dev[PRUNE ? OCCULT_MAX_E : 1];   // only pruning asks which device an expert is on
  if (PRUNE) {
    for (int e = threadIdx.x; e < E; e += blockDim.x) s_dev[e] = (expert_pos ? expert_pos[e] : e) / G;
    __syncthreads();
  }
  const int lane = threadIdx.x & 63, r = lane & (LANES - 1), row0 = lane & (64 - LANES);
  constexpr int SLOTS = OCCULT_MAX_K > LANES ? OCCULT_MAX_K / LANES : 1, DEVS = OCCULT_MAX_D / LANES;   // per lane
  const int t = block * (256 / LANES) + threadIdx.x / LANES;
  if (t >= T) return;   // all lanes of a token leave together; no barrier follows
  const float* row = logits + (size_t)t * E;

  float v0[EPL];     // the token's scores as read (with -0.0 folded onto +0.0)
  key_t64 key[EPL];  // 0: taken, not allowed or not there
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = r + LANES * i;
    // NaN and -inf scores are read as the lowest finite value and +inf as the highest: each round then selects a new
    // index below E whatever the scores hold (ids index other tables downstream), and the device sums and gates stay
    // finite
    v0[i] = (e < E) ? fminf(fmaxf(row[e] + 0.0f, -FLT_MAX), FLT_MAX) : 0.0f;
    key[i] = (e < E) ? argmax_key(v0[i], e) : 0ull;
  }
  auto select_round = [&]() {
    key_t64 best = key[0];
#pragma unroll
    for (int i = 1; i < EPL; ++i) best = key[i] > best ? key[i] : best;
    best = token_max<LANES>(best);
#pragma unroll
    for (int i = 0; i < EPL; ++i) key[i] = key[i] == best ? 0ull : key[i];
    return best;
  };

  key_t64 slot[SLOTS] = {};
  auto keep_slot = [&](int s, key_t64 best) {
#pragma unroll
    for (int h = 0; h < SLOTS; ++h)
      if (r + LANES * h == s) slot[h] = best;
  };
  float mx = 0.0f;
  float dev_sum[DEVS] = {};      // mode 1: scores of devices r, r + LANES, ...
  unsigned long long kept = 0;   // mode 2: devices kept so far (the same in a token's lanes)
  int n_kept = 0;

  for (int s = 0; s < k; ++s) {
    const key_t64 best = select_round();
    if (s == 0) mx = key_value(best);
    keep_slot(s, best);
    if (PRUNE) {
      const int dev = s_dev[key_index(best)];
      if (prune_mode == 1) {
        const float q = exp_ref(key_value(best) - mx);
#pragma unroll
        for (int h = 0; h < DEVS; ++h)
          if (r + LANES * h == dev) dev_sum[h] = dev_sum[h] + q;   // sequential in slot order
      } else if (!((kept >> dev) & 1ull) && n_kept < n_d) {
        kept |= 1ull << dev;
        ++n_kept;
      }
    }
  }

  if (PRUNE && prune_mode == 3) {
    // Expert-similarity-based pruning: routed experts on kept devices stay in their slots; the
    // others are replaced, in slot (= descending score) order, by the first entry of their table
    // row that is on a kept device and not taken.  `taken` = one bit per expert, the same in a token's lanes; the
    // control flow below differs between the tokens of a wave, never between the lanes of a token.
    unsigned long long taken[4] = {0ull, 0ull, 0ull, 0ull};
    auto expert_of = [&](int s) {   // expert in slot s
      const int lo = __shfl(key_index(slot[0]), row0 + (s & (LANES - 1)), 64);
      if (SLOTS == 1) return lo;
      const int hi = __shfl(key_index(slot[SLOTS - 1]), row0 + (s & (LANES - 1)), 64);
      return s < LANES ? lo : hi;
    };
    for (int s = 0; s < k; ++s) {
      const int e = expert_of(s);
      if ((kept >> s_dev[e]) & 1ull) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if ((e >> 6) == q) taken[q] |= 1ull << (e & 63);
      }
    }
    for (int s = 0; s < k; ++s) {
      const int e = expert_of(s);
      if ((kept >> s_dev[e]) & 1ull) continue;
      const int32_t* trow = sim_table + (size_t)e * (E - 1);
      int found = -1;
      for (int base = 0; base < E - 1 && found < 0; base += LANES) {
        const int q = base + r;
        int c = 0;
        bool ok = false;
        if (q < E - 1) {
          c = trow[q];
          unsigned long long word = taken[0];
#pragma unroll
          for (int m = 1; m < 4; ++m)
            if ((c >> 6) == m) word = taken[m];
          ok = ((kept >> s_dev[c]) & 1ull) && !((word >> (c & 63)) & 1ull);
        }
        const unsigned long long hits = (__ballot(ok) >> row0) & (~0ull >> (64 - LANES));
        const int c_hit = __shfl(c, row0 + (hits ? __ffsll((long long)hits) - 1 : 0), 64);
        if (hits) found = c_hit;
      }
      // host checks n_d * G >= k, so a free expert on a kept device always exists
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if ((found >> 6) == q) taken[q] |= 1ull << (found & 63);
      // its score sits in lane found % LANES of the token, register found / LANES
      float fv = v0[0];
#pragma unroll
      for (int i = 1; i < EPL; ++i)
        if (found / LANES == i) fv = v0[i];
      fv = __shfl(fv, row0 + (found & (LANES - 1)), 64);
      keep_slot(s, argmax_key(fv, found));
    }
  } else if (PRUNE) {
    if (prune_mode == 1) {
      key_t64 dk[DEVS];
#pragma unroll
      for (int h = 0; h < DEVS; ++h) dk[h] = r + LANES * h < D ? argmax_key(dev_sum[h], r + LANES * h) : 0ull;
      kept = 0;
      for (int q = 0; q < n_d; ++q) {
        key_t64 best = dk[0];
#pragma unroll
        for (int h = 1; h < DEVS; ++h) best = dk[h] > best ? dk[h] : best;
        best = token_max<LANES>(best);
        kept |= 1ull << key_index(best);
#pragma unroll
        for (int h = 0; h < DEVS; ++h) dk[h] = dk[h] == best ? 0ull : dk[h];
      }
    }
    // second pass: the k best experts on the surviving devices
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const int e = r + LANES * i;
      const bool ok = (e < E) && ((kept >> s_dev[e < E ? e : 0]) & 1ull);
      key[i] = ok ? argmax_key(v0[i], e) : 0ull;
    }
    for (int s = 0; s < k; ++s) keep_slot(s, select_round());
  }

  // gate values: softmax over all E experts at the selected ones
  constexpr int ROWS = 64 / LANES < EPL ? 64 / LANES : EPL;   // sums of sixteen columns that a lane takes part in: 1, 2 or 4
  float part[ROWS] = {};
#pragma unroll
  for (int i = 0; i < EPL; ++i)
    if (r + LANES * i < E) part[i % ROWS] += exp_ref(v0[i] - mx);
  const float denom = token_sum<LANES>(part);
  const bool second = SLOTS > 1 && k > LANES;   // uniform
  float g[SLOTS] = {r < k ? exp_ref(key_value(slot[0]) - mx) / denom : 0.0f};
  if (second) g[SLOTS - 1] = r + LANES < k ? exp_ref(key_value(slot[SLOTS - 1]) - mx) / denom : 0.0f;
  if (renorm) {
    float sel[1] = {g[0]}, sel2[SLOTS];
#pragma unroll
    for (int h = 0; h < SLOTS; ++h) sel2[h] = g[h];
    const float sum = second ? token_sum<LANES>(sel2) : token_sum<LANES>(sel);
    g[0] = g[0] / sum;
    if (second) g[SLOTS - 1] = g[SLOTS - 1] / sum;
  }
#pragma unroll
  for (int h = 0; h < SLOTS; ++h)
    if (r + LANES * h < k) {
      ids[(size_t)t * k + r + LANES * h] = key_index(slot[h]);
      w[(size_t)t * k + r + LANES * h] = g[h];
    }
}

}  // namespace occult

#pragma clang fp contract(fast)   // the compiler's default again
