// occult_plan: the dispatch plan for all D simulated devices at once
// (paper App. A.2 "Building BRIM_0" and "Building BRIM_1"; Sec. 2.2 replica count).
//
// The printed builders are sequential counters: BRIM_0 numbers (device, token) pairs
// device-major / token-ascending, BRIM_1 numbers (local expert, SFD row) pairs expert-major /
// row-ascending.  Both are stable ranks, so they are computed here without float atomics and in a
// fixed order:
//   pass 1  plan_count : one token per thread; per block of 256 tokens, the set of its tokens that
//                        touch each device and each placement position (bit-or into LDS), and the
//                        sets' sizes;
//   pass 2  plan_scan  : one block turns the [blocks][D+E] counts into exclusive bases
//                        (column scan over blocks, then a scan over devices / positions);
//   pass 3  plan_fill  : every workgroup rebuilds the sets of its block of tokens; a token's rank in a
//                        column is the block's base plus the number of set bits below its own, and
//                        every token writes its own entries of the rank-addressed tables.
// Ranks are token-ascending, which is the order the sequential counters would visit: every table
// is bit-reproducible.  What bounds the planner is the chain of launches and of dependent steps in each,
// so the third pass does the work of the others where every workgroup can afford it: it adds the counts of all
// blocks itself (no scan launch) up to kCountsMaxBlocks blocks, and counts all tokens itself (one launch) up
// to kSingleMaxTokens tokens.
#include "common.h"
#include "route_tokens.h"
#include "stream_gemm.h"

#include <mutex>

namespace occult {

constexpr int kTPB = kPlanTokensPerBlock;   // 256 threads = 4 waves, one token per thread
constexpr int kMaxCols = OCCULT_MAX_D + OCCULT_MAX_E;

// Per block of 256 tokens every column (device j: column j; placement position P: column D + P) gets a 256-bit set
// of the block's tokens that touch it, built in LDS with bit-or (order-free, so deterministic).  A column's count is
// the number of set bits, a token's rank inside its block the number of set bits below its own: the same
// token-ascending ranks the sequential counters give, without a wave vote per column.
typedef unsigned long long TokenSet[4];

__device__ __forceinline__ int bits_below(const unsigned long long* col, int tl) {
  const int tw = tl >> 6;
  const unsigned long long part = (1ull << (tl & 63)) - 1ull;
  int n = 0;
#pragma unroll
  for (int wd = 0; wd < 4; ++wd) n += __popcll(col[wd] & (wd < tw ? ~0ull : (wd == tw ? part : 0ull)));
  return n;
}

// A token's selected placement positions (a position named by several slots counts once, in the last of them) and their
// devices; -1 in unused slots.  k <= KMAX.
template <int KMAX>
struct TokenSlots {
  int pos[KMAX], dev[KMAX];
  unsigned long long devmask;
};

template <int KMAX>
__device__ __forceinline__ void load_token(TokenSlots<KMAX>& ts, const int32_t* __restrict__ ids, int t, int T, int k, int G,
                                           const int* s_pos) {
#pragma unroll
  for (int s = 0; s < KMAX; ++s) ts.pos[s] = (t < T) && (s < k) ? s_pos[ids[(size_t)t * k + s]] : -1;
#pragma unroll
  for (int s = 0; s < KMAX; ++s)
#pragma unroll
    for (int s2 = s + 1; s2 < KMAX; ++s2)
      if (ts.pos[s] >= 0 && ts.pos[s2] == ts.pos[s]) ts.pos[s] = -1;
  ts.devmask = 0;
#pragma unroll
  for (int s = 0; s < KMAX; ++s) {
    ts.dev[s] = ts.pos[s] >= 0 ? ts.pos[s] / G : -1;
    if (ts.pos[s] >= 0) ts.devmask |= 1ull << ts.dev[s];
  }
}

// the token at bit tl of its block joins the sets of its devices and positions
template <int KMAX>
__device__ __forceinline__ void join_sets(TokenSet* s_set, int D, int tl, const TokenSlots<KMAX>& ts) {
  const unsigned long long mybit = 1ull << (tl & 63);
#pragma unroll
  for (int s = 0; s < KMAX; ++s)
    if (ts.pos[s] >= 0) {
      atomicOr(&s_set[D + ts.pos[s]][tl >> 6], mybit);
      atomicOr(&s_set[ts.dev[s]][tl >> 6], mybit);
    }
}

// pass 1: per block of 256 tokens, how many of them touch each device and each placement position
template <int KMAX>
__global__ __launch_bounds__(kTPB) void plan_count(const int32_t* __restrict__ ids, int T, int k, int E, int D, int G,
                                                   const int32_t* __restrict__ expert_pos,
                                                   uint64_t* __restrict__ tok_devmask, int32_t* __restrict__ blk_cnt) {
  static_assert(kTPB == 256, "token sets are four 64-bit words");
  __shared__ int s_pos[OCCULT_MAX_E];
  __shared__ TokenSet s_set[kMaxCols];
  const int tl = threadIdx.x, t = blockIdx.x * kTPB + tl, C = D + E;
  for (int e = tl; e < E; e += kTPB) s_pos[e] = expert_pos ? expert_pos[e] : e;
  for (int i = tl; i < C * 4; i += kTPB) (&s_set[0][0])[i] = 0ull;
  __syncthreads();
  TokenSlots<KMAX> ts;
  load_token<KMAX>(ts, ids, t, T, k, G, s_pos);
  join_sets<KMAX>(s_set, D, tl, ts);
  if (t < T) tok_devmask[t] = ts.devmask;
  __syncthreads();
  for (int c = tl; c < C; c += kTPB)
    blk_cnt[(size_t)blockIdx.x * C + c] =
        __popcll(s_set[c][0]) + __popcll(s_set[c][1]) + __popcll(s_set[c][2]) + __popcll(s_set[c][3]);
}

// One block of 1024 threads.  Thread (part, c) owns rows [part*rpp, (part+1)*rpp) of column c.
constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void plan_scan(
    int32_t* __restrict__ blk_cnt, int nblk, int T, int k, int E, int D, int G,
    const int32_t* __restrict__ expert_pos, int32_t* __restrict__ dev_count,
    int32_t* __restrict__ dev_offset, int32_t* __restrict__ exp_count, int32_t* __restrict__ exp_offset,
    int32_t* __restrict__ pos_expert, uint64_t* __restrict__ counters) {
  __shared__ int s_part[kScanThreads];       // [parts][C] partial column sums
  __shared__ int s_total[kMaxCols];          // column totals
  __shared__ int s_start[kMaxCols + 2];      // exclusive scans: devices, then positions
  const int C = D + E;
  const int parts = kScanThreads / C;        // >= 3 since C <= 320
  const int rpp = (nblk + parts - 1) / parts;
  const int part = threadIdx.x / C, c = threadIdx.x % C;
  const bool active = part < parts;
  const int r0 = part * rpp, r1 = min(nblk, r0 + rpp);

  int sum = 0;
  if (active)
    for (int r = r0; r < r1; ++r) sum += blk_cnt[(size_t)r * C + c];
  if (active) s_part[part * C + c] = sum;
  __syncthreads();

  int base = 0;   // sum of this column over the parts before mine
  if (active)
    for (int p = 0; p < part; ++p) base += s_part[p * C + c];
  if (threadIdx.x < C) {
    int tot = 0;
    for (int p = 0; p < parts; ++p) tot += s_part[p * C + threadIdx.x];
    s_total[threadIdx.x] = tot;
  }
  __syncthreads();

  // exclusive scans over devices and over positions (<= 64 + 256 entries): one thread each
  if (threadIdx.x == 0) {
    int run = 0, mx = 0;
    for (int j = 0; j < D; ++j) {
      s_start[j] = run;
      dev_count[j] = s_total[j];
      dev_offset[j] = run;
      mx = max(mx, s_total[j]);
      run += s_total[j];
    }
    dev_offset[D] = run;
    counters[0] = (uint64_t)run;
    counters[3] = (uint64_t)mx;
  } else if (threadIdx.x == 64) {
    int run = 0, mx = 0;
    for (int P = 0; P < E; ++P) {
      s_start[D + P] = run;
      exp_count[P] = s_total[D + P];
      exp_offset[P] = run;
      mx = max(mx, s_total[D + P]);
      run += s_total[D + P];
    }
    exp_offset[E] = run;
    counters[1] = (uint64_t)run;
    counters[2] = (uint64_t)T * (uint64_t)k;
    counters[4] = (uint64_t)mx;
    counters[5] = counters[6] = counters[7] = 0;
  } else if (threadIdx.x >= 128 && threadIdx.x < 128 + E) {
    const int e = threadIdx.x - 128;
    pos_expert[expert_pos ? expert_pos[e] : e] = e;
  }
  // E can exceed the 896 threads after 128 only if E > 896: not possible (E <= 256)
  __syncthreads();

  if (active) {
    int run = s_start[c] + base;
    for (int r = r0; r < r1; ++r) {
      const int v = blk_cnt[(size_t)r * C + c];
      blk_cnt[(size_t)r * C + c] = run;   // count -> first rank of this block in this column
      run += v;
    }
  }
}

// pass 3.  A workgroup owns FT tokens of a block of 256 and gives every (token, device) and every (token, slot)
// entry a thread of its own: with a token per thread the D + k entries of a token were one thread's chain of LDS reads and
// scattered stores (15 us at any T).  Where the bases come from:
enum class Bases {
  kIds,      // the batch's own ids: every workgroup counts all tokens (T <= kSingleMaxTokens; the only launch)
  kCounts,   // blk holds pass 1's counts: every workgroup adds them up (at most kCountsMaxBlocks blocks)
  kScanned   // blk holds pass 2's ranks of each block's first token
};
// Where the lines lie (us for the whole planner, 64 experts, k = 8, D = 8, calls back to back):
//  - one launch, tokens x workgroups of counting: 256 tokens 7 against 12 with a counting launch, 500 9.6 / 11.9, 1000 14.6 / 12.0;
//  - adding the counts up, blocks x workgroups of reading: 2048 tokens 12.4 against 15.1 with a scan launch, 262144 81 / 98;
//    it grows with the square of the blocks, so the scan keeps what is beyond;
//  - 32 tokens per workgroup against 256, which build a block's sets once instead of eight times: 16384 tokens 17 / 22,
//    32768 21.5 / 23, 65536 33 / 30, 131072 57 / 47.
//  - the same lines for any number of columns, with 320 of them (E = 256, D = 64) as with 72: a scan launch has as many more to
//    walk (three launches with a token per thread in the last / these: 65536 tokens 120 / 69, 262144 404 / 201, 300000 419 / 281; E = 256,
//    D = 8: 72 / 44, 231 / 146, 263 / 241).
// (Three launches with a token per thread in the last: 256 tokens 12 (in one launch of one workgroup), 500 19.6, 16384 23,
// 65536 37, 262144 114.)
constexpr int kSingleMaxTokens = 512;
constexpr int kSmallMaxBlocks = 128;
constexpr int kCountsMaxBlocks = 1024;

// Exclusive scan of the columns' totals and, from one workgroup, the tables that hold them: wave 0 devices, wave 1 positions (64
// at a time, carrying the running total), waves 2 and 3 the inverse placement.
__device__ __forceinline__ void scan_columns(const int* s_total, int* s_start, const int* s_pos, bool write, int T, int k, int E,
                                             int D, const occult_plan_t& p) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave < 2) {
    const int n_cols = wave == 0 ? D : E, col0 = wave == 0 ? 0 : D;
    int32_t* cnt_out = wave == 0 ? p.dev_count : p.exp_count;
    int32_t* off_out = wave == 0 ? p.dev_offset : p.exp_offset;
    int run = 0, mx = 0;
    for (int c0 = 0; c0 < n_cols; c0 += 64) {
      const int c = c0 + lane;
      const int n = c < n_cols ? s_total[col0 + c] : 0;
      int incl = n;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      if (c < n_cols) {
        s_start[col0 + c] = run + incl - n;
        if (write) {
          cnt_out[c] = n;
          off_out[c] = run + incl - n;
        }
      }
      if (write) {   // uniform over the workgroup
        int m = n;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
        mx = max(mx, m);
      }
      run += __shfl(incl, 63, 64);
    }
    if (write && lane == 0) {
      off_out[n_cols] = run;
      if (wave == 0) {
        p.counters[0] = (uint64_t)run;
        p.counters[3] = (uint64_t)mx;
      } else {
        p.counters[1] = (uint64_t)run;
        p.counters[2] = (uint64_t)T * (uint64_t)k;
        p.counters[4] = (uint64_t)mx;
        p.counters[5] = p.counters[6] = p.counters[7] = 0;
      }
    }
  } else if (write) {
    for (int e = threadIdx.x - 128; e < E; e += kTPB - 128) p.pos_expert[s_pos[e]] = e;
  }
}

// The rows that plan_fill copies on the side: occult_dispatch's work for batches whose planner is one launch.
struct Rows {
  const u32x4* x;
  u32x4* sfd_x;
  int vecs;   // 16-byte vectors of a row, <= 64 * VPL
};

// FT: tokens of a workgroup.  VPL > 0: a wave has a token, whose row it requests at the start and copies to the SFD rows once
// it knows them (plan and dispatch in two launches, both chains of latencies: see launch_plan_dispatch).
template <int KMAX, Bases FROM, int FT, int VPL>
__device__ __forceinline__ void fill_block(int wg, const int32_t* __restrict__ ids, const float* __restrict__ w, int T, int k, int E,
                                           int D, int G, int M1, int nblk, const int32_t* __restrict__ expert_pos,
                                           const int32_t* __restrict__ blk, const occult_plan_t& p, const Rows& rows) {
  static_assert(VPL == 0 || FT == kTPB / 64, "a token per wave");
  constexpr int PER_BLOCK = kTPB / FT;   // workgroups that share a block of 256 tokens
  __shared__ int s_pos[OCCULT_MAX_E];
  __shared__ TokenSet s_set[kMaxCols];
  __shared__ int s_before[kMaxCols];   // tokens of the blocks before mine in each column
  __shared__ int s_total[kMaxCols];    // all tokens
  __shared__ int s_base[kMaxCols];     // rank of my block's first token
  __shared__ int s_slot[FT][KMAX];   // my tokens' slots: device << 16 | position, or -1
  const int tl = threadIdx.x, C = D + E;
  const int block = wg / PER_BLOCK, first = (wg % PER_BLOCK) * FT;   // first: my first bit
  const int t0 = block * kTPB;
  const int lane = tl & 63, wave = tl >> 6;
  u32x4 v[VPL > 0 ? VPL : 1];   // VPL: the row of token t0 + first + wave
  if constexpr (VPL > 0) {
    if (t0 + first + wave < T) {
      const u32x4* src = rows.x + (size_t)(t0 + first + wave) * rows.vecs;
#pragma unroll
      for (int i = 0; i < VPL; ++i)
        if (lane + 64 * i < rows.vecs) v[i] = __builtin_nontemporal_load(src + lane + 64 * i);
    }
  }
  for (int e = tl; e < E; e += kTPB) s_pos[e] = expert_pos ? expert_pos[e] : e;
  for (int i = tl; i < C * 4; i += kTPB) (&s_set[0][0])[i] = 0ull;
  for (int c = tl; c < C; c += kTPB) {
    s_before[c] = s_total[c] = 0;
    if (FROM == Bases::kScanned) s_base[c] = blk[(size_t)block * C + c];
  }
  __syncthreads();
  {
    TokenSlots<KMAX> ts;
    load_token<KMAX>(ts, ids, t0 + tl, T, k, G, s_pos);
    join_sets<KMAX>(s_set, D, tl, ts);
    if (tl >= first && tl < first + FT) {
#pragma unroll
      for (int s = 0; s < KMAX; ++s) s_slot[tl - first][s] = ts.pos[s] >= 0 ? ts.dev[s] << 16 | ts.pos[s] : -1;
      if (FROM == Bases::kIds && t0 + tl < T) p.tok_devmask[t0 + tl] = ts.devmask;
    }
  }
  if constexpr (FROM == Bases::kIds) {
    for (int b = 0; b < nblk; ++b) {   // the other blocks' tokens, before mine and after
      if (b == block) continue;
      TokenSlots<KMAX> ts;
      load_token<KMAX>(ts, ids, b * kTPB + tl, T, k, G, s_pos);
      int* into = b < block ? s_before : s_total;
#pragma unroll
      for (int s = 0; s < KMAX; ++s)
        if (ts.pos[s] >= 0) atomicAdd(&into[D + ts.pos[s]], 1);
      for (unsigned long long m = ts.devmask; m != 0; m &= m - 1) atomicAdd(&into[__ffsll((long long)m) - 1], 1);
    }
    __syncthreads();
    for (int c = tl; c < C; c += kTPB)
      s_total[c] += s_before[c] + __popcll(s_set[c][0]) + __popcll(s_set[c][1]) + __popcll(s_set[c][2]) + __popcll(s_set[c][3]);
  }
  if constexpr (FROM == Bases::kCounts) {
    const int parts = max(1, kTPB / C), rpp = (nblk + parts - 1) / parts;
    for (int i = tl; i < C * parts; i += kTPB) {
      const int c = i % C, r0 = i / C * rpp, r1 = min(nblk, r0 + rpp);
      int before = 0, total = 0;
#pragma unroll 8
      for (int r = r0; r < r1; ++r) {
        const int v = blk[(size_t)r * C + c];
        total += v;
        before += r < block ? v : 0;
      }
      atomicAdd(&s_total[c], total);   // integer sums: any order
      atomicAdd(&s_before[c], before);
    }
  }
  if constexpr (FROM != Bases::kScanned) {
    __syncthreads();
    scan_columns(s_total, s_base, s_pos, wg == 0, T, k, E, D, p);
    __syncthreads();
    for (int c = tl; c < C; c += kTPB) s_base[c] += s_before[c];
  }
  __syncthreads();

  // (token, device): the token's row of destinations, the row's token, the unused end of the row's merge list
  const int mine = min(FT, T - t0 - first);   // may be <= 0
  const int entries = VPL > 0 ? mine * 64 : mine * D;   // VPL: lane j of a wave for device j of its token (D <= 64)
  int my_row = -1;                                      // VPL: of this lane's device
  for (int i = tl; i < entries; i += kTPB) {
    const int m = VPL > 0 ? wave : i / D, j = VPL > 0 ? lane : i - m * D;
    if (VPL > 0 && j >= D) continue;
    int filled = 0;
#pragma unroll
    for (int s = 0; s < KMAX; ++s) filled += s_slot[m][s] >> 16 == j ? 1 : 0;   // (unused slots: -1 >> 16 = -1)
    const int r = filled > 0 ? s_base[j] + bits_below(s_set[j], first + m) : -1;
    p.tok_sfd_row[(size_t)(t0 + first + m) * D + j] = r;
    my_row = r;
    if (filled > 0) {
      p.sfd_token[r] = t0 + first + m;
      for (int e = filled; e < M1; ++e) p.sfd_epd_rows[(size_t)r * M1 + e] = -1;
    }
  }
  // (token, slot): the EPD row's source and gate, its entry of the merge list (position-ascending)
  for (int i = tl; i < mine * k; i += kTPB) {
    const int m = i / k, s = i - m * k, slot = s_slot[m][s];
    if (slot < 0) continue;
    const int j = slot >> 16, P = slot & 0xFFFF;
    const int r = s_base[j] + bits_below(s_set[j], first + m);
    const int q = s_base[D + P] + bits_below(s_set[D + P], first + m);
    int before = 0;   // this token's other positions on the same device below P
#pragma unroll
    for (int s2 = 0; s2 < KMAX; ++s2) {
      const int other = s_slot[m][s2];
      before += (other >> 16 == j && other < slot) ? 1 : 0;
    }
    p.epd_sfd_row[q] = r;
    p.epd_gate[q] = w[(size_t)(t0 + first) * k + i];
    p.sfd_epd_rows[(size_t)r * M1 + before] = q;
  }
  if constexpr (VPL > 0) {
    if (wave >= mine) return;
    for (int j = 0; j < D; ++j) {
      const int r = __builtin_amdgcn_readlane(my_row, j);
      if (r < 0) continue;
      u32x4* dst = rows.sfd_x + (size_t)r * rows.vecs;
#pragma unroll
      for (int i = 0; i < VPL; ++i)
        if (lane + 64 * i < rows.vecs) __builtin_nontemporal_store(v[i], dst + lane + 64 * i);
    }
  }
}

template <int KMAX, Bases FROM, int FT, int VPL>
__global__ __launch_bounds__(kTPB) void plan_fill(const int32_t* __restrict__ ids, const float* __restrict__ w, int T, int k,
                                                  int E, int D, int G, int M1, int nblk, const int32_t* __restrict__ expert_pos,
                                                  const int32_t* __restrict__ blk, const occult_plan_t p, const Rows rows) {
  fill_block<KMAX, FROM, FT, VPL>((int)blockIdx.x, ids, w, T, k, E, D, G, M1, nblk, expert_pos, blk, p, rows);
}

// A forward pass of at most kFrontTokens tokens up to the gate/up product in ONE launch: workgroups [0, plan_blocks) plan and copy
// rows as plan_fill does, the next a_blocks stream the routed experts' weights, the others the shared experts'.  Each of the first
// two kinds routes all tokens for itself, four at a time: a chain of about 2 us, in place of a launch of that length, one of 6 us and the
// gaps behind both.  The products read the rows of x that the plan's tables name as copies; same bits.
// Which batches (us per pass, separate / this, three layers in turn; d = 2048 unless given):
//  - up to 4 tokens, one round of routing: all with up to 2560 workgroups that route, or 6 d.  1 token: 60 + 4 experts of f = 1408, k = 4
//    53.0 / 44.0, 64 of 1024, k = 8 47.0 / 37.4, 256 of 512, d = 512 33.3 / 24.6; 4 tokens 75.2 / 65.0, 81.6 / 72.8, 36.9 / 27.2; pruned
//    92.7 / 84.0.  4 tokens, 64 experts, k = 8: 2560 workgroups, d = 64 48.0 / 48.0, 256 67.2 / 65.2; 3072, d = 64 53.1 / 54.8, 256 76.7 / 78.2;
//    4096, d = 64 62.9 / 68.5, 512 111 / 116, 1024 170 / 165, 2048 258 / 248; 6144, d = 1024 228 / 227, 2048 382 / 368.
//  - more where the workgroups that route are few for what each of them streams (128 bytes per element of K), since every round of them
//    over the CUs routes again: 8 tokens of 60 + 4 113 / 107, 64 + 2 135 / 125, 64 of 1024 116 / 110, d = 1024 and f = 704 53 / 45; 12 tokens
//    139 / 131, d = 4096 330 / 320, 64 of 1024 139 / 138.  Past the line: d = 1024, f = 1408, k = 8, 8 tokens 94 / 96, d = 512 66 / 72; 16 tokens
//    of 64 of 1024 147 / 149.  Not with a second round of selection or more than 64 experts to look at: 8 tokens pruned 130 / 134 and, by
//    similarity, 134 / 148, 256 experts of f = 1024, d = 1024 93 / 100.
constexpr int kFrontTokens = 12, kFrontSlots = 8;

template <int EPL, bool PRUNE, int VPL>
struct Few {
  static constexpr bool kOn = true;
  const float* logits;
  int T, E, k, D, G, M1;
  const int32_t* expert_pos;
  int n_d, prune_mode, renorm;
  const int32_t* sim_table;
  int32_t* ids;
  float* w;
  occult_plan_t p;
  Rows rows;
  int plan_blocks;

  struct Shared {
    int ids[kFrontTokens * kFrontSlots];
    float w[kFrontTokens * kFrontSlots];
    unsigned tokens[OCCULT_MAX_E];   // of each position, as bits
    int expert[OCCULT_MAX_E];        // at each position
  };
  __device__ static Shared& shared() {
    __shared__ Shared s;
    return s;
  }

  // true: the workgroup was one of the plan's
  __device__ __forceinline__ bool begin(int bid, int a_blocks) const {
    if (bid >= plan_blocks + a_blocks) return false;   // the shared experts' need no routing
    Shared& s = shared();
    const int tid = threadIdx.x;
    const bool plans = bid < plan_blocks;
    if (!plans)
      for (int e = tid; e < E; e += kTPB) {
        s.tokens[e] = 0;
        s.expert[expert_pos ? expert_pos[e] : e] = e;
      }
    for (int b = 0; b * 4 < T; ++b)
      route_tokens<64, EPL, PRUNE>(b, logits, T, E, k, D, G, expert_pos, n_d, prune_mode, renorm, sim_table, s.ids, s.w);
    __syncthreads();
    if (plans) {
      if (bid == 0 && tid < T * k) {
        ids[tid] = s.ids[tid];
        w[tid] = s.w[tid];
      }
      fill_block<kFrontSlots, Bases::kIds, 4, VPL>(bid, s.ids, s.w, T, k, E, D, G, M1, 1, expert_pos, nullptr, p, rows);
      return true;
    }
    if (tid < T * k) {
      const int e = s.ids[tid];
      atomicOr(&s.tokens[expert_pos ? expert_pos[e] : e], 1u << (tid / k));
    }
    __syncthreads();
    return false;
  }

  // the mt-th position that has rows (they are one tile); every wave for itself, wave-uniform.  group = -1: there are fewer
  __device__ __forceinline__ TileInfo tile(int mt) const {
    static_assert(kFrontTokens <= 32, "a position's tokens are the bits of a word, its rows one tile of the kernel");
    const unsigned* tokens = shared().tokens;
    const int lane = threadIdx.x & 63;
    TileInfo ti{-1, 0, 0, 0};
    for (int c0 = 0; c0 < E; c0 += 64) {
      const int n = c0 + lane < E ? __popc(tokens[c0 + lane]) : 0;
      unsigned long long active = __ballot(n > 0);
      const int here = __popcll(active);
      int at = 64;   // the position's lane, if it is among these
      if (mt < here) {
        for (int i = 0; i < mt; ++i) active &= active - 1;
        at = __ffsll((long long)active) - 1;
      }
      int before = lane < at ? n : 0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) before += __shfl_xor(before, o, 64);
      ti.row_base += before;
      if (at < 64) {
        ti.group = c0 + at;
        ti.rows = __shfl(n, at, 64);
        break;
      }
      mt -= here;
    }
    return ti;
  }
  __device__ __forceinline__ int matrix(int group) const { return shared().expert[group]; }
  __device__ __forceinline__ unsigned row(int group, int lr) const {   // the token of its row lr
    unsigned m = shared().tokens[group];
    for (int i = 0; i < lr; ++i) m &= m - 1;
    return __ffs((int)m) - 1;
  }
};

size_t plan_workspace_bytes(const occult_cfg_t& c);

#define OCC_PLAN_KMAX(LAUNCH)       \
  do {                              \
    if (c.k <= 8) LAUNCH(8);        \
    else if (c.k <= 16) LAUNCH(16); \
    else LAUNCH(32);                \
  } while (0)
#define OCC_PLAN_FILL(KM, FROM, FT, VPL)                                                                                 \
  hipLaunchKernelGGL((plan_fill<KM, FROM, FT, VPL>), dim3((unsigned)(c.T > 0 ? ((long long)c.T + FT - 1) / FT : 1)),     \
                     dim3(kTPB), 0, s, ids, w, c.T, c.k, c.E, c.D, G, merge_width(c), nblk, c.expert_pos, blk, p, rows)

// The launches of the planner on a block-count buffer `blk` of >= nblk * (D + E) ints.  plan_count writes every entry of the
// first nblk rows before they are read: the buffer need not be cleared.
static int launch_plan(const occult_cfg_t& c, const int32_t* ids, const float* w, const occult_plan_t& p,
                       int32_t* blk, hipStream_t s) {
  const int G = c.E / c.D;
  const int nblk = (c.T + kTPB - 1) / kTPB;
  const Rows rows{};
  const Bases from = c.T <= kSingleMaxTokens ? Bases::kIds : nblk <= kCountsMaxBlocks ? Bases::kCounts : Bases::kScanned;
  if (from != Bases::kIds) {
#define OCC_PLAN_COUNT(KM)                                                                               \
  hipLaunchKernelGGL(plan_count<KM>, dim3(nblk), dim3(kTPB), 0, s, ids, c.T, c.k, c.E, c.D, G, c.expert_pos, \
                     p.tok_devmask, blk)
    OCC_PLAN_KMAX(OCC_PLAN_COUNT);
#undef OCC_PLAN_COUNT
    OCC_LAUNCH_CHECK("plan_count");
  }
  if (from == Bases::kScanned) {
    hipLaunchKernelGGL(plan_scan, dim3(1), dim3(kScanThreads), 0, s, blk, nblk, c.T, c.k, c.E, c.D, G,
                       c.expert_pos, p.dev_count, p.dev_offset, p.exp_count, p.exp_offset, p.pos_expert,
                       p.counters);
    OCC_LAUNCH_CHECK("plan_scan");
  }
#define OCC_PLAN_FILL_IDS(KM) OCC_PLAN_FILL(KM, Bases::kIds, 32, 0)   // T = 0: one workgroup writes zero counts and offsets
#define OCC_PLAN_FILL_COUNTS(KM) OCC_PLAN_FILL(KM, Bases::kCounts, 32, 0)
#define OCC_PLAN_FILL_MANY(KM) OCC_PLAN_FILL(KM, Bases::kCounts, kTPB, 0)
#define OCC_PLAN_FILL_SCANNED(KM) OCC_PLAN_FILL(KM, Bases::kScanned, kTPB, 0)
  if (from == Bases::kIds) OCC_PLAN_KMAX(OCC_PLAN_FILL_IDS);
  else if (from == Bases::kScanned) OCC_PLAN_KMAX(OCC_PLAN_FILL_SCANNED);
  else if (nblk <= kSmallMaxBlocks) OCC_PLAN_KMAX(OCC_PLAN_FILL_COUNTS);
  else OCC_PLAN_KMAX(OCC_PLAN_FILL_MANY);
#undef OCC_PLAN_FILL_IDS
#undef OCC_PLAN_FILL_COUNTS
#undef OCC_PLAN_FILL_MANY
#undef OCC_PLAN_FILL_SCANNED
  OCC_LAUNCH_CHECK("plan_fill");
  return OCCULT_OK;
}

// Planner and row copies of at most kSingleMaxTokens tokens in one launch (us per forward pass, separate / together: 1 token
// of 60 experts 44.8 / 44.3, 8 of 64 119.8 / 118.3, 128 234.2 / 233.1, 256 246.9 / 244.1, 512 309.7 / 307.3; 256 tokens of the small
// f32 layer 29.9 / 28.4).  Rows of more than 8 KiB do not fit a wave's registers and are copied by the other kernel.
static int launch_plan_dispatch(const occult_cfg_t& c, const int32_t* ids, const float* w, const occult_plan_t& p,
                                const Rows& rows, hipStream_t s) {
  const int G = c.E / c.D;
  const int nblk = (c.T + kTPB - 1) / kTPB;
  const int32_t* blk = nullptr;   // (not read with kIds)
  const int vpl = (rows.vecs + 63) / 64;
#define OCC_PLAN_ROWS_1(KM) OCC_PLAN_FILL(KM, Bases::kIds, 4, 1)
#define OCC_PLAN_ROWS_2(KM) OCC_PLAN_FILL(KM, Bases::kIds, 4, 2)
#define OCC_PLAN_ROWS_4(KM) OCC_PLAN_FILL(KM, Bases::kIds, 4, 4)
#define OCC_PLAN_ROWS_8(KM) OCC_PLAN_FILL(KM, Bases::kIds, 4, 8)
  if (vpl <= 1) OCC_PLAN_KMAX(OCC_PLAN_ROWS_1);
  else if (vpl <= 2) OCC_PLAN_KMAX(OCC_PLAN_ROWS_2);
  else if (vpl <= 4) OCC_PLAN_KMAX(OCC_PLAN_ROWS_4);
  else OCC_PLAN_KMAX(OCC_PLAN_ROWS_8);
#undef OCC_PLAN_ROWS_1
#undef OCC_PLAN_ROWS_2
#undef OCC_PLAN_ROWS_4
#undef OCC_PLAN_ROWS_8
  OCC_LAUNCH_CHECK("plan_fill");
  return OCCULT_OK;
}
#undef OCC_PLAN_FILL
#undef OCC_PLAN_KMAX

static int check_plan_args(const occult_cfg_t& c, const int32_t* ids, const float* w, const occult_plan_t* plan) {
  OCC_REQUIRE(plan, OCCULT_ENULLPTR, "plan is NULL");
  const occult_plan_t& p = *plan;
  OCC_REQUIRE(p.tok_devmask && p.dev_count && p.dev_offset && p.tok_sfd_row && p.sfd_token &&
                  p.exp_count && p.exp_offset && p.pos_expert && p.epd_sfd_row && p.epd_gate &&
                  p.sfd_epd_rows && p.counters,
              OCCULT_ENULLPTR, "a plan table is NULL (use occult_plan_bind)");
  OCC_REQUIRE(c.T == 0 || (ids && w), OCCULT_ENULLPTR, "ids or w is NULL");
  return OCCULT_OK;
}

// Scratch of occult_plan_static: the planner's per-block counts in a device array of the library
// itself (4 MiB on every GPU the library runs on, held until the process ends).  On the host this
// name only stands for the array: its device address comes from hipGetSymbolAddress, once per
// device, and is what the kernels receive.
constexpr size_t kStaticPlanInts = (size_t)OCCULT_PLAN_STATIC_MAX_BYTES / sizeof(int32_t);
static __device__ __align__(256) int32_t scratch[kStaticPlanInts];

constexpr int kMaxHipDevices = 64;
static std::mutex g_scratch_mutex;
static int32_t* g_scratch_ptr[kMaxHipDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call for that device).
static int static_scratch(int32_t** out) {
  int dev = -1;
  OCC_HIP(hipGetDevice(&dev));
  OCC_REQUIRE(dev >= 0 && dev < kMaxHipDevices, OCCULT_EINVAL, "HIP device %d outside 0..%d", dev, kMaxHipDevices - 1);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    OCC_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    OCC_REQUIRE(ptr, OCCULT_EHIP, "hipGetSymbolAddress returned a NULL address for the planner's scratch");
    g_scratch_ptr[dev] = static_cast<int32_t*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return OCCULT_OK;
}

}  // namespace occult

using namespace occult;

static int check_plan_ws_args(const occult_cfg_t* cfg, const int32_t* ids, const float* w, const occult_plan_t* plan, void* ws,
                              size_t ws_bytes) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  rc = check_plan_args(c, ids, w, plan);
  if (rc) return rc;
  OCC_REQUIRE(ws, OCCULT_ENULLPTR, "workspace is NULL");
  OCC_REQUIRE(ws_bytes >= plan_workspace_bytes(c), OCCULT_EWORKSPACE, "workspace of %zu bytes < required %zu",
              ws_bytes, plan_workspace_bytes(c));
  return OCCULT_OK;
}

namespace occult {
// routed workgroups of the launch: a tile per position with rows
static long long front_blocks(const occult_cfg_t& c) { return (long long)min_i(c.T * c.k, c.E) * (c.f / skinny::BN_OUT); }

bool fits_front(const occult_cfg_t& c) {
  if (c.T < 1 || c.T > kFrontTokens || c.k > kFrontSlots || (size_t)c.d * elem_size(c) / 16 > 64 * 8) return false;
  if (c.T <= 4) return front_blocks(c) <= 2560 || front_blocks(c) <= 6ll * c.d;
  return c.n_d == 0 && c.E <= 64 && 10 * front_blocks(c) <= 11ll * c.d;
}

int check_plan_dispatch_args(const occult_cfg_t* cfg, const int32_t* ids, const float* w, const occult_plan_t* plan, void* ws,
                             size_t ws_bytes, const void* x, const void* sfd_x) {
  const int rc = check_plan_ws_args(cfg, ids, w, plan, ws, ws_bytes);
  return rc ? rc : check_dispatch_args(*cfg, plan, x, sfd_x);
}

int launch_front(const occult_cfg_t& c, const float* logits, int32_t* ids, float* w, const occult_plan_t& p, const void* x, void* sfd_x,
                 const GemmArgs& first, const GemmArgs* second, hipStream_t s) {
  const int vecs = c.d * elem_size(c) / 16, plan_blocks = (c.T + 3) / 4;
  const int a_blocks = (int)front_blocks(c);
  const Rows rows{static_cast<const u32x4*>(x), static_cast<u32x4*>(sfd_x), vecs};
  const long long blocks = plan_blocks + a_blocks + (second ? skinny::second_blocks(*second) : 0);
  OCC_REQUIRE(blocks < (1ll << 31), OCCULT_EINVAL, "grouped GEMM grid too large");
  const dim3 grid((unsigned)blocks), block(kTPB);
  const bool prune = c.n_d > 0, packed = first.Bp != nullptr, wide = vecs > 64 * 4, many = c.E > 64;
#define OCC_FRONT(N, P, V, K)                                                                                                \
  hipLaunchKernelGGL((skinny::grouped_gemm_bf16<true, 2, K, true, Few<N, P, V>>), grid, block, 0, s, first,                  \
                     second ? *second : first, a_blocks,                                                                     \
                     (Few<N, P, V>{logits, c.T, c.E, c.k, c.D, c.E / c.D, merge_width(c), c.expert_pos, c.n_d, c.prune_mode, \
                                   c.renorm, c.sim_table, ids, w, p, rows, plan_blocks}))
#define OCC_FRONT_K(N, P, V)              \
  do {                                    \
    if (packed) OCC_FRONT(N, P, V, true); \
    else OCC_FRONT(N, P, V, false);       \
  } while (0)
#define OCC_FRONT_V(N, P)           \
  do {                              \
    if (wide) OCC_FRONT_K(N, P, 8); \
    else OCC_FRONT_K(N, P, 4);      \
  } while (0)
#define OCC_FRONT_P(N)                \
  do {                                \
    if (prune) OCC_FRONT_V(N, true);  \
    else OCC_FRONT_V(N, false);       \
  } while (0)
  if (many) OCC_FRONT_P(4);
  else OCC_FRONT_P(1);
#undef OCC_FRONT_P
#undef OCC_FRONT_V
#undef OCC_FRONT_K
#undef OCC_FRONT
  OCC_LAUNCH_CHECK("grouped_gemm");
  return OCCULT_OK;
}

int plan_and_dispatch(const occult_cfg_t* cfg, const int32_t* ids, const float* w, const occult_plan_t* plan, void* ws,
                      size_t ws_bytes, const void* x, void* sfd_x, hipStream_t s) {
  int rc = check_plan_ws_args(cfg, ids, w, plan, ws, ws_bytes);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  const size_t vecs = (size_t)c.d * elem_size(c) / 16;
  if (c.T == 0 || c.T > kSingleMaxTokens || vecs > 64 * 8) {
    rc = launch_plan(c, ids, w, *plan, static_cast<int32_t*>(ws), s);
    return rc ? rc : occult_dispatch(cfg, plan, x, sfd_x, s);
  }
  rc = check_dispatch_args(c, plan, x, sfd_x);
  if (rc) return rc;
  return launch_plan_dispatch(c, ids, w, *plan, Rows{static_cast<const u32x4*>(x), static_cast<u32x4*>(sfd_x), (int)vecs}, s);
}
}  // namespace occult

extern "C" int occult_plan(const occult_cfg_t* cfg, const int32_t* ids, const float* w,
                           const occult_plan_t* plan, void* ws, size_t ws_bytes, occult_stream_t stream) {
  const int rc = check_plan_ws_args(cfg, ids, w, plan, ws, ws_bytes);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  return launch_plan(c, ids, w, *plan, static_cast<int32_t*>(ws), static_cast<hipStream_t>(stream));
}

extern "C" int occult_plan_static(const occult_cfg_t* cfg, const int32_t* ids, const float* w,
                                  const occult_plan_t* plan, occult_stream_t stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  const size_t need = plan_workspace_bytes(c);
  OCC_REQUIRE(need <= (size_t)OCCULT_PLAN_STATIC_MAX_BYTES, OCCULT_EWORKSPACE,
              "this layer's planner scratch (%zu bytes for T=%d, D+E=%d) exceeds the %zu bytes of the built-in "
              "buffer: use occult_plan with a caller workspace",
              need, c.T, c.D + c.E, (size_t)OCCULT_PLAN_STATIC_MAX_BYTES);
  rc = check_plan_args(c, ids, w, plan);
  if (rc) return rc;
  int32_t* blk = nullptr;
  rc = static_scratch(&blk);
  if (rc) return rc;
  return launch_plan(c, ids, w, *plan, blk, static_cast<hipStream_t>(stream));
}
