// Grouped expert GEMM, 128-row tiles: groups of a few dozen to a few hundred rows (a prompt chunk, a training
// micro-batch), where every expert's weights have to come from HBM for few rows each, and where 256-row tiles would
// be mostly padding.  Same products as ffn.hip (argument block in gemm.h), bf16 only.
#include "common.h"
#include "gemm.h"

#include <type_traits>

namespace occult {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Block = 256 threads = 4 waves (2 x 2), block tile 128 token rows x 256 weight rows, wave tile 64 x 128 = 4 x 8
// v_mfma_f32_16x16x32_bf16 tiles (128 accumulator registers per lane), one persistent block per CU.
//
// What bounds it: the weights' way from HBM while groups are small, the operand stream from L2 into LDS (48 KiB per K
// tile of 64 and 1024 matrix-pipe cycles) when they are not.  The operands go through a ring of three 48 KiB stages
// (global_load_lds), K tile j+3 requested as soon as every wave has read the last fragments of K tile j, so two K tiles
// are in flight at any time; a block walks its output tiles as one stream of K tiles, so the loads go on through the
// end of a tile and its epilogue.  Rows of a K tile are whole 128-byte lines: a first version with two blocks per CU and
// 64-byte rows (K tiles of 32) made twice the L2 requests and was bound by them.  16-byte chunk c of row r lives in slot
// c ^ ((r >> 1) & 7) of its LDS row: conflict-free for the fragment reads (ffn.hip).
//
// Order of the tiles: group by group, weight columns outside, row tiles inside, cut into eight equal runs, one per
// XCD (workgroups go to the XCDs round-robin).  The row tiles of one expert and weight block so run next to each
// other on one XCD and the weights leave HBM once; and no XCD gets a whole tile more than an eighth of both problems'.
//
// What is left of an XCD's run beyond whole rounds of its blocks is cut in two by columns where every half then still finds
// a block of its own (`halved`): a lone round costs the time of a whole tile whoever takes part in it, a half tile little more than
// half of that.  Its K loop multiplies half of the weight rows, and the ring's stages hold so many fewer.
// (gate/up product of 500 tokens of 64 + 2 experts, d = 2048, f = 1408, 24 tiles beyond three rounds: 161 us, 140 without these tiles, 150
// in halves, pass 273 -> 265; K = 1408 of a training step's 1000 tokens 107 -> 98.  More than half a round is left whole: the halves
// would need a second one.)
//
// One launch carries two problems of the same N: `second` (uniform groups: the shared experts) has its tiles at the
// front of every XCD's run because its K can be longer (the shared down projection walks S matrices).
namespace t128 {
constexpr int BM = 128, BN = 256, BK = 64, NST = 3;
constexpr int A_BYTES = BM * BK * 2;                // 16 KiB
constexpr int STAGE_BYTES = A_BYTES + BN * BK * 2;  // 48 KiB: token rows, then weight rows
constexpr int OUT_BYTES = 2048;                     // per wave: 16 rows x 64 output columns on their way out

__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// silu(g) * u in the form of the kernel that the rows of a group would otherwise take (silu_rcp, wave-uniform): with the
// 256-row tiles' hardware reciprocal (swiglu_rcp), or with the f32 division of the weight-streaming and small-tile kernels
__device__ __forceinline__ float swiglu_div(float g, float u) { return g / (1.0f + __expf(-g)) * u; }

// one output tile; every field is wave-uniform
struct Tile {
  int valid, is_second, group, m0, n0, rows, row_base, widx, half;   // half: BN_OUT / 2 columns from n0
};

// SAVE (with SWIGLU): the gate and up pre-activations are stored too (C2).
// PARTS: a problem's K may be summed in parts (GemmArgs.ksplit), whose sums are added in order: a result so has the bits
// that the weight-streaming or small-tile kernel gives the same rows.  The finished parts' sums have registers of
// their own (one wave per SIMD: there is room) and cost one addition per accumulator and part (500 tokens of 64 + 2 experts,
// shared down projection in parts: 312 -> 318 us; 300 of 60 + 4, gate/up in quarters as well: 305 -> 325 us).
// ONCE: the weights are requested, and the output stored, as not to be kept (launch_tile128).
// ROUNDS: with the half tiles and `span` (launch_tile128 says where).  One wave per SIMD hides no instruction, so their price is what a
// launch executes besides: about 0.4 us (1.3 before the two kinds of tiles shared one epilogue, whose copy alone cost 0.7,
// and the first tile was looked up without them).  Forward of 1280 tokens of 64 experts, d = 512, f = 448, none of them halved:
// 63.6 us without, 64.3 with, 66.1 then.
template <bool SWIGLU, bool SAVE, bool PARTS, bool ONCE, bool ROUNDS>
__global__ __launch_bounds__(256, 1) void grouped_gemm_bf16(const GemmArgs first, const GemmArgs second) {
  static_assert(SWIGLU || !SAVE, "pre-activations exist only with the fused activation");
  static_assert(!SAVE || !PARTS, "stored pre-activations are one sum over K");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE_BYTES];
  __shared__ __attribute__((aligned(16))) char s_out[4][OUT_BYTES];
  __shared__ int s_idx[4][64];               // source rows of the next tile's token rows, per loading wave
  __shared__ int s_goff[OCCULT_MAX_E + 1];   // first's row offsets and, before each group, its tile count
  __shared__ int s_tpre[OCCULT_MAX_E + 1];
  constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int n_tiles = (unsigned)(first.N + BN_OUT - 1) / BN_OUT;

  for (int i = tid; i <= first.ngroups; i += 256) s_goff[i] = first.grp_offset[i];
  if (wave == 0) {
    int before = 0;
    for (int c0 = 0; c0 < first.ngroups; c0 += 64) {
      const int g = c0 + lane;
      const int nt = g < first.ngroups ? (unsigned)(first.grp_offset[g + 1] - first.grp_offset[g] + BM - 1) / BM * n_tiles : 0;
      int incl = nt;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      if (g < first.ngroups) s_tpre[g] = before + incl - nt;
      before += __shfl(incl, 63, 64);
    }
    if (lane == 0) s_tpre[first.ngroups] = before;
  }
  __syncthreads();

  // this XCD's runs of the two problems' tiles: an eighth of each, the tiles left over of `second` one each to the first XCDs
  // and those of `first` to the last ones
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3;
  const unsigned mt2 = (unsigned)(second.M + BM - 1) / BM;   // (unsigned divisions are half as long)
  const int total1 = s_tpre[first.ngroups], total2 = second.ngroups * mt2 * n_tiles;   // host: their sum is below 2^28
  const int over1 = total1 & 7, over2 = total2 & 7;
  const int cnt1 = __builtin_amdgcn_readfirstlane((total1 >> 3) + (xcd >= 8 - over1));
  const int lo1 = __builtin_amdgcn_readfirstlane(xcd * (total1 >> 3) + max(0, xcd - (8 - over1)));
  const int cnt2 = (total2 >> 3) + (xcd < over2), lo2 = xcd * (total2 >> 3) + min(xcd, over2);
  // A tile of `second` with a longer K stands for `span` tiles of `first`: its block takes the next one so many rounds later.  (Shared
  // down projection of two experts beside 64, K = 2816 against 1408, d = 2048: forward of 500 tokens 265 -> 253 us, where it
  // now joins the launch, of 1000 tokens 303 -> 288)
  const int span = ROUNDS && cnt2 <= stride ? second.span : 1;
  int whole = 0;   // slots of whole rounds
  bool halved = false;
  // a block's first tile is a whole one of round 0: what the others take to find is left until its loads are on their way
  auto tile_at = [&](auto first_, int slot, int round) {
    constexpr bool FIRST = decltype(first_)::value;
    Tile t{};
    int second_half = 0;
    if (!FIRST && halved && slot >= whole) {
      t.half = 1;
      second_half = (slot - whole) & 1;
      slot = whole + ((slot - whole) >> 1);
    }
    if (slot < cnt2) {
      const unsigned n = lo2 + slot, per_group = mt2 * n_tiles, within = n % per_group;
      t.valid = t.is_second = 1;
      t.group = n / per_group;
      t.m0 = within % mt2 * BM; t.n0 = within / mt2 * BN_OUT;
      t.rows = second.M;
      t.widx = second.w_base + t.group;
    } else if (const int n1 = slot - cnt2 * (FIRST || !ROUNDS ? 1 : min(round + 1, span)); n1 < cnt1) {   // (slots of `second` in the rounds up to this one)
      const int n = lo1 + n1;
      for (int c0 = 0; c0 < first.ngroups; c0 += 64) {
        const int g = c0 + lane;
        const unsigned long long hit = __ballot(g < first.ngroups && n >= s_tpre[g] && n < s_tpre[g + 1]);
        if (hit) {   // wave-uniform
          t.group = c0 + __builtin_ctzll(hit);
          break;
        }
      }
      t.valid = 1;
      t.row_base = s_goff[t.group];
      t.rows = s_goff[t.group + 1] - t.row_base;
      const unsigned mt = (unsigned)(t.rows + BM - 1) / BM, within = n - s_tpre[t.group];
      t.m0 = within % mt * BM; t.n0 = within / mt * BN_OUT;
      t.widx = first.grp_widx ? first.grp_widx[t.group] : first.w_base + t.group;
    }
    t.half = ROUNDS && !FIRST ? __builtin_amdgcn_readfirstlane(t.half) : 0;
    t.group = __builtin_amdgcn_readfirstlane(t.group);
    t.m0 = __builtin_amdgcn_readfirstlane(t.m0);
    t.n0 = __builtin_amdgcn_readfirstlane(t.n0 + second_half * (BN_OUT / 2));
    t.rows = __builtin_amdgcn_readfirstlane(t.rows);
    t.row_base = __builtin_amdgcn_readfirstlane(t.row_base);
    t.widx = __builtin_amdgcn_readfirstlane(t.widx);
    return t;
  };
#define OCC_PICK(t, field) ((t).is_second ? second.field : first.field)

  int slot = blockIdx.x >> 3;
  int round = 0;
  Tile cur = tile_at(std::true_type{}, slot, 0);
  if (!cur.valid) return;   // uniform over the block, and so are its later tiles

  // loader role: a load covers 8 rows of 128 bytes, lane -> row lane/8, slot lane%8; four loads of token rows and eight
  // of weight rows per wave and K tile.  Token row i of this wave: tile row wave*32 + i*8 + lane/8.
  struct {
    const char *a, *w_even, *w_odd;   // scalar bases; w_odd: the up matrix
    unsigned a_off[4], b_off[8];      // per-lane byte offsets, constant over K
    long long kb;                     // byte offset of the K tile inside a token row (kt) and a weight row
    int kin, kseg;                    // K > kseg walks consecutive weight matrices
    long long ka, seg_step;
  } ld;
  // tile row of this lane for index slot `lane` (0..31) of s_idx, clamped to the group
  auto idx_row = [&](const Tile& t, int r) { return t.row_base + min(t.m0 + r, t.rows - 1); };
  auto request_rows = [&](const Tile& t) {   // source rows of tile t's token rows -> s_idx (nothing without a gather)
    const int32_t* a_rows = OCC_PICK(t, a_rows);
    if (a_rows)
      load_to_lds_4(reinterpret_cast<const char*>(a_rows + idx_row(t, wave * 32 + (lane & 31))),
                    __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) int*)&s_idx[wave][0]));
  };
  auto start_loading = [&](const Tile& t) {   // the rows requested for t have landed
    const bool gather = OCC_PICK(t, a_rows) != nullptr;
    const unsigned lda = OCC_PICK(t, lda), ldb = OCC_PICK(t, ldb);
    const int lrow = lane >> 3;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned chunk = (lane & 7) ^ ((i * 4 + (lane >> 4)) & 7);
      const unsigned src = gather ? s_idx[wave][i * 8 + lrow] : idx_row(t, wave * 32 + i * 8 + lrow);
      ld.a_off[i] = (src * lda + chunk * 8) * 2;   // host: A is below 4 GiB
    }
    // (a half tile's weight rows are loads 0..3 of the four waves, to where these go in any tile; what the tile before it
    // requests beyond them is not used)
    const int n_wave = t.n0 + (ROUNDS && t.half ? wave * (SWIGLU ? 16 : 32) : wave * (SWIGLU ? 32 : 64));
    // with SWIGLU a wave tile's 128 weight rows are [gate 16 | up 16] x 4, so MFMA row blocks 2j and 2j + 1 hold gate
    // and up of the same 16 output columns
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const unsigned chunk = (lane & 7) ^ ((i * 4 + (lane >> 4)) & 7);
      int ncol = n_wave + (SWIGLU ? (i >> 2) * 16 : (i >> 1) * 16) + (i & 1) * 8 + lrow;
      if (ncol >= first.N) ncol = first.N - 1;
      ld.b_off[i] = ((unsigned)ncol * ldb + chunk * 8) * 2;   // host: a weight matrix is below 4 GiB
    }
    const long long stride_b = OCC_PICK(t, b_group_stride);
    ld.a = static_cast<const char*>(OCC_PICK(t, A));
    ld.w_even = static_cast<const char*>(OCC_PICK(t, B)) + t.widx * stride_b * 2;
    ld.w_odd = SWIGLU ? static_cast<const char*>(OCC_PICK(t, B2)) + t.widx * stride_b * 2 : ld.w_even;
    ld.ka = ld.kb = 0;
    ld.kin = 0;
    ld.kseg = OCC_PICK(t, kseg);
    ld.seg_step = (stride_b - ld.kseg) * 2;
  };
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
  const unsigned lds_a = __builtin_amdgcn_readfirstlane(lds0 + wave * 4096);
  const unsigned lds_b = __builtin_amdgcn_readfirstlane(lds0 + A_BYTES + wave * 8192);
  constexpr int LOADS = 12;
  // load i (0..11) of the K tile being requested, into the stage at byte st; the last one moves on to the next K tile
  auto issue = [&](unsigned st, int i) {
    if (i < 8) {
      const char* w = (SWIGLU && (i & 2) ? ld.w_odd : ld.w_even) + ld.kb;
      if constexpr (ONCE) load_to_lds_16_streaming(w, ld.b_off[i], lds_b + st + i * 1024);
      else load_to_lds_16(w, ld.b_off[i], lds_b + st + i * 1024);
    } else load_to_lds_16(ld.a + ld.ka, ld.a_off[i - 8], lds_a + st + (i - 8) * 1024);
    if (i == LOADS - 1) {
      ld.ka += BK * 2;
      ld.kb += BK * 2;
      ld.kin += BK;
      if (ld.kin >= ld.kseg) {
        ld.kin = 0;
        ld.kb += ld.seg_step;
      }
    }
  };
  auto next = [](unsigned st) { return st == (NST - 1) * STAGE_BYTES ? 0u : st + STAGE_BYTES; };

  // fragments of the two K steps of 32: lane l holds row l%16, K group l/16 of a 16-row block
  int foff[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) foff[kk] = (lane & 15) * 128 + (((4 * kk + (lane >> 4)) ^ ((lane >> 1) & 7)) * 16);
  const char* frag_a = smem + wm * 8192;
  const char* frag_b = smem + A_BYTES + wn * 16384;
  bf16x8 fa[2][4], fb[8];
  auto read_a = [&](int kk, unsigned st, int i) {
    fa[kk][i] = *reinterpret_cast<const bf16x8*>(frag_a + st + foff[kk] + i * 2048);
  };
  auto read_b = [&](int kk, unsigned st, int i) {
    fb[i] = *reinterpret_cast<const bf16x8*>(frag_b + st + foff[kk] + i * 2048);
  };

  f32x4 acc[8][4];   // [weight-row block][token-row block]
  f32x4 tot[PARTS ? 8 : 1][4];   // PARTS: sums of the finished parts
  int nk = 0, parts = 1, edge = 0;   // of the current output tile: K tiles, parts, end of the part being summed
  auto part_after = [&](int done) {   // end of the part that K tile `done` is in: the smallest p * nk / parts above it
    const int p = ((done + 1) * parts + nk - 1) / nk;
    return __builtin_amdgcn_readfirstlane(p * nk / parts);
  };
  auto finish_part = [&](int done) {   // `done` < nk K tiles have been multiplied; the last part is added by sum()
    if constexpr (PARTS) {
      if (done != edge) return;   // wave-uniform
#pragma unroll
      for (int ni = 0; ni < 8; ++ni)
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
          tot[ni][mi] += acc[ni][mi];
          acc[ni][mi] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
      edge = part_after(done);
    }
  };
  auto sum = [&](int ni, int mi) { return PARTS ? tot[PARTS ? ni : 0][mi] + acc[ni][mi] : acc[ni][mi]; };
  // K step kk of the K tile in stage st: 8 groups of {4 products with, between them, one tile load into stage st_load
  // and up to two fragment reads of the next step (out of stage st_next)}, pinned in source order.  A fragment takes the registers of one
  // multiplied before; fb[7] follows in group 0 of its own step.  Step 1 has the block-wide wait between groups 1 and 2,
  // when the K tile's last fragments have been read: the next K tile has landed (for every wave) and stage st is free.
  // Its first six loads go out behind the wait, the other six in step 0 of the next K tile.
  auto step = [&](auto kk_, unsigned st, unsigned st_next, unsigned st_load) {
    constexpr int kk = decltype(kk_)::value;
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      if (kk == 1 && g == 2) wait_loads_and_barrier<LOADS>();
#pragma unroll
      for (int mi = 0; mi < 4; ++mi) {
        acc[g][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[g], fa[kk][mi], acc[g][mi], 0, 0, 0);
        // (fb[g] itself is free after the fourth product)
        if (mi == 0 && g >= 2) issue(st_load, kk == 1 ? g - 2 : g + 4);
        if (g == 2 || g == 3) {
          if (mi == 1) read_a(kk ^ 1, st_next, 2 * g - 4);
          if (mi == 2) read_a(kk ^ 1, st_next, 2 * g - 3);
        }
        if (g >= 4 && mi == 1) read_b(kk ^ 1, st_next, g - 4);
        if (g >= 5 && mi == 2) read_b(kk ^ 1, st_next, g - 1);
        if (g == 0 && mi == 3) read_b(kk, st, 7);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // The same of a half tile: 4 groups.  Fragments of the weight rows in two sets, fb[4 * kk ..], so that all of the next step's
  // can be read meanwhile.  Step 0 requests the token rows of the K tile two ahead, step 1, behind the wait, the weight rows of
  // the one three ahead.
  auto read_half_b = [&](int kk, unsigned st, int i) {   // (row blocks 2j and 2j + 1 of the wave tile came through one loading wave)
    fb[4 * kk + i] = *reinterpret_cast<const bf16x8*>(frag_b + st + foff[kk] + (i >> 1) * 8192 + (i & 1) * 2048);
  };
  auto half_step = [&](auto kk_, unsigned st_next, unsigned st_load) {
    constexpr int kk = decltype(kk_)::value, LEAD = kk == 1 ? 4 : 0;   // products before the wait
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (kk == 1 && g == 1) wait_loads_and_barrier<8>();
#pragma unroll
      for (int mi = 0; mi < 4; ++mi) {
        acc[g][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[4 * kk + g], fa[kk][mi], acc[g][mi], 0, 0, 0);
        const int at = 4 * g + mi - LEAD;
        if (at >= 0 && at < 12) {
          const int n = at - at / 3 - 1;   // two fragments behind every load
          if (at % 3 == 0) issue(st_load, (kk == 1 ? 0 : 8) + at / 3);
          else if (n < 4) read_a(kk ^ 1, st_next, n);
          else read_half_b(kk ^ 1, st_next, n - 4);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  const std::integral_constant<int, 0> k0{};
  const std::integral_constant<int, 1> k1{};

  // epilogue.  sum(ni, mi) element e of lane l: token row mi*16 + l%16, weight row ni*16 + (l/16)*4 + e of the wave
  // tile.  bf16 results pass through the wave's 2 KiB of LDS, 16 rows x 64 columns at a time (16-byte slots swizzled by
  // the row), and leave as row segments of 128 bytes; with ONCE marked as not to be kept: what lies dirty in the XCDs' L2s at the
  // end of a launch is written back before the next one may start (forward of 500 tokens of 64 + 2 experts 282 -> 271 us,
  // the products of a training step of 1000 tokens 712 -> 697; 2048 and 3500 tokens of 64 experts, whose next launch
  // finds some of it, 326.6 -> 329.4 and 467.6 -> 476.1: not there).
  auto store = [&](auto half_) {   // half_: cur.half, or the same known to the compiler
    const bool half = half_;
    char* stg = s_out[wave];
    constexpr int W_COLS = SWIGLU ? 64 : 128;      // output columns of a wave tile; of a half one the first half of them
    const int rows_left = cur.rows - cur.m0 - wm * 64;
    const int col_w = cur.n0 + (half ? wn * (W_COLS / 2) : wn * W_COLS);
    const int ccol = OCC_PICK(cur, c_col0) + cur.group * OCC_PICK(cur, c_group_cols);
    const int ldc = OCC_PICK(cur, ldc);
    const int scol = (lane & 7) * 8, srow = lane >> 3;
    const int col_end = min(first.N, SWIGLU && half ? col_w + W_COLS / 2 : first.N);
    constexpr int CHUNKS = SAVE ? 3 : W_COLS / 64;   // per 16-row block; SAVE: outputs, gate, up
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
      for (int ch = 0; ch < CHUNKS; ++ch) {
        if (!SWIGLU && ch == 1 && half) continue;   // wave-uniform
#pragma unroll
        for (int nn = 0; nn < 4; ++nn) {   // 16 output columns
          if (SWIGLU && nn > 1 && half) continue;
          float v[4];
          if (SWIGLU && ch == 0) {
            const f32x4 g = sum(2 * nn, mi), u = sum(2 * nn + 1, mi);
            if (OCC_PICK(cur, silu_rcp)) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = swiglu_rcp(g[e], u[e]);
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = swiglu_div(g[e], u[e]);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = SWIGLU ? sum(2 * nn + ch - 1, mi)[e] : sum(4 * ch + nn, mi)[e];
          }
          uint2 pk;
          pk.x = pack_bf16(v[0], v[1]);
          pk.y = pack_bf16(v[2], v[3]);
          const int row = lane & 15;
          *reinterpret_cast<uint2*>(stg + row * 128 + (((nn * 2 + (lane >> 5)) ^ ((row >> 1) & 7)) * 16) +
                                    ((lane >> 4) & 1) * 8) = pk;
        }
        const bool pre = SAVE && ch > 0;
        const int col = col_w + (SWIGLU ? 0 : ch * 64) + scol;
        __bf16* C = static_cast<__bf16*>(pre ? OCC_PICK(cur, C2) : OCC_PICK(cur, C));
        const long long pitch = pre ? 2ll * ldc : ldc;
        const int c0 = pre ? 2 * ccol + (ch - 1) * first.N : ccol;
        __bf16* dst = C + (cur.row_base + cur.m0 + wm * 64 + mi * 16) * pitch + c0 + col;
#pragma unroll
        for (int it = 0; it < 2; ++it) {
          const int row = it * 8 + srow;
          const u32x4 v = *reinterpret_cast<const u32x4*>(stg + row * 128 + (((lane & 7) ^ ((row >> 1) & 7)) * 16));
          if (mi * 16 + row < rows_left && col < col_end) {
            if constexpr (ONCE) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst + row * pitch));
            else *reinterpret_cast<u32x4*>(dst + row * pitch) = v;
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
  };

  // first tile: rows, K tiles 0 and 1, half of K tile 2
  request_rows(cur);
  wait_loads();   // a wave reads back only its own indices
  start_loading(cur);
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int i = 0; i < (k < 2 ? LOADS : LOADS / 2); ++i) issue(k * STAGE_BYTES, i);
  if constexpr (ROUNDS) {
    __builtin_amdgcn_sched_barrier(0);
    const int slots = cnt1 + cnt2 * span;
    whole = __builtin_amdgcn_readfirstlane((unsigned)slots / (unsigned)stride * stride);
    const int left = slots - whole;   // beyond the whole rounds
    halved = whole > 0 && whole >= span * stride && 2 * left <= stride;  // so a block takes at most one half, as its last tile and not its first
    __builtin_amdgcn_sched_barrier(0);
  }
  wait_loads_and_barrier<LOADS + LOADS / 2>();
  unsigned st = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) read_a(0, 0, i);
#pragma unroll
  for (int i = 0; i < 7; ++i) read_b(0, 0, i);
  __builtin_amdgcn_sched_barrier(0);

  auto begin_tile = [&]() {
    nk = (unsigned)OCC_PICK(cur, K) / BK;   // host: >= 3
    if (PARTS) {
      parts = OCC_PICK(cur, ksplit);   // host: >= 1
      edge = part_after(0);
    }
#pragma unroll
    for (int ni = 0; ni < 8; ++ni)
#pragma unroll
      for (int mi = 0; mi < 4; ++mi) acc[ni][mi] = tot[PARTS ? ni : 0][mi] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  // the block's last tile, a half one: its K tiles 0 and 1 and the weight rows of K tile 2 are on their way, K tile 0 has landed
  auto half_tile = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) read_half_b(0, st, i);
    half_step(k0, st, next(next(st)));
    for (int kt = 0; kt < nk - 1; ++kt) {
      const unsigned sn = next(st);
      if (kt == nk - 3) {   // what is requested past the end is its first K tiles again
        ld.ka = ld.kb = 0;
        ld.kin = 0;
      }
      half_step(k1, sn, st);
      finish_part(kt + 1);
      half_step(k0, sn, st);
      st = sn;
    }
    half_step(k1, next(st), st);
  };
  // Half and whole tiles share the epilogue's code, but for PARTS: the sums of both, in registers of their own, then meet in front of it and
  // are moved about in the whole tiles' K loop (down projection of 2314 tokens of 64 + 2 experts 159 us against 152).
  constexpr bool ONE_EPILOGUE = ROUNDS && !PARTS;
  bool more;
  do {
    const int ahead = ROUNDS && slot < cnt2 ? span : 1;
    slot += ahead * stride;
    round += ahead;
    Tile nxt = cur;   // keeps everything derived from it addressable where there is no next tile
    begin_tile();
    if (ONE_EPILOGUE && cur.half) {   // uniform over the block
      more = false;
      half_tile();
    } else {
      const Tile t = tile_at(std::false_type{}, slot, round);
      more = t.valid;
      if (more) nxt = t;
      request_rows(nxt);
      // step 0 of a K tile requests the second half of the K tile two ahead, step 1 the first half of the one three ahead
      step(k0, st, st, next(next(st)));
      for (int kt = 0; kt < nk - 3; ++kt) {
        const unsigned sn = next(st);
        step(k1, st, sn, st);
        finish_part(kt + 1);
        step(k0, sn, sn, st);
        st = sn;
      }
      if (nk < 5) wait_loads();   // the rows requested above have landed: two block-wide waits lie behind otherwise
      start_loading(nxt);
      const unsigned s1 = next(st), s2 = next(s1);
      step(k1, st, s1, st);
      finish_part(nk - 2);
      step(k0, s1, s1, st);
      step(k1, s1, s2, s1);
      finish_part(nk - 1);
      step(k0, s2, s2, s1);
      step(k1, s2, st, s2);
    }
    if constexpr (ONE_EPILOGUE) store(cur.half != 0);
    else store(std::false_type{});
    cur = nxt;
    if (ROUNDS && !ONE_EPILOGUE && cur.half) {
      more = false;
      begin_tile();
      half_tile();
      store(std::true_type{});
    }
  } while (more);   // uniform over the block
#undef OCC_PICK
  wait_loads();   // the loads issued for a tile that does not exist must land before the block's LDS is released
}
}  // namespace t128

// ONCE: the weights are read past the caches' keeping where almost every expert has one row tile, so that nobody reads them
// again, and where they are larger than the memory-side cache (256 MiB), which otherwise has some of them from the call before
// (us without / with: 64 experts, d = 2048, f = 1408, gate/up + down, 24 rows per expert 159 + 97 / 150 + 92, 47 rows
// 169 + 106 / 163 + 96; 38 rows of f = 1024, 537 MB of gate/up 100 / 92, 268 MB of down 47 / 52; d = 1152, f = 704, 207 MB of gate/up
// 44 / 55).  The line is put above the cache's size because it holds other tensors too; between 268 and 377 MB of weights
// nothing was measured that would move it.  By rows (GemmArgs::once_rows), forward passes of three layers in turn / of one again and again, without -> with: f = 1408,
// 64 + 2 experts, 75 rows 306 -> 303 / 303 -> 302, 94 rows 324 -> 320 / 312 -> 311, 112 rows 345 -> 366 / 334 -> 372; 60 + 4, 73 rows
// 369 -> 366 / 369 -> 349, 100 rows 406 -> 399 / 400 -> 392; f = 1024, 64 experts, 75 rows 259 -> 233 / 261 -> 214, 100 rows 232 -> 243 /
// 227 -> 250.  Below the line of bytes layers in turn gain by it what one layer loses (64 experts of 768 x 512, 47 rows, one layer
// 68.5 / 73.7, six in turn 463 / 441).  The shared experts' weights, which several row tiles read, go the same way: with 2 and
// 4 of them a forward takes 0.78 - 0.98 up to 47 rows and 0.87 - 1.04 at 60 and 70.  Where these have more rows than the routed experts,
// streaming loses beyond 72 (77 - 92 rows, streamed over kept, 2 - 4 shared experts, k = 1 and 2: 1.00 - 1.07); other
// forward passes from 88 on (20 sizes of 72 - 88 rows 0.94 - 1.00, 10 of 90 - 95 rows 0.97 - 1.04, three layers in turn).  One that keeps its
// pre-activations gains for the step behind it up to 95 rows (26 training steps 0.95 - 1.00).
// The backward's products keep their weights out of the memory-side cache in larger batches too, up to the line of the small weight-gradient
// tiles and while that cache holds the step's rows (ffn_backward.hip): these tiles read the rows of all products next, and wait for memory
// at every group if the weights have taken their place (1000 tokens of 64 + 2 experts, the three weight gradients 550 -> 400 us).  35 training steps of
// 80 - 230 rows per expert, streamed over kept, one layer again and again / three in turn: 0.955 / 0.950 on average, kept -> streamed
// 64 + 2 experts, d = 2048, f = 1408, 100 rows 1651 -> 1521 / 1665 -> 1509 us, 130 rows 1814 -> 1637 / 1838 -> 1646, 180 rows
// 2048 -> 1917 / 2070 -> 1900.  (With streamed weights and ordinary stores 0.962 / 0.967; with such stores alone 1.00.)
constexpr long long kOnceBytes = 320ll << 20;
int launch_tile128(const GemmArgs& a, const GemmArgs* b, bool swiglu, int total_rows, hipStream_t s) {
  const int bn_out = swiglu ? t128::BN / 2 : t128::BN;
  const long long n_tiles = (a.N + bn_out - 1) / bn_out;
  GemmArgs second{};
  if (b != nullptr) second = *b;
  OCC_REQUIRE(a.grp_offset != nullptr && a.K >= 3 * t128::BK && a.K % 64 == 0 && a.N % 64 == 0 &&
                  (b == nullptr || (b->grp_offset == nullptr && b->N == a.N && b->K >= 3 * t128::BK && b->K % 64 == 0)),
              OCCULT_EINVAL, "grouped GEMM shape outside the 128-row tiles' range");
  const long long t1 = (total_rows / t128::BM + a.ngroups) * n_tiles;   // at most one partial tile per group
  const long long t2 = (long long)second.ngroups * ((second.M + t128::BM - 1) / t128::BM) * n_tiles;
  OCC_REQUIRE(t1 + t2 < (1ll << 28), OCCULT_EINVAL, "grouped GEMM grid too large");
  int cus = 0;
  const int rc = device_cu_count(&cus);
  if (rc) return rc;
  long long blocks = ((t1 + 7) / 8 + (t2 + 7) / 8) * 8;   // one block per CU, a multiple of 8 so a block keeps its XCD
  const long long resident = cus >= 8 ? cus / 8 * 8 : 8;
  if (blocks > resident) blocks = resident;
  // Half tiles and `span` where a second round is likely: t1 counts a partly filled tile for every group, loads that differ leave half of
  // one on average, and one at least.  The kernel without takes any number of tiles.  (Forward passes of 45 batches whose t1 + t2 is 256 -
  // 1300, over those without half tiles anywhere: 0.968 on average, 0.88 - 1.02; by t1 + t2 alone 0.971, 0.88 - 1.025.)
  const long long likely1 = (total_rows / t128::BM + a.ngroups / 2) * n_tiles, least1 = (long long)min_i(total_rows, a.ngroups) * n_tiles;
  const bool rounds = t1 + t2 > blocks && 10 * ((likely1 > least1 ? likely1 : least1) + t2) > 9 * blocks;
  second.span = b != nullptr && b->K > a.K ? (b->K + a.K / 2) / a.K : 1;
  const bool save = swiglu && a.C2 != nullptr, parts = a.ksplit > 1 || second.ksplit > 1;
  OCC_REQUIRE(!(save && parts) && (!parts || (a.ksplit >= 1 && (b == nullptr || second.ksplit >= 1))), OCCULT_EINVAL,
              "grouped GEMM: parts of K outside the 128-row tiles' range");
  const dim3 grid((unsigned)blocks), block(256);
  const bool once = total_rows < (long long)a.once_rows * a.ngroups &&
                    (long long)a.ngroups * a.N * a.K * (swiglu ? 4 : 2) > kOnceBytes;
#define OCC_T128(SW, SAVE, PARTS)                                                                                        \
  do {                                                                                                                   \
    if (once && rounds) hipLaunchKernelGGL((t128::grouped_gemm_bf16<SW, SAVE, PARTS, true, true>), grid, block, 0, s, a, second); \
    else if (once) hipLaunchKernelGGL((t128::grouped_gemm_bf16<SW, SAVE, PARTS, true, false>), grid, block, 0, s, a, second);     \
    else if (rounds) hipLaunchKernelGGL((t128::grouped_gemm_bf16<SW, SAVE, PARTS, false, true>), grid, block, 0, s, a, second);   \
    else hipLaunchKernelGGL((t128::grouped_gemm_bf16<SW, SAVE, PARTS, false, false>), grid, block, 0, s, a, second);              \
  } while (0)
  if (save) OCC_T128(true, true, false);
  else if (swiglu && parts) OCC_T128(true, false, true);
  else if (swiglu) OCC_T128(true, false, false);
  else if (parts) OCC_T128(false, false, true);
  else OCC_T128(false, false, false);
#undef OCC_T128
  OCC_LAUNCH_CHECK("grouped_gemm");
  return OCCULT_OK;
}

}  // namespace occult
