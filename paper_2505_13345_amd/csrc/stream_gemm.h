// The weight-streaming kernel of the expert products: launched by ffn.hip, and by plan.hip with the routing and the plan of a few
// tokens in front of it (Front).  Not part of the public ABI.
#pragma once
#include "common.h"
#include "gemm.h"

namespace occult {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct TileInfo {
  int group, m0, rows, row_base;
};
// first output column of a group
__device__ __forceinline__ int group_col0(const GemmArgs& a, int group) { return a.c_col0 + group * a.c_group_cols; }

// Which group and row block does m-tile `mt` fall in?  Group g owns ceil(rows_g / BM) tiles.
// Executed by every thread of the first wave; result through LDS.  group = -1: past the end.
template <int BM>
__device__ __forceinline__ TileInfo find_tile(const GemmArgs& a, int mt, TileInfo* s_info) {
  const int lane = threadIdx.x & 63;
  if (threadIdx.x < 64) {
    TileInfo ti;
    ti.group = -1;
    ti.m0 = ti.rows = ti.row_base = 0;
    if (a.grp_offset == nullptr) {
      const int per_group = (a.M + BM - 1) / BM;
      if (mt < per_group * a.ngroups) {
        ti.group = mt / per_group;
        ti.m0 = (mt % per_group) * BM;
        ti.rows = a.M;
      }
      if (lane == 0) *s_info = ti;
    } else {
      if (lane == 0) *s_info = ti;
      int tiles_before = 0;
      for (int c0 = 0; c0 < a.ngroups; c0 += 64) {
        const int g = c0 + lane;
        const int lo = (g < a.ngroups) ? a.grp_offset[g] : 0;
        const int hi = (g < a.ngroups) ? a.grp_offset[g + 1] : 0;
        const int nt = (hi - lo + BM - 1) / BM;
        int incl = nt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int v = __shfl_up(incl, o, 64);
          if (lane >= o) incl += v;
        }
        const int excl = tiles_before + incl - nt;
        if (mt >= excl && mt < excl + nt) {   // at most one lane over all chunks
          ti.group = g;
          ti.m0 = (mt - excl) * BM;
          ti.rows = hi - lo;
          ti.row_base = lo;
          *s_info = ti;
        }
        tiles_before += __shfl(incl, 63, 64);
        if (tiles_before > mt) break;   // wave-uniform
      }
    }
  }
  __syncthreads();
  return *s_info;
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel for groups of a few rows (decode-shaped layers), where the work is streaming
// every active expert's weights from HBM once.  No LDS tiles, no barriers in the K loop: each wave
// owns 32 output columns x up to 16*MT tokens over the whole K (or a quarter of it: KSPLIT below)
// and loads both operands straight into MFMA fragment registers.  v_mfma_f32_16x16x32_bf16 takes 8 consecutive K elements per lane
// and 4 lanes per row, so one load instruction reads 16 rows x one whole 64-byte sector.  Weights
// are the row operand: a lane ends up with 4 consecutive output columns of one token (8-byte
// stores).  The operands of the next K step (4 or 8 KiB of weights per wave) are in flight while
// the current ones are multiplied; token blocks past the group's rows are skipped.
//
// One launch can carry two problems of the same shape class (N, SWIGLU, weight order): workgroups
// [0, a_blocks) work on `first`, the rest on `second`.  A small batch's shared experts ride with its
// routed experts this way: alone their few workgroups would stream weights at a fraction of the memory
// system's rate, and run after the routed experts they would add their whole duration to the call.
// The second problem has uniform groups and always splits K over the four waves of a workgroup (below);
// its K may walk several weight matrices (the shared experts' down projection: K = S * f), so that
// the sum over the shared experts happens in the accumulators and in the in-LDS addition, in K order.
namespace skinny {
constexpr int BN_OUT = 32;
typedef float f32x4v __attribute__((ext_vector_type(4)));

// KSPLIT (for the first problem; the second always does): the four waves of a workgroup take the four quarters of K
// of ONE column block and add their sums through LDS (quarters in ascending order, so the result is reproducible)
// instead of taking four column blocks over the whole K.  A wave's stream is then a quarter as long and there are four times as many workgroups, which the
// hardware hands to whichever CU has room: with whole-K waves a layer's 2000-4000 waves fill the chip's 1024 SIMDs
// two to four deep, all finish together, and a last partly filled layer of waves costs a whole stream's time.
// What a launch does before its products.  Nothing: the row tiles of the first problem are those of the plan's tables.
// (The kernel is a kernel and not a function that two call: inlined, its returns cost a branch in the loop, 128 tokens 225.7 -> 226.6 us.)
struct NoFront {
  static constexpr bool kOn = false;
};

template <bool SWIGLU, int MT, bool PACKED, bool KSPLIT, class Front = NoFront>   // MT token blocks of 16 per m-tile; PACKED: weights from a.Bp
__global__ __launch_bounds__(256) void grouped_gemm_bf16(const GemmArgs first, const GemmArgs second, const int a_blocks,
                                                         const Front front) {
  int bid = (int)blockIdx.x;
  if constexpr (Front::kOn) {
    if (front.begin(bid, a_blocks)) return;   // uniform: a workgroup of the plan
    bid -= front.plan_blocks;
  }
  constexpr int BM = 16 * MT;
  constexpr int KS = MT <= 2 ? 2 : 1;   // 32-wide K steps per pipeline stage
  constexpr int NW = SWIGLU ? 2 : 1;
  static_assert(!PACKED || KS == 2, "the packed order is written for two K steps per stage");
  __shared__ TileInfo s_info;
  const bool is_second = bid >= a_blocks;   // uniform over the workgroup
  const GemmArgs& a = is_second ? second : first;
  const bool ksplit = KSPLIT || is_second;   // uniform: the second problem's workgroups always split K
  const int cbw = ksplit ? 1 : 4;            // column blocks per workgroup
  const int n_cb = a.N / BN_OUT;   // column blocks (host: N % 32 == 0)
  const int wgs_per_mt = (n_cb + cbw - 1) / cbw;
  int mt, cbq;   // m-tile and group of cbw column blocks
  if (!is_second) {
    mt = bid / wgs_per_mt;
    cbq = bid % wgs_per_mt;
  } else {
    // Uniform groups of P m-tiles each: the P workgroups that stream the same weights (one per m-tile) get ids
    // 8 apart, so they run on the same XCD (workgroups go to the 8 XCDs round-robin) at about the same time and
    // all but the first of them find the weights in that XCD's L2.  unit = (group, column block).
    // (Measured against the four waves of one workgroup taking the m-tiles of one column block, which shares
    // the weights inside a CU: that was slower from 64 tokens on.)
    const int b = bid - a_blocks;
    const int P = (a.M + BM - 1) / BM;
    const int unit = b / (8 * P) * 8 + (b & 7), m = (b >> 3) % P;
    if (unit >= a.ngroups * wgs_per_mt) return;   // uniform: the grid is padded to whole sets of 8 units
    mt = unit / wgs_per_mt * P + m;
    cbq = unit % wgs_per_mt;
  }
  TileInfo ti;
  if constexpr (Front::kOn) ti = is_second ? find_tile<BM>(a, mt, &s_info) : front.tile(mt);
  else ti = find_tile<BM>(a, mt, &s_info);
  if (ti.group < 0) return;
  // what came through LDS is the same in every lane: kept in scalar registers, so that the addresses built from it
  // are a scalar base plus a per-lane 32-bit offset
  ti.group = __builtin_amdgcn_readfirstlane(ti.group);
  ti.m0 = __builtin_amdgcn_readfirstlane(ti.m0);
  ti.rows = __builtin_amdgcn_readfirstlane(ti.rows);
  ti.row_base = __builtin_amdgcn_readfirstlane(ti.row_base);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cb = ksplit ? cbq : cbq * 4 + wave;
  if (cb >= n_cb) return;   // whole-K workgroups meet no barrier after this; K-splitting ones never take it
  const int n0 = cb * BN_OUT;
  const int r = lane & 15, c = lane >> 4;
  int matrix;
  if constexpr (Front::kOn) matrix = is_second ? a.w_base + ti.group : front.matrix(ti.group);
  else matrix = a.grp_widx ? a.grp_widx[ti.group] : (a.w_base + ti.group);
  const long long widx = __builtin_amdgcn_readfirstlane(matrix);
  const int nblk = min(MT, (ti.rows - ti.m0 + 15) / 16);   // token blocks with any valid row
  const bool reread = is_second && a.M > BM;   // uniform

  // this lane's weight rows (column blocks 0 and 1 of the unit) and token rows, at its 16-byte K group
  const char* w[NW][2];
#pragma unroll
  for (int m = 0; m < NW; ++m)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
      w[m][nb] = static_cast<const char*>(m == 0 ? a.B : a.B2) +   // loaded like the token rows: lane l on row l / 4
                 ((widx * a.b_group_stride + (long long)(n0 + nb * 16 + (lane >> 2)) * a.ldb) * 2 + (lane & 3) * 16);
  // packed order: this wave's unit is one contiguous stream of stages, a load instruction reads 1 KiB of it
  const long long unit_bytes = (long long)(BN_OUT * NW * 2) * a.kseg;   // one unit's stream inside one weight matrix
  const char* wp = PACKED ? static_cast<const char*>(a.Bp) + widx * a.bp_group_stride + cb * unit_bytes
                          : nullptr;   // scalar; a lane reads at lane * 16 from it
  const unsigned lane16 = lane * 16;
  // token rows: a scalar base plus a 32-bit byte offset per lane (host: A < 4 GiB).  The MFMA wants lane l to hold row
  // l % 16, K group l / 16, which would make neighbouring lanes read rows that lie a whole row pitch apart (16 cache
  // lines looked up per 16 lanes).  The rows are loaded instead with lane l on row l / 4, K group l % 4 (four
  // neighbouring lanes = one 64-byte sector, 4 lines per 16 lanes) and put into the MFMA's order by a lane permutation
  // just before use (ds_bpermute: the LDS crossbar, no LDS memory).
  const char* xbase = static_cast<const char*>(a.A);
  unsigned xo[MT];
#pragma unroll
  for (int tb = 0; tb < MT; ++tb) {
    int lr = ti.m0 + tb * 16 + (lane >> 2);
    if (lr >= ti.rows) lr = ti.rows - 1;   // tokens past the group's end repeat its last row; dropped at the end
    const int logical = ti.row_base + lr;
    unsigned src;
    if constexpr (Front::kOn) src = is_second ? logical : front.row(ti.group, lr);
    else src = a.a_rows ? a.a_rows[logical] : logical;
    xo[tb] = (src * (unsigned)a.lda) * 2u + (lane & 3) * 16;
  }
  const int from_lane4 = (r * 4 + c) * 4;   // byte index of the lane that loaded what this lane multiplies
  auto to_mfma_order = [&](const bf16x8& v) {
    typedef int i32x4v __attribute__((ext_vector_type(4)));
    i32x4v t = __builtin_bit_cast(i32x4v, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = __builtin_amdgcn_ds_bpermute(from_lane4, t[e]);
    return __builtin_bit_cast(bf16x8, t);
  };

  f32x4v acc[NW][2][MT];
#pragma unroll
  for (int m = 0; m < NW; ++m)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int tb = 0; tb < MT; ++tb) acc[m][nb][tb] = f32x4v{0.0f, 0.0f, 0.0f, 0.0f};

  const int nst = a.K / (32 * KS);   // pipeline stages along K (host: K % 64 == 0)
  // byte offset of the current stage inside a weight row; K > kseg walks consecutive weight matrices
  long long w_off = 0, p_off = 0;   // caller's layout / packed order
  int w_kin = 0;
  auto w_advance = [&]() {
    w_off += 64 * KS;
    p_off += KS * NW * 2048;
    w_kin += 32 * KS;
    if (w_kin >= a.kseg) {   // host: kseg % 64 == 0, so a stage never straddles two matrices
      w_kin = 0;
      w_off += (a.b_group_stride - a.kseg) * 2;
      p_off += a.bp_group_stride - unit_bytes;
    }
  };
  struct Stage {
    bf16x8 wf[KS][NW][2], xf[KS][MT];
  };
  auto load_stage = [&](Stage& st, long long woff, long long poff, int i) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int m = 0; m < NW; ++m)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          {
            // measured: the streaming hint helps the single-matrix product and hurts the gate/up pair
            const bf16x8* src = PACKED ? reinterpret_cast<const bf16x8*>(wp + (poff + ((ks * NW + m) * 2 + nb) * 1024) +
                                                                           (size_t)lane16)
                                       : reinterpret_cast<const bf16x8*>(w[m][nb] + woff + ks * 64);
            // (a problem whose groups span several m-tiles reads its weights once per m-tile: those stay cacheable)
            st.wf[ks][m][nb] = (SWIGLU || reread) ? *src : __builtin_nontemporal_load(src);
          }
#pragma unroll
      for (int tb = 0; tb < MT; ++tb)
        if (tb < nblk) st.xf[ks][tb] = *reinterpret_cast<const bf16x8*>(xbase + ((long long)i * KS + ks) * 64 + (size_t)xo[tb]);
    }
  };
  auto multiply = [&](const Stage& st) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8 wfo[NW][2];   // the packed order is the MFMA's already
#pragma unroll
      for (int m = 0; m < NW; ++m)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) wfo[m][nb] = PACKED ? st.wf[ks][m][nb] : to_mfma_order(st.wf[ks][m][nb]);
#pragma unroll
      for (int tb = 0; tb < MT; ++tb)
        if (tb < nblk) {
          const bf16x8 xf = to_mfma_order(st.xf[ks][tb]);
#pragma unroll
          for (int m = 0; m < NW; ++m)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
              acc[m][nb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wfo[m][nb], xf, acc[m][nb][tb], 0, 0, 0);
        }
    }
  };

  // this wave's stages of K
  const int i_begin = ksplit ? wave * nst / 4 : 0, i_end = ksplit ? (wave + 1) * nst / 4 : nst;
  if (i_begin > 0) {
    const int kin = i_begin * 32 * KS, mat = kin / a.kseg;
    w_kin = kin - mat * a.kseg;
    w_off = ((long long)mat * a.b_group_stride + w_kin) * 2;
    p_off = mat * a.bp_group_stride + (long long)(w_kin / 32) * (NW * 2048);
  }
  if (i_begin < i_end) {   // wave-uniform
    Stage s0, s1;
    load_stage(s0, w_off, p_off, i_begin);
    for (int i = i_begin; i < i_end; i += 2) {
      // past the end the last stage is fetched again and not used
      const bool more1 = i + 1 < i_end;
      if (more1) w_advance();
      load_stage(s1, w_off, p_off, more1 ? i + 1 : i);
      multiply(s0);
      const bool more2 = i + 2 < i_end;
      if (more2) w_advance();
      load_stage(s0, w_off, p_off, more2 ? i + 2 : (more1 ? i + 1 : i));
      if (more1) multiply(s1);
    }
  }
  if (ksplit) {   // uniform over the workgroup
    // waves 1..3 hand their sums to wave 0, which adds them in that order and writes the tile
    __shared__ float s_red[3][NW * 2 * MT * 4][64];
    if (wave > 0) {
#pragma unroll
      for (int m = 0; m < NW; ++m)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int tb = 0; tb < MT; ++tb)
#pragma unroll
            for (int e = 0; e < 4; ++e) s_red[wave - 1][((m * 2 + nb) * MT + tb) * 4 + e][lane] = acc[m][nb][tb][e];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int wv = 0; wv < 3; ++wv)
#pragma unroll
      for (int m = 0; m < NW; ++m)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int tb = 0; tb < MT; ++tb)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[m][nb][tb][e] += s_red[wv][((m * 2 + nb) * MT + tb) * 4 + e][lane];
  }

  // acc element e of lane l: token l%16 of its block, output column nb*16 + (l/16)*4 + e of the unit
#pragma unroll
  for (int tb = 0; tb < MT; ++tb) {
    const int token = ti.m0 + tb * 16 + r;
    if (token < ti.rows) {
      __bf16* crow = static_cast<__bf16*>(a.C) + (long long)(ti.row_base + token) * a.ldc + group_col0(a, ti.group) + n0 + c * 4;
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g = acc[0][nb][tb][e];
          v[e] = SWIGLU ? g / (1.0f + __expf(-g)) * acc[NW - 1][nb][tb][e] : g;
        }
        uint2 pk;
        pk.x = pack_bf16(v[0], v[1]);
        pk.y = pack_bf16(v[2], v[3]);
        *reinterpret_cast<uint2*>(crow + nb * 16) = pk;
      }
    }
  }
}

// workgroups of the second problem
inline long long second_blocks(const GemmArgs& b) {
  return (b.ngroups * (b.N / BN_OUT) + 7) / 8 * 8 * (long long)((b.M + 31) / 32);   // whole sets of 8 units
}
}  // namespace skinny

}  // namespace occult
