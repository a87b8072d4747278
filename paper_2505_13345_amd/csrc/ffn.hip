// occult_expert_ffn: grouped SwiGLU expert computation (paper App. A.2 "SMM with Scattering" and
// the matrix product of "SMM with Merging"; Sec. 3.1: each operator bridges two tensor states).
//
//   GEMM-1 (SFD -> EPD): for the expert at placement position P, its EPD rows
//     [exp_offset[P], exp_offset[P+1]) gather their A rows from sfd_x through epd_sfd_row (the
//     replication happens in the load, no expanded copy of the input exists); B = [W_gate; W_up];
//     the epilogue applies silu(gate) * up and stores bf16 epd_h.
//   GEMM-2 (EPD -> EPD): epd_y rows = epd_h rows x W_down^T.  The reduction over a device's
//     experts is left to combine's first stage (order-fixed, no float atomics).
//   Shared experts: the same two kernels over all T rows of x with the shared weights.
//
// bf16 path: LDS-tiled MFMA, f32 accumulation.  Weights are
// K-contiguous ([out][in]), activations are K-contiguous rows, so both MFMA operands are read
// from LDS as 16-byte K-runs and no transpose is needed.
// f32 path: f32 matrix instructions, for small parity-sized layers.
#include "common.h"
#include "gemm.h"
#include "stream_gemm.h"

#include <type_traits>

namespace occult {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Workgroup id -> (m-tile, n-tile).  Workgroups are handed to the 8 XCDs round-robin and each XCD
// has its own L2, so the tiles an XCD runs at the same time should share operands: XCD x gets
// "chunks" x, x+8, ... of MC consecutive m-tiles times all n-tiles (about one tile per CU of the
// XCD), so that an A tile is fetched into one L2 only and a B tile is reused MC times there.
struct TileMap {
  int mt, nt;
};
__device__ __forceinline__ TileMap map_tile_id(unsigned b, int n_tiles) {
  const int mc = max(1, (32 + n_tiles / 2) / n_tiles);
  const unsigned per_chunk = mc * n_tiles;
  const int xcd = (int)(b & 7);
  const unsigned slot = b >> 3;
  const int chunk = (int)(slot / per_chunk) * 8 + xcd;
  const int within = (int)(slot % per_chunk);
  TileMap tm;
  tm.mt = chunk * mc + within / n_tiles;
  tm.nt = within % n_tiles;
  return tm;
}
__device__ __forceinline__ TileMap map_tile(int n_tiles) { return map_tile_id(blockIdx.x, n_tiles); }
// grid size covering m_tiles x n_tiles under map_tile (host)
static long long mapped_grid(long long m_tiles, int n_tiles) {
  const int mc = (32 + n_tiles / 2) / n_tiles > 1 ? (32 + n_tiles / 2) / n_tiles : 1;
  long long chunks = (m_tiles + mc - 1) / mc;
  chunks = (chunks + 7) / 8 * 8;
  return chunks * mc * n_tiles;
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel, small tile (few rows per expert: decode-shaped layers).  Block = 256 threads = 4 waves (2 x 2), block tile 128 x 128 x 64,
// wave tile 64 x 64 = 2 x 2 MFMA tiles of 32 x 32.  With SWIGLU the 128 B-rows of a tile are
// [gate n0..n0+31 | up n0..n0+31 | gate n0+32..n0+63 | up n0+32..n0+63], so the two MFMA
// columns of a wave hold gate and up of the same 32 output columns.
namespace small {
constexpr int BM = 128, BN = 128, BK = 64;
constexpr int LDS_STRIDE = BK + 8;   // 144-byte rows: 16-byte reads of 8 consecutive rows hit 8 distinct bank groups

template <bool SWIGLU>
__global__ __launch_bounds__(256) void grouped_gemm_bf16(const GemmArgs a) {
  __shared__ __attribute__((aligned(16))) __bf16 As[2][BM * LDS_STRIDE];   // two K tiles: one multiplied, one being written
  __shared__ __attribute__((aligned(16))) __bf16 Bs[2][BN * LDS_STRIDE];
  __shared__ TileInfo s_info;

  constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
  const int n_tiles = (a.N + BN_OUT - 1) / BN_OUT;
  TileMap tm = map_tile(n_tiles);
  if (a.plain_map) {
    tm.mt = blockIdx.x / n_tiles;
    tm.nt = blockIdx.x % n_tiles;
  }
  const int mt = tm.mt;
  const int n0 = tm.nt * BN_OUT;
  const TileInfo ti = find_tile<BM>(a, mt, &s_info);
  if (ti.group < 0) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const __bf16* A = static_cast<const __bf16*>(a.A);
  const long long widx = a.grp_widx ? a.grp_widx[ti.group] : (a.w_base + ti.group);

  // global -> LDS staging: thread owns 16-byte vector kv of rows (tid/8) + 32*i, i = 0..3
  const int kv = tid & 7, r_in = tid >> 3;
  const __bf16* a_src[4];
  const __bf16* b_src[4];   // row start inside the first weight matrix
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r_in + 32 * i;
    int lr = ti.m0 + r;
    if (lr >= ti.rows) lr = ti.rows - 1;   // clamp: rows past the group are computed and dropped
    const int logical = ti.row_base + lr;
    const long long src = a.a_rows ? a.a_rows[logical] : logical;
    a_src[i] = A + src * a.lda + kv * 8;
    int ncol;
    const __bf16* wbase;
    if (SWIGLU) {
      const int blk = r >> 5, within = r & 31;
      ncol = n0 + (blk >> 1) * 32 + within;
      wbase = static_cast<const __bf16*>((blk & 1) ? a.B2 : a.B);
    } else {
      ncol = n0 + r;
      wbase = static_cast<const __bf16*>(a.B);
    }
    if (ncol >= a.N) ncol = a.N - 1;
    b_src[i] = wbase + widx * a.b_group_stride + (long long)ncol * a.ldb + kv * 8;
  }

  f32x16 acc[2][2];
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.0f;

  const int nk_all = a.K / BK;
  const int split = a.ksplit > 1 ? a.ksplit : 1;
  const int kt_begin = (int)((long long)blockIdx.y * nk_all / split);   // this block's K tiles
  const int nk = (int)((long long)(blockIdx.y + 1) * nk_all / split);   // (end, exclusive)
  // A block is alone on its CU more often than not (few tiles), so nothing else hides its own latencies: the
  // K loop is software-pipelined.  While K tile kt is multiplied out of one LDS buffer, tile kt+1 (already in
  // registers) is written to the other, tile kt+2 is in flight into the second register set and tile kt+3 is
  // requested as soon as a set is free; inside a tile the fragments of K step kk+1 are read while step kk is
  // multiplied; one barrier per tile.
  u32x4 ga0[4], gb0[4], ga1[4], gb1[4];
  auto load_global = [&](int kt, u32x4 (&ga)[4], u32x4 (&gb)[4]) {
    const int k0 = kt * BK;
    const int seg = k0 / a.kseg;                 // which weight matrix along K (shared down-proj)
    const long long boff = (long long)seg * a.b_group_stride + (k0 - seg * a.kseg);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ga[i] = *reinterpret_cast<const u32x4*>(a_src[i] + k0);
      gb[i] = *reinterpret_cast<const u32x4*>(b_src[i] + boff);
    }
  };
  auto write_lds = [&](int buf, const u32x4 (&ga)[4], const u32x4 (&gb)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r_in + 32 * i;
      *reinterpret_cast<u32x4*>(&As[buf][r * LDS_STRIDE + kv * 8]) = ga[i];
      *reinterpret_cast<u32x4*>(&Bs[buf][r * LDS_STRIDE + kv * 8]) = gb[i];
    }
  };
  bf16x8 fa[2][2], fb[2][2];
  auto read_frags = [&](int buf, int kk, bf16x8 (&xa)[2], bf16x8 (&xb)[2]) {
    const int kof = kk * 16 + (lane >> 5) * 8;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
      xa[mi] = *reinterpret_cast<const bf16x8*>(&As[buf][(wm * 64 + mi * 32 + (lane & 31)) * LDS_STRIDE + kof]);
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
      xb[ni] = *reinterpret_cast<const bf16x8*>(&Bs[buf][(wn * 64 + ni * 32 + (lane & 31)) * LDS_STRIDE + kof]);
  };
  // K tile kt out of LDS buffer `buf`; (ga, gb) holds tile kt+1 on entry and is refilled with tile kt+3
  auto k_tile = [&](int kt, int buf, u32x4 (&ga)[4], u32x4 (&gb)[4]) {
    read_frags(buf, 0, fa[0], fb[0]);
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      if (kk + 1 < BK / 16) read_frags(buf, kk + 1, fa[(kk + 1) & 1], fb[(kk + 1) & 1]);
      if (kk == 1 && kt + 1 < nk) write_lds(buf ^ 1, ga, gb);
      if (kk == 2 && kt + 3 < nk) load_global(kt + 3, ga, gb);
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk & 1][mi], fb[kk & 1][ni], acc[mi][ni], 0, 0, 0);
    }
    __syncthreads();   // tile kt+1 is in the other buffer for everyone, and nobody reads this one any more
  };
  if (kt_begin < nk) {
    load_global(kt_begin, ga0, gb0);
    if (kt_begin + 1 < nk) load_global(kt_begin + 1, ga1, gb1);
    write_lds(0, ga0, gb0);
    if (kt_begin + 2 < nk) load_global(kt_begin + 2, ga0, gb0);
    __syncthreads();
    for (int kt = kt_begin; kt < nk; kt += 2) {
      k_tile(kt, 0, ga1, gb1);
      if (kt + 1 < nk) k_tile(kt + 1, 1, ga0, gb0);
    }
  }

  // epilogue.  Accumulator element r of lane l sits at row (r/4)*8 + (l/32)*4 + r%4, column l%32.
  __bf16* C = static_cast<__bf16*>(a.C);
  const int col_in = lane & 31;
#pragma unroll
  for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = ti.m0 + wm * 64 + mi * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
      if (row >= ti.rows) continue;
      __bf16* crow = C + (long long)(ti.row_base + row) * a.ldc + group_col0(a, ti.group);
      if (!SWIGLU && a.ksplit > 1) {   // partial sums of this K slice, f32
        float* prow = a.ws + ((long long)blockIdx.y * a.M + row) * a.N;
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
          const int col = n0 + wn * 64 + ni * 32 + col_in;
          if (col < a.N) prow[col] = acc[mi][ni][r];
        }
        continue;
      }
      if (SWIGLU) {
        const int col = n0 + wn * 32 + col_in;
        if (col < a.N) {
          const float g = acc[mi][0][r], u = acc[mi][1][r];
          crow[col] = static_cast<__bf16>(g / (1.0f + __expf(-g)) * u);
        }
      } else {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
          const int col = n0 + wn * 64 + ni * 32 + col_in;
          if (col < a.N) crow[col] = static_cast<__bf16>(acc[mi][ni][r]);
        }
      }
    }
  }
}
}  // namespace small


// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel, main variant (prefill-shaped layers).  Block = 256 threads = 4 waves (2 x 2),
// block tile 256 x 256 x 64, wave tile 128 x 128 = 8 x 8 MFMA tiles of 16 x 16 (256 accumulator
// registers per lane, one wave per SIMD, one block per CU).
//
// Persistent blocks.  With one block per CU nothing overlaps a tile's fixed costs (finding its
// group, gathering its row indices, the first operand loads, the store tail), so a block walks
// output tiles blockIdx.x, + gridDim.x, ... of the XCD-aware order and treats them as one stream
// of K tiles: the next output tile's group and row gather are fetched during the current K loop,
// its first K tile is loaded during the current tile's last two K tiles, and its second one
// during the epilogue.
//
// Global -> LDS.  Operand tiles go from global memory straight into LDS
// (global_load_lds_dwordx4: no VGPR staging, no ds_write), double buffered: while K tile j is
// multiplied, K tile j+1 lands in the other stage.  The loads are issued from inline assembly
// (wave-uniform base in SGPRs + a 32-bit per-lane offset that is constant over K, so advancing K
// costs two scalar adds) and waited for with an explicit vmcnt: the compiler's own wait insertion
// treats an LDS-directed load as a FLAT access and could only wait for all outstanding loads at
// every LDS read.  One such load writes 64 lanes x 16 bytes contiguously = 8 rows of 128 bytes,
// so rows cannot be padded; bank conflicts of the 16-byte fragment reads are avoided by an XOR
// swizzle instead: chunk c of row r lives at slot c ^ ((r >> 1) & 7), realised by the loading
// lane's choice of global chunk.  (LDS has 64 banks = 256 bytes per clock: two 128-byte rows share
// a bank line, so 16 consecutive rows x one chunk must cover the 16 slots of a line.)
//
// Matrix instruction.  v_mfma_f32_16x16x32_bf16 rather than 32x32x16: the clock under matrix load is power-limited, and
// the 16 x 16 form reads and writes half as many accumulator bytes per product.  Under the counters (GEMM-1 of the prefill
// batch) 941 us at 1697 MHz with the matrix pipe 70 % busy went to 905 us at 1888 MHz and 65 %: bound by the operand
// stream into LDS instead.
//
// Schedule.  With one wave per SIMD nothing hides an instruction clump, so a K step of 32 (64 MFMAs) is written as 16
// groups of {4 MFMAs, up to 2 LDS fragment reads for the next K step, up to 2 tile loads} pinned in source order: the
// matrix pipe keeps running while the other pipes are fed.  The block-wide wait for the next K tile sits between the two
// steps of a K tile, whose last fragments have been read by then; the next tile's step-0 fragments are read under
// step 1.  Step 0 of an output tile multiplies into a zero constant, so accumulators are never cleared.  No branch sits
// inside a K tile (each would make the register allocator shuffle the 256 accumulators).
//
// Epilogue.  The MFMA operands are swapped (weights as the row operand), so a lane holds 4
// consecutive output columns of one row; results go as bf16 through the wave's own 8 KiB of the
// idle stage (the region its own next loads will fill, so no block barrier is needed), 32 rows x
// 64 columns at a time, and leave as 16-byte stores of whole 128-byte row segments.  With SWIGLU
// the 128 B-rows of a wave's half tile are [gate c..c+31 | up c..c+31 | gate c+32..c+63 |
// up c+32..c+63], so the MFMA row blocks 0, 1 (4, 5) hold the gates to the up values in 2, 3 (6, 7)
// and the activation is applied in registers.
namespace t256 {
constexpr int BM = 256, BN = 256, BK = 64;
constexpr int A_BYTES = BM * BK * 2;             // 32 KiB
constexpr int STAGE_BYTES = 2 * A_BYTES;         // 64 KiB: A tile then B tile
constexpr int SMEM_BYTES = 2 * STAGE_BYTES;

// acc (16 x 16) += b (16 weight rows x 32 K) * a (16 token rows x 32 K)^T, accumulators in the accumulation registers.
// Written as assembly because the compiler, given the builtin, moves the 64 accumulator quads between the two register
// files; it cannot see that these are matrix instructions, so whoever reads acc has to leave the wait states itself
// (mfma_results_ready) and keep the reads behind them (behind).
__device__ __forceinline__ void mfma16(f32x4& acc, const bf16x8& b, const bf16x8& a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}
__device__ __forceinline__ void mfma16_first(f32x4& acc, const bf16x8& b, const bf16x8& a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(b), "v"(a));
}
// The wait states, and what ties acc to them: a value that the one leaves and the other takes.  (A volatile statement per
// accumulator would tie it as well, and hold the epilogue's LDS accesses in source order: prefill step 1673 -> 1688 us.)
__device__ __forceinline__ int mfma_results_ready() {
  int ready;
  asm volatile("s_nop 15\n\ts_nop 15" : "=s"(ready)::"memory");
  return ready;
}
__device__ __forceinline__ void behind(int ready, f32x4& acc) { asm("" : "+a"(acc) : "s"(ready)); }

// One output tile before its row gather has come back.  All fields but raw are wave-uniform.
struct Head {
  int valid, m0, rows, row_base, n0, widx, ccol;   // ccol: first output column of the tile's group
  int raw[8];   // source rows of this lane's 8 A-tile rows
};

// which group and row block is m-tile mt?  s_tpre[g] = m-tiles of the groups before g (s_tpre[ngroups]
// = all of them).  Every wave works this out for itself; the result is wave-uniform.
// group = -1: past the last tile.
__device__ __forceinline__ void locate(const GemmArgs& a, const int* s_goff, const int* s_tpre, int mt, int lane,
                                       int& group, int& m0, int& rows, int& row_base) {
  group = -1;
  m0 = rows = row_base = 0;
  if (a.grp_offset == nullptr) {
    const int per_group = (a.M + BM - 1) / BM;
    if (mt < per_group * a.ngroups) {
      group = mt / per_group;
      m0 = (mt % per_group) * BM;
      rows = a.M;
    }
    return;
  }
  for (int c0 = 0; c0 < a.ngroups; c0 += 64) {
    const int g = c0 + lane;
    const bool mine = g < a.ngroups && mt >= s_tpre[g] && mt < s_tpre[g + 1];
    const unsigned long long hit = __ballot(mine);
    if (hit) {   // wave-uniform
      group = c0 + __ffsll((long long)hit) - 1;
      m0 = (mt - s_tpre[group]) * BM;
      row_base = s_goff[group];
      rows = s_goff[group + 1] - row_base;
      return;
    }
  }
}


// SAVE (with SWIGLU): the gate and up pre-activations are stored too (a.C2).
// WIDE: the A operand is 4 GiB or larger, so its per-lane byte offsets take 64 bits (two registers per load
// and a 64-bit add before each) instead of one 32-bit offset beside a scalar base.
template <bool SWIGLU, bool SAVE, bool WIDE = false>
__global__ __launch_bounds__(256) void grouped_gemm_bf16(const GemmArgs a) {
  static_assert(SWIGLU || !SAVE, "pre-activations exist only with the fused activation");
  using aoff_t = typename std::conditional<WIDE, unsigned long long, unsigned>::type;
  __shared__ __attribute__((aligned(1024))) char smem[SMEM_BYTES];
  __shared__ int s_goff[OCCULT_MAX_E + 1];   // group row offsets
  __shared__ int s_widx[OCCULT_MAX_E];       // weight matrix of each group
  __shared__ int s_tpre[OCCULT_MAX_E + 1];   // m-tiles before each group

  constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
  const int n_tiles = (a.N + BN_OUT - 1) / BN_OUT;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  if (a.grp_offset) {
    for (int i = tid; i <= a.ngroups; i += 256) s_goff[i] = a.grp_offset[i];
    for (int i = tid; i < a.ngroups; i += 256) s_widx[i] = a.grp_widx ? a.grp_widx[i] : a.w_base + i;
    if (wave == 0) {   // exclusive scan of the groups' tile counts
      int before = 0;
      for (int c0 = 0; c0 < a.ngroups; c0 += 64) {
        const int g = c0 + lane;
        const int nt = g < a.ngroups ? (a.grp_offset[g + 1] - a.grp_offset[g] + BM - 1) / BM : 0;
        int incl = nt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int v = __shfl_up(incl, o, 64);
          if (lane >= o) incl += v;
        }
        if (g < a.ngroups) s_tpre[g] = before + incl - nt;
        before += __shfl(incl, 63, 64);
      }
      if (lane == 0) s_tpre[a.ngroups] = before;
    }
  }
  __syncthreads();

  // tile L of the XCD-aware order; past the end (or with nothing left) the fields of `fallback`
  // are kept, so that everything derived from a head stays addressable
  auto head_of = [&](unsigned L, const Head* fallback) {
    Head h;
    const TileMap tm = map_tile_id(L, n_tiles);
    int group;
    locate(a, s_goff, s_tpre, tm.mt, lane, group, h.m0, h.rows, h.row_base);
    h.valid = group >= 0;
    h.n0 = tm.nt * BN_OUT;
    h.widx = a.w_base;
    h.ccol = a.c_col0;
    if (h.valid) {
      h.widx = a.grp_offset ? s_widx[group] : a.w_base + group;
      h.ccol = group_col0(a, group);
    } else if (fallback) {
      h.m0 = fallback->m0; h.rows = fallback->rows; h.row_base = fallback->row_base;
      h.n0 = fallback->n0; h.widx = fallback->widx; h.ccol = fallback->ccol;
    }
    h.ccol = __builtin_amdgcn_readfirstlane(h.ccol);
    h.widx = __builtin_amdgcn_readfirstlane(h.widx);
    h.m0 = __builtin_amdgcn_readfirstlane(h.m0);
    h.rows = __builtin_amdgcn_readfirstlane(h.rows);
    h.row_base = __builtin_amdgcn_readfirstlane(h.row_base);
    h.n0 = __builtin_amdgcn_readfirstlane(h.n0);
    h.valid = __builtin_amdgcn_readfirstlane(h.valid);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = (wave * 8 + i) * 8 + (lane >> 3);
      int lr = h.m0 + r;
      if (lr >= h.rows) lr = h.rows - 1;   // rows past the group are computed and dropped
      if (lr < 0) lr = 0;
      const int logical = h.row_base + lr;
      h.raw[i] = a.a_rows ? a.a_rows[logical] : logical;
    }
    return h;
  };
  // loader role: load i (0..7) of this wave fills tile rows (wave*8 + i)*8 .. +7 of A and of B;
  // lane -> row lane/8, slot lane%8
  auto offsets_of = [&](const Head& h, aoff_t (&ao)[8], unsigned (&bo)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = (wave * 8 + i) * 8 + (lane >> 3);
      const int chunk = (lane & 7) ^ ((r >> 1) & 7);
      ao[i] = ((aoff_t)(unsigned)h.raw[i] * (aoff_t)(unsigned)a.lda + chunk * 8) * 2;   // host: A bytes < 2^32 unless WIDE
      int ncol;
      if (SWIGLU) {
        const int half = r >> 7, q = (r & 127) >> 5, within = r & 31;
        ncol = h.n0 + half * 64 + (q >> 1) * 32 + within;   // q odd -> up matrix: loads 4..7 of every wave
      } else {
        ncol = h.n0 + r;
      }
      if (ncol >= a.N) ncol = a.N - 1;
      bo[i] = (unsigned)(((long long)ncol * a.ldb + chunk * 8) * 2);
    }
  };

  const unsigned stride = gridDim.x;   // host: tile ids + stride stay below 2^31
  unsigned L = blockIdx.x;
  Head hd = head_of(L, nullptr);
  if (!hd.valid) return;   // uniform over the block; later tiles of this block are past the end too

  const char* a_base = static_cast<const char*>(a.A);
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
  const unsigned lds_w = __builtin_amdgcn_readfirstlane(lds0 + wave * 8192);
  // fragment read offsets inside a 16-row block for the two 32-wide K steps of a tile
  int foff[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
    foff[kk] = (lane & 15) * 128 + (((4 * kk + (lane >> 4)) ^ ((lane >> 1) & 7)) * 16);
  const int nk = a.K / BK;   // host: >= 2

  aoff_t a_off[8];
  unsigned b_off[8];
  offsets_of(hd, a_off, b_off);
  const char* w_lo = static_cast<const char*>(a.B) + (long long)hd.widx * a.b_group_stride * 2;   // loads 0..3
  const char* w_hi = SWIGLU ? static_cast<const char*>(a.B2) + (long long)hd.widx * a.b_group_stride * 2 : w_lo;

  bf16x8 fa[2][8], fb[2][8];
  // read r (0..15) of the fragments of K step kk of the tile in `stage`, in the order in which the products want them:
  // the first weight-row block, the token-row blocks, the other weight-row blocks
  auto read_frag = [&](int set, int stage, int kk, int r) {
    const char* As = smem + stage * STAGE_BYTES + wm * 128 * 128;
    const char* Bs = smem + stage * STAGE_BYTES + A_BYTES + wn * 128 * 128;
    if (r >= 1 && r <= 8)
      fa[set][r - 1] = *reinterpret_cast<const bf16x8*>(As + (r - 1) * 16 * 128 + foff[kk]);
    else {
      const int ni = r == 0 ? 0 : r - 8;
      fb[set][ni] = *reinterpret_cast<const bf16x8*>(Bs + ni * 16 * 128 + foff[kk]);
    }
  };
  // A rows / B rows of a K tile: load g (0..7) of this wave into `stage`
  auto load_a = [&](const aoff_t (&ao)[8], int ktile, int stage, int g) {
    if constexpr (WIDE)
      load_to_lds_16(a_base + (long long)ktile * (BK * 2) + ao[g], lds_w + stage * STAGE_BYTES + g * 1024);
    else
      load_to_lds_16(a_base + (long long)ktile * (BK * 2), ao[g], lds_w + stage * STAGE_BYTES + g * 1024);
  };
  auto load_b = [&](const unsigned (&bo)[8], const char* lo, const char* hi, long long kb, int stage, int g) {
    load_to_lds_16((g < 4 ? lo : hi) + kb, bo[g], lds_w + stage * STAGE_BYTES + A_BYTES + g * 1024);
  };
  // byte offset of K tile j inside a weight row; K > kseg walks consecutive weight matrices
  // (down projection of the shared experts)
  long long kb_next = 0;
  int kin_next = 0;
  auto kb_reset = [&]() { kb_next = 0; kin_next = 0; };
  auto kb_advance = [&]() {
    kb_next += BK * 2;
    kin_next += BK;
    if (kin_next >= a.kseg) {
      kin_next = 0;
      kb_next += (a.b_group_stride - a.kseg) * 2;
    }
  };

  // prologue of the block: K tile 0 -> stage 0, its first fragments, A half of K tile 1 -> stage 1
  int par = 0;   // stage holding K tile 0 of the current output tile
#pragma unroll
  for (int g = 0; g < 8; ++g) load_a(a_off, 0, 0, g);
#pragma unroll
  for (int g = 0; g < 8; ++g) load_b(b_off, w_lo, w_hi, 0, 0, g);
  wait_loads_and_barrier<0>();
#pragma unroll
  for (int r = 0; r < 16; ++r) read_frag(0, 0, 0, r);
#pragma unroll
  for (int g = 0; g < 8; ++g) load_a(a_off, 1, 1, g);
  __builtin_amdgcn_sched_barrier(0);

  __bf16* C = static_cast<__bf16*>(a.C);

  while (true) {
    // State here: K tile 0 of this output tile in stage par with its step-0 fragments in set 0;
    // the A half of K tile 1 on its way into stage par ^ 1.
    L += stride;
    const Head hn = head_of(L, &hd);   // the next tile's row gather flies during this tile's K loop
    kb_reset();
    kb_advance();

    f32x4 acc[8][8];   // [weight-row block ni][token-row block mi]
    // One K step: 16 groups of {4 products, the fragment reads of the next step, tile loads}, pinned in source order.
    // A K tile is multiplied in two steps and its successor but one is loaded meanwhile: tile load i (0..7: token rows,
    // 8..15: weight rows) of a wave goes out in group load_at(i) of the 32 (step 1, then step 0 of the next K tile).
    // Two loads per group hold up the products behind them (the path into LDS takes about one per group from each
    // wave), later ones have not landed at the wait: of eight placements (GEMM-1 of the prefill batch) this one is the
    // fastest, 941 us, against 963 (all in step 1, two per group) and 955 - 965 (8 + 8, or evenly over 28 or 32 groups).
    auto reads_of_group = [&](int set, int stage, int kk, int g, int half) {
      if (g < 4) read_frag(set, stage, kk, 2 * g + half);
      else if (g < 12 && half == 0) read_frag(set, stage, kk, g + 4);
    };
    auto group = [&](auto first, int set, int g, auto&& load, auto&& reads) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int t = 4 * g + q, ni = t >> 3, mi = t & 7;
        if constexpr (decltype(first)::value) mfma16_first(acc[ni][mi], fb[set][ni], fa[set][mi]);
        else mfma16(acc[ni][mi], fb[set][ni], fa[set][mi]);
        if (q == 0) load();
        if (q == 1) reads(0);
        if (q == 2) reads(1);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto load_at = [](int i) { return i < 12 ? i * 2 / 3 : i + 4; };   // 12 in step 1, groups 0..7; 4 in step 0, groups 0..3
    // step 0 of K tile kt in stage s: the rest of K tile kt+1 -> stage s^1, fragments of step 1.
    // head: the first step of an output tile, whose weight half of K tile 1 is all still to be requested
    auto step0 = [&](int s, const unsigned (&bo)[8], const char* lo, const char* hi, long long kb, auto head) {
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        group(head, 0, g,
              [&] {
                if constexpr (decltype(head)::value) {
                  if (g < 8) load_b(bo, lo, hi, kb, s ^ 1, g);
                } else {
#pragma unroll
                  for (int i = 8; i < 16; ++i)
                    if (load_at(i) == 16 + g) load_b(bo, lo, hi, kb, s ^ 1, i - 8);
                }
              },
              [&](int half) { reads_of_group(1, s, 1, g, half); });
      }
    };
    // step 1 of K tile kt in stage s, after the wait: first loads of K tile kt+2 -> stage s, step-0 fragments of K tile
    // kt+1.  tail: the last step of an output tile, whose epilogue uses the weight half of stage s: token half only
    auto step1 = [&](int s, const aoff_t (&ao)[8], int ktile, const unsigned (&bo)[8], const char* lo, const char* hi,
                     long long kb, auto tail) {
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        group(std::false_type{}, 1, g,
              [&] {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                  if (load_at(i) == g) {
                    if (i < 8) load_a(ao, ktile, s, i);
                    else if (!decltype(tail)::value) load_b(bo, lo, hi, kb, s, i - 8);
                  }
              },
              [&](int half) { reads_of_group(0, s ^ 1, 0, g, half); });
      }
    };
    step0(par, b_off, w_lo, w_hi, kb_next, std::true_type{});
    kb_advance();
    // K tiles 0 .. nk-3
    for (int kt = 0; kt < nk - 2; ++kt) {
      const int s = (par + kt) & 1;
      // K tile kt+1 has landed (this wave's loads, then every wave's), and every wave has issued
      // and completed its last reads of stage s, which may therefore be refilled
      wait_loads_and_barrier<0>();
      step1(s, a_off, kt + 2, b_off, w_lo, w_hi, kb_next, std::false_type{});
      step0(s ^ 1, b_off, w_lo, w_hi, kb_next, std::false_type{});
      kb_advance();
    }
    // K tile nk-2: its stage receives K tile 0 of the next output tile
    const int s = (par + nk - 2) & 1, s1 = s ^ 1;
    wait_loads_and_barrier<0>();
    aoff_t na_off[8];
    unsigned nb_off[8];
    offsets_of(hn, na_off, nb_off);   // the gather has long landed: nothing is outstanding here
    const char* nw_lo = static_cast<const char*>(a.B) + (long long)hn.widx * a.b_group_stride * 2;
    const char* nw_hi = SWIGLU ? static_cast<const char*>(a.B2) + (long long)hn.widx * a.b_group_stride * 2 : nw_lo;
    __builtin_amdgcn_sched_barrier(0);
    step1(s, na_off, 0, nb_off, nw_lo, nw_hi, 0, std::false_type{});
    step0(s1, nb_off, nw_lo, nw_hi, 0, std::false_type{});
    // K tile nk-1 (stage s1): the next tile's K tile 0 is complete in stage s and stage s1 is free: the token half of
    // the next tile's K tile 1 goes there
    wait_loads_and_barrier<0>();
    step1(s1, na_off, 1, nb_off, nw_lo, nw_hi, 0, std::true_type{});
    const int ready = mfma_results_ready();
#pragma unroll
    for (int ni = 0; ni < 8; ++ni)
#pragma unroll
      for (int mi = 0; mi < 8; ++mi) behind(ready, acc[ni][mi]);

    // epilogue.  acc[ni][mi] element e of lane l: output row (token) mi*16 + l%16, output column
    // ni*16 + (l/16)*4 + e of the wave tile: 4 consecutive columns per register quad.
    // Chunk c = 32 rows x 64 output columns = 4 KiB (128-byte rows, 16-byte slots swizzled like
    // the operand tiles), two buffers inside this wave's 8 KiB of stage s1's B region.
    {
      char* stg = smem + s1 * STAGE_BYTES + A_BYTES + wave * 8192;
      constexpr int NCH = SWIGLU ? 4 : 8;
      constexpr int W_COLS = SWIGLU ? 64 : 128;   // output columns of a wave tile
      char* wr = stg + (lane & 15) * 128 + ((lane >> 4) & 1) * 8;
      const int wsw = (lane >> 1) & 7;
      const int rrow = lane >> 3, rch = lane & 7;
      // A chunk sequence number cc alternates the two staging buffers (cc & 1).  Without SAVE chunk cc is
      // output chunk cc.  With SAVE the sequence is, per row block mi: the activated chunk, then the gate
      // and the up pre-activations of the same rows (kind 0, 1, 2), so that a row block's accumulators are
      // dead after its three chunks (keeping all of them live through a second pass spills registers, and
      // every reload of a spilled register waits for the next tile's loads as well).
      auto stage = [&](int cc) {
        char* buf = wr + (cc & 1) * 4096;
        const int kind = SAVE ? cc % 3 : 0;
        const int c = SAVE ? cc / 3 : cc;
        const int mi = SWIGLU ? c : (c >> 1), h = SWIGLU ? 0 : (c & 1);
#pragma unroll
        for (int m2 = 0; m2 < 2; ++m2)
#pragma unroll
          for (int nn = 0; nn < 4; ++nn) {   // 16 output columns
            const int gi = (nn >> 1) * 4 + (nn & 1);   // SWIGLU: weight-row block of the gate; the up block is gi + 2
            if (SAVE) {   // read again for every kind: values kept from one chunk to the next would not fit the registers
              asm volatile("" : "+a"(acc[gi][2 * mi + m2]));
              asm volatile("" : "+a"(acc[gi + 2][2 * mi + m2]));
            }
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if (SWIGLU && kind == 0)
                v[e] = swiglu_rcp(acc[gi][2 * mi + m2][e], acc[gi + 2][2 * mi + m2][e]);
              else if (SWIGLU)
                v[e] = acc[gi + 2 * (kind - 1)][2 * mi + m2][e];   // kind 1: gate, 2: up
              else
                v[e] = acc[4 * h + nn][2 * mi + m2][e];
            }
            uint2 pk;
            pk.x = pack_bf16(v[0], v[1]);
            pk.y = pack_bf16(v[2], v[3]);
            *reinterpret_cast<uint2*>(buf + m2 * 16 * 128 + (((nn * 2 + (lane >> 5)) ^ wsw) * 16)) = pk;
          }
      };
      // Stores go through a buffer descriptor over the wave tile's valid rows, so rows past the
      // group's end (and columns past N) are dropped by the hardware's range check: no branches.
      const int rows_left = min(hd.rows - hd.m0 - wm * 128, 128);
      const int col_w = hd.n0 + wn * W_COLS;   // first output column of the wave tile
      // (the last valid row counts only the wave tile's columns below N: with N < W_COLS and ldc = N a
      // whole tile width would reach into the next group's first row)
      // With the fused activation a wave tile is 64 columns and N a multiple of 64 (host), so a wave tile is whole
      // or wholly past N (every store of it redirected below): the constant keeps a scalar register free there.
      const int cols_left = SWIGLU ? W_COLS : min(a.N - col_w, W_COLS);
      const unsigned n_rec =
          rows_left > 0 && cols_left > 0 ? (unsigned)((rows_left - 1) * a.ldc + cols_left) * 2u : 0u;
      const unsigned long long c_tile = reinterpret_cast<unsigned long long>(
          C + (long long)(hd.row_base + hd.m0 + wm * 128) * a.ldc + hd.ccol + col_w);
      const unsigned long long c_tile_u =   // the descriptor has to sit in scalar registers
          ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(c_tile >> 32)) << 32) |
          (unsigned)__builtin_amdgcn_readfirstlane((unsigned)c_tile);
      const __amdgpu_buffer_rsrc_t c_rsrc = __builtin_amdgcn_make_buffer_rsrc(
          reinterpret_cast<void*>(c_tile_u), 0, __builtin_amdgcn_readfirstlane((int)n_rec), 0x00020000);
      // SAVE: the pre-activations go to rows of 2 * ldc elements, [gate | up] with the up half N columns
      // further.  One descriptor spans both halves of the wave tile's valid rows; an invalid row lies past
      // it because a row of that output is longer than N + 64 columns (2 * ldc >= 2 * N, N >= 64).
      const int ldc2 = 2 * a.ldc;
      const unsigned n_rec2 =
          SAVE && rows_left > 0 && cols_left > 0 ? (unsigned)((rows_left - 1) * ldc2 + a.N + cols_left) * 2u : 0u;
      const unsigned long long c2_tile = reinterpret_cast<unsigned long long>(
          static_cast<__bf16*>(SAVE ? a.C2 : a.C) + (long long)(hd.row_base + hd.m0 + wm * 128) * ldc2 + 2 * hd.ccol + col_w);
      const unsigned long long c2_tile_u =
          ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(c2_tile >> 32)) << 32) |
          (unsigned)__builtin_amdgcn_readfirstlane((unsigned)c2_tile);
      const __amdgpu_buffer_rsrc_t c2_rsrc = __builtin_amdgcn_make_buffer_rsrc(
          reinterpret_cast<void*>(c2_tile_u), 0, __builtin_amdgcn_readfirstlane((int)n_rec2), 0x00020000);
      u32x4 sv[4];
      auto read_chunk = [&](int cc) {
        const char* buf = stg + (cc & 1) * 4096;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int rl = it * 8 + rrow;   // row inside the 32-row chunk
          sv[it] = *reinterpret_cast<const u32x4*>(buf + rl * 128 + ((rch ^ ((rl >> 1) & 7)) * 16));
        }
      };
      auto store = [&](int cc) {
        const int kind = SAVE ? cc % 3 : 0;
        const int c = SAVE ? cc / 3 : cc;
        const int mi = SWIGLU ? c : (c >> 1), h = SWIGLU ? 0 : (c & 1);
        const int col = h * 64 + rch * 8;   // inside the wave tile
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int row = mi * 32 + it * 8 + rrow;
          if (kind == 0) {
            const unsigned off = col_w + col < a.N ? (unsigned)(row * a.ldc + col) * 2u : n_rec;
            __builtin_amdgcn_raw_buffer_store_b128(sv[it], c_rsrc, (int)off, 0, 0);
          } else {
            const unsigned off =
                col_w + col < a.N ? (unsigned)(row * ldc2 + col + (kind - 1) * a.N) * 2u : n_rec2;
            __builtin_amdgcn_raw_buffer_store_b128(sv[it], c2_rsrc, (int)off, 0, 0);
          }
        }
      };
      // chunk cc is converted and staged while the LDS reads of chunk cc-1 are in flight
      constexpr int NSEQ = SAVE ? 3 * NCH : NCH;
      stage(0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int cc = 1; cc < NSEQ; ++cc) {
        read_chunk(cc - 1);
        __builtin_amdgcn_sched_barrier(0);
        stage(cc);
        __builtin_amdgcn_sched_barrier(0);
        store(cc - 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      read_chunk(NSEQ - 1);
      store(NSEQ - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (!hn.valid) break;   // uniform over the block
    hd = hn;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      a_off[i] = na_off[i];
      b_off[i] = nb_off[i];
    }
    w_lo = nw_lo;
    w_hi = nw_hi;
    par = s;
  }
  // the loads issued for a tile that does not exist must land before the block's LDS is released
  wait_loads_and_barrier<0>();
}
}  // namespace t256

// ------------------------------------------------------------------------------------------
// f32 kernel (small layers for users who check numerics).  Block = 4 waves (2 x 2), block tile 32 x 64 x 64, wave tile
// 16 x 32 on v_mfma_f32_16x16x4_f32 (f32 products and sums; three 16-byte LDS reads of a lane feed eight of them, where a
// product on the vector unit takes two reads of its own).  Bound by latency where the layer is tiny (a
// chain of group offsets -> row index -> rows -> LDS -> products), by the matrix pipe where it is not.  The rows of 32
// tokens keep groups of a few dozen rows from being mostly padding and give a tiny layer blocks for every CU.
// A lane reads 16 bytes = 4 consecutive K of its row; product j of the four that follow takes element j of every lane, so
// the four products cover 16 K in an order of their own, the same for both operands.
// (256 tokens, d = 128, f = 256, 16 experts, k = 4: gate/up 15.6 -> 8.7 us, down 13.5 -> 7.3 us against one output per thread from
// 16 x 16 tiles on fma; 2048 tokens, d = f = 512, 32 experts, k = 4: 683 -> 171 us for both, 75 TFLOP/s.  Error against 64-bit sums
// the same to 1 %: 6.2e-7 relative in h, 4.1e-7 in y at d = f = 512.)
namespace f32t {
constexpr int BM = 32, BN = 64, BK = 64;
constexpr int STRIDE = BK + 4;   // 272-byte rows: the 16 rows of a fragment read start on 16 different bank quads

template <bool SWIGLU>
__global__ __launch_bounds__(256) void grouped_gemm_f32(const GemmArgs a) {
  __shared__ __attribute__((aligned(16))) float As[2][BM * STRIDE];   // two K tiles: one multiplied, one being written
  __shared__ __attribute__((aligned(16))) float Bs[2][BN * STRIDE];
  __shared__ TileInfo s_info;
  constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;   // SWIGLU: B rows 0..31 gate, 32..63 up of the same output columns
  const int n_tiles = (a.N + BN_OUT - 1) / BN_OUT;
  const int mt = blockIdx.x / n_tiles;
  const int n0 = (blockIdx.x % n_tiles) * BN_OUT;
  const TileInfo ti = find_tile<BM>(a, mt, &s_info);
  if (ti.group < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const long long widx = a.grp_widx ? a.grp_widx[ti.group] : (a.w_base + ti.group);

  // global -> LDS staging: a thread owns 16-byte vector kv of rows tid/16 + 16*i (rows are whole vectors: K % 4 == 0, host)
  const int kv = tid & 15, r_in = tid >> 4;
  const float* a_src[2];
  const float* b_src[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    int lr = ti.m0 + r_in + 16 * i;
    if (lr >= ti.rows) lr = ti.rows - 1;   // rows past the group are computed and dropped
    const int logical = ti.row_base + lr;
    const long long src = a.a_rows ? a.a_rows[logical] : logical;
    a_src[i] = static_cast<const float*>(a.A) + src * a.lda;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r_in + 16 * i;
    int ncol = n0 + (SWIGLU ? (r & 31) : r);
    if (ncol >= a.N) ncol = a.N - 1;
    b_src[i] = static_cast<const float*>(SWIGLU && i >= 2 ? a.B2 : a.B) + widx * a.b_group_stride + (long long)ncol * a.ldb;
  }
  const int nk = (a.K + BK - 1) / BK;
  f32x4 ga[2][2], gb[2][4];
  auto load_global = [&](int kt, f32x4 (&xa)[2], f32x4 (&xb)[4]) {
    const int k = kt * BK + kv * 4;
    const bool in = k < a.K;   // past K: zeros on both sides
    const int seg = a.K > a.kseg ? k / a.kseg : 0;   // which weight matrix along K (shared down projection)
    const long long boff = (long long)seg * a.b_group_stride + (k - seg * a.kseg);
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 2; ++i) xa[i] = in ? *reinterpret_cast<const f32x4*>(a_src[i] + k) : zero;
#pragma unroll
    for (int i = 0; i < 4; ++i) xb[i] = in ? *reinterpret_cast<const f32x4*>(b_src[i] + boff) : zero;
  };
  auto write_lds = [&](int buf, const f32x4 (&xa)[2], const f32x4 (&xb)[4]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) *reinterpret_cast<f32x4*>(&As[buf][(r_in + 16 * i) * STRIDE + kv * 4]) = xa[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4*>(&Bs[buf][(r_in + 16 * i) * STRIDE + kv * 4]) = xb[i];
  };
  f32x4 acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
  const int frag = (lane & 15) * STRIDE + (lane >> 4) * 4;
  const int b_row[2] = {SWIGLU ? wn * 16 : wn * 32, SWIGLU ? 32 + wn * 16 : wn * 32 + 16};
  // K tile kt out of LDS buffer `buf`; (xa, xb) holds tile kt+1 on entry and is refilled with tile kt+3
  auto k_tile = [&](int kt, int buf, f32x4 (&xa)[2], f32x4 (&xb)[4]) {
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const f32x4 fa = *reinterpret_cast<const f32x4*>(&As[buf][wm * 16 * STRIDE + frag + kk * 16]);
      f32x4 fb[2];
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) fb[nb] = *reinterpret_cast<const f32x4*>(&Bs[buf][b_row[nb] * STRIDE + frag + kk * 16]);
      if (kk == 0 && kt + 1 < nk) write_lds(buf ^ 1, xa, xb);
      if (kk == 1 && kt + 3 < nk) load_global(kt + 3, xa, xb);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[nb][j], fa[j], acc[nb], 0, 0, 0);
    }
    __syncthreads();   // tile kt+1 is in the other buffer for everyone, and nobody reads this one any more
  };
  load_global(0, ga[0], gb[0]);
  if (nk > 1) load_global(1, ga[1], gb[1]);
  write_lds(0, ga[0], gb[0]);
  if (nk > 2) load_global(2, ga[0], gb[0]);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    k_tile(kt, 0, ga[1], gb[1]);
    if (kt + 1 < nk) k_tile(kt + 1, 1, ga[0], gb[0]);
  }

  // element e of lane l: weight row (l/16)*4 + e, token l%16: four consecutive columns of one row (N % 4 == 0)
  const int row = ti.m0 + wm * 16 + (lane & 15);
  if (row >= ti.rows) return;
  float* crow = static_cast<float*>(a.C) + (long long)(ti.row_base + row) * a.ldc + group_col0(a, ti.group);
  if (SWIGLU) {
    const int col = n0 + wn * 16 + (lane >> 4) * 4;
    f32x4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = acc[0][e] / (1.0f + expf(-acc[0][e])) * acc[1][e];
    if (col < a.N) *reinterpret_cast<f32x4*>(crow + col) = out;
  } else {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int col = n0 + wn * 32 + nb * 16 + (lane >> 4) * 4;
      if (col < a.N) *reinterpret_cast<f32x4*>(crow + col) = acc[nb];
    }
  }
}
}  // namespace f32t

// compute units of the current device (the persistent kernel runs one block on each), cached
int device_cu_count(int* out) {
  static int cached[64];
  int dev = 0;
  OCC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64 || cached[dev] == 0) {
    int n = 0;
    OCC_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
    OCC_REQUIRE(n > 0, OCCULT_EHIP, "device reports %d compute units", n);
    if (dev < 0 || dev >= 64) {
      *out = n;
      return OCCULT_OK;
    }
    cached[dev] = n;
  }
  *out = cached[dev];
  return OCCULT_OK;
}

// sums the K slices of a split product in slice order and rounds once: out[row][col0 + col]
__global__ __launch_bounds__(256) void splitk_reduce_bf16(const float* __restrict__ ws, int ksplit, int M, int N,
                                                          __bf16* __restrict__ out, int ldc, int col0) {
  const size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;   // 4 columns per thread (N % 4 == 0)
  if (i >= (size_t)M * N) return;
  f32x4 sum = *reinterpret_cast<const f32x4*>(ws + i);
  for (int ks = 1; ks < ksplit; ++ks) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(ws + (size_t)ks * M * N + i);
    sum = sum + v;
  }
  const size_t row = i / N, col = i % N;
  uint2 pk;
  pk.x = pack_bf16(sum.x, sum.y);
  pk.y = pack_bf16(sum.z, sum.w);
  *reinterpret_cast<uint2*>(out + row * ldc + col0 + col) = pk;
}

// K slices for a product whose tiles alone would leave most of the chip idle (0 = do not split)
static int choose_ksplit(long long tiles, int nk) {
  if (tiles >= 384 || nk < 8) return 0;   // beyond that the tiles fill the chip by themselves
  long long ks = 1024 / tiles;   // about two rounds of 512 resident workgroups
  if (ks > nk / 4) ks = nk / 4;
  if (ks > 8) ks = 8;
  return ks >= 2 ? (int)ks : 0;
}

// Weights in the weight-streaming kernel's own order (bf16).  Region 1, gate and up, per weight
// matrix pair 4*f*d bytes: unit = 32 output columns, stage = 64 K elements; a stage is 8 blocks of
// 1 KiB in the order (K step ks, matrix m: gate or up, column block nb), block = 64 lanes x 16 bytes,
// lane l holding row nb*16 + l%16 of the unit at K offset ks*32 + (l/16)*8.  Region 2, down, per
// matrix 2*d*f bytes: the same with one matrix (4 blocks per stage).  One thread per 16-byte piece.
__global__ __launch_bounds__(256) void pack_weights_kernel(const u32x4* __restrict__ gate, const u32x4* __restrict__ up,
                                                           const u32x4* __restrict__ down, u32x4* __restrict__ out,
                                                           int n_mats, int d, int f) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long per1 = (long long)f * d / 4, per2 = (long long)d * f / 8;   // pieces per matrix pair / matrix
  const long long n1 = n_mats * per1;
  if (idx < n1) {
    const int e = (int)(idx / per1);
    long long rem = idx - e * per1;
    const int cb = (int)(rem / (8ll * d));           // unit: 32 columns x 2 matrices x d elements
    rem -= cb * 8ll * d;
    const int stage = (int)(rem / 512), blk = (int)(rem % 512) / 64, lane = (int)(rem % 64);
    const int ks = blk >> 2, m = (blk >> 1) & 1, nb = blk & 1;
    const int n = cb * 32 + nb * 16 + (lane & 15), k = stage * 64 + ks * 32 + (lane >> 4) * 8;
    out[idx] = (m ? up : gate)[(((long long)e * f + n) * d + k) / 8];
  } else if (idx < n1 + n_mats * per2) {
    const long long i2 = idx - n1;
    const int e = (int)(i2 / per2);
    long long rem = i2 - e * per2;
    const int cb = (int)(rem / (4ll * f));           // unit: 32 columns x f elements
    rem -= cb * 4ll * f;
    const int stage = (int)(rem / 256), blk = (int)(rem % 256) / 64, lane = (int)(rem % 64);
    const int ks = blk >> 1, nb = blk & 1;
    const int n = cb * 32 + nb * 16 + (lane & 15), k = stage * 64 + ks * 32 + (lane >> 4) * 8;
    out[idx] = down[(((long long)e * d + n) * f + k) / 8];
  }
}

// groups averaging under 24 rows take the weight-streaming kernel (one wave per 32 columns x 32 tokens)
static bool streams_weights(const GemmArgs& a, int total_rows) {
  // (that kernel addresses A rows with 32-bit byte offsets)
  return (long long)total_rows < 24ll * a.ngroups && a.N % skinny::BN_OUT == 0 &&
         (long long)a.a_rows_total * a.lda * 2 < (1ll << 32);
}

// Row tiles of bm rows over total_rows rows in groups: at most one partly filled one per group that has rows.  The grids are
// sized by this and workgroups beyond the last tile only look it up, but one token of 60 experts launched 2600 of them in
// front of the shared experts' workgroups (gate/up 20.2 -> 17.3 us, in the caller's weight layout 25.8 -> 19.1; 4 tokens 44 -> 38.5).
static long long row_tiles_max(const GemmArgs& a, int total_rows, int bm) {
  if (a.grp_offset == nullptr) return (long long)a.ngroups * ((a.M + bm - 1) / bm);
  return total_rows / bm + min_i(total_rows, a.ngroups);
}

// The weight-streaming kernel over `a` (grouped rows, total_rows of them) and, when b is not NULL, over `b` in the
// same launch (uniform groups of b->M rows; same N, K and weight order as `a`, one weight matrix along K in both).
static int launch_skinny(const GemmArgs& a, const GemmArgs* b, bool swiglu, int total_rows, hipStream_t s) {
  const bool ksplit = swiglu;   // the gate/up product's waves split K; the down projection's keep whole columns
  const long long n_cb = a.N / skinny::BN_OUT;
  const long long wgs_per_mt = ksplit ? n_cb : (n_cb + 3) / 4;
  const long long a_blocks = row_tiles_max(a, total_rows, 32) * wgs_per_mt;
  long long blocks = a_blocks;
  if (b != nullptr) {
    OCC_REQUIRE(b->N == a.N && b->grp_offset == nullptr && (b->Bp != nullptr) == (a.Bp != nullptr) && a.kseg == a.K &&
                    b->K % b->kseg == 0,
                OCCULT_EINVAL, "the two problems of one weight-streaming launch differ in shape class");
    blocks += skinny::second_blocks(*b);
  }
  OCC_REQUIRE(blocks < (1ll << 31), OCCULT_EINVAL, "grouped GEMM grid too large");
  const dim3 grid((unsigned)blocks), block(256);
  // the packed order holds whole matrices: a K that walks several of them steps from one matrix's stream to the next
  const bool packed = a.Bp != nullptr && (a.kseg == a.K || a.K % a.kseg == 0);
  const GemmArgs& b2 = b ? *b : a;
  const int ab = (int)a_blocks;
  if (swiglu && packed) hipLaunchKernelGGL((skinny::grouped_gemm_bf16<true, 2, true, true>), grid, block, 0, s, a, b2, ab, skinny::NoFront{});
  else if (swiglu) hipLaunchKernelGGL((skinny::grouped_gemm_bf16<true, 2, false, true>), grid, block, 0, s, a, b2, ab, skinny::NoFront{});
  else if (packed) hipLaunchKernelGGL((skinny::grouped_gemm_bf16<false, 2, true, false>), grid, block, 0, s, a, b2, ab, skinny::NoFront{});
  else hipLaunchKernelGGL((skinny::grouped_gemm_bf16<false, 2, false, false>), grid, block, 0, s, a, b2, ab, skinny::NoFront{});
  OCC_LAUNCH_CHECK("grouped_gemm");
  return OCCULT_OK;
}

constexpr int kStreamParts = 4;   // parts of K of that kernel where its waves split K: one per wave

// rows per group from which a product takes the 256-row tiles: uniform groups; grouped rows of the gate/up product
constexpr long long kBigRowsUniform = 192, kBigRowsSwiglu = 129;

// the large-tile kernels address a weight matrix's rows with 32-bit byte offsets
static bool weights_below_4gib(const GemmArgs& a) { return (long long)a.N * a.ldb * 2 < (1ll << 32); }

static bool uses_tile256(const GemmArgs& a, bool swiglu, int total_rows) {
  // 256-row tiles once groups average enough rows and there are at least two K tiles to pipeline
  // (measured on 60 experts, d = 2048, f = 1408: the gate/up product is weight-bound on the
  // 128-row tiles until an expert's rows no longer fit one of them; the down projection is
  // faster on the 256-row tiles from about 64 rows per expert)
  const long long big_rows = a.grp_offset == nullptr ? kBigRowsUniform : (swiglu ? kBigRowsSwiglu : 64);
  return (long long)total_rows >= big_rows * a.ngroups && a.ksplit <= 1 && a.K >= 2 * t256::BK && a.N % 64 == 0 &&
         weights_below_4gib(a);
}

// *fused_save: the pre-activations asked for through a.C2 were written by the launch itself
static int launch_gemm_main(const occult_cfg_t& c, const GemmArgs& a, bool swiglu, int total_rows, hipStream_t s,
                            bool* fused_save_out) {
  *fused_save_out = false;
  if (c.dtype == OCCULT_BF16) {
    const bool use_big = uses_tile256(a, swiglu, total_rows);
    // an A operand of 4 GiB or more takes the variant of the 256-row tiles with 64-bit row offsets
    const bool wide = (long long)a.a_rows_total * a.lda * 2 >= (1ll << 32);
    // of these kernels only the 256-row tiles store the pre-activations themselves (not with 64-bit offsets: registers)
    const bool fused_save = swiglu && a.C2 != nullptr && use_big && !wide;
    *fused_save_out = fused_save;
    const bool use_skinny = !use_big && streams_weights(a, total_rows);
    if (use_skinny) return launch_skinny(a, nullptr, swiglu, total_rows, s);
    const int bm = use_big ? t256::BM : small::BM;
    const int bn = use_big ? t256::BN : small::BN;
    const int bn_out = swiglu ? bn / 2 : bn;
    const long long m_tiles = row_tiles_max(a, total_rows, bm);
    long long blocks = mapped_grid(m_tiles, (a.N + bn_out - 1) / bn_out);
    OCC_REQUIRE(blocks < (1ll << 31), OCCULT_EINVAL, "grouped GEMM grid too large");
    if (use_big) {   // persistent: one block per CU, a multiple of 8 so a block keeps its XCD
      int cus = 0;
      const int rc = device_cu_count(&cus);
      if (rc) return rc;
      const long long resident = cus >= 8 ? cus / 8 * 8 : 8;
      if (blocks > resident) blocks = resident;
    }
    const bool split = !use_big && !swiglu && a.ksplit > 1;   // caller set ksplit and ws (one group)
    GemmArgs b = a;
    if (!split) b.ksplit = 0;
    // the XCD-aware order pads the grid to whole chunks per XCD: pointless when there are few tiles
    const long long plain_blocks = m_tiles * ((a.N + bn_out - 1) / bn_out);
    if (!use_big && plain_blocks <= 512) {
      b.plain_map = 1;
      blocks = plain_blocks;
    }
    const dim3 grid((unsigned)blocks, split ? (unsigned)b.ksplit : 1u), block(256);
    if (use_big) {
      if (swiglu && fused_save) hipLaunchKernelGGL((t256::grouped_gemm_bf16<true, true>), grid, block, 0, s, b);
      else if (swiglu && wide) hipLaunchKernelGGL((t256::grouped_gemm_bf16<true, false, true>), grid, block, 0, s, b);
      else if (swiglu) hipLaunchKernelGGL((t256::grouped_gemm_bf16<true, false>), grid, block, 0, s, b);
      else if (wide) hipLaunchKernelGGL((t256::grouped_gemm_bf16<false, false, true>), grid, block, 0, s, b);
      else hipLaunchKernelGGL((t256::grouped_gemm_bf16<false, false>), grid, block, 0, s, b);
    } else {
      if (swiglu) hipLaunchKernelGGL(small::grouped_gemm_bf16<true>, grid, block, 0, s, b);
      else hipLaunchKernelGGL(small::grouped_gemm_bf16<false>, grid, block, 0, s, b);
    }
    if (split) {
      OCC_LAUNCH_CHECK("grouped_gemm");
      const size_t quads = (size_t)b.M * b.N / 4;
      hipLaunchKernelGGL(splitk_reduce_bf16, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, b.ws, b.ksplit,
                         b.M, b.N, static_cast<__bf16*>(b.C), b.ldc, b.c_col0);
    }
  } else {
    const int bn_out = swiglu ? f32t::BN / 2 : f32t::BN;
    const long long blocks = row_tiles_max(a, total_rows, f32t::BM) * ((a.N + bn_out - 1) / bn_out);
    OCC_REQUIRE(blocks < (1ll << 31), OCCULT_EINVAL, "grouped GEMM grid too large");
    const dim3 grid((unsigned)blocks), block(256);
    if (swiglu) hipLaunchKernelGGL(f32t::grouped_gemm_f32<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(f32t::grouped_gemm_f32<false>, grid, block, 0, s, a);
  }
  OCC_LAUNCH_CHECK("grouped_gemm");
  return OCCULT_OK;
}

// one pre-activation (gate or up) of a gate/up product `a`, stored where a.C2 asks for it, as a product of its own
static GemmArgs preactivation(const GemmArgs& a, bool up) {
  GemmArgs p = a;
  p.C = a.C2; p.ldc = 2 * a.ldc; p.c_group_cols = 2 * a.c_group_cols; p.C2 = nullptr; p.B2 = nullptr; p.Bp = nullptr;
  p.B = up ? a.B2 : a.B;
  p.c_col0 = 2 * a.c_col0 + (up ? a.N : 0);
  p.ksplit = 0;
  return p;
}

int launch_gemm(const occult_cfg_t& c, const GemmArgs& a, bool swiglu, int total_rows, hipStream_t s) {
  if (total_rows == 0) return OCCULT_OK;
  bool fused_save = false;
  int rc = launch_gemm_main(c, a, swiglu, total_rows, s, &fused_save);
  if (rc) return rc;
  if (!swiglu || a.C2 == nullptr || fused_save) return rc;
  for (int up = 0; up < 2 && rc == OCCULT_OK; ++up)
    rc = launch_gemm_main(c, preactivation(a, up != 0), false, total_rows, s, &fused_save);
  return rc;
}

// Which products take the 128-row tiles (ffn_tile128.hip).  Rows per group, d = 2048, f = 1024 / 1408, 60 - 64 experts:
//  - below them stands the weight-streaming kernel, above the 256-row tiles, which need a third fewer operand bytes per
//    product but waste more on partly filled tiles and on the last round of tiles over the CUs;
//  - with shared experts one launch does both sets' work, which alone would leave most CUs idle (500 tokens: 118 of
//    357 us) or add a last round of its own: up to about 800 rows per group (656 rows: 1116 us against 1057; 768: equal),
//    and down to any number where shares_launch() says so;
//  - without, from 24 rows (32: 226 us against 220; 20: 215 against 218) up to 500: half as high, the tiles of a launch divide
//    more evenly over the CUs.  Time over that of the 256-row tiles, 242 - 490 rows per group of 32 - 128 experts, K = 384 - 2816, N = 384 -
//    2048: 336 gate/up products 0.84 on average (with and without stored pre-activations), 27 of them more than 1.03, at worst
//    1.16; 700 down projections, whose shapes are the backward's two products as well, 0.91, 108 more than 1.03, at worst 1.14, by
//    how the tiles happen to fill their last round.  The better of the two at every size would be 0.83 and 0.90.  750 rows: 1.08.
static bool fits_tile128(const GemmArgs& a) {
  return a.K >= 192 && a.K % 64 == 0 && a.N % 64 == 0 && (long long)a.a_rows_total * a.lda * 2 < (1ll << 32) &&
         weights_below_4gib(a);
}
static bool uses_tile128(const occult_cfg_t& c, const GemmArgs& a, const GemmArgs* b, int total_rows) {
  if (c.dtype != OCCULT_BF16 || a.grp_offset == nullptr || !fits_tile128(a) || (b != nullptr && !fits_tile128(*b)))
    return false;
  const long long lo = b != nullptr ? 0 : 24, hi = b != nullptr ? 800 : 500;
  return total_rows >= lo * a.ngroups && total_rows < hi * a.ngroups;
}

// Parts of K, summed one by one, of the kernel that would otherwise take a product: the 128-row tiles sum the same parts,
// so that a row's result does not depend on which of the two takes its batch.  The weight-streaming kernel's four waves
// take a quarter each of the gate/up product; a.ksplit: parts asked for.
static int k_parts(const GemmArgs& a, bool swiglu, int total_rows) {
  if (a.ksplit > 1) return a.ksplit;
  return swiglu && !uses_tile256(a, swiglu, total_rows) && streams_weights(a, total_rows) ? kStreamParts : 1;
}

// Whether the shared experts' product `b` runs in one launch of 128-row tiles with the routed experts' `a`, where those
// take it.  Apart, `a` goes to the kernel that takes it alone and `b` to its own.  What decides it (1000 pairs of times over
// 4 - 128 experts, 1 - 4 shared ones, d = 512 - 4096, f = 384 - 1536):
//  - a gate/up product that would stream its weights: the tiles spend a fixed time per expert, and gain the time that the
//    shared rows would take alone.  Joined from 6144 shared rows x K per expert, twice that where the weights are packed:
//    of 127 batches below 24 rows per expert 0.81 of the time apart on average (at worst 1.16), packed 0.88 (1.15).
//    (64 + 4 experts, 155 tokens, d = 1024, f = 512: 46 us against 43; 60 + 1, 169 tokens, the same widths: 27 against 37.)
//  - a down projection with scratch: apart, its K (S matrices long) is split over workgroups, joined it is one block's chain
//    of about 0.75 us per K tile of 64, and its block takes the fewer of the routed tiles (ffn_tile128.hip).  Joined while the
//    chain's excess over a block's share of all tiles stays within 9 K tiles of what it saves, twice the work of `b` spread over
//    256 CUs.  (Forward passes joined over apart, 8 - 128 experts, 1 - 4 shared ones, d = 512 - 4096: of 90 batches of 150 - 1722 tokens
//    from 24 rows per expert on the 69 taken 0.75 - 1.04, 0.90 on average, the 21 left apart 0.94 - 1.24; of 40 of 139 - 476 tokens
//    below 24 rows the 31 taken 0.85 - 1.00, with packed weights, which the tiles do not read, 0.91 - 1.00, the 9 left 0.95 - 1.10 and
//    0.99 - 1.12.  Joined / apart, d = 2048, f = 1408: 64 + 2 experts, 1000 tokens 311 / 358 us, 200 tokens 237 / 276, packed 238 / 259;
//    left apart: 60 + 4, 300 tokens 276 / 295, its worst miss, 200 tokens packed 256 / 248; 64 + 4, 476 tokens, 1024, 896 154 / 143.)
static bool shares_launch(const GemmArgs& a, const GemmArgs& b, bool swiglu, int total_rows) {
  if (swiglu && streams_weights(a, total_rows))
    return (long long)b.ngroups * b.M * a.K > (a.Bp != nullptr ? 2 : 1) * 6144ll * a.ngroups;
  if (b.ksplit <= 1) return true;
  const long long n_tiles = (a.N + 255) / 256;
  const long long groups = a.ngroups < total_rows ? a.ngroups : total_rows;
  const long long tiles_a = groups > 0 ? groups * ((total_rows / groups + 127) / 128) * n_tiles : 0;   // evenly loaded experts
  const long long tiles_b = (b.M + 127) / 128 * n_tiles, tiles = tiles_a + tiles_b;
  const long long share = (tiles_a * a.K + tiles_b * b.K) / (tiles < 256 ? tiles : 256);
  return b.K - share - tiles_b * b.K / 128 <= 9 * 64;
}

static int launch_preactivation_pair(const occult_cfg_t& c, const GemmArgs& a, const GemmArgs* b, int total_rows, int rows_b,
                                     hipStream_t s) {
  int rc = OCCULT_OK;
  for (int up = 0; up < 2 && rc == OCCULT_OK; ++up) {
    const GemmArgs p = preactivation(a, up != 0);
    GemmArgs q{};
    if (b != nullptr) q = preactivation(*b, up != 0);
    rc = launch_gemm_pair(c, p, b ? &q : nullptr, false, total_rows, rows_b, s);
  }
  return rc;
}

int launch_gemm_pair(const occult_cfg_t& c, const GemmArgs& a, const GemmArgs* b, bool swiglu, int total_rows, int rows_b,
                     hipStream_t s) {
  if (b != nullptr && !shares_launch(a, *b, swiglu, total_rows)) {
    const int rc = launch_gemm_pair(c, a, nullptr, swiglu, total_rows, 0, s);
    return rc ? rc : launch_gemm(c, *b, swiglu, rows_b, s);
  }
  if (total_rows > 0 && uses_tile128(c, a, b, total_rows)) {
    GemmArgs p = a, q{};
    if (b != nullptr) q = *b;
    p.silu_rcp = total_rows >= kBigRowsSwiglu * p.ngroups;   // as launch_gemm_main would choose
    q.silu_rcp = rows_b >= kBigRowsUniform * q.ngroups;
    p.ksplit = k_parts(a, swiglu, total_rows);
    if (b != nullptr) q.ksplit = k_parts(*b, swiglu, rows_b);
    // pre-activations are stored as one sum over K: by the launch itself unless it sums the activation's in parts
    const bool apart = a.C2 != nullptr && (p.ksplit > 1 || q.ksplit > 1);
    if (apart) p.C2 = q.C2 = nullptr;
    const int rc = launch_tile128(p, b ? &q : nullptr, swiglu, total_rows, s);
    return rc || !apart ? rc : launch_preactivation_pair(c, a, b, total_rows, rows_b, s);
  }
  const int rc = launch_gemm(c, a, swiglu, total_rows, s);
  if (rc || b == nullptr) return rc;
  return launch_gemm(c, *b, swiglu, rows_b, s);
}

}  // namespace occult

using namespace occult;


// Small batches whose routed experts take the weight-streaming kernel: the shared experts ride in the same two
// launches, the down projection as one product whose K walks the S matrices (no scratch, no extra launch).
constexpr int kPairMaxT = 128;   // a shared expert's weights are requested once per 32 tokens (from L2 after the first)
static bool pairs_shared_with_routed(const occult_cfg_t& c) {
  return c.dtype == OCCULT_BF16 && c.S > 0 && c.T > 0 && c.T <= kPairMaxT && (long long)c.T * c.k < 24ll * c.E &&
         c.f % skinny::BN_OUT == 0 && c.d % skinny::BN_OUT == 0 &&
         (long long)sfd_rows_max(c) * c.d * 2 < (1ll << 32) && (long long)c.T * c.k * c.f * 2 < (1ll << 32) &&
         (long long)c.T * c.S * c.f * 2 < (1ll << 32);
}

// Scratch that lets the shared experts' down projection of a small batch be split over K: the
// product has T/128 x d/128 tiles only (32 for T = 160, d = 2048) with a long K = S*f.
// Asked for by shape alone, also where the shared product then joins the routed experts' launch and sums its parts in
// registers: scratch sized for a server's largest batch serves the smaller ones, and a caller that gives it gets the sums
// in the same parts either way.
static size_t ffn_ws_need(const occult_cfg_t& c, int* ksplit_out) {
  *ksplit_out = 0;
  if (c.S == 0 || c.dtype != OCCULT_BF16 || c.T == 0) return 0;
  if (c.T < 24) return 0;   // those batches take the weight-streaming kernel
  if (pairs_shared_with_routed(c)) return 0;   // the shared experts run inside the routed experts' launches
  const long long tiles = (long long)((c.T + 127) / 128) * ((c.d + 127) / 128);
  const int ks = choose_ksplit(tiles, c.S * c.f / 64);
  if (ks == 0 || c.d % 4 != 0) return 0;
  *ksplit_out = ks;
  return (size_t)ks * c.T * c.d * sizeof(float);
}

extern "C" int occult_expert_ffn_ws_bytes(const occult_cfg_t* cfg, size_t* ws_bytes) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  OCC_REQUIRE(ws_bytes, OCCULT_ENULLPTR, "ws_bytes is NULL");
  int ks = 0;
  *ws_bytes = ffn_ws_need(*cfg, &ks);
  return OCCULT_OK;
}

namespace occult {
int check_ffn_args(const occult_cfg_t& c, const occult_plan_t* plan, const void* sfd_x, const void* x,
                   const occult_weights_t* weights, const void* epd_h, const void* epd_y, const void* h_shared, const void* y_shared) {
  OCC_REQUIRE(plan && plan->exp_offset && plan->pos_expert && plan->epd_sfd_row, OCCULT_ENULLPTR,
              "plan or one of its tables is NULL");
  OCC_REQUIRE(weights && weights->w_gate && weights->w_up && weights->w_down, OCCULT_ENULLPTR,
              "weights or one of its tensors is NULL");
  OCC_REQUIRE(sfd_x && epd_h && epd_y, OCCULT_ENULLPTR, "sfd_x, epd_h or epd_y is NULL");
  if (c.S > 0)
    OCC_REQUIRE(x && h_shared && y_shared, OCCULT_ENULLPTR, "x, h_shared or y_shared is NULL with S=%d", c.S);
  const int es = elem_size(c);
  OCC_REQUIRE(((size_t)c.d * es) % 16 == 0 && ((size_t)c.f * es) % 16 == 0, OCCULT_EALIGN,
              "rows of d=%d or f=%d elements are not multiples of 16 bytes", c.d, c.f);
  if (c.dtype == OCCULT_BF16)
    OCC_REQUIRE(c.d % 64 == 0 && c.f % 64 == 0, OCCULT_ESHAPE,
                "bf16 path needs d and f to be multiples of 64 (d=%d, f=%d)", c.d, c.f);
  OCC_REQUIRE(aligned16(sfd_x) && aligned16(epd_h) && aligned16(epd_y) && aligned16(x) &&
                  aligned16(h_shared) && aligned16(y_shared) && aligned16(weights->w_gate) &&
                  aligned16(weights->w_up) && aligned16(weights->w_down),
              OCCULT_EALIGN, "a buffer is not 16-byte aligned");
  return OCCULT_OK;
}

bool forward_uses_front(const occult_cfg_t& c) {
  return c.dtype == OCCULT_BF16 && c.ffn_phase == 0 && fits_front(c) && (long long)c.T * c.k < 24ll * c.E &&
         c.f % skinny::BN_OUT == 0 && (c.S == 0 || pairs_shared_with_routed(c));
}

// the two problems of the gate/up product: h = silu(x W_gate^T) * (x W_up^T); the shared experts as S groups over the rows of x
static void gate_up_products(const occult_cfg_t& c, const void* x, const occult_weights_t* weights, const void* packed, void* epd_h,
                             void* h_shared, GemmArgs* first, GemmArgs* second) {
  GemmArgs g1{}, a1{};
  a1.A = x; g1.lda = a1.lda = c.d;
  g1.B = a1.B = weights->w_gate; g1.B2 = a1.B2 = weights->w_up;
  g1.b_group_stride = a1.b_group_stride = (long long)c.f * c.d;
  g1.ldb = a1.ldb = g1.kseg = a1.kseg = g1.K = a1.K = c.d;
  g1.Bp = packed; g1.bp_group_stride = a1.bp_group_stride = 4ll * c.f * c.d;
  g1.N = a1.N = c.f;
  g1.C = epd_h; g1.ldc = c.f;
  a1.C = h_shared; a1.ldc = c.S * c.f; a1.c_group_cols = c.f;
  g1.ngroups = c.E;
  a1.w_base = c.E; a1.ngroups = c.S; a1.M = c.T; a1.a_rows_total = c.T;
  *first = g1;
  *second = a1;
}

void front_products(const occult_cfg_t& c, const void* x, const occult_weights_t* weights, const void* packed, void* epd_h,
                    void* h_shared, GemmArgs* first, GemmArgs* second) {
  gate_up_products(c, x, weights, packed, epd_h, h_shared, first, second);
  first->A = x;
  second->Bp = packed;
}
}  // namespace occult

static int expert_ffn_impl(const occult_cfg_t* cfg, const occult_plan_t* plan, const void* sfd_x,
                           const void* x, const occult_weights_t* weights, const void* packed, void* epd_h,
                           void* epd_y, void* h_shared, void* y_shared, void* ws, size_t ws_bytes,
                           occult_stream_t stream, void* epd_gu = nullptr, void* gu_shared = nullptr) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  if (c.T == 0) return OCCULT_OK;
  rc = check_ffn_args(c, plan, sfd_x, x, weights, epd_h, epd_y, h_shared, y_shared);
  if (rc) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int n_epd = c.T * c.k;

  const bool do1 = c.ffn_phase != 2, do2 = c.ffn_phase != 1;
  const int once_rows = epd_gu != nullptr ? kOnceTrain : c.S > c.k ? kOnceForwardShared : kOnceForward;

  if (do1) {   // h = silu(x W_gate^T) * (x W_up^T); the S shared experts as S groups over the same T rows
    GemmArgs g1, a1;
    gate_up_products(c, x, weights, packed, epd_h, h_shared, &g1, &a1);
    g1.A = sfd_x; g1.a_rows = plan->epd_sfd_row; g1.a_rows_total = sfd_rows_max(c);
    g1.C2 = epd_gu;      // rows of 2f: [gate | up]
    g1.once_rows = once_rows;
    a1.C2 = gu_shared;   // rows of S * 2f: per shared expert [gate | up]
    g1.grp_offset = plan->exp_offset; g1.grp_widx = plan->pos_expert;
    if (pairs_shared_with_routed(c)) {
      a1.Bp = packed;
      rc = launch_skinny(g1, &a1, true, n_epd, s);
      if (rc == OCCULT_OK && epd_gu != nullptr) rc = launch_preactivation_pair(c, g1, &a1, n_epd, c.T * c.S, s);
    } else {
      rc = launch_gemm_pair(c, g1, c.S > 0 ? &a1 : nullptr, true, n_epd, c.T * c.S, s);
    }
    if (rc) return rc;
  }
  if (do2) {   // y = h W_down^T; the shared experts as one product whose K dimension walks the S down matrices
    GemmArgs g2{}, a2{};
    g2.A = epd_h; g2.lda = c.f;
    a2.A = h_shared; a2.lda = c.S * c.f;
    g2.B = a2.B = weights->w_down;
    g2.b_group_stride = a2.b_group_stride = (long long)c.d * c.f;
    g2.ldb = a2.ldb = g2.kseg = a2.kseg = g2.K = c.f;
    a2.K = c.S * c.f;
    if (packed) g2.Bp = static_cast<const char*>(packed) + 4ll * c.f * c.d * (c.E + c.S);
    g2.bp_group_stride = a2.bp_group_stride = 2ll * c.d * c.f;
    g2.N = a2.N = c.d;
    g2.C = epd_y; g2.ldc = c.d;
    a2.C = y_shared; a2.ldc = c.d;
    g2.grp_offset = plan->exp_offset; g2.grp_widx = plan->pos_expert; g2.ngroups = c.E;
    g2.a_rows_total = n_epd;
    g2.once_rows = once_rows;
    a2.w_base = c.E; a2.ngroups = 1; a2.M = c.T; a2.a_rows_total = c.T;
    if (pairs_shared_with_routed(c)) {
      a2.Bp = g2.Bp;
      rc = launch_skinny(g2, &a2, false, n_epd, s);
    } else {
      int ks = 0;
      const size_t need = ffn_ws_need(c, &ks);
      if (ks > 1 && ws != nullptr && ws_bytes >= need) {
        a2.ksplit = ks;
        a2.ws = static_cast<float*>(ws);
      }
      rc = launch_gemm_pair(c, g2, c.S > 0 ? &a2 : nullptr, false, n_epd, c.T, s);
    }
    if (rc) return rc;
  }
  return OCCULT_OK;
}

extern "C" int occult_expert_ffn(const occult_cfg_t* cfg, const occult_plan_t* plan, const void* sfd_x,
                                 const void* x, const occult_weights_t* weights, void* epd_h, void* epd_y,
                                 void* h_shared, void* y_shared, occult_stream_t stream) {
  return expert_ffn_impl(cfg, plan, sfd_x, x, weights, nullptr, epd_h, epd_y, h_shared, y_shared, nullptr, 0, stream);
}

extern "C" int occult_expert_ffn_ws(const occult_cfg_t* cfg, const occult_plan_t* plan, const void* sfd_x,
                                    const void* x, const occult_weights_t* weights, void* epd_h, void* epd_y,
                                    void* h_shared, void* y_shared, void* ws, size_t ws_bytes,
                                    occult_stream_t stream) {
  if (ws != nullptr) OCC_REQUIRE(aligned16(ws), OCCULT_EALIGN, "ws is not 16-byte aligned");
  return expert_ffn_impl(cfg, plan, sfd_x, x, weights, nullptr, epd_h, epd_y, h_shared, y_shared, ws, ws_bytes, stream);
}

extern "C" int occult_expert_ffn_train(const occult_cfg_t* cfg, const occult_plan_t* plan, const void* sfd_x,
                                       const void* x, const occult_weights_t* weights, void* epd_h, void* epd_y,
                                       void* h_shared, void* y_shared, void* epd_gu, void* gu_shared, void* ws,
                                       size_t ws_bytes, occult_stream_t stream) {
  OCC_REQUIRE(epd_gu != nullptr, OCCULT_ENULLPTR, "epd_gu is NULL");
  OCC_REQUIRE(cfg == nullptr || cfg->S == 0 || gu_shared != nullptr, OCCULT_ENULLPTR, "gu_shared is NULL with shared experts");
  OCC_REQUIRE(aligned16(epd_gu) && aligned16(gu_shared) && aligned16(ws), OCCULT_EALIGN, "a buffer is not 16-byte aligned");
  return expert_ffn_impl(cfg, plan, sfd_x, x, weights, nullptr, epd_h, epd_y, h_shared, y_shared, ws, ws_bytes, stream,
                         epd_gu, gu_shared);
}

static size_t packed_bytes(const occult_cfg_t& c) {
  return c.dtype == OCCULT_BF16 ? (size_t)(c.E + c.S) * 3 * c.d * c.f * 2 : 0;
}

extern "C" int occult_pack_weights_bytes(const occult_cfg_t* cfg, size_t* bytes) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  OCC_REQUIRE(bytes, OCCULT_ENULLPTR, "bytes is NULL");
  *bytes = packed_bytes(*cfg);
  return OCCULT_OK;
}

extern "C" int occult_pack_weights(const occult_cfg_t* cfg, const occult_weights_t* weights, void* packed,
                                   size_t packed_size, occult_stream_t stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  if (c.dtype != OCCULT_BF16) return OCCULT_OK;   // the f32 path has no weight-streaming kernel
  OCC_REQUIRE(weights && weights->w_gate && weights->w_up && weights->w_down && packed, OCCULT_ENULLPTR,
              "weights, one of its tensors or packed is NULL");
  OCC_REQUIRE(c.d % 64 == 0 && c.f % 64 == 0, OCCULT_ESHAPE,
              "bf16 path needs d and f to be multiples of 64 (d=%d, f=%d)", c.d, c.f);
  OCC_REQUIRE(packed_size >= packed_bytes(c), OCCULT_EWORKSPACE, "packed buffer of %zu bytes < required %zu", packed_size,
              packed_bytes(c));
  OCC_REQUIRE(aligned16(weights->w_gate) && aligned16(weights->w_up) && aligned16(weights->w_down) && aligned16(packed),
              OCCULT_EALIGN, "a buffer is not 16-byte aligned");
  const long long pieces = (long long)packed_bytes(c) / 16;
  OCC_REQUIRE((pieces + 255) / 256 < (1ll << 31), OCCULT_EINVAL, "too many weights for one launch");
  hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), static_cast<const u32x4*>(weights->w_gate),
                     static_cast<const u32x4*>(weights->w_up), static_cast<const u32x4*>(weights->w_down),
                     static_cast<u32x4*>(packed), c.E + c.S, c.d, c.f);
  OCC_LAUNCH_CHECK("pack_weights_kernel");
  return OCCULT_OK;
}

extern "C" int occult_expert_ffn_packed(const occult_cfg_t* cfg, const occult_plan_t* plan, const void* sfd_x,
                                        const void* x, const occult_weights_t* weights, const void* packed,
                                        void* epd_h, void* epd_y, void* h_shared, void* y_shared, void* ws,
                                        size_t ws_bytes, occult_stream_t stream) {
  if (ws != nullptr) OCC_REQUIRE(aligned16(ws), OCCULT_EALIGN, "ws is not 16-byte aligned");
  if (packed != nullptr) OCC_REQUIRE(aligned16(packed), OCCULT_EALIGN, "packed is not 16-byte aligned");
  const void* use = (cfg && cfg->dtype == OCCULT_BF16) ? packed : nullptr;
  return expert_ffn_impl(cfg, plan, sfd_x, x, weights, use, epd_h, epd_y, h_shared, y_shared, ws, ws_bytes, stream);
}
