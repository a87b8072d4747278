// Backward pass of the expert computation: weight gradients of the grouped SwiGLU experts.
//
// Same sources as ffn_backward.hip (the paper trains through the layer and prints no backward
// algorithm; this is the chain rule through the forward's expert on the same plan).  For the
// expert at placement position P with EPD rows q in [exp_offset[P], exp_offset[P+1]):
//   dW_down = sum_q epd_dy[q] (x) epd_h[q]          [d][f]
//   dW_gate = sum_q dg[q] (x) x_q,  dW_up = sum_q du[q] (x) x_q     [f][d],  x_q = sfd_x[epd_sfd_row[q]]
// i.e. per expert C[m][n] = sum over its rows r of A[r][m] * B[src(r)][n]: a contraction over the
// ROW index of two row-major operands, the one GEMM shape the forward kernels do not cover (their
// operands are both contiguous along the contracted index).
//
// bf16 kernel (namespace wgd below).  Block = 256 threads = 4 waves (2 x 2), block tile 256 x 256
// outputs, wave tile 128 x 128 = 8 x 8 v_mfma_f32_16x16x32_bf16 tiles (256 accumulator registers, one
// block per CU).  Outputs are f32 (gradient accumulation across calls is exact to f32), stored
// as whole rows of a wave tile, 16 rows at a time through LDS, and marked as not to be kept in L2 (the operands are what is
// read again: 64 + 2 experts, 562 rows each, 1460 us for the three products with 64-byte pieces straight from the
// accumulators, 1359 with whole rows, 1290 not kept; gradients that a cache would hold, read once right behind, are even: 64 + 2
// experts of 768 x 512, 1000 tokens, 204 / 205, 12000 506 / 505).  With 8 groups or more a
// group's tiles are launched on one XCD (workgroup id % 8), so its rows are fetched into one L2.
#include "common.h"

#include <type_traits>

namespace occult {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct WgradArgs {
  const void* A;             // [rows][lda]: its columns index the output rows (M of them)
  int lda, a_col0, a_group_cols;   // group g reads columns a_col0 + g * a_group_cols ...
  const void* B;             // [rows][ldb]: its columns index the output columns (N of them)
  int ldb, b_col0, b_group_cols;
  const int32_t* b_rows;     // [rows] source row in B of each logical row, or NULL (identity)
  float* C;                  // [matrix][M][ldc]
  long long c_mat_stride;
  int ldc;
  const int32_t* grp_offset; // [ngroups+1] logical-row range per group, or NULL: every group takes rows [0, R)
  const int32_t* grp_widx;   // [ngroups] output matrix of each group, or NULL: w_base + group
  int w_base, ngroups, R;
  int M, N;
  int accumulate;            // 0: C = product, 1: C += product
  int rsplit;                // uniform groups only (grp_offset == NULL): the R rows are cut into rsplit slices of
                             // rslice rows (a multiple of the step), each a workgroup of its own that writes its f32
                             // partial product to ws[slice][group][M][N]; wgrad_reduce adds the slices in order.
                             // 0 or 1: no split
  int rslice;
  float* ws;
};

// ------------------------------------------------------------------------------------------
// The MFMA operands want 8 consecutive contracted elements per lane, which in memory are 8
// different rows.  A first version staged the operands through registers (16-byte loads of 4 rows,
// a 4 x 8 transpose with v_perm_b32, 8-byte LDS writes): it can keep only one step of operands
// (64 KiB per CU) in flight, which covers a step's products but not the latency of memory under
// load (measured: products alone 985 TFLOP/s, with the loads 480).  Here a step is 32 rows, the raw
// row-major tiles go from global memory straight into a ring of NST LDS stages
// (global_load_lds_dwordx4: no registers held while a load is in flight), NST steps ahead, and
// the transposition happens in the fragment reads: ds_read_b64_tr_b16 gives every lane
// of a 16-lane block the 4 contracted elements of its own column out of 4 rows x 16 columns that the
// block's lanes address (lanes 4e..4e+3 address row e).  Two such reads make one MFMA operand.
// One load instruction fills 1 KiB = 2 tile rows; 16-byte chunk c of tile row k sits at chunk
// c ^ ((k & 3) << 2) ^ ((k >> 3 & 1) << 1) (realised by the loading lane's choice of source chunk), so that
// the 2 x 4 rows x 32 bytes which two of a read's blocks address fall on different banks.  Rows past the
// group's end: the A side reads a page of zeros, the B side repeats the group's last row (0 * finite = 0).
// Gathered row indices take the same road two steps ahead of the rows they address: one 4-byte-per-lane
// LDS-directed load per wave and step into a small ring, read back with ordinary LDS reads.  Every step issues
// the same number of loads (steps past the end are clamped like rows past the end), so one
// constant vmcnt tells that the next step's tiles, and the indices about to be used, have landed.
//
// A step's fragments are read into registers under the products of the step before (two register sets), so a stage is
// free again one step earlier: four steps are in flight, and the LDS pipe (a step's 128 transposing reads at 64 B/clk
// and 32 KiB of writes, about 1130 cycles per CU) and the matrix pipe (1024) can work side by side.  Before, a
// step read its first fragments behind its barrier with nothing to multiply, and 32x32x16 products drew more power
// (ffn.hip).  Training step of 16384 tokens (64 experts, d = 2048, f = 1024) about 115 us less of 6000.
constexpr int kStreaming = 2;   // cache policy of a buffer store: not to be kept
namespace wgd {
constexpr int BM = 256, BN = 256, BK = 32;
constexpr int NST = 4;   // the index ring below assumes 4
constexpr int OP_BYTES = BK * 512;          // raw operand tile: 32 rows x 256 columns of bf16
constexpr int STAGE_BYTES = 2 * OP_BYTES;   // 32 KiB

__device__ __attribute__((aligned(16))) const unsigned zero_page[4] = {0u, 0u, 0u, 0u};

// acc (16 output rows x 16 columns) += A block^T * B block over 32 rows; assembly for the reason given in ffn.hip: the
// compiler, given the builtin, moves the 64 accumulator quads between the register files
__device__ __forceinline__ void mfma16(f32x4& acc, const bf16x8& b, const bf16x8& a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// GATHER: the first problem's B rows through b_rows.  TWO: workgroups [0, second_blocks) work on `second` (uniform groups, no
// gather), the rest on `first` (the shared experts' product alone had a few dozen workgroups: 6000 tokens of 64 + 2 experts
// 1290 -> 1267 us for the three products, 4000 of 60 + 4 1063 -> 882 together with the epilogue's stores below).
template <bool GATHER, bool TWO>
__global__ __launch_bounds__(256) void wgrad_bf16(const WgradArgs first, const WgradArgs second, const int second_blocks) {
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE_BYTES];
  __shared__ __attribute__((aligned(256))) int s_idx[4][4][64];   // [wave][step % 4][row of the wave's 8, repeated]
  const bool is_second = TWO && (int)blockIdx.x < second_blocks;   // uniform
  const WgradArgs& a = is_second ? second : first;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int nt_n = (a.N + BN - 1) / BN;
  const int tiles = ((a.M + BM - 1) / BM) * nt_n;
  // with 8 groups or more a group's tiles share an XCD (and its L2); fewer groups (shared experts: few
  // groups of many rows) are spread over all XCDs instead
  int group, tile, slice = 0;
  const int b = is_second ? (int)blockIdx.x : (int)blockIdx.x - second_blocks;
  if (!is_second && a.ngroups >= 8) {   // (host: second_blocks is a multiple of 8)
    const int xcd = b & 7, slot = b >> 3;
    group = (slot / tiles) * 8 + xcd;
    tile = slot % tiles;
  } else {
    const int per_slice = a.ngroups * tiles;
    const int bid = b % per_slice;
    slice = __builtin_amdgcn_readfirstlane(b / per_slice);   // 0 unless the rows are split
    if (slice >= max(1, a.rsplit)) return;   // whole block: the grid is padded to whole sets of XCDs
    group = bid / tiles;
    tile = bid % tiles;
  }
  if (group >= a.ngroups) return;   // whole block; before any barrier
  const bool split = a.rsplit > 1;
  // (the division runs in vector registers; the tile origin feeds scalar operands of the loads below)
  const int m0 = __builtin_amdgcn_readfirstlane((tile / nt_n) * BM), n0 = __builtin_amdgcn_readfirstlane((tile % nt_n) * BN);
  int r0 = 0, r1 = a.R;
  if (a.grp_offset) {
    r0 = a.grp_offset[group];
    r1 = a.grp_offset[group + 1];
  } else if (split) {
    r0 = min(a.R, slice * a.rslice);
    r1 = min(a.R, r0 + a.rslice);
  }
  r0 = __builtin_amdgcn_readfirstlane(r0);
  r1 = __builtin_amdgcn_readfirstlane(r1);
  const long long widx = a.grp_widx ? a.grp_widx[group] : (a.w_base + group);
  const int nk = (r1 - r0 + BK - 1) / BK;

  f32x4 acc[8][8];   // [output-row block][output-column block] of 16 x 16
#pragma unroll
  for (int mi = 0; mi < 8; ++mi)
#pragma unroll
    for (int ni = 0; ni < 8; ++ni) {
      acc[mi][ni] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      asm volatile("" : "+a"(acc[mi][ni]));   // cleared here, long before the first product reads it
    }

  if (nk > 0) {
    // loader role: a load instruction covers tile rows kb, kb + 1; lane = (row rr, chunk position p)
    const int rr = lane >> 5, p = lane & 31;
    const char* a_cols = static_cast<const char*>(a.A) + (long long)(a.a_col0 + group * a.a_group_cols + m0) * 2;
    const char* b_cols = static_cast<const char*>(a.B) + (long long)(a.b_col0 + group * a.b_group_cols + n0) * 2;
    const long long a_pitch = (long long)a.lda * 2, b_pitch = (long long)a.ldb * 2;
    const int a_chunks = min(32, (a.M - m0) / 8), b_chunks = min(32, (a.N - n0) / 8);   // valid 16-byte chunks per row
    const unsigned smem_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;   // LDS byte address
    const char* zeros = reinterpret_cast<const char*>(zero_page);

    // per-lane byte offsets of the 4 loads per operand inside a step's 32 rows: constant over the steps
    unsigned off_a[4], off_b[4], chunk_b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = wave * 8 + i * 2 + rr;           // tile row of this lane
      int ca = p ^ ((k & 3) << 2) ^ (((k >> 3) & 1) << 1), cb = ca;   // source chunk of this lane's position
      if (ca >= a_chunks) ca = 0;                     // columns past M or N: any valid chunk (never stored)
      if (cb >= b_chunks) cb = 0;
      off_a[i] = (unsigned)(k * a_pitch + ca * 16);
      off_b[i] = (unsigned)(k * b_pitch + cb * 16);
      chunk_b[i] = (unsigned)(cb * 16);
    }
    // the same for a step holding the group's last rows, or past them (issued to keep the load count constant)
    auto issue_tail = [&](int s) {
      const unsigned st = smem_base + (unsigned)(s % NST) * STAGE_BYTES;
      const int row0 = r0 + s * BK;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int kb = wave * 8 + i * 2;               // tile rows kb, kb + 1
        const long long ra = row0 + kb + rr;
        // A: rows past the end read zeros
        const char* src_a = (ra < r1) ? a_cols + ra * a_pitch + (off_a[i] - (unsigned)((kb + rr) * a_pitch)) : zeros;
        load_to_lds_16(src_a, st + (unsigned)kb * 512u);
        // B: rows past the end repeat the last row (the fetched indices are clamped the same way)
        long long rb = min(row0 + kb + rr, r1 - 1);
        if (GATHER && !is_second) rb = s_idx[wave][s & 3][i * 2 + rr];
        load_to_lds_16(b_cols + rb * b_pitch + chunk_b[i], st + (unsigned)OP_BYTES + (unsigned)kb * 512u);
      }
    };
    auto issue = [&](int s) {   // the 8 loads of this wave for step s into stage s % NST
      const unsigned st = smem_base + (unsigned)(s % NST) * STAGE_BYTES;
      const int row0 = r0 + s * BK;                    // first row of the step
      if (row0 + BK <= r1) {   // block-uniform: every row inside the group, addresses = uniform base + constant offsets
        const char* a_step = a_cols + (long long)row0 * a_pitch;
        const char* b_step = b_cols + (long long)row0 * b_pitch;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned kb = (unsigned)(wave * 8 + i * 2);
          load_to_lds_16(a_step, off_a[i], st + kb * 512u);
          if (GATHER) {
            const long long rb = is_second ? row0 + (int)kb + rr : s_idx[wave][s & 3][i * 2 + rr];   // fetched two steps ago
            load_to_lds_16(b_cols + rb * b_pitch + chunk_b[i], st + (unsigned)OP_BYTES + kb * 512u);
          } else {
            load_to_lds_16(b_step, off_b[i], st + (unsigned)OP_BYTES + kb * 512u);
          }
        }
      } else {
        issue_tail(s);
      }
    };

    // fragment reads: lane l = 16 b + j, j = 4 e + q: block b covers rows 8 b + e (first read), + 4 (second read) of 16
    // columns; the lane addresses 4 columns (8 bytes) of row e
    const int fb = lane >> 4, fe = (lane >> 2) & 3, fq = lane & 3;
    typedef __attribute__((address_space(3))) char lds_char;
    const int f_sw = (fe << 2) ^ ((fb & 1) << 1);
    int f_off[8];   // byte offset of 16-column block i (0..7) of a wave tile
#pragma unroll
    for (int i = 0; i < 8; ++i) f_off[i] = (8 * fb + fe) * 512 + (((2 * i + (fq >> 1)) ^ f_sw) * 16) + (fq & 1) * 8;
    bf16x8 fa[2][8], fbv[2][8];
    auto frag = [&](const lds_char* op, int i) -> bf16x8 {
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(op + f_off[i]));
      const bf16x4 hi =
          __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(op + f_off[i] + 4 * 512));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    // fragment r (0..15) of step s, in the order in which the products want them: the first block of A, the blocks of B,
    // the other blocks of A
    auto read_frag = [&](int set, int s, int r) {
      const lds_char* st = (const lds_char*)smem + (s % NST) * STAGE_BYTES;
      if (r >= 1 && r <= 8) fbv[set][r - 1] = frag(st + OP_BYTES + wn * 256, r - 1);
      else fa[set][r == 0 ? 0 : r - 8] = frag(st + wm * 256, r == 0 ? 0 : r - 8);
    };

    // source rows of this wave's 8 tile rows of step s (clamped to the group) -> its ring slot s % 4
    const unsigned idx_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)&s_idx[wave][0][0];
    auto issue_idx = [&](int s) {
      const int r = min(r0 + s * BK + wave * 8 + (lane & 7), r1 - 1);
      // (the second problem's rows are their own: a load that nobody reads keeps the count)
      load_to_lds_4(is_second ? zeros : reinterpret_cast<const char*>(a.b_rows + r), idx_base + (unsigned)(s & 3) * 256u);
    };
    constexpr int OPS = GATHER ? 9 : 8;   // loads per wave and step
    if (GATHER) {
#pragma unroll
      for (int s = 0; s < 4; ++s) issue_idx(s);          // one ring of indices
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // a wave reads only its own indices: no barrier
    }
    // Loads complete in order.  Per step a wave issues [indices of step s + 6,] 8 tile loads of step s + 4.  At the start
    // of step s the tiles of step s + 1 and the indices of step s + 4 have to have landed: behind them stand the tiles of
    // steps s + 2 and s + 3 and the indices of step s + 5.  The prologue issues in the order the loop continues; an index
    // slot is refilled once it has been read (the tile loads' addresses depend on the reads).
    issue(0);
    issue(1);
    if (GATHER) issue_idx(4);
    issue(2);
    if (GATHER) issue_idx(5);
    issue(3);
    wait_loads_and_barrier<3 * OPS - (GATHER ? 1 : 0)>();   // tiles of step 0
#pragma unroll
    for (int r = 0; r < 16; ++r) read_frag(0, 0, r);
    // One step: 16 groups of {4 products, fragment reads of the next step, a tile load}, pinned in source order (one wave
    // per SIMD: nothing else hides an instruction clump).  After its barrier the tiles of step s + 1 are in LDS, and every
    // wave has the fragments of step s in registers, so that step s + 4 may overwrite its stage.
    // full: all rows of step s + 4 lie inside the group
    auto step = [&](int set, int s, auto full) {
      wait_loads_and_barrier<2 * OPS - (GATHER ? 1 : 0)>();
      const int sn = s + NST;
      if (GATHER) issue_idx(s + NST + 2);
      const unsigned st = smem_base + (unsigned)(s % NST) * STAGE_BYTES + wave * 4096u;
      const char* a_step = a_cols + (long long)(r0 + sn * BK) * a_pitch;
      const char* b_step = b_cols + (long long)(r0 + sn * BK) * b_pitch;
      int rb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        rb[i] = GATHER ? s_idx[wave][sn & 3][i * 2 + rr] : 0;   // fetched two steps ago
        if (GATHER && is_second) rb[i] = min(r0 + sn * BK + wave * 8 + i * 2 + rr, r1 - 1);
      }
      auto tile_load = [&](int i) {   // 0..3: A, 4..7: B
        const int j = i & 3, row = r0 + sn * BK + wave * 8 + j * 2 + rr;
        const unsigned dst = st + (unsigned)j * 1024u;
        if (i < 4) {
          if constexpr (decltype(full)::value) load_to_lds_16(a_step, off_a[j], dst);
          else load_to_lds_16(row < r1 ? a_step + off_a[j] : zeros, dst);
        } else if (GATHER) {
          asm volatile("" : "+v"(rb[j]));   // nothing of the address is computed, and so waited for, before this place
          load_to_lds_16(b_cols + (long long)rb[j] * b_pitch + chunk_b[j], dst + (unsigned)OP_BYTES);
        } else {
          if constexpr (decltype(full)::value) load_to_lds_16(b_step, off_b[j], dst + (unsigned)OP_BYTES);
          else load_to_lds_16(b_cols + (long long)min(row, r1 - 1) * b_pitch + chunk_b[j], dst + (unsigned)OP_BYTES);
        }
      };
#pragma unroll
      for (int g = 0; g < 16; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int t = 4 * g + q, mi = t >> 3, ni = t & 7;
          mfma16(acc[mi][ni], fbv[set][ni], fa[set][mi]);
          if (q == 0 && (g & 1) == 0) tile_load(g / 2);
          if (q == 1 && g < 12) read_frag(set ^ 1, s + 1, g < 4 ? 2 * g : g + 4);
          if (q == 2 && g < 4) read_frag(set ^ 1, s + 1, 2 * g + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
    };
    // two loops, so that the first has no clamping: pairs of steps whose prefetched steps lie wholly inside the group
    const int n_main = max(0, (r1 - r0) / BK - NST) & ~1;
    int s = 0;
    for (; s < n_main; s += 2) {
      step(0, s, std::true_type{});
      step(1, s + 1, std::true_type{});
    }
    // then the steps that prefetch the group's last rows or past them
    for (; s < nk; s += 2) {
      step(0, s, std::false_type{});
      if (s + 1 >= nk) break;   // block-uniform
      step(1, s + 1, std::false_type{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the clamped loads past the end, before the block's LDS is released
  }

  // accumulator element e of lane l: output row l % 16, column (l / 16) * 4 + e of its 16 x 16 tile (the operands are
  // swapped).  16 rows of the wave tile at a time go through LDS, 16-byte chunk c of row r at c ^ r, and leave as two
  // whole rows of 512 bytes per store.
  // Stores (and, when accumulating, loads) go through a buffer descriptor over the wave tile's valid rows: rows
  // past M lie beyond its range and are dropped by the hardware, columns past N are sent there: no branches.
  const int rows_left = min(a.M - (m0 + wm * 128), 128);
  const int cols_left = min(a.N - (n0 + wn * 128), 128);
  // a row slice writes its partial product densely into the scratch tensor [slice][group][M][N] instead
  const int ldc = split ? a.N : a.ldc;
  const bool accumulate = !split && a.accumulate;
  float* c_mat = split ? a.ws + ((long long)slice * a.ngroups + group) * ((long long)a.M * a.N) : a.C + widx * a.c_mat_stride;
  const unsigned n_rec = rows_left > 0 && cols_left > 0 ? (unsigned)((rows_left - 1) * ldc + cols_left) * 4u : 0u;
  const unsigned long long c_tile = reinterpret_cast<unsigned long long>(
      c_mat + (long long)(m0 + wm * 128) * ldc + n0 + wn * 128);
  const unsigned long long c_tile_u =   // the descriptor has to sit in scalar registers
      ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(c_tile >> 32)) << 32) |
      (unsigned)__builtin_amdgcn_readfirstlane((unsigned)c_tile);
  const __amdgpu_buffer_rsrc_t c_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<void*>(c_tile_u), 0, __builtin_amdgcn_readfirstlane((int)n_rec), 0x00020000);
  // wait states of the last products' results (the compiler does not see that they are matrix instructions)
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  __syncthreads();   // every wave is past its last reads: the stages are free
  const int w_row = lane & 15, w_q = lane >> 4, o_row = lane >> 5, o_chunk = lane & 31;
  const bool col_ok = o_chunk * 4 < cols_left;   // N % 8 == 0 (host): four columns are inside together
#pragma unroll
  for (int mi = 0; mi < 8; ++mi) {
#pragma unroll
    for (int ni = 0; ni < 8; ++ni) asm volatile("" : "+a"(acc[mi][ni]));   // read from here on, not all of them at once
    char* buf = smem + wave * 16384 + (mi & 1) * 8192;
#pragma unroll
    for (int ni = 0; ni < 8; ++ni)
      *reinterpret_cast<f32x4*>(buf + w_row * 512 + ((ni * 4 + w_q) ^ w_row) * 16) = acc[mi][ni];
    wave_lds_order();   // (and the other half's reads before its next writes)
    f32x4 v[8];
    unsigned off[8];
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int r = it * 2 + o_row;
      v[it] = *reinterpret_cast<const f32x4*>(buf + r * 512 + (o_chunk ^ r) * 16);
      off[it] = col_ok ? (unsigned)((mi * 16 + r) * ldc + o_chunk * 4) * 4u : n_rec;
    }
    if (accumulate) {   // block-uniform; the 8 loads of a row block are in flight together
      u32x4 old[8];
#pragma unroll
      for (int it = 0; it < 8; ++it) old[it] = __builtin_amdgcn_raw_buffer_load_b128(c_rsrc, (int)off[it], 0, 0);
#pragma unroll
      for (int it = 0; it < 8; ++it) v[it] += __builtin_bit_cast(f32x4, old[it]);
    }
#pragma unroll
    for (int it = 0; it < 8; ++it)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[it]), c_rsrc, (int)off[it], 0, kStreaming);
  }
}
}  // namespace wgd

// ------------------------------------------------------------------------------------------
// Groups of a few hundred rows and fewer (small micro-batches): a product is then little more than writing its f32 outputs,
// and one block per CU does that with nothing beside it: a tile's first loads, its few steps and its stores stand in a row.
// Here a block takes 128 x 128 outputs (wave tile 64 x 64 = 4 x 4 MFMA tiles) and three blocks share a CU, one storing while the
// others load and multiply.  More operand bytes and LDS reads per product than the 256 x 256 tiles: from a few hundred rows
// those win (launch_wgrad_pair).  Bound by the stores: 1000 tokens of 64 + 2 experts, d = 2048, f = 1408, 694 -> 399 us for
// the three products = 5.7 TB/s of their 2.28 GB.  How the outputs are stored is half of that: in 64-byte pieces 800 us, marked
// as not to be kept 583 (the operands stay in L2, but with few rows 420 -> 690: half lines leave the cache), as whole rows
// through LDS and not to be kept 399 (388 with few rows).
// The routed experts' groups (`first`) and the shared experts' (`second`, uniform groups over all tokens) are one launch:
// alone the shared ones are a few dozen blocks.  They come first in the grid, since each of them runs longest.
// Staging, swizzle, transposing reads and the order of the sums are those of the kernel above; a step's fragments are read
// at its start (another block's products fill the gap) and the row indices of 1024 rows at a time are kept in LDS.
namespace wgs {
constexpr int BM = 128, BN = 128, BK = 32;
constexpr int NST = 3;
constexpr int OP_BYTES = BK * 256;          // raw operand tile: 32 rows x 128 columns of bf16
constexpr int STAGE_BYTES = 2 * OP_BYTES;   // 16 KiB
constexpr int IDX_ROWS = 1024;              // a multiple of BK
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256, 3) void wgrad_bf16(const WgradArgs first, const WgradArgs second, const int second_blocks) {
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE_BYTES];
  __shared__ int s_idx[IDX_ROWS];
  const bool is_second = (int)blockIdx.x < second_blocks;   // uniform
  const WgradArgs& a = is_second ? second : first;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int nt_n = (a.N + BN - 1) / BN;
  const int tiles = ((a.M + BM - 1) / BM) * nt_n;
  int group, tile;
  if (!is_second && a.ngroups >= 8) {   // a group's tiles share an XCD (second_blocks is a multiple of 8)
    const int b = (int)blockIdx.x - second_blocks, slot = b >> 3;
    group = (slot / tiles) * 8 + (b & 7);
    tile = slot % tiles;
  } else {
    const int b = is_second ? (int)blockIdx.x : (int)blockIdx.x - second_blocks;
    group = b / tiles;
    tile = b % tiles;
  }
  if (group >= a.ngroups) return;   // whole block; before any barrier
  const int m0 = __builtin_amdgcn_readfirstlane((tile / nt_n) * BM), n0 = __builtin_amdgcn_readfirstlane((tile % nt_n) * BN);
  int r0 = 0, r1 = a.R;
  if (a.grp_offset) {
    r0 = a.grp_offset[group];
    r1 = a.grp_offset[group + 1];
  }
  r0 = __builtin_amdgcn_readfirstlane(r0);
  r1 = __builtin_amdgcn_readfirstlane(r1);
  const long long widx = a.grp_widx ? a.grp_widx[group] : (a.w_base + group);
  const int nk = (r1 - r0 + BK - 1) / BK;
  const bool gather = a.b_rows != nullptr;   // uniform

  f32x4 acc[4][4];   // [output-row block][output-column block] of 16 x 16
#pragma unroll
  for (int mi = 0; mi < 4; ++mi)
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  if (nk > 0) {
    // loader role: load i (0, 1) of a wave covers tile rows wave*8 + i*4 .. +3; lane = (row rr, chunk position p)
    const int rr = lane >> 4, p = lane & 15;
    const char* a_cols = static_cast<const char*>(a.A) + (long long)(a.a_col0 + group * a.a_group_cols + m0) * 2;
    const char* b_cols = static_cast<const char*>(a.B) + (long long)(a.b_col0 + group * a.b_group_cols + n0) * 2;
    const long long a_pitch = (long long)a.lda * 2, b_pitch = (long long)a.ldb * 2;
    const int a_chunks = min(16, (a.M - m0) / 8), b_chunks = min(16, (a.N - n0) / 8);   // valid 16-byte chunks per row
    const int c_src = p ^ (rr << 2) ^ ((wave & 1) << 1);
    const int chunk_a = (c_src < a_chunks ? c_src : 0) * 16, chunk_b = (c_src < b_chunks ? c_src : 0) * 16;   // columns past M
    // or N: any valid chunk (never stored)
    const unsigned lds_w = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem + (unsigned)wave * 2048u;
    const char* zeros = reinterpret_cast<const char*>(wgd::zero_page);
    auto fetch_idx = [&](int from) {   // source rows of the group's rows from, from + 1, ...
      for (int i = tid; i < IDX_ROWS && r0 + from + i < r1; i += 256) s_idx[i] = a.b_rows[r0 + from + i];
    };
    auto issue = [&](int s) {   // this wave's 4 loads of step s; steps past the end too, so that the count stays constant
      const unsigned st = lds_w + (unsigned)(s % NST) * STAGE_BYTES;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = r0 + s * BK + wave * 8 + i * 4 + rr;
        load_to_lds_16(row < r1 ? a_cols + row * a_pitch + chunk_a : zeros, st + (unsigned)i * 1024u);   // past the end: zeros
        const int rb = min(row, r1 - 1);                                                                // the last row again
        const long long src = gather ? s_idx[(rb - r0) % IDX_ROWS] : rb;
        load_to_lds_16(b_cols + src * b_pitch + chunk_b, st + (unsigned)OP_BYTES + (unsigned)i * 1024u);
      }
    };
    // fragment reads: lane l = 16 b + j, j = 4 e + q, as in the kernel above
    const int fb = lane >> 4, fe = (lane >> 2) & 3, fq = lane & 3;
    typedef __attribute__((address_space(3))) char lds_char;
    const int f_sw = (fe << 2) ^ ((fb & 1) << 1), f_row = (8 * fb + fe) * 256 + (fq & 1) * 8;
    int a_off[4], b_off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a_off[i] = f_row + ((wm * 8 + 2 * i + (fq >> 1)) ^ f_sw) * 16;
      b_off[i] = f_row + ((wn * 8 + 2 * i + (fq >> 1)) ^ f_sw) * 16 + OP_BYTES;
    }
    auto frag = [&](const lds_char* at) -> bf16x8 {
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)at);
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(at + 4 * 256));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    if (gather) {
      fetch_idx(0);
      __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) issue(s);
    for (int s = 0; s < nk; ++s) {
      // the tiles of step s have landed for every wave, and every wave has read those of step s - 1, whose stage is free
      if (s == 0) {
        wait_loads_and_barrier<4 * (NST - 1)>();
      } else {
        wait_loads_and_barrier<4 * (NST - 2)>();
        const int next = s + NST - 1;
        if (gather && next * BK % IDX_ROWS == 0) {   // uniform; the indices of all steps before have been read
          fetch_idx(next * BK);
          __syncthreads();
        }
        issue(next);
      }
      const lds_char* st = (const lds_char*)smem + (s % NST) * STAGE_BYTES;
      bf16x8 fa[4], fbv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) fbv[i] = frag(st + b_off[i]);
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[i] = frag(st + a_off[i]);
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fbv[ni], fa[mi], acc[mi][ni], 0, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the loads of steps past the end, before the block's LDS is released
  }

  // Outputs leave as whole rows of the wave tile: element e of a lane is output row l % 16, column (l / 16) * 4 + e of its
  // 16 x 16 tile, and 16 rows x 64 columns at a time go through LDS (the stages are free: every wave is past its last read),
  // 16-byte chunk c of row r at c ^ r.  Rows past M lie beyond the descriptor's range and are dropped, columns past N are
  // sent there.
  const int rows_left = min(a.M - (m0 + wm * 64), 64);
  const int cols_left = min(a.N - (n0 + wn * 64), 64);
  const unsigned n_rec = rows_left > 0 && cols_left > 0 ? (unsigned)((rows_left - 1) * a.ldc + cols_left) * 4u : 0u;
  const unsigned long long c_tile = reinterpret_cast<unsigned long long>(
      a.C + widx * a.c_mat_stride + (long long)(m0 + wm * 64) * a.ldc + n0 + wn * 64);
  const unsigned long long c_tile_u =   // the descriptor has to sit in scalar registers
      ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned)(c_tile >> 32)) << 32) |
      (unsigned)__builtin_amdgcn_readfirstlane((unsigned)c_tile);
  const __amdgpu_buffer_rsrc_t c_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<void*>(c_tile_u), 0, __builtin_amdgcn_readfirstlane((int)n_rec), 0x00020000);
  __syncthreads();
  const int w_row = lane & 15, w_q = lane >> 4, o_row = lane >> 4, o_chunk = lane & 15;
  const bool col_ok = o_chunk * 4 < cols_left;   // N % 8 == 0 (host): four columns are inside together
#pragma unroll
  for (int mi = 0; mi < 4; ++mi) {
    char* buf = smem + wave * 8192 + (mi & 1) * 4096;
#pragma unroll
    for (int ni = 0; ni < 4; ++ni)
      *reinterpret_cast<f32x4*>(buf + w_row * 256 + ((ni * 4 + w_q) ^ w_row) * 16) = acc[mi][ni];
    wave_lds_order();   // (and the other half's reads before its next writes)
    f32x4 v[4];
    unsigned off[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int r = it * 4 + o_row;
      v[it] = *reinterpret_cast<const f32x4*>(buf + r * 256 + (o_chunk ^ r) * 16);
      off[it] = col_ok ? (unsigned)((mi * 16 + r) * a.ldc + o_chunk * 4) * 4u : n_rec;
    }
    if (a.accumulate) {   // block-uniform
      u32x4 old[4];
#pragma unroll
      for (int it = 0; it < 4; ++it) old[it] = __builtin_amdgcn_raw_buffer_load_b128(c_rsrc, (int)off[it], 0, 0);
#pragma unroll
      for (int it = 0; it < 4; ++it) v[it] += __builtin_bit_cast(f32x4, old[it]);
    }
#pragma unroll
    for (int it = 0; it < 4; ++it)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[it]), c_rsrc, (int)off[it], 0, kStreaming);
  }
}
}  // namespace wgs

// Adds the row slices' partial products in slice order and writes (or adds) the sum: C[group] (=|+=) ws[0][group]
// + ws[1][group] + ...  One thread per 4 output columns (host: N % 4 == 0, ldc % 4 == 0, 16-byte aligned bases).
__global__ __launch_bounds__(256) void wgrad_reduce(const WgradArgs a) {
  const long long quads_per_mat = (long long)a.M * (a.N / 4);
  const long long total = quads_per_mat * a.ngroups;
  const long long slice_stride = (long long)a.ngroups * a.M * a.N;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    const int group = (int)(i / quads_per_mat);
    const long long q = i - group * quads_per_mat;
    const int m = (int)(q / (a.N / 4)), n = (int)(q - (long long)m * (a.N / 4)) * 4;
    const float* src = a.ws + (long long)group * a.M * a.N + (long long)m * a.N + n;
    f32x4 sum = *reinterpret_cast<const f32x4*>(src);
    for (int sl = 1; sl < a.rsplit; ++sl) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + sl * slice_stride);
      sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
    }
    const long long widx = a.grp_widx ? a.grp_widx[group] : (a.w_base + group);
    f32x4* dst = reinterpret_cast<f32x4*>(a.C + widx * a.c_mat_stride + (long long)m * a.ldc + n);
    if (a.accumulate) {
      const f32x4 old = *dst;
      sum.x += old.x; sum.y += old.y; sum.z += old.z; sum.w += old.w;
    }
    *dst = sum;
  }
}

// f32 path for parity-sized layers: one thread per output element, rows summed in order
__global__ __launch_bounds__(256) void wgrad_f32(const WgradArgs a) {
  const int group = blockIdx.z;
  const int m = blockIdx.y * 16 + (threadIdx.x >> 4), n = blockIdx.x * 16 + (threadIdx.x & 15);
  if (m >= a.M || n >= a.N) return;
  int r0 = 0, r1 = a.R;
  if (a.grp_offset) {
    r0 = a.grp_offset[group];
    r1 = a.grp_offset[group + 1];
  }
  const long long widx = a.grp_widx ? a.grp_widx[group] : (a.w_base + group);
  const float* A = static_cast<const float*>(a.A) + a.a_col0 + group * a.a_group_cols + m;
  const float* B = static_cast<const float*>(a.B) + a.b_col0 + group * a.b_group_cols + n;
  float sum = 0.0f;
  for (int r = r0; r < r1; ++r) {
    const long long src = a.b_rows ? a.b_rows[r] : r;
    sum = fmaf(A[(long long)r * a.lda], B[src * a.ldb], sum);
  }
  float* p = a.C + widx * a.c_mat_stride + (long long)m * a.ldc + n;
  *p = a.accumulate ? *p + sum : sum;
}

// Row slices for a product with fewer than 8 uniform groups of many rows (shared experts of a large batch): its
// groups x tiles workgroups alone leave most of the chip idle.  Returns the number of slices (1 = no split) that
// minimises rounds of workgroups x rows per slice, at most 8, each of at least 2048 rows; *rslice = rows per slice.
// That is the price of the product in a launch of its own.  Beside the routed experts', where it runs, a split is still
// worth its partial sums and its second launch in narrow layers (us for the three products, split / not: 64 + 2 experts of 512 x 384,
// 4096 tokens 158 / 262, 16384 476 / 1005; 1024 x 704, 8192 474 / 588), and costs 6 % in wide ones (2048 x 1408, 4096 1133 / 1065, 16384 3218 /
// 2979) and up to a third with few experts (8 + 1, 8192 794 / 584).
static int choose_row_split(const occult_cfg_t& c, int ngroups, int M, int N, int R, int* rslice) {
  *rslice = R;
  if (c.dtype != OCCULT_BF16 || ngroups <= 0 || ngroups >= 8 || N % 4 != 0) return 1;
  static int cached_cus = 0;   // compute units of the device first asked about (one kind of GPU per process)
  if (cached_cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cached_cus = n;
    else
      cached_cus = 256;
  }
  const int cus = cached_cus;
  const long long tiles = (long long)((M + wgd::BM - 1) / wgd::BM) * ((N + wgd::BN - 1) / wgd::BN) * ngroups;
  int best = 1;
  double best_cost = (double)((tiles + cus - 1) / cus) * R;
  for (int r = 2; r <= 8; ++r) {
    const int rows = ((R + r - 1) / r + wgd::BK - 1) / wgd::BK * wgd::BK;
    if (rows < 2048) break;
    const double cost = (double)((tiles * r + cus - 1) / cus) * rows;
    if (cost < best_cost * 0.95) {
      best = r;
      best_cost = cost;
      *rslice = rows;
    }
  }
  return best;
}

// The routed experts' product and, unless b is NULL, the shared experts' (same M and N), which come first in the grid: their
// workgroups run longest.
// 128 x 128 tiles for fewer than 240 rows per group, shared ones included and their rows not split, where the products are mostly stores (us for the
// three, d = 2048, 128 / 256 tiles: 64 + 2 experts of f = 1408, 91 rows 388 / 441, 182 473 / 530, 242 624 / 595, 303 841 / 724;
// 64 of f = 1024, 125 rows 274 / 357, 250 387 / 419, 312 495 / 464; 60 + 4, 250 538 / 588, 375 873 / 767), and where the
// larger tiles would leave half of the CUs without one (4 + 1 experts, d = 256, f = 192, 420 rows: 38 / 66).
constexpr int kSmallRows = 240, kFewTiles = 128;
static int launch_wgrad_pair(const occult_cfg_t& c, const WgradArgs& a, const WgradArgs* b, hipStream_t s) {
  if (a.M == 0 || a.N == 0) return OCCULT_OK;
  if (c.dtype == OCCULT_BF16) {
    const bool split = b != nullptr && b->rsplit > 1;
    const long long groups = c.E + c.S;
    const bool small_groups = !split && ((long long)c.T * (c.k + c.S) < kSmallRows * groups ||
                                         groups * ((a.M + wgd::BM - 1) / wgd::BM) * ((a.N + wgd::BN - 1) / wgd::BN) < kFewTiles);
    const int bm = small_groups ? wgs::BM : wgd::BM, bn = small_groups ? wgs::BN : wgd::BN;
    const long long tiles = (long long)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn);
    // whole sets of XCDs: the routed groups keep theirs
    const long long second = b ? (b->ngroups * tiles * (split ? b->rsplit : 1) + 7) / 8 * 8 : 0;
    const long long blocks = second + (a.ngroups >= 8 ? (a.ngroups + 7) / 8 * 8 : a.ngroups) * tiles;
    OCC_REQUIRE(blocks < (1ll << 31), OCCULT_EINVAL, "weight-gradient grid too large");
    const dim3 grid((unsigned)blocks), block(256);
    const WgradArgs& b2 = b ? *b : a;
    if (small_groups) hipLaunchKernelGGL(wgs::wgrad_bf16, grid, block, 0, s, a, b2, (int)second);
    else if (a.b_rows && b) hipLaunchKernelGGL((wgd::wgrad_bf16<true, true>), grid, block, 0, s, a, b2, (int)second);
    else if (a.b_rows) hipLaunchKernelGGL((wgd::wgrad_bf16<true, false>), grid, block, 0, s, a, b2, (int)second);
    else if (b) hipLaunchKernelGGL((wgd::wgrad_bf16<false, true>), grid, block, 0, s, a, b2, (int)second);
    else hipLaunchKernelGGL((wgd::wgrad_bf16<false, false>), grid, block, 0, s, a, b2, (int)second);
    if (split) {
      OCC_LAUNCH_CHECK("wgrad");
      hipLaunchKernelGGL(wgrad_reduce, dim3(2048), dim3(256), 0, s, *b);
    }
  } else {
    for (const WgradArgs* p : {&a, b}) {
      if (p == nullptr || p->ngroups == 0) continue;
      OCC_REQUIRE(p->ngroups <= 65535, OCCULT_EINVAL, "too many groups");
      hipLaunchKernelGGL(wgrad_f32, dim3((p->N + 15) / 16, (p->M + 15) / 16, p->ngroups), dim3(256), 0, s, *p);
    }
  }
  OCC_LAUNCH_CHECK("wgrad");
  return OCCULT_OK;
}

}  // namespace occult

using namespace occult;

// chooses the row split of a uniform-group product when the caller's scratch holds its partial sums
static void set_row_split(const occult_cfg_t& c, WgradArgs& a, void* ws, size_t ws_bytes) {
  a.rsplit = 0;
  if (!ws) return;
  int rslice = 0;
  const int r = choose_row_split(c, a.ngroups, a.M, a.N, a.R, &rslice);
  if (r > 1 && ws_bytes >= (size_t)r * a.ngroups * a.M * a.N * sizeof(float)) {
    a.rsplit = r;
    a.rslice = rslice;
    a.ws = static_cast<float*>(ws);
  }
}

// scratch for the row-split products of the shared experts: the largest of the three (they run one after another)
static size_t wgrad_ws_need(const occult_cfg_t& c) {
  if (c.S <= 0 || c.T <= 0) return 0;
  int rs = 0;
  const int r1 = choose_row_split(c, c.S, c.d, c.f, c.T, &rs);
  const int r2 = choose_row_split(c, c.S, c.f, c.d, c.T, &rs);
  const int r = r1 > r2 ? r1 : r2;
  return r > 1 ? (size_t)r * c.S * c.d * c.f * sizeof(float) : 0;
}

extern "C" int occult_expert_ffn_backward_weights_ws_bytes(const occult_cfg_t* cfg, size_t* ws_bytes) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  OCC_REQUIRE(ws_bytes, OCCULT_ENULLPTR, "ws_bytes is NULL");
  *ws_bytes = wgrad_ws_need(*cfg);
  return OCCULT_OK;
}

static int backward_weights_impl(const occult_cfg_t* cfg, const occult_plan_t* plan, const void* sfd_x,
                                 const void* x, const void* epd_h, const void* h_shared,
                                 const void* epd_dy, const void* dy, const void* epd_gu,
                                 const void* gu_shared, float* dw_gate, float* dw_up, float* dw_down,
                                 int accumulate, void* ws, size_t ws_bytes, occult_stream_t stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  OCC_REQUIRE(aligned16(ws), OCCULT_EALIGN, "ws is not 16-byte aligned");
  OCC_REQUIRE(dw_gate && dw_up && dw_down, OCCULT_ENULLPTR, "dw_gate, dw_up or dw_down is NULL");
  OCC_REQUIRE(accumulate == 0 || accumulate == 1, OCCULT_EINVAL, "accumulate=%d must be 0 or 1", accumulate);
  const int es = elem_size(c);
  OCC_REQUIRE(((size_t)c.d * es) % 16 == 0 && ((size_t)c.f * es) % 16 == 0, OCCULT_EALIGN,
              "rows of d=%d or f=%d elements are not multiples of 16 bytes", c.d, c.f);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const long long mat = (long long)c.f * c.d;
  OCC_REQUIRE(plan && plan->exp_offset && plan->pos_expert && plan->epd_sfd_row, OCCULT_ENULLPTR,
              "plan or one of its tables is NULL");
  if (c.T > 0) {   // with no rows nothing is read and the products below write zeros (or add nothing)
    OCC_REQUIRE(sfd_x && epd_h && epd_dy && epd_gu, OCCULT_ENULLPTR, "sfd_x, epd_h, epd_dy or epd_gu is NULL");
    if (c.S > 0)
      OCC_REQUIRE(x && h_shared && dy && gu_shared, OCCULT_ENULLPTR, "x, h_shared, dy or gu_shared is NULL with S=%d",
                  c.S);
  }
  OCC_REQUIRE(aligned16(sfd_x) && aligned16(x) && aligned16(epd_h) && aligned16(h_shared) && aligned16(epd_dy) &&
                  aligned16(dy) && aligned16(epd_gu) && aligned16(gu_shared),
              OCCULT_EALIGN, "a buffer is not 16-byte aligned");

  WgradArgs routed{};
  routed.grp_offset = plan->exp_offset; routed.grp_widx = plan->pos_expert; routed.ngroups = c.E;
  routed.accumulate = accumulate;
  WgradArgs shared{};
  shared.grp_offset = nullptr; shared.grp_widx = nullptr; shared.w_base = c.E; shared.ngroups = c.S; shared.R = c.T;
  shared.accumulate = accumulate;
  for (int product = 0; product < 3; ++product) {
    WgradArgs a = routed, b = shared;
    if (product == 0) {   // dW_down [d][f] = sum_r dy_r (x) h_r
      a.A = epd_dy; a.B = epd_h; a.ldb = c.f;
      b.A = dy; b.B = h_shared; b.ldb = c.S * c.f; b.b_group_cols = c.f;
      a.lda = b.lda = a.M = b.M = c.d;
      a.N = b.N = a.ldc = b.ldc = c.f;
      a.C = b.C = dw_down;
    } else {              // dW_gate, dW_up [f][d] = sum_r dg_r (x) x_r, sum_r du_r (x) x_r
      a.A = epd_gu; a.lda = 2 * c.f; a.B = sfd_x; a.b_rows = plan->epd_sfd_row;
      b.A = gu_shared; b.lda = c.S * 2 * c.f; b.a_group_cols = 2 * c.f; b.B = x;
      a.a_col0 = b.a_col0 = product == 2 ? c.f : 0;
      a.M = b.M = c.f;
      a.N = b.N = a.ldb = b.ldb = a.ldc = b.ldc = c.d;
      a.C = b.C = product == 2 ? dw_up : dw_gate;
    }
    a.c_mat_stride = b.c_mat_stride = mat;
    if (c.S > 0) set_row_split(c, b, ws, ws_bytes);
    rc = launch_wgrad_pair(c, a, c.S > 0 ? &b : nullptr, s);
    if (rc) return rc;
  }
  return OCCULT_OK;
}

extern "C" int occult_expert_ffn_backward_weights(const occult_cfg_t* cfg, const occult_plan_t* plan, const void* sfd_x,
                                                  const void* x, const void* epd_h, const void* h_shared,
                                                  const void* epd_dy, const void* dy, const void* epd_gu,
                                                  const void* gu_shared, float* dw_gate, float* dw_up, float* dw_down,
                                                  int accumulate, occult_stream_t stream) {
  return backward_weights_impl(cfg, plan, sfd_x, x, epd_h, h_shared, epd_dy, dy, epd_gu, gu_shared, dw_gate, dw_up, dw_down,
                               accumulate, nullptr, 0, stream);
}

extern "C" int occult_expert_ffn_backward_weights_ws(const occult_cfg_t* cfg, const occult_plan_t* plan, const void* sfd_x,
                                                     const void* x, const void* epd_h, const void* h_shared,
                                                     const void* epd_dy, const void* dy, const void* epd_gu,
                                                     const void* gu_shared, float* dw_gate, float* dw_up, float* dw_down,
                                                     int accumulate, void* ws, size_t ws_bytes, occult_stream_t stream) {
  return backward_weights_impl(cfg, plan, sfd_x, x, epd_h, h_shared, epd_dy, dy, epd_gu, gu_shared, dw_gate, dw_up, dw_down,
                               accumulate, ws, ws_bytes, stream);
}
