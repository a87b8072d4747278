// Grouped GEMM of the expert computation: argument block and launcher, shared by the forward
// (ffn.hip) and backward (ffn_backward.hip) translation units.  Not part of the public ABI.
#pragma once
#include "common.h"

namespace occult {

struct GemmArgs {
  const void* A;            // activation rows, K-contiguous
  int lda;                  // elements between A rows
  const int32_t* a_rows;    // [rows] source row of each logical row, or NULL (identity)
  const void* B;            // weights [group][N][kseg]
  const void* B2;           // second weight matrix (up projection) when SWIGLU, same layout
  const void* Bp;           // the same weights in the weight-streaming kernel's own order (occult_pack_weights),
                            // or NULL; read instead of B / B2 when that kernel is chosen
  long long bp_group_stride;   // bytes between consecutive weight matrices (pairs, when SWIGLU) in Bp
  long long b_group_stride; // elements between consecutive weight matrices
  int ldb;                  // elements between B rows (= kseg)
  int kseg;                 // K elements held by one weight matrix; K > kseg walks consecutive matrices
  void* C;                  // output rows
  int ldc;                  // elements between C rows
  int c_col0;               // first output column written by group 0
  int c_group_cols;         // group g writes from column c_col0 + g * c_group_cols
  void* C2;                 // SWIGLU only, or NULL: the two pre-activations are stored as well, in rows of 2 * ldc
                            // elements: [gate | up] of group g from column 2 * (c_col0 + g * c_group_cols), the up
                            // half N columns after the gate half
  const int32_t* grp_offset;  // [ngroups+1] logical-row prefix per group, or NULL: every group takes rows [0, M)
  const int32_t* grp_widx;    // [ngroups] weight matrix of each group, or NULL: w_base + group
  int w_base;
  int ngroups;
  int M;                    // rows when grp_offset == NULL
  int a_rows_total;         // rows of the A buffer that may be addressed (bounds 32-bit offsets)
  int plain_map;            // small-tile kernel: workgroup id = m-tile * n_tiles + n-tile (tiny grids)
  int ksplit;               // K in consecutive parts, K tiles [y*nk/ksplit, (y+1)*nk/ksplit), whose f32 sums are added in
                            // order; 0 or 1 = one sum.  Small-tile kernel (one group, no SWIGLU): blockIdx.y takes part
                            // y and writes its sums to ws; 128-row tiles: a block adds the parts in registers
  float* ws;                // small-tile kernel: [ksplit][M][N] partial sums
  int silu_rcp;             // 128-row tiles, SWIGLU: activation as the 256-row tiles compute it (hardware reciprocal)
  int once_rows;            // 128-row tiles: rows per group below which large weights are read, and the output stored, as not to be kept
  int span;                 // 128-row tiles, second problem: tiles of the first that one of its tiles takes the time of (launch_tile128)
  int N;                    // output columns (for SWIGLU: columns of h)
  int K;
};

// Launches C[rows][N] = A[rows][K] x B[group][N][K]^T group by group (cfg.dtype: bf16 on MFMA with f32
// accumulation, or f32 matrix instructions); with `swiglu` the output is silu(A B^T) * (A B2^T).  `total_rows` = logical
// rows over all groups.  Picks the tile shape from the rows per group.  Returns an OCCULT_* code.
// GemmArgs::once_rows (figures at launch_tile128): a forward pass, one whose shared experts have more rows than the routed ones, and one
// that keeps pre-activations; the input gradients, and those whose rows the weight gradients find in the caches
constexpr int kOnceForward = 88, kOnceForwardShared = 72, kOnceTrain = 96, kOnceRowsAgain = 240;

int launch_gemm(const occult_cfg_t& c, const GemmArgs& a, bool swiglu, int total_rows, hipStream_t s);

// The same product for the routed experts (`a`, grouped rows) and, unless b is NULL, for the shared ones (`b`,
// uniform groups, rows_b rows over all of them, same N): one launch where the 128-row tiles take both, two otherwise.
int launch_gemm_pair(const occult_cfg_t& c, const GemmArgs& a, const GemmArgs* b, bool swiglu, int total_rows, int rows_b,
                     hipStream_t s);

// A forward pass of a few tokens up to the gate/up product of its experts in one launch (plan.hip): routing, plan, row copies, and the
// products `first` (routed experts; its rows are those of x, found by the launch's own routing) and `second` (shared ones, or NULL)
bool fits_front(const occult_cfg_t& c);
int launch_front(const occult_cfg_t& c, const float* logits, int32_t* ids, float* w, const occult_plan_t& p, const void* x, void* sfd_x,
                 const GemmArgs& first, const GemmArgs* second, hipStream_t s);
// whether the expert products of a forward pass without kept pre-activations take that launch, and its two problems
bool forward_uses_front(const occult_cfg_t& c);
void front_products(const occult_cfg_t& c, const void* x, const occult_weights_t* weights, const void* packed, void* epd_h,
                    void* h_shared, GemmArgs* first, GemmArgs* second);
int check_ffn_args(const occult_cfg_t& c, const occult_plan_t* plan, const void* sfd_x, const void* x,
                   const occult_weights_t* weights, const void* epd_h, const void* epd_y, const void* h_shared, const void* y_shared);

// compute units of the current device
int device_cu_count(int* out);

// 128-row tiles (ffn_tile128.hip): `a` grouped, `b` NULL or uniform; bf16.
int launch_tile128(const GemmArgs& a, const GemmArgs* b, bool swiglu, int total_rows, hipStream_t s);

}  // namespace occult
