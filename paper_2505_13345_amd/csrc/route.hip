// occult_route: softmax top-k gating with optional collaboration pruning
// (paper Eq. 1; Section 3.3, routing-score-based pruning).
//
// Sixteen lanes per token, four tokens per wavefront (a whole wavefront per token in small batches).  Lane r of a token's
// sixteen holds the scores of experts r, r+16, r+32, ... (E <= 256); a selection round is the lane's best followed by a
// 4-step arg-max over the sixteen lanes.
// Selection compares raw scores (softmax is monotone): larger first, equal -> lower expert index.
// Routing is bound by these vector operations, not by its 300 bytes per token; a whole wavefront per token spent them on
// one token instead of four (18.5 us at 16384 tokens of 64 experts, k = 8; 40 us pruned).
//
// The pruning decision of mode 1 compares per-device sums of exp(score - max); those sums are
// taken in one fixed float32 sequence (exp_ref below: separately rounded multiplies and adds,
// no contraction into FMAs) so that a CPU restatement of the same text reaches the same bits.
#include "common.h"
#include "route_tokens.h"

// every float operation in this file is rounded on its own
#pragma clang fp contract(off)

namespace occult {

template <int LANES, int EPL, bool PRUNE>
__global__ __launch_bounds__(256) void route_kernel(
    const float* __restrict__ logits, int T, int E, int k, int D, int G,
    const int32_t* __restrict__ expert_pos, int n_d, int prune_mode, int renorm,
    const int32_t* __restrict__ sim_table, int32_t* __restrict__ ids, float* __restrict__ w) {
  route_tokens<LANES, EPL, PRUNE>((int)blockIdx.x, logits, T, E, k, D, G, expert_pos, n_d, prune_mode, renorm, sim_table, ids, w);
}

// ------------------------------------------------------------------------------------------
// Router projection g(x) = x W_r^T (paper Eq. 1), bf16 inputs.
// The work is reading x once.  A block takes 32 tokens and all E expert rows on v_mfma_f32_16x16x32_bf16, wave tiles of 16
// tokens x half of the experts; K tiles of 64 of both operands go straight into a ring of LDS stages (global_load_lds),
// all but one of them in flight.  Every request is a whole 128-byte line: 16-byte chunk c of row r lives in slot
// c ^ ((r >> 1) & 7) of its LDS row, conflict-free for the fragment reads (ffn.hip).  Two blocks share a CU up to 128
// experts.  (Before, the four waves of a block took a quarter of K each and loaded fragments in 64-byte pieces of 16 rows,
// permuted through the LDS crossbar: 64 experts, d = 2048, us: 1000
// tokens 8.7 -> 7.8, 4096 13.7 -> 8.7, 16384 29 -> 15.3 = 4.4 TB/s of x, 65536 107 -> 63; same bits.)
// K is summed in quarters, added in ascending order: the sums that four waves with a quarter each add up to, shorter
// chains than one.  Routing runs as its own launch: a token
// is a chain of dependent cross-lane steps, which many resident waves hide and eight tokens in sequence on
// one wave of this kernel do not (measured with a wave per token: fused 75 us, separate 40 us at T = 2^14;
// the routing launch alone is 8 us there with sixteen lanes per token).
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kRouterTokens = 32;

template <int EB, bool QUARTERED>   // EB: blocks of 16 experts, E <= 16 * EB; even
__global__ __launch_bounds__(256) void router_kernel(const __bf16* __restrict__ x, const __bf16* __restrict__ wr,
                                                     int T, int d, int E, float* __restrict__ logits) {
  constexpr int X_BYTES = kRouterTokens * 128, STAGE_BYTES = X_BYTES + EB * 16 * 128;
  constexpr int NST = EB == 2 ? 8 : EB == 4 ? 6 : EB == 8 ? 3 : 4;   // 64, 72, 60, 144 KiB
  constexpr int LOADS = 1 + EB / 2;                                 // per wave and K tile
  constexpr int KPB = EB <= 4 ? 2 : 1;                              // K tiles per block-wide wait
  constexpr int LSTRIDE = 16 * EB + 4;
  static_assert(kRouterTokens * LSTRIDE * 4 <= NST * STAGE_BYTES, "the scores leave through the stages");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE_BYTES];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tok0 = blockIdx.x * kRouterTokens;

  // loader role: a load covers 8 rows of 128 bytes, lane -> row lane/8, slot lane%8; one load of token rows and EB / 2 of
  // expert rows per wave and K tile
  const int lrow = lane >> 3;
  auto chunk = [&](int row) { return ((lane & 7) ^ ((row >> 1) & 7)) * 16; };
  const int x_row = wave * 8 + lrow;
  const char* xp = reinterpret_cast<const char*>(x) + (size_t)min(tok0 + x_row, T - 1) * d * 2 + chunk(x_row);   // rows past
  // the end repeat the last token; not written
  const char* wp[EB / 2];
#pragma unroll
  for (int i = 0; i < EB / 2; ++i) {
    const int row = (wave * (EB / 2) + i) * 8 + lrow;
    wp[i] = reinterpret_cast<const char*>(wr) + (size_t)min(row, E - 1) * d * 2 + chunk(row);
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) char*)smem);
  const int nk = d / 64;   // host: d % 128 == 0, with QUARTERED d % 256 == 0
  // byte offset of K tile kt in a row.  QUARTERED: the four quarters in turn, so that the requests in flight at a time lie
  // in different places of the rows, whose pitch is a power of two as often as not and their memory channels then the
  // same (1000 tokens of 16 experts, d = 4096: 16 us one quarter after another, 8 in turn)
  auto k_offset = [&](int kt) {   // past the end the last K tile again: the number of loads in flight stays constant
    kt = min(kt, nk - 1);
    return QUARTERED ? (size_t)((kt & 3) * (nk >> 2) + (kt >> 2)) * 128 : (size_t)kt * 128;
  };
  auto issue = [&](int kt) {
    const unsigned st = lds0 + (unsigned)(kt % NST) * STAGE_BYTES;
    const size_t k0 = k_offset(kt);
    load_to_lds_16(xp + k0, st + wave * 1024u);
#pragma unroll
    for (int i = 0; i < EB / 2; ++i) load_to_lds_16(wp[i] + k0, st + X_BYTES + (wave * (EB / 2) + i) * 1024u);
  };
  int foff[2];   // fragments of the two K steps of 32: lane l holds row l%16, K group l/16 of a 16-row block
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) foff[kk] = (lane & 15) * 128 + (((4 * kk + (lane >> 4)) ^ ((lane >> 1) & 7)) * 16);
  const int tg = wave & 1, eh = wave >> 1;
  const char* frag_x = smem + tg * 2048;
  const char* frag_w = smem + X_BYTES + eh * (EB / 2) * 2048;

  constexpr int NACC = QUARTERED ? 4 : 1;
  f32x4 acc[NACC][EB / 2], sum[EB / 2];
#pragma unroll
  for (int j = 0; j < EB / 2; ++j) {
    sum[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int n = 0; n < NACC; ++n) acc[n][j] = sum[j];
  }
  const int per_quarter = d / 128;   // K steps
  int left = per_quarter;
#pragma unroll
  for (int kt = 0; kt < NST - KPB; ++kt) issue(kt);
  // K tiles kt .. kt + KPB - 1; n: accumulator of the first
  auto multiply = [&](int kt, auto n) {
    // they are there for every wave, and everyone is done with those before
    wait_loads_and_barrier<(NST - 2 * KPB) * LOADS>();
#pragma unroll
    for (int i = 0; i < KPB; ++i) issue(kt + NST - KPB + i);
    bf16x8 xf[2 * KPB], wf[2 * KPB][EB / 2];
#pragma unroll
    for (int q = 0; q < 2 * KPB; ++q) {
      const int at = ((kt + q / 2) % NST) * STAGE_BYTES + foff[q & 1];
      xf[q] = *reinterpret_cast<const bf16x8*>(frag_x + at);
#pragma unroll
      for (int j = 0; j < EB / 2; ++j) wf[q][j] = *reinterpret_cast<const bf16x8*>(frag_w + at + j * 2048);
    }
#pragma unroll
    for (int q = 0; q < 2 * KPB; ++q) {
      constexpr int first = decltype(n)::value;
#pragma unroll
      for (int j = 0; j < EB / 2; ++j) {
        f32x4& to = acc[QUARTERED ? first + q / 2 : 0][j];
        to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[q][j], xf[q], to, 0, 0, 0);
      }
      if (!QUARTERED && --left == 0) {   // uniform
        left = per_quarter;
#pragma unroll
        for (int j = 0; j < EB / 2; ++j) {
          sum[j] = sum[j] + acc[0][j];
          acc[0][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
      }
    }
  };
  if constexpr (QUARTERED) {
    for (int kt = 0; kt < nk; kt += 4) {
      multiply(kt, std::integral_constant<int, 0>{});
      if constexpr (KPB == 1) multiply(kt + 1, std::integral_constant<int, 1>{});
      if constexpr (KPB <= 2) multiply(kt + 2, std::integral_constant<int, 2>{});
      if constexpr (KPB == 1) multiply(kt + 3, std::integral_constant<int, 3>{});
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < EB / 2; ++j) sum[j] = sum[j] + acc[q][j];
  } else {
    for (int kt = 0; kt < nk; kt += KPB) multiply(kt, std::integral_constant<int, 0>{});
  }
  wait_loads_and_barrier<0>();   // the loads past the end as well: the stages are free

  // sum[j] element e of lane l: token tg*16 + l%16, expert (eh*EB/2 + j)*16 + (l/16)*4 + e
  float* s_lg = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int j = 0; j < EB / 2; ++j)
    *reinterpret_cast<f32x4*>(&s_lg[(tg * 16 + (lane & 15)) * LSTRIDE + (eh * (EB / 2) + j) * 16 + (lane >> 4) * 4]) = sum[j];
  __syncthreads();
  // scores out: wave w writes tokens w*8 .. w*8+7 of the block, rows of E floats
  for (int j = 0; j < kRouterTokens / 4; ++j) {
    const int tl = wave * (kRouterTokens / 4) + j;
    const int t = tok0 + tl;
    if (t >= T) break;   // wave-uniform; no barrier follows
    const float* row = &s_lg[tl * LSTRIDE];
    for (int e = lane; e < E; e += 64) logits[(size_t)t * E + e] = row[e];
  }
}

// float32 inputs (parity configuration): one thread per (token, expert), K summed in order
__global__ __launch_bounds__(256) void router_f32_kernel(const float* __restrict__ x, const float* __restrict__ wr,
                                                         int T, int d, int E, float* __restrict__ logits) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)T * E) return;
  const float* xr = x + (i / E) * d;
  const float* wrow = wr + (i % E) * d;
  float acc = 0.0f;
  for (int q = 0; q < d; ++q) acc = acc + xr[q] * wrow[q];
  logits[i] = acc;
}

// Gram matrix of router scores, H^T H in float64, on v_mfma_f64_16x16x4_f64.  A block takes a slice of tokens and a
// 64 x 64 tile of the matrix; wave w takes the tile's rows (w & 3)*16 .. +15 over part w / 4 of the slice.
// Four tokens per step go straight from the scores into the operands (a lane holds one score of token lane / 16, converted
// to double), the parts are added in LDS in ascending order and the tile is added to the result with double atomics.  Tiles
// below the diagonal are written by the block of their mirror image.  What bounds it is the chain of 64-cycle products of a
// wave and the atomics on the few thousand cells, a set of them per block: hence several parts to a block.
// (us with the clearing launch, 64 experts: 1000 tokens 10.9 -> 7.6, 16384 21 -> 15, 65536 29 -> 21; 128 experts 37 -> 25 and 89 ->
// 51 at the latter two.  Before: a wave per 64 tokens and row block, its loads behind a branch each.)
constexpr int kGramBlocks = 256, kGramMany = 12288;   // see occult_similarity_gram
template <int PARTS>   // of a slice
__global__ __launch_bounds__(256 * PARTS) void gram_kernel(const float* __restrict__ logits, int T, int E,
                                                                int tokens_per_block, double* __restrict__ gram) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  __shared__ double s_part[PARTS][64 * 64];
  // blockIdx.y -> tile (ti, tj), ti <= tj
  int ti = 0, tj = blockIdx.y;
  const int tiles = (E + 63) / 64;
  while (tj >= tiles - ti) {
    tj -= tiles - ti;
    ++ti;
  }
  tj += ti;
  const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) & 3, part = threadIdx.x >> 8;
  const int tk = lane >> 4, c = lane & 15;
  const int ea = ti * 64 + wave * 16 + c;
  const int per_part = tokens_per_block / PARTS;   // host: a multiple of 4 * PARTS
  const int t_begin = blockIdx.x * tokens_per_block + part * per_part, t_end = min(T, t_begin + per_part);
  f64x4 acc[4] = {};
  constexpr int UN = 4;   // steps of 4 tokens requested together, one such set ahead of the products
  struct Set {
    float a[UN], b[UN][4];
  };
  // past the slice or the experts the last score of each is read, and zero taken for it: no branch around a load
  const int ca = min(ea, E - 1);
  int cb[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) cb[j] = min(tj * 64 + j * 16 + c, E - 1);
  auto load = [&](Set& s, int t0) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const float* row = logits + (size_t)min(t0 + 4 * u + tk, T - 1) * E;
      s.a[u] = row[ca];
#pragma unroll
      for (int j = 0; j < 4; ++j) s.b[u][j] = row[cb[j]];
    }
  };
  auto multiply = [&](const Set& s, int t0) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const bool live = t0 + 4 * u + tk < t_end;   // (experts past E: their cells are not written)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(live ? (double)s.a[u] : 0.0, live ? (double)s.b[u][j] : 0.0, acc[j], 0, 0, 0);
    }
  };
  Set s0, s1;
  load(s0, t_begin);
  for (int t0 = t_begin; t0 < t_end; t0 += 8 * UN) {
    load(s1, t0 + 4 * UN);
    multiply(s0, t0);
    load(s0, t0 + 8 * UN);
    multiply(s1, t0 + 4 * UN);
  }
  // acc[j] element i of lane l: tile row wave*16 + i*4 + l/16, column j*16 + l%16
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) s_part[part][(wave * 16 + i * 4 + tk) * 64 + j * 16 + c] = acc[j][i];
  __syncthreads();
  for (int n = threadIdx.x; n < 64 * 64; n += 256 * PARTS) {
    // blocks begin at different cells; off the diagonal a wave takes 8 x 8 cells, so that neither they nor their mirror
    // images lie in 64 different rows (128 experts, 16384 tokens: 78 us with whole rows, 25 so)
    int at = (n + blockIdx.x * 256) & (64 * 64 - 1);
    if (ti != tj) at = (at >> 9) * 512 + (at >> 3 & 7) * 64 + (at >> 6 & 7) * 8 + (at & 7);
    const int ei = ti * 64 + (at >> 6), ej = tj * 64 + (at & 63);
    if (ei >= E || ej >= E) continue;
    double v = s_part[0][at];
#pragma unroll
    for (int q = 1; q < PARTS; ++q) v += s_part[q][at];
    atomicAdd(&gram[(size_t)ei * E + ej], v);
    if (ti != tj) atomicAdd(&gram[(size_t)ej * E + ei], v);
  }
}

__global__ void fill_f64(double* p, size_t n, double v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace occult

using namespace occult;

extern "C" int occult_similarity_gram(const occult_cfg_t* cfg, const float* logits, double* gram,
                                      int accumulate, occult_stream_t stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  OCC_REQUIRE(gram, OCCULT_ENULLPTR, "gram is NULL");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t n = (size_t)c.E * c.E;
  if (!accumulate) {   // a fill kernel rather than a memset node, so the call can be captured in a graph
    hipLaunchKernelGGL(fill_f64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, gram, n, 0.0);
    OCC_LAUNCH_CHECK("fill_f64");
  }
  if (c.T == 0) return OCCULT_OK;
  OCC_REQUIRE(logits, OCCULT_ENULLPTR, "logits is NULL");
  const int tiles = (c.E + 63) / 64;
  // As many slices as give a wave 32 tokens, within 256 blocks over all tiles (65536 tokens of 64 experts: 29 us with 128, 21
  // with 256).  Two parts to a block while the blocks are few, four beyond, for a quarter of the atomics per product (64
  // experts, two / four: 4000 tokens 8.0 / 10.2, 8192 9.5 / 10.8, 16384 17.9 / 14.8)
  const int n_tiles = tiles * (tiles + 1) / 2;
  const bool many = c.T * (long long)n_tiles >= kGramMany;
  const int parts = many ? 4 : 2, tokens = 32 * parts, step = 4 * parts;
  int slices = (c.T + tokens - 1) / tokens;
  const int most = kGramBlocks / n_tiles > 32 ? kGramBlocks / n_tiles : 32;
  if (slices > most) slices = most;
  const int per = ((c.T + slices - 1) / slices + step - 1) / step * step;
  slices = (c.T + per - 1) / per;
  const dim3 grid(slices, n_tiles);
  if (many) hipLaunchKernelGGL(gram_kernel<4>, grid, dim3(1024), 0, s, logits, c.T, c.E, per, gram);
  else hipLaunchKernelGGL(gram_kernel<2>, grid, dim3(512), 0, s, logits, c.T, c.E, per, gram);
  OCC_LAUNCH_CHECK("gram_kernel");
  return OCCULT_OK;
}

extern "C" int occult_similarity_table(const double* gram_host, int32_t E, int32_t* table_host) {
  OCC_REQUIRE(gram_host && table_host, OCCULT_ENULLPTR, "gram_host or table_host is NULL");
  OCC_REQUIRE(E >= 2 && E <= OCCULT_MAX_E, OCCULT_EINVAL, "E=%d outside 2..%d", E, OCCULT_MAX_E);
  for (int i = 0; i < E; ++i)
    OCC_REQUIRE(gram_host[(size_t)i * E + i] > 0.0, OCCULT_EINVAL, "gram[%d][%d] is not positive", i, i);
  double sim[OCCULT_MAX_E];
  for (int i = 0; i < E; ++i) {
    for (int j = 0; j < E; ++j) {
      // each product and the quotient rounded on its own (file-wide contraction is off)
      const double g = gram_host[(size_t)i * E + j];
      const double num = g * g;
      const double den = gram_host[(size_t)i * E + i] * gram_host[(size_t)j * E + j];
      sim[j] = num / den;
    }
    int32_t* row = table_host + (size_t)i * (E - 1);
    int n = 0;
    for (int j = 0; j < E; ++j)
      if (j != i) row[n++] = j;
    // insertion sort by (similarity descending, index ascending): stable, E <= 256
    for (int a = 1; a < n; ++a) {
      const int32_t v = row[a];
      int b = a - 1;
      while (b >= 0 && sim[row[b]] < sim[v]) {
        row[b + 1] = row[b];
        --b;
      }
      row[b + 1] = v;
    }
  }
  return OCCULT_OK;
}

namespace occult {
int check_route_args(const occult_cfg_t& c, const float* logits, const int32_t* ids, const float* w) {
  OCC_REQUIRE(logits && ids && w, OCCULT_ENULLPTR, "logits, ids or w is NULL");
  if (c.n_d > 0 && c.prune_mode == 3)
    OCC_REQUIRE(c.sim_table != nullptr, OCCULT_ENULLPTR, "prune_mode 3 needs cfg.sim_table");
  return OCCULT_OK;
}
}  // namespace occult

extern "C" int occult_route(const occult_cfg_t* cfg, const float* logits, int32_t* ids, float* w,
                            occult_stream_t stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  if (c.T == 0) return OCCULT_OK;
  rc = check_route_args(c, logits, ids, w);
  if (rc) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int G = c.E / c.D;
  // A wavefront per token while every token can have a SIMD of a 256-CU chip to itself: the call is then one token's
  // chain of dependent steps, shortest with few experts per lane (3.5 us with sixteen lanes, 2.4 with 64, at 128 tokens
  // of 60 experts).  Beyond that the steps are shared by four tokens (16384 tokens: 18 us with 64 lanes, 8 with sixteen).
  const bool few = c.T <= 1024;
  const int per_block = few ? 4 : 16;
  const dim3 grid((c.T + per_block - 1) / per_block), block(256);
#define OCC_ROUTE_LAUNCH(L, N, P)                                                                  \
  hipLaunchKernelGGL((route_kernel<L, N, P>), grid, block, 0, s, logits, c.T, c.E, c.k, c.D, G,    \
                     c.expert_pos, c.n_d, c.prune_mode, c.renorm, c.sim_table, ids, w)
#define OCC_ROUTE(L, N)                        \
  do {                                         \
    if (c.n_d > 0) OCC_ROUTE_LAUNCH(L, N, true); \
    else OCC_ROUTE_LAUNCH(L, N, false);          \
  } while (0)
  if (few) {
    if (c.E <= 64) OCC_ROUTE(64, 1);
    else if (c.E <= 128) OCC_ROUTE(64, 2);
    else OCC_ROUTE(64, 4);
  } else if (c.E <= 16) OCC_ROUTE(16, 1);
  else if (c.E <= 32) OCC_ROUTE(16, 2);
  else if (c.E <= 64) OCC_ROUTE(16, 4);
  else if (c.E <= 128) OCC_ROUTE(16, 8);
  else OCC_ROUTE(16, 16);
#undef OCC_ROUTE
#undef OCC_ROUTE_LAUNCH
  OCC_LAUNCH_CHECK("route_kernel");
  return OCCULT_OK;
}

extern "C" int occult_router(const occult_cfg_t* cfg, const void* x, const void* w_router, float* logits,
                             int32_t* ids, float* w, occult_stream_t stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  const occult_cfg_t c = *cfg;
  if (c.T == 0) return OCCULT_OK;
  OCC_REQUIRE(x && w_router && logits && ids && w, OCCULT_ENULLPTR, "x, w_router, logits, ids or w is NULL");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (c.dtype == OCCULT_F32) {
    const size_t n = (size_t)c.T * c.E;
    hipLaunchKernelGGL(router_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       static_cast<const float*>(x), static_cast<const float*>(w_router), c.T, c.d, c.E, logits);
    OCC_LAUNCH_CHECK("router_f32_kernel");
    return occult_route(cfg, logits, ids, w, stream);
  }
  OCC_REQUIRE(c.d % 128 == 0, OCCULT_ESHAPE, "bf16 router needs d to be a multiple of 128 (d=%d)", c.d);
  OCC_REQUIRE(aligned16(x) && aligned16(w_router), OCCULT_EALIGN, "x or w_router is not 16-byte aligned");
  const dim3 grid((c.T + kRouterTokens - 1) / kRouterTokens), block(256);
  const int eb = (c.E + 15) / 16;
#define OCC_ROUTER_KERNEL(N, Q)                                                            \
  hipLaunchKernelGGL((router_kernel<N, Q>), grid, block, 0, s, static_cast<const __bf16*>(x), \
                     static_cast<const __bf16*>(w_router), c.T, c.d, c.E, logits)
#define OCC_ROUTER_LAUNCH(N)                          \
  do {                                                \
    if (c.d % 256 == 0) OCC_ROUTER_KERNEL(N, true);   \
    else OCC_ROUTER_KERNEL(N, false);                 \
  } while (0)
  if (eb <= 2) OCC_ROUTER_LAUNCH(2);
  else if (eb <= 4) OCC_ROUTER_LAUNCH(4);
  else if (eb <= 8) OCC_ROUTER_LAUNCH(8);
  else OCC_ROUTER_LAUNCH(16);
#undef OCC_ROUTER_LAUNCH
#undef OCC_ROUTER_KERNEL
  OCC_LAUNCH_CHECK("router_kernel");
  return occult_route(cfg, logits, ids, w, stream);
}
