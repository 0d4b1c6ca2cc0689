// fp32 group attention for calls of few rows (v_mfma_f32_16x16x4_f32), head_dim 64 or 128: blocks of 16 stationary rows and
// four waves that share the streamed rows, 16 T per step.
//
// attn_f32.h cuts such a call into too few pieces: 4,096 rows x 2 heads in 8 groups are 264 of its 32-row blocks, one to a CU
// by their registers, so that eight CUs took two and the call twice as long.  These blocks are half as large and three or four
// share a CU: they also cover each other's waits.  dQ and dK/dV, which do not need each other, run in one launch.  A row of
// operands feeds half as many products here, so larger calls stay with the other kernels (see use_f32_small).
//
// Operand layout (lane = 16 g + r):
//   * scores: A holds 16 streamed rows, B the 16 stationary rows; the contraction over channels may run in any order, so lane
//     group g takes channels 16 j + 4 g .. + 3: 16-byte pieces of its row feed four instructions.  Stationary rows stay in
//     registers;
//   * a lane's four results are streamed rows 4 g + i of stationary row r: register i of the four groups is the B operand of a
//     second product over those four rows, so P and dS never move;
//   * second products: A is the streamed tensor transposed.  Channel (D / 16) i + dt is row i of output tile dt, so a lane
//     reads D / 16 adjacent channels of one streamed row and ends up with D / 4 adjacent channels of its stationary row.
#pragma once

#include "attn_f32.h"

namespace moga {

constexpr int kF32SmallRows = 16;
constexpr int kF32SmallWaves = 4;
template <int D> constexpr int kF32SmallTiles = D == 64 ? 2 : 1;   // T: with D = 128 two would not fit the registers

__device__ __forceinline__ floatx4_t f32s_mfma(float a, float b, floatx4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Channels 16 j + 4 g .. + 3 of one row.
template <int D> struct F32Frag { floatx4_t v[D / 16]; };

template <int D>
__device__ __forceinline__ void f32s_load(F32Frag<D>& f, const float* __restrict__ row, int g) {
#pragma unroll
  for (int j = 0; j < D / 16; ++j) f.v[j] = *(const floatx4_t*)(row + 16 * j + 4 * g);
}

// The 16 T streamed rows from row0 (clamped to the last of n) as A operands.
template <int D, int T>
__device__ __forceinline__ void f32s_load_rows(F32Frag<D> (&f)[T], const float* __restrict__ base, int row0, int n, int r, int g) {
#pragma unroll
  for (int t = 0; t < T; ++t) f32s_load<D>(f[t], base + (int64_t)min(row0 + 16 * t + r, n - 1) * D, g);
}

// (streamed rows) x (stationary rows)^T
template <int D, int T>
__device__ __forceinline__ void f32s_scores(floatx4_t (&acc)[T], const F32Frag<D> (&a)[T], const F32Frag<D>& b) {
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < D / 16; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] = f32s_mfma(a[t].v[j][e], b.v[j][e], acc[t]);
}

// Transposed operand: D / 16 adjacent channels of the lane's four streamed rows of every tile.  Rows past n lie outside the
// buffer of the step's rows and read as zero (see f32_accumulate).
template <int D, int T> struct F32Cols { floatx4_t v[T][4][D / 64]; };

template <int D, int T>
__device__ __forceinline__ void f32s_load_cols(F32Cols<D, T>& c, const float* __restrict__ base, int row0, int n, int r, int g) {
  const auto rows = __builtin_amdgcn_make_buffer_rsrc((void*)(base + (int64_t)row0 * D), 0, min(16 * T, n - row0) * D * 4, 0x00027000);
  const int lane_off = (4 * g * D + (D / 16) * r) * 4;
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int p = 0; p < D / 64; ++p)
        c.v[t][i][p] = __builtin_bit_cast(floatx4_t, __builtin_amdgcn_raw_buffer_load_b128(rows, lane_off + ((16 * t + i) * D + 4 * p) * 4, 0, 0));
}

// acc += (streamed rows)^T x b
template <int D, int T>
__device__ __forceinline__ void f32s_accumulate(floatx4_t (&acc)[D / 16], const F32Cols<D, T>& c, const floatx4_t (&b)[T]) {
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) acc[dt] = f32s_mfma(c.v[t][i][dt >> 2][dt & 3], b[t][i], acc[dt]);
}

// Four values per streamed row of the lane (lse, delta) from `base`, zero past n.
template <int T>
__device__ __forceinline__ void f32s_load_stats(floatx4_t (&v)[T], const float* __restrict__ base, int row0, int n, int g) {
  const auto rows = __builtin_amdgcn_make_buffer_rsrc((void*)(base + row0), 0, min(16 * T, n - row0) * 4, 0x00027000);
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      v[t][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows, (16 * t + 4 * g + i) * 4, 0, 0));
}

__device__ __forceinline__ float f32s_rows_max(float v) {   // over the four lanes of a stationary row
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f32_halves_max(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
}
__device__ __forceinline__ float f32s_rows_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f32_halves_sum(__uint_as_float(a[0]) + __uint_as_float(a[1]));
}

// The waves' accumulators, one row of D channels (and 16 bytes against bank conflicts) per stationary row.
template <int D> struct F32Sums { __attribute__((aligned(16))) float v[kF32SmallWaves][kF32SmallRows][D + 4]; };

template <int D>
__device__ __forceinline__ void f32s_put(F32Sums<D>& s, const floatx4_t (&acc)[D / 16], int wave, int r, int g) {
  float t[D / 4];   // channel (D / 16) (4 g + v) + dt
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) t[(D / 16) * v + dt] = acc[dt][v];
#pragma unroll
  for (int i = 0; i < D / 16; ++i)
    *(floatx4_t*)&s.v[wave][r][(D / 4) * g + 4 * i] = floatx4_t{t[4 * i], t[4 * i + 1], t[4 * i + 2], t[4 * i + 3]};
}

// Sixteen threads a row: four channels each, D / 64 times.  f: the waves' weights.
template <int D>
__device__ __forceinline__ void f32s_write(const F32Sums<D>& s, const float (&f)[kF32SmallWaves], float scale, float g, int row,
                                           float* __restrict__ out, float* __restrict__ tok) {
#pragma unroll
  for (int p = 0; p < D / 64; ++p) {
    const int c = 64 * p + 4 * (threadIdx.x & 15);
    floatx4_t q[kF32SmallWaves];
#pragma unroll
    for (int w = 0; w < kF32SmallWaves; ++w) q[w] = *(const floatx4_t*)&s.v[w][row][c] * f[w];
    const floatx4_t v = ((q[0] + q[1]) + (q[2] + q[3])) * scale;
    if (out) *(floatx4_t*)(out + c) = v;
    if (tok) *(floatx4_t*)(tok + c) = v * g;
  }
}

// Block -> (head, tile): false beyond the last tile.
__device__ __forceinline__ bool f32s_find(const int32_t* __restrict__ cu, const int32_t* __restrict__ tile_start, int M, int block,
                                          int tiles_per_head, int& head, TileInfo& ti) {
  head = block / tiles_per_head;
  const int tile = block - head * tiles_per_head;
  return tile_start ? find_tile_presummed(tile_start, cu, M, kF32SmallRows, tile, ti) : find_tile(cu, M, kF32SmallRows, tile, ti);
}

// ---- forward ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(64 * kF32SmallWaves, D == 64 ? 4 : 2) void attn_fwd_f32_small_kernel(
    const float* __restrict__ qh, const float* __restrict__ kh, const float* __restrict__ vh,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, int tiles_per_head, float* __restrict__ oh, float* __restrict__ lse,
    const int32_t* __restrict__ perm, const float* __restrict__ gate, float* __restrict__ o_tok) {
  constexpr int NW = kF32SmallWaves, T = kF32SmallTiles<D>, STEP = 16 * T;
  __shared__ F32Sums<D> s_o;
  __shared__ float s_m[NW][16], s_l[NW][16];
  int head;
  TileInfo ti;
  if (!f32s_find(cu_q, tile_start, M, blockIdx.x, tiles_per_head, head, ti)) return;
  const int gs = cu_k[ti.group], n = cu_k[ti.group + 1] - gs;   // keys of the group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t head_off = (int64_t)head * Nq;
  const float* kb = kh + ((int64_t)head * Nk + gs) * D;
  const float* vb = vh + ((int64_t)head * Nk + gs) * D;
  const float c = scale * 1.4426950408889634f;

  F32Frag<D> kf[T], qf;
  if (STEP * wave < n) f32s_load_rows<D, T>(kf, kb, STEP * wave, n, r, g);
  f32s_load<D>(qf, qh + (head_off + min(ti.tile_row + r, ti.row_end - 1)) * D, g);
  floatx4_t o[D / 16];
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) o[dt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  for (int row0 = STEP * wave; row0 < n; row0 += STEP * NW) {
    F32Cols<D, T> vf;
    f32s_load_cols<D, T>(vf, vb, row0, n, r, g);   // in flight during the scores
    floatx4_t p[T];
    f32s_scores<D, T>(p, kf, qf);
    if (row0 + STEP * NW < n) f32s_load_rows<D, T>(kf, kb, row0 + STEP * NW, n, r, g);
    if (row0 + STEP > n)
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (row0 + 16 * t + 4 * g + i >= n) p[t][i] = -INFINITY;
    float mx = p[0][0];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, p[t][i]);
    const float m_new = fmaxf(m, f32s_rows_max(mx));
    const float ref = m_new == -INFINITY ? 0.f : m_new;   // every score so far may be -inf: weights of zero, not NaN
    const float alpha = fast_exp2((m - ref) * c);
    m = m_new;
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[t][i] = fast_exp2((p[t][i] - ref) * c);
        sum += p[t][i];
      }
    l = fmaf(l, alpha, sum);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) o[dt] *= alpha;
    f32s_accumulate<D, T>(o, vf, p);
  }

  // common maximum of the waves (a wave without keys, or with none but scores of -inf, has m = -inf and weight 0)
  l = f32s_rows_sum(l);
  f32s_put<D>(s_o, o, wave, r, g);
  if (g == 0) { s_m[wave][r] = m; s_l[wave][r] = l; }
  __syncthreads();
  const int row = threadIdx.x >> 4, j = ti.tile_row + row;
  if (j >= ti.row_end) return;
  float mt = s_m[0][row];
#pragma unroll
  for (int w = 1; w < NW; ++w) mt = fmaxf(mt, s_m[w][row]);
  const float ref = mt == -INFINITY ? 0.f : mt;
  float f[NW], lt = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    f[w] = fast_exp2((s_m[w][row] - ref) * c);
    lt = fmaf(s_l[w][row], f[w], lt);
  }
  f32s_write<D>(s_o, f, n > 0 ? 1.f / lt : 0.f, o_tok ? gate[perm[j]] : 1.f, row, oh + (head_off + j) * D,
                f32_token_row<D>(o_tok, perm, j, head, H));
  if ((threadIdx.x & 15) == 0) lse[head_off + j] = n > 0 ? mt * scale + logf(lt) : -INFINITY;   // no keys: zero output, lse = -inf
}

// ---- backward: -delta = -rowsum(dO * O) comes from the caller ------------------------------
template <int D>
__device__ __forceinline__ void f32s_dq_block(
    F32Sums<D>& sums, int block, const float* __restrict__ d_oh, const float* __restrict__ qh, const float* __restrict__ kh,
    const float* __restrict__ vh, const float* __restrict__ lse, const float* __restrict__ neg_delta, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M, int64_t Nq, int64_t Nk, int H, float scale,
    int tiles_per_head, float* __restrict__ d_qh, const int32_t* __restrict__ perm, float* __restrict__ d_q_tok) {
  constexpr int NW = kF32SmallWaves, T = kF32SmallTiles<D>, STEP = 16 * T;
  int head;
  TileInfo ti;
  if (!f32s_find(cu_q, tile_start, M, block, tiles_per_head, head, ti)) return;
  const int gs = cu_k[ti.group], n = cu_k[ti.group + 1] - gs;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t head_off = (int64_t)head * Nq;
  const float* kb = kh + ((int64_t)head * Nk + gs) * D;
  const float* vb = vh + ((int64_t)head * Nk + gs) * D;
  const int64_t own = head_off + min(ti.tile_row + r, ti.row_end - 1);
  F32Frag<D> qf, of;
  f32s_load<D>(qf, qh + own * D, g);
  f32s_load<D>(of, d_oh + own * D, g);
  const float lv = lse[own], ndl = neg_delta[own];
  floatx4_t dq[D / 16];
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) dq[dt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  F32Frag<D> kf[T], vf[T];
  auto load_rows = [&](int row0) {
    f32s_load_rows<D, T>(kf, kb, row0, n, r, g);
    f32s_load_rows<D, T>(vf, vb, row0, n, r, g);
  };
  if (D == 64 && STEP * wave < n) load_rows(STEP * wave);
  for (int row0 = STEP * wave; row0 < n; row0 += STEP * NW) {
    F32Cols<D, T> kt;
    if (D == 128) load_rows(row0);
    f32s_load_cols<D, T>(kt, kb, row0, n, r, g);   // in flight during the scores
    floatx4_t p[T], dp[T];
    f32s_scores<D, T>(p, kf, qf);
    f32s_scores<D, T>(dp, vf, of);
    if (D == 64 && row0 + STEP * NW < n) load_rows(row0 + STEP * NW);   // during the rest of this step (D = 128 would spill)
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = f32_prob(p[t][i], scale, lv);
        p[t][i] = row0 + 16 * t + 4 * g + i < n ? e * (dp[t][i] + ndl) : 0.f;   // dS
      }
    f32s_accumulate<D, T>(dq, kt, p);
  }
  f32s_put<D>(sums, dq, wave, r, g);
  __syncthreads();
  const int row = threadIdx.x >> 4, j = ti.tile_row + row;
  if (j >= ti.row_end) return;
  const float one[NW] = {1.f, 1.f, 1.f, 1.f};
  f32s_write<D>(sums, one, scale, 1.f, row, f32_sorted_row<D>(d_qh, head_off + j), f32_token_row<D>(d_q_tok, perm, j, head, H));
}

template <int D>
__device__ __forceinline__ void f32s_dkdv_block(
    F32Sums<D>& s_dk, F32Sums<D>& s_dv, int block, const float* __restrict__ d_oh, const float* __restrict__ qh,
    const float* __restrict__ kh, const float* __restrict__ vh, const float* __restrict__ lse, const float* __restrict__ neg_delta,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M, int64_t Nq,
    int64_t Nk, int H, float scale, int tiles_per_head, float* __restrict__ d_kh, float* __restrict__ d_vh,
    const int32_t* __restrict__ perm, float* __restrict__ d_k_tok, float* __restrict__ d_v_tok) {
  constexpr int NW = kF32SmallWaves, T = kF32SmallTiles<D>, STEP = 16 * T;
  int head;
  TileInfo ti;   // tiles run over the key rows of the groups
  if (!f32s_find(cu_k, tile_start, M, block, tiles_per_head, head, ti)) return;
  const int gs = cu_q[ti.group], n = cu_q[ti.group + 1] - gs;   // queries of the group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t head_off = (int64_t)head * Nk, q_off = (int64_t)head * Nq + gs;
  const float* qb = qh + q_off * D;
  const float* ob = d_oh + q_off * D;
  const int64_t own = head_off + min(ti.tile_row + r, ti.row_end - 1);
  F32Frag<D> kf, vf;
  f32s_load<D>(kf, kh + own * D, g);
  f32s_load<D>(vf, vh + own * D, g);
  floatx4_t dk[D / 16], dv[D / 16];
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) dk[dt] = dv[dt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  F32Frag<D> qf[T], of[T];
  auto load_rows = [&](int row0) {
    f32s_load_rows<D, T>(qf, qb, row0, n, r, g);
    f32s_load_rows<D, T>(of, ob, row0, n, r, g);
  };
  if (D == 64 && STEP * wave < n) load_rows(STEP * wave);
  for (int row0 = STEP * wave; row0 < n; row0 += STEP * NW) {
    if (D == 128) load_rows(row0);
    F32Cols<D, T> ot, qt;
    floatx4_t lv[T], ndl[T], p[T], ds[T];
    f32s_load_stats<T>(lv, lse + q_off, row0, n, g);
    f32s_load_stats<T>(ndl, neg_delta + q_off, row0, n, g);
    f32s_load_cols<D, T>(ot, ob, row0, n, r, g);
    f32s_scores<D, T>(p, qf, kf);
    f32s_scores<D, T>(ds, of, vf);
    f32s_load_cols<D, T>(qt, qb, row0, n, r, g);
    if (D == 64 && row0 + STEP * NW < n) load_rows(row0 + STEP * NW);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = f32_prob(p[t][i], scale, lv[t][i]);
        const bool valid = row0 + 16 * t + 4 * g + i < n;
        p[t][i] = valid ? e : 0.f;
        ds[t][i] = valid ? e * (ds[t][i] + ndl[t][i]) : 0.f;
      }
    f32s_accumulate<D, T>(dv, ot, p);
    f32s_accumulate<D, T>(dk, qt, ds);
  }
  f32s_put<D>(s_dv, dv, wave, r, g);
  f32s_put<D>(s_dk, dk, wave, r, g);
  __syncthreads();
  const int row = threadIdx.x >> 4, j = ti.tile_row + row;
  if (j >= ti.row_end) return;
  const float one[NW] = {1.f, 1.f, 1.f, 1.f};
  f32s_write<D>(s_dv, one, 1.f, 1.f, row, f32_sorted_row<D>(d_vh, head_off + j), f32_token_row<D>(d_v_tok, perm, j, head, H));
  f32s_write<D>(s_dk, one, scale, 1.f, row, f32_sorted_row<D>(d_kh, head_off + j), f32_token_row<D>(d_k_tok, perm, j, head, H));
}

// Blocks below `k_blocks` are dK/dV's (four products to three: the longer ones first), the others dQ's.
template <int D>
__global__ __launch_bounds__(64 * kF32SmallWaves, 2) void attn_bwd_f32_small_kernel(
    const float* __restrict__ d_oh, const float* __restrict__ qh, const float* __restrict__ kh, const float* __restrict__ vh,
    const float* __restrict__ lse, const float* __restrict__ neg_delta, const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k,
    const int32_t* __restrict__ ts_q, const int32_t* __restrict__ ts_k, int M, int64_t Nq, int64_t Nk, int H, float scale, int q_tiles,
    int k_tiles, int k_blocks, float* __restrict__ d_qh, float* __restrict__ d_kh, float* __restrict__ d_vh,
    const int32_t* __restrict__ perm, float* __restrict__ d_q_tok, float* __restrict__ d_k_tok, float* __restrict__ d_v_tok) {
  __shared__ F32Sums<D> sums[2];
  if ((int)blockIdx.x < k_blocks)
    f32s_dkdv_block<D>(sums[0], sums[1], blockIdx.x, d_oh, qh, kh, vh, lse, neg_delta, cu_q, cu_k, ts_k, M, Nq, Nk, H, scale, k_tiles, d_kh,
                       d_vh, perm, d_k_tok, d_v_tok);
  else
    f32s_dq_block<D>(sums[0], blockIdx.x - k_blocks, d_oh, qh, kh, vh, lse, neg_delta, cu_q, cu_k, ts_q, M, Nq, Nk, H, scale, q_tiles, d_qh,
                     perm, d_q_tok);
}

// True where a call takes these kernels: up to kF32MaxTiles 32-row tiles of the others.  Groups as a router makes them (16- against
// 32-row kernels, forward / backward in us): 4,096 x 2 heads x 64, 8 groups 22.6 / 61.5 and 30.9 / 87.6; 3,000 x 4 x 64, 2
// groups 56 / 188 and 70 / 217; 8,192 x 4 x 64, 8 groups (1,056 tiles) 116 / 359 and 124 / 385, 2 groups 424 / 1,278 and 402 /
// 1,353; x 128, 2 groups 696 / 2,453 and 834 / 2,761.  Groups of 512 or 4,096 rows exactly, which leave the 32-row kernels
// no part-filled tile, are even up to 272 tiles and cost 5 to 13 % at 528 to 1,032 (D = 64; D = 128: forward faster, backward
// 4 to 8 %): beyond the line the two draw level for any groups.
constexpr int64_t kF32MaxTiles = 1152;
inline bool use_f32_small(int64_t rows, int H, int groups) {
  return use_small_group_kernels(rows, groups, max_tiles(rows, groups, kF32Rows) * H <= kF32MaxTiles ? INT64_MAX : 0);
}

}  // namespace moga
