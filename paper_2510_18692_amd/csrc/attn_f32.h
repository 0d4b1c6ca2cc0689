// fp32 group attention on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32), head_dim 64 or 128.
//
// A block owns 32 stationary rows (queries for the forward and dQ, keys for dK/dV) and its eight waves
// split the streamed rows of the group, 32 per step, step s going to wave s mod 8; the partial
// accumulators of the waves are added through LDS at the end (forward: after bringing them to a
// common maximum).  Full precision is used at a few thousand tokens: 4,096 tokens x 2 heads are only
// 256 such blocks, and the earlier kernels (one thread per row, plain FMAs against rows broadcast from
// LDS) kept 128 one-wave blocks busy for as long as one lane takes for a whole row.  Measured, before
// and after, forward / backward in us: 4,096 x 2 x 64, 8 groups of 512 341 / 1143 and 17.5 / 51; 8,192 x 4 x
// 128, 2 groups 9,133 / 36,215 and 692 / 2,180 (99 / 79 TFLOP/s of the 157 that the instruction has).
// Bound by the matrix instruction at large groups, at small ones by the latency of a few dependent steps and by
// the CUs that get a block more than others (8 groups of 480 to 534 make 262 blocks on 256 CUs: 33 / 93).  Two waves per SIMD: with one (more registers, D = 128) the large forward took 889 us.
//
// Operand layout (lane = (r, h), r = lane % 32, h = lane / 32):
//   * first products (scores): streamed rows are the A operand, one row per lane, stationary rows
//     the B operand, from LDS.  The contraction over channels may run in any order, so lane half h
//     takes channels 8j + 4h .. +3: 16-byte pieces of its row feed four instructions;
//   * the accumulator of a lane then holds streamed rows 8*(v/4) + 4h + v%4, v = 0..15, of the
//     stationary row r: register v of the two halves is exactly the B operand of a second product
//     whose contraction runs over the streamed rows, so P and dS never move;
//   * second products: the A operand is the streamed tensor transposed.  Channel d = DT*i + dt is
//     row i of output tile dt (DT = D / 32), so a lane reads DT adjacent channels of one streamed
//     row, and a wave half 128*DT contiguous bytes.
// Streamed rows go from L2 straight to registers: one 32-row step of the
// forward takes 64*D matrix cycles (4,096 at D = 64) for 256*D bytes of loads.
#pragma once

#include "attn_common.h"

namespace moga {

constexpr int kF32Rows = 32;   // stationary rows per block
constexpr int kF32Waves = 8;

// DT adjacent channels of a row, from a buffer.
template <int DT> struct F32Piece;
template <> struct F32Piece<2> {
  typedef floatx2_t type;
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t rows, int byte) {
    return __builtin_bit_cast(type, __builtin_amdgcn_raw_buffer_load_b64(rows, byte, 0, 0));
  }
};
template <> struct F32Piece<4> {
  typedef floatx4_t type;
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t rows, int byte) {
    return __builtin_bit_cast(type, __builtin_amdgcn_raw_buffer_load_b128(rows, byte, 0, 0));
  }
};

// Stationary rows in LDS: padded by 16 bytes, so that the 16-byte reads of 16 lanes (one row each)
// cover all banks.
template <int D> struct F32Tile { float v[kF32Rows][D + 4]; };

// Rows row0 .. row0 + 31 (clamped to last) of a [.., D] tensor into LDS, by `threads` threads.
template <int D, int THREADS>
__device__ __forceinline__ void f32_stage(F32Tile<D>& t, const float* __restrict__ base, int64_t row0, int64_t last) {
  constexpr int LPR = D / 4;
#pragma unroll
  for (int i = threadIdx.x; i < kF32Rows * LPR; i += THREADS) {
    const int row = i / LPR, c = (i % LPR) * 4;
    *(floatx4_t*)&t.v[row][c] = *(const floatx4_t*)(base + min(row0 + row, last) * D + c);
  }
}

// One streamed row as A operand of a score product.
template <int D> struct F32Row { floatx4_t v[D / 8]; };

template <int D>
__device__ __forceinline__ void f32_load_row(F32Row<D>& f, const float* __restrict__ row, int h) {
#pragma unroll
  for (int j = 0; j < D / 8; ++j) f.v[j] = *(const floatx4_t*)(row + 8 * j + 4 * h);
}

// acc += (streamed rows) x (stationary rows)^T
template <int D>
__device__ __forceinline__ void f32_scores(floatx16_t& acc, const F32Row<D>& f, const F32Tile<D>& t, int r, int h) {
#pragma unroll
  for (int j = 0; j < D / 8; ++j) {
    const floatx4_t b = *(const floatx4_t*)&t.v[r][8 * j + 4 * h];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f.v[j][e], b[e], acc, 0, 0, 0);
  }
}

// Streamed row of accumulator register v, relative to the step's first row.
__device__ __forceinline__ int f32_acc_row(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }

// acc[dt] += (streamed rows)^T x b, the streamed rows read with DT adjacent channels per lane.  Rows past `last` lie outside
// the buffer of the step's rows and read as zero: a copy of the last row times b = 0 would be NaN where that row has an
// infinity.  Selects for those rows made the D = 128 kernels spill (dQ, dK/dV and the forward 6 to 12 % slower); the buffer's
// own check needs fewer registers than clamped addresses (4,096 x 2 x 128, 8 groups: forward and backward 34.3 / 100.6 before,
// 33.4 / 97.4 us; x 64: 19.5 / 56.0 and 17.9 / 51.1).
template <int D>
__device__ __forceinline__ void f32_accumulate(floatx16_t (&acc)[D / 32], const float* __restrict__ base, int row0,
                                               int last, const floatx16_t& b, int r, int h) {
  constexpr int DT = D / 32;
  const auto rows = __builtin_amdgcn_make_buffer_rsrc((void*)(base + (int64_t)row0 * D), 0, min(32, last + 1 - row0) * D * 4, 0x00027000);
  int lane_off = (4 * h * D + DT * r) * 4;
  asm("" : "+v"(lane_off));   // not a loop invariant: the sixteen offsets are immediates, not registers kept through the loop
#pragma unroll
  for (int v0 = 0; v0 < 16; v0 += 8) {   // two batches of eight loads in flight
    typename F32Piece<DT>::type a[8];
#pragma unroll
    for (int v = 0; v < 8; ++v) a[v] = F32Piece<DT>::load(rows, lane_off + f32_acc_row(v0 + v, 0) * D * 4);
#pragma unroll
    for (int v = 0; v < 8; ++v)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        acc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[v][dt], b[v0 + v], acc[dt], 0, 0, 0);
  }
}

// Sum of the waves' accumulators, left in wave 0: halves of the waves hand theirs over in turn.
template <int NW, int DT>
__device__ __forceinline__ void f32_reduce_waves(floatx16_t (&acc)[DT], float (*buf)[DT * 16][64], int wave, int lane) {
#pragma unroll
  for (int s = NW / 2; s > 0; s >>= 1) {
    if (wave >= s && wave < 2 * s)
#pragma unroll
      for (int i = 0; i < DT * 16; ++i) buf[wave - s][i][lane] = acc[i >> 4][i & 15];
    __syncthreads();
    if (wave < s)
#pragma unroll
      for (int i = 0; i < DT * 16; ++i) acc[i >> 4][i & 15] += buf[wave][i][lane];
    __syncthreads();
  }
}

// Write acc * f (channel DT*i + dt of stationary row r) to `row`, and that times g to `tok`; either may be NULL.
template <int D>
__device__ __forceinline__ void f32_store_row(float* __restrict__ row, float* __restrict__ tok, const floatx16_t (&acc)[D / 32],
                                              float f, float g, int h) {
  constexpr int DT = D / 32;
#pragma unroll
  for (int b = 0; b < 4; ++b) {   // registers 4b .. 4b+3: channels DT*(8b + 4h) .. + 4*DT - 1
    float t[4 * DT];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) t[DT * e + dt] = acc[dt][4 * b + e] * f;
#pragma unroll
    for (int i = 0; i < DT; ++i) {
      const floatx4_t q = {t[4 * i], t[4 * i + 1], t[4 * i + 2], t[4 * i + 3]};
      if (row) *(floatx4_t*)(row + DT * (8 * b + 4 * h) + 4 * i) = q;
      if (tok) *(floatx4_t*)(tok + DT * (8 * b + 4 * h) + 4 * i) = floatx4_t{q[0] * g, q[1] * g, q[2] * g, q[3] * g};
    }
  }
}

// Row `row` of a [H, N, D] tensor and of its token-order counterpart [N, H, D]; NULL where the tensor is.
template <int D>
__device__ __forceinline__ float* f32_sorted_row(float* t, int64_t row) { return t ? t + row * D : nullptr; }
template <int D>
__device__ __forceinline__ float* f32_token_row(float* t, const int32_t* __restrict__ perm, int row, int head, int H) {
  return t ? t + ((int64_t)perm[row] * H + head) * D : nullptr;
}

__device__ __forceinline__ float f32_halves_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float f32_halves_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// P of the backward, exp(s * scale - lse): the difference first, in one rounding, and then to base 2.  With scale * log2(e)
// and lse * log2(e) rounded before the subtraction P was off by |lse| * 1e-7 (dV at logits around 100: 5.6e-6 from float64
// in the 2-norm, 3.5e-6 so; no change in time).
__device__ __forceinline__ float f32_prob(float s, float scale, float lse) {
  return fast_exp2(fmaf(s, scale, -lse) * 1.4426950408889634f);
}

// ---- forward ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(64 * kF32Waves) void attn_fwd_f32_mfma_kernel(
    const float* __restrict__ qh, const float* __restrict__ kh, const float* __restrict__ vh,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, int tiles_per_head, float* __restrict__ oh, float* __restrict__ lse,
    const int32_t* __restrict__ perm, const float* __restrict__ gate, float* __restrict__ o_tok) {
  constexpr int NW = kF32Waves, DT = D / 32;
  __shared__ __attribute__((aligned(16))) F32Tile<D> Qs;
  __shared__ float s_buf[NW / 2][DT * 16][64];
  __shared__ float s_m[NW][32], s_l[NW][32];
  const int head = blockIdx.x / tiles_per_head;
  const int tile = blockIdx.x - head * tiles_per_head;
  TileInfo ti;
  if (tile_start) {
    if (!find_tile_presummed(tile_start, cu_q, M, kF32Rows, tile, ti)) return;
  } else if (!find_tile(cu_q, M, kF32Rows, tile, ti)) {
    return;
  }
  const int gs = cu_k[ti.group], n = cu_k[ti.group + 1] - gs;   // keys of the group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int64_t head_off = (int64_t)head * Nq;
  const float* kb = kh + ((int64_t)head * Nk + gs) * D;
  const float* vb = vh + ((int64_t)head * Nk + gs) * D;
  const float c = scale * 1.4426950408889634f;
  const int nsteps = (n + 31) >> 5;

  F32Row<D> kf;
  if (wave < nsteps) f32_load_row<D>(kf, kb + (int64_t)min(32 * wave + r, n - 1) * D, h);
  f32_stage<D, 64 * NW>(Qs, qh, head_off + ti.tile_row, head_off + ti.row_end - 1);
  __syncthreads();

  floatx16_t o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.f;
  float m = -INFINITY, l = 0.f;
  for (int s = wave; s < nsteps; s += NW) {
    floatx16_t p;
#pragma unroll
    for (int v = 0; v < 16; ++v) p[v] = 0.f;
    f32_scores<D>(p, kf, Qs, r, h);
    if (s + NW < nsteps) f32_load_row<D>(kf, kb + (int64_t)min(32 * (s + NW) + r, n - 1) * D, h);
    if (32 * s + 32 > n)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (32 * s + f32_acc_row(v, h) >= n) p[v] = -INFINITY;
    float mx = p[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, p[v]);
    const float m_new = fmaxf(m, f32_halves_max(mx));
    const float ref = m_new == -INFINITY ? 0.f : m_new;   // every score so far may be -inf: weights of zero, not NaN
    const float alpha = fast_exp2((m - ref) * c);
    m = m_new;
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p[v] = fast_exp2((p[v] - ref) * c);
      sum += p[v];
    }
    l = fmaf(l, alpha, sum);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[dt][v] *= alpha;
    f32_accumulate<D>(o, vb, 32 * s, n - 1, p, r, h);
  }

  // common maximum of the waves (a wave without keys, or with none but scores of -inf, has m = -inf and weight 0)
  l = f32_halves_sum(l);
  if (h == 0) { s_m[wave][r] = m; s_l[wave][r] = l; }
  __syncthreads();
  float mt = s_m[0][r];
#pragma unroll
  for (int w = 1; w < NW; ++w) mt = fmaxf(mt, s_m[w][r]);
  float lt = 0.f;
  if (nsteps > 0) {
    const float ref = mt == -INFINITY ? 0.f : mt;
#pragma unroll
    for (int w = 0; w < NW; ++w) lt = fmaf(s_l[w][r], fast_exp2((s_m[w][r] - ref) * c), lt);
    const float f = fast_exp2((m - ref) * c);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[dt][v] *= f;
  }
  f32_reduce_waves<NW, DT>(o, s_buf, wave, lane);
  const int row = ti.tile_row + r;
  if (wave == 0 && row < ti.row_end) {   // no keys: zero output, lse = -inf
    f32_store_row<D>(oh + (head_off + row) * D, f32_token_row<D>(o_tok, perm, row, head, H), o, nsteps > 0 ? 1.f / lt : 0.f,
                     o_tok ? gate[perm[row]] : 1.f, h);
    if (h == 0) lse[head_off + row] = nsteps > 0 ? mt * scale + logf(lt) : -INFINITY;
  }
}

// ---- backward, query-stationary: delta and dQ --------------------------------------------
// Writes delta = rowsum(dO * O) of its rows for the dK/dV kernel that follows.
template <int D>
__global__ __launch_bounds__(64 * kF32Waves) void attn_bwd_dq_f32_mfma_kernel(
    const float* __restrict__ d_oh, const float* __restrict__ qh, const float* __restrict__ kh,
    const float* __restrict__ vh, const float* __restrict__ oh, const float* __restrict__ lse,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, int tiles_per_head, float* __restrict__ delta, float* __restrict__ d_qh,
    const int32_t* __restrict__ perm, float* __restrict__ d_q_tok) {
  constexpr int NW = kF32Waves, DT = D / 32, LPR = D / 4;
  __shared__ __attribute__((aligned(16))) F32Tile<D> Qs, Ds;
  __shared__ float s_buf[NW / 2][DT * 16][64];
  __shared__ float s_delta[kF32Rows];
  const int head = blockIdx.x / tiles_per_head;
  const int tile = blockIdx.x - head * tiles_per_head;
  TileInfo ti;
  if (tile_start) {
    if (!find_tile_presummed(tile_start, cu_q, M, kF32Rows, tile, ti)) return;
  } else if (!find_tile(cu_q, M, kF32Rows, tile, ti)) {
    return;
  }
  const int gs = cu_k[ti.group], n = cu_k[ti.group + 1] - gs;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int64_t head_off = (int64_t)head * Nq, first = head_off + ti.tile_row, last = head_off + ti.row_end - 1;
  const float* kb = kh + ((int64_t)head * Nk + gs) * D;
  const float* vb = vh + ((int64_t)head * Nk + gs) * D;
  const int nsteps = (n + 31) >> 5;

  f32_stage<D, 64 * NW>(Qs, qh, first, last);
#pragma unroll
  for (int i = threadIdx.x; i < kF32Rows * LPR; i += 64 * NW) {   // dO rows, and delta on the way
    const int row = i / LPR, cc = (i % LPR) * 4;
    const int64_t off = min(first + row, last) * D + cc;
    const floatx4_t a = *(const floatx4_t*)(d_oh + off), b = *(const floatx4_t*)(oh + off);
    *(floatx4_t*)&Ds.v[row][cc] = a;
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fmaf(a[e], b[e], s);
    s = lanes_sum<LPR>(s);
    if (i % LPR == 0) {
      s_delta[row] = s;
      if (first + row <= last) delta[first + row] = s;
    }
  }
  const float lv = lse[min(first + r, last)];
  __syncthreads();
  const float dl = s_delta[r];

  floatx16_t dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) dq[dt][v] = 0.f;
  for (int s = wave; s < nsteps; s += NW) {
    const int64_t row = (int64_t)min(32 * s + r, n - 1) * D;
    F32Row<D> kf, vf;
    f32_load_row<D>(kf, kb + row, h);
    f32_load_row<D>(vf, vb + row, h);
    floatx16_t p, dp;
#pragma unroll
    for (int v = 0; v < 16; ++v) { p[v] = 0.f; dp[v] = 0.f; }
    f32_scores<D>(p, kf, Qs, r, h);
    f32_scores<D>(dp, vf, Ds, r, h);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = f32_prob(p[v], scale, lv);
      p[v] = 32 * s + f32_acc_row(v, h) < n ? e * (dp[v] - dl) : 0.f;   // dS
    }
    f32_accumulate<D>(dq, kb, 32 * s, n - 1, p, r, h);
  }
  f32_reduce_waves<NW, DT>(dq, s_buf, wave, lane);
  if (wave == 0 && first + r <= last)
    f32_store_row<D>(f32_sorted_row<D>(d_qh, first + r), f32_token_row<D>(d_q_tok, perm, ti.tile_row + r, head, H), dq, scale, 1.f, h);
}

// ---- backward, key-stationary: dK and dV --------------------------------------------------
template <int D>
__global__ __launch_bounds__(64 * kF32Waves) void attn_bwd_dkdv_f32_mfma_kernel(
    const float* __restrict__ d_oh, const float* __restrict__ qh, const float* __restrict__ kh,
    const float* __restrict__ vh, const float* __restrict__ lse, const float* __restrict__ delta,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, int tiles_per_head, float* __restrict__ d_kh, float* __restrict__ d_vh,
    const int32_t* __restrict__ perm, float* __restrict__ d_k_tok, float* __restrict__ d_v_tok) {
  constexpr int NW = kF32Waves, DT = D / 32;
  __shared__ __attribute__((aligned(16))) F32Tile<D> Ks, Vs;
  __shared__ float s_buf[NW / 2][DT * 16][64];
  const int head = blockIdx.x / tiles_per_head;
  const int tile = blockIdx.x - head * tiles_per_head;
  TileInfo ti;   // tiles run over the key rows of the groups
  if (tile_start) {
    if (!find_tile_presummed(tile_start, cu_k, M, kF32Rows, tile, ti)) return;
  } else if (!find_tile(cu_k, M, kF32Rows, tile, ti)) {
    return;
  }
  const int gs = cu_q[ti.group], n = cu_q[ti.group + 1] - gs;   // queries of the group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int64_t first = (int64_t)head * Nk + ti.tile_row, last = (int64_t)head * Nk + ti.row_end - 1;
  const int64_t q_off = (int64_t)head * Nq + gs;
  const float* qb = qh + q_off * D;
  const float* ob = d_oh + q_off * D;
  const int nsteps = (n + 31) >> 5;

  f32_stage<D, 64 * NW>(Ks, kh, first, last);
  f32_stage<D, 64 * NW>(Vs, vh, first, last);
  __syncthreads();

  floatx16_t dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) { dk[dt][v] = 0.f; dv[dt][v] = 0.f; }
  for (int s = wave; s < nsteps; s += NW) {
    const int64_t row = (int64_t)min(32 * s + r, n - 1) * D;
    F32Row<D> qf, of;
    f32_load_row<D>(qf, qb + row, h);
    if (D == 64) f32_load_row<D>(of, ob + row, h);
    floatx16_t p, ds;
#pragma unroll
    for (int v = 0; v < 16; ++v) { p[v] = 0.f; ds[v] = 0.f; }
    f32_scores<D>(p, qf, Ks, r, h);
    if (D == 128) {   // 128 accumulator registers: one row of operands at a time, or the kernel spills
      __builtin_amdgcn_sched_barrier(0);
      f32_load_row<D>(of, ob + row, h);
    }
    f32_scores<D>(ds, of, Vs, r, h);
    if (D == 128) __builtin_amdgcn_sched_barrier(0);
    float lv[16], dl[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t q = q_off + min(32 * s + f32_acc_row(v, h), n - 1);
      lv[v] = lse[q];
      dl[v] = delta[q];
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = f32_prob(p[v], scale, lv[v]);
      const bool valid = 32 * s + f32_acc_row(v, h) < n;
      p[v] = valid ? e : 0.f;
      ds[v] = valid ? e * (ds[v] - dl[v]) : 0.f;
    }
    f32_accumulate<D>(dv, ob, 32 * s, n - 1, p, r, h);
    f32_accumulate<D>(dk, qb, 32 * s, n - 1, ds, r, h);
  }
  f32_reduce_waves<NW, DT>(dv, s_buf, wave, lane);
  f32_reduce_waves<NW, DT>(dk, s_buf, wave, lane);
  if (wave == 0 && first + r <= last) {
    const int row = ti.tile_row + r;
    f32_store_row<D>(f32_sorted_row<D>(d_vh, first + r), f32_token_row<D>(d_v_tok, perm, row, head, H), dv, 1.f, 1.f, h);
    f32_store_row<D>(f32_sorted_row<D>(d_kh, first + r), f32_token_row<D>(d_k_tok, perm, row, head, H), dk, scale, 1.f, h);
  }
}

}  // namespace moga
