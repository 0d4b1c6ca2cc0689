// fp32 group attention on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32), head_dim 64 or 128: blocks of 16 stationary rows
// (queries for the forward and dQ, keys for dK/dV) and four waves that share the streamed rows of the group, 16 T per step, step
// s going to wave s mod 4; the waves' partial accumulators are added through LDS at the end (forward: after bringing them to a
// common maximum).  Small blocks, because full precision is used at a few thousand tokens: 4,096 rows x 2 heads are 512 of them,
// two to four share a CU and cover each other's waits.  dQ and dK/dV, which do not need each other, run in one launch.
//
// Operand layout (lane = 16 g + r):
//   * scores: A holds 16 streamed rows, B the 16 stationary rows; the contraction over channels may run in any order, so lane
//     group g takes channels 16 j + 4 g .. + 3: 16-byte pieces of its row feed four instructions.  Stationary rows stay in
//     registers;
//   * a lane's four results are streamed rows 4 g + i of stationary row r: register i of the four groups is the B operand of a
//     second product over those four rows, so P and dS never move;
//   * second products: A is the streamed tensor transposed.  Channel 64 p + 4 i + e is row i of output tile 4 p + e, so a lane
//     reads 4 adjacent channels of one streamed row.
//
// Streamed rows reach the scores, and in the backward the second products too, through the wave's own LDS.  Loaded straight as A
// operands, the 16 lanes that a load serves at a time were in 16 rows, a cache line each for 16 bytes, and the vector cache's rate
// of lines was the bound (10 TB/s from L2).  Forward / backward in us, so and now: 4,096 x 2 heads x 64, 8 groups 22.6 / 61.2 and
// 20.9 / 51.6; 8,192 x 4 x 64, 8 groups 116 / 354 and 88 / 284; 16,384 x 4 x 64, 4 groups 822 / 2,591 and 594 / 1,986 (116 and 121
// TFLOP/s executed of the 157 that the instruction has); x 128 1,328 / 4,775 and 1,184 / 3,902.  Bound by the matrix instruction
// at large groups, at small ones by a few dependent steps between launch, first loads and the final sums.  The 32-row blocks of
// eight waves that these replaced (32x32x2 instruction, rows straight from memory) took 29.5 / 86.3, 124 / 384, 739 / 2,454 and
// 1,515 / 4,953.
#pragma once

#include "attn_common.h"

namespace moga {

constexpr int kF32Rows = 16;
constexpr int kF32Waves = 4;
// T, the 16-row tiles of a step, is one in calls of at most kF32ShortCall rows with D = 64, else two (with D = 128 two would not fit the
// registers).  One tile leaves registers for three waves per SIMD in the backward instead of two (1,024 rows x 2 heads, 4 groups 15.2 and 17.0 us)
// but adds twice as many sums to the results, which in long groups shows.  Errors against float64 in the 2-norm, in 1e-7, with one tile and two,
// by the rows of one group: O 512 3.04 and 3.10, 1,536 3.22 and 3.24, 2,048 3.28 and 3.28, 4,096 3.42 and 3.35, 8,192 3.76 and 3.56, 30,000 5.04
// and 4.28; dQ 512 4.21 and 4.25, 1,536 4.58 and 4.59, 2,048 5.19 and 5.19, 4,096 5.40 and 5.35, 8,192 5.76 and 5.62, 30,000 6.98 and 6.44; dK and
// dV alike.  The line is by the rows of the call, which no group can exceed and empty groups do not change: by the mean group, one tile took
// 4,096 x 2, 8 groups from 51.6 to 49.0 us backward, and a group that has most of the rows with it.
constexpr int kF32ShortCall = 1536;

__device__ __forceinline__ floatx4_t f32_mfma(float a, float b, floatx4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
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

// Channels 16 j + 4 g .. + 3 of one row.
template <int D> struct F32Frag { floatx4_t v[D / 16]; };

template <int D>
__device__ __forceinline__ void f32_load(F32Frag<D>& f, const float* __restrict__ row, int g) {
#pragma unroll
  for (int j = 0; j < D / 16; ++j) f.v[j] = *(const floatx4_t*)(row + 16 * j + 4 * g);
}

// The compiler waits for the loads here, and not in the loop, where it would count them against later ones.
template <int D>
__device__ __forceinline__ void f32_settle(F32Frag<D>& f) {
#pragma unroll
  for (int j = 0; j < D / 16; ++j) asm volatile("" : "+v"(f.v[j]));
}

// A wave's 16 T streamed rows of one tensor in its own LDS, in direct-to-LDS loads of 1 KB (whole rows).  Straight from
// memory as A operands, every lane of a load is in a row of its own: sixteen cache lines for 256 bytes.  Chunk c (16 bytes) of
// row j is stored at c ^ swizzle(j), which spreads both kinds of reads below over all banks.
__device__ __forceinline__ constexpr int f32_swizzle(int row) { return (row & 15) ^ ((row & 4) << 1); }

template <int D, int T>
__device__ __forceinline__ void f32_stage(unsigned lds, const float* __restrict__ base, int row0, int n, int lane) {
  constexpr int LPR = D / 4, RPI = 64 / LPR;   // lanes per row, rows per load
  const void* rows = uniform_ptr(base + (int64_t)row0 * D);
  const int last = n - 1 - row0;   // rows past n: the last one, not used
#pragma unroll
  for (int q = 0; q < 16 * T / RPI; ++q) {
    const int row = RPI * q + lane / LPR;
    lds_dma16_soff(rows, (unsigned)((min(row, last) * D + 4 * ((lane % LPR) ^ f32_swizzle(row))) * 4), lds + q * 1024);
  }
}

__device__ __forceinline__ floatx4_t f32_lds(unsigned addr) {
  return *(const floatx4_t __attribute__((address_space(3)))*)(uintptr_t)addr;
}

// The staged rows as A operands.
template <int D, int T>
__device__ __forceinline__ void f32_read_rows(F32Frag<D> (&f)[T], unsigned lds, int r, int g) {
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int j = 0; j < D / 16; ++j) f[t].v[j] = f32_lds(lds + r * D * 4 + (((4 * (j & 3) + g) ^ f32_swizzle(r)) << 4) + 16 * t * D * 4 + (j >> 2) * 256);
}

// (streamed rows) x (stationary rows)^T
template <int D, int T>
__device__ __forceinline__ void f32_scores(floatx4_t (&acc)[T], const F32Frag<D> (&a)[T], const F32Frag<D>& b) {
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < D / 16; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] = f32_mfma(a[t].v[j][e], b.v[j][e], acc[t]);
}

// Transposed operand: channels 64 p + 4 r .. + 3 of the lane's four streamed rows of every tile.  Rows past n are zero (a copy of the last
// row times a weight of 0 would be NaN where that row has an infinity).
template <int D, int T> struct F32Cols { floatx4_t v[T][4][D / 64]; };

template <int D, int T>   // from memory; rows past n lie outside the buffer
__device__ __forceinline__ void f32_load_cols(F32Cols<D, T>& c, const float* __restrict__ base, int row0, int n, int r, int g) {
  const auto rows = __builtin_amdgcn_make_buffer_rsrc((void*)(base + (int64_t)row0 * D), 0, min(16 * T, n - row0) * D * 4, 0x00027000);
  const int lane_off = (4 * g * D + 4 * r) * 4;
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int p = 0; p < D / 64; ++p)
        c.v[t][i][p] = __builtin_bit_cast(floatx4_t, __builtin_amdgcn_raw_buffer_load_b128(rows, lane_off + ((16 * t + i) * D + 64 * p) * 4, 0, 0));
}

template <int D, int T>   // from the staged rows
__device__ __forceinline__ void f32_read_cols(F32Cols<D, T>& c, unsigned lds, int rows, int r, int g) {
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int p = 0; p < D / 64; ++p) c.v[t][i][p] = f32_lds(lds + 4 * g * D * 4 + ((r ^ f32_swizzle(4 * g + i)) << 4) + (16 * t + i) * D * 4 + p * 256);
  if (rows < 16 * T)   // a group's last step
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int p = 0; p < D / 64; ++p)
          if (16 * t + 4 * g + i >= rows) c.v[t][i][p] = floatx4_t{0.f, 0.f, 0.f, 0.f};
}

__device__ __forceinline__ void f32_wait_stage() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void f32_wait_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }   // before they are staged over

// acc = alpha acc + (streamed rows)^T x b.  The step's products are summed by themselves first.  In one chain over the group, whose
// waves take twice the rows of the 32-row kernels', the errors against float64 were up to a third larger than theirs (one group of
// 16,384 rows: O 1.14e-6 in the 2-norm, 0.83e-6 theirs, 0.38e-6 so; 512 rows: 3.5e-7, 3.2e-7, 3.1e-7).  Costs 2 % at D = 64, 4 at 128.
template <int D, int T>
__device__ __forceinline__ void f32_accumulate(floatx4_t (&acc)[D / 16], const F32Cols<D, T>& c, const floatx4_t (&b)[T], float alpha = 1.f) {
#pragma unroll
  for (int p = 0; p < D / 64; ++p) {
    floatx4_t sum[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] = f32_mfma(c.v[t][i][p][e], b[t][i], sum[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[4 * p + e][v] = fmaf(acc[4 * p + e][v], alpha, sum[e][v]);
  }
}

// Row constants of the streamed rows: lanes 0 .. 31 load lse, the others -delta, one value per row (past n: the last one's), and
// the wave hands them round through its LDS.
template <int T>
__device__ __forceinline__ float f32_load_stat(const float* __restrict__ lse, const float* __restrict__ neg_delta, int row0, int n, int lane) {
  return (lane < 32 ? lse : neg_delta)[min(row0 + lane % (16 * T), n - 1)];
}

__device__ __forceinline__ float f32_rows_max(float v) {   // over the four lanes of a stationary row
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f32_halves_max(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
}
__device__ __forceinline__ float f32_rows_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f32_halves_sum(__uint_as_float(a[0]) + __uint_as_float(a[1]));
}

// The waves' accumulators, one row of D channels (and 16 bytes against bank conflicts) per stationary row.
template <int D> struct F32Sums { __attribute__((aligned(16))) float v[kF32Waves][kF32Rows][D + 4]; };

// LDS of a block that stages `tensors` tensors and then holds as many sums.
template <int D>
constexpr int f32_lds_bytes(int tensors, int tile) {
  return tensors * (kF32Waves * tile > (int)sizeof(F32Sums<D>) ? kF32Waves * tile : (int)sizeof(F32Sums<D>));
}

template <int D>
__device__ __forceinline__ void f32_put(F32Sums<D>& s, const floatx4_t (&acc)[D / 16], int wave, int r, int g) {
#pragma unroll
  for (int p = 0; p < D / 64; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v)   // tile 4 p + e, row 4 g + v: channel 64 p + 4 (4 g + v) + e
      *(floatx4_t*)&s.v[wave][r][64 * p + 16 * g + 4 * v] = floatx4_t{acc[4 * p][v], acc[4 * p + 1][v], acc[4 * p + 2][v], acc[4 * p + 3][v]};
}

// Sixteen threads a row: four channels each, D / 64 times.  f: the waves' weights.
template <int D>
__device__ __forceinline__ void f32_write(const F32Sums<D>& s, const float (&f)[kF32Waves], float scale, float g, int row,
                                           float* __restrict__ out, float* __restrict__ tok) {
#pragma unroll
  for (int p = 0; p < D / 64; ++p) {
    const int c = 64 * p + 4 * (threadIdx.x & 15);
    floatx4_t q[kF32Waves];
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) q[w] = *(const floatx4_t*)&s.v[w][row][c] * f[w];
    const floatx4_t v = ((q[0] + q[1]) + (q[2] + q[3])) * scale;
    if (out) *(floatx4_t*)(out + c) = v;
    if (tok) *(floatx4_t*)(tok + c) = v * g;
  }
}

// Block -> (head, tile): false beyond the last tile.
__device__ __forceinline__ bool f32_find(const int32_t* __restrict__ cu, const int32_t* __restrict__ tile_start, int M, int block,
                                          int tiles_per_head, int& head, TileInfo& ti) {
  head = block / tiles_per_head;
  const int tile = block - head * tiles_per_head;
  return tile_start ? find_tile_presummed(tile_start, cu, M, kF32Rows, tile, ti) : find_tile(cu, M, kF32Rows, tile, ti);
}

// ---- forward ---------------------------------------------------------------------------
template <int D, int T>
__global__ __launch_bounds__(64 * kF32Waves, D == 64 ? 4 : 2) void attn_fwd_f32_kernel(
    const float* __restrict__ qh, const float* __restrict__ kh, const float* __restrict__ vh,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, int tiles_per_head, float* __restrict__ oh, float* __restrict__ lse,
    const int32_t* __restrict__ perm, const float* __restrict__ gate, float* __restrict__ o_tok) {
  constexpr int NW = kF32Waves, STEP = 16 * T;
  __shared__ __attribute__((aligned(1024))) unsigned char s_mem[f32_lds_bytes<D>(1, 16 * T * D * 4)];
  __shared__ float s_m[NW][16], s_l[NW][16];
  F32Sums<D>& s_o = *(F32Sums<D>*)s_mem;   // after the loop
  int head;
  TileInfo ti;
  if (!f32_find(cu_q, tile_start, M, blockIdx.x, tiles_per_head, head, ti)) return;
  const int gs = cu_k[ti.group], n = cu_k[ti.group + 1] - gs;   // keys of the group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t head_off = (int64_t)head * Nq;
  const float* kb = kh + ((int64_t)head * Nk + gs) * D;
  const float* vb = vh + ((int64_t)head * Nk + gs) * D;
  const float c = scale * 1.4426950408889634f;

  const unsigned lds = lds_addr_uniform(s_mem) + wave * (16 * T * D * 4);
  if (STEP * wave < n) f32_stage<D, T>(lds, kb, STEP * wave, n, lane);
  F32Frag<D> qf;
  f32_load<D>(qf, qh + (head_off + min(ti.tile_row + r, ti.row_end - 1)) * D, g);
  f32_settle(qf);
  floatx4_t o[D / 16];
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) o[dt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  for (int row0 = STEP * wave; row0 < n; row0 += STEP * NW) {
    F32Frag<D> kf[T];
    f32_wait_stage();
    f32_read_rows<D, T>(kf, lds, r, g);
    F32Cols<D, T> vf;
    f32_load_cols<D, T>(vf, vb, row0, n, r, g);   // in flight during the scores
    f32_wait_reads();
    if (row0 + STEP * NW < n) f32_stage<D, T>(lds, kb, row0 + STEP * NW, n, lane);
    floatx4_t p[T];
    f32_scores<D, T>(p, kf, qf);
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
    const float m_new = fmaxf(m, f32_rows_max(mx));
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
    f32_accumulate<D, T>(o, vf, p, alpha);
  }

  // common maximum of the waves (a wave without keys, or with none but scores of -inf, has m = -inf and weight 0)
  l = f32_rows_sum(l);
  __syncthreads();   // the staged rows' memory now takes the sums
  f32_put<D>(s_o, o, wave, r, g);
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
  f32_write<D>(s_o, f, n > 0 ? 1.f / lt : 0.f, o_tok ? gate[perm[j]] : 1.f, row, oh + (head_off + j) * D,
                f32_token_row<D>(o_tok, perm, j, head, H));
  if ((threadIdx.x & 15) == 0) lse[head_off + j] = n > 0 ? mt * scale + logf(lt) : -INFINITY;   // no keys: zero output, lse = -inf
}

// ---- backward: -delta = -rowsum(dO * O) comes from the caller ------------------------------
template <int D, int T>
__device__ __forceinline__ void f32_dq_block(
    unsigned char* s_mem, int block, const float* __restrict__ d_oh, const float* __restrict__ qh, const float* __restrict__ kh,
    const float* __restrict__ vh, const float* __restrict__ lse, const float* __restrict__ neg_delta, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M, int64_t Nq, int64_t Nk, int H, float scale,
    int tiles_per_head, float* __restrict__ d_qh, const int32_t* __restrict__ perm, float* __restrict__ d_q_tok) {
  constexpr int NW = kF32Waves, STEP = 16 * T, kTile = 16 * T * D * 4;
  int head;
  TileInfo ti;
  if (!f32_find(cu_q, tile_start, M, block, tiles_per_head, head, ti)) return;
  const int gs = cu_k[ti.group], n = cu_k[ti.group + 1] - gs;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t head_off = (int64_t)head * Nq;
  const float* kb = kh + ((int64_t)head * Nk + gs) * D;
  const float* vb = vh + ((int64_t)head * Nk + gs) * D;
  const int64_t own = head_off + min(ti.tile_row + r, ti.row_end - 1);
  F32Frag<D> qf, of;
  f32_load<D>(qf, qh + own * D, g);
  f32_load<D>(of, d_oh + own * D, g);
  const float lv = lse[own], ndl = neg_delta[own];
  floatx4_t dq[D / 16];
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) dq[dt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  const unsigned lds_k = lds_addr_uniform(s_mem) + wave * 2 * kTile, lds_v = lds_k + kTile;
  auto stage = [&](int row0) {
    f32_stage<D, T>(lds_k, kb, row0, n, lane);
    f32_stage<D, T>(lds_v, vb, row0, n, lane);
  };
  if (STEP * wave < n) stage(STEP * wave);
  f32_settle(qf);
  f32_settle(of);
  for (int row0 = STEP * wave; row0 < n; row0 += STEP * NW) {
    f32_wait_stage();
    F32Frag<D> kf[T], vf[T];
    F32Cols<D, T> kt;
    f32_read_rows<D, T>(kf, lds_k, r, g);
    f32_read_rows<D, T>(vf, lds_v, r, g);
    floatx4_t p[T], dp[T];
    f32_scores<D, T>(p, kf, qf);
    f32_scores<D, T>(dp, vf, of);
    f32_read_cols<D, T>(kt, lds_k, n - row0, r, g);
    f32_wait_reads();
    if (row0 + STEP * NW < n) stage(row0 + STEP * NW);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = f32_prob(p[t][i], scale, lv);
        p[t][i] = row0 + 16 * t + 4 * g + i < n ? e * (dp[t][i] + ndl) : 0.f;   // dS
      }
    f32_accumulate<D, T>(dq, kt, p);
  }
  F32Sums<D>& sums = *(F32Sums<D>*)s_mem;
  __syncthreads();   // the staged rows' memory now takes the sums
  f32_put<D>(sums, dq, wave, r, g);
  __syncthreads();
  const int row = threadIdx.x >> 4, j = ti.tile_row + row;
  if (j >= ti.row_end) return;
  const float one[NW] = {1.f, 1.f, 1.f, 1.f};
  f32_write<D>(sums, one, scale, 1.f, row, f32_sorted_row<D>(d_qh, head_off + j), f32_token_row<D>(d_q_tok, perm, j, head, H));
}

template <int D, int T>
__device__ __forceinline__ void f32_dkdv_block(
    unsigned char* s_mem, int block, const float* __restrict__ d_oh, const float* __restrict__ qh,
    const float* __restrict__ kh, const float* __restrict__ vh, const float* __restrict__ lse, const float* __restrict__ neg_delta,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M, int64_t Nq,
    int64_t Nk, int H, float scale, int tiles_per_head, float* __restrict__ d_kh, float* __restrict__ d_vh,
    const int32_t* __restrict__ perm, float* __restrict__ d_k_tok, float* __restrict__ d_v_tok) {
  constexpr int NW = kF32Waves, STEP = 16 * T, kTile = 16 * T * D * 4;
  int head;
  TileInfo ti;   // tiles run over the key rows of the groups
  if (!f32_find(cu_k, tile_start, M, block, tiles_per_head, head, ti)) return;
  const int gs = cu_q[ti.group], n = cu_q[ti.group + 1] - gs;   // queries of the group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int64_t head_off = (int64_t)head * Nk, q_off = (int64_t)head * Nq + gs;
  const float* qb = qh + q_off * D;
  const float* ob = d_oh + q_off * D;
  const int64_t own = head_off + min(ti.tile_row + r, ti.row_end - 1);
  F32Frag<D> kf, vf;
  f32_load<D>(kf, kh + own * D, g);
  f32_load<D>(vf, vh + own * D, g);
  floatx4_t dk[D / 16], dv[D / 16];
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) dk[dt] = dv[dt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  __shared__ __attribute__((aligned(16))) float s_stat[NW][2][32];
  const unsigned lds_q = lds_addr_uniform(s_mem) + wave * 2 * kTile, lds_o = lds_q + kTile;
  float stat = 0.f;
  auto stage = [&](int row0) {
    stat = f32_load_stat<T>(lse + q_off, neg_delta + q_off, row0, n, lane);
    f32_stage<D, T>(lds_q, qb, row0, n, lane);
    f32_stage<D, T>(lds_o, ob, row0, n, lane);
  };
  if (STEP * wave < n) stage(STEP * wave);
  f32_settle(kf);
  f32_settle(vf);
  for (int row0 = STEP * wave; row0 < n; row0 += STEP * NW) {
    f32_wait_stage();
    s_stat[wave][lane >> 5][lane & 31] = stat;
    asm volatile("" ::: "memory");
    F32Frag<D> qf[T], of[T];
    F32Cols<D, T> ot, qt;
    floatx4_t p[T], ds[T];
    f32_read_rows<D, T>(qf, lds_q, r, g);
    f32_read_rows<D, T>(of, lds_o, r, g);
    f32_scores<D, T>(p, qf, kf);
    f32_scores<D, T>(ds, of, vf);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const floatx4_t lv = *(const floatx4_t*)&s_stat[wave][0][16 * t + 4 * g], ndl = *(const floatx4_t*)&s_stat[wave][1][16 * t + 4 * g];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = f32_prob(p[t][i], scale, lv[i]);
        const bool valid = row0 + 16 * t + 4 * g + i < n;
        p[t][i] = valid ? e : 0.f;
        ds[t][i] = valid ? e * (ds[t][i] + ndl[i]) : 0.f;
      }
    }
    f32_read_cols<D, T>(ot, lds_o, n - row0, r, g);
    f32_read_cols<D, T>(qt, lds_q, n - row0, r, g);
    f32_wait_reads();
    if (row0 + STEP * NW < n) stage(row0 + STEP * NW);
    f32_accumulate<D, T>(dv, ot, p);
    f32_accumulate<D, T>(dk, qt, ds);
  }
  F32Sums<D>&s_dk = *(F32Sums<D>*)s_mem, &s_dv = ((F32Sums<D>*)s_mem)[1];
  __syncthreads();   // the staged rows' memory now takes the sums
  f32_put<D>(s_dv, dv, wave, r, g);
  f32_put<D>(s_dk, dk, wave, r, g);
  __syncthreads();
  const int row = threadIdx.x >> 4, j = ti.tile_row + row;
  if (j >= ti.row_end) return;
  const float one[NW] = {1.f, 1.f, 1.f, 1.f};
  f32_write<D>(s_dv, one, 1.f, 1.f, row, f32_sorted_row<D>(d_vh, head_off + j), f32_token_row<D>(d_v_tok, perm, j, head, H));
  f32_write<D>(s_dk, one, scale, 1.f, row, f32_sorted_row<D>(d_kh, head_off + j), f32_token_row<D>(d_k_tok, perm, j, head, H));
}

// Blocks below `k_blocks` are dK/dV's (four products to three: the longer ones first), the others dQ's.
template <int D, int T>
__global__ __launch_bounds__(64 * kF32Waves, D == 64 && T == 1 ? 3 : 2) void attn_bwd_f32_kernel(
    const float* __restrict__ d_oh, const float* __restrict__ qh, const float* __restrict__ kh, const float* __restrict__ vh,
    const float* __restrict__ lse, const float* __restrict__ neg_delta, const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k,
    const int32_t* __restrict__ ts_q, const int32_t* __restrict__ ts_k, int M, int64_t Nq, int64_t Nk, int H, float scale, int q_tiles,
    int k_tiles, int k_blocks, float* __restrict__ d_qh, float* __restrict__ d_kh, float* __restrict__ d_vh,
    const int32_t* __restrict__ perm, float* __restrict__ d_q_tok, float* __restrict__ d_k_tok, float* __restrict__ d_v_tok) {
  __shared__ __attribute__((aligned(1024))) unsigned char s_mem[f32_lds_bytes<D>(2, 16 * T * D * 4)];
  if ((int)blockIdx.x < k_blocks)
    f32_dkdv_block<D, T>(s_mem, blockIdx.x, d_oh, qh, kh, vh, lse, neg_delta, cu_q, cu_k, ts_k, M, Nq, Nk, H, scale, k_tiles, d_kh,
                       d_vh, perm, d_k_tok, d_v_tok);
  else
    f32_dq_block<D, T>(s_mem, blockIdx.x - k_blocks, d_oh, qh, kh, vh, lse, neg_delta, cu_q, cu_k, ts_q, M, Nq, Nk, H, scale, q_tiles, d_qh,
                     perm, d_q_tok);
}

}  // namespace moga
