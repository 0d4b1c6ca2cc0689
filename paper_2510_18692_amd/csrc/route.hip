// Token router of MoGA (Eqs. 2-4 of the paper) and its backward through the gate of Eq. 5.
//
//   logits = X W^T, probs = softmax(logits), group = argmax, gate = probs[group].
//
// Two forward kernels:
//   * route_mfma_kernel: bf16 X.  logits^T = W X^T on bf16 MFMA with fp32-GEMM semantics:
//     each fp32 weight is split exactly into three bf16 limbs (hi + mid + lo == w), every
//     limb product with a bf16 activation is exact in fp32, and only the accumulation
//     rounds.  Groups are the MFMA rows and tokens the columns, so a lane ends up holding
//     half of one token's logits: argmax / softmax need one exchange between wave halves.
//   * route_generic_kernel: any dtype / shape; one wave per token, fp32 FMA.
// Backward: dr = d_gate * gate * (onehot(group) - probs), dW = dr^T X on bf16 MFMA (dr split in two
// bf16 limbs) for bf16 X, else with fp32 FMAs; optional dX = dr W.
#include <algorithm>

#include "lds_pipe.h"

namespace moga {

// ---------------------------------------------------------------------------------------
// generic: one wave per token
// ---------------------------------------------------------------------------------------
template <typename XT> __device__ __forceinline__ float load_x(const XT* p);
template <> __device__ __forceinline__ float load_x<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float load_x<unsigned short>(const unsigned short* p) {
  return bf16_bits_to_f32(*p);
}

constexpr int64_t kGenericTokens = (int64_t)1 << 25;   // of a launch: 64 threads each, 2^32 are too many

template <typename XT>
__global__ __launch_bounds__(256) void route_generic_kernel(
    const XT* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias,
    int64_t N, int d, int M, int32_t* __restrict__ group, float* __restrict__ gate,
    float* __restrict__ probs, float* __restrict__ logits) {
  __shared__ float s_logit[4][MOGA_MAX_GROUPS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int64_t tok = (int64_t)blockIdx.x * 4 + wave;
  const bool valid = tok < N;
  if (!valid) tok = N - 1;
  const XT* xr = x + tok * (int64_t)d;

  for (int j0 = 0; j0 < M; j0 += 8) {
    float acc[8];
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) acc[jj] = 0.f;
    for (int c = lane; c < d; c += 64) {
      const float xv = load_x<XT>(xr + c);
#pragma unroll
      for (int jj = 0; jj < 8; ++jj) {
        const int j = min(j0 + jj, M - 1);
        acc[jj] = fmaf(xv, w[(int64_t)j * d + c], acc[jj]);
      }
    }
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
      const float r = wave_sum(acc[jj]);
      if (lane == jj && j0 + jj < M) s_logit[wave][j0 + jj] = r + (bias ? bias[j0 + jj] : 0.f);
    }
  }
  __syncthreads();

  // argmax (lowest index on ties) and softmax over the M logits of this wave's token
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int j = lane; j < M; j += 64) {
    const float r = s_logit[wave][j];
    if (r > best) { best = r; bi = j; }
  }
  const float top = wave_max(best);
  bi = lanes_reduce<64>(best == top ? bi : 0x7fffffff, [](int a, int b) { return a < b ? a : b; });
  best = top;
  float sum = 0.f;
  for (int j = lane; j < M; j += 64) sum += expf(s_logit[wave][j] - best);
  sum = wave_sum(sum);
  const float g = 1.f / sum;
  if (valid) {
    if (lane == 0) { group[tok] = bi; gate[tok] = g; }
    for (int j = lane; j < M; j += 64) {
      const float r = s_logit[wave][j];
      if (probs) probs[tok * M + j] = expf(r - best) * g;
      if (logits) logits[tok * M + j] = r;
    }
  }
}

// ---------------------------------------------------------------------------------------
// bf16 MFMA path (M <= 32, d_model % 64 == 0)
// ---------------------------------------------------------------------------------------
constexpr int kRouteKC = 128;              // k-chunk of W staged in LDS (two 64-wide k blocks)
constexpr int kRouteStride = kRouteKC + 8; // bf16 elements per LDS row (+16 B against bank conflicts)
// float4 loads of W per thread and chunk in a block of NWV waves
template <int NWV> constexpr int kRouteWLoads = 32 * (kRouteKC / 4) / (64 * NWV);

// Split an fp32 value into three bf16 limbs whose sum is exactly the value.
__device__ __forceinline__ void split3(float w, unsigned short& hi, unsigned short& mid,
                                       unsigned short& lo) {
  hi = f32_to_bf16_bits(w);
  const float r1 = w - bf16_bits_to_f32(hi);
  mid = f32_to_bf16_bits(r1);
  const float r2 = r1 - bf16_bits_to_f32(mid);
  lo = f32_to_bf16_bits(r2);
}

// One thread's share of a weight chunk: rows of W beyond M and columns beyond d read as zero.
template <int NWV>
__device__ __forceinline__ void route_load_w(const float* __restrict__ w, int d, int M, int k0,
                                             floatx4_t (&wv)[kRouteWLoads<NWV>]) {
#pragma unroll
  for (int i = 0; i < kRouteWLoads<NWV>; ++i) {
    const int idx = threadIdx.x + 64 * NWV * i;
    const int row = idx / (kRouteKC / 4), c = (idx % (kRouteKC / 4)) * 4;
    const floatx4_t z = {0.f, 0.f, 0.f, 0.f};
    wv[i] = (row < M && k0 + c < d) ? *(const floatx4_t*)(w + (int64_t)row * d + k0 + c) : z;
  }
}

template <int NWV>
__device__ __forceinline__ void route_store_w(unsigned short (&sw)[3][32][kRouteStride],
                                              const floatx4_t (&wv)[kRouteWLoads<NWV>]) {
#pragma unroll
  for (int i = 0; i < kRouteWLoads<NWV>; ++i) {
    const int idx = threadIdx.x + 64 * NWV * i;
    const int row = idx / (kRouteKC / 4), c = (idx % (kRouteKC / 4)) * 4;
    unsigned short hi[4], mid[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split3(wv[i][e], hi[e], mid[e], lo[e]);
    const uintx2_t ph = {hi[0] | ((unsigned)hi[1] << 16), hi[2] | ((unsigned)hi[3] << 16)};
    const uintx2_t pm = {mid[0] | ((unsigned)mid[1] << 16), mid[2] | ((unsigned)mid[3] << 16)};
    const uintx2_t pl = {lo[0] | ((unsigned)lo[1] << 16), lo[2] | ((unsigned)lo[3] << 16)};
    *(uintx2_t*)&sw[0][row][c] = ph;
    *(uintx2_t*)&sw[1][row][c] = pm;
    *(uintx2_t*)&sw[2][row][c] = pl;
  }
}

// A 64-wide k block of X as a wave's MFMA B operands: lane half h holds elements [32h, 32h+32) of
// its token's row as four 16-byte pieces; piece s feeds MFMA k-step s (the weight operand uses
// the same map).
template <int TT>
struct RouteXBlock {
  uintx4_t v[TT][4];
};

template <int TT>
__device__ __forceinline__ void route_load_x(RouteXBlock<TT>& b, const unsigned short* const (&xrow)[TT],
                                             int koff) {
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int s = 0; s < 4; ++s) b.v[t][s] = *(const uintx4_t*)(xrow[t] + koff + 8 * s);
}

template <int TT>
__device__ __forceinline__ void route_mfma_block(floatx16_t (&acc)[TT],
                                                 const unsigned short (&sw)[3][32][kRouteStride],
                                                 int col0, int r, int h, const RouteXBlock<TT>& b) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int limb = 0; limb < 3; ++limb) {
      const bf16x8_t a = *(const bf16x8_t*)&sw[limb][r][col0 + 32 * h + 8 * s];
#pragma unroll
      for (int t = 0; t < TT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            a, __builtin_bit_cast(bf16x8_t, b.v[t][s]), acc[t], 0, 0, 0);
    }
  }
}

// argmax, softmax and stores of one 32-token tile: accumulator register v of lane (r, h) is group row 8*(v/4) + 4*h + v%4 of
// token `tok`, the tile's r-th.
__device__ __forceinline__ void route_finish(const floatx16_t& total, int64_t tok, int h, const float* __restrict__ bias, int64_t N,
                                             int M, int32_t* __restrict__ group, float* __restrict__ gate, float* __restrict__ probs,
                                             float* __restrict__ logits) {
  const bool vec4 = (M & 3) == 0 && (((uintptr_t)probs | (uintptr_t)logits) & 15) == 0;
  float vals[16];
  float best = -INFINITY;
  int bi = 0x7fffffff;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = 8 * (v >> 2) + 4 * h + (v & 3);
    float val = total[v];
    if (row < M) {
      if (bias) val += bias[row];
    } else {
      val = -INFINITY;
    }
    vals[v] = val;
    if (val > best) { best = val; bi = row; }
  }
  const float ob = other_half(best);
  const int oi = other_half_i(bi);
  if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
  float sum = 0.f;
  float e[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) { e[v] = expf(vals[v] - best); sum += e[v]; }
  sum += other_half(sum);
  const float g = 1.f / sum;
  if (tok < N) {
    if (h == 0) { group[tok] = bi; gate[tok] = g; }
    if (vec4) {   // a lane's registers 4q .. 4q+3 are four consecutive groups: one 16-byte store
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = 8 * q + 4 * h;
        if (row < M) {
          if (probs) {
            const floatx4_t pv = {e[4 * q] * g, e[4 * q + 1] * g, e[4 * q + 2] * g, e[4 * q + 3] * g};
            *(floatx4_t*)(probs + tok * M + row) = pv;
          }
          if (logits) {
            const floatx4_t lv = {vals[4 * q], vals[4 * q + 1], vals[4 * q + 2], vals[4 * q + 3]};
            *(floatx4_t*)(logits + tok * M + row) = lv;
          }
        }
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = 8 * (v >> 2) + 4 * h + (v & 3);
        if (row < M) {
          if (probs) probs[tok * M + row] = e[v] * g;
          if (logits) logits[tok * M + row] = vals[v];
        }
      }
    }
  }
}

// Few tokens: a block per 32 tokens, whose waves share the k blocks (wave w takes w, w + NWV, ..) and add their logits through
// LDS.  The kernel below has 128 tokens per block and walks all of W with a barrier per chunk: at 1,560 tokens its 13 blocks took
// as long as a full chip.  A wave's k block of W (fp32) and of X goes to its own LDS with direct-to-LDS loads, whole rows of 256
// and 128 bytes at a time, and is read from there as operands: straight from memory every lane would touch a cache line of its
// own in each of twelve loads (10,007 x 1536, 20 groups: 17.1 us).  16-byte chunks are XOR-swizzled by the row so that the reads
// hit all banks.  W is split into its limbs in registers.  The other kernel's time and this one's, in us: 1,560 x 512, 8 groups
// 9.5 and 5.1; 1,560 x 1536, 16 groups 18.6 and 8.1; 10,007 x 1536, 20 groups 19.1 and 11.7; 8,192 x 5120, 16 groups 60 and 23;
// 16,384 x 1536, 8 groups 21.7 and 13.8 (3.6 TB/s).  A block alone on its CU waits for its waves' own chains (splitting W, twelve dependent
// products a k block; two more k blocks in flight: 1 us slower): eight waves instead of four where a CU has one block and they have many
// k blocks, 1,253 x 5120, 4 groups 17.6 -> 15.4, 5,225 x 5120, 20 groups 19.3 -> 17.3, but 8,192 x 5120, 16 groups 20.6 and 20.8, 1,560 x 1536 8.3
// and 8.1, 10,007 x 1536 11.9 and 15.0.
constexpr int kFewW = 32 * 256, kFewX = 32 * 128;   // bytes of a wave's k block

template <int NWV>
__global__ __launch_bounds__(64 * NWV, NWV == 4 ? 3 : 1) void route_mfma_few_kernel(
    const unsigned short* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias, int64_t N, int d, int M,
    int32_t* __restrict__ group, float* __restrict__ gate, float* __restrict__ probs, float* __restrict__ logits) {
  __shared__ __attribute__((aligned(1024))) unsigned char s_k[NWV][kFewW + kFewX];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int64_t tok0 = (int64_t)blockIdx.x * 32;
  const void* xb = uniform_ptr(x + tok0 * d);
  const void* wb = uniform_ptr(w);
  const int last = (int)min((int64_t)31, N - 1 - tok0);
  const unsigned lds = lds_addr_uniform(&s_k[0][0]) + wave * (kFewW + kFewX);
  auto issue = [&](int k0) {   // rows of W beyond M and of X beyond N: the last one, not used
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int row = 4 * q + (lane >> 4), chunk = (lane & 15) ^ (row & 15);
      lds_dma16_soff(wb, (unsigned)((min(row, M - 1) * d + k0 + 4 * chunk) * 4), lds + q * 1024);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = 8 * q + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
      lds_dma16_soff(xb, (unsigned)((min(row, last) * d + k0 + 8 * chunk) * 2), lds + kFewW + q * 1024);
    }
  };
  // lane half h takes elements 32 h .. 32 h + 31 of its rows' k block
  unsigned wa[8], xa[4];
#pragma unroll
  for (int s = 0; s < 8; ++s) wa[s] = lds + r * 256 + (((8 * h + s) ^ (r & 15)) << 4);
#pragma unroll
  for (int s = 0; s < 4; ++s) xa[s] = lds + kFewW + r * 128 + (((4 * h + s) ^ ((r >> 1) & 7)) << 4);

  floatx16_t total;
#pragma unroll
  for (int v = 0; v < 16; ++v) total[v] = 0.f;
  if (64 * wave < d) issue(64 * wave);
  for (int k0 = 64 * wave; k0 < d; k0 += 64 * NWV) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uintx4_t xv[4];
    floatx4_t wv[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) wv[s] = *(const floatx4_t __attribute__((address_space(3)))*)(uintptr_t)wa[s];
#pragma unroll
    for (int s = 0; s < 4; ++s) xv[s] = *(const uintx4_t __attribute__((address_space(3)))*)(uintptr_t)xa[s];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the next block overwrites it
    if (k0 + 64 * NWV < d) issue(k0 + 64 * NWV);
    floatx16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uintx4_t limb[3];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float w0 = wv[2 * s + (e >> 1)][2 * (e & 1)], w1 = wv[2 * s + (e >> 1)][2 * (e & 1) + 1];
        if (r >= M) w0 = w1 = 0.f;
#pragma unroll
        for (int l = 0; l < 3; ++l) {   // as split3: what is left after each limb is exact
          limb[l][e] = pack_bf16x2(w0, w1);
          w0 -= bf16_lo_to_f32(limb[l][e]);
          w1 -= bf16_hi_to_f32(limb[l][e]);
        }
      }
#pragma unroll
      for (int l = 0; l < 3; ++l)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, limb[l]), __builtin_bit_cast(bf16x8_t, xv[s]), acc, 0, 0, 0);
    }
    total += acc;   // short chains
  }
  __syncthreads();   // the k blocks' memory now takes the waves' logits
  float (*s_tot)[16][64] = (float (*)[16][64])&s_k[0][0];
#pragma unroll
  for (int v = 0; v < 16; ++v) s_tot[wave][v][lane] = total[v];
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int v = 0; v < 16; ++v)
#pragma unroll
    for (int k = 1; k < NWV; ++k) total[v] += s_tot[k][v][lane];
  route_finish(total, tok0 + r, h, bias, N, M, group, gate, probs, logits);
}

// The other kernel's blocks of 128 tokens run 256 at a time; it is the better one where their last round is well filled, from an
// earlier point on where a token brings few channels.  Its time and that of the kernel above in us: 24,000 tokens x 1536, 20 groups 20.9
// and 18.7, x 128, 8 groups 7.1 and 5.8; 28,672 x 1536 21.5 and 21.9, x 5120, 32 groups 71 and 80, x 128 7.1 and 8.0; 35,000 x 1536
// 34.3 and 25.6, x 512 15.1 and 12.5, x 128 8.9 and 9.0; 50,000 x 128 8.9 and 11.0, x 512 15.7 and 17.0, x 1536 34.6 and 33.2;
// 53,000 x 5120, 16 groups 135 and 125, 32 groups 143 and 148.
inline bool use_route_few(int64_t N, int d_model, int M) {
  if (d_model > (1 << 20)) return false;   // 32-bit offsets within W
  const int64_t blocks = (N + 127) / 128;
  if (blocks <= 256) return blocks <= 192;
  return d_model >= 256 && blocks > 257 && blocks <= (d_model >= 2560 && M <= 20 ? 448 : 384);
}

// The weight chunk is double-buffered: while the matrix cores work on chunk c, the fp32 weights of
// chunk c+1 are in flight from L2; they are split and stored after the chunk's MFMAs, one block
// barrier per chunk.  X lives in a ring of four k-block register sets with fixed roles (the loop
// is unrolled over two chunks, so no set is ever copied): a set is refilled, four k blocks ahead,
// right after its MFMAs, which keeps 16-32 KB of loads per wave in flight across the barriers.
template <int TT, int NWV>  // 32-token tiles per wave, waves per block
__global__ __launch_bounds__(64 * NWV, 2) void route_mfma_kernel(
    const unsigned short* __restrict__ x, const float* __restrict__ w,
    const float* __restrict__ bias, int64_t N, int d, int M, int32_t* __restrict__ group,
    float* __restrict__ gate, float* __restrict__ probs, float* __restrict__ logits) {
  __shared__ __attribute__((aligned(16))) unsigned short s_w[2][3][32][kRouteStride];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int64_t tok0 = ((int64_t)blockIdx.x * NWV + wave) * (32 * TT);

  const unsigned short* xrow[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    int64_t tok = tok0 + 32 * t + r;
    if (tok > N - 1) tok = N - 1;
    xrow[t] = x + tok * (int64_t)d + 32 * h;
  }

  floatx16_t total[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) total[t][v] = 0.f;

  // k blocks past the end of the row are clamped to the last one (loaded, never used)
  const int last_kb = d - 64;
  RouteXBlock<TT> b0, b1, b2, b3;
  route_load_x<TT>(b0, xrow, 0);
  route_load_x<TT>(b1, xrow, min(64, last_kb));
  route_load_x<TT>(b2, xrow, min(128, last_kb));
  route_load_x<TT>(b3, xrow, min(192, last_kb));
  floatx4_t wv[kRouteWLoads<NWV>];
  route_load_w<NWV>(w, d, M, 0, wv);
  route_store_w<NWV>(s_w[0], wv);
  __syncthreads();

  const int nchunks = (d + kRouteKC - 1) / kRouteKC;
  // One chunk: k blocks (BA, BB) against weight buffer BUF.
#define MOGA_ROUTE_CHUNK(BA, BB, BUF, C)                                          \
  {                                                                                \
    const int k0 = (C) * kRouteKC;                                                 \
    const bool more = (C) + 1 < nchunks;                                           \
    if (more) route_load_w<NWV>(w, d, M, k0 + kRouteKC, wv);                         \
    floatx16_t acc[TT];                                                            \
    _Pragma("unroll") for (int t = 0; t < TT; ++t)                                 \
      _Pragma("unroll") for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;              \
    route_mfma_block<TT>(acc, s_w[BUF], 0, r, h, BA);                              \
    route_load_x<TT>(BA, xrow, min(k0 + 256, last_kb));                            \
    if (k0 + 64 < d) route_mfma_block<TT>(acc, s_w[BUF], 64, r, h, BB);            \
    route_load_x<TT>(BB, xrow, min(k0 + 320, last_kb));                            \
    _Pragma("unroll") for (int t = 0; t < TT; ++t)                                 \
      _Pragma("unroll") for (int v = 0; v < 16; ++v) total[t][v] += acc[t][v];     \
    if (more) route_store_w<NWV>(s_w[(BUF) ^ 1], wv);                                \
    __syncthreads();                                                               \
  }
  for (int c = 0; c < nchunks; c += 2) {
    MOGA_ROUTE_CHUNK(b0, b1, 0, c)
    if (c + 1 < nchunks) MOGA_ROUTE_CHUNK(b2, b3, 1, c + 1)
  }
#undef MOGA_ROUTE_CHUNK

#pragma unroll
  for (int t = 0; t < TT; ++t) route_finish(total[t], tok0 + 32 * t + r, h, bias, N, M, group, gate, probs, logits);
}

// ---------------------------------------------------------------------------------------
// backward: dr = d_gate * gate * (onehot(group) - probs);  dW = dr^T X;  dX = dr W
// ---------------------------------------------------------------------------------------
// The gate's gradient: d_gate, and with frac the balancing loss's, rounded as moga_balance_loss_bwd adds it.
struct GateGrad {
  const float* d_gate;
  const float* frac;
  float coef;
  const float* d_loss;   // or NULL: on the device
};
__device__ __forceinline__ float gate_grad(const GateGrad& gg, int64_t tok, int g, int M) {
  const float d = gg.d_gate[tok];
  if (!gg.frac) return d;
  const float c = gg.d_loss ? gg.coef * gg.d_loss[0] : gg.coef;
  return d + (g >= 0 && g < M ? c * gg.frac[g] : 0.f);
}

constexpr int kRbTok = 64;  // tokens per staged tile
constexpr int kRbMB = 32;   // groups per pass

// dW for fp32 X and for shapes the matrix-core path below does not cover, with fp32 FMAs.  A block takes
// 64 columns and a range of tokens; its four waves take 16 tokens each of every 64-token tile, a lane one
// column with all MB groups, and are added through LDS at the end.  The 16 activations of a tile are
// loaded together (one round trip per tile), dr comes from LDS as broadcast 16-byte pieces.  The token
// range is cut until about a thousand blocks exist or a block has a single tile: with one thread per
// column and 2,048 tokens per block, 4,096 x 128 x 8 groups ran on two blocks (437 us for the call, 16 us now).
template <typename XT, int MB>
__global__ __launch_bounds__(256) void route_bwd_dw_partial_kernel(
    const XT* __restrict__ x, const float* __restrict__ probs, const int32_t* __restrict__ group,
    const float* __restrict__ gate, GateGrad gg, int64_t N, int d, int M,
    int64_t tokens_per_split, float* __restrict__ partial /* [splits][M][d] */) {
  constexpr int WT = kRbTok / 4;   // tokens per wave and tile
  __shared__ __attribute__((aligned(16))) float s_dr[kRbTok][MB];
  __shared__ float s_acc[3][MB][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c = blockIdx.x * 64 + lane;
  const int split = blockIdx.y;
  const int j0 = blockIdx.z * MB;
  const int mb = min(MB, M - j0);
  const int64_t t0 = (int64_t)split * tokens_per_split;
  const int64_t t1 = min(N, t0 + tokens_per_split);
  const XT* xc = x + min(c, d - 1);
  float acc[MB];
#pragma unroll
  for (int j = 0; j < MB; ++j) acc[j] = 0.f;

  for (int64_t tb = t0; tb < t1; tb += kRbTok) {
    float xv[WT];   // tokens past the end of the range have dr = 0 and x = 0 (not a copy: 0 times an infinity is NaN)
#pragma unroll
    for (int i = 0; i < WT; ++i) {
      const int64_t tok = tb + WT * wave + i;
      xv[i] = load_x<XT>(xc + min(tok, t1 - 1) * d);
      if (tok >= t1) xv[i] = 0.f;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < kRbTok * MB; idx += 256) {
      const int ti = idx / MB, j = idx % MB;
      float v = 0.f;
      if (tb + ti < t1 && j < mb) {
        const int64_t tok = tb + ti;
        const int g = group[tok];
        const float coef = gate_grad(gg, tok, g, M) * gate[tok];
        const float onehot = (g == j0 + j) ? 1.f : 0.f;
        v = coef * (onehot - probs[tok * M + j0 + j]);
      }
      s_dr[ti][j] = v;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int j4 = 0; j4 < MB; j4 += 4) {
        const floatx4_t dr = *(const floatx4_t*)&s_dr[WT * wave + i][j4];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j4 + e] = fmaf(dr[e], xv[i], acc[j4 + e]);
      }
  }
  if (wave > 0)
#pragma unroll
    for (int j = 0; j < MB; ++j) s_acc[wave - 1][j][lane] = acc[j];
  __syncthreads();
  if (wave == 0 && c < d)
#pragma unroll
    for (int j = 0; j < MB; ++j)
      if (j < mb)
        partial[((int64_t)split * M + j0 + j) * d + c] = (acc[j] + s_acc[0][j][lane]) + (s_acc[1][j][lane] + s_acc[2][j][lane]);
}

// dW of up to 65,536 tokens (where the matrix-core path below applies; route_bwd_few_plan has the lines): a block takes 64 columns and a run of tokens, its
// sixteen waves every sixteenth 16 of them, and they are added through LDS at the end; the sums of several blocks by
// route_bwd_dw_reduce_kernel.  dr is made in registers, in two bf16 limbs as in route_bwd_dr_pack_kernel, as the A operand (groups x
// tokens) of the 32x32x16 matrix instruction; X is the B operand: a lane loads columns 2 r and 2 r + 1 of eight tokens, one column for
// each of two accumulators, 64 KB of a CU's loads in flight.  The three launches of that path against this one, in us: 64 x 512, 8 groups
// 10.3 and 4.6; 390 x 1536, 8 groups 12.3 and 4.9; split over blocks, 5,000 x 1536, 20 groups 17.5 and 8.7; 10,007 x 1536, 20 groups
// 19.5 and 13.1 (2.3 TB/s of X); 16,384 x 512, 8 groups 15.1 and 8.3; 32,760 x 1536, 20 groups 32.3 and 26.5 (3.8 TB/s); 10,007 x 5120, 32
// groups 33.5 and 27.3.
constexpr int kDwFewWaves = 16, kDwFewTok = 16;   // waves per block, tokens per run
constexpr int kDwFewTokens = 8192;                // of one block

__global__ __launch_bounds__(64 * kDwFewWaves) void route_bwd_dw_few_kernel(
    const unsigned short* __restrict__ x, const float* __restrict__ probs, const int32_t* __restrict__ group, const float* __restrict__ gate,
    GateGrad gg, int64_t n_all, int tokens, int d, int M, float* __restrict__ out) {
  constexpr int STEP = kDwFewTok * kDwFewWaves;
  typedef float Acc[2][16][64];
  __shared__ __attribute__((aligned(16))) unsigned char s_mem[kDwFewWaves * sizeof(Acc)];
  float* s_coef = (float*)s_mem;                         // of the block's tokens, 0 past the end
  int* s_group = (int*)s_mem + kDwFewTokens;
  Acc* s_acc = (Acc*)s_mem;                              // after the loop
  static_assert(8 * kDwFewTokens <= (int)sizeof(s_mem));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int64_t first_tok = (int64_t)blockIdx.y * tokens;
  const int N = (int)min((int64_t)tokens, n_all - first_tok);   // the block's tokens
  x += first_tok * d;
  probs += first_tok * M;
  const unsigned short* xc = x + 64 * blockIdx.x + 2 * r;
  const float* pc = probs + min(r, M - 1);
  struct Run {
    unsigned x[8];
    float p[8];
  };
  auto load = [&](Run& b, int t0) {   // tokens past the end: the last one, not used
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int tok = min(t0 + 8 * h + e, N - 1);
      b.x[e] = *(const unsigned*)(xc + (int64_t)tok * d);
      b.p[e] = pc[tok * M];
    }
  };
  Run cur, next;
  const int first = kDwFewTok * wave;
  if (first < N) load(cur, first);
  for (int t = threadIdx.x; t < (N + kDwFewTok - 1) / kDwFewTok * kDwFewTok; t += 64 * kDwFewWaves) {
    const int g = t < N ? group[first_tok + t] : -1;
    s_coef[t] = t < N ? gate_grad(gg, first_tok + t, g, M) * gate[first_tok + t] : 0.f;
    s_group[t] = g;
  }
  __syncthreads();
  floatx16_t acc[2];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
  for (int t0 = first; t0 < N; t0 += STEP) {
    load(next, t0 + STEP);
    uintx4_t hi, lo, xe, xo;
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      const floatx4_t coef = *(const floatx4_t*)&s_coef[t0 + 8 * h + e];
      const uintx4_t g = *(const uintx4_t*)&s_group[t0 + 8 * h + e];
      float v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float onehot = (int)g[k] == r ? 1.f : 0.f;
        v[k] = coef[k] * (onehot - cur.p[e + k]);
        if (r >= M || t0 + 8 * h + e + k >= N) v[k] = 0.f;
      }
#pragma unroll
      for (int k = 0; k < 4; k += 2) {
        const unsigned top = pack_bf16x2(v[k], v[k + 1]);
        hi[(e + k) / 2] = top;
        lo[(e + k) / 2] = pack_bf16x2(v[k] - bf16_lo_to_f32(top), v[k + 1] - bf16_hi_to_f32(top));
      }
    }
    if (t0 + kDwFewTok > N)   // not a copy of the last row: 0 times an infinity is NaN
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (t0 + 8 * h + e >= N) cur.x[e] = 0u;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      xe[e / 2] = __builtin_amdgcn_perm(cur.x[e + 1], cur.x[e], 0x05040100u);
      xo[e / 2] = __builtin_amdgcn_perm(cur.x[e + 1], cur.x[e], 0x07060302u);
    }
    const bf16x8_t a0 = __builtin_bit_cast(bf16x8_t, hi), a1 = __builtin_bit_cast(bf16x8_t, lo);
    const bf16x8_t b0 = __builtin_bit_cast(bf16x8_t, xe), b1 = __builtin_bit_cast(bf16x8_t, xo);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b1, acc[1], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b0, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, acc[1], 0, 0, 0);
    cur = next;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) s_acc[wave][c][v][lane] = acc[c][v];
  __syncthreads();
  // wave w: register w of both accumulators, group 8 (w / 4) + 4 h + w % 4, columns 2 r and 2 r + 1
  floatx2_t sum = {0.f, 0.f};
#pragma unroll
  for (int k = 0; k < kDwFewWaves; ++k) {
    sum[0] += s_acc[k][0][wave][lane];
    sum[1] += s_acc[k][1][wave][lane];
  }
  const int j = 8 * (wave >> 2) + 4 * h + (wave & 3);
  if (j < M) *(floatx2_t*)(out + ((int64_t)blockIdx.y * M + j) * d + 64 * blockIdx.x + 2 * r) = sum;
}

// Sum of the splits, in a fixed order: 64 elements per block, eight waves that take every eighth split
// each with eight loads in flight, then a sum over the waves.  (One thread per element took 59 us for the
// 50 MB of 256 splits at d = 1536; the call at 62,400 x 1536, M = 5 went from 105 to 48 us with this and
// with the groups rounded up to 8 instead of 32.)  Element i of a split is (j, c) = (i / d,
// i % d), or for the matrix-core path (TRANSPOSED) (c, j) = (i / mp, i % mp).
template <bool TRANSPOSED>
__global__ __launch_bounds__(512) void route_bwd_dw_reduce_kernel(const float* __restrict__ partial, int splits, int64_t n,
                                                                  int d, int M, int mp, float* __restrict__ d_w) {
  __shared__ float s_sum[8][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const float* p = partial + min(i, n - 1);
  float s = 0.f;
#pragma unroll 8
  for (int k = wave; k < splits; k += 8) s += p[(int64_t)k * n];
  s_sum[wave][lane] = s;
  __syncthreads();
  if (wave != 0 || i >= n) return;
  s = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) s += s_sum[w][lane];
  if (!TRANSPOSED) {
    d_w[i] = s;
  } else {
    const int c = (int)(i / mp), j = (int)(i - (int64_t)c * mp);
    if (j < M) d_w[(int64_t)j * d + c] = s;
  }
}

// dX as fp32 or rounded to bf16: 4 or 8 adjacent columns of a row leave as one store of 8 or 16 bytes.
template <int COLS>
__device__ __forceinline__ void store_dx(float* p, const float (&v)[COLS]) {
#pragma unroll
  for (int i = 0; i < COLS; i += 4) *(floatx4_t*)(p + i) = floatx4_t{v[i], v[i + 1], v[i + 2], v[i + 3]};
}
template <int COLS>
__device__ __forceinline__ void store_dx(unsigned short* p, const float (&v)[COLS]) {
  unsigned u[COLS / 2];
#pragma unroll
  for (int i = 0; i < COLS; i += 2) u[i / 2] = pack_bf16x2(v[i], v[i + 1]);
  if constexpr (COLS == 8) *(uintx4_t*)p = uintx4_t{u[0], u[1], u[2], u[3]};
  else *(uintx2_t*)p = uintx2_t{u[0], u[1]};
}
__device__ __forceinline__ void store_dx1(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_dx1(unsigned short* p, float v) { *p = f32_to_bf16_bits(v); }

template <typename OT>
__global__ __launch_bounds__(256) void route_bwd_dx_kernel(
    const float* __restrict__ w, const float* __restrict__ probs,
    const int32_t* __restrict__ group, const float* __restrict__ gate,
    GateGrad gg, int64_t N, int d, int M, OT* __restrict__ d_x) {
  __shared__ float s_dr[kRbTok][kRbMB];
  const int c = blockIdx.y * 256 + threadIdx.x;
  const int64_t tb = (int64_t)blockIdx.x * kRbTok;
  const int nt = (int)min((int64_t)kRbTok, N - tb);
  float out[kRbTok];
#pragma unroll
  for (int ti = 0; ti < kRbTok; ++ti) out[ti] = 0.f;
  for (int j0 = 0; j0 < M; j0 += kRbMB) {
    const int mb = min(kRbMB, M - j0);
    __syncthreads();
    for (int idx = threadIdx.x; idx < kRbTok * kRbMB; idx += 256) {
      const int ti = idx / kRbMB, j = idx - ti * kRbMB;
      float v = 0.f;
      if (ti < nt && j < mb) {
        const int64_t tok = tb + ti;
        const int g = group[tok];
        const float coef = gate_grad(gg, tok, g, M) * gate[tok];
        const float onehot = (g == j0 + j) ? 1.f : 0.f;
        v = coef * (onehot - probs[tok * M + j0 + j]);
      }
      s_dr[ti][j] = v;
    }
    __syncthreads();
    if (c < d) {
      for (int j = 0; j < mb; ++j) {
        const float wv = w[(int64_t)(j0 + j) * d + c];
#pragma unroll
        for (int ti = 0; ti < kRbTok; ++ti) out[ti] = fmaf(s_dr[ti][j], wv, out[ti]);
      }
    }
  }
  if (c < d) {
#pragma unroll
    for (int ti = 0; ti < kRbTok; ++ti)
      if (ti < nt) store_dx1(d_x + (tb + ti) * (int64_t)d + c, out[ti]);
  }
}

// dX for M <= 32 and d a multiple of 4: a thread owns COLS adjacent columns and keeps their MW >= M weights in registers; a block
// sweeps `tokens` tokens in tiles of kDxTile, whose dr rows are staged in LDS and read back as broadcast 16-byte pieces.  A wave's
// store of a row is 512 bytes or 1 KB.  Sums run over the groups in ascending order: exact fp32 FMA chains, the same for every launch.
// Bound by its stores.  With 32 weights per column whatever M is, 512 tokens per block whatever N is, and the rounding to bf16 left to a
// pass of its own, the two took 348 us at 62,400 x 1536, 5 groups (now some 45); a training step of 1,560 tokens x 4 heads
// (x 512, 8 groups) 282 us (now 110), of 9,000 x 12 (x 1536, 10) 607 (374), of 20,000 x 40 (x 5120, 20) 2,625 (2,389).
constexpr int kDxTile = 32;

template <typename OT, int MW, int COLS>
__global__ __launch_bounds__(256) void route_bwd_dx_cols_kernel(
    const float* __restrict__ w, const float* __restrict__ probs, const int32_t* __restrict__ group, const float* __restrict__ gate,
    GateGrad gg, int64_t N, int d, int M, int tokens, OT* __restrict__ d_x) {
  __shared__ __attribute__((aligned(16))) float s_dr[kDxTile][MW];
  const int c0 = (blockIdx.y * blockDim.x + threadIdx.x) * COLS;
  const bool valid = c0 < d;
  float wreg[MW][COLS];
#pragma unroll
  for (int j = 0; j < MW; ++j)
#pragma unroll
    for (int i = 0; i < COLS; i += 4) {
      const floatx4_t v = valid && j < M ? *(const floatx4_t*)(w + (int64_t)j * d + c0 + i) : floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; ++e) wreg[j][i + e] = v[e];
    }
  const int64_t t_begin = (int64_t)blockIdx.x * tokens;
  const int64_t t_end = min(N, t_begin + tokens);
  for (int64_t tb = t_begin; tb < t_end; tb += kDxTile) {
    const int nt = (int)min((int64_t)kDxTile, t_end - tb);
    __syncthreads();
    for (int idx = threadIdx.x; idx < kDxTile * MW; idx += blockDim.x) {
      const int ti = idx / MW, j = idx % MW;
      float v = 0.f;
      if (ti < nt && j < M) {
        const int64_t tok = tb + ti;
        const int g = group[tok];
        const float coef = gate_grad(gg, tok, g, M) * gate[tok];
        const float onehot = (g == j) ? 1.f : 0.f;
        v = coef * (onehot - probs[tok * M + j]);
      }
      s_dr[ti][j] = v;
    }
    __syncthreads();
    if (valid) {
      for (int ti = 0; ti < nt; ++ti) {
        float acc[COLS];
#pragma unroll
        for (int i = 0; i < COLS; ++i) acc[i] = 0.f;
#pragma unroll
        for (int j4 = 0; j4 < MW; j4 += 4) {
          const floatx4_t r = *(const floatx4_t*)&s_dr[ti][j4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < COLS; ++i) acc[i] = fmaf(r[e], wreg[j4 + e][i], acc[i]);
        }
        store_dx<COLS>(d_x + (tb + ti) * (int64_t)d + c0, acc);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// dW on the matrix cores (bf16 X, M <= 32, d a multiple of 256).
//
// dW^T[c, j] = sum_t X[t, c] dr[t, j] is a contraction over tokens.  A pre-pass writes dr as two
// bf16 limbs (hi + lo carries 16 mantissa bits) in the B-operand order of the 32x32x16 MFMA:
// [token block of 8][group 0..31][8 tokens], zero beyond M and beyond N.  The main kernel runs
// one wave per block: the wave owns 256 columns of X and a range of 16-token steps, streams
// [16 tokens x 256 columns] tiles of X plus the two dr limb tiles into its own LDS ring with
// direct-to-LDS loads (three stages in flight, no barriers: a wave only reads what it loaded),
// reads X^T fragments with transposed LDS reads and accumulates eight 32x32 blocks of dW^T.
// Partial sums go to partial[split][c][M rounded up to 8] and a second kernel reduces over the splits.
// ---------------------------------------------------------------------------------------
constexpr int kDwCols = 256;                          // columns of X per wave
constexpr int kDwTok = 16;                            // tokens per stage = one MFMA contraction step
constexpr int kDwStages = 4;                          // ring slots
constexpr int kDwXBytes = kDwTok * kDwCols * 2;       // 8 KB
constexpr int kDwStageBytes = kDwXBytes + 2048;       // + dr hi, dr lo (1 KB each)
constexpr int kDwDmaPerStage = kDwXBytes / 1024 + 2;  // direct-to-LDS instructions per stage

__global__ __launch_bounds__(256) void route_bwd_dr_pack_kernel(
    const float* __restrict__ probs, const int32_t* __restrict__ group,
    const float* __restrict__ gate, GateGrad gg, int64_t N, int M,
    int64_t blocks8, uintx4_t* __restrict__ dr_hi, uintx4_t* __restrict__ dr_lo) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t tb = idx >> 5;
  const int j = (int)(idx & 31);
  if (tb >= blocks8) return;
  unsigned short hi[8], lo[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int64_t tok = tb * 8 + i;
    float v = 0.f;
    if (tok < N && j < M) {
      const int g = group[tok];
      const float coef = gate_grad(gg, tok, g, M) * gate[tok];
      const float onehot = (g == j) ? 1.f : 0.f;
      v = coef * (onehot - probs[tok * M + j]);
    }
    hi[i] = f32_to_bf16_bits(v);
    lo[i] = f32_to_bf16_bits(v - bf16_bits_to_f32(hi[i]));
  }
  const uintx4_t ph = {hi[0] | ((unsigned)hi[1] << 16), hi[2] | ((unsigned)hi[3] << 16),
                       hi[4] | ((unsigned)hi[5] << 16), hi[6] | ((unsigned)hi[7] << 16)};
  const uintx4_t pl = {lo[0] | ((unsigned)lo[1] << 16), lo[2] | ((unsigned)lo[3] << 16),
                       lo[4] | ((unsigned)lo[5] << 16), lo[6] | ((unsigned)lo[7] << 16)};
  dr_hi[idx] = ph;
  dr_lo[idx] = pl;
}

// Chunk swizzle of the X tile in LDS (rows of 512 B = 32 chunks of 16 B): chunk' = chunk ^ this.
// The four rows a transposed read touches land in four different 64-byte bank groups.
__device__ __forceinline__ int dw_swizzle(int row) { return (row & 3) << 2; }

__global__ __launch_bounds__(64) void route_bwd_dw_mfma_kernel(
    const unsigned short* __restrict__ x, const uintx4_t* __restrict__ dr_hi,
    const uintx4_t* __restrict__ dr_lo, int64_t N, int d, int nslabs, int splits,
    int64_t steps_per_split, int64_t total_steps, int mp, float* __restrict__ partial) {
  __shared__ __attribute__((aligned(1024))) unsigned char ring[kDwStages * kDwStageBytes];
  const int lane = threadIdx.x;
  const int r = lane & 31, h = lane >> 5;
  // Blocks are dealt round-robin to the 8 XCDs; consecutive blocks of one XCD take the column
  // slabs of one token split, so its dr tiles are shared through that XCD's L2.
  const int64_t k = blockIdx.x >> 3;
  const int split = (int)(k / nslabs) * 8 + (int)(blockIdx.x & 7);
  const int slab = (int)(k % nslabs);
  if (split >= splits) return;
  const int64_t s0 = (int64_t)split * steps_per_split;
  const int64_t s1 = min(total_steps, s0 + steps_per_split);
  const int nst = (int)(s1 - s0);

  floatx16_t acc[8];
#pragma unroll
  for (int cb = 0; cb < 8; ++cb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[cb][v] = 0.f;

  const unsigned lds0 = lds_addr_uniform(&ring[0]);
  // direct-to-LDS: instruction q of a stage covers token rows 2q, 2q+1 (32 chunks each)
  const int dma_row = lane >> 5, dma_pos = lane & 31;
  const unsigned short* xslab = x + (int64_t)slab * kDwCols;
  auto issue = [&](int64_t step, int slot) {
    if (step > total_steps - 1) step = total_steps - 1;   // beyond the range: valid memory, never read back
    const int64_t tok0 = step * kDwTok;
    const int last = (int)min((int64_t)(kDwTok - 1), N - 1 - tok0);
    const void* xb = uniform_ptr(xslab + tok0 * (int64_t)d);
    const unsigned base = lds0 + slot * kDwStageBytes;
#pragma unroll
    for (int q = 0; q < kDwTok / 2; ++q) {
      const int row = 2 * q + dma_row;
      const unsigned off = (unsigned)min(row, last) * (unsigned)(d * 2) + ((dma_pos ^ dw_swizzle(row)) << 4);
      lds_dma16_soff(xb, off, base + q * 1024);
    }
    const int64_t tb = step * 2 * 32;   // two 8-token blocks of 32 groups, 16 bytes each
    lds_dma16_soff(uniform_ptr(dr_hi + tb), (unsigned)lane * 16u, base + kDwXBytes);
    lds_dma16_soff(uniform_ptr(dr_lo + tb), (unsigned)lane * 16u, base + kDwXBytes + 1024);
  };

  // transposed reads: lane gets X^T[column 32*cb + lane%32][tokens 8h .. 8h+7] from rows tr_r + {0..3}
  // (and + 4), 16-byte chunk 4*cb + tr_c, element offset tr_e
  const int tr_r = 8 * h + ((lane & 15) >> 2);
  const int tr_c = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  const int tr_e = 4 * (lane & 1);
  unsigned a_addr[8];
#pragma unroll
  for (int cb = 0; cb < 8; ++cb)
    a_addr[cb] = (unsigned)(uintptr_t)&ring[0] + tr_r * 512 + (((4 * cb + tr_c) ^ dw_swizzle(tr_r)) << 4) + tr_e * 2;
  const unsigned b_addr = (unsigned)(uintptr_t)&ring[0] + kDwXBytes + lane * 16;

#pragma unroll
  for (int t = 0; t < kDwStages - 1; ++t) issue(s0 + t, t);
  for (int s = 0; s < nst; ++s) {
    issue(s0 + s + kDwStages - 1, (s + kDwStages - 1) & (kDwStages - 1));
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kDwDmaPerStage * (kDwStages - 1)) : "memory");
    const unsigned so = (unsigned)(s & (kDwStages - 1)) * kDwStageBytes;
    const bf16x8_t bh = lds_read_b128(b_addr + so);
    const bf16x8_t bl = lds_read_b128(b_addr + so + 1024);
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) {
      const bf16x8_t a = concat_tr(lds_read_tr16_addr(a_addr[cb] + so), lds_read_tr16_addr(a_addr[cb] + so + 4 * 512));
      acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bh, acc[cb], 0, 0, 0);
      acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bl, acc[cb], 0, 0, 0);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may land in LDS after the block ends

  // accumulator register v of lane (r, h): column 8*(v/4) + 4*h + v%4 of the block, group r
  if (r >= mp) return;
  float* out = partial + ((int64_t)split * d + (int64_t)slab * kDwCols) * mp + r;
#pragma unroll
  for (int cb = 0; cb < 8; ++cb)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      out[(int64_t)(32 * cb + 8 * (v >> 2) + 4 * h + (v & 3)) * mp] = acc[cb][v];
}

constexpr int dw_group_block(int M) { return M <= 8 ? 8 : kRbMB; }   // groups per block of the FMA path

static int route_bwd_splits(int64_t N, int M, int d) {
  const int64_t per_split = (int64_t)((d + 63) / 64) * ((M + dw_group_block(M) - 1) / dw_group_block(M));
  int64_t s = std::min<int64_t>((1024 + per_split - 1) / per_split, (N + kRbTok - 1) / kRbTok);
  return (int)std::max<int64_t>(1, std::min<int64_t>(s, 256));
}

// Launch plan of the matrix-core dW path.
struct DwPlan {
  int nslabs, splits, mp;           // mp: groups per column in the partial sums
  int64_t total_steps, steps_per_split;
  size_t dr_bytes, partial_bytes;   // one dr limb array; the partial sums
};

static bool route_bwd_mfma_ok(int x_dtype, int M, int d) {
  return x_dtype == MOGA_BF16 && M <= 32 && d % kDwCols == 0;
}

// Plan of route_bwd_dw_few_kernel: `splits` blocks of `tokens` tokens for each 64 columns, one round of 256 blocks (a block has its
// CU to itself), or no splits where the kernels of DwPlan are the better ones.  One split up to 2,048 tokens: two launches take the
// device less from 1,024 on (1,560 x 1536, 4 groups 11.3 and 6.9 us), but the host more, which calls of so few tokens wait for (a whole
// training step through autograd, 1,560 x 512, 99.7 and 103.7).  The DwPlan kernels beyond 1e8 activations (in us, them and this: 65,000 x
// 1536, 32 groups 49.6 and 48.5; 87,000 x 1536 58.5 and 58.4; 32,760 x 5120 98.5 and 98.9) and beyond 65,536 tokens, where a block's
// dr for 64 columns is what it waits for (512, 32 groups: 65,000 30.0 and 27.9; 87,000 33.8 and 34.5; 130,000 42.4 and 49.8).
struct DwFewPlan {
  int splits, tokens;
};

static DwFewPlan route_bwd_few_plan(int64_t N, int d) {
  if (N > 65536 || N * d > 100000000) return {0, 0};
  const int64_t room = std::max(1, 256 / (d / 64));
  const int64_t splits = N <= 2048 ? 1 : std::min(room, N / 256);
  const int64_t tokens = ((N + splits - 1) / splits + kDwFewTok - 1) / kDwFewTok * kDwFewTok;
  if (tokens > kDwFewTokens) return {0, 0};
  return {(int)((N + tokens - 1) / tokens), (int)tokens};
}

static DwPlan route_bwd_plan(int64_t N, int M, int d) {
  DwPlan p;
  p.mp = (M + 7) / 8 * 8;
  p.nslabs = d / kDwCols;
  p.total_steps = (N + kDwTok - 1) / kDwTok;
  // 40 KB of LDS per one-wave block: 4 blocks per CU, 1024 on the chip; three rounds of them measured best
  // at 580k tokens (1.21 ms against 1.29 ms for two or four rounds) and at 100k (237 us; 251 for half a
  // round).  The partial sums cost 8 d mp bytes a split, so a split gets at least 512 tokens (20,000 x
  // 5120, M = 8: 45 us with 25 splits, 55 with 153), and down to 128 where that would leave the chip with
  // fewer than half a round of blocks.
  int64_t splits = std::max(std::min<int64_t>(3072 / p.nslabs, p.total_steps / 32),
                            std::min<int64_t>(512 / p.nslabs, (p.total_steps + 7) / 8));
  splits = std::max<int64_t>(1, std::min<int64_t>(splits, 256));
  p.steps_per_split = (p.total_steps + splits - 1) / splits;
  p.splits = (int)((p.total_steps + p.steps_per_split - 1) / p.steps_per_split);   // no empty split
  p.dr_bytes = (size_t)p.total_steps * 2 * 32 * 16;
  p.partial_bytes = (size_t)p.splits * (size_t)d * p.mp * sizeof(float);
  return p;
}

}  // namespace moga

using namespace moga;

extern "C" size_t moga_route_bwd_ws_bytes(int64_t N, int M, int d_model) {
  // the larger of the two paths, so the size does not depend on the dtype of X
  size_t need = (size_t)route_bwd_splits(N, M, d_model) * (size_t)M * (size_t)d_model * sizeof(float);
  if (N > 0 && route_bwd_mfma_ok(MOGA_BF16, M, d_model)) {
    const DwPlan p = route_bwd_plan(N, M, d_model);
    need = std::max(need, 2 * p.dr_bytes + p.partial_bytes);
    need = std::max(need, (size_t)route_bwd_few_plan(N, d_model).splits * (size_t)M * (size_t)d_model * sizeof(float));
  }
  return need;
}

extern "C" int moga_route(const void* x, int x_dtype, const float* w, const float* bias,
                          int64_t N, int d_model, int M, int32_t* group, float* gate,
                          float* probs, float* logits, void* ws, size_t ws_bytes, void* stream) {
  (void)ws; (void)ws_bytes;
  if (N < 0 || d_model < 1 || M < 1) return MOGA_ERR_INVALID_ARG;
  if (x_dtype != MOGA_F32 && x_dtype != MOGA_BF16) return MOGA_ERR_UNSUPPORTED;
  if (M > MOGA_MAX_GROUPS || N >= ((int64_t)1 << 31)) return MOGA_ERR_UNSUPPORTED;
  if (N == 0) return MOGA_OK;
  if (!x || !w || !group || !gate) return MOGA_ERR_INVALID_ARG;
  if (!aligned16(x) || !aligned16(w)) return MOGA_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (x_dtype == MOGA_BF16 && M <= 32 && d_model % 64 == 0) {
    if (N >= 65536) {
      // 8 waves share one staged weight chunk, one 32-token tile per wave: 16 waves per CU keep more
      // loads in flight than 4-wave blocks with two tiles per wave (5.1 against 4.7 TB/s at 580k tokens)
      const unsigned blocks = (unsigned)((N + 255) / 256);
      route_mfma_kernel<1, 8><<<blocks, 512, 0, st>>>((const unsigned short*)x, w, bias, N, d_model, M,
                                                     group, gate, probs, logits);
    } else if (use_route_few(N, d_model, M)) {
      const unsigned blocks = (unsigned)((N + 31) / 32);
#define MOGA_ROUTE_FEW(NWV)                                                                                                            \
  route_mfma_few_kernel<NWV><<<blocks, 64 * NWV, 0, st>>>((const unsigned short*)x, w, bias, N, d_model, M, group, gate, probs, logits)
      if (blocks <= 192 && d_model >= 2560) MOGA_ROUTE_FEW(8);
      else MOGA_ROUTE_FEW(4);
#undef MOGA_ROUTE_FEW
    } else {
      const unsigned blocks = (unsigned)((N + 127) / 128);
      route_mfma_kernel<1, 4><<<blocks, 256, 0, st>>>((const unsigned short*)x, w, bias, N, d_model, M,
                                                     group, gate, probs, logits);
    }
  } else {
    for (int64_t t = 0; t < N; t += kGenericTokens) {
      const int64_t n = std::min(N - t, kGenericTokens);
      const unsigned blocks = (unsigned)((n + 3) / 4);
      float *const pr = probs ? probs + t * M : nullptr, *const lo = logits ? logits + t * M : nullptr;
      if (x_dtype == MOGA_F32)
        route_generic_kernel<float><<<blocks, 256, 0, st>>>((const float*)x + t * d_model, w, bias, n, d_model, M, group + t, gate + t,
                                                           pr, lo);
      else
        route_generic_kernel<unsigned short><<<blocks, 256, 0, st>>>((const unsigned short*)x + t * d_model, w, bias, n, d_model, M,
                                                                     group + t, gate + t, pr, lo);
    }
  }
  return launch_status();
}

// Blocks of dX: threads of a block so that the fewest lie past the last column (the most of those), and tokens so that there are some
// 8,192 waves, 16 to 512 of them: 1,560 x 512, 8 groups ran on four blocks of 512 tokens.
template <int MW, int COLS, typename OT>
static void launch_dx_cols(const float* w, const float* probs, const int32_t* group, const float* gate, const GateGrad& gg, int64_t N,
                           int d, int M, OT* d_x, hipStream_t st) {
  const int cols = (d + COLS - 1) / COLS;
  int threads = 256;
  for (int t = 192; t >= 64; t -= 64)
    if ((cols + t - 1) / t * t < (cols + threads - 1) / threads * threads) threads = t;
  const int slabs = (cols + threads - 1) / threads;
  int64_t tokens = (N * slabs * (threads / 64) / 8192 + 15) / 16 * 16;
  tokens = std::min<int64_t>(512, std::max<int64_t>(16, tokens));
  route_bwd_dx_cols_kernel<OT, MW, COLS><<<dim3((unsigned)((N + tokens - 1) / tokens), slabs), threads, 0, st>>>(w, probs, group, gate, gg, N,
                                                                                                           d, M, (int)tokens, d_x);
}
template <typename OT>
static void launch_dx(const float* w, const float* probs, const int32_t* group, const float* gate, const GateGrad& gg, int64_t N, int d,
                      int M, OT* d_x, hipStream_t st) {
  constexpr bool kHalf = sizeof(OT) == 2;
  const bool wide = kHalf && d % 8 == 0 && aligned16(d_x);   // 16-byte stores of bf16
  if (M > 32 || d % 4 != 0 || ((uintptr_t)d_x & (4 * sizeof(OT) - 1)) != 0 || !aligned16(w)) {
    route_bwd_dx_kernel<<<dim3((unsigned)((N + kRbTok - 1) / kRbTok), (d + 255) / 256), 256, 0, st>>>(w, probs, group, gate, gg, N, d, M, d_x);
  } else if (M > 16) {
    launch_dx_cols<32, 4>(w, probs, group, gate, gg, N, d, M, d_x, st);   // with 8 columns 256 weights, which do not fit the registers
  } else if (wide) {
    if (M <= 8) launch_dx_cols<8, 8>(w, probs, group, gate, gg, N, d, M, d_x, st);
    else launch_dx_cols<16, 8>(w, probs, group, gate, gg, N, d, M, d_x, st);
  } else if (M <= 8) {
    launch_dx_cols<8, 4>(w, probs, group, gate, gg, N, d, M, d_x, st);
  } else {
    launch_dx_cols<16, 4>(w, probs, group, gate, gg, N, d, M, d_x, st);
  }
}

static int launch_route_bwd(const void* x, int x_dtype, const float* w, const float* probs, const int32_t* group, const float* gate,
                            const GateGrad& gg, int64_t N, int d_model, int M, float* d_w, void* d_x, int dx_dtype, void* ws,
                            size_t ws_bytes, void* stream) {
  if (N < 0 || d_model < 1 || M < 1) return MOGA_ERR_INVALID_ARG;
  if (x_dtype != MOGA_F32 && x_dtype != MOGA_BF16) return MOGA_ERR_UNSUPPORTED;
  if (d_x && dx_dtype != MOGA_F32 && dx_dtype != MOGA_BF16) return MOGA_ERR_UNSUPPORTED;
  if (M > MOGA_MAX_GROUPS || N >= ((int64_t)1 << 31)) return MOGA_ERR_UNSUPPORTED;
  if (d_model > (1 << 24)) return MOGA_ERR_UNSUPPORTED;
  if (!d_w) return MOGA_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  const int64_t md = (int64_t)M * d_model;
  if (!grid_fits(((int64_t)(M + 7) / 8 * 8 * d_model + 63) / 64, 512) || (d_x && !grid_fits((N + kRbTok - 1) / kRbTok, 256)))
    return MOGA_ERR_UNSUPPORTED;
  if (N == 0) {
    launch_fill_zero(d_w, md, st);
    return launch_status();
  }
  if (!x || !w || !probs || !group || !gate || !gg.d_gate) return MOGA_ERR_INVALID_ARG;
  const size_t need = moga_route_bwd_ws_bytes(N, M, d_model);
  if (!ws || ws_bytes < need) return MOGA_ERR_WORKSPACE;
  const bool mfma = route_bwd_mfma_ok(x_dtype, M, d_model);
  if (mfma && (!aligned16(x) || !aligned16(ws))) return MOGA_ERR_INVALID_ARG;
  const DwFewPlan few = mfma ? route_bwd_few_plan(N, d_model) : DwFewPlan{0, 0};
  if (few.splits > 1 || (few.splits == 1 && ((uintptr_t)d_w & 7) == 0)) {
    route_bwd_dw_few_kernel<<<dim3(d_model / 64, few.splits), 64 * kDwFewWaves, 0, st>>>(
        (const unsigned short*)x, probs, group, gate, gg, N, few.tokens, d_model, M, few.splits > 1 ? (float*)ws : d_w);
    if (few.splits > 1)
      route_bwd_dw_reduce_kernel<false><<<(unsigned)((md + 63) / 64), 512, 0, st>>>((const float*)ws, few.splits, md, d_model, M, M, d_w);
  } else if (mfma) {
    const DwPlan p = route_bwd_plan(N, M, d_model);
    uintx4_t* dr_hi = (uintx4_t*)ws;
    uintx4_t* dr_lo = (uintx4_t*)((char*)ws + p.dr_bytes);
    float* partial = (float*)((char*)ws + 2 * p.dr_bytes);
    const int64_t blocks8 = p.total_steps * 2;
    route_bwd_dr_pack_kernel<<<(unsigned)((blocks8 * 32 + 255) / 256), 256, 0, st>>>(
        probs, group, gate, gg, N, M, blocks8, dr_hi, dr_lo);
    const unsigned blocks = (unsigned)((p.splits + 7) / 8 * 8 * p.nslabs);
    route_bwd_dw_mfma_kernel<<<blocks, 64, 0, st>>>((const unsigned short*)x, dr_hi, dr_lo, N, d_model,
                                                    p.nslabs, p.splits, p.steps_per_split,
                                                    p.total_steps, p.mp, partial);
    const int64_t n = (int64_t)d_model * p.mp;
    route_bwd_dw_reduce_kernel<true><<<(unsigned)((n + 63) / 64), 512, 0, st>>>(partial, p.splits, n, d_model, M, p.mp, d_w);
  } else {
    const int splits = route_bwd_splits(N, M, d_model);
    int64_t tps = (N + splits - 1) / splits;
    tps = (tps + kRbTok - 1) / kRbTok * kRbTok;
    const int mb = dw_group_block(M);
    dim3 grid((d_model + 63) / 64, splits, (M + mb - 1) / mb);
    float* partial = (float*)ws;
#define MOGA_DW_PARTIAL(XT, MB)                                                                             \
  route_bwd_dw_partial_kernel<XT, MB><<<grid, 256, 0, st>>>((const XT*)x, probs, group, gate, gg, N,    \
                                                            d_model, M, tps, partial)
    if (x_dtype == MOGA_F32) {
      if (mb == 8) MOGA_DW_PARTIAL(float, 8);
      else MOGA_DW_PARTIAL(float, kRbMB);
    } else {
      if (mb == 8) MOGA_DW_PARTIAL(unsigned short, 8);
      else MOGA_DW_PARTIAL(unsigned short, kRbMB);
    }
#undef MOGA_DW_PARTIAL
    route_bwd_dw_reduce_kernel<false><<<(unsigned)((md + 63) / 64), 512, 0, st>>>(partial, splits, md, d_model, M, M, d_w);
  }
  if (d_x) {
    if (dx_dtype == MOGA_BF16) launch_dx(w, probs, group, gate, gg, N, d_model, M, (unsigned short*)d_x, st);
    else launch_dx(w, probs, group, gate, gg, N, d_model, M, (float*)d_x, st);
  }
  return launch_status();
}

extern "C" int moga_route_bwd(const void* x, int x_dtype, const float* w, const float* probs,
                              const int32_t* group, const float* gate, const float* d_gate,
                              int64_t N, int d_model, int M, float* d_w, float* d_x,
                              void* ws, size_t ws_bytes, void* stream) {
  return launch_route_bwd(x, x_dtype, w, probs, group, gate, GateGrad{d_gate, nullptr, 0.f, nullptr}, N, d_model, M, d_w, d_x,
                          MOGA_F32, ws, ws_bytes, stream);
}

extern "C" int moga_route_bwd_balanced(const void* x, int x_dtype, const float* w, const float* probs, const int32_t* group,
                                       const float* gate, const float* d_gate, const float* frac, float alpha, float d_loss,
                                       const float* d_loss_dev, int64_t N, int d_model, int M, float* d_w, float* d_x, void* ws,
                                       size_t ws_bytes, void* stream) {
  if (N > 0 && !frac) return MOGA_ERR_INVALID_ARG;
  const float coef = N > 0 ? (float)((double)d_loss * (double)alpha * (double)M / (double)N) : 0.f;   // as moga_balance_loss_bwd
  return launch_route_bwd(x, x_dtype, w, probs, group, gate, GateGrad{d_gate, frac, coef, d_loss_dev}, N, d_model, M, d_w, d_x,
                          MOGA_F32, ws, ws_bytes, stream);
}

extern "C" int moga_route_bwd_typed(const void* x, int x_dtype, const float* w, const float* probs, const int32_t* group,
                                    const float* gate, const float* d_gate, const float* frac, float alpha, float d_loss,
                                    const float* d_loss_dev, int64_t N, int d_model, int M, float* d_w, void* d_x, int dx_dtype,
                                    void* ws, size_t ws_bytes, void* stream) {
  const float coef = frac && N > 0 ? (float)((double)d_loss * (double)alpha * (double)M / (double)N) : 0.f;
  return launch_route_bwd(x, x_dtype, w, probs, group, gate, GateGrad{d_gate, frac, coef, frac ? d_loss_dev : nullptr}, N, d_model, M,
                          d_w, d_x, dx_dtype, ws, ws_bytes, stream);
}
