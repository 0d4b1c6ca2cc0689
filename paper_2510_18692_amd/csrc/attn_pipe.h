// Software-pipelined bf16 forward kernel of the group attention (head_dim 128).
//
// 8 waves per block, two per SIMD, 48 query rows per wave (384-row query tiles; 32 and 256 where that suits the call better).
// Keys are consumed in steps of 32.  While the matrix cores compute the scores of step s+1
// (S^T = K Q^T), the vector units exponentiate the exponents of step s; while the matrix cores
// accumulate O^T += V^T P^T of step s, the vector units turn the scores of step s+1 into exponents and take their maximum.
// K/V tiles of 64 keys (two steps) are streamed global -> LDS with direct-to-LDS loads into
// a ring of four buffers, two tiles ahead of their use; one block-wide barrier per tile.
//
// Bound by energy at the board's power cap, that of the matrix instructions and of what goes with them: fragment reads, which 48 rows share
// instead of 32, vector instructions (1.6 per product) and the stream of tiles, which 384 rows share instead of 256.  580,320 x 40 heads, 32
// groups: 1.90 -> 1.62 vector instructions per product with 0.71 -> 0.47 LDS ones; 145,080 x 40, 8 groups 43.6 -> 41.0 ms (on zeros
// 33.2 -> 31.2), 99,840 x 40, 16 groups 10.55 -> 10.1, 62,400 x 12, 5 groups 3.74 -> 3.63, 32,760 x 12, 8 groups 0.685 -> 0.670.  64 rows
// per wave do not fit 256 registers.
#pragma once

#include <type_traits>

#include "attn_common.h"

namespace moga {

constexpr int kPipeNBuf = 4;                      // LDS ring: tiles of 64 keys
constexpr int kPipeAhead = 2;                     // tiles in flight beyond the one being waited for
constexpr int kPipeTileBytes = 64 * kHeadDim * 2; // 16 KB per K (or V) tile

__device__ __forceinline__ float uniform_float(float x) {
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

// A value that the compiler takes as it is: what is added to it later is not folded into it.
__device__ __forceinline__ unsigned in_register(unsigned x) {
  asm("" : "+v"(x));
  return x;
}

// All waves of the block are here.  Unlike __syncthreads it does not wait for the wave's own LDS reads.
__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

struct PipeLane {
  unsigned k;      // K rows
  unsigned v[2];   // V transposed
  bf16x8_t ones;   // A operand of the row sums
};

__device__ __forceinline__ bf16x8_t all_ones() {
  uintx4_t v = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
#pragma unroll
  for (int i = 0; i < 4; ++i) asm("" : "+v"(v[i]));   // in registers, not made again in every step
  return __builtin_bit_cast(bf16x8_t, v);
}

// Scores of a step, or the exponents s*c - m*c of its weights: [key operand t][query column]; register i is key 8 g + 4 t + i of
// query 16 q + r
template <int NC>
using Scores = floatx4_t[2][NC];
typedef Scores<2> StepScores;

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// Maximum of a lane's own eight values of a query (the other keys of the step are in three other lanes)
template <int NC>
__device__ __forceinline__ float column_max(const floatx4_t (&s)[2][NC], int q) {
  float t = max3(s[0][q][0], s[0][q][1], s[0][q][2]);
  t = max3(t, s[0][q][3], s[1][q][0]);
  t = max3(t, s[1][q][1], s[1][q][2]);
  return fmaxf(t, s[1][q][3]);
}
template <int NC>
__device__ __forceinline__ void step_max(const floatx4_t (&s)[2][NC], float (&mx)[NC]) {
#pragma unroll
  for (int q = 0; q < NC; ++q) mx[q] = column_max(s, q);
}

template <int NC>
__device__ __forceinline__ void mask_step(floatx4_t (&s)[2][NC], int first_key, int g, int end) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (first_key + 8 * g + 4 * t + i >= end) s[t][q][i] = -INFINITY;
}

template <int NC>
__device__ __forceinline__ void copy_scores(floatx4_t (&to)[2][NC], const floatx4_t (&from)[2][NC]) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int q = 0; q < NC; ++q) to[t][q] = from[t][q];
}

__device__ __forceinline__ floatx4_t quarter(const floatx16_t& v, int k) {
  return floatx4_t{v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]};
}

template <int NC>
struct PipeState {
  // O^T: [d tiles 4 D .. 4 D + 3][query column], 16 registers each.  As sixteen vectors of four the compiler joins the two
  // sides of the rare branch in maybe_rescale by moving all 64 registers in every step.
  floatx16_t o[2][NC];
  float l[NC];       // row sums
  float negmc[NC];   // -m*c of the running maximum m (0: none yet)
  float thresh[NC];  // an exponent s*c - m*c above it raises the maximum: 8, or -inf before the first one
};

template <int NC>
__device__ __forceinline__ void pipe_state_init(PipeState<NC>& st) {
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    st.l[q] = st.negmc[q] = 0.f;
    st.thresh[q] = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) st.o[0][q][e] = st.o[1][q][e] = 0.f;
  }
}

// The four lanes of a query compare their own maxima with the common threshold; only when one exceeds it is the
// maximum taken over all four, and what depends on it brought to the new one: the sums and the exponents `x` of the coming step.
template <int NC>
__device__ __forceinline__ void maybe_rescale(PipeState<NC>& st, const float (&mx)[NC], floatx4_t (&x)[2][NC]) {
  bool up = false;
#pragma unroll
  for (int q = 0; q < NC; ++q) up = up || mx[q] > st.thresh[q];
  if (__builtin_amdgcn_ballot_w64(up) != 0) {   // wave-uniform; after the first step this is rare
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      float all = fmaxf(mx[q], __shfl_xor(mx[q], 16, kWave));
      all = fmaxf(all, __shfl_xor(all, 32, kWave));
      const bool first = st.thresh[q] == -INFINITY;
      const float by = first ? (all == -INFINITY ? 0.f : all) : fmaxf(all, 0.f);
      const float alpha = first ? 0.f : fast_exp2(-by);
      if (all != -INFINITY) st.thresh[q] = 8.f;
      st.negmc[q] -= by;
      st.l[q] *= alpha;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[t][q][i] -= by;
#pragma unroll
      for (int D = 0; D < 2; ++D)
#pragma unroll
        for (int i = 0; i < 16; ++i) st.o[D][q][i] *= alpha;
    }
  }
}

// Exponents of a column's keys from its scores, and their maximum.
template <int NC>
__device__ __forceinline__ float column_exponents(floatx4_t (&s)[2][NC], int q, float c, float negmc) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) s[t][q][i] = fmaf(s[t][q][i], c, negmc);
  return column_max(s, q);
}

// Scores of a whole step from its K rows at byte offset `off`.
template <int ROWS, int NC>
__device__ __forceinline__ void step_scores(const PipeLane& ln, unsigned off, const bf16x8_t (&qf)[NC][4], floatx4_t (&s)[2][NC]) {
  bf16x8_t kf[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kf[t][ks] = read_nat<ROWS>(ln.k + off, t, ks);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < NC; ++q)
        s[t][q] = mfma16(kf[t][ks], qf[q][ks], ks == 0 ? floatx4_t{0.f, 0.f, 0.f, 0.f} : s[t][q]);
}

// One pipeline step.  KOFF: byte offset (half of a tile, or ring slot too) of the NEXT step's keys; VOFF: of the CURRENT step's
// values; with SLOT koff and voff are added to them.  s_cur holds the current step's exponents; s_next
// receives those of the next step (if HAS_NEXT) and mx their lane maxima.
//
// The step's sixteen fragments (K rows, then V transposed) are read kWin ahead of their products, three products each, and the
// exponentials stay where they are put among the products: with all fragments read first, as 32 rows per wave allow, the registers
// spill, and the compiler's own order of loads and exponentials takes 2 to 5 % longer.  The exponents are made where the scores are, not
// where they are used: the vector instructions are spread over both halves of the step, the maximum needs no canonical copies of
// its operands, and no maximum but the scaled one is kept (zeros, 145,080 x 40 heads: 33.1 -> 31.4 ms with the addresses).
// `mid` is called among the PV products, kWin d tiles before their end: the barrier of the tiles.  There, once a tile, it also keeps
// the two waves of a SIMD in step, one at its scores while the other is at its PV products; with a barrier for two tiles zeros take 8 % longer.
constexpr int kWin = 2, kSumAt = 3, kMaxAt = 3;   // d tile where the row sums, and from which on the maxima, are taken
template <int ROWS, bool SLOT, bool PRIO, bool HAS_NEXT, int KOFF, int VOFF, int NC, typename F>
__device__ __forceinline__ void pipe_step(const PipeLane& ln, unsigned koff, unsigned voff, const bf16x8_t (&qf)[NC][4],
                                          PipeState<NC>& st, const floatx4_t (&s_cur)[2][NC], floatx4_t (&s_next)[2][NC],
                                          float (&mx)[NC], float c, F&& mid) {
  // The scores and exponentials are the long chain of a step: they go first when the SIMD's two waves compete, and the
  // other wave's PV products fill the gaps (without priorities 4 % slower, on zeros 8 %).
  wave_priority<PRIO, 1>();
  unsigned int pk[NC][4];
  constexpr int kKeep = 0x2 | 0x4 | 0x400;   // what may cross: vector, scalar and transcendental instructions
  bf16x8_t fr[16];   // K rows (t, ks), then V transposed (dt)
  // One address per kind of read, so that everything else is an immediate of the read: left to itself the compiler adds
  // each offset by an instruction of its own.
  unsigned ka = ln.k, va[2] = {ln.v[0], ln.v[1]};
  if (SLOT) {
    ka = in_register(ka + koff);
#pragma unroll
    for (int p = 0; p < 2; ++p) va[p] = in_register(va[p] + voff);
  }
  auto load = [&](int f) {
    if (f < 8) {
      if constexpr (HAS_NEXT) fr[f] = read_nat<ROWS>(ka + KOFF, f >> 2, f & 3);
    } else if (f < 16) {
      fr[f] = read_tr<ROWS>(va, VOFF, f - 8);
    }
  };
#pragma unroll
  for (int f = 0; f < kWin; ++f) load(f);
  if constexpr (HAS_NEXT) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < NC; ++q) s_next[t][q] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
  // P = exp2 of the exponents, packed to bf16
  auto word = [&](int q, int w) {   // keys 8 g + 2 w and + 1
    const floatx4_t& v = s_cur[w >> 1][q];
    pk[q][w] = pack_bf16x2(fast_exp2(v[2 * (w & 1)]), fast_exp2(v[2 * (w & 1) + 1]));
  };
#pragma unroll
  for (int f = 0; f < 8; ++f) {
    __builtin_amdgcn_sched_barrier(0);
    load(f + kWin);
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if constexpr (HAS_NEXT) s_next[f >> 2][q] = mfma16(fr[f], qf[q][f & 3], s_next[f >> 2][q]);
#pragma unroll
    for (int j = 4 * NC * f / 8; j < 4 * NC * (f + 1) / 8; ++j) word(j % NC, j / NC);
  }
  __builtin_amdgcn_sched_barrier(0);
  wave_priority<PRIO, 0>();
  bf16x8_t pf[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) pf[q] = __builtin_bit_cast(bf16x8_t, uintx4_t{pk[q][0], pk[q][1], pk[q][2], pk[q][3]});
  floatx4_t sum[NC];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) {
    // The row sums are one more d tile, of ones (two weights at a time v_dot2c_f32_bf16 would sum, but that does not run beside the
    // matrix instructions: it adds its 8 cycles to their 16), and are added up where no product waits for them.
    if (dt == kSumAt) {
#pragma unroll
      for (int q = 0; q < NC; ++q) sum[q] = mfma16(ln.ones, pf[q], floatx4_t{0.f, 0.f, 0.f, 0.f});
    }
    if (dt == 7)
#pragma unroll
      for (int q = 0; q < NC; ++q) st.l[q] += sum[q][0];
    if (dt == 8 - kWin) mid();
    if constexpr (HAS_NEXT)   // a column's maximum at a time
      if (dt >= kMaxAt && dt < kMaxAt + NC) mx[dt - kMaxAt] = column_exponents(s_next, dt - kMaxAt, c, st.negmc[dt - kMaxAt]);
    __builtin_amdgcn_sched_barrier(kKeep);
    load(8 + dt + kWin);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      floatx16_t& o = st.o[dt >> 2][q];
      const floatx4_t t = mfma16(fr[8 + dt], pf[q], quarter(o, dt & 3));
#pragma unroll
      for (int e = 0; e < 4; ++e) o[4 * (dt & 3) + e] = t[e];
    }
  }
  if constexpr (HAS_NEXT) {   // in its registers here: not after the products, behind the branches that follow
#pragma unroll
    for (int q = 0; q < NC; ++q) asm volatile("" : "+v"(mx[q]));
  }
}

// Output rows of a wave (query columns r, 16 + r .. of its 16 NC rows from q0w): O / l, times the row's gate in gather mode,
// and the log-sum-exp.  Register i of d tile dt is d = 16 dt + 4 g + i.
// o_tok (not in gather mode): NULL, or where the rows also go in token order [N, H, 128], rounded and then times the gate.
template <bool GATHER, int NC>
__device__ __forceinline__ void store_output(const PipeState<NC>& st, int q0w, int ge, int head, int64_t head_off, int H,
                                             unsigned short* __restrict__ oh, float* __restrict__ lse,
                                             const int32_t* __restrict__ perm, const float* __restrict__ gate,
                                             unsigned short* __restrict__ o_tok) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const float lt = st.l[q];
    float inv = 1.f / lt;
    const int qrow = q0w + 16 * q + r;
    if (qrow < ge) {
      int64_t orow = head_off + qrow;
      if (GATHER) {
        const int tok = perm[qrow];
        orow = (int64_t)tok * H + head;
        inv *= gate[tok];
      }
      unsigned short* op = oh + orow * kHeadDim + join_channel(g);
      unsigned short* tp = nullptr;
      float gt = 1.f;
      if (!GATHER && o_tok) {
        const int tok = perm[qrow];
        tp = o_tok + ((int64_t)tok * H + head) * kHeadDim + join_channel(g);
        gt = gate[tok];
      }
#pragma unroll
      for (int dt = 0; dt < 8; dt += 2) {
        const floatx16_t& o = st.o[dt >> 2][q];
        const uintx4_t v = join_tiles(pack4(quarter(o, dt & 3), inv), pack4(quarter(o, (dt & 3) + 1), inv));
        *(uintx4_t*)(op + 16 * dt) = v;
        if (!GATHER && o_tok) *(uintx4_t*)(tp + 16 * dt) = scale8(v, gt);
      }
      if (g == 0) lse[head_off + qrow] = logf(lt) - st.negmc[q] * 0.6931471805599453f;
    }
  }
}

// A piece's O, maximum and sum of this wave's rows (row0 on, of the workspace), not yet divided.
template <int NC>
__device__ __forceinline__ void store_piece(const PipeState<NC>& st, const SplitWs& sw, size_t row0) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const float lt = st.l[q];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) store_partial(sw.part + row0 * kHeadDim, dt, q, quarter(st.o[dt >> 2][q], dt & 3));
    if (lane < 16) *(floatx2_t*)(sw.stat + (row0 + 16 * q + lane) * 2) = floatx2_t{st.thresh[q] == -INFINITY ? -INFINITY : -st.negmc[q], lt};
  }
}
template <int NC>
__device__ __forceinline__ void store_empty_piece(const SplitWs& sw, size_t row0) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) store_partial(sw.part + row0 * kHeadDim, dt, q, floatx4_t{0.f, 0.f, 0.f, 0.f});
    if (lane < 16) *(floatx2_t*)(sw.stat + (row0 + 16 * q + lane) * 2) = floatx2_t{-INFINITY, 0.f};
  }
}

// Zero output rows of a wave whose group has no keys (lse = -inf if given); `tok`: NULL, or the rows in token order.
template <bool GATHER, int NC>
__device__ __forceinline__ void store_zero_rows(int row0, int ge, int head, int64_t head_off, int H, unsigned short* __restrict__ out,
                                                float* __restrict__ lse, const int32_t* __restrict__ perm,
                                                unsigned short* __restrict__ tok) {
  const int lane = threadIdx.x & 63, h = lane >> 5;
  const uintx4_t z = {0u, 0u, 0u, 0u};
  for (int row = row0 + (lane & 31); row < min(ge, row0 + 16 * NC); row += 32) {
    if (out) {
      const int64_t orow = GATHER ? (int64_t)perm[row] * H + head : head_off + row;
      uintx4_t* op = (uintx4_t*)(out + orow * kHeadDim + 64 * h);
#pragma unroll
      for (int i = 0; i < 8; ++i) op[i] = z;
    }
    if (!GATHER && tok) {
      uintx4_t* op = (uintx4_t*)(tok + ((int64_t)perm[row] * H + head) * kHeadDim + 64 * h);
#pragma unroll
      for (int i = 0; i < 8; ++i) op[i] = z;
    }
    if (lse && h == 0) lse[head_off + row] = -INFINITY;
  }
}

// B fragments of a wave's 16 NC rows from row0 (clamped to the last row of the group): columns 16 c + r, d = 32 ks + 8 g ..
template <bool GATHER, int NC>
__device__ __forceinline__ void load_columns(bf16x8_t (&f)[NC][4], const unsigned short* __restrict__ src, int row0, int ge, int head,
                                             int64_t head_off, int H, const int32_t* __restrict__ perm) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int row = min(row0 + 16 * c + (lane & 15), ge - 1);
    const int64_t irow = GATHER ? (int64_t)perm[row] * H + head : head_off + row;
    const unsigned short* p = src + irow * kHeadDim + 8 * (lane >> 4);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) f[c][ks] = *(const bf16x8_t*)(p + 32 * ks);
  }
}

// The fragments are in their registers: the compiler waits for their loads here and nowhere later.
template <int NC>
__device__ __forceinline__ void settle(bf16x8_t (&f)[NC][4]) {
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(f[c][ks]));
}

// Direct-to-LDS loads of tiles of ROWS rows: a load of a wave moves one quarter of 16 rows (1 KB), and a wave moves
// neighbouring quarters of the same rows, ROWS / (4 NW) of them per tensor.
struct PipeDma {
  const void* kbase;   // first K row of this head's group (wave-uniform)
  const void* vbase;
  unsigned lds_k, lds_v;   // LDS byte address of this wave's first load in buffer 0 (wave-uniform)
  int row0;                // this lane's row inside a tile
  unsigned chunk_off;      // its 16-byte chunk inside the row, in bytes
  int last_row;            // last valid row, relative to the group's first row
  // gather mode: rows are fetched through an index list from token-major tensors; kbase / vbase
  // then point at token 0 of this head
  const void* rows;        // index list at the group's first row (wave-uniform)
  int64_t tok_stride;      // bytes between two tokens
  unsigned lds_tok;        // LDS byte address of the tokens of a tile, eight slots of 256 bytes (wave-uniform)
};

__device__ __forceinline__ void lds_dma4_soff(const void* base, unsigned byte_off, unsigned lds_wave_base) {
  lds_wave_base = __builtin_amdgcn_readfirstlane(lds_wave_base);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :
               : "s"(lds_wave_base), "v"(byte_off), "s"(base)
               : "memory");
}

template <int NW, int ROWS>
constexpr int kDmaLoads = ROWS / (4 * NW);   // per tensor, wave and tile

template <int NW, int ROWS>
__device__ __forceinline__ void dma_lanes(PipeDma& d, const void* lds_k, const void* lds_v, int wave, int lane) {
  const int unit = wave * kDmaLoads<NW, ROWS>, quarter = unit & 3;   // first of the wave's loads
  const unsigned lds_off = quarter * kQuarterBytes<ROWS> + (unit >> 2) * 1024;
  d.lds_k = lds_addr_uniform(lds_k) + lds_off;
  d.lds_v = lds_addr_uniform(lds_v) + lds_off;
  d.row0 = 16 * (unit >> 2) + (lane >> 2);
  d.chunk_off = (unsigned)(quarter * 64 + (((lane & 3) ^ lds_swizzle(d.row0)) << 4));
}

// Gather mode: the tokens of the tile at kv0, two tiles before its rows are issued: the kernels' waits, which count the loads of
// rows only, cover them by then (every wave moves the same 256 bytes).  Eight slots: before the first barrier a wave may be five
// tiles ahead of one that has not read its first tokens.
__device__ __forceinline__ void pipe_issue_tokens(const PipeDma& d, int kv0) {
  lds_dma4_soff(d.rows, (unsigned)min(kv0 + (int)(threadIdx.x & 63), d.last_row) * 4u, d.lds_tok + ((kv0 >> 6) & 7) * 256);
}

// Issue the loads of the tile starting at group-relative row kv0 into the ring slot `boff` bytes into the ring.
template <int NW, int ROWS, bool GATHER>
__device__ __forceinline__ void pipe_issue(const PipeDma& d, int kv0, unsigned boff) {
  if constexpr (GATHER) {
    static_assert(ROWS == 64, "64 tokens at a time");
    pipe_issue_tokens(d, kv0 + 2 * ROWS);
    const unsigned slot = d.lds_tok + ((kv0 >> 6) & 7) * 256;
    const int tok = *(const int __attribute__((address_space(3)))*)(uintptr_t)(slot + d.row0 * 4);
    const int64_t off = tok * d.tok_stride + d.chunk_off;
#pragma unroll
    for (int i = 0; i < kDmaLoads<NW, ROWS>; ++i) {
      lds_dma16((const char*)d.kbase + off + 64 * i, d.lds_k + boff + i * kQuarterBytes<ROWS>);
      lds_dma16((const char*)d.vbase + off + 64 * i, d.lds_v + boff + i * kQuarterBytes<ROWS>);
    }
  } else {
    const unsigned off = (unsigned)min(kv0 + d.row0, d.last_row) * (kHeadDim * 2) + d.chunk_off;
#pragma unroll
    for (int i = 0; i < kDmaLoads<NW, ROWS>; ++i) {
      lds_dma16_soff(d.kbase, off + 64 * i, d.lds_k + boff + i * kQuarterBytes<ROWS>);
      lds_dma16_soff(d.vbase, off + 64 * i, d.lds_v + boff + i * kQuarterBytes<ROWS>);
    }
  }
}

// Queries are the rows cu_q[g] .. cu_q[g+1] of qh [H, Nq, 128]; their keys and values the rows
// cu_k[g] .. cu_k[g+1] of kh, vh [H, Nk, 128] (cu_k == cu_q and Nk == Nq for MoGA's groups).
// tile_start: NULL (tile lookup from cu_q inside the block, M <= MOGA_MAX_GROUPS) or the
// pre-summed first-tile index of every group.
//
// o_tok: NULL, or [N, H, 128] for the rows in token order times their gate as well (Alg. 1 step 4, the scatter, without
// reading the output again): row j is token perm[j].
// GATHER: qh, kh, vh and oh are token-major [N, H, 128]; row j of a group is token perm[j] (the
// permutation of Alg. 1 is applied while loading, nothing is materialised) and the output row is
// multiplied by gate[token] (Eq. 5) and written to its token.  lse stays in sorted order [H, N].
// SPLIT: the last round is cut into pieces (find_work).
// ROWS: query rows of a block, 384 or 256 (query_blocks chooses).
template <int ROWS, bool GATHER, bool SPLIT>
__device__ __forceinline__ void attn_fwd_block(
    int block, const unsigned short* __restrict__ qh, const unsigned short* __restrict__ kh,
    const unsigned short* __restrict__ vh, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, unsigned short* __restrict__ oh,
    float* __restrict__ lse, const int32_t* __restrict__ perm,
    const float* __restrict__ gate, SplitWs sw, unsigned short* __restrict__ o_tok) {
  constexpr int NW = 8;
  constexpr int kDmaPerTile = 2 * kDmaLoads<NW, 64>;   // direct-to-LDS instructions per thread per tile
  __shared__ __attribute__((aligned(1024))) unsigned short Ks[kPipeNBuf][64 * kHeadDim];
  __shared__ __attribute__((aligned(1024))) unsigned short Vs[kPipeNBuf][64 * kHeadDim];
  __shared__ __attribute__((aligned(256))) int toks[GATHER ? 512 : 1];   // gather mode: tokens of eight tiles

  WorkTile sp;
  if (!find_work<SPLIT>(cu_q, tile_start, M, H, ROWS, block, sp)) return;
  const TileInfo& ti = sp.ti;
  const int head = sp.head;
  const int ge = ti.row_end, q0 = ti.tile_row;   // query rows of the group end at ge
  int gs = cu_k[ti.group];                       // first key row of the group
  int n = cu_k[ti.group + 1] - gs;               // number of keys
  const bool piece = SPLIT && sp.splits > 1;
  if (piece) split_range(sp, gs, n);

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t head_off = (int64_t)head * Nq;
  const int64_t head_off_k = (int64_t)head * Nk;
  const float c = uniform_float(scale * 1.4426950408889634f);

  // A wave owns 16 NC query rows: three columns, or two where that is enough for the last tile of a group, which then takes
  // two thirds of the time.
  auto sweep = [&](auto columns) {
    constexpr int NC = columns.value;
    const int q0w = q0 + wave * 16 * NC;   // first query row of this wave
    const size_t piece_row = (size_t)sp.slot * ROWS + 16 * NC * wave;
    if (n <= 0) {   // queries without keys: zero output, lse = -inf (block-uniform branch)
      if (piece) store_empty_piece<NC>(sw, piece_row);
      else store_zero_rows<GATHER, NC>(q0w, ge, head, head_off, H, oh, lse, perm, o_tok);
      return;
    }

    bf16x8_t qf[NC][4];
    load_columns<GATHER>(qf, qh, q0w, ge, head, head_off, H, perm);

    // the first kPipeAhead + 1 tiles (always issued; rows are clamped)
    PipeDma dma;
    dma.kbase = uniform_ptr(GATHER ? kh + (int64_t)head * kHeadDim : kh + (head_off_k + gs) * kHeadDim);
    dma.vbase = uniform_ptr(GATHER ? vh + (int64_t)head * kHeadDim : vh + (head_off_k + gs) * kHeadDim);
    dma_lanes<NW, 64>(dma, &Ks[0][0], &Vs[0][0], wave, lane);
    dma.last_row = n - 1;
    if constexpr (GATHER) {
      dma.rows = uniform_ptr(perm + gs);
      dma.tok_stride = (int64_t)H * kHeadDim * 2;
      dma.lds_tok = lds_addr_uniform(&toks[0]);
      pipe_issue_tokens(dma, 0);
      pipe_issue_tokens(dma, 64);
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    }
#pragma unroll
    for (int t = 0; t <= kPipeAhead; ++t) {
      if (GATHER && t == 2) __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kDmaPerTile));   // its tokens
      pipe_issue<NW, 64, GATHER>(dma, 64 * t, t * kPipeTileBytes);
    }

    PipeLane ln;
    ln.k = nat_address(&Ks[0][0], lane);
    tr_addresses(ln.v, &Vs[0][0], lane);
    ln.ones = all_ones();
    PipeState<NC> st;
    pipe_state_init(st);

    // Tile T (64 keys, two steps) lives in ring slot T % 4.  Step 2T reads its values and the next step's keys from that slot;
    // then the block waits for tile T+1, refills the slot of tile T-1 with tile T+3, and step 2T+1 reads the keys of step 2T+2
    // from the slot of tile T+1.
    auto next_tile = [&](int T) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kPipeAhead - 1)));
      block_barrier();
      pipe_issue<NW, 64, GATHER>(dma, 64 * (T + 1 + kPipeAhead), ((T + 1 + kPipeAhead) & 3) * kPipeTileBytes);
    };
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * kPipeAhead));
    __syncthreads();
    const int last = (n - 1) >> 6;   // the last tile
    if (q0w >= ge) {
      // Every query row of this wave lies past the end of the group (last tile of a group): it only moves
      // its share of the K/V tiles and keeps the barriers of the loop below, one for one, so that no
      // matrix or vector work is spent on padding.
      for (int T = 0; T < last; ++T) next_tile(T);
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      return;
    }
    Scores<NC> s_a, s_b;   // scores of even / odd steps
    float mx[NC];
    step_scores<64>(ln, 0, qf, s_a);
#pragma unroll
    for (int q = 0; q < NC; ++q) mx[q] = column_exponents(s_a, q, c, 0.f);
    for (int T = 0; T < last; ++T) {
      const unsigned slot = (T & 3) * kPipeTileBytes, next = ((T + 1) & 3) * kPipeTileBytes;
      maybe_rescale(st, mx, s_a);
      pipe_step<64, true, true, true, kRow32Bytes, 0>(ln, slot, slot, qf, st, s_a, s_b, mx, c, [&]() { next_tile(T); });
      maybe_rescale(st, mx, s_b);
      pipe_step<64, true, true, true, 0, kRow32Bytes>(ln, next, slot, qf, st, s_b, s_a, mx, c, []() {});
    }
    // the last tile, possibly partial
    unsigned voff = (last & 3) * kPipeTileBytes;
    if (n - 64 * last < 32) {
      mask_step(s_a, 64 * last, lane >> 4, n);
      step_max(s_a, mx);
    }
    if (n - 64 * last > 32) {
      maybe_rescale(st, mx, s_a);
      pipe_step<64, true, true, true, kRow32Bytes, 0>(ln, voff, voff, qf, st, s_a, s_b, mx, c, []() {});
      mask_step(s_b, 64 * last + 32, lane >> 4, n);
      step_max(s_b, mx);
      copy_scores(s_a, s_b);
      voff += kRow32Bytes;
    }
    maybe_rescale(st, mx, s_a);
    pipe_step<64, true, true, false, 0, 0>(ln, 0, voff, qf, st, s_a, s_b, mx, c, []() {});

    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // drain the look-ahead loads before the LDS is released
    if (piece) store_piece(st, sw, piece_row);
    else store_output<GATHER>(st, q0w, ge, head, head_off, H, oh, lse, perm, gate, o_tok);
  };
  if (ROWS > 256 && ge - q0 > 256) sweep(std::integral_constant<int, ROWS / 128>());
  else sweep(std::integral_constant<int, 2>());
}

template <int ROWS, bool GATHER = false, bool SPLIT = false>
__global__ __launch_bounds__(512) void attn_fwd_bf16_pipe_kernel(
    const unsigned short* __restrict__ qh, const unsigned short* __restrict__ kh,
    const unsigned short* __restrict__ vh, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, unsigned short* __restrict__ oh,
    float* __restrict__ lse, const int32_t* __restrict__ perm = nullptr,
    const float* __restrict__ gate = nullptr, SplitWs sw = {}, unsigned short* __restrict__ o_tok = nullptr) {
  attn_fwd_block<ROWS, GATHER, SPLIT>(blockIdx.x, qh, kh, vh, cu_q, cu_k, tile_start, M, Nq, Nk, H, scale, oh, lse, perm, gate, sw, o_tok);
}

// Several calls in one launch (the branches of Section 3.2's block): call i takes the blocks from first[i] on, a multiple of 8 (the XCDs).
struct AttnFwdCall {
  const unsigned short *qh, *kh, *vh;
  const int32_t *cu_q, *cu_k, *tile_start;
  int64_t Nq, Nk;
  unsigned short* oh;
  float* lse;
  int M;
};
struct AttnFwdCalls {
  AttnFwdCall c[kMaxCalls];
  int first[kMaxCalls];   // INT_MAX: none
};
template <typename T>
__device__ __forceinline__ int call_of_block(const T& calls, int block) {
  int i = 0;
#pragma unroll
  for (int k = 1; k < kMaxCalls; ++k) i += block >= calls.first[k];
  return i;
}
template <int ROWS>
__global__ __launch_bounds__(512) void attn_fwd_bf16_pipe_calls_kernel(AttnFwdCalls calls, int H, float scale) {
  const int i = call_of_block(calls, blockIdx.x);
  const AttnFwdCall& c = calls.c[i];
  attn_fwd_block<ROWS, false, false>(blockIdx.x - calls.first[i], c.qh, c.kh, c.vh, c.cu_q, c.cu_k, c.tile_start, c.M, c.Nq, c.Nk, H, scale,
                                     c.oh, c.lse, nullptr, nullptr, SplitWs{}, nullptr);
}

// Pieces of every query tile of the last round, with their maxima m_k in exponents of two: O = sum O_k 2^(m_k - m) / l,
// l = sum l_k 2^(m_k - m).  NaN and infinite scores end as in a whole tile; only a group without keys gets zero rows.
static __global__ __launch_bounds__(256) void split_fwd_kernel(SplitWs sw, int rows, const int32_t* __restrict__ cu_q,
                                                               const int32_t* __restrict__ cu_k, int M, int H, int64_t N,
                                                               unsigned short* __restrict__ oh,
                                                               float* __restrict__ lse, const int32_t* __restrict__ perm,
                                                               const float* __restrict__ gate, unsigned short* __restrict__ o_tok) {
  const int per_head = count_tiles(cu_q, M, rows);
  const SplitShape s = split_shape(per_head * H);
  if (s.splits == 1 || (int)blockIdx.x >= s.left) return;
  int head, tile;
  decode_work(s.full + blockIdx.x, per_head, H, head, tile);
  TileInfo ti;
  if (!find_tile(cu_q, M, rows, tile, ti)) return;
  const bool keys = cu_k[ti.group + 1] > cu_k[ti.group];
  const int col = (threadIdx.x & 31) * 4, r = blockIdx.y * 8 + (threadIdx.x >> 5);
  if (ti.tile_row + r >= ti.row_end) return;
  const size_t first = (size_t)blockIdx.x * s.splits * rows + r;   // piece k is k * rows further
  floatx4_t v[kMaxSplits];
  floatx2_t ml[kMaxSplits];
#pragma unroll
  for (int k = 0; k < kMaxSplits; ++k) {
    const size_t row = first + (k < s.splits ? k : 0) * (size_t)rows;
    v[k] = *(const floatx4_t*)(sw.part + row * kHeadDim + col);
    ml[k] = *(const floatx2_t*)(sw.stat + row * 2);
  }
  float m = -INFINITY, l = 0.f;
#pragma unroll
  for (int k = 0; k < kMaxSplits; ++k) m = fmaxf(m, ml[k][0]);
  floatx4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < kMaxSplits; ++k)
    if (k < s.splits) {
      const float w = ml[k][0] == m ? 1.f : fast_exp2(ml[k][0] - m);   // equal: also both -inf
      l += ml[k][1] * w;
      o += v[k] * w;
    }
  const int64_t orow = (int64_t)head * N + ti.tile_row + r;
  const uintx2_t w = pack4(o, keys ? 1.f / l : 0.f);
  *(uintx2_t*)(oh + orow * kHeadDim + col) = w;
  if (o_tok) {
    const int tok = perm[ti.tile_row + r];
    *(uintx2_t*)(o_tok + ((int64_t)tok * H + head) * kHeadDim + col) = scale4(w, gate[tok]);
  }
  if (col == 0) lse[orow] = keys ? m * 0.6931471805599453f + logf(l) : -INFINITY;
}

}  // namespace moga
