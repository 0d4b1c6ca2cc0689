// Software-pipelined bf16 forward kernel of the group attention (head_dim 128).
//
// 8 waves per block, 32 query rows per wave (256-row query tiles), two waves per SIMD.
// Keys are consumed in steps of 32.  While the matrix cores compute the scores of step s+1
// (S^T = K Q^T), the vector units exponentiate the scores of step s; while the matrix cores
// accumulate O^T += V^T P^T of step s, the vector units reduce the maximum of step s+1.
// K/V tiles of 64 keys (two steps) are streamed global -> LDS with direct-to-LDS loads into
// a ring of four buffers, two tiles ahead of their use; one block-wide barrier per tile.
//
// Bound by the energy of the matrix instructions at the board's power cap and by the issue of a wave's own
// instruction stream.  Against the same kernel on 32x32x16: 182.1 -> 175.4 ms at 580,320 x 40 heads, 32 groups,
// 0.817 -> 0.793 ms at 32,760 x 12, 8 groups (clock 1.80 -> 1.94 GHz for 8 % more cycles).
#pragma once

#include "attn_common.h"

namespace moga {

constexpr int kPipeNBuf = 4;                      // LDS ring: tiles of 64 keys
constexpr int kPipeAhead = 2;                     // tiles in flight beyond the one being waited for
constexpr int kPipeTileBytes = 64 * kHeadDim * 2; // 16 KB per K (or V) tile

struct PipeLane {
  unsigned k[4];   // K rows
  unsigned v[8];   // V transposed
  bf16x8_t pairs;  // A operand of the row sums: lane (r, g) has row r's ones if they are among its keys 8 g .. 8 g + 7
};

__device__ __forceinline__ bf16x8_t pair_ones(int lane) {
  const int r = lane & 15;
  uintx4_t v;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = r == 4 * (lane >> 4) + i ? 0x3f803f80u : 0u;
  return __builtin_bit_cast(bf16x8_t, v);
}

// The sum of a row's sixteen shares, four in each of its four lanes.
__device__ __forceinline__ float row_sum(const floatx4_t& l) {
  float s = (l[0] + l[1]) + (l[2] + l[3]);
  s += __shfl_xor(s, 16, kWave);
  return s + __shfl_xor(s, 32, kWave);
}

// Raw scores of a step: [key operand t][query half]; register i is key 8 g + 4 t + i of query column r
typedef floatx4_t StepScores[2][2];

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// Maximum of a lane's own eight scores per query (the other keys of the step are in three other lanes)
__device__ __forceinline__ void step_max(const StepScores& s, float (&mx)[2]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float t = max3(s[0][q][0], s[0][q][1], s[0][q][2]);
    t = max3(t, s[0][q][3], s[1][q][0]);
    t = max3(t, s[1][q][1], s[1][q][2]);
    mx[q] = fmaxf(t, s[1][q][3]);
  }
}

__device__ __forceinline__ void mask_step(StepScores& s, int first_key, int g, int end) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (first_key + 8 * g + 4 * t + i >= end) s[t][q][i] = -INFINITY;
}

__device__ __forceinline__ void copy_scores(StepScores& to, const StepScores& from) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int q = 0; q < 2; ++q) to[t][q] = from[t][q];
}

__device__ __forceinline__ floatx4_t quarter(const floatx16_t& v, int k) {
  return floatx4_t{v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]};
}

struct PipeState {
  // O^T: [d tiles 4 D .. 4 D + 3][query half], 16 registers each.  As sixteen vectors of four the compiler joins the two
  // sides of the rare branch in maybe_rescale by moving all 64 registers in every step.
  floatx16_t o[2][2];
  floatx4_t l[2];                 // this lane's shares of the row sum: register i has the keys 8 g + 2 i and + 1 of all steps
  float m[2], negmc[2];           // running max (raw score units), -m*c
  float thresh[2];                // m + tau: the max is raised only when a score exceeds this
};

__device__ __forceinline__ void pipe_state_init(PipeState& st) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    st.m[q] = -INFINITY;
    st.l[q] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    st.negmc[q] = 0.f;
    st.thresh[q] = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) st.o[0][q][e] = st.o[1][q][e] = 0.f;
  }
}

// The four lanes of a query compare their own maxima with the common threshold; only when one exceeds it is the
// maximum taken over all four.
__device__ __forceinline__ void maybe_rescale(PipeState& st, const float (&mx)[2], float c, float tau) {
  if (__builtin_amdgcn_ballot_w64(mx[0] > st.thresh[0] || mx[1] > st.thresh[1]) != 0) {   // wave-uniform; after the first step this is rare
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float all = fmaxf(mx[q], __shfl_xor(mx[q], 16, kWave));
      all = fmaxf(all, __shfl_xor(all, 32, kWave));
      const float m_new = fmaxf(st.m[q], all);
      const float alpha = fast_exp2((st.m[q] - m_new) * c);
      st.m[q] = m_new;
      st.negmc[q] = -m_new * c;
      st.thresh[q] = m_new + tau;
      st.l[q] *= alpha;
#pragma unroll
      for (int D = 0; D < 2; ++D)
#pragma unroll
        for (int i = 0; i < 16; ++i) st.o[D][q][i] *= alpha;
    }
  }
}

// Scores of a whole step from its K rows at byte offset `off`.
__device__ __forceinline__ void step_scores(const PipeLane& ln, unsigned off, const bf16x8_t (&qf)[2][4], StepScores& s) {
  bf16x8_t kf[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kf[t][ks] = lds_read_b128(ln.k[ks] + off + t * kRow4Bytes);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        s[t][q] = mfma16(kf[t][ks], qf[q][ks], ks == 0 ? floatx4_t{0.f, 0.f, 0.f, 0.f} : s[t][q]);
}

// One pipeline step.  koff: byte offset (ring slot + half) of the NEXT step's keys; voff: byte
// offset of the CURRENT step's values.  s_cur holds the current step's raw scores; s_next
// receives the next step's raw scores (if HAS_NEXT) and mx their lane maxima.
template <bool PRIO, bool HAS_NEXT, int KOFF = 0, int VOFF = 0>
__device__ __forceinline__ void pipe_step(const PipeLane& ln, unsigned koff, unsigned voff, const bf16x8_t (&qf)[2][4],
                                          PipeState& st, const StepScores& s_cur, StepScores& s_next, float (&mx)[2],
                                          float c) {
  // The scores and exponentials are the long chain of a step: they go first when the SIMD's two waves compete, and the
  // other wave's PV products fill the gaps (580,320 x 40 heads: 175.4 -> 169.4 ms; the other way round 5 % slower).
  // From the step's first LDS reads on, and the row sums last among the products: 62,400 x 12 heads on zeros 3.08 -> 3.00 ms,
  // 32,760 x 12 669 -> 666 us, within the noise where the power limit binds.
  wave_priority<PRIO, 1>();
  bf16x8_t kf[2][4];
  if (HAS_NEXT) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int t = 0; t < 2; ++t) kf[t][ks] = lds_read_b128(ln.k[ks] + koff + KOFF + t * kRow4Bytes);
  }
  bf16x8_t vf[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) vf[dt] = lds_read_tr_frag(ln.v[dt] + voff + VOFF);

  // P = exp2(S*c - m*c), packed to bf16; row sum from the rounded values
  unsigned int pk[2][4];
  if (HAS_NEXT) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < 2; ++q) s_next[t][q] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (HAS_NEXT) {
        s_next[0][q] = mfma16(kf[0][ks], qf[q][ks], s_next[0][q]);
        s_next[1][q] = mfma16(kf[1][ks], qf[q][ks], s_next[1][q]);
      }
      const floatx4_t& v = s_cur[ks >> 1][q];
      const float p0 = fast_exp2(fmaf(v[2 * (ks & 1)], c, st.negmc[q]));
      const float p1 = fast_exp2(fmaf(v[2 * (ks & 1) + 1], c, st.negmc[q]));
      pk[q][ks] = pack_bf16x2(p0, p1);
    }
  }
  wave_priority<PRIO, 0>();
  bf16x8_t pf[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) pf[q] = __builtin_bit_cast(bf16x8_t, uintx4_t{pk[q][0], pk[q][1], pk[q][2], pk[q][3]});
  // The row sums are one more d tile, whose row j has ones at keys 2 j and 2 j + 1 of the step: v_dot2c_f32_bf16, which summed two of the rounded weights at a time, does not run
  // beside the matrix instructions (alternating with them it adds its 8 cycles to their 16, where an fma or a conversion adds
  // none), and eight of them a step cost more than these two products: 62,400 x 12 heads, 5 groups 3.89 -> 3.70 ms (on zeros
  // 3.33 -> 3.07), 32,760 x 12, 8 groups 698 -> 676 us, 99,840 x 40, 16 groups 10.7 -> 10.35 ms.
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      floatx16_t& o = st.o[dt >> 2][q];
      const floatx4_t t = mfma16(vf[dt], pf[q], quarter(o, dt & 3));
#pragma unroll
      for (int e = 0; e < 4; ++e) o[4 * (dt & 3) + e] = t[e];
    }
#pragma unroll
  for (int q = 0; q < 2; ++q) st.l[q] = mfma16(ln.pairs, pf[q], st.l[q]);
  if (HAS_NEXT) step_max(s_next, mx);
}

// Output rows of a wave (query columns r and 16 + r of its 32 rows from q0w): O / l, times the row's gate in gather mode,
// and the log-sum-exp.  Register i of d tile dt is d = 16 dt + 4 g + i.
// o_tok (not in gather mode): NULL, or where the rows also go in token order [N, H, 128], rounded and then times the gate.
template <bool GATHER>
__device__ __forceinline__ void store_output(const PipeState& st, int q0w, int ge, int head, int64_t head_off, int H, float scale,
                                             unsigned short* __restrict__ oh, float* __restrict__ lse,
                                             const int32_t* __restrict__ perm, const float* __restrict__ gate,
                                             unsigned short* __restrict__ o_tok) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float lt = row_sum(st.l[q]);
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
      if (g == 0) lse[head_off + qrow] = st.m[q] * scale + logf(lt);
    }
  }
}

// A piece's O, maximum and sum of this wave's rows, not yet divided.
__device__ __forceinline__ void store_piece(const PipeState& st, const SplitWs& sw, int slot, int wave) {
  const int lane = threadIdx.x & 63;
  const size_t row0 = slot * kSplitRows + 32 * wave;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float lt = row_sum(st.l[q]);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) store_partial(sw.part + row0 * kHeadDim, dt, q, quarter(st.o[dt >> 2][q], dt & 3));
    if (lane < 16) *(floatx2_t*)(sw.stat + (row0 + 16 * q + lane) * 2) = floatx2_t{st.m[q], lt};
  }
}
__device__ __forceinline__ void store_empty_piece(const SplitWs& sw, int slot, int wave) {
  const int lane = threadIdx.x & 63;
  const size_t row0 = slot * kSplitRows + 32 * wave;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) store_partial(sw.part + row0 * kHeadDim, dt, q, floatx4_t{0.f, 0.f, 0.f, 0.f});
    if (lane < 16) *(floatx2_t*)(sw.stat + (row0 + 16 * q + lane) * 2) = floatx2_t{-INFINITY, 0.f};
  }
}

// Zero output rows of a wave whose group has no keys (lse = -inf if given); `tok`: NULL, or the rows in token order.
template <bool GATHER>
__device__ __forceinline__ void store_zero_rows(int row0, int ge, int head, int64_t head_off, int H, unsigned short* __restrict__ out,
                                                float* __restrict__ lse, const int32_t* __restrict__ perm,
                                                unsigned short* __restrict__ tok) {
  const int lane = threadIdx.x & 63, row = row0 + (lane & 31), h = lane >> 5;
  if (row >= ge) return;
  const uintx4_t z = {0u, 0u, 0u, 0u};
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

// B fragments of a wave's 32 rows from row0 (clamped to the last row of the group): columns 16 c + r, d = 32 ks + 8 g ..
template <bool GATHER>
__device__ __forceinline__ void load_columns(bf16x8_t (&f)[2][4], const unsigned short* __restrict__ src, int row0, int ge, int head,
                                             int64_t head_off, int H, const int32_t* __restrict__ perm) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int row = min(row0 + 16 * c + (lane & 15), ge - 1);
    const int64_t irow = GATHER ? (int64_t)perm[row] * H + head : head_off + row;
    const unsigned short* p = src + irow * kHeadDim + 8 * (lane >> 4);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) f[c][ks] = *(const bf16x8_t*)(p + 32 * ks);
  }
}

// The fragments are in their registers: the compiler waits for their loads here and nowhere later.
__device__ __forceinline__ void settle(bf16x8_t (&f)[2][4]) {
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(f[c][ks]));
}

struct PipeDma {
  const void* kbase;   // first K row of this head's group (wave-uniform)
  const void* vbase;
  unsigned lds_k, lds_v;   // LDS byte address of this wave's first row in buffer 0 (wave-uniform)
  int row0;                // this lane's row inside a tile for round 0 (round i is + 4*NW*i)
  unsigned chunk_off;      // swizzled 16-byte chunk inside the row, in bytes
  int last_row;            // last valid row, relative to the group's first row
  // gather mode: rows are fetched through an index list from token-major tensors; kbase / vbase
  // then point at token 0 of this head
  const int32_t* rows;     // index list at the group's first row (wave-uniform)
  int64_t tok_stride;      // bytes between two tokens
  int wave_row;            // 4 * wave (wave-uniform)
  int last_index;          // last readable entry of `rows` (the list ends there; entries past the
                           // group's own rows belong to other groups and are harmless: those rows are masked)
  // tokens of the rows this wave moves in the next tile to be issued, rounds 0 and 1 (wave-uniform;
  // separate scalars so that they stay in scalar registers)
  int ta0, ta1, ta2, ta3, tb0, tb1, tb2, tb3;
};

// Issue the loads of the 64-key tile starting at group-relative row kv0 into ring slot `buf`:
// 16/NW rounds, each wave moving 4 rows of K and 4 rows of V per round.
template <int NW>
__device__ __forceinline__ void pipe_issue_tile(const PipeDma& d, int kv0, int buf) {
  const unsigned boff = (unsigned)buf * kPipeTileBytes;
#pragma unroll
  for (int i = 0; i < 16 / NW; ++i) {
    const int row = min(kv0 + d.row0 + 4 * NW * i, d.last_row);
    // four waves: every other round is 16 rows further, which the swizzle turns into chunk ^ 3
    const unsigned off = (unsigned)row * (kHeadDim * 2) + (NW == 4 && (i & 1) ? d.chunk_off ^ 48u : d.chunk_off);
    lds_dma16_soff(d.kbase, off, d.lds_k + boff + i * 4 * NW * 256);
    lds_dma16_soff(d.vbase, off, d.lds_v + boff + i * 4 * NW * 256);
  }
}

// Gather mode: the tokens of the tile's rows were read (as scalars) while the previous tile was
// issued; select this lane's token, form the two 64-bit addresses, issue, then read the tokens of
// the following tile.
// Scalar (constant-address-space) read of one index: address and result are wave-uniform.
__device__ __forceinline__ int scalar_load_index(const int32_t* p, int i) {
  typedef const int32_t __attribute__((address_space(4))) * cptr;
  return __builtin_amdgcn_readfirstlane(((cptr)(uintptr_t)p)[i]);
}

typedef int intx4_t __attribute__((ext_vector_type(4)));

// Four consecutive indices with one 16-byte scalar load.
__device__ __forceinline__ intx4_t scalar_load_index4(const int32_t* p, int i) {
  typedef const intx4_t __attribute__((address_space(4), aligned(4))) * cptr4;
  return *(cptr4)(uintptr_t)(p + i);
}

template <int NW>
__device__ __forceinline__ void pipe_load_tokens(PipeDma& d, int kv0) {
  const int r0 = kv0 + d.wave_row;
  if (NW == 8 && r0 + 35 <= d.last_index) {   // the common case: two 16-byte scalar loads, no clamping
    const intx4_t a = scalar_load_index4(d.rows, r0), b = scalar_load_index4(d.rows, r0 + 32);
    d.ta0 = __builtin_amdgcn_readfirstlane(a[0]);
    d.ta1 = __builtin_amdgcn_readfirstlane(a[1]);
    d.ta2 = __builtin_amdgcn_readfirstlane(a[2]);
    d.ta3 = __builtin_amdgcn_readfirstlane(a[3]);
    d.tb0 = __builtin_amdgcn_readfirstlane(b[0]);
    d.tb1 = __builtin_amdgcn_readfirstlane(b[1]);
    d.tb2 = __builtin_amdgcn_readfirstlane(b[2]);
    d.tb3 = __builtin_amdgcn_readfirstlane(b[3]);
    return;
  }
  d.ta0 = scalar_load_index(d.rows, min(r0 + 0, d.last_row));
  d.ta1 = scalar_load_index(d.rows, min(r0 + 1, d.last_row));
  d.ta2 = scalar_load_index(d.rows, min(r0 + 2, d.last_row));
  d.ta3 = scalar_load_index(d.rows, min(r0 + 3, d.last_row));
  if (NW == 8) {
    d.tb0 = scalar_load_index(d.rows, min(r0 + 32, d.last_row));
    d.tb1 = scalar_load_index(d.rows, min(r0 + 33, d.last_row));
    d.tb2 = scalar_load_index(d.rows, min(r0 + 34, d.last_row));
    d.tb3 = scalar_load_index(d.rows, min(r0 + 35, d.last_row));
  }
}

__device__ __forceinline__ int select4(int sub, int a, int b, int c, int e) {
  int t = a;
  t = sub == 1 ? b : t;
  t = sub == 2 ? c : t;
  t = sub == 3 ? e : t;
  return t;
}

template <int NW>
__device__ __forceinline__ void pipe_issue_tile_gather(PipeDma& d, int kv0, int buf) {
  static_assert(NW == 8, "gather mode moves two rounds of four rows per wave");
  const unsigned boff = (unsigned)buf * kPipeTileBytes;
  const int sub = d.row0 & 3;
  const int64_t off_a = (int64_t)select4(sub, d.ta0, d.ta1, d.ta2, d.ta3) * d.tok_stride + d.chunk_off;
  const int64_t off_b = (int64_t)select4(sub, d.tb0, d.tb1, d.tb2, d.tb3) * d.tok_stride + d.chunk_off;
  lds_dma16((const char*)d.kbase + off_a, d.lds_k + boff);
  lds_dma16((const char*)d.vbase + off_a, d.lds_v + boff);
  lds_dma16((const char*)d.kbase + off_b, d.lds_k + boff + 4 * NW * 256);
  lds_dma16((const char*)d.vbase + off_b, d.lds_v + boff + 4 * NW * 256);
  pipe_load_tokens<NW>(d, kv0 + 64);
}

template <int NW, bool GATHER>
__device__ __forceinline__ void pipe_issue(PipeDma& d, int kv0, int buf) {
  if constexpr (GATHER) pipe_issue_tile_gather<NW>(d, kv0, buf);
  else pipe_issue_tile<NW>(d, kv0, buf);
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
template <int NW, bool GATHER = false, bool SPLIT = false>
__global__ __launch_bounds__(NW * 64) void attn_fwd_bf16_pipe_kernel(
    const unsigned short* __restrict__ qh, const unsigned short* __restrict__ kh,
    const unsigned short* __restrict__ vh, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, unsigned short* __restrict__ oh,
    float* __restrict__ lse, const int32_t* __restrict__ perm = nullptr,
    const float* __restrict__ gate = nullptr, SplitWs sw = {}, unsigned short* __restrict__ o_tok = nullptr) {
  constexpr int BM = NW * 32;
  constexpr int kDmaPerTile = 2 * (16 / NW);   // direct-to-LDS instructions per thread per tile
  static_assert(NW == 4 || NW == 8, "4 or 8 waves");
  __shared__ __attribute__((aligned(1024))) unsigned short Ks[kPipeNBuf][64 * kHeadDim];
  __shared__ __attribute__((aligned(1024))) unsigned short Vs[kPipeNBuf][64 * kHeadDim];

  WorkTile sp;
  if (!find_work<SPLIT>(cu_q, tile_start, M, H, BM, blockIdx.x, sp)) return;
  const TileInfo& ti = sp.ti;
  const int head = sp.head;
  const int ge = ti.row_end, q0 = ti.tile_row;   // query rows of the group end at ge
  int gs = cu_k[ti.group];                       // first key row of the group
  int n = cu_k[ti.group + 1] - gs;               // number of keys
  const bool piece = SPLIT && sp.splits > 1;
  if (piece) split_range(sp, gs, n);

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int q0w = q0 + wave * 32;   // first query row of this wave
  const int64_t head_off = (int64_t)head * Nq;
  const int64_t head_off_k = (int64_t)head * Nk;
  const float c = scale * 1.4426950408889634f;
  const float tau = 8.f / c;

  if (n <= 0) {   // queries without keys: zero output, lse = -inf (block-uniform branch)
    if (piece) store_empty_piece(sw, sp.slot, wave);
    else store_zero_rows<GATHER>(q0w, ge, head, head_off, H, oh, lse, perm, o_tok);
    return;
  }

  bf16x8_t qf[2][4];
  load_columns<GATHER>(qf, qh, q0w, ge, head, head_off, H, perm);

  // ---- direct-to-LDS loads: first kPipeAhead + 1 tiles (always issued; rows are clamped)
  PipeDma dma;
  dma.kbase = uniform_ptr(GATHER ? kh + (int64_t)head * kHeadDim : kh + (head_off_k + gs) * kHeadDim);
  dma.vbase = uniform_ptr(GATHER ? vh + (int64_t)head * kHeadDim : vh + (head_off_k + gs) * kHeadDim);
  dma.lds_k = lds_addr_uniform(&Ks[0][0]) + wave * 1024;
  dma.lds_v = lds_addr_uniform(&Vs[0][0]) + wave * 1024;
  dma.row0 = 4 * wave + (lane >> 4);
  dma.chunk_off = (unsigned)(((lane & 15) ^ lds_swizzle(dma.row0)) * 16);
  dma.last_row = n - 1;
  if constexpr (GATHER) {
    dma.rows = (const int32_t*)uniform_ptr(perm + gs);
    dma.tok_stride = (int64_t)H * kHeadDim * 2;
    dma.wave_row = 4 * wave;
    dma.last_index = (int)(Nk - 1) - gs;
    pipe_load_tokens<NW>(dma, 0);
  }
#pragma unroll
  for (int t = 0; t <= kPipeAhead; ++t) pipe_issue<NW, GATHER>(dma, 64 * t, t);

  PipeLane ln;
  nat_addresses(ln.k, &Ks[0][0], lane);
  tr_addresses(ln.v, &Vs[0][0], lane);
  ln.pairs = pair_ones(lane);
  PipeState st;
  pipe_state_init(st);

  const int nsteps = (n + 31) >> 5;
  const int nfull = n >> 5;   // steps whose 32 keys are all inside the group

  // ---- prologue: scores of step 0
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * kPipeAhead));
  __syncthreads();
  if (q0w >= ge) {
    // Every query row of this wave lies past the end of the group (last tile of a group): it only moves
    // its share of the K/V tiles and keeps the barriers of the loops below, one for one, so that no
    // matrix or vector work is spent on padding.
    int s = 0;
    for (; s + 8 <= nfull - 1; s += 8) {
#pragma unroll
      for (int B = 0; B < 4; ++B) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kPipeAhead - 1)));
        __syncthreads();
        pipe_issue<NW, GATHER>(dma, 32 * s + 64 * (B + 1 + kPipeAhead), (B + 1 + kPipeAhead) & 3);
      }
    }
    while (s + 2 <= nfull - 1) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kPipeAhead - 1)));
      __syncthreads();
      pipe_issue<NW, GATHER>(dma, 32 * (s + 2) + 64 * kPipeAhead, ((s >> 1) + 1 + kPipeAhead) & 3);
      s += 2;
    }
    for (; s < nsteps; ++s) {
      if ((s & 1) == 1 && s + 1 < nsteps) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kPipeAhead - 1)));
        __syncthreads();
        pipe_issue<NW, GATHER>(dma, 32 * (s + 1) + 64 * kPipeAhead, (((s >> 1) & 3) + 1 + kPipeAhead) & 3);
      }
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    return;
  }
  StepScores s_a, s_b;   // scores of even / odd steps
  float mx[2];
  step_scores(ln, 0, qf, s_a);
  if (nfull == 0) mask_step(s_a, 0, lane >> 4, n);
  step_max(s_a, mx);

  // ---- main loop.  Tile T (64 keys, two steps) lives in ring slot T % 4.  Step 2T reads its
  // values and the next step's keys from that slot; then the block waits for tile T+1, refills
  // the slot of tile T-1 with tile T+3, and step 2T+1 reads the keys of step 2T+2 from the slot
  // of tile T+1.  Four tiles per iteration so that every LDS offset is an immediate.
  int s = 0;
#define MOGA_FWD_TILE(B)                                                                        \
  maybe_rescale(st, mx, c, tau);                                                            \
  pipe_step<true, true, (B) * kPipeTileBytes + 8192, (B) * kPipeTileBytes>(ln, 0, 0, qf, st, s_a, s_b, mx, c); \
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kPipeAhead - 1)));                       \
  __syncthreads();                                                                              \
  pipe_issue<NW, GATHER>(dma, 32 * s + 64 * ((B) + 1 + kPipeAhead), ((B) + 1 + kPipeAhead) & 3); \
  maybe_rescale(st, mx, c, tau);                                                            \
  pipe_step<true, true, (((B) + 1) & 3) * kPipeTileBytes, (B) * kPipeTileBytes + 8192>(ln, 0, 0, qf, st, s_b, s_a, mx, c);
  for (; s + 8 <= nfull - 1; s += 8) {   // steps s .. s+7 and their successors are full
    MOGA_FWD_TILE(0)
    MOGA_FWD_TILE(1)
    MOGA_FWD_TILE(2)
    MOGA_FWD_TILE(3)
  }
#undef MOGA_FWD_TILE
  // remaining whole tiles, ring offsets at run time (s / 2 is a multiple of 4 on entry)
  while (s + 2 <= nfull - 1) {
    const unsigned slot = ((unsigned)(s >> 1) & 3u) * kPipeTileBytes;
    const unsigned slot_next = ((unsigned)((s >> 1) + 1) & 3u) * kPipeTileBytes;
    maybe_rescale(st, mx, c, tau);
    pipe_step<true, true>(ln, slot + 8192, slot, qf, st, s_a, s_b, mx, c);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kPipeAhead - 1)));
    __syncthreads();
    pipe_issue<NW, GATHER>(dma, 32 * (s + 2) + 64 * kPipeAhead, ((s >> 1) + 1 + kPipeAhead) & 3);
    maybe_rescale(st, mx, c, tau);
    pipe_step<true, true>(ln, slot_next, slot + 8192, qf, st, s_b, s_a, mx, c);
    s += 2;
  }

  // ---- tail: at most three steps (s is even here), the last one possibly partial
  for (; s < nsteps; ++s) {
    const int buf = (s >> 1) & 3, half = s & 1;
    const bool has_next = s + 1 < nsteps;
    if (half == 1 && has_next) {   // the next step starts a new tile
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kPipeAhead - 1)));
      __syncthreads();
      pipe_issue<NW, GATHER>(dma, 32 * (s + 1) + 64 * kPipeAhead, (buf + 1 + kPipeAhead) & 3);
    }
    maybe_rescale(st, mx, c, tau);
    const unsigned voff = buf * kPipeTileBytes + half * 8192;
    const unsigned koff = (half ? ((buf + 1) & 3) : buf) * kPipeTileBytes + (half ? 0 : 8192);
    if (has_next) {
      pipe_step<true, true>(ln, koff, voff, qf, st, s_a, s_b, mx, c);
      if (s + 1 >= nfull) {
        mask_step(s_b, 32 * (s + 1), lane >> 4, n);
        step_max(s_b, mx);
      }
      copy_scores(s_a, s_b);
    } else {
      pipe_step<true, false>(ln, koff, voff, qf, st, s_a, s_b, mx, c);
    }
  }

  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // drain the look-ahead loads before the LDS is released
  if (piece) store_piece(st, sw, sp.slot, wave);
  else store_output<GATHER>(st, q0w, ge, head, head_off, H, scale, oh, lse, perm, gate, o_tok);
}

// Pieces of every query tile of the last round: O = sum O_k 2^((m_k - m) c) / l, l = sum l_k 2^((m_k - m) c).  NaN and
// infinite scores end as in a whole tile; only a group without keys gets zero rows.
static __global__ __launch_bounds__(256) void split_fwd_kernel(SplitWs sw, const int32_t* __restrict__ cu_q,
                                                               const int32_t* __restrict__ cu_k, int M, int H, int64_t N,
                                                               float scale, unsigned short* __restrict__ oh,
                                                               float* __restrict__ lse, const int32_t* __restrict__ perm,
                                                               const float* __restrict__ gate, unsigned short* __restrict__ o_tok) {
  const int per_head = count_tiles(cu_q, M, kSplitRows);
  const SplitShape s = split_shape(per_head * H);
  if (s.splits == 1 || (int)blockIdx.x >= s.left) return;
  int head, tile;
  decode_work(s.full + blockIdx.x, per_head, H, head, tile);
  TileInfo ti;
  if (!find_tile(cu_q, M, kSplitRows, tile, ti)) return;
  const bool keys = cu_k[ti.group + 1] > cu_k[ti.group];
  const float c = scale * 1.4426950408889634f;
  const int col = (threadIdx.x & 31) * 4, r = blockIdx.y * 8 + (threadIdx.x >> 5);
  if (ti.tile_row + r >= ti.row_end) return;
  const size_t first = (size_t)blockIdx.x * s.splits * kSplitRows + r;   // piece k is k * kSplitRows rows further
  floatx4_t v[kMaxSplits];
  floatx2_t ml[kMaxSplits];
#pragma unroll
  for (int k = 0; k < kMaxSplits; ++k) {
    const size_t row = first + (k < s.splits ? k : 0) * kSplitRows;
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
      const float w = ml[k][0] == m ? 1.f : fast_exp2((ml[k][0] - m) * c);   // equal: also both -inf
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
  if (col == 0) lse[orow] = keys ? m * scale + logf(l) : -INFINITY;
}

}  // namespace moga
