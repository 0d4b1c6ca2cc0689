// bf16 forward kernel of the group attention for SMALL groups (head_dim 128): the static groups of
// Section 3.2 have a few hundred to a few thousand rows, where the 8-wave kernel of attn_pipe.h, in a call of few
// rounds, leaves CUs idle with its 384- or 256-row tiles and its three-tile prologue is not amortised.
//
// Same step (pipe_step) and operand layouts, but a block is 4 waves x 32 query rows (128-row
// tiles) and streams K/V in tiles of 32 keys through a ring of four 8 KB + 8 KB slots: 64 KB of
// LDS, so TWO blocks share a CU.  They run independently: one block's prologue, epilogue and
// barrier waits are covered by the other block's waves on the same SIMDs.
#pragma once

#include "attn_pipe.h"

namespace moga {

constexpr int kSmallTileBytes = 32 * kHeadDim * 2;   // 8 KB per K (or V) tile of 32 keys

// Arguments as attn_fwd_bf16_pipe_kernel (no gather mode); tiles of 128 query rows.
__device__ __forceinline__ void attn_fwd_small_block(
    int block, const unsigned short* __restrict__ qh, const unsigned short* __restrict__ kh,
    const unsigned short* __restrict__ vh, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, unsigned short* __restrict__ oh,
    float* __restrict__ lse, const int32_t* __restrict__ perm, const float* __restrict__ gate,
    unsigned short* __restrict__ o_tok) {
  constexpr int BM = 128;
  constexpr int kDmaPerTile = 2 * kDmaLoads<4, 32>;   // direct-to-LDS instructions per thread per tile
  constexpr int kAhead = 2;        // tiles in flight beyond the one being waited for
  __shared__ __attribute__((aligned(1024))) unsigned short Ks[4][32 * kHeadDim];
  __shared__ __attribute__((aligned(1024))) unsigned short Vs[4][32 * kHeadDim];

  WorkTile sp;
  if (!find_work<false>(cu_q, tile_start, M, H, BM, block, sp)) return;
  const TileInfo& ti = sp.ti;
  const int head = sp.head;
  const int ge = ti.row_end, q0 = ti.tile_row;   // query rows of the group end at ge
  const int gs = cu_k[ti.group];                 // first key row of the group
  const int n = cu_k[ti.group + 1] - gs;         // number of keys

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int q0w = q0 + wave * 32;   // first query row of this wave
  const int64_t head_off = (int64_t)head * Nq;
  const int64_t head_off_k = (int64_t)head * Nk;
  const float c = scale * 1.4426950408889634f;

  if (n <= 0) {   // queries without keys: zero output, lse = -inf (block-uniform branch)
    store_zero_rows<false, 2>(q0w, ge, head, head_off, H, oh, lse, perm, o_tok);
    return;
  }

  bf16x8_t qf[2][4];
  load_columns<false>(qf, qh, q0w, ge, head, head_off, H, nullptr);

  PipeDma dma;
  dma.kbase = uniform_ptr(kh + (head_off_k + gs) * kHeadDim);
  dma.vbase = uniform_ptr(vh + (head_off_k + gs) * kHeadDim);
  dma_lanes<4, 32>(dma, &Ks[0][0], &Vs[0][0], wave, lane);
  dma.last_row = n - 1;
#pragma unroll
  for (int t = 0; t <= kAhead; ++t) pipe_issue<4, 32, false>(dma, 32 * t, t * kSmallTileBytes);   // rows are clamped: always issued

  PipeLane ln;
  ln.k = nat_address(&Ks[0][0], lane);
  tr_addresses(ln.v, &Vs[0][0], lane);
  ln.ones = all_ones();
  PipeState<2> st;
  pipe_state_init(st);

  const int nsteps = (n + 31) >> 5;
  const int nfull = n >> 5;   // steps whose 32 keys are all inside the group

  // prologue: scores of step 0 (tile 0)
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * kAhead));
  __syncthreads();
  if (q0w >= ge) {
    // every query row of this wave lies past the end of the group: it only moves its share of the K/V
    // tiles and keeps the barriers of the loops below, one per step
    for (int s = 0; s < nsteps; ++s) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kAhead - 1)));
      __syncthreads();
      pipe_issue<4, 32, false>(dma, 32 * (s + 1 + kAhead), ((s + 1 + kAhead) & 3) * kSmallTileBytes);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    return;
  }
  StepScores s_a, s_b;   // scores of even / odd steps
  float mx[2];
  step_scores<32>(ln, 0, qf, s_a);
#pragma unroll
  for (int q = 0; q < 2; ++q) mx[q] = column_exponents(s_a, q, c, 0.f);
  if (nfull == 0) {
    mask_step(s_a, 0, lane >> 4, n);
    step_max(s_a, mx);
  }

  // main loop.  Step s (= tile s) lives in ring slot s % 4: it reads its values from that slot and
  // the keys of step s+1 from the next one.  At the top of a step the block waits for tile s+1 and
  // refills the slot of tile s-1 with tile s+3.  Four steps per iteration: every LDS offset is an
  // immediate.
  int s = 0;
#define MOGA_SMALL_STEP(B, SA, SB)                                                        \
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kAhead - 1)));                     \
  __syncthreads();                                                                        \
  pipe_issue<4, 32, false>(dma, 32 * (s + (B) + 1 + kAhead), (((B) + 1 + kAhead) & 3) * kSmallTileBytes);             \
  maybe_rescale(st, mx, SA);                                                          \
  pipe_step<32, false, false, true, (((B) + 1) & 3) * kSmallTileBytes, (B) * kSmallTileBytes>(ln, 0, 0, qf, st, SA, SB, mx, c, []() {});
  for (; s + 4 <= nfull - 1; s += 4) {   // steps s .. s+3 and their successors are full
    MOGA_SMALL_STEP(0, s_a, s_b)
    MOGA_SMALL_STEP(1, s_b, s_a)
    MOGA_SMALL_STEP(2, s_a, s_b)
    MOGA_SMALL_STEP(3, s_b, s_a)
  }
#undef MOGA_SMALL_STEP

  // tail: at most four steps and a partial one (s is a multiple of 4 here), ring offsets at run time
  for (; s < nsteps; ++s) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kAhead - 1)));
    __syncthreads();
    pipe_issue<4, 32, false>(dma, 32 * (s + 1 + kAhead), ((s + 1 + kAhead) & 3) * kSmallTileBytes);
    const bool has_next = s + 1 < nsteps;
    maybe_rescale(st, mx, s_a);
    const unsigned voff = (unsigned)(s & 3) * kSmallTileBytes;
    const unsigned koff = (unsigned)((s + 1) & 3) * kSmallTileBytes;
    if (has_next) {
      pipe_step<32, true, false, true, 0, 0>(ln, koff, voff, qf, st, s_a, s_b, mx, c, []() {});
      if (s + 1 >= nfull) {
        mask_step(s_b, 32 * (s + 1), lane >> 4, n);
        step_max(s_b, mx);
      }
      copy_scores(s_a, s_b);
    } else {
      pipe_step<32, true, false, false, 0, 0>(ln, koff, voff, qf, st, s_a, s_b, mx, c, []() {});
    }
  }

  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // drain the look-ahead loads before the LDS is released
  store_output<false>(st, q0w, ge, head, head_off, H, oh, lse, perm, gate, o_tok);
}

__global__ __launch_bounds__(256, 2) void attn_fwd_bf16_small_kernel(
    const unsigned short* __restrict__ qh, const unsigned short* __restrict__ kh,
    const unsigned short* __restrict__ vh, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ cu_k, const int32_t* __restrict__ tile_start, int M,
    int64_t Nq, int64_t Nk, int H, float scale, unsigned short* __restrict__ oh,
    float* __restrict__ lse, const int32_t* __restrict__ perm, const float* __restrict__ gate,
    unsigned short* __restrict__ o_tok) {
  attn_fwd_small_block(blockIdx.x, qh, kh, vh, cu_q, cu_k, tile_start, M, Nq, Nk, H, scale, oh, lse, perm, gate, o_tok);
}

__global__ __launch_bounds__(256, 2) void attn_fwd_bf16_small_calls_kernel(AttnFwdCalls calls, int H, float scale) {
  const int i = call_of_block(calls, blockIdx.x);
  const AttnFwdCall& c = calls.c[i];
  attn_fwd_small_block(blockIdx.x - calls.first[i], c.qh, c.kh, c.vh, c.cu_q, c.cu_k, c.tile_start, c.M, c.Nq, c.Nk, H, scale, c.oh, c.lse,
                       nullptr, nullptr, nullptr);
}

}  // namespace moga
