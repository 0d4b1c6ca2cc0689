// bf16 backward kernels of the group attention (head_dim 128) on the LDS ring of attn_pipe.h.
//
//   attn_bwd_dq_pipe_kernel   : a wave owns 48 (or 32) query rows (Q, dO fragments, lse, delta and
//                               the dQ^T accumulators in registers) and sweeps 64-key tiles of
//                               K and V; three MFMA products per tile (S^T, dP^T, dQ^T).
//   attn_bwd_dkdv_ab_kernel   : a pair of waves on one SIMD owns 48 (or 32) key rows and sweeps 64-query
//                               tiles of Q, dO, lse and delta; one wave computes S, P and dV^T,
//                               the other dP, dS and dK^T (P handed over through LDS).
// Tiles are streamed global -> LDS by direct-to-LDS loads into a ring of four slots, two tiles
// ahead; one block-wide barrier per tile.  Both also come as 4-wave blocks with a two-slot ring (64 KB of
// LDS), 32 query rows per wave and 32 key rows per pair, two blocks per CU, in one launch (attn_bwd_small_kernel), for groups of a few thousand rows or less.
// All are at the power cap.  LDS fragments read beside the products cost matrix time too: a loop of 16x16x32 products takes 7.2 ns each
// at the top clock, and with a fragment read for every two 8.3 (row fragments) or 8.6 (transposing reads).
#pragma once

#include <type_traits>

#include "attn_pipe.h"

namespace moga {

__device__ __forceinline__ floatx4_t lds_read_f32x4(unsigned addr) {
  return *(const floatx4_t __attribute__((address_space(3)))*)(uintptr_t)addr;
}

// ---------------------------------------------------------------------------------------
// dQ: query-stationary
// ---------------------------------------------------------------------------------------
// A step of 32 keys: for either 16-key operand t of it the scores and dP, then dQ over all 32 keys, the vector work of one among the products
// of the next:
//   S(0) | dP(0), P(0) | S(1), dS(0) | dP(1), P(1) | dS(1), dQ
// Bound by energy at the power cap, as the forward is: with 48 rows per wave a fragment read from LDS feeds three products instead of two,
// and the stream of K/V tiles is a third smaller.  48 rows leave 64 registers beside Q, dO and dQ^T.  What fits them: the scores and dP of 16
// keys at a time instead of 64; delta subtracted from dP (an accumulator that starts from it takes four registers per
// column, for good); one address for K and V, which lie side by side in a slot; the factor c in a scalar register; and only one fragment
// read ahead where scores, P and dP are all there (with two the 96 registers of Q and dO are kept in memory and read in every tile).
// Whole backward, 32 and 48 rows per wave: 99,840 x 40 heads, 16 groups 32.2 -> 31.3 ms, 62,400 x 12, 5 groups 11.70 -> 11.40, 32,760 x
// 12, 8 groups 2.15 -> 2.12, 99,840 x 12, 99 groups 2.155 -> 2.08, 8,000 x 3, 1 group 0.296 -> 0.279 (with 256-row blocks too, to which the
// order of the work is common).  Without priorities 1 to 4 % slower, with scheduling barriers that vector work does not cross 0 to 0.5 %.
//
// nat, tr: the lane's addresses in the tile's slot.  The 24 fragments are read across the step's end, into `ahead` for the next step; `mid` is
// called before the first of those, and may move nat on to the next tile.
constexpr int kDqWin = 2;   // fragments read ahead
// the last fragment that is read before the products of fragment i
constexpr int dq_read_up_to(int i, int nc) { return i + (nc > 2 && i >= 4 && i < 16 ? 1 : kDqWin); }
template <int NC>
struct DqRows {   // a wave's own operands
  bf16x8_t qf[NC][4], dof[NC][4];
  float lse2[NC], neg_dlt[NC];
};
template <bool PRIO, int U, bool MASK, bool NEXT, int NC, typename F>
__device__ __forceinline__ void dq_step(unsigned& nat, const unsigned (&tr)[2], const DqRows<NC>& w, floatx4_t (&dq)[8][NC],
                                        bf16x8_t (&ahead)[kDqWin], float c, int g, int left, F&& mid) {
  constexpr int kKeep = 0x2 | 0x4 | 0x400;   // what may cross: vector, scalar and transcendental instructions
  bf16x8_t fr[24];   // K rows, V rows of operand 0 (ks), of operand 1, then K transposed (dt)
  floatx4_t s[NC], dp[NC];
  unsigned dd[NC][4];
  auto load = [&](int f) {
    if (f < 16) fr[f] = read_nat<64>(nat + ((f >> 2) & 1) * kPipeTileBytes + U * kRow32Bytes, f >> 3, f & 3);
    else if (f < 24) fr[f] = read_tr<64>(tr, U * kRow32Bytes, f - 16);
    else if (NEXT) ahead[f - 24] = read_nat<64>(nat + (U == 0 ? kRow32Bytes : 0), 0, f - 24);
  };
  auto load_at = [&](int i) {
#pragma unroll
    for (int f = dq_read_up_to(i - 1, NC) + 1; f <= dq_read_up_to(i, NC); ++f) load(f);
  };
  auto make_ds = [&](int t, int q) {
#pragma unroll
    for (int i = 0; i < 4; i += 2)
      dd[q][2 * t + (i >> 1)] = pack_bf16x2(s[q][i] * (dp[q][i] + w.neg_dlt[q]), s[q][i + 1] * (dp[q][i + 1] + w.neg_dlt[q]));
  };
#pragma unroll
  for (int f = 0; f < kDqWin; ++f) fr[f] = ahead[f];
  wave_priority<PRIO, 1>();
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    floatx4_t sn[NC];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int f = 8 * t + ks;
      __builtin_amdgcn_sched_barrier(kKeep);
      load_at(f);
#pragma unroll
      for (int q = 0; q < NC; ++q) sn[q] = mfma16(fr[f], w.qf[q][ks], ks == 0 ? floatx4_t{0.f, 0.f, 0.f, 0.f} : sn[q]);
      if (t == 1 && ks < NC) make_ds(0, ks);
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) s[q] = sn[q];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int f = 8 * t + 4 + ks;
      __builtin_amdgcn_sched_barrier(kKeep);
      load_at(f);
#pragma unroll
      for (int q = 0; q < NC; ++q) dp[q] = mfma16(fr[f], w.dof[q][ks], ks == 0 ? floatx4_t{0.f, 0.f, 0.f, 0.f} : dp[q]);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        s[q][ks] = fast_exp2(fmaf(s[q][ks], c, -w.lse2[q]));
        if (MASK && 32 * U + 8 * g + 4 * t + ks >= left) s[q][ks] = 0.f;
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  wave_priority<PRIO, 0>();
  bf16x8_t dsf[NC];
  auto operand = [&](int q) {
    make_ds(1, q);
    dsf[q] = __builtin_bit_cast(bf16x8_t, uintx4_t{dd[q][0], dd[q][1], dd[q][2], dd[q][3]});
  };
  operand(0);
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) {
    if (dt == 8 - kDqWin) mid();
    __builtin_amdgcn_sched_barrier(kKeep);
    load_at(16 + dt);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      dq[dt][q] = mfma16(fr[16 + dt], dsf[q], dq[dt][q]);
      if (dt == 0 && q + 1 < NC) operand(q + 1);
    }
  }
}

// Gradient rows of a wave (columns r, 16 + r .. of its 16 NC rows from row0), times f: to `out` (sorted order, or token order in
// gather mode) and, not in gather mode, to `tok` in token order; either may be NULL.
template <bool GATHER, int NC>
__device__ __forceinline__ void store_gradient(const floatx4_t (&acc)[8][NC], float f, int row0, int ge, int head, int64_t head_off,
                                               int H, unsigned short* __restrict__ out, unsigned short* __restrict__ tok,
                                               const int32_t* __restrict__ perm) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int row = row0 + 16 * c + r;
    if (row < ge) {
      const int64_t trow = GATHER || tok ? (int64_t)perm[row] * H + head : 0;
      unsigned short* op = out + (GATHER ? trow : head_off + row) * kHeadDim + join_channel(g);
      unsigned short* tp = tok + trow * kHeadDim + join_channel(g);
#pragma unroll
      for (int dt = 0; dt < 8; dt += 2) {
        const uintx4_t v = join_tiles(pack4(acc[dt][c], f), pack4(acc[dt + 1][c], f));
        if (GATHER || out) *(uintx4_t*)(op + 16 * dt) = v;
        if (!GATHER && tok) *(uintx4_t*)(tp + 16 * dt) = v;
      }
    }
  }
}

template <int NC>
__device__ __forceinline__ void store_gradient_piece(const floatx4_t (&acc)[8][NC], float* rows) {
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) store_partial(rows, dt, c, acc[dt][c]);
}
template <int NC>
__device__ __forceinline__ void store_zero_piece(float* rows) {
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) store_partial(rows, dt, c, floatx4_t{0.f, 0.f, 0.f, 0.f});
}

// SPLIT (both backward kernels): the last round is cut into pieces (find_work), partial sums in `part`.
// GATHER (both backward kernels): d_oh, qh, kh, vh and the gradient outputs are token-major
// [N, H, 128] and row j of a group is token perm[j]; neg_lse_over_scale / neg_delta stay in
// sorted order [H, N] and carry the gate (see attn_bwd_fused_prepass_kernel), so d_oh is the
// raw upstream gradient of the gated output.
// NB: ring slots of 64 keys (4: two tiles ahead, one block per CU; 2: one tile ahead, 64 KB of LDS, so
// that two 4-wave blocks share a CU -- the variant for small groups).
template <int NB, bool GATHER>
struct DqLds {
  __attribute__((aligned(1024))) unsigned short kv[NB][2][64 * kHeadDim];   // a tile of K, then of V: one address for both
  __attribute__((aligned(256))) int tok[GATHER ? 512 : 1];   // gather mode: tokens of eight tiles
};
constexpr int kDqSlotBytes = 2 * kPipeTileBytes;

// ROWS: query rows of a block, 48 or 32 per wave.
template <int NW, bool GATHER, int NB, int ROWS, bool SPLIT>
__device__ __forceinline__ void attn_bwd_dq_block(
    DqLds<NB, GATHER>& lds, int block, const unsigned short* __restrict__ d_oh, const unsigned short* __restrict__ qh,
    const unsigned short* __restrict__ kh, const unsigned short* __restrict__ vh,
    const float* __restrict__ neg_lse_over_scale, const float* __restrict__ neg_delta,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k,
    const int32_t* __restrict__ tile_start, int M, int64_t Nq, int64_t Nk, int H, float scale,
    unsigned short* __restrict__ d_qh, const int32_t* __restrict__ perm, float* __restrict__ part,
    unsigned short* __restrict__ d_q_tok) {
  constexpr int kDmaPerTile = 2 * kDmaLoads<NW, 64>;
  constexpr int kAhead = NB - 2;   // tiles in flight beyond the one being waited for

  WorkTile sp;
  if (!find_work<SPLIT>(cu_q, tile_start, M, H, ROWS, block, sp)) return;
  const TileInfo& ti = sp.ti;
  const int head = sp.head;
  const int ge = ti.row_end, q0 = ti.tile_row;   // query rows of the group end at ge
  int gs = cu_k[ti.group];                       // first key row of the group
  int n = cu_k[ti.group + 1] - gs;               // number of keys
  const bool piece = SPLIT && sp.splits > 1;
  if (piece) split_range(sp, gs, n);
  gs = __builtin_amdgcn_readfirstlane(gs);
  n = __builtin_amdgcn_readfirstlane(n);

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t head_off = (int64_t)head * Nq;
  const int64_t head_off_k = (int64_t)head * Nk;
  // In a scalar register; the builtin is dropped where the compiler knows that the value is uniform.  The waits are those between a vector
  // instruction and a lane read of its result, and between a lane read and a vector instruction.
  float c;
  asm("s_nop 1\n\tv_readfirstlane_b32 %0, %1\n\ts_nop 2" : "=s"(c) : "v"(scale * 1.4426950408889634f));

  // A wave owns 16 NC query rows: three columns, or two where that is enough for the last tile of a group, which then takes
  // two thirds of the time.
  auto sweep = [&](auto columns) {
    constexpr int NC = columns.value;
    const int q0w = q0 + wave * 16 * NC;   // first query row of this wave
    float* const piece_rows = piece ? part + ((size_t)sp.slot * ROWS + 16 * NC * wave) * kHeadDim : nullptr;
    if (n <= 0) {   // queries without keys: zero gradient (block-uniform branch)
      if (piece) store_zero_piece<NC>(piece_rows);
      else store_zero_rows<GATHER, NC>(q0w, ge, head, head_off, H, d_qh, nullptr, perm, d_q_tok);
      return;
    }

    DqRows<NC> w;
    load_columns<GATHER>(w.qf, qh, q0w, ge, head, head_off, H, perm);
    load_columns<GATHER>(w.dof, d_oh, q0w, ge, head, head_off, H, perm);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const int qrow = min(q0w + 16 * q + (lane & 15), ge - 1);
      w.lse2[q] = -neg_lse_over_scale[head_off + qrow] * c;   // lse * log2(e)
      w.neg_dlt[q] = neg_delta[head_off + qrow];
    }

    PipeDma dma;
    dma.kbase = uniform_ptr(GATHER ? kh + (int64_t)head * kHeadDim : kh + (head_off_k + gs) * kHeadDim);
    dma.vbase = uniform_ptr(GATHER ? vh + (int64_t)head * kHeadDim : vh + (head_off_k + gs) * kHeadDim);
    dma_lanes<NW, 64>(dma, &lds.kv[0][0][0], &lds.kv[0][1][0], wave, lane);
    dma.last_row = n - 1;
    if constexpr (GATHER) {
      dma.rows = uniform_ptr(perm + gs);
      dma.tok_stride = (int64_t)H * kHeadDim * 2;
      dma.lds_tok = lds_addr_uniform(&lds.tok[0]);
      pipe_issue_tokens(dma, 0);
      pipe_issue_tokens(dma, 64);
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    }
    auto issue_tile = [&](int T) { pipe_issue<NW, 64, GATHER>(dma, 64 * T, (T & (NB - 1)) * kDqSlotBytes); };
#pragma unroll
    for (int t = 0; t <= kAhead; ++t) {
      if (GATHER && t == 2) __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kDmaPerTile));   // its tokens
      issue_tile(t);
    }

    // All of the wave's own operands are here before the loop.  Otherwise the compiler, which sees the loads above and not the
    // direct-to-LDS loads, waits for them at their first use, inside the loop: vmcnt(4) .. vmcnt(0) in every tile, that is for
    // the tiles that were issued a moment ago.
    settle(w.qf);
    settle(w.dof);
#pragma unroll
    for (int q = 0; q < NC; ++q) asm volatile("" : "+v"(w.lse2[q]), "+v"(w.neg_dlt[q]));

    floatx4_t dq[8][NC];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int q = 0; q < NC; ++q) dq[dt][q] = floatx4_t{0.f, 0.f, 0.f, 0.f};

    const int g = lane >> 4, last = (n - 1) >> 6;   // the last tile
    const bool active = q0w < ge;   // a wave whose query rows all lie past the end of the group only moves its share of the tiles
    unsigned nat = nat_address(&lds.kv[0][0][0], lane), tr[2];   // in the slot of the tile
    tr_addresses(tr, &lds.kv[0][0][0], lane);
    bf16x8_t ahead[kDqWin];
    auto first_fragments = [&]() {
#pragma unroll
      for (int f = 0; f < kDqWin; ++f) ahead[f] = read_nat<64>(nat, 0, f);
    };
    auto nothing = []() {};
    // tile T lives in ring slot T % NB
    if constexpr (NB == 4) {
      // In tile T the block waits for tile T + 1 and refills the slot of tile T - 1, which every wave has left, with tile T + 3.
      auto next_tile = [&](int T) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kAhead - 1)));
        block_barrier();
        issue_tile(T + 1 + kAhead);
      };
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * kAhead));
      __syncthreads();
      if (!active) {
        for (int T = 0; T < last; ++T) next_tile(T);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        return;
      }
      first_fragments();
      for (int T = 0; T < last; ++T) {
        const unsigned by = (T & 3) == 3 ? -3u * kDqSlotBytes : kDqSlotBytes;
        dq_step<NB == 4, 0, false, true>(nat, tr, w, dq, ahead, c, g, 64, nothing);
        dq_step<NB == 4, 1, false, true>(nat, tr, w, dq, ahead, c, g, 64, [&]() {
          next_tile(T);
          nat = in_register(nat + by);
        });
        tr[0] = in_register(tr[0] + by);
        tr[1] = in_register(tr[1] + by);
      }
    } else {
      for (int T = 0; T < last; ++T) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        __syncthreads();
        issue_tile(T + 1);
        if (active) {
          first_fragments();
          dq_step<NB == 4, 0, false, true>(nat, tr, w, dq, ahead, c, g, 64, nothing);
          dq_step<NB == 4, 1, false, false>(nat, tr, w, dq, ahead, c, g, 64, nothing);
        }
        const unsigned by = T & 1 ? -kDqSlotBytes : kDqSlotBytes;
        nat = in_register(nat + by);
        tr[0] = in_register(tr[0] + by);
        tr[1] = in_register(tr[1] + by);
      }
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      __syncthreads();
      if (!active) return;
      first_fragments();
    }
    // the last tile, possibly partial: masked keys contribute zero
    const int left = n - 64 * last;
    dq_step<NB == 4, 0, true, true>(nat, tr, w, dq, ahead, c, g, left, nothing);
    if (left > 32) dq_step<NB == 4, 1, true, false>(nat, tr, w, dq, ahead, c, g, left, nothing);

    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // drain the look-ahead loads before the LDS is released
    if (piece) store_gradient_piece(dq, piece_rows);
    else store_gradient<GATHER>(dq, scale, q0w, ge, head, head_off, H, d_qh, d_q_tok, perm);
  };
  if (ROWS > 32 * NW && ge - q0 > 32 * NW) sweep(std::integral_constant<int, ROWS / (16 * NW)>());
  else sweep(std::integral_constant<int, 2>());
}

template <int ROWS, bool GATHER = false, bool SPLIT = false>
__global__ __launch_bounds__(512, 1) void attn_bwd_dq_pipe_kernel(
    const unsigned short* __restrict__ d_oh, const unsigned short* __restrict__ qh,
    const unsigned short* __restrict__ kh, const unsigned short* __restrict__ vh,
    const float* __restrict__ neg_lse_over_scale, const float* __restrict__ neg_delta,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k,
    const int32_t* __restrict__ tile_start, int M, int64_t Nq, int64_t Nk, int H, float scale,
    unsigned short* __restrict__ d_qh, const int32_t* __restrict__ perm = nullptr,
    float* __restrict__ part = nullptr, unsigned short* __restrict__ d_q_tok = nullptr) {
  __shared__ DqLds<4, GATHER> lds;
  attn_bwd_dq_block<8, GATHER, 4, ROWS, SPLIT>(lds, blockIdx.x, d_oh, qh, kh, vh, neg_lse_over_scale, neg_delta, cu_q, cu_k, tile_start,
                                               M, Nq, Nk, H, scale, d_qh, perm, part, d_q_tok);
}

// ---------------------------------------------------------------------------------------
// dK, dV with two waves per SIMD: the four products are split between two waves that own the
// same key rows.  Wave A (waves 0-3) holds K and the dV^T accumulators: it computes S = Q K^T,
// P = exp2(c*S - lse*log2e), hands P to its partner through LDS and accumulates dV^T += dO^T P.
// Wave B (waves 4-7, same SIMD as its partner) holds V and the dK^T accumulators: it computes
// dP = dO V^T - delta, takes P, forms dS = P * dP and accumulates dK^T += Q^T dS.  Each wave
// needs half of the accumulators (96 registers for 48 keys), so two waves fit on a SIMD and fill each other's
// waits.  There is one block-wide barrier per 64-query tile (tile landed, ring slot free) and one P buffer
// per pair, and P is handed over in one of two ways:
//   * two-slot ring (small groups, ab_tile): by a stamp in LDS.  A writes P and then the tile's number
//     (release), B spins on the number (acquire); the roles drift apart between the barriers.  A publishes
//     the stamp of a tile before it reaches the next barrier and waits for B nowhere else, so the spin ends,
//     and it rewrites P only behind that barrier, which B reaches after it has taken P.
//   * four-slot ring (AbTile): by the barrier itself, which stands behind A's writes of P.  B takes P
//     behind it and then counts the tile in LDS (release); A spins on that count (acquire) before it rewrites
//     P in the next tile.  B waits for nothing between the barrier and the count, so the spin ends.
// Both spins are bounded (spin_until), so the kernels drain whatever happens.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void lds_write_b128(unsigned addr, bf16x8_t v) {
  *(bf16x8_t __attribute__((address_space(3)))*)(uintptr_t)addr = v;
}

struct AbLane {
  unsigned nat;         // rows of Q (A) or dO (B): A operand of the score product, slot 0, half 0
  unsigned tr[2];       // dO (A) or Q (B) transposed
  unsigned init_addr;   // -lse/scale (A) or -delta (B) of the lane's first row
  unsigned p_addr;      // this lane's 16 bytes in the pair's P buffer (unit 0, key half 0)
};

// Row fragments and row constants of one 32-query unit.
template <int SOFF, int SROW>
__device__ __forceinline__ void ab_load_nat(const AbLane& ln, unsigned off, unsigned off_row, bf16x8_t (&nat)[2][4], floatx4_t (&ini)[2]) {
#pragma unroll
  for (int t = 0; t < 2; ++t) ini[t] = lds_read_f32x4(ln.init_addr + off_row + SROW + t * 16);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int t = 0; t < 2; ++t) nat[t][ks] = read_nat<64>(ln.nat + off + SOFF, t, ks);
}
// Its scores ([query operand t][key half]), started from the constants.
__device__ __forceinline__ void ab_scores(const bf16x8_t (&nat)[2][4], const floatx4_t (&ini)[2],
                                          const bf16x8_t (&kvf)[2][4], StepScores& acc) {
#pragma unroll
  for (int t = 0; t < 2; ++t) acc[t][0] = acc[t][1] = ini[t];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k = 0; k < 2; ++k) acc[t][k] = mfma16(nat[t][ks], kvf[k][ks], acc[t][k]);
}

template <int SOFF>
__device__ __forceinline__ void ab_load_tr(const AbLane& ln, unsigned off, bf16x8_t (&tr)[8]) {
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) tr[dt] = read_tr<64>(ln.tr, off + SOFF, dt);
}

__device__ __forceinline__ void ab_accumulate(const bf16x8_t (&tr)[8], const bf16x8_t (&bop)[2], floatx4_t (&acc)[8][2]) {
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int k = 0; k < 2; ++k) acc[dt][k] = mfma16(tr[dt], bop[k], acc[dt][k]);
}

// A: P of one 32-query unit from its scores, also written to LDS for the partner.
template <bool MASK, int NC>
__device__ __forceinline__ void ab_make_p(const AbLane& ln, const floatx4_t (&sc)[2][NC], float c, int g, int left, int u,
                                          bf16x8_t (&pf)[NC]) {
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    unsigned int pp[4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        float pa = fast_exp2(sc[t][k][i] * c), pb = fast_exp2(sc[t][k][i + 1] * c);
        if (MASK) {
          const int idx = 32 * u + 8 * g + 4 * t + i;
          if (idx >= left) pa = 0.f;
          if (idx + 1 >= left) pb = 0.f;
        }
        pp[2 * t + (i >> 1)] = pack_bf16x2(pa, pb);
      }
    pf[k] = __builtin_bit_cast(bf16x8_t, uintx4_t{pp[0], pp[1], pp[2], pp[3]});
    lds_write_b128(ln.p_addr + (u * NC + k) * 1024, pf[k]);
  }
}

// B: dS = P * dP of one unit, P read from LDS.
template <int NC>
__device__ __forceinline__ void ab_take_p(const AbLane& ln, const floatx4_t (&dp)[2][NC], int u, bf16x8_t (&dsf)[NC]) {
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const uintx4_t pu = __builtin_bit_cast(uintx4_t, lds_read_b128(ln.p_addr + (u * NC + k) * 1024));
    unsigned int dd[4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        const unsigned w = pu[2 * t + (i >> 1)];
        dd[2 * t + (i >> 1)] = pack_bf16x2(bf16_lo_to_f32(w) * dp[t][k][i], bf16_hi_to_f32(w) * dp[t][k][i + 1]);
      }
    dsf[k] = __builtin_bit_cast(bf16x8_t, uintx4_t{dd[0], dd[1], dd[2], dd[3]});
  }
}

// Waits until *flag reaches `value`; after `spin_limit` polls it records a give-up in *status and goes on.
__device__ __forceinline__ void spin_until(int* flag, int value, int spin_limit, int* status) {
  int polls = 0;
  while (__hip_atomic_load(flag, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < value) {
    if (++polls > spin_limit) {   // wave-uniform
      if ((threadIdx.x & 63) == 0) atomicOr(status, 1);
      break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// One 64-query tile of the two-slot kernel for either role (role is wave-uniform; the common parts are written once so that
// the two roles share one instruction stream, with one short role-specific piece in the middle):
//   A: S(u0), S(u1) | P -> LDS, stamp          | dV(u0), dV(u1)
//   B: dP(u0), dP(u1) | wait for the stamp, dS = P * dP | dK(u0), dK(u1)
// `left`: valid query rows of the tile (MASK only).  The stamp of tile t is t + 1.
// The wait of B is bounded: after `spin_limit` polls it records a give-up in *status and goes on
// with whatever P holds (wrong numbers, but the kernel drains normally and the host can tell).
// Progress does not depend on the bound: A publishes the stamp of tile t before it reaches the
// block barrier of tile t + 1 and never waits for B anywhere else, and the single P buffer of a
// pair is only rewritten after that barrier, which B reaches only after it has consumed P.
template <bool MASK, int SOFF, int SROW>
__device__ __forceinline__ void ab_tile(const AbLane& ln, int role, unsigned off, unsigned off_row,
                                        const bf16x8_t (&kvf)[2][4], floatx4_t (&acc)[8][2], float c, int g, int left,
                                        int* flag, int tile_no, int spin_limit, int* status) {
  StepScores sc[2];      // S (A) or dP (B) of the two 32-query units
  bf16x8_t bop[2][2];    // B operand of the second product: P (A) or dS (B), per unit and key half
  bf16x8_t tr0[8], tr1[8];
  bf16x8_t nat0[2][4], nat1[2][4];
  floatx4_t ini0[2], ini1[2];
  ab_load_nat<SOFF, SROW>(ln, off, off_row, nat0, ini0);   // all fragments on their way before the first product
  ab_load_nat<SOFF + kRow32Bytes, SROW + 128>(ln, off, off_row, nat1, ini1);
  __builtin_amdgcn_sched_barrier(0);
  ab_scores(nat0, ini0, kvf, sc[0]);
  __builtin_amdgcn_sched_barrier(0);
  ab_load_tr<SOFF>(ln, off, tr0);   // in flight while P is computed (A) or awaited (B)
  ab_scores(nat1, ini1, kvf, sc[1]);
  __builtin_amdgcn_sched_barrier(0);
  if (role == 0) {
    ab_make_p<MASK>(ln, sc[0], c, g, left, 0, bop[0]);
    ab_make_p<MASK>(ln, sc[1], c, g, left, 1, bop[1]);
    __hip_atomic_store(flag, tile_no, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);   // P of this tile is in LDS
  } else {
    spin_until(flag, tile_no, spin_limit, status);
    ab_take_p(ln, sc[0], 0, bop[0]);
    ab_take_p(ln, sc[1], 1, bop[1]);
  }
  ab_load_tr<SOFF + kRow32Bytes>(ln, off, tr1);   // in flight while the first unit is accumulated
  ab_accumulate(tr0, bop[0], acc);
  ab_accumulate(tr1, bop[1], acc);
}

// The tile of the four-slot kernel, a stream of instructions for each role:
//   A: S(u0) | S(u1), P(u0) | dV(u0), P(u1) | wait until B has taken the P before, P -> LDS | barrier | dV(u1)
//   B: dP(u0) | dP(u1) | barrier | take P(u0), dS(u0) | dK(u0), take P(u1), dS(u1) | dK(u1)
// The tile's 32 fragments (row fragments of both units, then transposed ones) are read kAbWin ahead of their products, across the
// tile's end, so that no wave starts a tile with its matrix pipe waiting for LDS.  `left`: valid query rows of the tile.  `taken`: tiles
// whose P B has taken; the single P buffer of a pair is rewritten only then.
//
// 48 keys per pair: a fragment feeds three products instead of two, and a tile's waits (barrier, hand-over) weigh a third less.  A's exponentials
// stand among products of its own: as one piece between its products, in a stream that both roles shared, they took 1,480 of a tile's
// 4,780 cycles in A, for 400 of which B waited at the barrier.  B moves the tiles: A is the longer chain.  Whole backward, 145,080 x 40 heads,
// 8 groups 149.2 -> 138.1 ms, 62,400 x 12, 5 groups 13.5 -> 12.4, 32,760 x 12, 8 groups 2.32 -> 2.23, 16,384 x 4, 2 groups 0.764 -> 0.758; matrix
// pipes of this kernel busy 0.604 -> 0.709.  At the power cap: variants that take 3 % fewer cycles take the same time.
constexpr int kAbWin = 3;
constexpr int kAbKeep = 0x2 | 0x4 | 0x400;   // what may cross a scheduling barrier: vector, scalar and transcendental instructions
struct AbAhead {   // the next tile's first fragments and row constants
  bf16x8_t fr[kAbWin];
  floatx4_t ini;
};
template <int NC>
struct AbTile {
  const AbLane& ln;
  const bf16x8_t (&kvf)[NC][4];
  floatx4_t (&acc)[8][NC];
  AbAhead& ahead;
  unsigned nat, tr[2], init;   // the lane's addresses in this tile (AbLane's in slot 0)
  unsigned nnat, ninit;        // and in the next one
  Scores<NC> sc[2];       // S (A) or dP (B) of the two 32-query units
  bf16x8_t bop[2][NC];    // B operand of the second product: P (A) or dS (B), per unit and key column
  bf16x8_t fr[32];
  floatx4_t ini[4];

  __device__ __forceinline__ void load(int f) {
    if (f < 16) {
      fr[f] = read_nat<64>(nat + (f >> 3) * kRow32Bytes, (f >> 2) & 1, f & 3);
      if (!(f & 3)) ini[f >> 2] = lds_read_f32x4(init + (f >> 3) * 128 + ((f >> 2) & 1) * 16);
    } else if (f < 32) {
      fr[f] = read_tr<64>(tr, ((f - 16) >> 3) * kRow32Bytes, f & 7);
    } else {
      ahead.fr[f - 32] = read_nat<64>(nnat, (f >> 2) & 1, f & 3);
      if (f == 32) ahead.ini = lds_read_f32x4(ninit);
    }
  }
  __device__ __forceinline__ void begin() {
#pragma unroll
    for (int f = 0; f < kAbWin; ++f) fr[f] = ahead.fr[f];
    ini[0] = ahead.ini;
  }
  // The products of fragments 8 U .. 8 U + 7, and among them the 4 NC steps of `vec`, which stay where they are put: left to
  // itself the compiler collects them in front of the products.
  template <int U, bool VEC, typename V>
  __device__ __forceinline__ void products(V&& vec) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int f = 8 * U + i;
      __builtin_amdgcn_sched_barrier(VEC ? 0 : kAbKeep);
      load(f + kAbWin);
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        if constexpr (U < 2) {
          floatx4_t& a = sc[U][i >> 2][k];
          a = mfma16(fr[f], kvf[k][f & 3], f & 3 ? a : ini[f >> 2]);
        } else {
          acc[i][k] = mfma16(fr[f], bop[U - 2][k], acc[i][k]);
        }
      }
      if constexpr (VEC)
#pragma unroll
        for (int j = 4 * NC * i / 8; j < 4 * NC * (i + 1) / 8; ++j) vec(j % NC, j / NC);
    }
    if constexpr (VEC) __builtin_amdgcn_sched_barrier(0);
  }
  // A: word w (0 .. 3) of the B operand of unit U: P = exp2(S c)
  template <int U>
  __device__ __forceinline__ void make_p(int k, int w, float c) {
    const floatx4_t& v = sc[U][w >> 1][k];
    unsigned p = pack_bf16x2(fast_exp2(v[2 * (w & 1)] * c), fast_exp2(v[2 * (w & 1) + 1] * c));
    asm volatile("" : "+v"(p));   // here and not behind the wait for B
    set_word(bop[U][k], w, p);
  }
  // B: dS = P * dP, P as A wrote it
  template <int U>
  __device__ __forceinline__ void make_ds(int k, int w, unsigned p) {
    const floatx4_t& v = sc[U][w >> 1][k];
    set_word(bop[U][k], w, pack_bf16x2(bf16_lo_to_f32(p) * v[2 * (w & 1)], bf16_hi_to_f32(p) * v[2 * (w & 1) + 1]));
  }
  static __device__ __forceinline__ void set_word(bf16x8_t& f, int w, unsigned x) {
    uintx4_t u = __builtin_bit_cast(uintx4_t, f);
    u[w] = x;
    f = __builtin_bit_cast(bf16x8_t, u);
  }
  // Queries past the end of the group: P = 0
  template <int U>
  __device__ __forceinline__ void mask(int g, int left) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k = 0; k < NC; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (32 * U + 8 * g + 4 * t + i >= left) sc[U][t][k][i] = -INFINITY;
  }

  template <bool MASK, typename F>
  __device__ __forceinline__ void run_a(float c, int g, int left, int* taken, int tile_no, int spin_limit, int* status, F&& barrier) {
    begin();
    products<0, false>([](int, int) {});
    if (MASK) mask<0>(g, left);
    products<1, true>([&](int k, int w) { make_p<0>(k, w, c); });
    if (MASK) mask<1>(g, left);
    products<2, true>([&](int k, int w) { make_p<1>(k, w, c); });
    spin_until(taken, tile_no, spin_limit, status);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = 0; k < NC; ++k) lds_write_b128(ln.p_addr + (u * NC + k) * 1024, bop[u][k]);
    barrier();
    products<3, false>([](int, int) {});
  }

  template <typename F>
  __device__ __forceinline__ void run_b(int* taken, int tile_no, F&& barrier) {
    begin();
    products<0, false>([](int, int) {});
    products<1, false>([](int, int) {});
    __builtin_amdgcn_sched_barrier(0);
    barrier();
    wave_priority<true, 1>();   // A has half a tile's products left, B needs its dS first (without: 3 % slower on zeros, 1 % else)
    uintx4_t p[NC];
    auto take = [&](int u) {
#pragma unroll
      for (int k = 0; k < NC; ++k) p[k] = __builtin_bit_cast(uintx4_t, lds_read_b128(ln.p_addr + (u * NC + k) * 1024));
    };
    take(0);
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int w = 0; w < 4; ++w) make_ds<0>(k, w, p[k][w]);
    __builtin_amdgcn_sched_barrier(0);
    take(1);
    products<2, true>([&](int k, int w) { make_ds<1>(k, w, p[k][w]); });
    __hip_atomic_store(taken, tile_no + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    wave_priority<true, 0>();
    products<3, false>([](int, int) {});
  }
};

// NPAIR: wave pairs per block (4: partners on one SIMD; 2: for small groups).
// NB: ring slots of 64 queries (4 or 2, as in the dQ kernel).
// NC: columns of 16 keys per pair, at most.
template <int NPAIR, int NB, int NC, bool GATHER>
struct DkdvLds {
  __attribute__((aligned(1024))) unsigned short q[NB][64 * kHeadDim], d_o[NB][64 * kHeadDim];
  __attribute__((aligned(1024))) unsigned char p[NPAIR][NC * 2048];   // P of one tile, per pair
  __attribute__((aligned(256))) float l[NB][64], d[NB][64];      // -lse / scale, -delta
  __attribute__((aligned(256))) int tok[GATHER ? 512 : 1];       // gather mode: tokens of eight tiles
  int flag[NPAIR];   // per pair: number of tiles whose P has been written (NB == 2) or taken (NB == 4)
};

template <bool GATHER, int NPAIR, int NB, int MAXNC, bool SPLIT>
__device__ __forceinline__ void attn_bwd_dkdv_block(
    DkdvLds<NPAIR, NB, MAXNC, GATHER>& lds, int block, const unsigned short* __restrict__ d_oh, const unsigned short* __restrict__ qh,
    const unsigned short* __restrict__ kh, const unsigned short* __restrict__ vh,
    const float* __restrict__ neg_lse_over_scale, const float* __restrict__ neg_delta,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k,
    const int32_t* __restrict__ tile_start, int M, int64_t Nq, int64_t Nk, int H, float scale,
    unsigned short* __restrict__ d_kh, unsigned short* __restrict__ d_vh,
    int spin_limit, int* __restrict__ status, const int32_t* __restrict__ perm, float* __restrict__ part,
    unsigned short* __restrict__ d_k_tok, unsigned short* __restrict__ d_v_tok) {
  constexpr int NW = 2 * NPAIR;
  constexpr int BK = 16 * MAXNC * NPAIR;           // keys of a tile
  constexpr int kAhead = NB - 2;
  // Who moves the tiles: the large kernel leaves it to the waves B, which wait for A's P anyway.
  constexpr int kDmaWaves = NB == 4 ? NPAIR : NW;
  constexpr int kDmaPerTile = 2 * kDmaLoads<kDmaWaves, 64> + 2;

  // Ordered before its first use by the barriers below.  With NB == 4 and no polls the first wait (of P nobody needs yet) finds its
  // word not there, so that a test reaches the give-up for certain.
  if (threadIdx.x < NPAIR) lds.flag[threadIdx.x] = NB == 4 && spin_limit == 0 ? -1 : 0;
  WorkTile sp;
  if (!find_work<SPLIT>(cu_k, tile_start, M, H, BK, block, sp)) return;
  const TileInfo& ti = sp.ti;
  const int head = sp.head;
  const int ge = ti.row_end, k0 = ti.tile_row;
  int gs = cu_q[ti.group];
  int n = cu_q[ti.group + 1] - gs;
  const bool piece = SPLIT && sp.splits > 1;
  if (piece) split_range(sp, gs, n);

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int role = wave / NPAIR, pair = wave % NPAIR;
  int* flag = &lds.flag[pair];
  const int64_t head_off = (int64_t)head * Nk;
  const int64_t head_off_q = (int64_t)head * Nq;
  const float c = uniform_float(scale * 1.4426950408889634f);
  // A pair of waves owns 16 NC keys: three columns, or two where that is enough for the last tile of a group, which then takes
  // two thirds of the time.
  auto sweep = [&](auto columns) {
    constexpr int NC = columns.value;
    const int k0w = k0 + pair * 16 * NC;   // first key row of this pair
    unsigned short* outp = role == 0 ? d_vh : d_kh;
    unsigned short* tokp = role == 0 ? d_v_tok : d_k_tok;

    float* const piece_rows = piece ? part + ((size_t)sp.slot * 2 * BK + BK * role + 16 * NC * pair) * kHeadDim : nullptr;   // dV, then dK
    if (n <= 0) {   // keys without queries: zero gradient (block-uniform branch)
      if (piece) store_zero_piece<NC>(piece_rows);
      else store_zero_rows<GATHER, NC>(k0w, ge, head, head_off, H, outp, nullptr, perm, tokp);
      return;
    }

    bf16x8_t kvf[NC][4];   // K (A) or V (B) of the pair's key rows
    load_columns<GATHER>(kvf, role == 0 ? kh : vh, k0w, ge, head, head_off, H, perm);

    PipeDma dma;   // "k" = Q rows, "v" = dO rows of this head's group
    dma.kbase = uniform_ptr(GATHER ? qh + (int64_t)head * kHeadDim : qh + (head_off_q + gs) * kHeadDim);
    dma.vbase = uniform_ptr(GATHER ? d_oh + (int64_t)head * kHeadDim : d_oh + (head_off_q + gs) * kHeadDim);
    dma_lanes<kDmaWaves, 64>(dma, &lds.q[0][0], &lds.d_o[0][0], wave % kDmaWaves, lane);
    const bool moves = NB == 2 || role == 1;
    dma.last_row = n - 1;
    if constexpr (GATHER) {
      dma.rows = uniform_ptr(perm + gs);
      dma.tok_stride = (int64_t)H * kHeadDim * 2;
      dma.lds_tok = lds_addr_uniform(&lds.tok[0]);
      if (moves) {
        pipe_issue_tokens(dma, 0);
        pipe_issue_tokens(dma, 64);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      }
    }
    const void* lbase = uniform_ptr(neg_lse_over_scale + head_off_q + gs);
    const void* dbase = uniform_ptr(neg_delta + head_off_q + gs);
    const unsigned lds_l = lds_addr_uniform(&lds.l[0][0]), lds_d = lds_addr_uniform(&lds.d[0][0]);
    auto issue_tile = [&](int T) {   // every wave that moves tiles issues the (identical) row-constant loads so that all count alike
      const int slot = T & (NB - 1);
      pipe_issue<kDmaWaves, 64, GATHER>(dma, 64 * T, slot * kPipeTileBytes);
      const unsigned roff = (unsigned)min(64 * T + lane, n - 1) * 4u;
      lds_dma4_soff(lbase, roff, lds_l + slot * 256);
      lds_dma4_soff(dbase, roff, lds_d + slot * 256);
    };
    if (moves) {
#pragma unroll
      for (int t = 0; t <= kAhead; ++t) {
        if (GATHER && t == 2) __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kDmaPerTile));   // its tokens
        issue_tile(t);
      }
    }

    AbLane ln;
    ln.nat = nat_address(role == 0 ? &lds.q[0][0] : &lds.d_o[0][0], lane);
    tr_addresses(ln.tr, role == 0 ? &lds.d_o[0][0] : &lds.q[0][0], lane);
    ln.init_addr = (role == 0 ? (unsigned)(uintptr_t)&lds.l[0][0] : (unsigned)(uintptr_t)&lds.d[0][0]) + 8 * (lane >> 4) * 4;
    ln.p_addr = (unsigned)(uintptr_t)&lds.p[0][0] + pair * (NC * 2048) + lane * 16;

    settle(kvf);
    floatx4_t acc[8][NC];   // dV^T (A) or dK^T (B): d tile, key column
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int k = 0; k < NC; ++k) acc[dt][k] = floatx4_t{0.f, 0.f, 0.f, 0.f};

    const int nfull = n >> 6;   // tiles whose 64 queries are all inside the group
    // a pair whose key rows all lie past the end of the group (both of its waves) only moves its share of the tiles
    const bool active = k0w < ge;
    int T = 0;
    if constexpr (NB == 4) {
      const int ntiles = (n + 63) >> 6;
      AbAhead ahead;
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * kAhead));
      __syncthreads();
      if (active) {
#pragma unroll
        for (int f = 0; f < kAbWin; ++f) ahead.fr[f] = read_nat<64>(ln.nat, f >> 2, f & 3);
        ahead.ini = lds_read_f32x4(ln.init_addr);
      }
      // In tile t: tile t + 1 has landed (for the wave that moved it, then for all), and every wave has left the slot of tile t - 1.
      auto barrier_b = [&]() {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * (kAhead - 1)));
        block_barrier();
        issue_tile(T + 3);
      };
      auto addresses = [&](AbTile<NC>& t) {   // one register each, everything else is an immediate of the reads
        const unsigned slot = (unsigned)T & 3u, next = (unsigned)(T + 1) & 3u;
        t.nat = in_register(ln.nat + slot * kPipeTileBytes);
        t.tr[0] = in_register(ln.tr[0] + slot * kPipeTileBytes);
        t.tr[1] = in_register(ln.tr[1] + slot * kPipeTileBytes);
        t.init = in_register(ln.init_addr + slot * 256);
        t.nnat = in_register(ln.nat + next * kPipeTileBytes);
        t.ninit = ln.init_addr + next * 256;
      };
      if (!active) {
        for (; T < ntiles; ++T) {
          if (role == 1) barrier_b();
          else block_barrier();
        }
      } else if (role == 0) {
        for (; T < (n >> 6); ++T) {
          AbTile<NC> t = {ln, kvf, acc, ahead};
          addresses(t);
          t.template run_a<false>(c, lane >> 4, 64, flag, T, spin_limit, status, []() { __syncthreads(); });
        }
        if (n & 63) {
          AbTile<NC> t = {ln, kvf, acc, ahead};
          addresses(t);
          t.template run_a<true>(c, lane >> 4, n & 63, flag, T, spin_limit, status, []() { __syncthreads(); });
        }
      } else {
        for (; T < ntiles; ++T) {
          AbTile<NC> t = {ln, kvf, acc, ahead};
          addresses(t);
          t.run_b(flag, T, barrier_b);
        }
      }
    } else {
#define MOGA_AB_TILE(B)                                                          \
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * kAhead));                  \
    __syncthreads();                                                               \
    issue_tile(T + (B) + 1 + kAhead);                                              \
    if (active)                                                                    \
      ab_tile<false, ((B) & (NB - 1)) * kPipeTileBytes, ((B) & (NB - 1)) * 256>(ln, role, 0, 0, kvf, acc, c, lane >> 4, 64, flag, \
                                                                                T + (B) + 1, spin_limit, status);
      for (; T + 4 <= nfull; T += 4) {
        MOGA_AB_TILE(0)
        MOGA_AB_TILE(1)
        MOGA_AB_TILE(2)
        MOGA_AB_TILE(3)
      }
#undef MOGA_AB_TILE
      for (; T < nfull; ++T) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * kAhead));
        __syncthreads();
        issue_tile(T + 1 + kAhead);
        if (active)
          ab_tile<false, 0, 0>(ln, role, ((unsigned)T & (unsigned)(NB - 1)) * kPipeTileBytes,
                               ((unsigned)T & (unsigned)(NB - 1)) * 256, kvf, acc, c, lane >> 4, 64, flag, T + 1, spin_limit, status);
      }
      if (n & 63) {   // last, partial tile: masked queries get P = 0 and contribute nothing
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(kDmaPerTile * kAhead));
        __syncthreads();
        if (active)
          ab_tile<true, 0, 0>(ln, role, ((unsigned)T & (unsigned)(NB - 1)) * kPipeTileBytes,
                              ((unsigned)T & (unsigned)(NB - 1)) * 256, kvf, acc, c, lane >> 4, n - 64 * T, flag, T + 1, spin_limit, status);
      }
    }

    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // drain the look-ahead loads before the LDS is released
    if (piece) store_gradient_piece(acc, piece_rows);
    else store_gradient<GATHER>(acc, role == 0 ? 1.f : scale, k0w, ge, head, head_off, H, outp, tokp, perm);
  };
  if (MAXNC > 2 && ge - k0 > 32 * NPAIR) sweep(std::integral_constant<int, MAXNC>());
  else sweep(std::integral_constant<int, 2>());
}

// KEYS: keys of a block, 192 or 128 (key_blocks chooses): 48 or 32 for each of its four pairs of waves.
template <int KEYS, bool GATHER = false, bool SPLIT = false>
__global__ __launch_bounds__(512, 1) void attn_bwd_dkdv_ab_kernel(
    const unsigned short* __restrict__ d_oh, const unsigned short* __restrict__ qh,
    const unsigned short* __restrict__ kh, const unsigned short* __restrict__ vh,
    const float* __restrict__ neg_lse_over_scale, const float* __restrict__ neg_delta,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k,
    const int32_t* __restrict__ tile_start, int M, int64_t Nq, int64_t Nk, int H, float scale,
    unsigned short* __restrict__ d_kh, unsigned short* __restrict__ d_vh,
    int spin_limit, int* __restrict__ status, const int32_t* __restrict__ perm = nullptr,
    float* __restrict__ part = nullptr, unsigned short* __restrict__ d_k_tok = nullptr,
    unsigned short* __restrict__ d_v_tok = nullptr) {
  __shared__ DkdvLds<4, 4, KEYS / 64, GATHER> lds;
  attn_bwd_dkdv_block<GATHER, 4, 4, KEYS / 64, SPLIT>(lds, blockIdx.x, d_oh, qh, kh, vh, neg_lse_over_scale, neg_delta, cu_q, cu_k,
                                           tile_start, M, Nq, Nk, H, scale, d_kh, d_vh, spin_limit, status, perm, part, d_k_tok, d_v_tok);
}

// Both for small groups, in one launch: blocks below `dq_blocks` (a multiple of 8, for the XCDs) are dQ's, the others dK/dV's.
// Neither needs the other, and each alone leaves the chip idle in its last round and at a few hundred blocks from the first.
__global__ __launch_bounds__(256, 2) void attn_bwd_small_kernel(
    const unsigned short* __restrict__ d_oh, const unsigned short* __restrict__ qh,
    const unsigned short* __restrict__ kh, const unsigned short* __restrict__ vh,
    const float* __restrict__ neg_lse_over_scale, const float* __restrict__ neg_delta,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_k,
    const int32_t* __restrict__ ts_q, const int32_t* __restrict__ ts_k, int M, int64_t Nq, int64_t Nk, int H, float scale,
    unsigned short* __restrict__ d_qh, unsigned short* __restrict__ d_kh, unsigned short* __restrict__ d_vh,
    int spin_limit, int* __restrict__ status, const int32_t* __restrict__ perm, unsigned short* __restrict__ d_q_tok,
    unsigned short* __restrict__ d_k_tok, unsigned short* __restrict__ d_v_tok, int dq_blocks) {
  __shared__ union {
    DqLds<2, false> dq;
    DkdvLds<2, 2, 2, false> dkdv;
  } lds;
  if ((int)blockIdx.x < dq_blocks)
    attn_bwd_dq_block<4, false, 2, 128, false>(lds.dq, blockIdx.x, d_oh, qh, kh, vh, neg_lse_over_scale, neg_delta, cu_q, cu_k, ts_q, M, Nq,
                                          Nk, H, scale, d_qh, perm, nullptr, d_q_tok);
  else
    attn_bwd_dkdv_block<false, 2, 2, 2, false>(lds.dkdv, blockIdx.x - dq_blocks, d_oh, qh, kh, vh, neg_lse_over_scale, neg_delta, cu_q,
                                            cu_k, ts_k, M, Nq, Nk, H, scale, d_kh, d_vh, spin_limit, status, perm, nullptr, d_k_tok,
                                            d_v_tok);
}

// Several calls in one launch: the blocks of dQ and of dK/dV of each are a segment of the grid, from first[s] on (a multiple of 8), in an order
// that the host chooses: longest blocks first (by product, or shortest first, up to 24 % slower).  The branches of Section 3.2's block, whose last
// rounds are short blocks of other calls instead of pieces: attention backward of 8 frames x 3 heads 0.41 -> 0.27 ms, whole block forward and
// backward 2 x 16 0.60 -> 0.46, 8 x 3 0.66 -> 0.51, 11 x 12 2.47 -> 2.22, 5 x 40 3.50 -> 3.15, 30 x 12 9.93 -> 9.64, 21 x 12 with longer groups
// 8.73 -> 8.54; 64 x 40 75.9 and 75.6, within what two runs of one side differ by.
struct AttnBwdCall {
  const unsigned short *d_oh, *qh, *kh, *vh;
  const float *neg_lse_over_scale, *neg_delta;
  const int32_t *cu_q, *cu_k, *ts_q, *ts_k;
  int64_t Nq, Nk;
  unsigned short *d_qh, *d_kh, *d_vh;      // NULL where only the token-order rows are wanted
  unsigned short *d_q_tok, *d_k_tok, *d_v_tok;   // NULL, or the rows in token order as well
  const int32_t* perm;
  int* status;
  int M;
};
// The host sizes a segment for the most tiles that its groups can have, so blocks without a tile lie behind its real ones.  Between the two segments
// of a call by itself they cost a round: an XCD deals its blocks to its four shader engines of eight CUs in turn, whether they have work or not, and
// with the turn shifted one engine gets a ninth block while another keeps a CU free.  Where the blocks may be one round (rows0) the second segment
// starts where the tiles of the first really end (rounded up to 8): 243 blocks (2,304 rows x 9 heads) 115 us -> 84, 252 (1,536 x 14) 82 -> 62, 253 (1,920 x 11) 98 -> 74; 240 (2,560 x 8)
// 90 and 91.
struct AttnBwdCalls {
  AttnBwdCall c[kMaxCalls];
  int first[2 * kMaxCalls];   // INT_MAX: none
  int what[2 * kMaxCalls];    // 2 * call, + 1 for dK/dV
  int rows0, sure;            // rows of a tile of the first segment, blocks that it has at least; 0: the segments start at first
};
struct BwdPlace { int segment, block; };
__device__ __forceinline__ BwdPlace place_of_block(const AttnBwdCalls& calls, int H, int block) {
  if (calls.rows0 > 0) {
    if (block < calls.sure) return {0, block};
    const AttnBwdCall& c = calls.c[0];
    const int tiles = (max(count_tiles(calls.what[0] & 1 ? c.cu_k : c.cu_q, c.M, calls.rows0) * H, calls.sure) + 7) & ~7;
    return block < tiles ? BwdPlace{0, block} : BwdPlace{1, block - tiles};
  }
  int s = 0;
#pragma unroll
  for (int k = 1; k < 2 * kMaxCalls; ++k) s += block >= calls.first[k];
  return {s, block - calls.first[s]};
}
template <int KEYS, int ROWS, bool GATHER>
__global__ __launch_bounds__(512, 1) void attn_bwd_calls_kernel(AttnBwdCalls calls, int H, float scale, int spin_limit) {
  __shared__ union {
    DqLds<4, GATHER> dq;
    DkdvLds<4, 4, KEYS / 64, GATHER> dkdv;
  } lds;
  const BwdPlace at = place_of_block(calls, H, blockIdx.x);
  const int what = calls.what[at.segment], block = at.block;
  const AttnBwdCall& c = calls.c[what >> 1];
  if (what & 1)
    attn_bwd_dkdv_block<GATHER, 4, 4, KEYS / 64, false>(lds.dkdv, block, c.d_oh, c.qh, c.kh, c.vh, c.neg_lse_over_scale, c.neg_delta, c.cu_q,
                                                        c.cu_k, c.ts_k, c.M, c.Nq, c.Nk, H, scale, c.d_kh, c.d_vh, spin_limit, c.status,
                                                        c.perm, nullptr, c.d_k_tok, c.d_v_tok);
  else
    attn_bwd_dq_block<8, GATHER, 4, ROWS, false>(lds.dq, block, c.d_oh, c.qh, c.kh, c.vh, c.neg_lse_over_scale, c.neg_delta, c.cu_q, c.cu_k,
                                                 c.ts_q, c.M, c.Nq, c.Nk, H, scale, c.d_qh, c.perm, nullptr, c.d_q_tok);
}
__global__ __launch_bounds__(256, 2) void attn_bwd_small_calls_kernel(AttnBwdCalls calls, int H, float scale, int spin_limit) {
  __shared__ union {
    DqLds<2, false> dq;
    DkdvLds<2, 2, 2, false> dkdv;
  } lds;
  const BwdPlace at = place_of_block(calls, H, blockIdx.x);
  const int what = calls.what[at.segment], block = at.block;
  const AttnBwdCall& c = calls.c[what >> 1];
  if (what & 1)
    attn_bwd_dkdv_block<false, 2, 2, 2, false>(lds.dkdv, block, c.d_oh, c.qh, c.kh, c.vh, c.neg_lse_over_scale, c.neg_delta, c.cu_q, c.cu_k,
                                               c.ts_k, c.M, c.Nq, c.Nk, H, scale, c.d_kh, c.d_vh, spin_limit, c.status, c.perm, nullptr,
                                               c.d_k_tok, c.d_v_tok);
  else
    attn_bwd_dq_block<4, false, 2, 128, false>(lds.dq, block, c.d_oh, c.qh, c.kh, c.vh, c.neg_lse_over_scale, c.neg_delta, c.cu_q, c.cu_k,
                                               c.ts_q, c.M, c.Nq, c.Nk, H, scale, c.d_qh, c.perm, nullptr, c.d_q_tok);
}

}  // namespace moga
