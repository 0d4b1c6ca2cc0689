// Backward of the variable-length group attention (derivative of Eq. 1 inside each group).
//
// With P = exp(scale*S - lse) and delta = rowsum(dO * O):
//   dV = P^T dO,  dP = dO V^T,  dS = P * (dP - delta),  dQ = scale dS K,  dK = scale dS^T Q.
//
// No atomics; results do not depend on scheduling, only (in their rounding) on whether the workspace has room
// to split the last round:
//   attn_bwd_delta   : -delta[h][j] = -sum_c dO[h][j][c] * O[h][j][c], and in bf16 -lse / scale; the calls that
//                      write dO themselves (_tokens) or are given these constants (_rows) do without it;
//   attn_bwd_dkdv_ab : a pair of waves owns 48 (or 32) key rows and sweeps the query tiles of its group, one wave with
//                      the K fragments and the dV^T accumulators, the other with the V fragments and dK^T;
//   attn_bwd_dq_pipe : a wave owns 48 (or 32) query rows and sweeps the key tiles (mirror of forward);
//   attn_bwd_small   : both with smaller tiles in one launch, for small groups;
//   attn_bwd_calls   : dq_pipe's and dkdv_ab's blocks in one launch, of one call or of several (attn_bwd_small_calls: of small groups).
// The bf16 MFMA kernels are in attn_bwd_pipe.h: they keep the contraction index of the second
// product in the accumulator registers of the first (row permutation of the LDS operand), and
// read the transposed operands (dO^T, Q^T, K^T) from row-major LDS tiles with the transposing
// LDS read.  fp32 (attn_f32.h): delta, then dQ and dK/dV in one launch.
#include <algorithm>
#include <atomic>
#include <climits>

#include "attn_common.h"
#include "attn_bwd_pipe.h"
#include "attn_f32.h"

namespace moga {

// ---------------------------------------------------------------------------------------
// LPR lanes of 16 bytes a row.  neg_lse_over_scale and its lse: bf16 only.
template <int LPR, bool BF16>
__global__ __launch_bounds__(256) void attn_bwd_delta_kernel(const uintx4_t* __restrict__ d_oh,
                                                             const uintx4_t* __restrict__ oh,
                                                             const float* __restrict__ lse, int64_t rows,
                                                             float inv_scale, float* __restrict__ neg_delta,
                                                             float* __restrict__ neg_lse_over_scale,
                                                             int* __restrict__ status) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *status = 0;   // read by the kernels that follow
  const int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LPR;
  const int part = threadIdx.x % LPR;
  float s = 0.f;
  if (row < rows) {
    const uintx4_t a = d_oh[row * LPR + part], b = oh[row * LPR + part];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (BF16) {
        s = fmaf(bf16_lo_to_f32(a[i]), bf16_lo_to_f32(b[i]), s);
        s = fmaf(bf16_hi_to_f32(a[i]), bf16_hi_to_f32(b[i]), s);
      } else {
        s = fmaf(__uint_as_float(a[i]), __uint_as_float(b[i]), s);
      }
    }
  }
  s = lanes_sum<LPR>(s);
  if (row < rows && part == 0) {   // both negated, ready to start an accumulator from
    neg_delta[row] = -s;
    if (BF16) neg_lse_over_scale[row] = -lse[row] * inv_scale;
  }
}

template <int LPR, bool BF16>
static void launch_delta(const void* d_oh, const void* oh, const float* lse, int64_t rows, float inv_scale, float* neg_delta,
                         float* neg_lse_over_scale, int* status, hipStream_t st) {
  constexpr int64_t kRows = (int64_t)1 << 26;   // of a launch: 16 or 32 threads each, 2^32 are too many
  for (int64_t r = 0; r < rows; r += kRows)
    attn_bwd_delta_kernel<LPR, BF16><<<(unsigned)((std::min(rows - r, kRows) * LPR + 255) / 256), 256, 0, st>>>(
        (const uintx4_t*)d_oh + r * LPR, (const uintx4_t*)oh + r * LPR, lse + r, std::min(rows - r, kRows), inv_scale, neg_delta + r,
        BF16 ? neg_lse_over_scale + r : nullptr, status);
}

// Pre-pass of the gather-fused backward (bf16, head_dim 128; token-major inputs).  With O = gate * A
// (Eq. 5) and dO the upstream gradient of O:  delta = rowsum(dA * A) = rowsum(dO * O) =: dot, and the
// kernels can consume the raw dO rows if the gate is folded into the per-row constants:
//   P' = gate * P = exp(S - (lse - ln gate)),   dS = P' * (dO V^T - dot / gate),   dV = P'^T dO.
// Writes, in sorted order [H, N]:  -(lse - ln gate) / scale  and  -dot / gate;  and per token
// d_gate = sum over heads of dot / gate.  Four tokens per block, 16 lanes per (token, head) row; a wave takes every fourth head, four heads
// at a time: with 16 tokens per block and a row's loads behind the stores of the one before, 1,253 x 40 heads 42.5 us (8.7 so), 5,000 x 40
// 61.5 (22.4), 16,000 x 40 91.5 (70.0), 99,840 x 40 485 (453).
constexpr int kPrepassTokens = 4;
__global__ __launch_bounds__(256) void attn_bwd_fused_prepass_kernel(
    const uintx4_t* __restrict__ d_o, const uintx4_t* __restrict__ o, const float* __restrict__ lse,
    const int32_t* __restrict__ inv_perm, const float* __restrict__ gate, int64_t N, int H,
    float inv_scale, float* __restrict__ neg_lse_over_scale, float* __restrict__ neg_delta,
    float* __restrict__ d_gate, int* __restrict__ status) {
  constexpr int SLOTS = kPrepassTokens, IT = SLOTS / 4, HU = 4;
  __shared__ float s_part[4][SLOTS];
  if (blockIdx.x == 0 && threadIdx.x == 0) *status = 0;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int part = lane & 15, rsub = lane >> 4;
  const int64_t t0 = (int64_t)blockIdx.x * SLOTS;
  float acc[IT];
  int64_t tok[IT], slot[IT];
  float g[IT], lg[IT];
  bool ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t t = t0 + it * 4 + rsub;
    ok[it] = t < N;
    tok[it] = ok[it] ? t : N - 1;
    slot[it] = inv_perm[tok[it]];
    g[it] = gate[tok[it]];
    lg[it] = logf(g[it]);
    acc[it] = 0.f;
  }
  for (int h0 = wave; h0 < H; h0 += 4 * HU) {
    uintx4_t a[HU][IT], b[HU][IT];
    float l[HU][IT];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = min(h0 + 4 * u, H - 1);
        a[u][it] = d_o[(tok[it] * H + h) * 16 + part];
        b[u][it] = o[(tok[it] * H + h) * 16 + part];
        l[u][it] = lse[(int64_t)h * N + slot[it]];
      }
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        if (h >= H) continue;   // the same for all lanes
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s = fmaf(bf16_lo_to_f32(a[u][it][i]), bf16_lo_to_f32(b[u][it][i]), s);
          s = fmaf(bf16_hi_to_f32(a[u][it][i]), bf16_hi_to_f32(b[u][it][i]), s);
        }
        s = lanes_sum<16>(s);
        const float dg = s / g[it];
        acc[it] += dg;
        if (part == 0 && ok[it]) {
          const int64_t idx = (int64_t)h * N + slot[it];
          neg_lse_over_scale[idx] = -(l[u][it] - lg[it]) * inv_scale;
          neg_delta[idx] = -dg;
        }
      }
  }
#pragma unroll
  for (int it = 0; it < IT; ++it)
    if (part == 0) s_part[wave][it * 4 + rsub] = acc[it];
  __syncthreads();
  if (threadIdx.x < SLOTS) {
    const int64_t t = t0 + threadIdx.x;
    if (t < N)
      d_gate[t] = (s_part[0][threadIdx.x] + s_part[1][threadIdx.x]) + (s_part[2][threadIdx.x] + s_part[3][threadIdx.x]);
  }
}

// Mean rows per group below which the small-group bf16 kernels run, by rounds of 256 blocks of 256 rows: their finer tiles win
// where there are few.  Time of the small kernels against the large ones' (blocks by large_blocks) with room to split a round, groups of
// equal / Zipf(1.1) sizes, in %; in brackets equal groups without room:
//   rounds 0.15  1,250 rows -42 / 0 [-53], 2,500 -17 / +11 [-52], 5,000 +9 / +22 [-51];  0.25  2,500 -15 / -1 [-31], 8,000 +25 / +36 [-31]
//          0.4   1,560 +6 / -5 [+3], 2,500 +19 / -8 [+7];                0.6   1,560 +2 / -20 [+6], 2,500 +5 / -20 [+9]
//          0.85  1,000 +3 / -9 [+9], 1,560 +9 / -3 [+13];                1.05  850 -3 / -4 [+2], 1,250 -1 / -16 [+4], 1,560 +3 / -3 [+7]
//          1.2   850 -6 / -15 [-2], 1,250 +3 / -16 [+8], 1,560 +8 / -13 [+11];   1.6  1,000 -3 / -12 [0], 1,560 +5 / -10 [+4]
//          1.8   850 -2 / +4 [+2], 1,250 +10 / -12 [+14];                2.9   700 -5 / +8 [-1], 1,000 +4 / +4 [+5]
//          4.5   600 -6 / +7 [-3], 700 -1 / +13 [+1];                    6.6   400 -5 / +11 [-3], 500 -1 / +11 [+3]
//          8     400 -7 / +11 [-3], 500 -3 / +11 [+4];                   12    400 -2 / +17 [0], 500 +1 / +15 [+5]
// The lines are where equal groups, what a balanced router makes, take the same time; between 0.33 and 2 rounds they are higher, to where
// equal groups lose up to 10 %, since Zipf groups gain up to twice that.  The host knows only the mean.  Without room below a third
// of a round most CUs have no block of the large kernels, and these are never the faster ones (measured to 8,000 rows).  A line with room
// may not lie above the one without: a call that it sends to the small kernels asks for no room, and comes here again without.
static int64_t small_group_rows(int64_t Nq, int H, bool room) {
  const int64_t rounds = 100 * Nq * H / (256 * kCus);   // in hundredths
  if (rounds < 33) return room ? 2800 : 8192;
  if (rounds < 100) return rounds < 75 ? 2000 : 1450;
  return rounds < 200 ? 1300 : rounds < 350 ? 860 : rounds < 600 ? 650 : rounds < 1000 ? 450 : 400;
}

// The same for the calls of one launch, all of them with `rows` queries: a second launch, for the other kernels, costs more than the finer tiles
// of some give.  Blocks of three branches from one to eight rounds, over the time of the calls one by one, with the large kernels for all / with the small
// ones for the windows, mean and range: windows of 4 tokens 1.34 (1.07 to 1.64) / 0.97 (0.88 to 1.08), 6 to 15 1.14 (0.93 to 1.35) / 0.92 (0.82 to 0.97),
// 15 to 24 1.03 (0.87 to 1.17) / 0.92 (0.81 to 1.06), 24 to 40 0.95 (0.81 to 1.02) / 0.92 (0.80 to 1.06), 40 to 100 0.90 / 0.88, 100 to 300 0.88 / 0.86.  Forward and
// backward with the large kernels for all against the small ones for groups of less than 300 / 700 / 1,200 rows: 2.6 rounds 0.538 ms and
// 0.590 / 0.590 / 0.569, 3.4 0.743 and 0.743 / 0.742 / 0.799, 5.1 1.200 and 1.241 / 1.241 / 1.241; groups of 104 queries, 4.3 rounds 0.883 and 0.901,
// 34 rounds 9.12 and 8.92, 69 rounds 15.5 and 15.25.
static int64_t calls_small_group_rows(int64_t rows, int H) {
  const int64_t rounds = 100 * rows * H / (256 * kCus);
  return rounds < 100 ? small_group_rows(rows, H, false) : rounds < 800 ? 24 : 300;
}

AttnPlan bwd_plan(int64_t Nq, int64_t Nk, int H, int M, int room) {
  if (use_small_group_kernels(Nq, M, small_group_rows(Nq, H, room > 0))) return {true, {128, false}, {64, false}};
  return {false, query_blocks(Nq, Nk, H, M, room), key_blocks(Nq, Nk, H, M, room)};
}

// dQ and dK/dV of one call in one launch: mean rows per group below which the small-group kernels run.  Time of the large kernels against
// the small ones', both in one launch, groups of iid / Zipf(1.1) tokens, in %:
//   rounds 0.5   400 rows -2 / -7, 500 +6 / -4, 650 -10 / -15;    1.0   400 +5 / -10, 500 +8 / -14, 650 -2 / -8
//          1.4   400 +11 / -11, 500 +3 / -11, 650 +2 / -9;        1.9   400 +9 / -4, 500 +1 / -9, 650 -3 / -9
//          3.5   300 +10 / -8, 400 +9 / -7, 500 +1 / -10, 650 -5 / -14;   8   400 +7 / -8, 500 -1 / -9, 650 -7 / -14
// Below a fifth of a round most CUs have no large block: 0.14 rounds, 650 rows +27 / +27, 1,700 +23 / +24, 3,200 +8 / +8; 0.2 rounds 650 -5 /
// -10, 1,700 -12 / -12, 3,200 -12 / -12.  About one round the blocks of 500 equal groups often just miss the first round (+6), those of 650 less so.
static int64_t joint_small_rows(int64_t N, int H) {
  const int64_t rounds = 100 * N * H / (256 * kCus);   // in hundredths
  return rounds < 18 ? 8192 : rounds < 50 ? 500 : rounds < 300 ? 650 : 500;
}

// Blocks of dQ and of dK/dV of up to kMaxCalls calls as one list, longest first.
struct BwdSegment {
  int what;          // 2 * call, + 1 for dK/dV
  int64_t blocks;
  double length;     // of a block: products times rows swept
};
struct BwdBlocks { int bm, bk; };   // query rows of a block, keys
static double list_end(const BwdSegment* seg, int n, int places) {
  struct { double time; int64_t places; } free[2 * kMaxCalls + 1] = {{0., places}};   // soonest first; a segment adds one at most
  int count = 1;
  double end = 0;
  for (int i = 0; i < n; ++i)
    for (int64_t left = seg[i].blocks; left > 0;) {
      const double t = free[0].time + seg[i].length;
      const int64_t k = std::min(left, free[0].places);
      left -= k;
      if ((free[0].places -= k) == 0) std::copy(free + 1, free + count--, free);
      int at = count;
      while (at > 0 && free[at - 1].time >= t) --at;
      if (at < count && free[at].time == t) {
        free[at].places += k;
      } else {
        std::copy_backward(free + at, free + count, free + count + 1);
        free[at] = {t, k};
        ++count;
      }
      end = std::max(end, t);
    }
  return end;
}
// Price of blocks of bm query rows and bk keys, in the units of large_blocks: three products a pair of rows in dQ, four in dK/dV (whose blocks have
// half the rows).  With equal groups; a block sweeps kStartRows more rows than there are.  Up to 1.2 rounds (of 256
// blocks of 256 rows) the end of the list.  Beyond, work per CU and half of a last block, since the blocks get out of step: over 72 calls of 1.2 to
// 20 rounds 1 % faster than by the list with iid groups, 2.5 % with Zipf's.
static bool few_rounds(int64_t rows, int H) { return 10 * rows * H < 12 * 256 * kCus; }
static double bwd_price(const SideShape* q, int n, int H, int bm, int bk, double weight, bool listed, int places) {
  BwdSegment seg[2 * kMaxCalls];
  double work = 0;
  for (int i = 0; i < n; ++i) {
    const SideShape& c = q[i];
    const int64_t nk = (c.other + c.M - 1) / c.M, nq = (c.N + c.M - 1) / c.M, tq = (nq + bm - 1) / bm, tk = (nk + bk - 1) / bk;
    seg[2 * i] = {2 * i, tq * c.M * H, 3 * weight * (nk + kStartRows)};
    seg[2 * i + 1] = {2 * i + 1, tk * c.M * H, 2 * weight * (nq + kStartRows)};
    // a group's last block, of two columns a wave
    work += (tq - (nq - (tq - 1) * bm <= 256 ? 1 - 10 / weight : 0)) * c.M * H * seg[2 * i].length;
    work += (tk - (nk - (tk - 1) * bk <= 128 ? 1 - 10 / weight : 0)) * c.M * H * seg[2 * i + 1].length;
  }
  std::stable_sort(seg, seg + 2 * n, [](const BwdSegment& x, const BwdSegment& y) { return x.length > y.length; });
  return listed ? list_end(seg, 2 * n, places) : work / kCus + seg[2 * n - 1].length / 2;
}
// Where the list ends in few rounds the long blocks, of which one may be the whole call's time, have to be a fifth cheaper: 0.33 rounds, groups of
// 800 iid / Zipf(1.1) rows 51 / 87 us with the short ones and 49 / 118 with the long ones.  With the rows read through perm a seventh (27 of 1,350
// calls more than 3 % slower than with two launches; with a fifth 35).
static BwdBlocks bwd_blocks(const SideShape* q, int n, int H, bool gather) {
  int64_t rows = 0;
  for (int i = 0; i < n; ++i) rows += q[i].N;
  const bool listed = few_rounds(rows, H);
  const double few = bwd_price(q, n, H, 256, 128, 10, listed, kCus), many = bwd_price(q, n, H, 384, 192, 13, listed, kCus);
  return few < (!listed ? 1. : gather ? 1.15 : 1.2) * many ? BwdBlocks{256, 128} : BwdBlocks{384, 192};
}

// How dQ and dK/dV of one call are launched, if the caller lets the call choose: together, as small-group blocks, or apart as by the other
// entry points (the large kernels with their last rounds split, or the small ones).  Time of what is chosen here over the time apart, 730 calls of 0.1 to 14
// rounds, groups of 100 to 20,000 rows of equal, iid and Zipf(1.1) sizes: mean 0.975, 37 of the 2,190 above 1.03, the worst
// with few or many Zipf groups, whose largest decides when the list ends (24,059 rows x 4 heads, 20 groups 1.20; 12,364 x 1, 5 groups 1.19).  Always together
// between four and 16 rounds and by the price of equal groups alone below: 65 of 1,350 above 1.03, with equal groups to 1.29.
enum class BwdForm { kApart, kSmall, kTogether };
// Apart in many rounds, where a last one is little (10 to 18 rounds together: 0.97 to 1.01).
static bool many_rounds(int64_t N, int H, int M) { return N * H >= 10 * 256 * kCus || (N * H >= 7 * 256 * kCus && N >= 8000 * (int64_t)M); }
// Long groups, with room to split a round: few blocks, each of them long.  Together 0.83 to 1.14 of the time apart from 3,400 rows on and 0.15 to three rounds,
// 67 of 231 sets above 1.03 (up to a fifth of a round the small-group kernels are the others, from 2,800 rows on); from three to seven rounds 0.90 to 1.04
// (3 of 54) with up to 8,000 rows, 0.89 to 1.06 (8 of 111) with more.
static bool long_groups(int64_t N, int H, int M) {
  return N >= (5 * N * H < 256 * kCus ? 2800 : N * H < 3 * 256 * kCus ? 3400 : 8000) * (int64_t)M;
}
// Places of the 256 that count where the end of a list is held against small blocks: routed groups have some blocks more than equal ones (4,900 x 4,
// 5 groups, 240 blocks if equal: 45 us, iid 59 and 46 as small blocks), and the first of the two kinds is rounded up to 8.
constexpr int kSurePlaces = 240;
static bool together_fits(int64_t N, int H, int M) { return grid_fits((max_tiles(N, M, 128) + max_tiles(N, M, 256)) * H + 14, 512); }
static BwdForm bwd_form(int64_t N, int H, int M, int room) {
  if (many_rounds(N, H, M) || (room > 0 && long_groups(N, H, M)) || !together_fits(N, H, M)) return BwdForm::kApart;
  const SideShape side = {N, N, M};
  const bool listed = few_rounds(N, H);
  auto price = [&](int bm, int places) { return bwd_price(&side, 1, H, bm, bm / 2, bm == 256 ? 10 : 13, listed, places); };
  int64_t line = joint_small_rows(N, H);
  if (N / M >= line && N / M < small_group_rows(N, H, room > 0)) {
    // Between the lines the small kernels are what runs apart.  They stay up to a quarter of a round with more than five groups (the largest of
    // Zipf groups, alone on its CUs: 13,228 rows, 10 groups 140 us together, 116 so), and in few rounds where their list ends sooner: a small block
    // starts for 500 rows and takes 12 per row, on half a CU.  Over 80 calls the two ends are in the proportion of the times to 5 %.
    bool small = 4 * N * H < 256 * kCus && M > 5;
    if (!small && listed) {
      const int64_t rows = (N + M - 1) / M;
      const BwdSegment seg[2] = {{0, (rows + 127) / 128 * M * H, 36. * (rows + 500)}, {1, (rows + 63) / 64 * M * H, 24. * (rows + 500)}};
      small = std::min(price(256, kSurePlaces), price(384, kSurePlaces)) > 0.95 * list_end(seg, 2, 2 * kCus);
    }
    if (small) line = INT64_MAX;
  }
  if (use_small_group_kernels(N, M, line)) return BwdForm::kSmall;
  if (room > 0 && N * H <= 4 * 256 * kCus && !bwd_plan(N, N, H, M, room).small) {   // from four rounds on at most 2 %
    double pq, pk;
    const Blocks q = large_blocks(N, N, H, M, 256, 1, room, &pq), k = large_blocks(N, N, H, M, 128, 2, room, &pk);
    if ((q.split || k.split) && 3 * pq + 2 * pk < 0.95 * price(bwd_blocks(&side, 1, H, false).bm, kCus)) return BwdForm::kApart;
  }
  return BwdForm::kTogether;
}
// The gather-fused call has no small kernels and splits nothing: together 0.89 of the time apart over 1,440 sets of groups of 0.15 to 9 rounds, 49 of them above 1.03, to 1.16
// (48,188 rows x 2 heads, 15 Zipf groups).  No line at long groups: apart from 2,800 rows and half a round on, the mean is 0.906 (15 above 1.03), and two
// groups of 5,777 rows x 12 and five of 7,374 x 3 take 6 % longer than together.
static bool fused_apart(int64_t N, int H, int M) { return many_rounds(N, H, M) || !together_fits(N, H, M); }

}  // namespace moga

using namespace moga;

// Workspace layout of the backward calls: [-delta: rows floats][-lse/scale: rows floats][status:
// 16 bytes, first int32 used], rows = Nq * H; the varlen call appends its two tile-start lists.
static size_t bwd_rows_bytes(int64_t Nq, int H) { return round_up(2 * (size_t)Nq * (size_t)H * sizeof(float), 16); }

extern "C" size_t moga_attn_bwd_status_offset(int64_t Nq, int H) {
  if (Nq <= 0 || H < 1) return 0;
  return bwd_rows_bytes(Nq, H);
}

extern "C" size_t moga_attn_bwd_ws_bytes(int64_t N, int H, int D, int dtype) {
  (void)D; (void)dtype;
  if (N <= 0 || H < 1) return 0;
  return bwd_rows_bytes(N, H) + 16;
}

// Polls after which a wave of the dK/dV kernels that waits for its partner gives up (and sets the
// status word).  In normal operation a wait lasts a few hundred polls at most.
static std::atomic<int> g_spin_limit{1 << 24};
extern "C" void moga_debug_set_spin_limit(int polls) { g_spin_limit.store(polls < 0 ? 0 : polls); }

// The bf16 kernels form per-lane byte offsets `row * 256` in 32 bits, relative to the first row of
// a group: a group (hence a tensor) must have fewer than 2^24 rows.
static bool bf16_rows_ok(int64_t Nq, int64_t Nk) { return Nq < ((int64_t)1 << 24) && Nk < ((int64_t)1 << 24); }

// The gradients in token order [N, H, D] as well, row j of the sorted order at token perm[j]; all NULL: none.  With them the
// sorted ones (d_qh, d_kh, d_vh) may be NULL.
struct TokenGrads {
  void *d_q, *d_k, *d_v;
  const int32_t* perm;
  bool row_constants;   // already in the workspace
};

// dQ and dK/dV of n bf16 calls in one launch: the blocks of one fill the last round of the other.  Against two launches with their last rounds
// split (32 MB of pieces, and a launch to add them up, each), groups of iid / Zipf(1.1) rows, backward of the attention in us: 9,000 x 12, 5 groups
// 317 -> 287 / 497 -> 432; 20,000 x 12, 10 groups 717 -> 679 / 1,437 -> 1,332; 15,000 x 40, 16 groups 974 -> 931; gather-fused step, whose launches
// cannot split, 700 x 12 71 -> 48, 1,253 x 40 159 -> 137, 5,225 x 40 720 -> 660.  Of the kernels for small groups or of the large ones (with their rows read through perm: GATHER).
// c: everything but ts_q and ts_k, for which ts[i] has room if call i has more than MOGA_MAX_GROUPS groups.
enum class BwdKernels { kSmall, kLarge, kGather };
static int launch_bwd_calls(const AttnBwdCall* c, int32_t* const* ts, int n, BwdKernels kernels, int H, float softmax_scale, hipStream_t st) {
  int bm = 128, bk = 64;
  const int threads = kernels == BwdKernels::kSmall ? 256 : 512;
  if (kernels != BwdKernels::kSmall) {
    SideShape q[kMaxCalls];
    for (int i = 0; i < n; ++i) q[i] = {c[i].Nq, c[i].Nk, c[i].M};
    const BwdBlocks rows = bwd_blocks(q, n, H, kernels == BwdKernels::kGather);
    bm = rows.bm, bk = rows.bk;
  }
  BwdSegment seg[2 * kMaxCalls];
  int segments = 0;
  for (int i = 0; i < n; ++i) {   // three products of bm rows a key, four of bk keys a query
    seg[segments++] = {2 * i, (max_tiles(c[i].Nq, c[i].M, bm) * H + 7) / 8 * 8, 3. * bm * (double)c[i].Nk / c[i].M};
    if (c[i].Nk > 0) seg[segments++] = {2 * i + 1, (max_tiles(c[i].Nk, c[i].M, bk) * H + 7) / 8 * 8, 4. * bk * (double)c[i].Nq / c[i].M};
  }
  std::stable_sort(seg, seg + segments, [](const BwdSegment& x, const BwdSegment& y) { return x.length > y.length; });
  AttnBwdCalls a = {};
  std::copy(c, c + n, a.c);
  // the blocks of the segments [first, last) as one grid, or 0 if it cannot hold them
  auto grid = [&](int first, int last) -> int64_t {
    std::fill(a.first, a.first + 2 * kMaxCalls, INT_MAX);
    int64_t blocks = 0;
    for (int s = first; s < last; ++s) {
      a.first[s - first] = (int)blocks;
      a.what[s - first] = seg[s].what;
      blocks += seg[s].blocks;
      if (!grid_fits(blocks, threads)) return 0;
    }
    return blocks;
  };
  // dK/dV of all calls, then dQ of all, from 12 rounds on: what one launch saves of a last round is little there, and blocks of both kinds side
  // by side take longer.  Step of a three-branch block, two launches before (apart call by call, last rounds split), one and these two, in us, in brackets
  // the rounds: 8 x 3 heads (4.5 of small and large blocks) 1,001, 793 and 903; 11 x 12 (9) 3,955, 3,440 and 3,508; 5 x 40 (14) 2,838, 2,545 and
  // 2,565; 15 x 12 (13) 5,120, 5,001 and 4,927; 21 x 12 (18) 4,385, 4,257 and 4,179, with fewer and longer groups 8,615, 8,535 and 8,451 (8,788 and 8,904 with
  // one on another card); 30 x 12 (26) 15,960, 15,705 and 15,637.
  int64_t rows = 0;
  for (int i = 0; i < n; ++i) rows += c[i].Nq;
  const int mid = n > 1 && kernels == BwdKernels::kLarge && rows * H >= 12 * 256 * kCus
                      ? (int)(std::stable_partition(seg, seg + segments, [](const BwdSegment& x) { return (x.what & 1) != 0; }) - seg) : segments;
  if ((mid > 0 && grid(0, mid) == 0) || (mid < segments && grid(mid, segments) == 0)) return MOGA_ERR_UNSUPPORTED;
  if (n == 1 && segments == 2 && c[0].M <= MOGA_MAX_GROUPS) {
    auto sure = [&](const BwdSegment& x) { return x.what & 1 ? (c[0].Nk + bk - 1) / bk * H : (c[0].Nq + bm - 1) / bm * H; };
    // where the blocks may be a round: elsewhere the count costs its 2 us and gives nothing (gather-fused, 1,146 rows x 40 heads, 16 groups 105.8 -> 107.3)
    if (sure(seg[0]) + sure(seg[1]) <= kCus && seg[0].blocks + seg[1].blocks > kCus) {
      a.rows0 = seg[0].what & 1 ? bk : bm;
      a.sure = (int)sure(seg[0]);
    }
  }
  for (int i = 0; i < n; ++i)
    if (c[i].M > MOGA_MAX_GROUPS) {
      int32_t *ts_q = ts[i], *ts_k = ts_q + (c[i].M + 1);
      if (c[i].Nk > 0) tile_start_kernel<<<1, 1024, 0, st>>>(c[i].cu_k, c[i].M, bk, ts_k);
      tile_start_kernel<<<1, 1024, 0, st>>>(c[i].cu_q, c[i].M, bm, ts_q);
      a.c[i].ts_q = ts_q, a.c[i].ts_k = ts_k;
    }
  const int spin = g_spin_limit.load();
#define MOGA_BWD_CALLS(KK, RR)                                                                                                            \
  if (kernels == BwdKernels::kGather) attn_bwd_calls_kernel<KK, RR, true><<<(unsigned)blocks, 512, 0, st>>>(a, H, softmax_scale, spin); \
  else attn_bwd_calls_kernel<KK, RR, false><<<(unsigned)blocks, 512, 0, st>>>(a, H, softmax_scale, spin)
  for (int first = 0, last = mid; first < segments; first = last, last = segments) {
    if (first == last) continue;   // no keys
    const int64_t blocks = grid(first, last);
    if (kernels == BwdKernels::kSmall) {
      attn_bwd_small_calls_kernel<<<(unsigned)blocks, 256, 0, st>>>(a, H, softmax_scale, spin);
    } else if (bm == 384) {
      MOGA_BWD_CALLS(192, 384);
    } else {
      MOGA_BWD_CALLS(128, 256);
    }
  }
#undef MOGA_BWD_CALLS
  return launch_status();
}

// Shared launcher.  ts_q / ts_k: NULL (tile lookup inside the kernels, M <= MOGA_MAX_GROUPS) or
// space for the pre-summed first-tile indices over query rows / key rows (M + 1 ints each).  split: room for
// the pieces of a last round, if any (dK/dV and dQ use it one after the other; only without ts_q / ts_k).  form: bf16; together and small
// need neither lists nor room (M <= MOGA_MAX_GROUPS).
static int launch_attn_bwd(const void* d_oh, const void* qh, const void* kh, const void* vh,
                           const void* oh, const float* lse, int dtype, int64_t Nq, int64_t Nk, int H, int D,
                           const int32_t* cu_q, const int32_t* cu_k, int32_t* ts_q, int32_t* ts_k,
                           int M, float softmax_scale, void* d_qh, void* d_kh, void* d_vh,
                           float* delta, const TokenGrads& tok, const SplitRoom& split, BwdForm form, hipStream_t st) {
  unsigned short *d_q_tok = (unsigned short*)tok.d_q, *d_k_tok = (unsigned short*)tok.d_k, *d_v_tok = (unsigned short*)tok.d_v;
  const int64_t rows = Nq * (int64_t)H;
  int* status = (int*)((char*)delta + bwd_rows_bytes(Nq, H));
  if (dtype == MOGA_BF16) {
    if (!bf16_rows_ok(Nq, Nk)) return MOGA_ERR_UNSUPPORTED;
    if (form == BwdForm::kTogether) {
      if (!tok.row_constants) launch_delta<16, true>(d_oh, oh, lse, rows, 1.f / softmax_scale, delta, delta + rows, status, st);
      const AttnBwdCall c = {(const unsigned short*)d_oh, (const unsigned short*)qh, (const unsigned short*)kh, (const unsigned short*)vh,
                             delta + rows, delta, cu_q, cu_k, nullptr, nullptr, Nq, Nk, (unsigned short*)d_qh, (unsigned short*)d_kh,
                             (unsigned short*)d_vh, d_q_tok, d_k_tok, d_v_tok, tok.perm, status, M};
      return launch_bwd_calls(&c, nullptr, 1, BwdKernels::kLarge, H, softmax_scale, st);
    }
    // groups of a few thousand rows or less (the static groups of Section 3.2): 4-wave blocks with a
    // two-slot ring, two blocks per CU, and smaller tiles; the host only knows the mean group size
    const AttnPlan plan = form == BwdForm::kSmall ? AttnPlan{true, {128, false}, {64, false}} : bwd_plan(Nq, Nk, H, M, split.rows);
    const bool small = plan.small;
    const int bk = plan.k.rows, bm = plan.q.rows;
    const int64_t k_tiles = Nk > 0 ? max_tiles(Nk, M, bk) : 0, q_tiles = max_tiles(Nq, M, bm);
    const int64_t k_blocks = (k_tiles * H + 7) / 8 * 8, q_blocks = (q_tiles * H + 7) / 8 * 8;
    if (!grid_fits(std::max(k_blocks, q_blocks), small ? 256 : 512)) return MOGA_ERR_UNSUPPORTED;
    float* lse2 = delta + rows;   // holds -lse/scale; `delta` holds -delta
    if (!tok.row_constants) launch_delta<16, true>(d_oh, oh, lse, rows, 1.f / softmax_scale, delta, lse2, status, st);
    if (ts_k && Nk > 0) tile_start_kernel<<<1, 1024, 0, st>>>(cu_k, M, bk, ts_k);
    if (ts_q) tile_start_kernel<<<1, 1024, 0, st>>>(cu_q, M, bm, ts_q);
    if (small) {
      auto launch = [&](int64_t dq_blocks, int64_t dkdv_blocks) {
        attn_bwd_small_kernel<<<(unsigned)(dq_blocks + dkdv_blocks), 256, 0, st>>>(
            (const unsigned short*)d_oh, (const unsigned short*)qh, (const unsigned short*)kh, (const unsigned short*)vh, lse2, delta,
            cu_q, cu_k, ts_q, ts_k, M, Nq, Nk, H, softmax_scale, (unsigned short*)d_qh, (unsigned short*)d_kh, (unsigned short*)d_vh,
            g_spin_limit.load(), status, tok.perm, d_q_tok, d_k_tok, d_v_tok, (int)dq_blocks);
      };
      if (grid_fits(q_blocks + k_blocks, 256)) {
        launch(q_blocks, k_blocks);
      } else {   // millions of groups
        launch(q_blocks, 0);
        if (k_blocks > 0) launch(0, k_blocks);
      }
      return launch_status();
    }
    if (Nk > 0) {
      const bool split_k = plan.k.split;
#define MOGA_BWD_DKDV(KK, SPLIT)                                                                                               \
  attn_bwd_dkdv_ab_kernel<KK, false, SPLIT><<<(unsigned)(k_blocks + (SPLIT ? kCus : 0)), 512, 0, st>>>(                        \
      (const unsigned short*)d_oh, (const unsigned short*)qh, (const unsigned short*)kh, (const unsigned short*)vh, lse2, delta, \
      cu_q, cu_k, SPLIT ? nullptr : ts_k, M, Nq, Nk, H, softmax_scale, (unsigned short*)d_kh, (unsigned short*)d_vh,            \
      g_spin_limit.load(), status, tok.perm, SPLIT ? (float*)split.ws : nullptr, d_k_tok, d_v_tok)
      if (split_k && bk == 192) MOGA_BWD_DKDV(192, true);
      else if (split_k) MOGA_BWD_DKDV(128, true);
      else if (bk == 192) MOGA_BWD_DKDV(192, false);
      else MOGA_BWD_DKDV(128, false);
#undef MOGA_BWD_DKDV
      if (split_k)
        split_sum_kernel<<<dim3(kCus / 2, 2 * bk / 8), 256, 0, st>>>((const float*)split.ws, cu_k, M, H, Nk, bk, 1.f, softmax_scale,
                                                                     (unsigned short*)d_vh, (unsigned short*)d_kh, d_v_tok, d_k_tok, tok.perm);
    }
    const bool split_q = plan.q.split;
#define MOGA_BWD_DQ(RR, SPLIT)                                                                                                  \
  attn_bwd_dq_pipe_kernel<RR, false, SPLIT><<<(unsigned)(q_blocks + (SPLIT ? kCus : 0)), 512, 0, st>>>(                        \
      (const unsigned short*)d_oh, (const unsigned short*)qh, (const unsigned short*)kh, (const unsigned short*)vh, lse2, delta, \
      cu_q, cu_k, SPLIT ? nullptr : ts_q, M, Nq, Nk, H, softmax_scale, (unsigned short*)d_qh, tok.perm,                         \
      SPLIT ? (float*)split.ws : nullptr, d_q_tok)
    if (split_q && bm == 384) MOGA_BWD_DQ(384, true);
    else if (split_q) MOGA_BWD_DQ(256, true);
    else if (bm == 384) MOGA_BWD_DQ(384, false);
    else MOGA_BWD_DQ(256, false);
#undef MOGA_BWD_DQ
    if (split_q)
      split_sum_kernel<<<dim3(kCus / 2, bm / 8), 256, 0, st>>>((const float*)split.ws, cu_q, M, H, Nq, bm, softmax_scale, 0.f,
                                                                   (unsigned short*)d_qh, nullptr, d_q_tok, nullptr, tok.perm);
  } else {
    const int64_t q_tiles = max_tiles(Nq, M, kF32Rows), k_tiles = Nk > 0 ? max_tiles(Nk, M, kF32Rows) : 0;
    if (!grid_fits(std::max(q_tiles, k_tiles) * H, 64 * kF32Waves)) return MOGA_ERR_UNSUPPORTED;
    if (!tok.row_constants && D == 64) launch_delta<16, false>(d_oh, oh, lse, rows, 0.f, delta, nullptr, status, st);
    if (!tok.row_constants && D == 128) launch_delta<32, false>(d_oh, oh, lse, rows, 0.f, delta, nullptr, status, st);
    if (ts_k && Nk > 0) tile_start_kernel<<<1, 1024, 0, st>>>(cu_k, M, kF32Rows, ts_k);
    if (ts_q) tile_start_kernel<<<1, 1024, 0, st>>>(cu_q, M, kF32Rows, ts_q);
    auto launch = [&](int64_t dq_blocks, int64_t dkdv_blocks) {
#define MOGA_BWD_F32(DD, TT)                                                                                          \
  attn_bwd_f32_kernel<DD, TT><<<(unsigned)(dq_blocks + dkdv_blocks), 64 * kF32Waves, 0, st>>>(                       \
      (const float*)d_oh, (const float*)qh, (const float*)kh, (const float*)vh, lse, delta, cu_q, cu_k, ts_q, ts_k, M, Nq,   \
      Nk, H, softmax_scale, (int)q_tiles, (int)k_tiles, (int)dkdv_blocks, (float*)d_qh, (float*)d_kh, (float*)d_vh,          \
      tok.perm, (float*)tok.d_q, (float*)tok.d_k, (float*)tok.d_v)
      if (D == 64 && std::max(Nq, Nk) > kF32ShortCall) MOGA_BWD_F32(64, 2);
      else if (D == 64) MOGA_BWD_F32(64, 1);
      else MOGA_BWD_F32(128, 1);
#undef MOGA_BWD_F32
    };
    if (grid_fits((q_tiles + k_tiles) * H, 64 * kF32Waves)) {
      launch(q_tiles * H, k_tiles * H);
    } else {
      if (k_tiles > 0) launch(0, k_tiles * H);
      launch(q_tiles * H, 0);
    }
  }
  return launch_status();
}

static int check_attn_bwd_args(int64_t Nq, int64_t Nk, int H, int D, int M, float softmax_scale, int dtype) {
  if (Nq < 0 || Nk < 0 || H < 1 || D < 1 || M < 1) return MOGA_ERR_INVALID_ARG;
  if (!(softmax_scale > 0.f) || !(softmax_scale < INFINITY)) return MOGA_ERR_INVALID_ARG;
  if (dtype != MOGA_F32 && dtype != MOGA_BF16) return MOGA_ERR_UNSUPPORTED;
  if (Nq >= ((int64_t)1 << 31) || Nk >= ((int64_t)1 << 31)) return MOGA_ERR_UNSUPPORTED;
  if (dtype == MOGA_BF16 && D != 128) return MOGA_ERR_UNSUPPORTED;
  if (dtype == MOGA_F32 && D != 64 && D != 128) return MOGA_ERR_UNSUPPORTED;
  return MOGA_OK;
}

static int group_attn_bwd(bool joint, const void* d_oh, const void* qh, const void* kh, const void* vh,
                                   const void* oh, const float* lse, int dtype, int64_t N, int H,
                                   int D, const int32_t* cu_seqlens, int M, float softmax_scale,
                                   void* d_qh, void* d_kh, void* d_vh, void* ws, size_t ws_bytes,
                                   void* stream) {
  const int bad = check_attn_bwd_args(N, N, H, D, M, softmax_scale, dtype);
  if (bad) return bad;
  if (M > MOGA_MAX_GROUPS) return MOGA_ERR_UNSUPPORTED;
  if (N == 0) return MOGA_OK;
  if (!d_oh || !qh || !kh || !vh || !oh || !lse || !cu_seqlens || !d_qh || !d_kh || !d_vh)
    return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(d_oh) && aligned16(qh) && aligned16(kh) && aligned16(vh) && aligned16(oh) &&
        aligned16(d_qh) && aligned16(d_kh) && aligned16(d_vh)))
    return MOGA_ERR_INVALID_ARG;
  const size_t need = moga_attn_bwd_ws_bytes(N, H, D, dtype);
  if (!ws || ws_bytes < need) return MOGA_ERR_WORKSPACE;
  const SplitRoom room = split_room(ws, need, ws_bytes);
  const BwdForm form = joint && dtype == MOGA_BF16 ? bwd_form(N, H, M, room.rows) : BwdForm::kApart;
  return launch_attn_bwd(d_oh, qh, kh, vh, oh, lse, dtype, N, N, H, D, cu_seqlens, cu_seqlens, nullptr,
                         nullptr, M, softmax_scale, d_qh, d_kh, d_vh, (float*)ws, TokenGrads{},
                         form == BwdForm::kApart ? room : SplitRoom{}, form, (hipStream_t)stream);
}

static int group_attn_bwd_tokens(bool joint, const void* d_o, const void* qh, const void* kh, const void* vh, const void* oh,
                                          const float* lse, int dtype, int64_t N, int H, int D, const int32_t* cu_seqlens, int M,
                                          float softmax_scale, const int32_t* perm, const float* gate, void* d_oh, float* d_gate,
                                          void* d_qh, void* d_kh, void* d_vh, void* d_q, void* d_k, void* d_v, void* ws,
                                          size_t ws_bytes, void* stream) {
  const int bad = check_attn_bwd_args(N, N, H, D, M, softmax_scale, dtype);
  if (bad) return bad;
  if (M > MOGA_MAX_GROUPS) return MOGA_ERR_UNSUPPORTED;
  if (dtype == MOGA_BF16 && !bf16_rows_ok(N, N)) return MOGA_ERR_UNSUPPORTED;
  if (N == 0) return MOGA_OK;
  if (!d_o || !qh || !kh || !vh || !oh || !lse || !cu_seqlens || !perm || !gate || !d_oh || !d_gate || !d_q || !d_k || !d_v)
    return MOGA_ERR_INVALID_ARG;
  if (!d_qh != !d_kh || !d_qh != !d_vh) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(d_o) && aligned16(d_oh) && aligned16(qh) && aligned16(kh) && aligned16(vh) && aligned16(oh) &&
        aligned16(d_qh) && aligned16(d_kh) && aligned16(d_vh) && aligned16(d_q) && aligned16(d_k) && aligned16(d_v)))
    return MOGA_ERR_INVALID_ARG;
  const size_t need = moga_attn_bwd_ws_bytes(N, H, D, dtype);
  if (!ws || ws_bytes < need) return MOGA_ERR_WORKSPACE;
  const SplitRoom room = split_room(ws, need, ws_bytes);
  const BwdForm form = joint && dtype == MOGA_BF16 ? bwd_form(N, H, M, room.rows) : BwdForm::kApart;
  float* delta = (float*)ws;
  const RowConstants rc = {lse, 1.f / softmax_scale, delta, delta + N * (int64_t)H, (int*)((char*)ws + bwd_rows_bytes(N, H))};
  const int rows = launch_unpermute_bwd(d_o, oh, dtype, perm, gate, N, H, D, d_oh, d_gate, &rc, (hipStream_t)stream);
  if (rows != MOGA_OK) return rows;
  return launch_attn_bwd(d_oh, qh, kh, vh, oh, lse, dtype, N, N, H, D, cu_seqlens, cu_seqlens, nullptr, nullptr, M,
                         softmax_scale, d_qh, d_kh, d_vh, delta, TokenGrads{d_q, d_k, d_v, perm, true},
                         form == BwdForm::kApart ? room : SplitRoom{}, form, (hipStream_t)stream);
}

extern "C" int moga_group_attn_bwd(
    const void* d_oh, const void* qh, const void* kh, const void* vh, const void* oh, const float* lse, int dtype, int64_t N, int H, int D,
    const int32_t* cu_seqlens, int M, float softmax_scale, void* d_qh, void* d_kh, void* d_vh, void* ws, size_t ws_bytes, void* stream) {
  return group_attn_bwd(false, d_oh, qh, kh, vh, oh, lse, dtype, N, H, D, cu_seqlens, M, softmax_scale, d_qh, d_kh, d_vh, ws, ws_bytes, stream);
}
extern "C" int moga_group_attn_bwd_joint(
    const void* d_oh, const void* qh, const void* kh, const void* vh, const void* oh, const float* lse, int dtype, int64_t N, int H, int D,
    const int32_t* cu_seqlens, int M, float softmax_scale, void* d_qh, void* d_kh, void* d_vh, void* ws, size_t ws_bytes, void* stream) {
  return group_attn_bwd(true, d_oh, qh, kh, vh, oh, lse, dtype, N, H, D, cu_seqlens, M, softmax_scale, d_qh, d_kh, d_vh, ws, ws_bytes, stream);
}
extern "C" int moga_group_attn_bwd_tokens(
    const void* d_o, const void* qh, const void* kh, const void* vh, const void* oh, const float* lse, int dtype, int64_t N, int H, int D,
    const int32_t* cu_seqlens, int M, float softmax_scale, const int32_t* perm, const float* gate, void* d_oh, float* d_gate, void* d_qh,
    void* d_kh, void* d_vh, void* d_q, void* d_k, void* d_v, void* ws, size_t ws_bytes, void* stream) {
  return group_attn_bwd_tokens(false, d_o, qh, kh, vh, oh, lse, dtype, N, H, D, cu_seqlens, M, softmax_scale, perm, gate, d_oh, d_gate, d_qh,
                               d_kh, d_vh, d_q, d_k, d_v, ws, ws_bytes, stream);
}
extern "C" int moga_group_attn_bwd_tokens_joint(
    const void* d_o, const void* qh, const void* kh, const void* vh, const void* oh, const float* lse, int dtype, int64_t N, int H, int D,
    const int32_t* cu_seqlens, int M, float softmax_scale, const int32_t* perm, const float* gate, void* d_oh, float* d_gate, void* d_qh,
    void* d_kh, void* d_vh, void* d_q, void* d_k, void* d_v, void* ws, size_t ws_bytes, void* stream) {
  return group_attn_bwd_tokens(true, d_o, qh, kh, vh, oh, lse, dtype, N, H, D, cu_seqlens, M, softmax_scale, perm, gate, d_oh, d_gate, d_qh,
                               d_kh, d_vh, d_q, d_k, d_v, ws, ws_bytes, stream);
}

extern "C" size_t moga_varlen_attn_bwd_ws_bytes(int64_t Nq, int H, int G) {
  if (Nq <= 0 || H < 1) return 0;
  return bwd_rows_bytes(Nq, H) + 16 + 2 * ((size_t)G + 1) * sizeof(int32_t);
}

static int check_varlen_bwd(const moga_attn_bwd_call& c, int dtype, int H, int D, float softmax_scale) {
  const int bad = check_attn_bwd_args(c.Nq, c.Nk, H, D, c.G, softmax_scale, dtype);
  if (bad) return bad;
  if (c.G > MOGA_MAX_SEGMENTS) return MOGA_ERR_UNSUPPORTED;
  if (c.Nq == 0 && c.Nk == 0) return MOGA_OK;
  if (!c.cu_seqlens_q || !c.cu_seqlens_k) return MOGA_ERR_INVALID_ARG;
  if (c.Nq > 0 && (!c.d_oh || !c.qh || !c.oh || !c.lse || !c.d_qh)) return MOGA_ERR_INVALID_ARG;
  if (c.Nk > 0 && (!c.kh || !c.vh || !c.d_kh || !c.d_vh)) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(c.d_oh) && aligned16(c.qh) && aligned16(c.kh) && aligned16(c.vh) && aligned16(c.oh) &&
        aligned16(c.d_qh) && aligned16(c.d_kh) && aligned16(c.d_vh)))
    return MOGA_ERR_INVALID_ARG;
  if (c.Nq > 0 && (!c.ws || c.ws_bytes < moga_varlen_attn_bwd_ws_bytes(c.Nq, H, c.G) || !aligned16(c.ws))) return MOGA_ERR_WORKSPACE;
  return MOGA_OK;
}

static int varlen_attn_bwd(const moga_attn_bwd_call& c, int dtype, int H, int D, float softmax_scale, bool row_constants, void* stream) {
  const int bad = check_varlen_bwd(c, dtype, H, D, softmax_scale);
  if (bad || (c.Nq == 0 && c.Nk == 0)) return bad;
  hipStream_t st = (hipStream_t)stream;
  if (c.Nq == 0) {   // keys without any query: zero gradients
    const int64_t nf = c.Nk * (int64_t)H * D / (dtype == MOGA_BF16 ? 2 : 1);
    launch_fill_zero((float*)c.d_kh, nf, st);
    launch_fill_zero((float*)c.d_vh, nf, st);
    return launch_status();
  }
  const size_t need = moga_varlen_attn_bwd_ws_bytes(c.Nq, H, c.G);
  const bool presum = c.G > MOGA_MAX_GROUPS;   // few groups: every block looks its tile up itself
  int32_t* ts_q = presum ? (int32_t*)((char*)c.ws + bwd_rows_bytes(c.Nq, H) + 16) : nullptr;
  int32_t* ts_k = presum ? ts_q + (c.G + 1) : nullptr;
  return launch_attn_bwd(c.d_oh, c.qh, c.kh, c.vh, c.oh, c.lse, dtype, c.Nq, c.Nk, H, D, c.cu_seqlens_q, c.cu_seqlens_k, ts_q, ts_k, c.G,
                         softmax_scale, c.d_qh, c.d_kh, c.d_vh, (float*)c.ws, TokenGrads{nullptr, nullptr, nullptr, nullptr, row_constants},
                         presum ? SplitRoom{} : split_room(c.ws, need, c.ws_bytes), BwdForm::kApart, st);
}

extern "C" int moga_varlen_attn_bwd(const void* d_oh, const void* qh, const void* kh, const void* vh,
                                    const void* oh, const float* lse, int dtype, int64_t Nq,
                                    int64_t Nk, int H, int D, const int32_t* cu_seqlens_q,
                                    const int32_t* cu_seqlens_k, int G, float softmax_scale,
                                    void* d_qh, void* d_kh, void* d_vh, void* ws, size_t ws_bytes,
                                    void* stream) {
  return varlen_attn_bwd({d_oh, qh, kh, vh, oh, lse, cu_seqlens_q, cu_seqlens_k, Nq, Nk, G, d_qh, d_kh, d_vh, ws, ws_bytes}, dtype, H, D,
                         softmax_scale, false, stream);
}

extern "C" int moga_varlen_attn_bwd_rows(const void* d_oh, const void* qh, const void* kh, const void* vh,
                                         const void* oh, const float* lse, int dtype, int64_t Nq,
                                         int64_t Nk, int H, int D, const int32_t* cu_seqlens_q,
                                         const int32_t* cu_seqlens_k, int G, float softmax_scale,
                                         void* d_qh, void* d_kh, void* d_vh, void* ws, size_t ws_bytes,
                                         void* stream) {
  return varlen_attn_bwd({d_oh, qh, kh, vh, oh, lse, cu_seqlens_q, cu_seqlens_k, Nq, Nk, G, d_qh, d_kh, d_vh, ws, ws_bytes}, dtype, H, D,
                         softmax_scale, true, stream);
}

extern "C" int moga_varlen_attn_bwd_rows_calls(const moga_attn_bwd_call* calls, int n, int dtype, int H, int D, float softmax_scale,
                                               void* stream) {
  if (!calls || n < 1 || n > MOGA_MAX_CALLS) return MOGA_ERR_INVALID_ARG;
  int64_t rows = 0;
  int order[kMaxCalls], count = 0;
  bool together = dtype == MOGA_BF16;
  for (int i = 0; i < n; ++i) {
    const moga_attn_bwd_call& c = calls[i];
    const int bad = check_varlen_bwd(c, dtype, H, D, softmax_scale);
    if (bad) return bad;
    if (dtype == MOGA_BF16 && !bf16_rows_ok(c.Nq, c.Nk)) return MOGA_ERR_UNSUPPORTED;
    rows += c.Nq;
    if (c.Nq > 0) order[count++] = i;
    else if (c.Nk > 0) together = false;   // keys without any query
  }
  if (!together || count < 2) {
    for (int i = 0; i < n; ++i) {
      const int rc = varlen_attn_bwd(calls[i], dtype, H, D, softmax_scale, true, stream);
      if (rc != MOGA_OK) return rc;
    }
    return MOGA_OK;
  }
  auto small = [&](int i) { return use_small_group_kernels(calls[i].Nq, calls[i].G, calls_small_group_rows(rows, H)); };
  int* const mid = std::stable_partition(order, order + count, [&](int i) { return !small(i); });
  auto launch = [&](const int* first, const int* last, BwdKernels kernels) -> int {
    if (first == last) return MOGA_OK;
    AttnBwdCall a[kMaxCalls];
    int32_t* ts[kMaxCalls];
    const int m = (int)(last - first);
    for (int i = 0; i < m; ++i) {
      const moga_attn_bwd_call& c = calls[first[i]];
      char* ws = (char*)c.ws;
      ts[i] = (int32_t*)(ws + bwd_rows_bytes(c.Nq, H) + 16);
      a[i] = {(const unsigned short*)c.d_oh, (const unsigned short*)c.qh, (const unsigned short*)c.kh, (const unsigned short*)c.vh,
              (float*)ws + c.Nq * (int64_t)H, (float*)ws, c.cu_seqlens_q, c.cu_seqlens_k, nullptr, nullptr, c.Nq, c.Nk,
              (unsigned short*)c.d_qh, (unsigned short*)c.d_kh, (unsigned short*)c.d_vh, nullptr, nullptr, nullptr, nullptr,
              (int*)(ws + bwd_rows_bytes(c.Nq, H)), c.G};
    }
    int rc = launch_bwd_calls(a, ts, m, kernels, H, softmax_scale, (hipStream_t)stream);
    if (rc == MOGA_ERR_UNSUPPORTED) {   // millions of groups: together too many threads for a grid
      rc = MOGA_OK;
      for (int i = 0; i < m && rc == MOGA_OK; ++i) rc = varlen_attn_bwd(calls[first[i]], dtype, H, D, softmax_scale, true, stream);
    }
    return rc;
  };
  const int rc = launch(order, mid, BwdKernels::kLarge);
  return rc != MOGA_OK ? rc : launch(mid, order + count, BwdKernels::kSmall);
}

extern "C" int moga_fused_attn_bwd(const void* d_o, const void* q, const void* k, const void* v,
                                   const void* o, const float* lse, int dtype, int64_t N, int H, int D,
                                   const int32_t* perm, const int32_t* inv_perm, const float* gate,
                                   const int32_t* cu_seqlens, int M, float softmax_scale, void* d_q,
                                   void* d_k, void* d_v, float* d_gate, void* ws, size_t ws_bytes,
                                   void* stream) {
  const int bad = check_attn_bwd_args(N, N, H, D, M, softmax_scale, dtype);
  if (bad) return bad;
  if (M > MOGA_MAX_GROUPS || dtype != MOGA_BF16 || !bf16_rows_ok(N, N)) return MOGA_ERR_UNSUPPORTED;
  if (N == 0) return MOGA_OK;
  if (!d_o || !q || !k || !v || !o || !lse || !perm || !inv_perm || !gate || !cu_seqlens || !d_q || !d_k ||
      !d_v || !d_gate)
    return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(d_o) && aligned16(q) && aligned16(k) && aligned16(v) && aligned16(o) && aligned16(d_q) &&
        aligned16(d_k) && aligned16(d_v)))
    return MOGA_ERR_INVALID_ARG;
  const size_t need = moga_attn_bwd_ws_bytes(N, H, D, dtype);
  if (!ws || ws_bytes < need) return MOGA_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  float* delta = (float*)ws;
  float* lse2 = delta + N * (int64_t)H;
  int* status = (int*)((char*)ws + bwd_rows_bytes(N, H));
  const bool apart = fused_apart(N, H, M);
  const int rows_q = query_blocks(N, N, H, M, 0).rows, keys = key_blocks(N, N, H, M, 0).rows;   // apart
  const int64_t k_blocks = (max_tiles(N, M, keys) * H + 7) / 8 * 8, q_blocks = (max_tiles(N, M, rows_q) * H + 7) / 8 * 8;
  if (apart && !grid_fits(std::max(k_blocks, q_blocks), 512)) return MOGA_ERR_UNSUPPORTED;
  attn_bwd_fused_prepass_kernel<<<(unsigned)((N + kPrepassTokens - 1) / kPrepassTokens), 256, 0, st>>>(
      (const uintx4_t*)d_o, (const uintx4_t*)o, lse, inv_perm, gate, N, H, 1.f / softmax_scale, lse2, delta, d_gate, status);
  if (apart) {
#define MOGA_BWD_DKDV(KK)                                                                                                   \
  attn_bwd_dkdv_ab_kernel<KK, true><<<(unsigned)k_blocks, 512, 0, st>>>(                                                    \
      (const unsigned short*)d_o, (const unsigned short*)q, (const unsigned short*)k, (const unsigned short*)v, lse2, delta, \
      cu_seqlens, cu_seqlens, nullptr, M, N, N, H, softmax_scale, (unsigned short*)d_k, (unsigned short*)d_v,               \
      g_spin_limit.load(), status, perm)
    if (keys == 192) MOGA_BWD_DKDV(192);
    else MOGA_BWD_DKDV(128);
#undef MOGA_BWD_DKDV
#define MOGA_BWD_DQ(RR)                                                                                                     \
  attn_bwd_dq_pipe_kernel<RR, true><<<(unsigned)q_blocks, 512, 0, st>>>(                                                    \
      (const unsigned short*)d_o, (const unsigned short*)q, (const unsigned short*)k, (const unsigned short*)v, lse2, delta, \
      cu_seqlens, cu_seqlens, nullptr, M, N, N, H, softmax_scale, (unsigned short*)d_q, perm)
    if (rows_q == 384) MOGA_BWD_DQ(384);
    else MOGA_BWD_DQ(256);
#undef MOGA_BWD_DQ
    return launch_status();
  }
  const AttnBwdCall c = {(const unsigned short*)d_o, (const unsigned short*)q, (const unsigned short*)k, (const unsigned short*)v, lse2, delta,
                         cu_seqlens, cu_seqlens, nullptr, nullptr, N, N, (unsigned short*)d_q, (unsigned short*)d_k, (unsigned short*)d_v,
                         nullptr, nullptr, nullptr, perm, status, M};
  return launch_bwd_calls(&c, nullptr, 1, BwdKernels::kGather, H, softmax_scale, st);
}

extern "C" size_t moga_workspace_preferred_bytes(int op, int64_t N, int64_t Nk, int H, int D, int M, int d_model, int dtype) {
  const size_t need = moga_workspace_bytes(op, N, H, D, M, d_model, dtype);
  if (dtype != MOGA_BF16 || D != 128 || N <= 0 || Nk <= 0 || H < 1 || M < 1) return need;
  const bool fwd = op == MOGA_OP_ATTN_FWD || op == MOGA_OP_VARLEN_ATTN_FWD;
  const bool bwd = op == MOGA_OP_ATTN_BWD || op == MOGA_OP_VARLEN_ATTN_BWD || op == MOGA_OP_ATTN_BWD_JOINT;
  if (M > MOGA_MAX_GROUPS) return need;
  if (op == MOGA_OP_ATTN_FWD_CALL) return fwd_call_alone(N, H, M) ? moga_workspace_preferred_bytes(MOGA_OP_VARLEN_ATTN_FWD, N, Nk, H, D, M, d_model, dtype) : need;
  if (op == MOGA_OP_ATTN_BWD_JOINT && (N != Nk || bwd_form(N, H, M, 384) != BwdForm::kApart)) return need;
  if (!fwd && !bwd) return need;
  auto plan = [&](int room) { return fwd ? fwd_plan(N, Nk, H, M, room) : bwd_plan(N, Nk, H, M, room); };
  const AttnPlan p = plan(384), q = plan(256);
  if (!p.q.split && !p.k.split) return need;
  const bool same = p.small == q.small && p.q.rows == q.q.rows && p.q.split == q.q.split && p.k.rows == q.k.rows && p.k.split == q.k.split;
  return round_up(need, 256) + 256 + split_bytes(same ? 256 : 384);
}

extern "C" void moga_debug_attn_blocks(int op, int64_t Nq, int64_t Nk, int H, int M, size_t ws_bytes, int blocks[4]) {
  const bool fwd = op == MOGA_OP_ATTN_FWD || op == MOGA_OP_VARLEN_ATTN_FWD;
  const int room = M > MOGA_MAX_GROUPS ? 0 : split_room((void*)256, moga_workspace_bytes(op, Nq, H, 128, M, 0, MOGA_BF16), ws_bytes).rows;
  const bool gather = op == MOGA_OP_FUSED_ATTN_BWD;
  const BwdForm form = gather ? (fused_apart(Nq, H, M) ? BwdForm::kApart : BwdForm::kTogether)
                              : op == MOGA_OP_ATTN_BWD_JOINT ? bwd_form(Nq, H, M, room) : BwdForm::kApart;
  AttnPlan p = fwd ? fwd_plan(Nq, Nk, H, M, room) : bwd_plan(Nq, Nk, H, M, room);
  if (form == BwdForm::kSmall) p = {true, {128, false}, {64, false}};
  if (gather) p = {false, query_blocks(Nq, Nk, H, M, 0), key_blocks(Nq, Nk, H, M, 0)};
  blocks[0] = p.q.rows, blocks[1] = p.q.split, blocks[2] = p.k.rows, blocks[3] = p.k.split;
  if (form == BwdForm::kTogether) {
    const SideShape side = {Nq, Nq, M};
    const BwdBlocks b = bwd_blocks(&side, 1, H, gather);
    blocks[0] = b.bm, blocks[2] = b.bk;
    blocks[1] = blocks[3] = 2;
  }
}

extern "C" int moga_debug_small_calls(int op, int n, const int64_t* Nq, const int* G, int H) {
  int64_t rows = 0, shortest = INT64_MAX;
  for (int i = 0; i < n; ++i) {
    rows += Nq[i];
    shortest = std::min(shortest, Nq[i] / G[i]);
  }
  const int64_t line = op == MOGA_OP_VARLEN_ATTN_FWD ? fwd_calls_small_rows(rows, H, shortest) : calls_small_group_rows(rows, H);
  int small = 0;
  for (int i = 0; i < n; ++i) small |= use_small_group_kernels(Nq[i], G[i], line) << i;
  return small;
}
