// Variable-length attention inside groups (Alg. 1 step 3 of the paper; Eq. 1 per group/head).
//
// bf16 kernel, head_dim 128, 16x16x32 bf16 MFMA:
//   * scores are computed transposed, S^T = K Q^T, so that each lane owns two or three query columns:
//     their softmax statistics are per-lane scalars, and the four lanes of a query only meet when
//     its maximum is raised and at the end;
//   * the K rows fed to the MFMA are permuted (attn_common.h, step_row) so a lane's eight scores of a
//     query are eight consecutive keys -- exactly the B operand of the second product
//     O^T = V^T P^T, which therefore needs no data movement for P;
//   * V^T is read from the row-major V tile in LDS with the transposing LDS read;
//   * the kernel itself (software pipeline, LDS ring, direct-to-LDS loads) is in attn_pipe.h.
// fp32 kernel (fp32 matrix instruction, full precision throughout): attn_f32.h.
#include <algorithm>
#include <climits>

#include "attn_common.h"
#include "attn_f32.h"
#include "attn_pipe.h"
#include "attn_pipe_small.h"

namespace moga {

// Mean rows per group below which the small-group bf16 kernel runs, by rounds of 256 blocks of 256 rows.  Time of the small kernel
// against the large one's (blocks by large_blocks) with room to split a round, groups of equal / Zipf(1.1) sizes, in %; in brackets without room:
//   rounds 0.15  1,560 rows -6 / +63 [-26 / -28], 2,000 +6 / +74 [-26 / -28];   0.25  2,500 -3 / +49 [-24 / -28], 3,200 +4 / +55 [-25 / -28]
//          0.4   5,000 -2 / +21 [-26 / -28], 6,200 +4 / +23;                    0.6   3,200 +7 / -24 [+13 / -22], 5,000 +12 / -2 [+12 / -23]
//          0.85  2,500 +8 / +1 [+13 / +3], 5,000 +7 / -18 [+10 / -17];          1.1   1,250 +11 / -16 [+18 / -15], 2,500 +21 / -20
//          1.2   1,560 +8 / -17 [+13 / -18], 2,500 +19 / -16;                   1.6   1,560 +5 / -20 [+7 / -19], 2,500 +8 / -1
//          2.6   1,560 +1 / 0, 2,000 +4 / -1;                                   3.4   2,000 -4 / +2, 3,200 +2 / +2
//          4.5   1,000 -6 / -4, 1,560 +5 / +2;                                  6.6   600 -8 / +1, 700 +4 / -4
//          8     600 -6 / +1, 700 +7 / +1;       12    600 -7 / +2, 700 +10 / 0;       20    600 -5 / +9, 700 +10 / +7
// Below half a round and above two the lines are where groups of equal size take about the same time by both.  Between, the small kernel costs
// equal groups, what a balanced router makes, up to 20 %, and gains 16 to 24 % where groups are as unequal as Zipf's, since its finer tiles end
// together: the lines there are those of the unequal groups, and equal ones of 1,000 rows and more pay for them.  Below a third of a round it is the other
// way round: with room the large kernel splits a long group's keys and would be the faster one for Zipf groups down to 1,000 rows.
// Below three quarters of a round the large kernel needs room to split its tiles; without, the line is that of the kernels unsplit.
static int64_t small_group_rows(int64_t Nq, int H, bool split) {
  const int64_t rounds = 100 * Nq * H / (256 * kCus);   // in hundredths
  if (split && rounds < 75) return rounds < 20 ? 1500 : rounds < 33 ? 2700 : rounds < 50 ? 5632 : 4500;
  return rounds < 50 ? 5632 : rounds < 100 ? 6144 : rounds < 370 ? 2560 : rounds < 600 ? 1300 : 700;
}

// The same for the calls of one launch, all of them with `rows` queries, the shortest groups with `shortest` rows on average.  From one to eight rounds
// all take the small kernels unless all have long groups.  Blocks of three branches (windows, frames of 1,560 tokens, routed groups of up to 8,400), over
// the time of the calls one by one, with the large kernels for all / with the small ones, mean and range: windows of 4 tokens 1.28 (1.10 to 1.43) /
// 0.91 (0.77 to 1.00), 6 to 15 1.07 (0.85 to 1.24) / 0.86 (0.70 to 0.98), 24 to 40 0.93 (0.74 to 1.05) / 0.85 (0.72 to 0.98), 100 to 300 0.86 (0.70 to
// 1.05) / 0.85 (0.72 to 0.97), 300 to 1,500 0.90 (0.75 to 1.07) / 0.87 (0.73 to 0.99), longer ones 0.91 (0.86 to 0.94) / 0.93 (0.88 to 0.98).  From
// eight rounds on windows of less than 300 tokens take them: 4 tokens 0.96 (with the large kernels 1.38), 40 to 100 0.92 (0.94).
int64_t fwd_calls_small_rows(int64_t rows, int H, int64_t shortest) {
  const int64_t rounds = 100 * rows * H / (256 * kCus);
  if (rounds < 100) return small_group_rows(rows, H, false);
  return rounds < 800 ? (shortest < 1500 ? INT64_MAX : 0) : 300;
}
// One of the calls of a launch that runs by itself, with its last round split: long groups, whose few blocks the others are too short to even out.
// With it in the launch the three took up to 1.42 of the time of the calls one by one (24,960 x 4 heads, 2 groups, windows of 64 tokens 1.25; 99,840 x 1,
// 4 groups 1.40), with the small kernels for all up to 1.19.  The bound is on its rows and stands for eight rounds of three branches.
bool fwd_call_alone(int64_t Nq, int H, int G) { return G <= MOGA_MAX_GROUPS && Nq >= 8192 * (int64_t)G && 3 * Nq * H < 8 * 256 * kCus; }

AttnPlan fwd_plan(int64_t Nq, int64_t Nk, int H, int M, int room) {
  if (use_small_group_kernels(Nq, M, small_group_rows(Nq, H, room > 0))) return {true, {128, false}, {}};
  return {false, query_blocks(Nq, Nk, H, M, room), {}};
}

}  // namespace moga

using namespace moga;

// Where the output rows go in token order as well: o [N, H, D] or NULL, row j of the sorted order at token perm[j], times
// gate[perm[j]].
struct TokenRows {
  void* o;
  const int32_t* perm;
  const float* gate;
};

// Shared launcher.  tile_start == NULL: tile lookup inside the kernels (M <= MOGA_MAX_GROUPS).  split: room
// for the pieces of the last round, if any (only with tile_start == NULL).
static int launch_attn_fwd(const void* qh, const void* kh, const void* vh, int dtype, int64_t Nq,
                           int64_t Nk, int H, int D, const int32_t* cu_q, const int32_t* cu_k,
                           int32_t* tile_start, int M, float softmax_scale, void* oh, float* lse,
                           const TokenRows& tok, const SplitRoom& split, hipStream_t st) {
  // bf16: groups of a few thousand rows or less (the static groups of Section 3.2) take the kernel
  // with 128-row tiles and two 4-wave blocks per CU; the host only knows the mean group size
  const AttnPlan plan = dtype == MOGA_BF16 ? fwd_plan(Nq, Nk, H, M, split.rows) : AttnPlan{};
  const bool small = plan.small;
  const int rows = plan.q.rows, bm = dtype == MOGA_BF16 ? rows : kF32Rows;
  const int64_t tiles = max_tiles(Nq, M, bm);
  const int64_t blocks = dtype == MOGA_BF16 ? (tiles * H + 7) / 8 * 8 : tiles * H;
  if (!grid_fits(blocks, dtype == MOGA_BF16 && !small ? 512 : 256)) return MOGA_ERR_UNSUPPORTED;
  if (tile_start) tile_start_kernel<<<1, 1024, 0, st>>>(cu_q, M, bm, tile_start);
  if (dtype == MOGA_F32) {
#define MOGA_FWD_F32(DD, TT)                                                                                               \
  attn_fwd_f32_kernel<DD, TT><<<(unsigned)blocks, 64 * kF32Waves, 0, st>>>(                                                \
      (const float*)qh, (const float*)kh, (const float*)vh, cu_q, cu_k, tile_start, M, Nq, Nk, H, softmax_scale, (int)tiles, \
      (float*)oh, lse, tok.perm, tok.gate, (float*)tok.o)
    if (D == 64 && Nk > kF32ShortCall) MOGA_FWD_F32(64, 2);
    else if (D == 64) MOGA_FWD_F32(64, 1);
    else MOGA_FWD_F32(128, 1);
#undef MOGA_FWD_F32
  } else if (small) {
    attn_fwd_bf16_small_kernel<<<(unsigned)blocks, 256, 0, st>>>(
        (const unsigned short*)qh, (const unsigned short*)kh, (const unsigned short*)vh, cu_q, cu_k,
        tile_start, M, Nq, Nk, H, softmax_scale, (unsigned short*)oh, lse, tok.perm, tok.gate, (unsigned short*)tok.o);
  } else if (plan.q.split) {
    const SplitWs sw = split_ws(split.ws, rows);
#define MOGA_FWD_SPLIT(RR)                                                                                                     \
  attn_fwd_bf16_pipe_kernel<RR, false, true><<<(unsigned)(blocks + kCus), 512, 0, st>>>(                                       \
      (const unsigned short*)qh, (const unsigned short*)kh, (const unsigned short*)vh, cu_q, cu_k, nullptr, M, Nq, Nk, H,      \
      softmax_scale, (unsigned short*)oh, lse, tok.perm, tok.gate, sw, (unsigned short*)tok.o)
    if (rows == 384) MOGA_FWD_SPLIT(384);
    else MOGA_FWD_SPLIT(256);
#undef MOGA_FWD_SPLIT
    split_fwd_kernel<<<dim3(kCus / 2, rows / 8), 256, 0, st>>>(sw, rows, cu_q, cu_k, M, H, Nq, (unsigned short*)oh, lse, tok.perm,
                                                               tok.gate, (unsigned short*)tok.o);
  } else {
#define MOGA_FWD(RR)                                                                                                           \
  attn_fwd_bf16_pipe_kernel<RR><<<(unsigned)blocks, 512, 0, st>>>(                                                             \
      (const unsigned short*)qh, (const unsigned short*)kh, (const unsigned short*)vh, cu_q, cu_k, tile_start, M, Nq, Nk, H,   \
      softmax_scale, (unsigned short*)oh, lse, tok.perm, tok.gate, SplitWs{}, (unsigned short*)tok.o)
    if (rows == 384) MOGA_FWD(384);
    else MOGA_FWD(256);
#undef MOGA_FWD
  }
  return launch_status();
}

static int check_attn_args(int64_t Nq, int64_t Nk, int H, int D, int M, float softmax_scale, int dtype) {
  if (Nq < 0 || Nk < 0 || H < 1 || D < 1 || M < 1) return MOGA_ERR_INVALID_ARG;
  if (!(softmax_scale > 0.f) || !(softmax_scale < INFINITY)) return MOGA_ERR_INVALID_ARG;
  if (dtype != MOGA_F32 && dtype != MOGA_BF16) return MOGA_ERR_UNSUPPORTED;
  if (Nq >= ((int64_t)1 << 31) || Nk >= ((int64_t)1 << 31)) return MOGA_ERR_UNSUPPORTED;
  if (dtype == MOGA_BF16 && D != 128) return MOGA_ERR_UNSUPPORTED;
  if (dtype == MOGA_F32 && D != 64 && D != 128) return MOGA_ERR_UNSUPPORTED;
  // the bf16 kernels form per-lane byte offsets `row * 256` in 32 bits, relative to the first row
  // of a group: a group (hence a tensor) must have fewer than 2^24 rows
  if (dtype == MOGA_BF16 && (Nq >= ((int64_t)1 << 24) || Nk >= ((int64_t)1 << 24))) return MOGA_ERR_UNSUPPORTED;
  return MOGA_OK;
}

static int group_attn_fwd(const void* qh, const void* kh, const void* vh, int dtype, int64_t N, int H, int D,
                          const int32_t* cu_seqlens, int M, float softmax_scale, void* oh, float* lse, const TokenRows& tok,
                          void* ws, size_t ws_bytes, void* stream) {
  const int bad = check_attn_args(N, N, H, D, M, softmax_scale, dtype);
  if (bad) return bad;
  if (M > MOGA_MAX_GROUPS) return MOGA_ERR_UNSUPPORTED;
  if (N == 0) return MOGA_OK;
  if (!qh || !kh || !vh || !cu_seqlens || !oh || !lse) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(qh) && aligned16(kh) && aligned16(vh) && aligned16(oh) && aligned16(tok.o))) return MOGA_ERR_INVALID_ARG;
  return launch_attn_fwd(qh, kh, vh, dtype, N, N, H, D, cu_seqlens, cu_seqlens, nullptr, M,
                         softmax_scale, oh, lse, tok, split_room(ws, 0, ws_bytes), (hipStream_t)stream);
}

extern "C" int moga_group_attn_fwd_ws(const void* qh, const void* kh, const void* vh, int dtype,
                                      int64_t N, int H, int D, const int32_t* cu_seqlens, int M,
                                      float softmax_scale, void* oh, float* lse, void* ws,
                                      size_t ws_bytes, void* stream) {
  return group_attn_fwd(qh, kh, vh, dtype, N, H, D, cu_seqlens, M, softmax_scale, oh, lse, TokenRows{}, ws, ws_bytes, stream);
}

extern "C" int moga_group_attn_fwd_tokens(const void* qh, const void* kh, const void* vh, int dtype,
                                          int64_t N, int H, int D, const int32_t* cu_seqlens, int M,
                                          float softmax_scale, const int32_t* perm, const float* gate,
                                          void* oh, float* lse, void* o, void* ws, size_t ws_bytes, void* stream) {
  if (N > 0 && (!perm || !gate || !o)) return MOGA_ERR_INVALID_ARG;
  return group_attn_fwd(qh, kh, vh, dtype, N, H, D, cu_seqlens, M, softmax_scale, oh, lse, TokenRows{o, perm, gate}, ws,
                        ws_bytes, stream);
}

// Needs no workspace and touches none: a caller may pass one that other streams are using.
extern "C" int moga_group_attn_fwd(const void* qh, const void* kh, const void* vh, int dtype,
                                   int64_t N, int H, int D, const int32_t* cu_seqlens, int M,
                                   float softmax_scale, void* oh, float* lse, void* ws,
                                   size_t ws_bytes, void* stream) {
  (void)ws; (void)ws_bytes;
  return moga_group_attn_fwd_ws(qh, kh, vh, dtype, N, H, D, cu_seqlens, M, softmax_scale, oh, lse, nullptr, 0, stream);
}

extern "C" int moga_fused_attn_fwd(const void* q, const void* k, const void* v, int dtype, int64_t N,
                                   int H, int D, const int32_t* perm, const float* gate,
                                   const int32_t* cu_seqlens, int M, float softmax_scale, void* o,
                                   float* lse, void* stream) {
  const int bad = check_attn_args(N, N, H, D, M, softmax_scale, dtype);
  if (bad) return bad;
  if (M > MOGA_MAX_GROUPS || dtype != MOGA_BF16) return MOGA_ERR_UNSUPPORTED;
  if (N == 0) return MOGA_OK;
  if (!q || !k || !v || !perm || !gate || !cu_seqlens || !o || !lse) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(q) && aligned16(k) && aligned16(v) && aligned16(o))) return MOGA_ERR_INVALID_ARG;
  const int rows = query_blocks(N, N, H, M, 0).rows;
  const int64_t blocks = (max_tiles(N, M, rows) * H + 7) / 8 * 8;
  if (!grid_fits(blocks, 512)) return MOGA_ERR_UNSUPPORTED;
#define MOGA_FWD(RR)                                                                                                             \
  attn_fwd_bf16_pipe_kernel<RR, true><<<(unsigned)blocks, 512, 0, (hipStream_t)stream>>>(                                        \
      (const unsigned short*)q, (const unsigned short*)k, (const unsigned short*)v, cu_seqlens, cu_seqlens, nullptr, M, N, N, H, \
      softmax_scale, (unsigned short*)o, lse, perm, gate)
  if (rows == 384) MOGA_FWD(384);
  else MOGA_FWD(256);
#undef MOGA_FWD
  return launch_status();
}

extern "C" size_t moga_varlen_attn_fwd_ws_bytes(int G) { return ((size_t)G + 1) * sizeof(int32_t); }

static int check_varlen_fwd(const moga_attn_fwd_call& c, int dtype, int H, int D, float softmax_scale) {
  const int bad = check_attn_args(c.Nq, c.Nk, H, D, c.G, softmax_scale, dtype);
  if (bad) return bad;
  if (c.G > MOGA_MAX_SEGMENTS) return MOGA_ERR_UNSUPPORTED;
  if (c.Nq == 0) return MOGA_OK;
  if (!c.qh || !c.cu_seqlens_q || !c.cu_seqlens_k || !c.oh || !c.lse) return MOGA_ERR_INVALID_ARG;
  if (c.Nk > 0 && (!c.kh || !c.vh)) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(c.qh) && aligned16(c.kh) && aligned16(c.vh) && aligned16(c.oh))) return MOGA_ERR_INVALID_ARG;
  if (!c.ws || c.ws_bytes < moga_varlen_attn_fwd_ws_bytes(c.G)) return MOGA_ERR_WORKSPACE;
  return MOGA_OK;
}

extern "C" int moga_varlen_attn_fwd(const void* qh, const void* kh, const void* vh, int dtype,
                                    int64_t Nq, int64_t Nk, int H, int D,
                                    const int32_t* cu_seqlens_q, const int32_t* cu_seqlens_k, int G,
                                    float softmax_scale, void* oh, float* lse, void* ws,
                                    size_t ws_bytes, void* stream) {
  const int bad = check_varlen_fwd({qh, kh, vh, cu_seqlens_q, cu_seqlens_k, Nq, Nk, G, oh, lse, ws, ws_bytes}, dtype, H, D, softmax_scale);
  if (bad) return bad;
  if (Nq == 0) return MOGA_OK;
  int32_t* ts = G <= MOGA_MAX_GROUPS ? nullptr : (int32_t*)ws;   // few groups: every block looks its tile up itself
  const SplitRoom split = ts ? SplitRoom{} : split_room(ws, moga_varlen_attn_fwd_ws_bytes(G), ws_bytes);
  return launch_attn_fwd(qh, kh, vh, dtype, Nq, Nk, H, D, cu_seqlens_q, cu_seqlens_k, ts, G,
                         softmax_scale, oh, lse, TokenRows{}, split, (hipStream_t)stream);
}

// The bf16 calls `which` in one launch of the kernels for small groups, or of the large ones with `rows` per block.
static int launch_fwd_calls(const moga_attn_fwd_call* calls, const int* which, int n, bool small, int rows, int H, float softmax_scale,
                            hipStream_t st) {
  AttnFwdCalls a = {};
  int64_t blocks = 0;
  std::fill(a.first, a.first + kMaxCalls, INT_MAX);
  for (int i = 0; i < n; ++i) {
    const moga_attn_fwd_call& c = calls[which[i]];
    a.first[i] = (int)blocks;
    blocks += (max_tiles(c.Nq, c.G, rows) * H + 7) / 8 * 8;
    if (!grid_fits(blocks, small ? 256 : 512)) return MOGA_ERR_UNSUPPORTED;
    int32_t* ts = c.G <= MOGA_MAX_GROUPS ? nullptr : (int32_t*)c.ws;
    a.c[i] = {(const unsigned short*)c.qh, (const unsigned short*)c.kh, (const unsigned short*)c.vh, c.cu_seqlens_q, c.cu_seqlens_k, ts, c.Nq,
              c.Nk, (unsigned short*)c.oh, c.lse, c.G};
  }
  for (int i = 0; i < n; ++i)
    if (a.c[i].tile_start) tile_start_kernel<<<1, 1024, 0, st>>>(a.c[i].cu_q, a.c[i].M, rows, (int32_t*)calls[which[i]].ws);
  if (small) attn_fwd_bf16_small_calls_kernel<<<(unsigned)blocks, 256, 0, st>>>(a, H, softmax_scale);
  else if (rows == 384) attn_fwd_bf16_pipe_calls_kernel<384><<<(unsigned)blocks, 512, 0, st>>>(a, H, softmax_scale);
  else attn_fwd_bf16_pipe_calls_kernel<256><<<(unsigned)blocks, 512, 0, st>>>(a, H, softmax_scale);
  return launch_status();
}

extern "C" int moga_varlen_attn_fwd_calls(const moga_attn_fwd_call* calls, int n, int dtype, int H, int D, float softmax_scale,
                                          void* stream) {
  if (!calls || n < 1 || n > MOGA_MAX_CALLS) return MOGA_ERR_INVALID_ARG;
  int order[kMaxCalls], count = 0;
  for (int i = 0; i < n; ++i) {
    const int bad = check_varlen_fwd(calls[i], dtype, H, D, softmax_scale);
    if (bad) return bad;
    if (calls[i].Nq > 0) order[count++] = i;
  }
  auto one_by_one = [&](const int* first, const int* last) {
    int rc = MOGA_OK;
    for (; first != last && rc == MOGA_OK; ++first) {
      const moga_attn_fwd_call& c = calls[*first];
      rc = moga_varlen_attn_fwd(c.qh, c.kh, c.vh, dtype, c.Nq, c.Nk, H, D, c.cu_seqlens_q, c.cu_seqlens_k, c.G, softmax_scale, c.oh, c.lse,
                                c.ws, c.ws_bytes, stream);
    }
    return rc;
  };
  if (dtype != MOGA_BF16 || count < 2) return one_by_one(order, order + count);
  int* const first = std::stable_partition(order, order + count, [&](int i) {
    const moga_attn_fwd_call& c = calls[i];
    return fwd_call_alone(c.Nq, H, c.G) && split_room(c.ws, moga_varlen_attn_fwd_ws_bytes(c.G), c.ws_bytes).rows > 0;
  });
  const int alone = one_by_one(order, first);
  if (alone != MOGA_OK || order + count - first < 2) return alone != MOGA_OK ? alone : one_by_one(first, order + count);
  int64_t rows = 0, shortest = INT64_MAX;
  for (const int* i = first; i != order + count; ++i) {
    rows += calls[*i].Nq;
    shortest = std::min(shortest, calls[*i].Nq / calls[*i].G);
  }
  // longest blocks first, the calls of the large kernels before those of the small ones
  std::stable_sort(first, order + count, [&](int a, int b) { return calls[a].Nk * calls[b].G > calls[b].Nk * calls[a].G; });
  auto small = [&](int i) { return use_small_group_kernels(calls[i].Nq, calls[i].G, fwd_calls_small_rows(rows, H, shortest)); };
  int* const mid = std::stable_partition(first, order + count, [&](int i) { return !small(i); });
  const int large = (int)(mid - first);
  auto launch = [&](const int* from, const int* last, bool few, int block) {
    if (from == last) return (int)MOGA_OK;
    const int rc = launch_fwd_calls(calls, from, (int)(last - from), few, block, H, softmax_scale, (hipStream_t)stream);
    return rc == MOGA_ERR_UNSUPPORTED ? one_by_one(from, last) : rc;   // millions of groups: together too many threads for a grid
  };
  SideShape q[kMaxCalls];
  for (int i = 0; i < large; ++i) q[i] = {calls[first[i]].Nq, calls[first[i]].Nk, calls[first[i]].G};
  const int bm = calls_cost(q, large, H, 256, 256, 10) < calls_cost(q, large, H, 384, 256, 13) ? 256 : 384;
  const int rc = launch(first, mid, false, bm);
  return rc != MOGA_OK ? rc : launch(mid, order + count, true, 128);
}
