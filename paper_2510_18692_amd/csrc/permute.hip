// permute / repermute of MoGA (Alg. 1 steps 2 and 4) and their backward.
//
// Integer part: a stable counting sort of tokens by group id, without atomics deciding any
// order.  Tokens are cut into chunks, one wave per chunk:
//   1. chunk_hist  : per-chunk histogram by wave ballots, accumulated in LDS owned by the wave;
//   2. chunk_scan  : one block; per group a wave scan over the chunks gives every chunk its
//                    first slot for that group; also counts, cu_seqlens, max_seqlen;
//   3. chunk_rank  : each wave walks its chunk in token order; a token's slot is its chunk's
//                    running base for the group plus its rank among equal ids in the batch.
// Up to 16,384 tokens and 32 groups one block does all three (permute_single_block), and with rows to move, where that pays,
// every block of the gather for itself (permute_gather).
// Data part: 16-byte-per-lane row copies between token order [N, H, D] and head-major
// group-contiguous order [H, N, D]; the scatter back multiplies by the gate (Eq. 5).
#include <mutex>
#include <type_traits>

#include "moga_common.h"

namespace moga {

// Lanes of this wave (among `valid` ones) that hold the same group id as the caller.
__device__ __forceinline__ unsigned long long match_group(int g, bool valid, int nbits) {
  const unsigned long long v = __ballot(valid);
  unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
  for (int b = 0; b < nbits; ++b) {
    const int bit = __builtin_amdgcn_sbfe(g, b, 1);   // 0 or -1
    const unsigned long long bal = __ballot(bit != 0);
    lo &= ~((unsigned)bal ^ (unsigned)bit);
    hi &= ~((unsigned)(bal >> 32) ^ (unsigned)bit);
  }
  return lo | ((unsigned long long)hi << 32);
}

__device__ __forceinline__ int clamp_group(int g, int M) { return g < 0 ? 0 : (g >= M ? M - 1 : g); }

// Group ids of eight consecutive 64-token batches starting at tb, -1 past `end`: all loads in flight
// together.
constexpr int kBatches = 8;
__device__ __forceinline__ void load_groups(int (&g)[kBatches], const int32_t* __restrict__ group, int64_t tb, int64_t end,
                                            int M) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int b = 0; b < kBatches; ++b) {
    const int64_t tok = tb + 64 * b + lane;
    g[b] = tok < end ? clamp_group(group[tok], M) : -1;
  }
}

// hist is [M][num_chunks], so that the scan below reads it in rows.
__global__ __launch_bounds__(256) void chunk_hist_kernel(const int32_t* __restrict__ group,
                                                         int64_t N, int M, int nbits,
                                                         int chunk_len, int num_chunks,
                                                         int32_t* __restrict__ hist) {
  __shared__ int s_hist[4][MOGA_MAX_GROUPS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int chunk = blockIdx.x * 4 + wave;
  if (chunk >= num_chunks) return;  // no block-wide barrier below
  volatile int* my = s_hist[wave];
  for (int j = lane; j < M; j += 64) my[j] = 0;
  const int64_t t0 = (int64_t)chunk * chunk_len;
  const int64_t t1 = min(N, t0 + chunk_len);
  for (int64_t tb = t0; tb < t1; tb += 64 * kBatches) {
    int g[kBatches];
    load_groups(g, group, tb, t1, M);
#pragma unroll
    for (int b = 0; b < kBatches; ++b) {
      const unsigned long long mask = match_group(g[b], g[b] >= 0, nbits);
      const unsigned long long below = mask & ((1ull << lane) - 1ull);
      if (g[b] >= 0 && below == 0) my[g[b]] += __popcll(mask);  // one leader per distinct id
    }
  }
  for (int j = lane; j < M; j += 64) hist[(int64_t)j * num_chunks + chunk] = my[j];
}

// counts, exclusive prefix sum and largest count of the groups: wave 0 of a block, from s_count.
__device__ __forceinline__ void scan_groups(const int* s_count, int* s_cu, int M, int32_t* __restrict__ counts,
                                            int32_t* __restrict__ cu_seqlens, int32_t* __restrict__ max_seqlen) {
  const int lane = threadIdx.x & 63;
  int running = 0, mx = 0;
  for (int g0 = 0; g0 < M; g0 += 64) {
    const int g = g0 + lane;
    const int v = g < M ? s_count[g] : 0;
    const int incl = running + wave_scan_add(v);
    if (g < M) {
      s_cu[g] = incl - v;
      cu_seqlens[g] = incl - v;
      counts[g] = v;
    }
    running = __builtin_amdgcn_readlane(incl, 63);
    mx = max(mx, v);
  }
  mx = wave_max_i(mx);
  if (lane == 0) {
    cu_seqlens[M] = running;
    max_seqlen[0] = mx;
  }
}

// One block of 1024 threads.  hist [M][num_chunks] is overwritten with each chunk's first slot for the group.
__global__ __launch_bounds__(1024) void chunk_scan_kernel(int32_t* __restrict__ hist,
                                                          int num_chunks, int M, int64_t N,
                                                          int32_t* __restrict__ counts,
                                                          int32_t* __restrict__ cu_seqlens,
                                                          int32_t* __restrict__ max_seqlen) {
  __shared__ int s_count[MOGA_MAX_GROUPS];
  __shared__ int s_cu[MOGA_MAX_GROUPS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int g = wave; g < M; g += 16) {
    const int32_t* row = hist + (int64_t)g * num_chunks;
    int tot = 0;
#pragma unroll 8
    for (int c = lane; c < num_chunks; c += 64) tot += row[c];
    tot = wave_sum_i(tot);
    if (lane == 0) s_count[g] = tot;
  }
  __syncthreads();
  if (wave == 0) scan_groups(s_count, s_cu, M, counts, cu_seqlens, max_seqlen);
  __syncthreads();
  for (int g = wave; g < M; g += 16) {
    int32_t* row = hist + (int64_t)g * num_chunks;
    int running = s_cu[g];
    for (int c0 = 0; c0 < num_chunks; c0 += 64 * 8) {
      int v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = c0 + 64 * i + lane;
        v[i] = c < num_chunks ? row[c] : 0;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = c0 + 64 * i + lane;
        const int incl = running + wave_scan_add(v[i]);
        if (c < num_chunks) row[c] = incl - v[i];
        running = __builtin_amdgcn_readlane(incl, 63);
      }
    }
  }
}

__global__ __launch_bounds__(256) void chunk_rank_kernel(const int32_t* __restrict__ group,
                                                         int64_t N, int M, int nbits,
                                                         int chunk_len, int num_chunks,
                                                         const int32_t* __restrict__ base,
                                                         int32_t* __restrict__ perm,
                                                         int32_t* __restrict__ inv_perm) {
  __shared__ int s_next[4][MOGA_MAX_GROUPS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int chunk = blockIdx.x * 4 + wave;
  if (chunk >= num_chunks) return;  // no block-wide barrier below
  volatile int* next = s_next[wave];
  for (int j = lane; j < M; j += 64) next[j] = base[(int64_t)j * num_chunks + chunk];
  const int64_t t0 = (int64_t)chunk * chunk_len;
  const int64_t t1 = min(N, t0 + chunk_len);
  for (int64_t tb = t0; tb < t1; tb += 64 * kBatches) {
    int g[kBatches];
    load_groups(g, group, tb, t1, M);
#pragma unroll
    for (int b = 0; b < kBatches; ++b) {
      const bool valid = g[b] >= 0;
      const unsigned long long mask = match_group(g[b], valid, nbits);
      const int rank = __popcll(mask & ((1ull << lane) - 1ull));
      int slot = 0;
      if (valid) slot = next[g[b]] + rank;
      __builtin_amdgcn_wave_barrier();
      if (valid) {
        const int64_t tok = tb + 64 * b + lane;
        perm[slot] = (int32_t)tok;
        inv_perm[tok] = slot;
        if (rank == 0) next[g[b]] += __popcll(mask);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// The whole counting sort in one block, for up to 16,384 tokens and 32 groups, where three launches cost
// more than the work.  A thread takes PER consecutive tokens and counts them in counters of its own
// (16 bits, [group][thread] in LDS: no conflict and no ballots), which also gives each token its rank among
// the thread's; a wave then scans a group's 1,024 counters, 16 per lane.  Ids come in and both lists leave
// through LDS, so that every access to memory is coalesced: one CU takes a cycle per cache line, and with
// scattered stores 10,007 tokens took 14 us.
// 4.4 us up to 4,096 and 9.8 us at 10,007 tokens, against 16.5 us for the three kernels.
constexpr int64_t kSingleBlockTokens = 16384;
constexpr int kSingleBlockGroups = 32;

template <int PER>
__global__ __launch_bounds__(1024) void permute_single_block_kernel(const int32_t* __restrict__ group, int N, int M,
                                                                    int32_t* __restrict__ counts,
                                                                    int32_t* __restrict__ cu_seqlens,
                                                                    int32_t* __restrict__ max_seqlen,
                                                                    int32_t* __restrict__ perm,
                                                                    int32_t* __restrict__ inv_perm) {
  constexpr int CAP = 1024 * PER, W = PER / 4;
  typedef unsigned __attribute__((may_alias)) word_t;   // four ids, or two counters, at once
  __shared__ __attribute__((aligned(16))) unsigned short s_cnt[kSingleBlockGroups][1024];
  __shared__ __attribute__((aligned(16))) unsigned char s_id[CAP];
  __shared__ unsigned short s_perm[CAP], s_inv[CAP];
  __shared__ int s_count[kSingleBlockGroups];
  __shared__ int s_cu[kSingleBlockGroups];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int t = 1024 * i + tid;
    s_id[t] = (unsigned char)(t < N ? clamp_group(group[t], M) : 255);
  }
  for (int j = 0; j < M; ++j) s_cnt[j][tid] = 0;
  __syncthreads();
  unsigned id[W];
#pragma unroll
  for (int w = 0; w < W; ++w) id[w] = ((const word_t*)s_id)[tid * W + w];
  int pos[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const unsigned g = (id[i >> 2] >> (8 * (i & 3))) & 255u;
    if (g != 255u) {
      pos[i] = s_cnt[g][tid];
      s_cnt[g][tid] = (unsigned short)(pos[i] + 1);
    }
  }
  __syncthreads();
  for (int j = wave; j < M; j += 16) {   // counters of group j -> exclusive sums over the threads
    word_t* p = (word_t*)&s_cnt[j][16 * lane];
    unsigned c[8];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      c[i] = p[i];
      sum += (c[i] & 0xffff) + (c[i] >> 16);
    }
    const int incl = wave_scan_add(sum);
    int run = incl - sum;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int next = run + (c[i] & 0xffff);
      p[i] = (unsigned)run | ((unsigned)next << 16);
      run = next + (c[i] >> 16);
    }
    if (lane == 63) s_count[j] = incl;
  }
  __syncthreads();
  if (wave == 0) scan_groups(s_count, s_cu, M, counts, cu_seqlens, max_seqlen);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const unsigned g = (id[i >> 2] >> (8 * (i & 3))) & 255u;
    if (g != 255u) {
      const int slot = s_cu[g] + s_cnt[g][tid] + pos[i];
      s_perm[slot] = (unsigned short)(tid * PER + i);
      s_inv[tid * PER + i] = (unsigned short)slot;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int t = 1024 * i + tid;
    if (t < N) {
      perm[t] = s_perm[t];
      inv_perm[t] = s_inv[t];
    }
  }
}

// ---------------------------------------------------------------------------------------
// row movers.  A (token, head) row is D*elem bytes = LPR lanes of 16 bytes.
// ---------------------------------------------------------------------------------------
// A block of four waves takes SLOTS tokens or slots and all heads, a wave every fourth head; a wave has 16 rows of a tensor in flight, of one
// head (SLOTS = 16) or of four (4).  Four slots: four times the blocks, which few tokens need, and writes that are as good (1 KB to a place).
// us with 16 and 4: gather for three branches 3,120 x 16 heads 38.3 and 34.0, 99,840 x 40 2,423 and 2,390; its backward 40.1 and 34.4, 2,417
// and 2,379; mean of three branches 15.7 and 10.9, 800 and 776; gather 62,400 x 12 205 and 202; scatter 1,253 x 40 12.8 and 8.4, 60,000 x 40 251
// and 243.
constexpr int kManySlots = 16, kFewSlots = 4;
// HIP takes fewer than 2^32 threads in a grid.
inline bool few_slots(int64_t N) { return grid_fits((N + kFewSlots - 1) / kFewSlots, 256); }
// The kernels that also sum over the heads of a token and write its row constants keep more in registers: 3,120 x 16 heads 30.6 and 24.3 us
// (backward of the mean of three branches), 4,680 x 12 29.0 and 28.5, 6,240 x 12 33.0 and 37.9, 32,760 x 12 151 and 161; scatter backward
// 1,253 x 40 18.3 and 10.8, 5,600 x 12 15.4 and 13.6, 8,000 x 12 18.1 and 18.6, 16,000 x 12 28.8 and 31.8.
inline bool few_slots_of_sums(int64_t N) { return N <= 6000; }
constexpr int kGatherSlots = 16;   // tokens per block of permute_gather

struct Rows3 {
  const void* src[3];
  void* dst[3];
};

// token order -> head-major sorted order:  dst[h][j] = src[perm[j]][h]
template <int LPR, int SLOTS>
__global__ __launch_bounds__(256) void gather_rows_kernel(Rows3 p, const int32_t* __restrict__ perm,
                                                          int64_t N, int H) {
  constexpr int RPW = 64 / LPR;  // rows per wave instruction
  constexpr int IT = SLOTS / RPW;
  constexpr int HU = kManySlots / SLOTS;   // heads in flight
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int part = lane % LPR, rsub = lane / LPR;
  const int64_t j0 = (int64_t)blockIdx.x * SLOTS;
  const uintx4_t* __restrict__ src = (const uintx4_t*)p.src[blockIdx.y];
  uintx4_t* __restrict__ dst = (uintx4_t*)p.dst[blockIdx.y];
  int64_t tok[IT];
  bool ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t j = j0 + it * RPW + rsub;
    ok[it] = j < N;
    tok[it] = ok[it] ? perm[j] : 0;
  }
  for (int h0 = wave; h0 < H; h0 += 4 * HU) {
    uintx4_t v[HU][IT];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it)
        if (ok[it] && h0 + 4 * u < H) v[u][it] = src[(tok[it] * H + h0 + 4 * u) * LPR + part];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int64_t j = j0 + it * RPW + rsub;
        if (ok[it] && h0 + 4 * u < H) dst[((int64_t)(h0 + 4 * u) * N + j) * LPR + part] = v[u][it];
      }
  }
}

// Sort and gather in one launch, for up to 16,384 tokens and 32 groups.  A block moves the rows of 16 tokens (of one tensor, or
// of all three) and finds their slots by itself: it counts the ids of all tokens and of those before its own (up to 64 per
// thread, 8-bit counters packed four to a word, summed over the waves) while its first rows are on the way.  The sort as a launch
// of its own is one block that the chip waits for.  Two launches against this one, in us: 4,096 x 12 heads x 128 bf16, 8 groups
// 18.3 and 13.7 (5.5 TB/s); 10,007 x 12, 20 groups 39.3 and 37.8; 16,384 x 12, 8 groups 64 and 54, 32 groups 71 and 59.
// The count is paid back by a token's rows (bytes of one tensor) where the tokens are many, doubles at 8,193 tokens, and has four
// times the counters above 8 groups.  Two launches against one, up to 8 groups: 256-byte rows 7.6 and 6.3 at 4,096 tokens, 10.1 and
// 22.8 at 16,384; 1 KB rows 16.1 and 12.1 at 8,192, 29.3 and 21.5 at 16,384.  20 groups: 256-byte rows 6.8 and 5.7 at 2,048, 7.3 and
// 8.8 at 3,000 (in a graph; call by call, where the host's time counts, 12.4 and 9.9); 1.5 KB 10.7 and 11.0 at 3,500, 14.8 and 15.4 at
// 5,000, 16.9 and 16.2 at 6,000; 1 KB 16.5 and 14.7 at 8,192, 17.3 and 22.2 at 8,193; 2 KB 27.8 and 27.2 at 9,000, 30.2 and 27.7 at
// 10,007; 4 KB, 9 groups 44.0 and 46.9 at 9,300, 65.4 and 62.3 at 12,288.
inline bool use_permute_gather(int64_t N, int M, int64_t row_bytes) {
  if (M <= 8) return N <= 4096 || (N <= 16384 && row_bytes >= 1024);
  if (M > 32 || N > 16384) return false;
  if (N <= 2048) return true;
  if (N <= 4096) return row_bytes >= 1536;
  if (N <= 5600) return row_bytes >= 6144 && N > 4608;
  if (N <= 8192) return row_bytes >= 1024;
  return row_bytes >= 6144 || N > (row_bytes >= 4096 ? 10240 : row_bytes >= 2048 ? 9216 : 16384);
}
// A block per 16 tokens and tensor instead of one for all three: three times the counts, but no second or third round of blocks that
// holds a few long ones.  Two launches, one block for all, one per tensor, 40 heads: 5,000 tokens, 8 groups 59.7, 68.4 and 54.8, 9
// groups 59.6, 71.6 and 56.5; 9,000, 8 groups 121, 123 and 114; 8,192 (two full rounds) 107, 97 and 103.  16 heads, 10,007, 8 groups
// 53.7, 52.3 and 48.0, 9 groups 54.7, 56.1 and 57.5.
inline bool permute_gather_per_tensor(int64_t N, int M, int64_t row_bytes) {
  return N <= 4096 || (row_bytes >= (M <= 8 ? 4096 : 6144) && (N - 1) / kGatherSlots % 256 < 224);
}

template <int LPR, int WORDS, int PER>   // WORDS * 4 >= groups, PER * 256 >= tokens
__global__ __launch_bounds__(256) void permute_gather_kernel(Rows3 p, const int32_t* __restrict__ group, int N, int H, int M, int nbits,
                                                             int32_t* __restrict__ counts, int32_t* __restrict__ cu_seqlens,
                                                             int32_t* __restrict__ max_seqlen, int32_t* __restrict__ perm,
                                                             int32_t* __restrict__ inv_perm) {
  constexpr int RPW = 64 / LPR;  // rows per wave instruction
  constexpr int IT = kGatherSlots / RPW;
  __shared__ int s_sum[4][2][2 * WORDS];   // per wave: all tokens, those before the block's; groups 4 w + f and 4 w + f + 2 at 2 w + f
  __shared__ int s_count[4 * WORDS], s_cu[4 * WORDS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int part = lane % LPR, rsub = lane / LPR;
  const int t0 = blockIdx.x * kGatherSlots;
  constexpr int BATCH = PER < 16 ? PER : 16;
  int id[BATCH], ahead[BATCH];   // a batch of ids in flight together, and the next one
  auto load_ids = [&](int (&to)[BATCH], int i0) {
#pragma unroll
    for (int i = 0; i < BATCH; ++i) to[i] = group[min(256 * (i0 + i) + (int)threadIdx.x, N - 1)];
  };
  load_ids(id, 0);
  const bool own = lane < kGatherSlots && t0 + lane < N;
  const int g = clamp_group(group[min(t0 + (lane & (kGatherSlots - 1)), N - 1)], M);
  uintx4_t v[IT];
  auto load_rows = [&](const uintx4_t* __restrict__ src, int h) {
#pragma unroll
    for (int it = 0; it < IT; ++it) v[it] = src[((int64_t)min(t0 + it * RPW + rsub, N - 1) * H + h) * LPR + part];
  };
  if (wave < H) load_rows((const uintx4_t*)p.src[blockIdx.y], wave);

  unsigned all[WORDS], before[WORDS];
#pragma unroll
  for (int w = 0; w < WORDS; ++w) all[w] = before[w] = 0u;
#pragma unroll 1
  for (int i0 = 0; i0 < PER; i0 += BATCH) {
    if (PER > BATCH) load_ids(ahead, i0 + BATCH);
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int t = 256 * (i0 + i) + threadIdx.x, k = clamp_group(id[i], M);
      const unsigned one = t < N ? 1u << (8 * (k & 3)) : 0u, b = t < t0 ? one : 0u;
#pragma unroll
      for (int w = 0; w < WORDS; ++w) {
        all[w] += (k >> 2) == w ? one : 0u;
        before[w] += (k >> 2) == w ? b : 0u;
      }
    }
    if (PER > BATCH)
#pragma unroll
      for (int i = 0; i < BATCH; ++i) id[i] = ahead[i];
  }
#pragma unroll
  for (int w = 0; w < WORDS; ++w)
#pragma unroll
    for (int f = 0; f < 2; ++f) {   // two 16-bit sums at once: at most 4,096 per wave
      const int x = wave_scan_add((int)((all[w] >> (8 * f)) & 0x00ff00ffu));
      const int y = wave_scan_add((int)((before[w] >> (8 * f)) & 0x00ff00ffu));
      if (lane == 63) { s_sum[wave][0][2 * w + f] = x; s_sum[wave][1][2 * w + f] = y; }
    }
  const int rank = __popcll(match_group(g, own, nbits) & ((1ull << lane) - 1ull));
  __syncthreads();
  int sum[2] = {0, 0};   // of group `lane`; every wave for itself
  if (lane < 4 * WORDS) {
    const int idx = 2 * (lane >> 2) + (lane & 1), shift = 8 * (lane & 2);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int b = 0; b < 2; ++b) sum[b] += (s_sum[k][b][idx] >> shift) & 0xffff;
  }
  const int base = wave_scan_add(sum[0]) - sum[0] + sum[1];
  const int slot = __shfl(base, g, kWave) + rank;   // lane i < 16: of token t0 + i
  if (blockIdx.y == 0 && wave == 0) {
    if (own) { perm[slot] = t0 + lane; inv_perm[t0 + lane] = slot; }
    if (blockIdx.x == 0) {
      if (lane < 4 * WORDS) s_count[lane] = sum[0];
      scan_groups(s_count, s_cu, M, counts, cu_seqlens, max_seqlen);
    }
  }
  int64_t to[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) to[it] = (int64_t)__shfl(slot, it * RPW + rsub, kWave) * LPR + part;
  for (int y = blockIdx.y; y < 3; y += gridDim.y) {
    const uintx4_t* __restrict__ src = (const uintx4_t*)p.src[y];
    uintx4_t* __restrict__ dst = (uintx4_t*)p.dst[y];
    if (y != (int)blockIdx.y && wave < H) load_rows(src, wave);
    for (int h = wave; h < H; h += 4) {
#pragma unroll
      for (int it = 0; it < IT; ++it)
        if (t0 + it * RPW + rsub < N) dst[(int64_t)h * N * LPR + to[it]] = v[it];
      if (h + 4 < H) load_rows(src, h + 4);
    }
  }
}

template <bool BF16>
__device__ __forceinline__ uintx4_t scale16(uintx4_t v, float g) {
  uintx4_t r;
  if (BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      r[i] = pack_bf16x2(bf16_lo_to_f32(v[i]) * g, bf16_hi_to_f32(v[i]) * g);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __float_as_uint(__uint_as_float(v[i]) * g);
  }
  return r;
}

template <bool BF16>
__device__ __forceinline__ float dot16(uintx4_t a, uintx4_t b) {
  float s = 0.f;
  if (BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s = fmaf(bf16_lo_to_f32(a[i]), bf16_lo_to_f32(b[i]), s);
      s = fmaf(bf16_hi_to_f32(a[i]), bf16_hi_to_f32(b[i]), s);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) s = fmaf(__uint_as_float(a[i]), __uint_as_float(b[i]), s);
  }
  return s;
}

// head-major sorted order -> token order: dst[perm[j]][h] = gate[perm[j]] * src[h][j]
template <int LPR, bool BF16, int SLOTS>
__global__ __launch_bounds__(256) void scatter_rows_kernel(Rows3 p, const int32_t* __restrict__ perm,
                                                           const float* __restrict__ gate,
                                                           int64_t N, int H) {
  constexpr int RPW = 64 / LPR;
  constexpr int IT = SLOTS / RPW;
  constexpr int HU = kManySlots / SLOTS;   // heads in flight
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int part = lane % LPR, rsub = lane / LPR;
  const int64_t j0 = (int64_t)blockIdx.x * SLOTS;
  const uintx4_t* __restrict__ src = (const uintx4_t*)p.src[blockIdx.y];
  uintx4_t* __restrict__ dst = (uintx4_t*)p.dst[blockIdx.y];
  int64_t tok[IT];
  float g[IT];
  bool ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t j = j0 + it * RPW + rsub;
    ok[it] = j < N;
    tok[it] = ok[it] ? perm[j] : 0;
    g[it] = (gate && ok[it]) ? gate[tok[it]] : 1.f;
  }
  for (int h0 = wave; h0 < H; h0 += 4 * HU) {
    uintx4_t v[HU][IT];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int64_t j = j0 + it * RPW + rsub;
        if (ok[it] && h0 + 4 * u < H) v[u][it] = src[((int64_t)(h0 + 4 * u) * N + j) * LPR + part];
      }
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it)
        if (ok[it] && h0 + 4 * u < H)
          dst[(tok[it] * H + h0 + 4 * u) * LPR + part] = gate ? scale16<BF16>(v[u][it], g[it]) : v[u][it];
  }
}

// d_oh[h][j] = gate[t] * d_o[t][h],  d_gate[t] = sum_{h,c} d_o[t][h][c] * oh[h][j][c],  t = perm[j]
// DELTA: also the row constants of the attention backward, -delta = -rowsum(d_oh * oh) (of the rounded d_oh) and, in bf16,
// -lse / scale, and its status word.  Both tensors are in registers here; attn_bwd_delta_kernel reads them again (10,007 x 12
// heads: 12 us, 32,760 x 12: 38 us).  Same sums in the same order as there.
template <int LPR, bool BF16, bool DELTA, int SLOTS>
__global__ __launch_bounds__(256) void unpermute_bwd_kernel(
    const uintx4_t* __restrict__ d_o, const uintx4_t* __restrict__ oh,
    const int32_t* __restrict__ perm, const float* __restrict__ gate, int64_t N, int H,
    uintx4_t* __restrict__ d_oh, float* __restrict__ d_gate, RowConstants rc) {
  constexpr int RPW = 64 / LPR;
  constexpr int IT = SLOTS / RPW;
  constexpr int HU = kManySlots / SLOTS;   // heads in flight
  __shared__ float s_part[4][SLOTS];
  if (DELTA && blockIdx.x == 0 && threadIdx.x == 0) *rc.status = 0;   // read by the kernels that follow
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int part = lane % LPR, rsub = lane / LPR;
  const int64_t j0 = (int64_t)blockIdx.x * SLOTS;
  int64_t tok[IT];
  float g[IT], acc[IT];
  bool ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t j = j0 + it * RPW + rsub;
    ok[it] = j < N;
    tok[it] = ok[it] ? perm[j] : 0;
    g[it] = ok[it] ? gate[tok[it]] : 0.f;
    acc[it] = 0.f;
  }
  for (int h0 = wave; h0 < H; h0 += 4 * HU) {
    uintx4_t a[HU][IT], b[HU][IT];
    float l[HU][IT];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        const int64_t j = j0 + it * RPW + rsub;
        if (ok[it] && h < H) {
          a[u][it] = d_o[(tok[it] * H + h) * LPR + part];
          b[u][it] = oh[((int64_t)h * N + j) * LPR + part];
          if (DELTA && BF16) l[u][it] = rc.lse[(int64_t)h * N + j];
        }
      }
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        const int64_t j = j0 + it * RPW + rsub;
        if (ok[it] && h < H) {   // the same for all lanes of a row
          acc[it] += dot16<BF16>(a[u][it], b[u][it]);
          const uintx4_t s = scale16<BF16>(a[u][it], g[it]);
          d_oh[((int64_t)h * N + j) * LPR + part] = s;
          if (DELTA) {
            float dl = dot16<BF16>(s, b[u][it]);
            dl = lanes_sum<LPR>(dl);
            if (part == 0) {
              rc.neg_delta[(int64_t)h * N + j] = -dl;
              if (BF16) rc.neg_lse_over_scale[(int64_t)h * N + j] = -l[u][it] * rc.inv_scale;
            }
          }
        }
      }
  }
  // reduce over the LPR lanes of a row, then over the four waves
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const float s = lanes_sum<LPR>(acc[it]);
    if (part == 0) s_part[wave][it * RPW + rsub] = s;
  }
  __syncthreads();
  if (threadIdx.x < SLOTS) {
    const int64_t j = j0 + threadIdx.x;
    if (j < N) {
      const float s = (s_part[0][threadIdx.x] + s_part[1][threadIdx.x]) +
                      (s_part[2][threadIdx.x] + s_part[3][threadIdx.x]);
      d_gate[perm[j]] = s;
    }
  }
}

// ---------------------------------------------------------------------------------------
// Static branches (Section 3.2): gradient of a gather whose index lists a token several times,
// and the mean of the dynamic branch and two static branches fused into one scatter.
// ---------------------------------------------------------------------------------------
template <bool BF16>
__device__ __forceinline__ void add16(float (&acc)[8], uintx4_t v) {
  if (BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { acc[2 * i] += bf16_lo_to_f32(v[i]); acc[2 * i + 1] += bf16_hi_to_f32(v[i]); }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] += __uint_as_float(v[i]);
  }
}

template <bool BF16>
__device__ __forceinline__ uintx4_t pack16(const float (&acc)[8]) {
  uintx4_t r;
  if (BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = pack_bf16x2(acc[2 * i], acc[2 * i + 1]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __float_as_uint(acc[i]);
  }
  return r;
}

// d_src[t][h] (+)= sum over the slots j that list token t (inv_slots[inv_cu[t] .. inv_cu[t+1]),
// ascending) of d_dst[h][j]; fp32 sums in a fixed order.
template <int LPR, bool BF16>
__global__ __launch_bounds__(256) void gather_rows_bwd_kernel(
    const uintx4_t* __restrict__ d_dst, const int32_t* __restrict__ inv_cu,
    const int32_t* __restrict__ inv_slots, int64_t N, int64_t Nk, int H, int accumulate,
    uintx4_t* __restrict__ d_src) {
  constexpr int RPW = 64 / LPR;
  constexpr int IT = kManySlots / RPW;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int part = lane % LPR, rsub = lane / LPR;
  const int64_t t0 = (int64_t)blockIdx.x * kManySlots;
  for (int it = 0; it < IT; ++it) {
    const int64_t t = t0 + it * RPW + rsub;
    if (t >= N) continue;
    const int beg = inv_cu[t], end = inv_cu[t + 1];
    for (int h = wave; h < H; h += 4) {
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      uintx4_t* dp = d_src + (t * H + h) * LPR + part;
      if (accumulate) add16<BF16>(acc, *dp);
      for (int j = beg; j < end; ++j)
        add16<BF16>(acc, d_dst[((int64_t)h * Nk + inv_slots[j]) * LPR + part]);
      *dp = pack16<BF16>(acc);
    }
  }
}

// Q, K and V rows to all three branches (Section 3.2): the dynamic groups' slot, the slots of the static lists, the frame order.
// Every row is read once; as separate gathers it was read three times (32,760 x 12 heads: 324 us for the seven launches).
struct Gather3 {
  const uintx4_t* src[3];
  uintx4_t *m[3], *s[3], *f[3];
  const int32_t *inv_cu[3], *slots[3];   // slots of token t in the static list: slots[inv_cu[t] .. inv_cu[t + 1]); inv_cu NULL: slots[t]
  int64_t rows[3];                       // of the static list
};

template <int LPR, int SLOTS>
__global__ __launch_bounds__(256) void gather3_kernel(Gather3 p, const int32_t* __restrict__ inv_m, const int32_t* __restrict__ inv_f,
                                                      int64_t N, int H) {
  constexpr int RPW = 64 / LPR;
  constexpr int IT = SLOTS / RPW;
  constexpr int HU = kManySlots / SLOTS;   // heads in flight
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, y = blockIdx.y;
  const int part = lane % LPR, rsub = lane / LPR;
  const int64_t t0 = (int64_t)blockIdx.x * SLOTS;
  const uintx4_t* __restrict__ src = p.src[y];
  const int32_t* __restrict__ slots = p.slots[y];
  const int32_t* __restrict__ inv_cu = p.inv_cu[y];
  int64_t jm[IT], jf[IT], tok[IT];
  int beg[IT], end[IT], first[IT];
  bool ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t t = t0 + it * RPW + rsub;
    ok[it] = t < N;
    tok[it] = ok[it] ? t : N - 1;
    jm[it] = inv_m[tok[it]];
    jf[it] = inv_f ? inv_f[tok[it]] : tok[it];
    beg[it] = inv_cu ? inv_cu[tok[it]] : (int)tok[it];
    end[it] = inv_cu ? inv_cu[tok[it] + 1] : (int)tok[it] + 1;
    first[it] = beg[it] < end[it] ? slots[beg[it]] : -1;
  }
  for (int h0 = wave; h0 < H; h0 += 4 * HU) {
    uintx4_t v[HU][IT];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) v[u][it] = src[(tok[it] * H + min(h0 + 4 * u, H - 1)) * LPR + part];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        if (ok[it] && h < H) {
          p.m[y][((int64_t)h * N + jm[it]) * LPR + part] = v[u][it];
          p.f[y][((int64_t)h * N + jf[it]) * LPR + part] = v[u][it];
          if (first[it] >= 0) p.s[y][((int64_t)h * p.rows[y] + first[it]) * LPR + part] = v[u][it];
          for (int j = beg[it] + 1; j < end[it]; ++j) p.s[y][((int64_t)h * p.rows[y] + slots[j]) * LPR + part] = v[u][it];
        }
      }
  }
}

// Gradient of a token-order tensor that fed all three branches (Q, K or V of Section 3.2's block):
//   d_src[t][h] = g_m[h][inv_m[t]] + sum over the slots j of t of g_s[h][j] + g_f[h][inv_f[t]]
// (inv_f NULL = identity).  One fp32 sum per element in this fixed order, rounded once: a single
// pass instead of a scatter followed by two accumulating gather-backwards.
// The slots of a token do not depend on the head: the first two (keys of a boundary frame are listed twice) are read once, and their
// rows are in flight with the others.
struct Gather3Bwd {
  const uintx4_t *g_m[3], *g_s[3], *g_f[3];
  const int32_t *inv_cu[3], *slots[3];   // as in Gather3
  int64_t rows[3];
  uintx4_t* d_src[3];
};
template <int LPR, bool BF16, int SLOTS>
__global__ __launch_bounds__(256) void gather3_bwd_kernel(Gather3Bwd p, const int32_t* __restrict__ inv_m, const int32_t* __restrict__ inv_f,
                                                          int64_t N, int H) {
  constexpr int RPW = 64 / LPR;
  constexpr int IT = SLOTS / RPW;
  constexpr int HU = kManySlots / SLOTS;   // heads in flight
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, y = blockIdx.y;
  const int part = lane % LPR, rsub = lane / LPR;
  const int64_t t0 = (int64_t)blockIdx.x * SLOTS;
  const uintx4_t* __restrict__ g_m = p.g_m[y];
  const uintx4_t* __restrict__ g_s = p.g_s[y];
  const uintx4_t* __restrict__ g_f = p.g_f[y];
  const int32_t* __restrict__ slots = p.slots[y];
  const int32_t* __restrict__ inv_cu = p.inv_cu[y];
  uintx4_t* __restrict__ d_src = p.d_src[y];
  const int64_t Nk = p.rows[y];
  int64_t jm[IT], jf[IT];
  int beg[IT], end[IT], js[IT][2];
  bool ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t t = t0 + it * RPW + rsub;
    ok[it] = t < N;
    jm[it] = ok[it] ? inv_m[t] : 0;
    jf[it] = ok[it] ? (inv_f ? inv_f[t] : t) : 0;
    beg[it] = ok[it] ? (inv_cu ? inv_cu[t] : (int)t) : 0;
    end[it] = ok[it] ? (inv_cu ? inv_cu[t + 1] : (int)t + 1) : 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) js[it][i] = beg[it] + i < end[it] ? slots[beg[it] + i] : -1;
  }
  for (int h0 = wave; h0 < H; h0 += 4 * HU) {
    uintx4_t vm[HU][IT], vf[HU][IT], vs[HU][IT][2];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        if (ok[it] && h < H) {
          vm[u][it] = g_m[((int64_t)h * N + jm[it]) * LPR + part];
          vf[u][it] = g_f[((int64_t)h * N + jf[it]) * LPR + part];
#pragma unroll
          for (int i = 0; i < 2; ++i)
            if (js[it][i] >= 0) vs[u][it][i] = g_s[((int64_t)h * Nk + js[it][i]) * LPR + part];
        }
      }
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        if (ok[it] && h < H) {
          const int64_t t = t0 + it * RPW + rsub;
          float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          add16<BF16>(acc, vm[u][it]);
#pragma unroll
          for (int i = 0; i < 2; ++i)
            if (js[it][i] >= 0) add16<BF16>(acc, vs[u][it][i]);
          for (int j = beg[it] + 2; j < end[it]; ++j) add16<BF16>(acc, g_s[((int64_t)h * Nk + slots[j]) * LPR + part]);
          add16<BF16>(acc, vf[u][it]);
          d_src[(t * H + h) * LPR + part] = pack16<BF16>(acc);
        }
      }
  }
}

// o[t][h] = alpha * (gate[t] * a_m[h][inv_m[t]] + a_s[h][inv_s[t]] + a_f[h][inv_f[t]]); a NULL
// inverse list means the identity (the branch keeps token order).
template <int LPR, bool BF16, int SLOTS>
__global__ __launch_bounds__(256) void merge3_fwd_kernel(
    const uintx4_t* __restrict__ a_m, const uintx4_t* __restrict__ a_s, const uintx4_t* __restrict__ a_f,
    const int32_t* __restrict__ inv_m, const int32_t* __restrict__ inv_s, const int32_t* __restrict__ inv_f,
    const float* __restrict__ gate, float alpha, int64_t N, int H, uintx4_t* __restrict__ o) {
  constexpr int RPW = 64 / LPR;
  constexpr int IT = SLOTS / RPW;
  constexpr int HU = kManySlots / SLOTS;   // heads in flight
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int part = lane % LPR, rsub = lane / LPR;
  const int64_t t0 = (int64_t)blockIdx.x * SLOTS;
  int64_t jm[IT], js[IT], jf[IT];
  float g[IT];
  bool ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t t = t0 + it * RPW + rsub;
    ok[it] = t < N;
    jm[it] = ok[it] ? (inv_m ? inv_m[t] : t) : 0;
    js[it] = ok[it] ? (inv_s ? inv_s[t] : t) : 0;
    jf[it] = ok[it] ? (inv_f ? inv_f[t] : t) : 0;
    g[it] = ok[it] ? gate[t] : 0.f;
  }
  for (int h0 = wave; h0 < H; h0 += 4 * HU) {
    uintx4_t vm[HU][IT], vs[HU][IT], vf[HU][IT];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        if (ok[it] && h < H) {
          vm[u][it] = a_m[((int64_t)h * N + jm[it]) * LPR + part];
          vs[u][it] = a_s[((int64_t)h * N + js[it]) * LPR + part];
          vf[u][it] = a_f[((int64_t)h * N + jf[it]) * LPR + part];
        }
      }
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        if (ok[it] && h < H) {
          float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          add16<BF16>(acc, vm[u][it]);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] *= g[it];
          add16<BF16>(acc, vs[u][it]);
          add16<BF16>(acc, vf[u][it]);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] *= alpha;
          const int64_t t = t0 + it * RPW + rsub;
          o[(t * H + h) * LPR + part] = pack16<BF16>(acc);
        }
      }
  }
}

// Backward of merge3_fwd: d_m[h][inv_m[t]] = alpha * gate[t] * d_o[t][h], d_s / d_f = alpha * d_o[t][h],
// d_gate[t] = alpha * sum_{h,c} d_o[t][h][c] * a_m[h][inv_m[t]][c].
// ROWS: also the row constants of the three attention backwards (see unpermute_bwd_kernel), for which the outputs of the static
// branches are read here: two passes instead of the six of three attn_bwd_delta_kernel.  At 62,400 x 12 heads this launch takes 293
// us instead of 199 (4.6 TB/s) and each of the three backward calls 69 less; 4,096 x 4: 9.2 instead of 7.0, and 3 less.
struct Merge3Rows {
  const uintx4_t *a_s, *a_f;
  RowConstants m, s, f;
};
template <bool BF16, int LPR>
__device__ __forceinline__ void put_row_constants(const RowConstants& rc, int64_t row, uintx4_t d, uintx4_t a, float lse, int part) {
  const float dl = lanes_sum<LPR>(dot16<BF16>(d, a));
  if (part == 0) {
    rc.neg_delta[row] = -dl;
    if (BF16) rc.neg_lse_over_scale[row] = -lse * rc.inv_scale;
  }
}

template <int LPR, bool BF16, bool ROWS, int SLOTS>
__global__ __launch_bounds__(256) void merge3_bwd_kernel(
    const uintx4_t* __restrict__ d_o, const uintx4_t* __restrict__ a_m,
    const int32_t* __restrict__ inv_m, const int32_t* __restrict__ inv_s, const int32_t* __restrict__ inv_f,
    const float* __restrict__ gate, float alpha, int64_t N, int H, uintx4_t* __restrict__ d_m,
    uintx4_t* __restrict__ d_s, uintx4_t* __restrict__ d_f, float* __restrict__ d_gate, Merge3Rows rows) {
  constexpr int RPW = 64 / LPR;
  constexpr int IT = SLOTS / RPW;
  constexpr int HU = kManySlots / SLOTS;   // heads in flight
  __shared__ float s_part[4][SLOTS];
  if (ROWS && blockIdx.x == 0 && threadIdx.x == 0) *rows.m.status = *rows.s.status = *rows.f.status = 0;   // read by the kernels that follow
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int part = lane % LPR, rsub = lane / LPR;
  const int64_t t0 = (int64_t)blockIdx.x * SLOTS;
  int64_t jm[IT], js[IT], jf[IT];
  float g[IT], acc[IT];
  bool ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int64_t t = t0 + it * RPW + rsub;
    ok[it] = t < N;
    jm[it] = ok[it] ? (inv_m ? inv_m[t] : t) : 0;
    js[it] = ok[it] ? (inv_s ? inv_s[t] : t) : 0;
    jf[it] = ok[it] ? (inv_f ? inv_f[t] : t) : 0;
    g[it] = ok[it] ? gate[t] * alpha : 0.f;
    acc[it] = 0.f;
  }
  for (int h0 = wave; h0 < H; h0 += 4 * HU) {
    uintx4_t a[HU][IT], b[HU][IT], as[HU][IT], af[HU][IT];
    float l[HU][IT][3];
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        if (ok[it] && h < H) {
          const int64_t t = t0 + it * RPW + rsub;
          a[u][it] = d_o[(t * H + h) * LPR + part];
          b[u][it] = a_m[((int64_t)h * N + jm[it]) * LPR + part];
          if (ROWS) {
            as[u][it] = rows.a_s[((int64_t)h * N + js[it]) * LPR + part];
            af[u][it] = rows.a_f[((int64_t)h * N + jf[it]) * LPR + part];
            if (BF16) {
              l[u][it][0] = rows.m.lse[(int64_t)h * N + jm[it]];
              l[u][it][1] = rows.s.lse[(int64_t)h * N + js[it]];
              l[u][it][2] = rows.f.lse[(int64_t)h * N + jf[it]];
            }
          }
        }
      }
#pragma unroll
    for (int u = 0; u < HU; ++u)
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int h = h0 + 4 * u;
        if (ok[it] && h < H) {
          acc[it] += dot16<BF16>(a[u][it], b[u][it]);
          const uintx4_t sm = scale16<BF16>(a[u][it], g[it]);
          d_m[((int64_t)h * N + jm[it]) * LPR + part] = sm;
          const uintx4_t sc = scale16<BF16>(a[u][it], alpha);
          d_s[((int64_t)h * N + js[it]) * LPR + part] = sc;
          d_f[((int64_t)h * N + jf[it]) * LPR + part] = sc;
          if (ROWS) {
            put_row_constants<BF16, LPR>(rows.m, (int64_t)h * N + jm[it], sm, b[u][it], l[u][it][0], part);
            put_row_constants<BF16, LPR>(rows.s, (int64_t)h * N + js[it], sc, as[u][it], l[u][it][1], part);
            put_row_constants<BF16, LPR>(rows.f, (int64_t)h * N + jf[it], sc, af[u][it], l[u][it][2], part);
          }
        }
      }
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const float s = lanes_sum<LPR>(acc[it]);
    if (part == 0) s_part[wave][it * RPW + rsub] = s;
  }
  __syncthreads();
  if (threadIdx.x < SLOTS) {
    const int64_t t = t0 + threadIdx.x;
    if (t < N)
      d_gate[t] = alpha * ((s_part[0][threadIdx.x] + s_part[1][threadIdx.x]) +
                           (s_part[2][threadIdx.x] + s_part[3][threadIdx.x]));
  }
}

static int bits_for(int M) {
  int b = 0;
  while ((1 << b) < M) ++b;
  return b;
}

// Runs f(std::integral_constant<int, SLOTS>, blocks).
template <typename F>
static void with_slots(bool few, int64_t N, F&& f) {
  if (few) f(std::integral_constant<int, kFewSlots>(), (unsigned)((N + kFewSlots - 1) / kFewSlots));
  else f(std::integral_constant<int, kManySlots>(), (unsigned)((N + kManySlots - 1) / kManySlots));
}

template <int LPR>
static void launch_gather(const Rows3& p, int ntensors, const int32_t* perm, int64_t N, int H,
                          hipStream_t st) {
  with_slots(few_slots(N), N, [&](auto slots, unsigned blocks) {
    gather_rows_kernel<LPR, slots.value><<<dim3(blocks, ntensors), 256, 0, st>>>(p, perm, N, H);
  });
}

template <int LPR, bool BF16>
static void launch_scatter(const Rows3& p, int ntensors, const int32_t* perm, const float* gate,
                           int64_t N, int H, hipStream_t st) {
  with_slots(few_slots(N), N, [&](auto slots, unsigned blocks) {
    scatter_rows_kernel<LPR, BF16, slots.value><<<dim3(blocks, ntensors), 256, 0, st>>>(p, perm, gate, N, H);
  });
}

// Returns lanes per (token, head) row, or 0 when the combination is not covered.
static int lanes_per_row(int dtype, int D) {
  if (dtype == MOGA_F32 && (D == 64 || D == 128)) return D / 4;
  if (dtype == MOGA_BF16 && D == 128) return 16;
  return 0;
}

static int check_rows_args(int dtype, int64_t N, int H, int D) {
  if (N < 0 || H < 1 || D < 1) return MOGA_ERR_INVALID_ARG;
  if (dtype != MOGA_F32 && dtype != MOGA_BF16) return MOGA_ERR_UNSUPPORTED;
  if (!grid_fits((N + kManySlots - 1) / kManySlots, 256) || lanes_per_row(dtype, D) == 0) return MOGA_ERR_UNSUPPORTED;
  return MOGA_OK;
}

}  // namespace moga

using namespace moga;

extern "C" size_t moga_permute_ws_bytes(int64_t N, int M) {
  return (size_t)perm_num_chunks(N) * (size_t)M * sizeof(int32_t);
}

// Shared body of moga_permute and moga_permute_static: `hist` holds num_chunks * M int32.
static int permute_impl(const int32_t* group, int64_t N, int M, const void* q, const void* k,
                        const void* v, int dtype, int H, int D, int32_t* counts,
                        int32_t* cu_seqlens, int32_t* max_seqlen, int32_t* perm,
                        int32_t* inv_perm, void* qh, void* kh, void* vh, int32_t* hist,
                        hipStream_t st) {
  const bool with_data = q || k || v;
  const int chunk_len = perm_chunk_len(N);
  const int num_chunks = perm_num_chunks(N);
  const int nbits = bits_for(M);
  const int64_t row_bytes = (int64_t)H * lanes_per_row(dtype, D) * 16;
  if (with_data && N > 0 && use_permute_gather(N, M, row_bytes)) {
    const Rows3 p = {{q, k, v}, {qh, kh, vh}};
    const dim3 grid((unsigned)((N + kGatherSlots - 1) / kGatherSlots), permute_gather_per_tensor(N, M, row_bytes) ? 3 : 1);
#define MOGA_PERMUTE_GATHER(LPR, WORDS, PER)                                                                                  \
  permute_gather_kernel<LPR, WORDS, PER><<<grid, 256, 0, st>>>(p, group, (int)N, H, M, nbits, counts, cu_seqlens, max_seqlen, \
                                                               perm, inv_perm)
#define MOGA_PERMUTE_GATHER_N(LPR, WORDS)                         \
  if (N <= 2048) MOGA_PERMUTE_GATHER(LPR, WORDS, 8);              \
  else if (N <= 4096) MOGA_PERMUTE_GATHER(LPR, WORDS, 16);        \
  else if (N <= 8192) MOGA_PERMUTE_GATHER(LPR, WORDS, 32);        \
  else MOGA_PERMUTE_GATHER(LPR, WORDS, 64)
    if (lanes_per_row(dtype, D) == 16) {
      if (M <= 8) { MOGA_PERMUTE_GATHER_N(16, 2); } else { MOGA_PERMUTE_GATHER_N(16, 8); }
    } else {
      if (M <= 8) { MOGA_PERMUTE_GATHER_N(32, 2); } else { MOGA_PERMUTE_GATHER_N(32, 8); }
    }
#undef MOGA_PERMUTE_GATHER_N
#undef MOGA_PERMUTE_GATHER
    return launch_status();
  }
  if (N <= kSingleBlockTokens && M <= kSingleBlockGroups) {
#define MOGA_PERMUTE_ONE(PER) \
  permute_single_block_kernel<PER><<<1, 1024, 0, st>>>(group, (int)N, M, counts, cu_seqlens, max_seqlen, perm, inv_perm)
    if (N <= 4096) MOGA_PERMUTE_ONE(4);
    else if (N <= 8192) MOGA_PERMUTE_ONE(8);
    else MOGA_PERMUTE_ONE(16);
#undef MOGA_PERMUTE_ONE
  } else {
    if (num_chunks > 0)
      chunk_hist_kernel<<<(num_chunks + 3) / 4, 256, 0, st>>>(group, N, M, nbits, chunk_len,
                                                             num_chunks, hist);
    chunk_scan_kernel<<<1, 1024, 0, st>>>(hist, num_chunks, M, N, counts, cu_seqlens, max_seqlen);
    if (num_chunks > 0)
      chunk_rank_kernel<<<(num_chunks + 3) / 4, 256, 0, st>>>(group, N, M, nbits, chunk_len,
                                                             num_chunks, hist, perm, inv_perm);
  }
  if (with_data && N > 0) {
    Rows3 p;
    p.src[0] = q; p.src[1] = k; p.src[2] = v;
    p.dst[0] = qh; p.dst[1] = kh; p.dst[2] = vh;
    switch (lanes_per_row(dtype, D)) {
      case 16: launch_gather<16>(p, 3, perm, N, H, st); break;
      case 32: launch_gather<32>(p, 3, perm, N, H, st); break;
      default: return MOGA_ERR_UNSUPPORTED;
    }
  }
  return launch_status();
}

// Host-side argument checks shared by the two permute entry points.
static int permute_check(const int32_t* group, int64_t N, int M, const void* q, const void* k,
                         const void* v, int dtype, int H, int D, const int32_t* counts,
                         const int32_t* cu_seqlens, const int32_t* max_seqlen,
                         const int32_t* perm, const int32_t* inv_perm, const void* qh,
                         const void* kh, const void* vh) {
  if (N < 0 || M < 1) return MOGA_ERR_INVALID_ARG;
  if (M > MOGA_MAX_GROUPS || N >= ((int64_t)1 << 31)) return MOGA_ERR_UNSUPPORTED;
  const bool with_data = q || k || v;
  if (with_data) {
    const int rc = check_rows_args(dtype, N, H, D);
    if (rc != MOGA_OK) return rc;
  }
  if (!counts || !cu_seqlens || !max_seqlen) return MOGA_ERR_INVALID_ARG;
  if (N > 0) {
    if (!group || !perm || !inv_perm) return MOGA_ERR_INVALID_ARG;
    if (with_data && (!q || !k || !v || !qh || !kh || !vh)) return MOGA_ERR_INVALID_ARG;
    if (with_data && !(aligned16(q) && aligned16(k) && aligned16(v) && aligned16(qh) &&
                       aligned16(kh) && aligned16(vh)))
      return MOGA_ERR_INVALID_ARG;
  }
  return MOGA_OK;
}

extern "C" int moga_permute(const int32_t* group, int64_t N, int M, const void* q, const void* k,
                            const void* v, int dtype, int H, int D, int32_t* counts,
                            int32_t* cu_seqlens, int32_t* max_seqlen, int32_t* perm,
                            int32_t* inv_perm, void* qh, void* kh, void* vh, void* ws,
                            size_t ws_bytes, void* stream) {
  const int rc = permute_check(group, N, M, q, k, v, dtype, H, D, counts, cu_seqlens, max_seqlen,
                               perm, inv_perm, qh, kh, vh);
  if (rc != MOGA_OK) return rc;
  const size_t need = moga_permute_ws_bytes(N, M);
  if (need > 0 && (!ws || ws_bytes < need)) return MOGA_ERR_WORKSPACE;
  return permute_impl(group, N, M, q, k, v, dtype, H, D, counts, cu_seqlens, max_seqlen, perm,
                      inv_perm, qh, kh, vh, (int32_t*)ws, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------
// moga_permute_static: the same call for callers that cannot allocate.  The per-chunk
// histograms live in a file-scope device array; every GPU holds its own copy, whose address is
// looked up once per device (the array's name is only a host-side handle, never a device
// address).  chunk_hist overwrites every entry it later reads, so nothing has to be cleared
// between calls; two calls that overlap on one GPU would share the array and race.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) int32_t scratch[MOGA_PERMUTE_STATIC_MAX_BYTES / sizeof(int32_t)];

static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static int32_t* g_scratch_ptr[kMaxDevices];  // per device, filled on the first call there

// Device address of `scratch` on the current device, or nullptr when HIP reports an error.
static int32_t* static_scratch_for_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = (int32_t*)ptr;
  }
  return g_scratch_ptr[dev];
}

extern "C" int moga_permute_static(const int32_t* group, int64_t N, int M, const void* q,
                                   const void* k, const void* v, int dtype, int H, int D,
                                   int32_t* counts, int32_t* cu_seqlens, int32_t* max_seqlen,
                                   int32_t* perm, int32_t* inv_perm, void* qh, void* kh,
                                   void* vh, void* stream) {
  const int rc = permute_check(group, N, M, q, k, v, dtype, H, D, counts, cu_seqlens, max_seqlen,
                               perm, inv_perm, qh, kh, vh);
  if (rc != MOGA_OK) return rc;
  if (moga_permute_ws_bytes(N, M) > (size_t)MOGA_PERMUTE_STATIC_MAX_BYTES)
    return MOGA_ERR_UNSUPPORTED;  // more chunk histograms than the static array holds
  int32_t* hist = static_scratch_for_current_device();
  if (!hist) return MOGA_ERR_HIP;
  return permute_impl(group, N, M, q, k, v, dtype, H, D, counts, cu_seqlens, max_seqlen, perm,
                      inv_perm, qh, kh, vh, hist, (hipStream_t)stream);
}

static int scatter_dispatch(const Rows3& p, int ntensors, int dtype, int D, const int32_t* perm,
                            const float* gate, int64_t N, int H, hipStream_t st) {
  const int lpr = lanes_per_row(dtype, D);
  if (dtype == MOGA_BF16) {
    launch_scatter<16, true>(p, ntensors, perm, gate, N, H, st);
  } else if (lpr == 16) {
    launch_scatter<16, false>(p, ntensors, perm, gate, N, H, st);
  } else {
    launch_scatter<32, false>(p, ntensors, perm, gate, N, H, st);
  }
  return launch_status();
}

extern "C" int moga_unpermute(const void* oh, int dtype, const int32_t* perm, const float* gate,
                              int64_t N, int H, int D, void* o, void* stream) {
  const int rc = check_rows_args(dtype, N, H, D);
  if (rc != MOGA_OK) return rc;
  if (N == 0) return MOGA_OK;
  if (!oh || !perm || !o) return MOGA_ERR_INVALID_ARG;
  if (!aligned16(oh) || !aligned16(o)) return MOGA_ERR_INVALID_ARG;
  Rows3 p;
  p.src[0] = oh; p.dst[0] = o;
  p.src[1] = p.src[2] = nullptr; p.dst[1] = p.dst[2] = nullptr;
  return scatter_dispatch(p, 1, dtype, D, perm, gate, N, H, (hipStream_t)stream);
}

extern "C" int moga_permute_bwd(const void* d_qh, const void* d_kh, const void* d_vh, int dtype,
                                const int32_t* perm, int64_t N, int H, int D, void* d_q,
                                void* d_k, void* d_v, void* stream) {
  const int rc = check_rows_args(dtype, N, H, D);
  if (rc != MOGA_OK) return rc;
  if (N == 0) return MOGA_OK;
  if (!d_qh || !d_kh || !d_vh || !perm || !d_q || !d_k || !d_v) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(d_qh) && aligned16(d_kh) && aligned16(d_vh) && aligned16(d_q) &&
        aligned16(d_k) && aligned16(d_v)))
    return MOGA_ERR_INVALID_ARG;
  Rows3 p;
  p.src[0] = d_qh; p.src[1] = d_kh; p.src[2] = d_vh;
  p.dst[0] = d_q; p.dst[1] = d_k; p.dst[2] = d_v;
  return scatter_dispatch(p, 3, dtype, D, perm, nullptr, N, H, (hipStream_t)stream);
}

int moga::launch_unpermute_bwd(const void* d_o, const void* oh, int dtype, const int32_t* perm, const float* gate, int64_t N,
                               int H, int D, void* d_oh, float* d_gate, const RowConstants* rc, hipStream_t st) {
  const int bad = check_rows_args(dtype, N, H, D);
  if (bad != MOGA_OK) return bad;
  if (N == 0) return MOGA_OK;
  if (!d_o || !oh || !perm || !gate || !d_oh || !d_gate) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(d_o) && aligned16(oh) && aligned16(d_oh))) return MOGA_ERR_INVALID_ARG;
  const int lpr = lanes_per_row(dtype, D);
#define MOGA_UNPERMUTE_BWD(LPR, BF, DELTA)                                                                                          \
  with_slots(few_slots_of_sums(N), N, [&](auto slots, unsigned blocks) {                                                            \
    unpermute_bwd_kernel<LPR, BF, DELTA, slots.value><<<blocks, 256, 0, st>>>((const uintx4_t*)d_o, (const uintx4_t*)oh, perm, gate, \
                                                                              N, H, (uintx4_t*)d_oh, d_gate, rc ? *rc : RowConstants{}); \
  })
  if (dtype == MOGA_BF16 && rc) MOGA_UNPERMUTE_BWD(16, true, true);
  else if (dtype == MOGA_BF16) MOGA_UNPERMUTE_BWD(16, true, false);
  else if (lpr == 16 && rc) MOGA_UNPERMUTE_BWD(16, false, true);
  else if (lpr == 16) MOGA_UNPERMUTE_BWD(16, false, false);
  else if (rc) MOGA_UNPERMUTE_BWD(32, false, true);
  else MOGA_UNPERMUTE_BWD(32, false, false);
#undef MOGA_UNPERMUTE_BWD
  return launch_status();
}

extern "C" int moga_unpermute_bwd(const void* d_o, const void* oh, int dtype, const int32_t* perm,
                                  const float* gate, int64_t N, int H, int D, void* d_oh,
                                  float* d_gate, void* stream) {
  return launch_unpermute_bwd(d_o, oh, dtype, perm, gate, N, H, D, d_oh, d_gate, nullptr, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------
// static branches
// ---------------------------------------------------------------------------------------
extern "C" int moga_gather_rows(const void* src, int dtype, const int32_t* index, int64_t Nk, int H,
                                int D, void* dst, void* stream) {
  const int bad = check_rows_args(dtype, Nk, H, D);
  if (bad) return bad;
  if (Nk == 0) return MOGA_OK;
  if (!src || !index || !dst || !aligned16(src) || !aligned16(dst)) return MOGA_ERR_INVALID_ARG;
  Rows3 p{};
  p.src[0] = src;
  p.dst[0] = dst;
  const int lpr = lanes_per_row(dtype, D);
  if (lpr == 16) launch_gather<16>(p, 1, index, Nk, H, (hipStream_t)stream);
  else launch_gather<32>(p, 1, index, Nk, H, (hipStream_t)stream);
  return launch_status();
}

extern "C" int moga_gather_rows_bwd(const void* d_dst, int dtype, const int32_t* inv_cu,
                                    const int32_t* inv_slots, int64_t N, int64_t Nk, int H, int D,
                                    int accumulate, void* d_src, void* stream) {
  const int bad = check_rows_args(dtype, N, H, D);
  if (bad) return bad;
  if (Nk < 0 || Nk >= ((int64_t)1 << 31)) return MOGA_ERR_INVALID_ARG;
  if (N == 0) return MOGA_OK;
  if (!inv_cu || !d_src || (Nk > 0 && (!d_dst || !inv_slots))) return MOGA_ERR_INVALID_ARG;
  if (!aligned16(d_dst) || !aligned16(d_src)) return MOGA_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  const unsigned blocks = (unsigned)((N + kManySlots - 1) / kManySlots);
  const int lpr = lanes_per_row(dtype, D);
  if (dtype == MOGA_BF16)
    gather_rows_bwd_kernel<16, true><<<blocks, 256, 0, st>>>((const uintx4_t*)d_dst, inv_cu, inv_slots, N, Nk, H,
                                                             accumulate, (uintx4_t*)d_src);
  else if (lpr == 16)
    gather_rows_bwd_kernel<16, false><<<blocks, 256, 0, st>>>((const uintx4_t*)d_dst, inv_cu, inv_slots, N, Nk, H,
                                                              accumulate, (uintx4_t*)d_src);
  else
    gather_rows_bwd_kernel<32, false><<<blocks, 256, 0, st>>>((const uintx4_t*)d_dst, inv_cu, inv_slots, N, Nk, H,
                                                              accumulate, (uintx4_t*)d_src);
  return launch_status();
}

extern "C" int moga_gather3_fwd(const void* q, const void* k, const void* v, int dtype, int64_t N, int H, int D,
                                const int32_t* inv_moga, const int32_t* q_slot, const int32_t* inv_cu, const int32_t* inv_slots,
                                int64_t Nk, const int32_t* inv_frame, void* qm, void* km, void* vm, void* qs, void* ks, void* vs,
                                void* qf, void* kf, void* vf, void* stream) {
  const int bad = check_rows_args(dtype, N, H, D);
  if (bad) return bad;
  if (Nk < 0 || Nk >= ((int64_t)1 << 31)) return MOGA_ERR_INVALID_ARG;
  if (N == 0) return MOGA_OK;
  if (!q || !k || !v || !inv_moga || !q_slot || !inv_cu || !qm || !km || !vm || !qs || !qf || !kf || !vf ||
      (Nk > 0 && (!inv_slots || !ks || !vs)))
    return MOGA_ERR_INVALID_ARG;
  for (const void* t : {q, k, v, (const void*)qm, (const void*)km, (const void*)vm, (const void*)qs, (const void*)ks, (const void*)vs,
                        (const void*)qf, (const void*)kf, (const void*)vf})
    if (!aligned16(t)) return MOGA_ERR_INVALID_ARG;
  typedef const uintx4_t* in;
  typedef uintx4_t* out;
  const Gather3 p = {{(in)q, (in)k, (in)v}, {(out)qm, (out)km, (out)vm}, {(out)qs, (out)ks, (out)vs}, {(out)qf, (out)kf, (out)vf},
                     {nullptr, inv_cu, inv_cu}, {q_slot, inv_slots, inv_slots}, {N, Nk, Nk}};
  hipStream_t st = (hipStream_t)stream;
  with_slots(few_slots(N), N, [&](auto slots, unsigned blocks) {
    if (lanes_per_row(dtype, D) == 16) gather3_kernel<16, slots.value><<<dim3(blocks, 3), 256, 0, st>>>(p, inv_moga, inv_frame, N, H);
    else gather3_kernel<32, slots.value><<<dim3(blocks, 3), 256, 0, st>>>(p, inv_moga, inv_frame, N, H);
  });
  return launch_status();
}

static int gather3_bwd(const Gather3Bwd& p, int tensors, const int32_t* inv_moga, const int32_t* inv_frame, int dtype, int64_t N, int H,
                       int D, hipStream_t st) {
  for (int i = 0; i < tensors; ++i)
    for (const void* t : {(const void*)p.g_m[i], (const void*)p.g_s[i], (const void*)p.g_f[i], (const void*)p.d_src[i]})
      if (!aligned16(t)) return MOGA_ERR_INVALID_ARG;
  const int lpr = lanes_per_row(dtype, D);
#define MOGA_GATHER3(LPR, BF)                                                                                        \
  with_slots(few_slots(N), N, [&](auto slots, unsigned blocks) {                                                     \
    gather3_bwd_kernel<LPR, BF, slots.value><<<dim3(blocks, tensors), 256, 0, st>>>(p, inv_moga, inv_frame, N, H);   \
  })
  if (dtype == MOGA_BF16) MOGA_GATHER3(16, true);
  else if (lpr == 16) MOGA_GATHER3(16, false);
  else MOGA_GATHER3(32, false);
#undef MOGA_GATHER3
  return launch_status();
}

extern "C" int moga_gather3_bwd(const void* g_moga, const int32_t* inv_moga, const void* g_stga,
                                const int32_t* inv_cu, const int32_t* inv_slots, int64_t Nk,
                                const void* g_frame, const int32_t* inv_frame, int dtype, int64_t N,
                                int H, int D, void* d_src, void* stream) {
  const int bad = check_rows_args(dtype, N, H, D);
  if (bad) return bad;
  if (Nk < 0 || Nk >= ((int64_t)1 << 31)) return MOGA_ERR_INVALID_ARG;
  if (N == 0) return MOGA_OK;
  if (!g_moga || !inv_moga || !inv_cu || !g_frame || !d_src || (Nk > 0 && (!g_stga || !inv_slots)))
    return MOGA_ERR_INVALID_ARG;
  typedef const uintx4_t* in;
  const Gather3Bwd p = {{(in)g_moga}, {(in)g_stga}, {(in)g_frame}, {inv_cu}, {inv_slots}, {Nk}, {(uintx4_t*)d_src}};
  return gather3_bwd(p, 1, inv_moga, inv_frame, dtype, N, H, D, (hipStream_t)stream);
}

extern "C" int moga_gather3_bwd_qkv(const void* gq_moga, const void* gk_moga, const void* gv_moga, const int32_t* inv_moga,
                                    const void* gq_stga, const void* gk_stga, const void* gv_stga, const int32_t* q_slot,
                                    const int32_t* inv_cu, const int32_t* inv_slots, int64_t Nk, const void* gq_frame,
                                    const void* gk_frame, const void* gv_frame, const int32_t* inv_frame, int dtype, int64_t N, int H,
                                    int D, void* d_q, void* d_k, void* d_v, void* stream) {
  const int bad = check_rows_args(dtype, N, H, D);
  if (bad) return bad;
  if (Nk < 0 || Nk >= ((int64_t)1 << 31)) return MOGA_ERR_INVALID_ARG;
  if (N == 0) return MOGA_OK;
  if (!gq_moga || !gk_moga || !gv_moga || !inv_moga || !gq_stga || !q_slot || !inv_cu || !gq_frame || !gk_frame || !gv_frame || !d_q ||
      !d_k || !d_v || (Nk > 0 && (!gk_stga || !gv_stga || !inv_slots)))
    return MOGA_ERR_INVALID_ARG;
  typedef const uintx4_t* in;
  typedef uintx4_t* out;
  const Gather3Bwd p = {{(in)gq_moga, (in)gk_moga, (in)gv_moga}, {(in)gq_stga, (in)gk_stga, (in)gv_stga},
                        {(in)gq_frame, (in)gk_frame, (in)gv_frame}, {nullptr, inv_cu, inv_cu}, {q_slot, inv_slots, inv_slots},
                        {N, Nk, Nk}, {(out)d_q, (out)d_k, (out)d_v}};
  return gather3_bwd(p, 3, inv_moga, inv_frame, dtype, N, H, D, (hipStream_t)stream);
}

extern "C" int moga_merge3_fwd(const void* a_moga, const void* a_stga, const void* a_frame, int dtype,
                               const int32_t* inv_moga, const int32_t* inv_stga, const int32_t* inv_frame,
                               const float* gate, int64_t N, int H, int D, void* o, void* stream) {
  const int bad = check_rows_args(dtype, N, H, D);
  if (bad) return bad;
  if (N == 0) return MOGA_OK;
  if (!a_moga || !a_stga || !a_frame || !gate || !o) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(a_moga) && aligned16(a_stga) && aligned16(a_frame) && aligned16(o))) return MOGA_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  const float alpha = 1.f / 3.f;
  const int lpr = lanes_per_row(dtype, D);
#define MOGA_MERGE_FWD(LPR, BF)                                                                                                    \
  with_slots(few_slots(N), N, [&](auto slots, unsigned blocks) {                                                                   \
    merge3_fwd_kernel<LPR, BF, slots.value><<<blocks, 256, 0, st>>>((const uintx4_t*)a_moga, (const uintx4_t*)a_stga,              \
                                                                    (const uintx4_t*)a_frame, inv_moga, inv_stga, inv_frame, gate, \
                                                                    alpha, N, H, (uintx4_t*)o);                                    \
  })
  if (dtype == MOGA_BF16) MOGA_MERGE_FWD(16, true);
  else if (lpr == 16) MOGA_MERGE_FWD(16, false);
  else MOGA_MERGE_FWD(32, false);
#undef MOGA_MERGE_FWD
  return launch_status();
}

static int merge3_bwd(const void* d_o, const void* a_moga, int dtype, const int32_t* inv_moga, const int32_t* inv_stga,
                      const int32_t* inv_frame, const float* gate, int64_t N, int H, int D, void* d_a_moga, void* d_a_stga,
                      void* d_a_frame, float* d_gate, const Merge3Rows* rows, void* stream) {
  const int bad = check_rows_args(dtype, N, H, D);
  if (bad) return bad;
  if (N == 0) return MOGA_OK;
  if (!d_o || !a_moga || !gate || !d_a_moga || !d_a_stga || !d_a_frame || !d_gate) return MOGA_ERR_INVALID_ARG;
  if (!(aligned16(d_o) && aligned16(a_moga) && aligned16(d_a_moga) && aligned16(d_a_stga) && aligned16(d_a_frame)))
    return MOGA_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  const float alpha = 1.f / 3.f;
  const int lpr = lanes_per_row(dtype, D);
#define MOGA_MERGE_BWD(LPR, BF, ROWS)                                                                                                  \
  with_slots(few_slots_of_sums(N), N, [&](auto slots, unsigned blocks) {                                                               \
    merge3_bwd_kernel<LPR, BF, ROWS, slots.value><<<blocks, 256, 0, st>>>((const uintx4_t*)d_o, (const uintx4_t*)a_moga, inv_moga,     \
                                                                          inv_stga, inv_frame, gate, alpha, N, H, (uintx4_t*)d_a_moga, \
                                                                          (uintx4_t*)d_a_stga, (uintx4_t*)d_a_frame, d_gate,           \
                                                                          rows ? *rows : Merge3Rows{});                                \
  })
  if (dtype == MOGA_BF16 && rows) MOGA_MERGE_BWD(16, true, true);
  else if (dtype == MOGA_BF16) MOGA_MERGE_BWD(16, true, false);
  else if (lpr == 16 && rows) MOGA_MERGE_BWD(16, false, true);
  else if (lpr == 16) MOGA_MERGE_BWD(16, false, false);
  else if (rows) MOGA_MERGE_BWD(32, false, true);
  else MOGA_MERGE_BWD(32, false, false);
#undef MOGA_MERGE_BWD
  return launch_status();
}

extern "C" int moga_merge3_bwd(const void* d_o, const void* a_moga, int dtype, const int32_t* inv_moga,
                               const int32_t* inv_stga, const int32_t* inv_frame, const float* gate,
                               int64_t N, int H, int D, void* d_a_moga, void* d_a_stga, void* d_a_frame,
                               float* d_gate, void* stream) {
  return merge3_bwd(d_o, a_moga, dtype, inv_moga, inv_stga, inv_frame, gate, N, H, D, d_a_moga, d_a_stga, d_a_frame, d_gate,
                    nullptr, stream);
}

extern "C" int moga_merge3_bwd_rows(const void* d_o, const void* a_moga, const void* a_stga, const void* a_frame, int dtype,
                                    const int32_t* inv_moga, const int32_t* inv_stga, const int32_t* inv_frame,
                                    const float* gate, const float* lse_moga, const float* lse_stga, const float* lse_frame,
                                    float softmax_scale, int64_t N, int H, int D, void* d_a_moga, void* d_a_stga,
                                    void* d_a_frame, float* d_gate, void* ws_moga, void* ws_stga, void* ws_frame,
                                    size_t ws_bytes, void* stream) {
  const int bad = check_rows_args(dtype, N, H, D);
  if (bad) return bad;
  if (N == 0) return MOGA_OK;
  if (!a_stga || !a_frame || !lse_moga || !lse_stga || !lse_frame || !aligned16(a_stga) || !aligned16(a_frame) || !(softmax_scale > 0.f) ||
      !(softmax_scale < INFINITY))
    return MOGA_ERR_INVALID_ARG;
  const size_t status = moga_attn_bwd_status_offset(N, H);
  if (!ws_moga || !ws_stga || !ws_frame || ws_bytes < status + 16) return MOGA_ERR_WORKSPACE;
  auto rc = [&](void* ws, const float* lse) {
    float* f = (float*)ws;
    return RowConstants{lse, 1.f / softmax_scale, f, f + N * (int64_t)H, (int*)((char*)ws + status)};
  };
  const Merge3Rows rows = {(const uintx4_t*)a_stga, (const uintx4_t*)a_frame, rc(ws_moga, lse_moga), rc(ws_stga, lse_stga),
                           rc(ws_frame, lse_frame)};
  return merge3_bwd(d_o, a_moga, dtype, inv_moga, inv_stga, inv_frame, gate, N, H, D, d_a_moga, d_a_stga, d_a_frame, d_gate, &rows,
                    stream);
}
