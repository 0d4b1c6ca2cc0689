// Pieces shared by the forward and backward group-attention kernels.
#pragma once

#include <algorithm>
#include <cmath>

#include "lds_pipe.h"

namespace moga {

constexpr int kHeadDim = 128;  // head_dim of the bf16 MFMA kernels
constexpr int kMaxCalls = MOGA_MAX_CALLS;   // of one launch

// Tile schedule.  Every group g with n_g rows contributes ceil(n_g / rows_per_tile) tiles;
// tiles never straddle a group boundary.  `tile` is a flat index over all groups in order.
// Both lookups are done by every wave for itself, with all 64 lanes and no LDS or barrier, and
// return wave-uniform values (scalar registers).  They return false when `tile` lies beyond the
// last real tile (the grid is sized from an upper bound because the group sizes live on the device).
struct TileInfo {
  int group;      // group id
  int row_begin;  // first row of the group (sorted slot)
  int row_end;    // one past the last row of the group
  int tile_row;   // first row of this tile
};

// A lane per group, 64 groups at a time: one round trip to memory and some twenty instructions.  (Through
// LDS, with two barriers and the group's bounds read again, it took 2 us more of a block's prologue.)
__device__ __forceinline__ bool find_tile(const int32_t* __restrict__ cu_seqlens, int M, int rows_per_tile, int tile,
                                          TileInfo& out) {
  const int lane = threadIdx.x & 63;
  int running = 0;
  for (int g0 = 0; g0 < M; g0 += 64) {
    const int beg = cu_seqlens[min(g0 + lane, M)], end = cu_seqlens[min(g0 + lane + 1, M)];
    const int t = (end - beg + rows_per_tile - 1) / rows_per_tile;
    const int incl = running + wave_scan_add(t);
    const unsigned long long hit = __ballot(incl - t <= tile && tile < incl);
    if (hit) {
      const int l = __builtin_ctzll(hit);
      out.group = g0 + l;
      out.row_begin = __builtin_amdgcn_readlane(beg, l);
      out.row_end = __builtin_amdgcn_readlane(end, l);
      out.tile_row = out.row_begin + (tile - __builtin_amdgcn_readlane(incl - t, l)) * rows_per_tile;
      return true;
    }
    running = __builtin_amdgcn_readlane(incl, 63);
  }
  return false;
}

// The lookup of find_tile for calls with more than MOGA_MAX_GROUPS groups: `tile_start[g]` (M + 1 entries, written
// by tile_start_kernel) is the flat index of group g's first tile.  The 64 lanes probe 64 entries at
// once, so 4,096 groups take two dependent loads (a binary search: twelve).
__device__ __forceinline__ bool find_tile_presummed(const int32_t* __restrict__ tile_start,
                                                    const int32_t* __restrict__ cu_seqlens, int M,
                                                    int rows_per_tile, int tile, TileInfo& out) {
  if (tile >= tile_start[M]) return false;
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = M, step;   // tile_start[lo] <= tile, and tile < tile_start[hi]
  do {
    step = (hi - lo + 63) >> 6;
    const int idx = lo + lane * step;
    const unsigned long long below = __ballot(idx < hi && tile_start[min(idx, M)] <= tile);   // lane 0 always
    lo += (63 - __builtin_clzll(below)) * step;
    hi = min(hi, lo + step);
  } while (step > 1);
  out.group = lo;
  out.row_begin = cu_seqlens[lo];
  out.row_end = cu_seqlens[lo + 1];
  out.tile_row = out.row_begin + (tile - tile_start[lo]) * rows_per_tile;
  return true;
}

// Splitting the last round.  Blocks of one size run in rounds of kCus; the tiles of the
// last, partly filled round are cut along the other side into equal runs of 64-row tiles, so that the round is full and
// shorter.  Such a piece writes fp32 partial results to slot `slot` of the workspace, and split_*_kernel puts the pieces
// of a tile together.  Without: 6.2 rounds of work took the time of 7 (forward, 32,760 rows x 12 heads, 8 groups).
constexpr int kCus = 256;
constexpr int kMaxSplits = 8;
struct WorkTile {
  TileInfo ti;
  int head;
  int split, splits;   // splits == 1: a whole tile
  int slot;
};
struct SplitShape { int full, left, splits; };   // whole tiles in full rounds, tiles of the last round, pieces of each

__device__ __forceinline__ SplitShape split_shape(int tiles) {
  SplitShape s = {tiles / kCus * kCus, tiles % kCus, 1};
  if (s.left > 0) s.splits = min(kMaxSplits, kCus / s.left);
  return s;
}

// Tiles of one head.
__device__ __forceinline__ int count_tiles(const int32_t* __restrict__ cu_seqlens, int M, int rows_per_tile) {
  const int lane = threadIdx.x & 63;
  int sum = 0;
  for (int g0 = 0; g0 < M; g0 += 64) {
    const int n = cu_seqlens[min(g0 + lane + 1, M)] - cu_seqlens[min(g0 + lane, M)];
    sum += __builtin_amdgcn_readlane(wave_scan_add((n + rows_per_tile - 1) / rows_per_tile), 63);
  }
  return sum;
}

// Position w of the work list -> (head, tile of the head).  The hardware deals blocks round-robin to the 8 XCDs, so
// w % 8 is the XCD: each gets an eighth of the heads whole (a head's K/V tiles are streamed through a single L2), and the
// tiles of the remaining heads are dealt in runs of 16, the last ones singly, so that the XCDs' shares are equal whatever
// the group sizes are.  (As one list with bounds per head, cut into eighths, 62,400 rows x 4 heads in 8 Zipf(1.1) groups
// took 8.1 ms instead of 5.3; dealt singly throughout, groups of 1,560 rows lose 6 %: their rows go to every L2.)
__device__ __forceinline__ void decode_work(int w, int per_head, int H, int& head, int& tile) {
  const int whole = (H & ~7) * per_head;
  const bool rest = w >= whole;
  int i = rest ? w - whole : w >> 3;
  if (rest && i < ((H & 7) * per_head & ~127)) i = (i & ~127) + (i & 7) * 16 + ((i >> 3) & 15);
  const int h = i / per_head;
  head = rest ? (H & ~7) + h : (w & 7) * (H >> 3) + h;
  tile = i - h * per_head;
}

// What block `block` works on; false: nothing.  tile_start: NULL, or the pre-summed tiles (more than MOGA_MAX_GROUPS groups).
template <bool SPLIT>
__device__ __forceinline__ bool find_work(const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ tile_start, int M, int H,
                                          int rows_per_tile, int block, WorkTile& out) {
  // up to 64 groups (a lane each) the bounds are read once, for the count and for the lookup
  const int lane = threadIdx.x & 63;
  const bool one_scan = !tile_start && M <= 64;
  int beg = 0, end = 0, incl = 0, per_head;
  if (one_scan) {
    beg = cu_seqlens[min(lane, M)];
    end = cu_seqlens[min(lane + 1, M)];
    incl = wave_scan_add((end - beg + rows_per_tile - 1) / rows_per_tile);
    per_head = __builtin_amdgcn_readlane(incl, 63);
  } else {
    per_head = tile_start ? tile_start[M] : count_tiles(cu_seqlens, M, rows_per_tile);
  }
  const int total = per_head * H;
  int w = block, tile;
  out.split = out.slot = 0;
  out.splits = 1;
  if constexpr (SPLIT) {
    const SplitShape s = split_shape(total);
    if (block >= s.full) {
      const int p = block - s.full;
      if (p >= s.left * s.splits) return false;
      w = s.full + p % s.left;
      out.split = p / s.left;
      out.splits = s.splits;
      out.slot = (p % s.left) * s.splits + out.split;
    }
  }
  if (w >= total) return false;
  decode_work(w, per_head, H, out.head, tile);
  if (!one_scan)
    return tile_start ? find_tile_presummed(tile_start, cu_seqlens, M, rows_per_tile, tile, out.ti)
                      : find_tile(cu_seqlens, M, rows_per_tile, tile, out.ti);
  const int g = __builtin_ctzll(__ballot(incl > tile));
  out.ti.group = g;
  out.ti.row_begin = __builtin_amdgcn_readlane(beg, g);
  out.ti.row_end = __builtin_amdgcn_readlane(end, g);
  const int first = __builtin_amdgcn_readlane(incl, g) - (out.ti.row_end - out.ti.row_begin + rows_per_tile - 1) / rows_per_tile;
  out.ti.tile_row = out.ti.row_begin + (tile - first) * rows_per_tile;
  return true;
}

// Rows (first, count) of the other side that a piece sweeps.
__device__ __forceinline__ void split_range(const WorkTile& s, int& first, int& n) {
  const int tiles = (n + 63) >> 6, t0 = tiles * s.split / s.splits, t1 = tiles * (s.split + 1) / s.splits;
  const int end = min(n, 64 * t1);
  first += 64 * t0;
  n = end - 64 * t0;
}

// Column `col` (16 result rows) of a wave, d tile dt, as fp32 rows of a slot; `base` is the wave's first row.
__device__ __forceinline__ void store_partial(float* base, int dt, int col, const floatx4_t& v) {
  const int lane = threadIdx.x & 63;
  *(floatx4_t*)(base + (16 * col + (lane & 15)) * kHeadDim + 16 * dt + 4 * (lane >> 4)) = v;
}

// A round of pieces of `rows` result rows each (dV and dK: of both), 34 MB for 256 and 51 MB for 384: results, then (max, sum) of the forward.
constexpr size_t split_bytes(int rows) { return (size_t)kCus * rows * (kHeadDim + 2) * sizeof(float); }
struct SplitWs {
  float *part, *stat;
};
inline SplitWs split_ws(void* ws, int rows) { return {(float*)ws, (float*)ws + (size_t)kCus * rows * kHeadDim}; }
// The part of a workspace past its first `used` bytes, and the rows of the longest pieces that fit there (0: none do).
struct SplitRoom {
  void* ws;
  int rows;
};
inline SplitRoom split_room(void* ws, size_t used, size_t ws_bytes) {
  if (!ws) return {nullptr, 0};
  const size_t off = round_up((size_t)(uintptr_t)ws + used, 256) - (size_t)(uintptr_t)ws;
  const int rows = ws_bytes >= off + split_bytes(384) ? 384 : ws_bytes >= off + split_bytes(256) ? 256 : 0;
  return {rows ? (char*)ws + off : nullptr, rows};
}
// Worth it for a few rounds of the kernels with long blocks; beyond 32 rounds the last one is under 3 %.
inline bool split_pays(int64_t tiles) { return tiles <= 32 * kCus; }

// Sum of the pieces of every tile of the last round, times f, as bf16 rows of `out` (sorted order) and `tok` (token order),
// each of which may be NULL.  A tile has `arrays` results of
// `rows` rows each.  Grid (kCus / 2, arrays * rows / 8): eight rows per block, one trip
// to memory (with 64 rows per block, one after the other, 45 us instead of 9).
static __global__ __launch_bounds__(256) void split_sum_kernel(const float* __restrict__ part, const int32_t* __restrict__ cu, int M,
                                                               int H, int64_t N, int rows, float f0, float f1,
                                                               unsigned short* __restrict__ out0,
                                                               unsigned short* __restrict__ out1,
                                                               unsigned short* __restrict__ tok0,
                                                               unsigned short* __restrict__ tok1,
                                                               const int32_t* __restrict__ perm) {
  const int per_head = count_tiles(cu, M, rows);
  const SplitShape s = split_shape(per_head * H);
  if (s.splits == 1 || (int)blockIdx.x >= s.left) return;
  int head, tile;
  decode_work(s.full + blockIdx.x, per_head, H, head, tile);
  TileInfo ti;
  if (!find_tile(cu, M, rows, tile, ti)) return;
  const int col = (threadIdx.x & 31) * 4, r = blockIdx.y * 8 + (threadIdx.x >> 5);
  const int a = r / rows, row = ti.tile_row + r % rows;
  if (row >= ti.row_end) return;
  const size_t piece = 8 * gridDim.y;   // rows
  const float* p = part + ((size_t)blockIdx.x * s.splits * piece + r) * kHeadDim + col;
  floatx4_t v[kMaxSplits];   // all in flight together
#pragma unroll
  for (int k = 0; k < kMaxSplits; ++k) v[k] = k < s.splits ? *(const floatx4_t*)(p + k * piece * kHeadDim) : floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 1; k < kMaxSplits; ++k) v[0] += v[k];
  unsigned short *o = a ? out1 : out0, *t = a ? tok1 : tok0;
  const float f = a ? f1 : f0;
  const uintx2_t w = {pack_bf16x2(v[0][0] * f, v[0][1] * f), pack_bf16x2(v[0][2] * f, v[0][3] * f)};
  if (o) *(uintx2_t*)(o + ((int64_t)head * N + row) * kHeadDim + col) = w;
  if (t) *(uintx2_t*)(t + ((int64_t)perm[row] * H + head) * kHeadDim + col) = w;
}

// One block: exclusive scan of ceil(n_g / rows_per_tile) over the groups, M + 1 results.
static __global__ __launch_bounds__(1024) void tile_start_kernel(const int32_t* __restrict__ cu_seqlens, int M,
                                                                 int rows_per_tile, int32_t* __restrict__ tile_start) {
  __shared__ int s_wave[16];
  __shared__ int s_carry;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (int g0 = 0; g0 < M; g0 += 1024) {
    const int g = g0 + threadIdx.x;
    const int n = g < M ? cu_seqlens[g + 1] - cu_seqlens[g] : 0;
    const int t = n > 0 ? (n + rows_per_tile - 1) / rows_per_tile : 0;
    int incl = t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += up;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = s_carry;
    for (int w = 0; w < wave; ++w) before += s_wave[w];
    if (g < M) tile_start[g] = before + incl - t;
    __syncthreads();
    if (threadIdx.x == 1023) s_carry = before + incl;
    __syncthreads();
  }
  if (threadIdx.x == 0) tile_start[M] = s_carry;
}

// Upper bound on the number of tiles for N rows in M groups (host side).
inline int64_t max_tiles(int64_t N, int M, int rows_per_tile) {
  return (N + rows_per_tile - 1) / rows_per_tile + M;
}

// Rows of a block of the large kernels (forward and dQ: 256 or 384 query rows; dK/dV: 128 or 192 keys), and whether the call splits its
// last round.  Per row the longer blocks take less time (a fragment read from LDS feeds three products instead of two, the stream of the
// other side is shared by more), but alone on its CU one takes 1.3 times as long as a short one: a call of less than a round that does not
// split takes that much longer.  So the rounds are priced: for every row of the other side a step, kStartRows of them for a block's start
// and end (prologue, row fragments, stores), the last round by its pieces if it is split, which costs kMergeRows more.  With every round the
// blocks get further out of step, and the price goes over from whole rounds to the work per CU and half a block.
// Constants from 374 calls of equal groups, 0.07 to 21 rounds of 256 blocks, groups of 500 to 20,000 rows, either size of block forced: where
// these kernels run by default the choice is the faster one or within (mean / worst) 0.3 / 8 % forward, 0.1 / 3 % by dK/dV, and of the whole
// backward 0.5 / 6 % by dQ, split or not (by whole rounds only 0.7 / 10, 0.2 / 6 and 0.5 / 6).  The host knows the
// mean group only and takes it for all.  Where groups are unequal the longest block may be the whole call's time: from two to four rounds of
// 256-row blocks 384 rows took Zipf(1.1) groups 9 % more time than 256 without a split and 11 % with, up to 36 %, and gained 3 % with equal
// groups, so there they have to be a fifth cheaper (nobody slower on average, at worst 2 %).  Over 172 calls of Zipf(1.1) groups the
// choice is within 4 % of the faster one forward, 2 % backward.  Milliseconds with 256 and 384 rows, forward without a split: 5,000 x 3 heads, 5 groups 0.029 and
// 0.039; 7,000 x 4, 2 groups 0.081 and 0.111; 40,000 x 3, 4 groups 0.52 and 0.65; 99,840 x 12, 16 groups 3.33 and 3.09.
struct Blocks {
  int rows;
  bool split;
};
// N: rows of this side, in blocks of `few` or 3/2 of that; other: rows of the side that they sweep; arrays: results per row; room: result
// rows of the longest piece there is room for.
constexpr double kStartRows = 640, kMergeRows = 1000;
inline Blocks large_blocks(int64_t N, int64_t other, int H, int M, int few, int arrays, int room, double* price = nullptr) {
  const int64_t mean = (N + M - 1) / M, swept = (other + M - 1) / M;
  auto splits = [&](int rows) { return room >= arrays * rows && split_pays(max_tiles(N, M, rows) * H); };
  auto cost = [&](int rows, double weight) {
    const int64_t of_group = (mean + rows - 1) / rows, tiles = of_group * M * H, full = tiles / kCus, left = tiles % kCus;
    const int64_t pieces = left > 0 && splits(rows) ? std::min<int64_t>(kMaxSplits, kCus / left) : 1;
    const double block = swept + kStartRows, last = left > 0 ? swept / pieces + kStartRows : 0;
    const double in_step = full > 1 ? std::pow(0.8, full - 1) : 1;
    const double short_end = mean - (of_group - 1) * rows <= few ? (weight - 10) * M * H : 0;   // a group's last block, of two columns a wave
    return in_step * weight * (full * block + last) + (1 - in_step) * ((weight * tiles - short_end) / kCus * block + weight * last / 2) +
           (pieces > 1 ? 10 * kMergeRows : 0);
  };
  const bool by_far = arrays == 1 && N * H >= 2 * 256 * kCus && N * H < 4 * 256 * kCus;
  const double short_cost = cost(few, 10), long_cost = cost(few / 2 * 3, 13);
  const int rows = short_cost < (by_far ? 1.2 : 1.) * long_cost ? few : few / 2 * 3;
  if (price) *price = rows == few ? short_cost : long_cost;
  return {rows, splits(rows)};
}
inline Blocks query_blocks(int64_t Nq, int64_t Nk, int H, int M, int room) { return large_blocks(Nq, Nk, H, M, 256, 1, room); }
inline Blocks key_blocks(int64_t Nq, int64_t Nk, int H, int M, int room) { return large_blocks(Nk, Nq, H, M, 128, 2, room); }

// The same for the large-group calls of one launch, by work per CU: tiles of all of them, and half a block of the shortest for the end.
struct SideShape {
  int64_t N, other;   // rows of this side; of the side that they sweep
  int M;
};
inline double calls_cost(const SideShape* c, int n, int H, int rows, int few, double weight) {
  double work = 0, last = 0;
  for (int i = 0; i < n; ++i) {
    const int64_t mean = (c[i].N + c[i].M - 1) / c[i].M, of_group = (mean + rows - 1) / rows;
    const double block = (double)((c[i].other + c[i].M - 1) / c[i].M) + kStartRows;
    const double short_end = mean - (of_group - 1) * rows <= few ? weight - 10 : 0;
    work += (weight * of_group - short_end) * c[i].M * H * block;
    last = i == 0 ? block : std::min(last, block);
  }
  return work / kCus + weight * last / 2;
}

// What a bf16 call runs: the kernels for small groups, or the large ones and their blocks of queries (and of keys, backward).  room:
// that of split_room (0 where M > MOGA_MAX_GROUPS).
struct AttnPlan {
  bool small;
  Blocks q, k;
};
AttnPlan fwd_plan(int64_t Nq, int64_t Nk, int H, int M, int room);
AttnPlan bwd_plan(int64_t Nq, int64_t Nk, int H, int M, int room);
int64_t fwd_calls_small_rows(int64_t rows, int H, int64_t shortest);
bool fwd_call_alone(int64_t Nq, int H, int G);   // of moga_varlen_attn_fwd_calls: by itself, if its last round can be split

// Matrix products of the bf16 kernels: 16x16x32 (A 16 x 32, B 32 x 16).  Lane l = 16 g + r holds row (A) or
// column (B) r at k = 8 g .. 8 g + 7, and rows 4 g .. 4 g + 3 of column r of the result.  At the board's power cap a
// register-resident loop of random operands reaches 1.94-2.18 PFLOP/s (card to card) with this shape and 1.83-1.86 with 32x32x16
// (whose accumulators are read and written twice as often per product), and an A fragment from LDS feeds 16 columns for every B
// fragment that a wave keeps (two or three).
__device__ __forceinline__ floatx4_t mfma16(bf16x8_t a, bf16x8_t b, floatx4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// A step takes 32 rows of an LDS tile as two 16-row A operands t = 0, 1; operand row 4 a + b is tile row
// 8 a + 4 t + b.  A lane's eight results are then eight consecutive rows: the B operand of the second product.
__device__ __forceinline__ int step_row(int r) { return 8 * (r >> 2) + (r & 3); }   // t = 0; t = 1 is 4 rows further

// LDS layout of a tile of ROWS rows of 128 bf16: four quarters (channels 32 ks .. 32 ks + 31), each [ROWS][64 bytes], so that the
// quarter is an immediate offset of a read and a lane needs one address register for row fragments and two for transposed ones
// (as [ROWS][256 bytes], with the 16-byte chunk index XOR-swizzled by the row, it needs 4 and 8).  Inside a row the four
// 16-byte chunks are XOR-swizzled by row bits 4:3 (a) as 0, 2, 3, 1: a 16-byte
// read is served in groups of lanes {0-3, 12-15, 20-27} and {4-11, 16-19, 28-31} (and the same plus 32), which then
// hit all banks once, and so do both halves of a transposed read (rows 8 g .. 8 g + 3).  Row bit 2 does not count: the second
// operand and the upper rows of a transposed fragment are constant offsets, and so are the upper 32 rows.
constexpr int kRow4Bytes = 4 * 64, kRow32Bytes = 32 * 64;
template <int ROWS>
constexpr int kQuarterBytes = ROWS * 64;
__device__ __forceinline__ int lds_swizzle(int row) { return (((row >> 2) ^ (row >> 3)) & 2) | ((row >> 4) & 1); }

// Per-lane LDS byte addresses (slot 0, first step) of the A operands of a tile at `base`.
// nat: rows as they are, d = 8 g .. of a quarter; operand t adds t * kRow4Bytes.
// tr: transposed, d = 16 p + r of a quarter for p = 0, 1, 32 tile rows.
__device__ __forceinline__ unsigned nat_address(const void* base, int lane) {
  const int g = lane >> 4, row = step_row(lane & 15);
  return (unsigned)(uintptr_t)base + row * 64 + ((g ^ lds_swizzle(row)) << 4);
}
__device__ __forceinline__ void tr_addresses(unsigned (&tr)[2], const void* base, int lane) {
  const int row = 8 * (lane >> 4) + ((lane & 15) >> 2), c = (lane & 3) >> 1;
#pragma unroll
  for (int p = 0; p < 2; ++p) tr[p] = (unsigned)(uintptr_t)base + row * 64 + (((2 * p + c) ^ lds_swizzle(row)) << 4) + (lane & 1) * 8;
}
// The fragments: rows of operand t at k block ks; transposed d tile dt.
template <int ROWS>
__device__ __forceinline__ bf16x8_t read_nat(unsigned nat, int t, int ks) {
  return lds_read_b128(nat + ks * kQuarterBytes<ROWS> + t * kRow4Bytes);
}
template <int ROWS>
__device__ __forceinline__ bf16x8_t read_tr(const unsigned (&tr)[2], unsigned off, int dt) {
  const unsigned a = tr[dt & 1] + off + (dt >> 1) * kQuarterBytes<ROWS>;
  return concat_tr(lds_read_tr16_addr(a), lds_read_tr16_addr(a + kRow4Bytes));
}

// Priority of this wave among the waves of its SIMD, in the kernels with one block per CU.  Where two blocks share a
// CU their waves are out of step by themselves, and priorities cost 3 % (10,007 rows x 12 heads, 20 groups).
template <bool ON, int P>
__device__ __forceinline__ void wave_priority() {
  if constexpr (ON) __builtin_amdgcn_s_setprio(P);
}

// Four results of a column (d = 16 dt + 4 g ..) as bf16, scaled.
__device__ __forceinline__ uintx2_t pack4(const floatx4_t& v, float f) {
  return uintx2_t{pack_bf16x2(v[0] * f, v[1] * f), pack_bf16x2(v[2] * f, v[3] * f)};
}

// Results of two neighbouring d tiles (dt even, dt + 1) of a column, four values of each per lane, as 16 adjacent bytes per
// lane: lane groups g and g ^ 1 exchange halves, so that an even group ends up with eight values of tile dt and an odd one with
// eight of tile dt + 1, from channel 16 dt + join_channel(g) on.  A store then covers 64 bytes of each of 16 rows instead of
// 32, in half as many instructions.  Lanes of a column are active together.
__device__ __forceinline__ uintx4_t join_tiles(uintx2_t lo, uintx2_t hi) {
  const auto a = __builtin_amdgcn_permlane16_swap(lo[0], hi[0], false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(lo[1], hi[1], false, false);
  return uintx4_t{a[0], b[0], a[1], b[1]};
}
__device__ __forceinline__ int join_channel(int g) { return 16 * (g & 1) + 4 * (g & 2); }

// Eight bf16 values times f, rounded again.
__device__ __forceinline__ uintx4_t scale8(uintx4_t v, float f) {
  uintx4_t r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = pack_bf16x2(bf16_lo_to_f32(v[i]) * f, bf16_hi_to_f32(v[i]) * f);
  return r;
}
__device__ __forceinline__ uintx2_t scale4(uintx2_t v, float f) {
  return uintx2_t{pack_bf16x2(bf16_lo_to_f32(v[0]) * f, bf16_hi_to_f32(v[0]) * f),
                  pack_bf16x2(bf16_lo_to_f32(v[1]) * f, bf16_hi_to_f32(v[1]) * f)};
}

}  // namespace moga
