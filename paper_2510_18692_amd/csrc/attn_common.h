// Pieces shared by the forward and backward group-attention kernels.
#pragma once

#include "lds_pipe.h"

namespace moga {

constexpr int kHeadDim = 128;  // head_dim of the bf16 MFMA kernels

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

// The same lookup for calls with more than MOGA_MAX_GROUPS groups: `tile_start[g]` (M + 1 entries, written
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

// Work item of a block: blocks are dealt round-robin to the 8 XCDs by the hardware, so block
// b runs on XCD b % 8.  Give each XCD one contiguous eighth of the (head-major) work list, so
// that the K/V tiles of a head are streamed through a single L2.
__device__ __forceinline__ int64_t xcd_work_index(int64_t block, int64_t total) {
  const int64_t per = (total + 7) / 8;
  return (block & 7) * per + (block >> 3);
}

// Row permutation that makes the 32x32 MFMA accumulator registers of a lane hold eight
// consecutive contraction indices: swap bits 2 and 3 of the row index.
__device__ __forceinline__ int swap_bits_2_3(int x) {
  return (x & ~12) | ((x & 4) << 1) | ((x & 8) >> 1);
}

// XOR swizzle of the 16-byte chunk index inside an unpadded 256-byte LDS row (128 bf16):
// chunk' = chunk ^ lds_swizzle(row).  The two low row bits land in chunk bits 3:2 and row bits
// 3:2 in chunk bits 1:0, which spreads both the row-per-lane 16-byte reads and the 4-row
// transposed reads over all banks.
__device__ __forceinline__ int lds_swizzle(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

}  // namespace moga
