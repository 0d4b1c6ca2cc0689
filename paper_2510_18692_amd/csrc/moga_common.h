// Shared device helpers and host-side launch checks for the gfx950 MoGA kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "moga.h"

namespace moga {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float floatx2_t __attribute__((ext_vector_type(2)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef unsigned int uintx2_t __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// fp32 <-> bf16 (round to nearest even), packed two at a time (one v_cvt_pk_bf16_f32).
__device__ __forceinline__ unsigned int pack_bf16x2(float lo, float hi) {
  floatx2_t f = {lo, hi};
  bf16x2_t b = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(unsigned int, b);
}
__device__ __forceinline__ float bf16_lo_to_f32(unsigned int packed) {
  return __uint_as_float(packed << 16);
}
__device__ __forceinline__ float bf16_hi_to_f32(unsigned int packed) {
  return __uint_as_float(packed & 0xffff0000u);
}
__device__ __forceinline__ float bf16_bits_to_f32(unsigned short b) {
  return __uint_as_float(((unsigned int)b) << 16);
}
__device__ __forceinline__ unsigned short f32_to_bf16_bits(float f) {
  return (unsigned short)(pack_bf16x2(f, 0.f) & 0xffffu);
}

// Butterfly reductions over L = 16, 32 or 64 neighbouring lanes (distances L / 2 .. 1) with cross-lane data paths of the vector
// unit.  (__shfl_xor goes through LDS, some 120 cycles a step: the fp32 router at 4,096 x 128, 8 groups and the row sums of the
// scatter backward wait for little else.)  All L lanes are active.
template <int CTRL>
__device__ __forceinline__ int dpp_lane(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false); }
// The value X lanes away (xor), X = 1, 2, 4, 8.
template <int X>
__device__ __forceinline__ int xor_lane(int v) {
  if (X == 8) return dpp_lane<0x128>(v);                  // rotation of a row of 16 by 8
  if (X == 4) return dpp_lane<0x1b>(dpp_lane<0x141>(v));  // 7 - i of eight, then 3 - i of four
  return X == 2 ? dpp_lane<0x4e>(v) : dpp_lane<0xb1>(v);  // within four lanes
}
template <int X, typename F>
__device__ __forceinline__ int combine_xor(int v, F f) {
  if constexpr (X == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);   // the lower halves, the upper halves
    return f((int)r[0], (int)r[1]);
  } else if constexpr (X == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // the even rows, the odd rows
    return f((int)r[0], (int)r[1]);
  } else {
    return f(v, xor_lane<X>(v));
  }
}
template <int L, typename F>
__device__ __forceinline__ int lanes_reduce(int v, F f) {
  if constexpr (L >= 64) v = combine_xor<32>(v, f);
  if constexpr (L >= 32) v = combine_xor<16>(v, f);
  v = combine_xor<8>(v, f);
  v = combine_xor<4>(v, f);
  v = combine_xor<2>(v, f);
  return combine_xor<1>(v, f);
}
struct AddF { __device__ int operator()(int a, int b) const { return __float_as_int(__int_as_float(a) + __int_as_float(b)); } };
struct MaxF { __device__ int operator()(int a, int b) const { return __float_as_int(fmaxf(__int_as_float(a), __int_as_float(b))); } };
struct AddI { __device__ int operator()(int a, int b) const { return a + b; } };
struct MaxI { __device__ int operator()(int a, int b) const { return a > b ? a : b; } };
template <int L> __device__ __forceinline__ float lanes_sum(float v) { return __int_as_float(lanes_reduce<L>(__float_as_int(v), AddF{})); }
__device__ __forceinline__ float wave_sum(float v) { return lanes_sum<64>(v); }
__device__ __forceinline__ float wave_max(float v) { return __int_as_float(lanes_reduce<64>(__float_as_int(v), MaxF{})); }
__device__ __forceinline__ int wave_sum_i(int v) { return lanes_reduce<64>(v, AddI{}); }
__device__ __forceinline__ int wave_max_i(int v) { return lanes_reduce<64>(v, MaxI{}); }

// Inclusive sum over the lanes of a wave with cross-lane data paths of the vector unit (no LDS).
__device__ __forceinline__ int wave_scan_add(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // rows of 16 lanes: shift by 1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // last lane of row 0 / 2 into row 1 / 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // last lane of row 1 into rows 2 and 3
  return x;
}

// Value held by the lane 32 away (the other half of the wave).
__device__ __forceinline__ float other_half(float v) { return __shfl_xor(v, 32, kWave); }
__device__ __forceinline__ int other_half_i(int v) { return __shfl_xor(v, 32, kWave); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Zero fill as a kernel (a memset node inside a captured graph is avoided on purpose).
[[maybe_unused]] static __global__ __launch_bounds__(256) void fill_zero_kernel(float* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0.f;
}

// ---- host side ------------------------------------------------------------
// true when groups of mean size rows / groups should run on the small-group bf16 attention kernels
bool use_small_group_kernels(int64_t rows, int groups, int64_t default_threshold);
// Row constants of the attention backward, [H, N] in sorted order, and its status word (fp32: -delta and the word).
struct RowConstants {
  const float* lse;
  float inv_scale;
  float *neg_delta, *neg_lse_over_scale;
  int* status;
};
// moga_unpermute_bwd; rc: NULL, or the row constants as well
int launch_unpermute_bwd(const void* d_o, const void* oh, int dtype, const int32_t* perm, const float* gate, int64_t N, int H,
                         int D, void* d_oh, float* d_gate, const RowConstants* rc, hipStream_t st);
// HIP takes fewer than 2^32 threads in a grid; of more it launches what is left of the number in 32 bits, without an error.
inline bool grid_fits(int64_t blocks, int threads) { return blocks * threads < ((int64_t)1 << 32); }
[[maybe_unused]] static void launch_fill_zero(float* p, int64_t n, hipStream_t st) {
  fill_zero_kernel<<<(unsigned)((n + 255) / 256 < (1 << 20) ? (n + 255) / 256 : 1 << 20), 256, 0, st>>>(p, n);
}
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int launch_status() { return hipGetLastError() == hipSuccess ? MOGA_OK : MOGA_ERR_HIP; }
inline size_t round_up(size_t a, size_t b) { return (a + b - 1) / b * b; }
inline size_t elem_size(int dtype) { return dtype == MOGA_F32 ? 4 : 2; }

// Number of wave-sized token chunks the permutation uses for N tokens, and their length.
inline int perm_chunk_len(int64_t N) {
  int64_t len = 512;
  while ((N + len - 1) / len > 8192) len *= 2;
  return (int)len;
}
inline int perm_num_chunks(int64_t N) {
  int len = perm_chunk_len(N);
  return (int)((N + len - 1) / len);
}

}  // namespace moga
