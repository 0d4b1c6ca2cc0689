// Group balancing loss of MoGA (Eqs. 6-8 of the paper) and its gradient with respect to the gate.
//
//   F_i = (1/N) #{x : g(x) = i}                      fraction of tokens assigned to group i (Eq. 7)
//   P_i = (1/N) sum_{x : g(x) = i} p(g(x) | x)       router probability mass of those tokens (Eq. 8)
//   L   = alpha * M * sum_i F_i * P_i                (Eq. 6)
//
// The per-group sums are accumulated as integers (counts, and gates in 2^-32 fixed point), so
// the result does not depend on the order in which tokens are added: LDS atomics per block,
// then one global atomic per block and group.  A last block turns the sums into F, P and L in
// double precision.  F is piecewise constant in the router weights, so the gradient flows through
// P only: dL/d gate[x] = alpha * M * F_{g(x)} / N.
#include <algorithm>

#include "moga_common.h"

namespace moga {

constexpr double kGateFixedScale = 4294967296.0;   // 2^32

struct BalanceAcc {
  unsigned long long gate_sum;   // sum of round(gate * 2^32), two's complement
  unsigned long long count;
};

// Sums of the tokens t, t + stride, ... of every thread, in LDS.  COPIES per group, for the lanes in turn: lanes that add to one
// word do so one after the other.
template <int COPIES>
__device__ __forceinline__ void balance_sums(const int32_t* __restrict__ group, const float* __restrict__ gate, int64_t N, int M,
                                             int64_t t, int64_t stride, unsigned long long* s_sum, unsigned int* s_cnt) {
  for (int j = threadIdx.x; j < M * COPIES; j += blockDim.x) { s_sum[j] = 0ull; s_cnt[j] = 0u; }
  __syncthreads();
  for (; t < N; t += stride) {
    const int g = group[t];
    if (g >= 0 && g < M) {
      const long long fx = __double2ll_rn((double)gate[t] * kGateFixedScale);
      const int w = g * COPIES + threadIdx.x % COPIES;
      atomicAdd(&s_sum[w], (unsigned long long)fx);
      atomicAdd(&s_cnt[w], 1u);
    }
  }
  __syncthreads();
}

// F, P and L from the sums, by one block.
__device__ __forceinline__ void balance_result(unsigned long long gate_sum, unsigned long long count, int j, double inv_n, double* s_fp,
                                               float* __restrict__ frac, float* __restrict__ prob) {
  const double f = (double)count * inv_n;
  const double p = (double)(long long)gate_sum / kGateFixedScale * inv_n;
  frac[j] = (float)f;
  prob[j] = (float)p;
  s_fp[j] = f * p;
}
__device__ __forceinline__ void balance_loss_value(const double* s_fp, int M, float alpha, float* __restrict__ loss) {
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int j = 0; j < M; ++j) s += s_fp[j];
    loss[0] = (float)((double)alpha * (double)M * s);
  }
}

__global__ __launch_bounds__(256) void balance_accumulate_kernel(
    const int32_t* __restrict__ group, const float* __restrict__ gate, int64_t N, int M,
    BalanceAcc* __restrict__ acc) {
  __shared__ unsigned long long s_sum[MOGA_MAX_GROUPS];
  __shared__ unsigned int s_cnt[MOGA_MAX_GROUPS];
  balance_sums<1>(group, gate, N, M, (int64_t)blockIdx.x * 256 + threadIdx.x, (int64_t)gridDim.x * 256, s_sum, s_cnt);
  for (int j = threadIdx.x; j < M; j += 256) {
    if (s_cnt[j]) {
      atomicAdd(&acc[j].gate_sum, s_sum[j]);
      atomicAdd(&acc[j].count, (unsigned long long)s_cnt[j]);
    }
  }
}

__global__ __launch_bounds__(256) void balance_finalize_kernel(
    const BalanceAcc* __restrict__ acc, int64_t N, int M, float alpha, float* __restrict__ loss,
    float* __restrict__ frac, float* __restrict__ prob) {
  __shared__ double s_fp[MOGA_MAX_GROUPS];
  const double inv_n = 1.0 / (double)N;
  for (int j = threadIdx.x; j < M; j += 256) balance_result(acc[j].gate_sum, acc[j].count, j, inv_n, s_fp, frac, prob);
  balance_loss_value(s_fp, M, alpha, loss);
}

// All of it in one block for up to kBalanceOneBlock tokens, where the three launches (fill, accumulate, finalize) cost more than
// the work.  The same integers, so the same bits.  With one sum per group, tokens that all chose one group were added one after the
// other by this block alone (8,192 tokens 16.0 us, with eight sums 4.4, by the three launches 7.3; 4,096: 9.1, 3.5 and 7.3; evenly
// over 8 groups 8,192 take 4.4 and 6.5).
constexpr int64_t kBalanceOneBlock = 8192;
constexpr int kBalanceCopies = 8;
__global__ __launch_bounds__(1024) void balance_one_block_kernel(
    const int32_t* __restrict__ group, const float* __restrict__ gate, int64_t N, int M, float alpha, float* __restrict__ loss,
    float* __restrict__ frac, float* __restrict__ prob) {
  __shared__ unsigned long long s_sum[MOGA_MAX_GROUPS * kBalanceCopies];
  __shared__ unsigned int s_cnt[MOGA_MAX_GROUPS * kBalanceCopies];
  __shared__ double s_fp[MOGA_MAX_GROUPS];
  balance_sums<kBalanceCopies>(group, gate, N, M, threadIdx.x, 1024, s_sum, s_cnt);
  const double inv_n = 1.0 / (double)N;
  for (int j = threadIdx.x; j < M; j += 1024) {
    unsigned long long sum = 0ull;
    unsigned int cnt = 0u;
#pragma unroll
    for (int k = 0; k < kBalanceCopies; ++k) {
      sum += s_sum[j * kBalanceCopies + k];
      cnt += s_cnt[j * kBalanceCopies + k];
    }
    balance_result(sum, cnt, j, inv_n, s_fp, frac, prob);
  }
  balance_loss_value(s_fp, M, alpha, loss);
}

__global__ __launch_bounds__(256) void balance_bwd_kernel(
    const int32_t* __restrict__ group, const float* __restrict__ frac, int64_t N, int M, float coef,
    const float* __restrict__ d_loss_dev, int accumulate, float* __restrict__ d_gate) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= N) return;
  if (d_loss_dev) coef *= d_loss_dev[0];   // upstream gradient kept on the device: no host synchronisation
  const int g = group[t];
  const float v = (g >= 0 && g < M) ? coef * frac[g] : 0.f;
  d_gate[t] = accumulate ? d_gate[t] + v : v;
}

}  // namespace moga

using namespace moga;

extern "C" size_t moga_balance_ws_bytes(int M) { return (size_t)M * sizeof(BalanceAcc); }

extern "C" int moga_balance_loss(const int32_t* group, const float* gate, int64_t N, int M,
                                 float alpha, float* loss, float* frac, float* prob, void* ws,
                                 size_t ws_bytes, void* stream) {
  if (N < 0 || M < 1) return MOGA_ERR_INVALID_ARG;
  if (M > MOGA_MAX_GROUPS || N >= ((int64_t)1 << 31)) return MOGA_ERR_UNSUPPORTED;
  if (!loss || !frac || !prob) return MOGA_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (N == 0) {   // no tokens: F = P = 0, L = 0
    launch_fill_zero(frac, M, st);
    launch_fill_zero(prob, M, st);
    launch_fill_zero(loss, 1, st);
    return launch_status();
  }
  if (!group || !gate) return MOGA_ERR_INVALID_ARG;
  if (!ws || ws_bytes < moga_balance_ws_bytes(M)) return MOGA_ERR_WORKSPACE;
  if (!aligned16(ws)) return MOGA_ERR_INVALID_ARG;
  if (N <= kBalanceOneBlock) {
    balance_one_block_kernel<<<1, 1024, 0, st>>>(group, gate, N, M, alpha, loss, frac, prob);
    return launch_status();
  }
  BalanceAcc* acc = (BalanceAcc*)ws;
  const int64_t ws_floats = (int64_t)(moga_balance_ws_bytes(M) / sizeof(float));
  launch_fill_zero((float*)ws, ws_floats, st);
  const unsigned blocks = (unsigned)std::min<int64_t>(1024, (N + 1023) / 1024);
  balance_accumulate_kernel<<<blocks, 256, 0, st>>>(group, gate, N, M, acc);
  balance_finalize_kernel<<<1, 256, 0, st>>>(acc, N, M, alpha, loss, frac, prob);
  return launch_status();
}

extern "C" int moga_balance_loss_bwd(const int32_t* group, const float* frac, int64_t N, int M,
                                     float alpha, float d_loss, const float* d_loss_device_or_null,
                                     int accumulate, float* d_gate, void* stream) {
  if (N < 0 || M < 1) return MOGA_ERR_INVALID_ARG;
  if (M > MOGA_MAX_GROUPS || N >= ((int64_t)1 << 31)) return MOGA_ERR_UNSUPPORTED;
  if (N == 0) return MOGA_OK;
  if (!group || !frac || !d_gate) return MOGA_ERR_INVALID_ARG;
  const float coef = (float)((double)d_loss * (double)alpha * (double)M / (double)N);
  balance_bwd_kernel<<<(unsigned)((N + 255) / 256), 256, 0, (hipStream_t)stream>>>(
      group, frac, N, M, coef, d_loss_device_or_null, accumulate, d_gate);
  return launch_status();
}
