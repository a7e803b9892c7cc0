// Per-token log-probability: logp = x[y] - logsumexp(x), x = logits * inv_temperature.
//
// One workgroup (1024 threads) per row.  Thread t streams the row's 16-byte
// vectors t, t+1024, t+2048, ... in batches, keeping an online (max, sum) pair;
// the 1024 pairs are then combined by a fixed butterfly inside each wave and a
// fixed pairing of the waves.  The reduction structure depends only on vocab,
// never on the number of rows or a row's position, so a row's result is
// bit-identical in any batch (the precondition for reusing rollout
// log-probabilities with ratio exactly 1).
//
// The temperature is folded into the exponent: with k = inv_temperature *
// log2(e) and m the row max of the raw logits (inv_temperature > 0),
//   sum = sum_v exp2(fma(logit_v, k, -m*k)),
//   logp = (logit_y - m) * inv_temperature - log2(sum) * ln(2).
#include "uattn_internal.h"
#include "uattn_numerics.h"

#pragma clang fp contract(off)

namespace uattn {
namespace {

// A row is one workgroup's, so few rows (a decode step) leave most CUs idle and
// what counts is how fast one CU streams: 16 waves with kBatch loads each in
// flight.  8 rows of 151,936: 35 us with 256 threads and one load in flight, 17.6
// with 256 x 8, 13.6 with 512 x 5, 12.7 so; 8192 rows 403 -> 391 us (6.4 TB/s).
constexpr int kThreads = 1024;
constexpr int kBatch = 5;  // 16-byte loads in flight per thread

struct MaxSum {
  float m, s;
};

// Factor that moves a sum kept relative to max `from` to max `to` (to >= from).
__device__ __forceinline__ float rebase(float from, float to, float k) {
  return from == neg_inf() ? 0.f : hw_exp2(from * k - to * k);
}

__device__ __forceinline__ MaxSum combine(MaxSum a, MaxSum b, float k) {
  MaxSum r;
  r.m = fmaxf(a.m, b.m);
  r.s = a.s * rebase(a.m, r.m, k) + b.s * rebase(b.m, r.m, k);
  return r;
}

constexpr u32x4 kNegInfVec = {0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u};  // eight bf16 -inf
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__global__ __launch_bounds__(kThreads) void logprob_kernel(const uint16_t* __restrict__ logits, int64_t stride,
                                                           const int32_t* __restrict__ targets, int vocab, float it,
                                                           float k, int first, float* __restrict__ logp) {
  const int row = first + blockIdx.x, tid = threadIdx.x;
  const uint16_t* x = logits + static_cast<int64_t>(row) * stride;
  MaxSum acc{neg_inf(), 0.f};
  const int nvec = vocab / 8;
  for (int i0 = tid; i0 < nvec; i0 += kBatch * kThreads) {
    u32x4 w[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int i = i0 + b * kThreads;
      w[b] = i < nvec ? *reinterpret_cast<const u32x4*>(x + 8 * static_cast<int64_t>(i)) : kNegInfVec;
    }
    float m_new = acc.m;
#pragma unroll
    for (int b = 0; b < kBatch; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j) m_new = fmaxf(m_new, fmaxf(bf16_lo(w[b][j]), bf16_hi(w[b][j])));
    // entries of -inf (a masked vocabulary) add nothing, also where all so far are -inf
    const float mk = m_new == neg_inf() ? 0.f : m_new * k;
    float sum = 0.f;
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      float e[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        e[2 * j] = hw_exp2(__builtin_fmaf(bf16_lo(w[b][j]), k, -mk));
        e[2 * j + 1] = hw_exp2(__builtin_fmaf(bf16_hi(w[b][j]), k, -mk));
      }
      sum = sum + (((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7])));
    }
    acc.s = acc.s * rebase(acc.m, m_new, k) + sum;
    acc.m = m_new;
  }
  for (int i = 8 * nvec + tid; i < vocab; i += kThreads)
    acc = combine(acc, MaxSum{__uint_as_float(static_cast<uint32_t>(x[i]) << 16), 1.f}, k);
  // wave butterfly (combine is commutative, so every lane ends with the same pair)
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    MaxSum o{__shfl_xor(acc.m, off, 64), __shfl_xor(acc.s, off, 64)};
    acc = combine(acc, o, k);
  }
  __shared__ MaxSum part[kThreads / 64];
  if ((tid & 63) == 0) part[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    // the waves' pairs, neighbours first
#pragma unroll
    for (int n = 1; n < kThreads / 64; n *= 2)
#pragma unroll
      for (int w = 0; w < kThreads / 64; w += 2 * n) part[w] = combine(part[w], part[w + n], k);
    const MaxSum r = part[0];
    const int y = targets[row];
    if (y < 0 || y >= vocab) {
      logp[row] = __builtin_nanf("");
    } else {
      const float xy = __uint_as_float(static_cast<uint32_t>(x[y]) << 16);
      logp[row] = (xy - r.m) * it - hw_log2(r.s) * 0.69314718055994530942f;
    }
  }
}

}  // namespace

hipError_t launch_logprob(const LogprobLaunch& a, hipStream_t stream) {
  const float k = static_cast<float>(static_cast<double>(a.inv_temperature) * 1.4426950408889634);
  return launch_parts(a.num_rows, kThreads, [&](int first, unsigned n) {
    hipLaunchKernelGGL(logprob_kernel, dim3(n), dim3(kThreads), 0, stream, static_cast<const uint16_t*>(a.logits),
                       a.row_stride, a.targets, a.vocab, a.inv_temperature, k, first, a.logp);
  });
}

}  // namespace uattn
