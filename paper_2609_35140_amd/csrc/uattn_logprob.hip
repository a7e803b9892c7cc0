// Per-token log-probability: logp = x[y] - logsumexp(x), x = logits * inv_temperature.
//
// One workgroup per row, of 64 to 1024 threads by the vocabulary (launch_logprob).
// Thread t streams the row's 16-byte vectors t, t+threads, t+2*threads, ... in
// batches, keeping an online (max, sum) pair; the pairs are then combined by a
// fixed butterfly inside each wave and a fixed pairing of the waves.  The reduction
// structure depends only on vocab, never on the number of rows or a row's
// position, so a row's result is bit-identical in any batch (the precondition for
// reusing rollout log-probabilities with ratio exactly 1).
//
// The temperature is folded into the exponent: with k = inv_temperature *
// log2(e) and m the row max of the raw logits (inv_temperature > 0),
//   sum = sum_v exp2(fma(logit_v, k, -m*k)),
//   logp = (logit_y - m) * inv_temperature - log2(sum) * ln(2).
#include <type_traits>

#include "uattn_internal.h"
#include "uattn_numerics.h"

#pragma clang fp contract(off)

namespace uattn {
namespace {

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

// kBatch 16-byte loads in flight per thread; a batch's loads past the row's end are
// skipped by the wave, and those of its last vector's wave read as -inf.
template <int kThreads, int kBatch>
__global__ __launch_bounds__(kThreads) void logprob_kernel(const uint16_t* __restrict__ logits, int64_t stride,
                                                           const int32_t* __restrict__ targets, int vocab, float it,
                                                           float k, int first, float* __restrict__ logp) {
  constexpr int kWaves = kThreads / 64;
  const int row = first + blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint16_t* x = logits + static_cast<int64_t>(row) * stride;
  const int y = targets[row];
  MaxSum acc{neg_inf(), 0.f};
  const int nvec = vocab / 8;
  for (int i0 = 64 * wave; i0 < nvec; i0 += kBatch * kThreads) {
    u32x4 w[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      const int i = i0 + b * kThreads + lane;
      w[b] = kNegInfVec;
      if (i < nvec) w[b] = *reinterpret_cast<const u32x4*>(x + 8 * static_cast<int64_t>(i));
    }
    float m_new = acc.m;
#pragma unroll
    for (int b = 0; b < kBatch; ++b)
      if (i0 + b * kThreads < nvec)
#pragma unroll
        for (int j = 0; j < 4; ++j) m_new = fmaxf(m_new, fmaxf(bf16_lo(w[b][j]), bf16_hi(w[b][j])));
    // entries of -inf (a masked vocabulary) add nothing, also where all so far are -inf
    const float mk = m_new == neg_inf() ? 0.f : m_new * k;
    float sum = 0.f;
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      if (i0 + b * kThreads >= nvec) break;
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
  MaxSum part[kWaves];
  part[0] = acc;
  if constexpr (kWaves > 1) {
    __shared__ MaxSum all[kWaves];
    if (lane == 0) all[wave] = acc;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) part[w] = all[w];
  }
  if (tid == 0) {
    // the waves' pairs, neighbours first
#pragma unroll
    for (int n = 1; n < kWaves; n *= 2)
#pragma unroll
      for (int w = 0; w < kWaves; w += 2 * n) part[w] = combine(part[w], part[w + n], k);
    const MaxSum r = part[0];
    if (y < 0 || y >= vocab) {
      logp[row] = __builtin_nanf("");
    } else {
      const float xy = __uint_as_float(static_cast<uint32_t>(x[y]) << 16);
      logp[row] = (xy - r.m) * it - hw_log2(r.s) * 0.69314718055994530942f;
    }
  }
}

}  // namespace

// Threads to a row by the vocabulary alone (a row's bits do not depend on the
// number of rows).  Few rows (a decode step) leave most CUs idle, so what counts
// there is how fast one CU streams a row, many loads in flight; many rows
// want no idle waves, whose launch and reduction cost as much as a busy one's.  us
// for 8 and for 8192 rows (vocab 1000 and 2048: 65536), by threads x batch:
//   1,000     64 x 4   2.7 / 28     256 x 1   2.8 / 63     1024 x 5   3.5 / 283
//   2,048    128 x 4   2.9 / 52     256 x 4   2.9 / 81      64 x 4    3.1 / 45
//   16,384   256 x 4   4.0 / 40.7   512 x 5   3.8 / 41.6   1024 x 5   4.3 / 56
//   28,000   256 x 4   5.2 / 79     512 x 5   4.6 / 82     256 x 1   5.6 / 78
//   32,000   512 x 5   4.9 / 89.5   256 x 4   5.5 / 90.5   256 x 1   6.2 / 90
//   50,257   512 x 5   6.2 / 135    256 x 4   7.4 / 142    1024 x 5   6.3 / 147
//   151,936 1024 x 5  11.5 / 407    512 x 5  12.4 / 412     256 x 1  19 / 424
// The vectors of a thread stay between one and about twenty.
hipError_t launch_logprob(const LogprobLaunch& a, hipStream_t stream) {
  const float k = static_cast<float>(static_cast<double>(a.inv_temperature) * 1.4426950408889634);
  auto launch = [&](auto threads_const, auto batch_const) {
    constexpr int kThreads = decltype(threads_const)::value, kBatch = decltype(batch_const)::value;
    return launch_parts(a.num_rows, kThreads, [&](int first, unsigned n) {
      hipLaunchKernelGGL((logprob_kernel<kThreads, kBatch>), dim3(n), dim3(kThreads), 0, stream,
                         static_cast<const uint16_t*>(a.logits), a.row_stride, a.targets, a.vocab, a.inv_temperature, k,
                         first, a.logp);
    });
  };
  using std::integral_constant;
  if (a.vocab <= 1024) return launch(integral_constant<int, 64>{}, integral_constant<int, 4>{});
  if (a.vocab <= 3072) return launch(integral_constant<int, 128>{}, integral_constant<int, 4>{});
  if (a.vocab <= 28672) return launch(integral_constant<int, 256>{}, integral_constant<int, 4>{});
  if (a.vocab <= 65536) return launch(integral_constant<int, 512>{}, integral_constant<int, 5>{});
  return launch(integral_constant<int, 1024>{}, integral_constant<int, 5>{});
}

}  // namespace uattn
