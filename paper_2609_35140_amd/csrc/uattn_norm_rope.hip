// Q/K RMSNorm + NeoX rotary embedding (one pass), and its rotary table.
//
// A workgroup takes one token's head rows; one row of head_dim bf16 is
// handled by head_dim/8 lanes, 16 bytes (8 elements) each.  The sum of squares
// is summed by each lane over its 8 elements in order, then across the row's
// lanes by an xor butterfly, so every lane of the row holds the same total
// computed in one fixed order.  NeoX pairs element i with i + head_dim/2,
// which lives in the lane head_dim/16 positions away; the two exchange their
// normalized values.  Nothing depends on how many rows
// there are or where a row sits, so the full-sequence and token-wise regimes
// produce identical rows.
#include <math.h>

#include <type_traits>

#include "uattn_internal.h"
#include "uattn_numerics.h"

namespace uattn {
namespace {

struct NormRopeParams {
  const __bf16* q;
  const __bf16* k;
  const int32_t* positions;
  const __bf16* qw;
  const __bf16* kw;
  const float* cos_sin;
  __bf16* q_out;
  __bf16* k_out;
  float eps;
  int32_t max_position, num_tokens, hq, hkv;
  int32_t first;  // tokens of the launches before this one
};

// DPP: lanes exchange values within 16 without an LDS round trip.  Every lane
// of the patterns below has a source lane.
template <int ctrl>
__device__ __forceinline__ float dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), ctrl, 0xF, 0xF, true));
}
constexpr int kRowRor = 0x120;                 // + n: rotate 16 lanes by n
constexpr int kQuadSwap2 = 0x4E, kQuadSwap1 = 0xB1;  // lane ^ 2, lane ^ 1
constexpr int kQuadBroadcast = 0x55;           // * n: lane n of each 4
// The value of lane j ^ n, n = LPR / 2 (half a row of D elements).
template <int n>
__device__ __forceinline__ float lane_xor(float x) {
  static_assert(n == 4 || n == 8, "half a row of 64 or 128 elements");
  if constexpr (n == 8) {
    return dpp<kRowRor + 8>(x);
  } else {
    // lanes with bit 2 clear from j + 4 (row_shl:4), the others from j - 4 (row_shr:4)
    const uint32_t u = __float_as_uint(x);
    const uint32_t up = __builtin_amdgcn_update_dpp(u, u, 0x104, 0xF, 0x5, false);
    return __uint_as_float(__builtin_amdgcn_update_dpp(up, u, 0x114, 0xF, 0xA, false));
  }
}
// Sum over the LPR lanes of a row by an xor butterfly from the largest distance
// down.  After distance n the sums repeat with period n, so a rotation by n/2
// reads the same value as lane j ^ n/2.
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
  x = x + lane_xor<LPR / 2>(x);
  if constexpr (LPR == 16) x = x + dpp<kRowRor + 4>(x);
  x = x + dpp<kQuadSwap2>(x);
  return x + dpp<kQuadSwap1>(x);
}

// Two values rounded to bf16 by one instruction.
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ void round_pairs(float (&y)[8]) {
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const uint32_t w = bf16_pair(y[e], y[e + 1]);
    y[e] = __uint_as_float(w << 16);
    y[e + 1] = __uint_as_float(w & 0xFFFF0000u);
  }
}

// One workgroup per token (its position and rotary row are uniform); an item is
// the 64 / (head_dim/8) head rows of q or of k that one wave handles at a time,
// and the four waves take the token's items in turn, kAhead of them at once.
//
// Bound by memory, with the vector instructions close behind (a wave instruction
// takes a SIMD about four cycles, an item some 130 of them), so: values pass
// between lanes as DPP operands of the instructions that use them; the sign of
// the NeoX pair sits in the sine; the weights are unpacked once; one square
// root and division serve kAhead items, each in its own lane of four; and the
// rows of kAhead items are requested before the first is used.
// 39,855 tokens, 32/8 heads, d = 128: 168 us with about 230 instructions, LDS
// shuffles and a pass at a time, 163 with the loads ahead alone, 140 so (5.8 TB/s);
// one token 4.1 -> 2.8 us.  A token of fewer items is handled by as many as its
// waves have (launch_qk_norm_rope): 9818 tokens, 12/12 heads, d = 64 (one to a wave)
// 21.7 us as three, 19.2 as one.
constexpr int kNormWaves = 4;
template <int D, int kAhead>
__global__ __launch_bounds__(kNormWaves * 64) void qk_norm_rope_kernel(NormRopeParams p) {
  constexpr int LPR = D / 8;          // lanes per row
  constexpr int RPI = 64 / LPR;       // rows per item
  constexpr int HALF = LPR / 2;       // lane distance of a NeoX pair
  static_assert(kAhead <= 4, "an item's reciprocal in its own lane of four");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane % LPR;           // 16-byte piece of the row
  const bool first = j < HALF;
  const int i0 = 8 * (first ? j : j - HALF);  // rotary index of element 0 of this lane
  const int64_t t = p.first + blockIdx.x;
  const int q_items = (p.hq + RPI - 1) / RPI, items = q_items + (p.hkv + RPI - 1) / RPI;
  if (wave >= items) return;
  const int32_t pos = p.positions[t];

  bf16x8 xs[kAhead] = {};
  // row of this lane in item `it`, counted in its own matrix
  auto row_of = [&](int it) { return (it < q_items ? it : it - q_items) * RPI + lane / LPR; };
  auto load = [&](int it0) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int it = it0 + u * kNormWaves, r = row_of(it);
      const bool is_q = it < q_items;
      const int heads = is_q ? p.hq : p.hkv;
      // lanes past the last head read it again (not written)
      if (it < items)
        xs[u] = *reinterpret_cast<const bf16x8*>((is_q ? p.q : p.k) + t * heads * D + min(r, heads - 1) * D + 8 * j);
    }
  };
  load(wave);
  float wq[8], wk[8];
  {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(p.qw + 8 * j), b = *reinterpret_cast<const bf16x8*>(p.kw + 8 * j);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      wq[e] = static_cast<float>(a[e]);
      wk[e] = static_cast<float>(b[e]);
    }
  }
  // cosines, and the sines with the sign they get in this lane's half: the first
  // half of a row is y c - z s, the second y c + z s, z the partner's value
  float cosv[8], sinv[8];
  if (pos >= 0 && pos < p.max_position) {
    const float4* cp = reinterpret_cast<const float4*>(p.cos_sin + (static_cast<int64_t>(pos) * (D / 2) + i0) * 2);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float4 v4 = cp[u];
      cosv[2 * u] = v4.x;
      cosv[2 * u + 1] = v4.z;
      sinv[2 * u] = first ? -v4.y : v4.y;
      sinv[2 * u + 1] = first ? -v4.w : v4.w;
    }
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) cosv[u] = sinv[u] = __builtin_nanf("");
  }
  for (int it0 = wave;;) {
    float ss[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      ss[u] = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = static_cast<float>(xs[u][e]);
        ss[u] = ss[u] + x * x;
      }
      ss[u] = row_sum<LPR>(ss[u]);
    }
    float mine = ss[0];
#pragma unroll
    for (int u = 1; u < kAhead; ++u) mine = (lane & 3) == u ? ss[u] : mine;
    const float r_mine = 1.0f / __builtin_sqrtf(mine / static_cast<float>(D) + p.eps);
    float r_inv[kAhead];
    r_inv[0] = dpp<0>(r_mine);
    if constexpr (kAhead > 1) r_inv[1] = dpp<kQuadBroadcast>(r_mine);
    if constexpr (kAhead > 2) r_inv[2] = dpp<2 * kQuadBroadcast>(r_mine);
    if constexpr (kAhead > 3) r_inv[3] = dpp<3 * kQuadBroadcast>(r_mine);
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int it = it0 + u * kNormWaves;
      if (it >= items) break;
      const bool is_q = it < q_items;
      float y[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = static_cast<float>(xs[u][e]) * r_inv[u];
      round_pairs(y);
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = (is_q ? wq[e] : wk[e]) * y[e];
      round_pairs(y);
      u32x4 ov;
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = y[e] * cosv[e] + lane_xor<HALF>(y[e]) * sinv[e];
#pragma unroll
      for (int e = 0; e < 4; ++e) ov[e] = bf16_pair(y[2 * e], y[2 * e + 1]);
      // keeps the products here: moved into the branch below they could not
      // take the other lanes' values as DPP operands
      asm volatile("" : "+v"(ov));
      const int r = row_of(it), heads = is_q ? p.hq : p.hkv;
      if (r < heads) *reinterpret_cast<u32x4*>((is_q ? p.q_out : p.k_out) + t * heads * D + r * D + 8 * j) = ov;
    }
    it0 += kAhead * kNormWaves;
    if (it0 >= items) break;
    load(it0);
  }
}

__global__ __launch_bounds__(256) void rope_cache_kernel(float* cos_sin, int32_t max_position, int32_t d, double theta) {
  const int64_t n = static_cast<int64_t>(max_position) * (d / 2);
  for (int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; idx < n;
       idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t pos = idx / (d / 2);
    const int i = static_cast<int>(idx % (d / 2));
    const double inv_freq = pow(theta, -2.0 * i / d);
    const double ang = static_cast<double>(pos) * inv_freq;
    cos_sin[2 * idx] = static_cast<float>(cos(ang));
    cos_sin[2 * idx + 1] = static_cast<float>(sin(ang));
  }
}

}  // namespace

hipError_t launch_qk_norm_rope(const NormRopeLaunch& a, hipStream_t stream) {
  NormRopeParams p;
  p.q = static_cast<const __bf16*>(a.q);
  p.k = static_cast<const __bf16*>(a.k);
  p.positions = a.positions;
  p.qw = static_cast<const __bf16*>(a.q_weight);
  p.kw = static_cast<const __bf16*>(a.k_weight);
  p.cos_sin = a.cos_sin;
  p.q_out = static_cast<__bf16*>(a.q_out);
  p.k_out = static_cast<__bf16*>(a.k_out);
  p.eps = a.eps;
  p.max_position = a.max_position;
  p.num_tokens = a.num_tokens;
  p.hq = a.num_q_heads;
  p.hkv = a.num_kv_heads;
  // one workgroup per token
  return launch_parts(a.num_tokens, kNormWaves * 64, [&](int first, unsigned n) {
    p.first = first;
    auto launch = [&](auto d_const, auto ahead_const) {
      hipLaunchKernelGGL((qk_norm_rope_kernel<decltype(d_const)::value, decltype(ahead_const)::value>), dim3(n),
                         dim3(kNormWaves * 64), 0, stream, p);
    };
    auto pick = [&](auto d_const) {
      constexpr int kRows = 64 / (decltype(d_const)::value / 8);  // of an item
      const int items = (p.hq + kRows - 1) / kRows + (p.hkv + kRows - 1) / kRows;
      if (items <= kNormWaves)
        launch(d_const, std::integral_constant<int, 1>{});
      else if (items <= 2 * kNormWaves)
        launch(d_const, std::integral_constant<int, 2>{});
      else
        launch(d_const, std::integral_constant<int, 3>{});
    };
    if (a.head_dim == 128)
      pick(std::integral_constant<int, 128>{});
    else
      pick(std::integral_constant<int, 64>{});
  });
}

hipError_t launch_rope_cache(float* cos_sin, int32_t max_position, int32_t head_dim, double theta, hipStream_t stream) {
  const int64_t n = static_cast<int64_t>(max_position) * (head_dim / 2);
  const int64_t want = (n + 255) / 256;
  const int64_t cap = static_cast<int64_t>(device_cus()) * 16;
  hipLaunchKernelGGL(rope_cache_kernel, dim3(static_cast<unsigned>(want < cap ? want : cap)), dim3(256), 0, stream,
                     cos_sin, max_position, head_dim, theta);
  return hipGetLastError();
}

}  // namespace uattn
