// Batch-invariant LM head: logits = bf16(hidden . weight^T).
//
// Each MFMA computes a 16 (vocab) x 16 (token) block of logits^T = W H^T, so
// a lane's four results are four consecutive vocab entries of one token (one
// 8-byte store).  Workgroup = 8 waves = 256 vocab rows x 256 tokens (smaller
// tiles for few tokens, see launch_rows); wave
// (wm, wn) owns 64 vocab x 128 tokens (4 x 8 blocks), so each 16-byte LDS
// operand read feeds 4 or 8 MFMAs.  K (the hidden dimension) is walked in
// 64-wide chunks (up to 256-wide in the small tiles) through a two-stage LDS ring
// filled by direct-to-LDS loads
// (16-byte pieces XOR-swizzled by row, so the lanes of an operand read's
// LDS cycle hit distinct banks), and every accumulator steps K in ascending 32-wide MFMA
// steps from zero: a row's logits never depend on the batch, its size or the
// row's place in a tile.
//
// Workgroup order: the hardware deals consecutive ids to the 8 XCDs in turn;
// id -> (vocab tile, token tile) keeps one vocab tile's weights (2 MB for
// hidden 4096) on one XCD while all token tiles pass, so they stay in that
// XCD's L2 and the hidden rows stream from the shared cache.
//
// Fused log-probability epilogue (uattn_lm_head_logprob): instead of (or as
// well as) storing the bf16 logits, the workgroup reduces each token's 256
// logits of its vocab tile to a partial (max, sum of exp) pair and picks out
// the target's logit when the target lies in the tile; a second kernel folds
// each token's partials in 16 runs of consecutive vocab tiles, ascending inside a
// run, then run by run.  Every reduction has a structure fixed by vocab positions
// alone (lane, wave, tile and run order), so a token's result does not depend on
// the batch or its place in it.
#include <type_traits>

#include "uattn_internal.h"
#include "uattn_numerics.h"
#include "uattn_tile_io.h"

namespace uattn {
namespace {

constexpr int kVocabTile = 256;  // vocab rows of a workgroup, and of a log-prob partial
constexpr int kLmXcds = 8;

struct LmHeadParams {
  const __bf16* h;
  const __bf16* w;
  __bf16* out;          // logits, or nullptr (fused log-prob without stored logits)
  int64_t hs, ws, os;
  int32_t T, V, K, n_vt, n_tt;
  int32_t first;        // workgroups of the launches before this one
  // fused log-prob epilogue
  const int32_t* targets;
  float* part_m;        // [n_vt][T] tile max of the raw bf16 logits
  float* part_s;        // [n_vt][T] sum over the tile of exp2(fma(x, k, -m*k))
  float* y_logit;       // [T] the target's raw bf16 logit
  float k;              // inv_temperature * log2(e)
};

// VT vocab rows x TT tokens per workgroup, WM x WN waves (wave tile
// VT/WM x TT/WN), a ring of STAGES chunks of kKC hidden elements.
template <int VT, int TT, int WM, int WN, int STAGES, int kKC>
struct LmCfg {
  static constexpr int kPieces = kKC / 8;  // 16-byte pieces of a row's chunk
  // pieces are XOR-swizzled by row so that the lanes of an LDS cycle hit distinct banks
  __device__ __forceinline__ static int swz(int row) { return row & (kPieces - 1) & 15; }
  static constexpr int NW = WM * WN;       // waves per workgroup
  static constexpr int BI = VT / WM / 16;   // 16-row vocab blocks per wave
  static constexpr int BJ = TT / WN / 16;   // 16-column token blocks per wave
  static constexpr int kAInstr = VT * kKC * 2 / 1024 / NW;  // 1 KB direct-to-LDS loads per wave per chunk
  static constexpr int kBInstr = TT * kKC * 2 / 1024 / NW;
  static_assert(kAInstr * 1024 * NW == VT * kKC * 2 && kBInstr * 1024 * NW == TT * kKC * 2, "chunk split");
  static constexpr int kChunkOps = kAInstr + kBInstr;
  struct Smem {
    __bf16 a[STAGES][VT * kKC];   // weight rows, kKC elements each, pieces swizzled
    __bf16 b[STAGES][TT * kKC];   // hidden rows
  };
};

// What becomes of a workgroup's accumulators: the bf16 logits (if p.out), and
// the log-prob partials of its vocab tile.  `red`: LDS of the K loop.
template <int VT, int TT, int WM, int WN, bool kLogprob>
__device__ __forceinline__ void lm_head_epilogue(const LmHeadParams& p, const f32x4 (&acc)[VT / WM / 16][TT / WN / 16],
                                                 float* red /* [WM][TT] per-wave maxima, then sums */,
                                                 const int (&ytgt)[kLogprob ? TT / WN / 16 : 1], int v0, int t0, int vt,
                                                 int tid) {
  constexpr int BI = VT / WM / 16, BJ = TT / WN / 16;
  const int lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM;
  // lane: token 16j + r16 of the wave's columns, vocab 16i + 4g .. +3 of its rows
  if (p.out != nullptr) {
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int t = t0 + (TT / WN) * wn + 16 * j + r16;
      if (t >= p.T) continue;
      __bf16* orow = p.out + static_cast<int64_t>(t) * p.os;
#pragma unroll
      for (int i = 0; i < BI; ++i) {
        const int v = v0 + (VT / WM) * wm + 16 * i + 4 * g;
        bf16x4 o;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) o[jj] = to_bf16(acc[i][j][jj]);
        if (v + 3 < p.V) {
          *reinterpret_cast<bf16x4*>(orow + v) = o;
        } else {
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
            if (v + jj < p.V) orow[v + jj] = o[jj];
        }
      }
    }
  }
  if constexpr (kLogprob) {
    static_assert(VT == 256 && WM == 4 && TT <= 256, "reduction layout: four waves of 64 vocab entries");
    // the K loop's LDS is free once every wave is past its last chunk
    lds_barrier();
    const float k = p.k;
    // x = the stored bf16 logit (raw; the temperature sits in k), -inf past the vocabulary
    float x[BJ][BI][4];
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int tl = (TT / WN) * wn + 16 * j + r16;
      const int t = t0 + tl;
      const int y = ytgt[j];
#pragma unroll
      for (int i = 0; i < BI; ++i) {
        const int v = v0 + (VT / WM) * wm + 16 * i + 4 * g;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const float xv = static_cast<float>(to_bf16(acc[i][j][jj]));
          x[j][i][jj] = (v + jj < p.V) ? xv : neg_inf();
          if (v + jj == y) p.y_logit[t] = xv;
        }
      }
      // the wave's maximum over its 64 entries of this token (max is exact: any order)
      float mx = neg_inf();
#pragma unroll
      for (int i = 0; i < BI; ++i) mx = vmax(vmax(mx, vmax(x[j][i][0], x[j][i][1])), vmax(x[j][i][2], x[j][i][3]));
      mx = max_xor32(max_xor16(mx));
      if (g == 0) red[wm * TT + tl] = mx;
    }
    lds_barrier();
    float m_tile[BJ];
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int tl = (TT / WN) * wn + 16 * j + r16;
      m_tile[j] = vmax(vmax(red[tl], red[TT + tl]), vmax(red[2 * TT + tl], red[3 * TT + tl]));
    }
    lds_barrier();
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int tl = (TT / WN) * wn + 16 * j + r16;
      const float mk = m_tile[j] * k;
      // fixed order: the four values of a block in pairs, then the blocks in pairs
      float sb[BI];
#pragma unroll
      for (int i = 0; i < BI; ++i) {
        float e[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) e[jj] = hw_exp2(__builtin_fmaf(x[j][i][jj], k, -mk));
        sb[i] = (e[0] + e[1]) + (e[2] + e[3]);
      }
      float sum = (sb[0] + sb[1]) + (sb[2] + sb[3]);
      // the four lane groups of the column: the same pairs in every lane
      sum = sum + __shfl_xor(sum, 16, 64);
      sum = sum + __shfl_xor(sum, 32, 64);
      if (g == 0) red[wm * TT + tl] = sum;
    }
    lds_barrier();
    if (tid < TT) {
      const int t = t0 + tid;
      if (t < p.T) {
        const float s4 = (red[tid] + red[TT + tid]) + (red[2 * TT + tid] + red[3 * TT + tid]);
        p.part_s[static_cast<int64_t>(vt) * p.T + t] = s4;
      }
    }
    // the tile maxima (the same value in every wave): lanes g == 0 of the waves wm == 0 write them
    if (wm == 0 && g == 0) {
#pragma unroll
      for (int j = 0; j < BJ; ++j) {
        const int t = t0 + (TT / WN) * wn + 16 * j + r16;
        if (t < p.T) p.part_m[static_cast<int64_t>(vt) * p.T + t] = m_tile[j];
      }
    }
  }
}

// One workgroup tile: vocab tile vt, tokens t0 .. t0 + TT - 1.
template <int VT, int TT, int WM, int WN, int STAGES, int kKC, bool kLogprob>
__device__ __forceinline__ void lm_head_tile(const LmHeadParams& p, typename LmCfg<VT, TT, WM, WN, STAGES, kKC>::Smem& sm,
                                             int vt, int t0) {
  using C = LmCfg<VT, TT, WM, WN, STAGES, kKC>;
  constexpr int BI = C::BI, BJ = C::BJ;
  const int v0 = vt * VT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const __bf16* zero = reinterpret_cast<const __bf16*>(g_zero_rows) + 8 * (lane & 15);

  // chunk c (hidden elements kKC*c .. kKC*c + kKC-1) of this workgroup's rows into stage c % STAGES
  auto issue_chunk = [&](int c) {
    const int k0 = c * kKC;
    __bf16* a = &sm.a[c % STAGES][0];
    __bf16* b = &sm.b[c % STAGES][0];
#pragma unroll
    for (int i = 0; i < C::kAInstr; ++i) {
      const int slot = (wave * C::kAInstr + i) * 64 + lane;
      const int row = slot / C::kPieces, lp = (slot % C::kPieces) ^ C::swz(row);
      const __bf16* src = (v0 + row < p.V) ? p.w + static_cast<int64_t>(v0 + row) * p.ws + k0 + 8 * lp : zero;
      dma_b128(src, __builtin_amdgcn_readfirstlane(lds_addr(a + (wave * C::kAInstr + i) * 512)));
    }
#pragma unroll
    for (int i = 0; i < C::kBInstr; ++i) {
      const int slot = (wave * C::kBInstr + i) * 64 + lane;
      const int row = slot / C::kPieces, lp = (slot % C::kPieces) ^ C::swz(row);
      const __bf16* src = (t0 + row < p.T) ? p.h + static_cast<int64_t>(t0 + row) * p.hs + k0 + 8 * lp : zero;
      dma_b128(src, __builtin_amdgcn_readfirstlane(lds_addr(b + (wave * C::kBInstr + i) * 512)));
    }
  };

  f32x4 acc[BI][BJ];
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = p.K / kKC;
#pragma unroll
  for (int c = 0; c < STAGES - 1; ++c)
    if (c < nk) issue_chunk(c);
  const int r16 = lane & 15, g = lane >> 4;
  // the fused epilogue's targets, read before the K loop so that their round trip hides behind it
  int ytgt[kLogprob ? BJ : 1];
  if constexpr (kLogprob) {
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int t = t0 + (TT / WN) * wn + 16 * j + r16;
      ytgt[j] = t < p.T ? p.targets[t] : -1;
    }
  }
#pragma unroll 1
  for (int c = 0; c < nk; ++c) {
    // chunk c has landed once only the chunks issued after it may still load;
    // after the barrier every wave is also done with chunk c-1, whose stage
    // takes chunk c + STAGES - 1
    wait_tiles_barrier<C::kChunkOps>(min(STAGES - 2, nk - 1 - c));
    if (c + STAGES - 1 < nk) issue_chunk(c + STAGES - 1);
    const __bf16* a = &sm.a[c % STAGES][0];
    const __bf16* b = &sm.b[c % STAGES][0];
#pragma unroll
    for (int s = 0; s < kKC / 32; ++s) {
      const int lp = 4 * s + g;
      bf16x8 av[BI], bv[BJ];
#pragma unroll
      for (int i = 0; i < BI; ++i) {
        const int row = (VT / WM) * wm + 16 * i + r16;
        av[i] = *reinterpret_cast<const bf16x8*>(a + row * kKC + 8 * (lp ^ C::swz(row)));
      }
#pragma unroll
      for (int j = 0; j < BJ; ++j) {
        const int row = (TT / WN) * wn + 16 * j + r16;
        bv[j] = *reinterpret_cast<const bf16x8*>(b + row * kKC + 8 * (lp ^ C::swz(row)));
      }
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int j = 0; j < BJ; ++j) acc[i][j] = mfma16(av[i], bv[j], acc[i][j]);
    }
  }

  lm_head_epilogue<VT, TT, WM, WN, kLogprob>(p, acc, reinterpret_cast<float*>(&sm), ytgt, v0, t0, vt, tid);
}

template <int VT, int TT, int WM, int WN, int STAGES, int kKC, bool kLogprob>
__global__ __launch_bounds__(WM * WN * 64, 1) void lm_head_kernel(LmHeadParams p) {
  __shared__ __attribute__((aligned(1024))) typename LmCfg<VT, TT, WM, WN, STAGES, kKC>::Smem sm;
  const int pid = p.first + blockIdx.x;
  const int xcd = pid % kLmXcds, kk = pid / kLmXcds;
  const int vt = xcd + kLmXcds * (kk / p.n_tt);
  const int tt = kk % p.n_tt;
  if (vt >= p.n_vt) return;
  lm_head_tile<VT, TT, WM, WN, STAGES, kKC, kLogprob>(p, sm, vt, tt * TT);
}

// The 256 x 256 tile of a large call, 8 waves of 64 vocab x 128 tokens, bound by
// matrix issue.  Each wave holds the operands of two K steps of 32: while the
// 32 products of one run, the LDS reads of the next go out between them, so no
// product waits for LDS.  One barrier per 64-wide chunk, placed in the middle
// of it: by then every wave has read the rest of the chunk into registers, so
// its stage can be refilled at once (chunk c + 2, a whole chunk ahead of its
// use) and every wave leaves the barrier with 32 products ready to issue.
// The loads take a uniform base per matrix and one 32-bit offset per
// instruction; rows past the vocabulary or the batch are clamped to the last
// valid one (their results are not written).
// 4100 x 151,936 x 4096 (5.1 TFLOP): 4.60 ms with a chunk's reads before its
// products, 4.19 so, 4.05 with the last 4 tokens in a tile of 64 instead of 256
// (1.26 PFLOP/s).  Matrix units busy 71% of the cycles at 1.73 GHz: the clock
// falls as they get busier.  64% of the L2 requests miss, but blocks of 4 x 8,
// 4 x 16 and 8 x 4 (vocab x token tiles) to an XCD instead of one vocab tile at
// a time all take the same time.
constexpr int kWideVT = kVocabTile, kWideTT = 256, kWideWM = 4, kWideWN = 2;
constexpr int kWideKC = 64;
constexpr int64_t kWideMaxStride = int64_t{1} << 22;  // 255 rows of it in a 32-bit byte offset

template <bool kLogprob>
__global__ __launch_bounds__(512, 1) void lm_head_wide_kernel(LmHeadParams p) {
  constexpr int BI = kWideVT / kWideWM / 16, BJ = kWideTT / kWideWN / 16;  // 4 x 8 blocks of 16 x 16
  constexpr int kStage = (kWideVT + kWideTT) * kWideKC;                  // elements: weight rows, then hidden rows
  __shared__ __attribute__((aligned(1024))) __bf16 sm[2 * kStage];
  const int pid = p.first + blockIdx.x;
  const int xcd = pid % kLmXcds, kk = pid / kLmXcds;
  const int vt = xcd + kLmXcds * (kk / p.n_tt);
  const int tt = kk % p.n_tt;
  if (vt >= p.n_vt) return;
  const int v0 = vt * kWideVT, t0 = tt * kWideTT;
  // a last tile of few tokens: not padded to 256
  if (p.T - t0 <= 64) {
    lm_head_tile<kWideVT, 64, 4, 2, 2, kWideKC, kLogprob>(
        p, *reinterpret_cast<typename LmCfg<kWideVT, 64, 4, 2, 2, kWideKC>::Smem*>(sm), vt, t0);
    return;
  }
  if (p.T - t0 <= 128) {
    lm_head_tile<kWideVT, 128, 4, 2, 2, kWideKC, kLogprob>(
        p, *reinterpret_cast<typename LmCfg<kWideVT, 128, 4, 2, 2, kWideKC>::Smem*>(sm), vt, t0);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % kWideWM, wn = wave / kWideWM;
  const int r16 = lane & 15, g = lane >> 4;

  // wave w loads rows 32w .. 32w + 31 of both matrices, 8 rows (1 KB) per
  // instruction; lane piece p of row r holds logical piece p ^ (r & 7)
  uint32_t aoff[4], boff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 32 * wave + 8 * i + (lane >> 3);
    const int piece = (lane & 7) ^ (lane >> 3);
    aoff[i] = static_cast<uint32_t>((min(row, p.V - 1 - v0) * p.ws + 8 * piece) * 2);
    boff[i] = static_cast<uint32_t>((min(row, p.T - 1 - t0) * p.hs + 8 * piece) * 2);
  }
  const __bf16* abase = p.w + static_cast<int64_t>(v0) * p.ws;
  const __bf16* bbase = p.h + static_cast<int64_t>(t0) * p.hs;
  const uint32_t ld0 = __builtin_amdgcn_readfirstlane(lds_addr(sm)) + 4096 * wave;
  auto issue = [&](int c, int i) {  // instruction i of chunk c
    const uint32_t d = ld0 + (c & 1) * (kStage * 2);
    if (i < 4)
      dma_b128_based(abase + c * kWideKC, aoff[i], d + 1024 * i);
    else
      dma_b128_based(bbase + c * kWideKC, boff[i - 4], d + kWideVT * kWideKC * 2 + 1024 * (i - 4));
  };

  f32x4 acc[BI][BJ];
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct Operands {
    bf16x8 a[BI], b[BJ];
  };
  // LDS address of this lane's operand rows, K step 0; step 1 is one XOR away
  const uint32_t sw = 16 * (g ^ (r16 & 7));
  const uint32_t ra = lds_addr(sm) + (64 * wm + r16) * (kWideKC * 2) + sw;
  const uint32_t rb = lds_addr(sm) + (kWideVT + 128 * wn + r16) * (kWideKC * 2) + sw;
  typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
  auto read = [&](Operands& o, int c, int s, int i) {  // operand i of step s of chunk c
    const uint32_t st = (c & 1) * (kStage * 2);
    const uint32_t base = ((i < BI ? ra : rb) ^ (64u * s)) + st;
    const lds_bf16x8* q = reinterpret_cast<const lds_bf16x8*>(static_cast<uintptr_t>(base));
    if (i < BI)
      o.a[i] = q[16 * i * kWideKC / 8];
    else
      o.b[i - BI] = q[16 * (i - BI) * kWideKC / 8];
  };
  int ytgt[kLogprob ? BJ : 1];
  if constexpr (kLogprob) {
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int t = t0 + 128 * wn + 16 * j + r16;
      ytgt[j] = t < p.T ? p.targets[t] : -1;
    }
  }

  const int nk = p.K / kWideKC;
#pragma unroll
  for (int i = 0; i < 8; ++i) issue(0, i);
  if (nk > 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i) issue(1, i);
  }
  wait_vmem_below<0>();  // the compiler's own wait: the targets and both chunks have landed
  lds_barrier();
  Operands o0, o1;
#pragma unroll
  for (int i = 0; i < BI + BJ; ++i) read(o0, 0, 0, i);

  // the 32 products of one K step; between them the next step's reads (kNext)
  // and a chunk's loads (kLoad), in this order
  auto products = [&](const Operands& o, Operands& nx, int c, int s, auto next_const, auto load_const) {
    constexpr bool kNext = decltype(next_const)::value, kLoad = decltype(load_const)::value;
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
#pragma unroll
      for (int i = 0; i < BI; ++i) acc[i][j] = mfma16(o.a[i], o.b[j], acc[i][j]);
      if constexpr (kNext) {
        if (2 * j < BI + BJ) {
          read(nx, c, s, 2 * j);
          read(nx, c, s, 2 * j + 1);
        }
      }
      if constexpr (kLoad) issue(c + 1, j);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kNext) {
      // said here, where the last two groups have covered the reads: at the
      // loop's head the compiler would wait for the reads it has just issued
      if (s == 0) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    }
  };
  auto chunk = [&](int c, auto next_const, auto load_const) {
    products(o0, o1, c, 1, std::true_type{}, std::false_type{});
    // chunk c + 1 has landed (the only one in flight), and every wave has read all of chunk c
    if constexpr (decltype(next_const)::value) {
      wait_barrier<0>();
      __builtin_amdgcn_sched_barrier(0);
    }
    products(o1, o0, c + 1, 0, next_const, load_const);
  };
  int c = 0;
#pragma unroll 1
  for (; c + 2 < nk; ++c) chunk(c, std::true_type{}, std::true_type{});
  if (c + 1 < nk) {
    chunk(c, std::true_type{}, std::false_type{});
    ++c;
  }
  chunk(c, std::false_type{}, std::false_type{});

  lm_head_epilogue<kWideVT, kWideTT, kWideWM, kWideWN, kLogprob>(p, acc, reinterpret_cast<float*>(sm), ytgt, v0, t0, vt,
                                                                 tid);
}

// Fold of a token's vocab-tile partials, then
//   logp = (x_y - M) * inv_temperature - log2(S) * ln 2
// (S is the sum of exp2((x - M) * inv_temperature * log2 e)).  A token's tiles
// are cut into kFoldSegs runs of consecutive tiles, one thread each, folded in
// ascending order inside a run and then run by run: the order depends on the
// tile count alone.  One thread per token walked 594 tiles in 37 dependent
// round trips (90 us, whatever the number of tokens); a run of 38 takes three.
constexpr int kFoldBatch = 16;
constexpr int kFoldSegs = 16;
constexpr int kFoldTokens = 256 / kFoldSegs;  // tokens per workgroup
__global__ __launch_bounds__(256) void logprob_fold_kernel(const float* __restrict__ part_m,
                                                           const float* __restrict__ part_s,
                                                           const float* __restrict__ y_logit,
                                                           const int32_t* __restrict__ targets, int32_t T, int32_t V,
                                                           int32_t n_vt, float it, float k, int32_t first_wg,
                                                           float* __restrict__ logp) {
  __shared__ float2 run[kFoldSegs][kFoldTokens];
  const int tok = threadIdx.x % kFoldTokens, seg = threadIdx.x / kFoldTokens;
  const int t = (first_wg + blockIdx.x) * kFoldTokens + tok;
  const int len = (n_vt + kFoldSegs - 1) / kFoldSegs;
  const int first = seg * len, last = min(first + len, n_vt);
  float M = 0.f, S = 0.f;
  auto fold = [&](float m, float s) {
    const float mn = vmax(M, m);
    const float mk = mn * k;
    S = S * hw_exp2(M * k - mk) + s * hw_exp2(m * k - mk);
    M = mn;
  };
  if (t < T) {
    for (int v0 = first; v0 < last; v0 += kFoldBatch) {
      float bm[kFoldBatch], bs[kFoldBatch];
#pragma unroll
      for (int i = 0; i < kFoldBatch; ++i) {
        const int64_t vt = min(v0 + i, n_vt - 1);
        bm[i] = part_m[vt * T + t];
        bs[i] = part_s[vt * T + t];
      }
#pragma unroll
      for (int i = 0; i < kFoldBatch; ++i) {
        const int vt = v0 + i;
        if (vt >= last) break;
        if (vt == first) {
          M = bm[i];
          S = bs[i];
        } else {
          fold(bm[i], bs[i]);
        }
      }
    }
  }
  run[seg][tok] = float2{M, S};
  __syncthreads();
  if (seg != 0 || t >= T) return;
  for (int i = 1; i < kFoldSegs && i * len < n_vt; ++i) fold(run[i][tok].x, run[i][tok].y);
  const int y = targets[t];
  const float xy = (y >= 0 && y < V) ? y_logit[t] : 0.f;
  logp[t] = (y < 0 || y >= V) ? __builtin_nanf("") : (xy - M) * it - hw_log2(S) * 0.69314718055994530942f;
}

template <int VT, int TT, int WM, int WN, int STAGES, int kKC, bool kLogprob>
hipError_t launch_cfg(LmHeadParams p, hipStream_t stream) {
  p.n_vt = (p.V + VT - 1) / VT;
  p.n_tt = (p.T + TT - 1) / TT;
  const int64_t nblocks = static_cast<int64_t>((p.n_vt + kLmXcds - 1) / kLmXcds) * kLmXcds * p.n_tt;
  return launch_parts(nblocks, WM * WN * 64, [&](int first, unsigned n) {
    p.first = first;
    hipLaunchKernelGGL((lm_head_kernel<VT, TT, WM, WN, STAGES, kKC, kLogprob>), dim3(n), dim3(WM * WN * 64), 0, stream, p);
  });
}

template <bool kLogprob>
hipError_t launch_wide(LmHeadParams p, hipStream_t stream) {
  p.n_vt = (p.V + kWideVT - 1) / kWideVT;
  p.n_tt = (p.T + kWideTT - 1) / kWideTT;
  const int64_t nblocks = static_cast<int64_t>((p.n_vt + kLmXcds - 1) / kLmXcds) * kLmXcds * p.n_tt;
  return launch_parts(nblocks, 512, [&](int first, unsigned n) {
    p.first = first;
    hipLaunchKernelGGL(lm_head_wide_kernel<kLogprob>, dim3(n), dim3(512), 0, stream, p);
  });
}

// Tile shape by the number of rows.  Every shape adds the same products in the
// same order to an accumulator, so a row has the same bits in all of them.
//
// Up to about 128 rows the product is bound by the stream of the weights
// (1.24 GB for 151,936 x 4096: 190 us at the read ceiling), and a tile padded to
// 256 tokens spends 345 us on it at 8 rows.  What the stream wants is bytes in
// flight that a barrier does not drain, so up to 64 rows two workgroups to a CU
// (32 to 80 KB of LDS each), and long runs of a row per load: a power-of-two row length puts
// the same chunk of all rows on few memory channels.  Measured at 8 rows,
// 151,936 x 4096 (and with rows 128 bytes longer): 64 vocab rows x 256-wide
// chunks 229 us (201), x 128 256 us (206) with 64 token columns; 256 vocab
// rows x 64-wide chunks 266 us (254), x 128 285 us (229); deeper rings of one
// workgroup to a CU 276-286 us; operands straight to registers, 16 waves to a
// CU, 299 us (284).
// The log-prob epilogue reduces 256 vocab entries in one workgroup, so its
// shapes keep 256 rows.
//
// The lines at 64 and 128 rows, us at 151,936 x 4096 (fused): 64 rows 274 (288) in
// tiles of 64, 65 rows 342 (342) in the tile of 128, whose 96 KB of LDS let one
// workgroup to a CU, 128 rows 355 (344); 129 rows in the wide kernel 374 (375), in
// two tiles of 128 401 (397).  The line at 64 is where the smaller tile ends and not
// the best one: two 64-token tiles on one XCD take 306 (306) at 65 rows and 330
// (319) at 128, a 128 x 128 tile, of which two fit a CU, 312 and 331.
template <bool kLogprob>
hipError_t launch_rows(const LmHeadParams& p, hipStream_t stream) {
  if constexpr (kLogprob) {
    if (p.T <= 64) return launch_cfg<kVocabTile, 64, 4, 2, 2, 64, true>(p, stream);
  } else {
    if (p.T <= 16 && p.K % 256 == 0) return launch_cfg<64, 16, 4, 1, 2, 256, false>(p, stream);
    if (p.T <= 64 && p.K % 128 == 0) return launch_cfg<64, 64, 4, 1, 2, 128, false>(p, stream);
    if (p.T <= 64) return launch_cfg<64, 64, 4, 1, 2, 64, false>(p, stream);
  }
  // 128-token tiles: up to 128 rows, and for strides past the wide kernel's 32-bit
  // offsets while the tiles fit the CUs at once (1024 rows, vocab 4096: 100 us, 122
  // with 256-token tiles); more of them read the weights too often (260 rows, hidden
  // stride 2^22 + 8, vocab 32,000: 146 us, 131 with 256; 1024 rows 357, 262).
  const bool far = p.ws > kWideMaxStride || p.hs > kWideMaxStride;
  const int64_t tiles128 = static_cast<int64_t>((p.V + kVocabTile - 1) / kVocabTile) * ((p.T + 127) / 128);
  if (p.T <= 128 || (far && tiles128 <= device_cus()))
    return launch_cfg<kVocabTile, 128, 4, 2, 2, 64, kLogprob>(p, stream);
  if (far) return launch_cfg<kVocabTile, 256, 4, 2, 2, 64, kLogprob>(p, stream);
  return launch_wide<kLogprob>(p, stream);
}

}  // namespace

hipError_t launch_lm_head(const LmHeadLaunch& a, hipStream_t stream) {
  LmHeadParams p;
  p.h = static_cast<const __bf16*>(a.hidden);
  p.w = static_cast<const __bf16*>(a.weight);
  p.out = static_cast<__bf16*>(a.logits);
  p.hs = a.hidden_stride;
  p.ws = a.weight_stride;
  p.os = a.logits_stride;
  p.T = a.num_rows;
  p.V = a.vocab;
  p.K = a.hidden_dim;
  p.targets = nullptr;
  p.part_m = p.part_s = p.y_logit = nullptr;
  p.k = 0.f;
  return launch_rows<false>(p, stream);
}

size_t lm_head_logprob_ws_bytes(int64_t num_rows, int64_t vocab) {
  const int64_t n_vt = (vocab + kVocabTile - 1) / kVocabTile;
  return static_cast<size_t>((2 * n_vt + 1) * num_rows) * sizeof(float);
}

hipError_t launch_lm_head_logprob(const LmHeadLaunch& a, const int32_t* targets, float inv_temperature, float* logp,
                                  void* workspace, hipStream_t stream) {
  LmHeadParams p;
  p.h = static_cast<const __bf16*>(a.hidden);
  p.w = static_cast<const __bf16*>(a.weight);
  p.out = static_cast<__bf16*>(a.logits);
  p.hs = a.hidden_stride;
  p.ws = a.weight_stride;
  p.os = a.logits_stride;
  p.T = a.num_rows;
  p.V = a.vocab;
  p.K = a.hidden_dim;
  const int64_t n_vt = (a.vocab + kVocabTile - 1) / kVocabTile;
  float* ws = static_cast<float*>(workspace);
  p.targets = targets;
  p.part_m = ws;
  p.part_s = ws + n_vt * a.num_rows;
  p.y_logit = ws + 2 * n_vt * a.num_rows;
  p.k = static_cast<float>(static_cast<double>(inv_temperature) * 1.4426950408889634);
  hipError_t e = launch_rows<true>(p, stream);
  if (e != hipSuccess) return e;
  const int64_t folds = (static_cast<int64_t>(a.num_rows) + kFoldTokens - 1) / kFoldTokens;
  return launch_parts(folds, 256, [&](int first, unsigned n) {
    hipLaunchKernelGGL(logprob_fold_kernel, dim3(n), dim3(256), 0, stream, p.part_m, p.part_s, p.y_logit, targets,
                       a.num_rows, a.vocab, static_cast<int32_t>(n_vt), inv_temperature, p.k, first, logp);
  });
}

}  // namespace uattn
