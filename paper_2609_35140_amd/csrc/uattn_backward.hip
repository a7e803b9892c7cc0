// Backward of the full-sequence path: dQ, dK and dV of causal GQA attention
// over a packed varlen batch, from the forward's output and log-sum-exp.
//
// For one (sequence, q head), with S = scale * Q K^T masked causally,
// P = softmax(S), O = P V (Section 3.2) and an upstream gradient dO:
//   dV = P^T dO,   dP = dO V^T,   dS = P * (dP - D) with D_i = dO_i . O_i,
//   dQ = scale * dS K,   dK = scale * dS^T Q,
// and the q heads of a group add their dK and dV.  P is recomputed from the
// saved log-sum-exp: P_ij = exp2(s_ij * c - lse_i * log2(e)), c = scale * log2(e).
//
// Deterministic and batch-invariant by construction: there are no atomics,
// and every output row is accumulated by exactly one workgroup, in an order
// that depends on nothing but its own sequence:
//   bwd_prep_kernel  D_i and lse_i * log2(e) of every (token, q head), written
//                    head-major into the workspace;
//   bwd_grads_kernel, both of:
//   bwd_dkdv         one workgroup per (128-key tile, sequence, kv head); waves w
//                    and w+4 own keys 32w .. 32w+31, one with the K operands and the
//                    dV^T accumulator in registers, the other with V and dK^T, and
//                    walk the 64-query tiles from the sequence's end down to their
//                    keys, every q head of the group at each tile (S = Q K^T with
//                    the keys as MFMA columns, so P and dS already sit in the
//                    layout the dV^T and dK^T products consume);
//   bwd_dq           one workgroup per (256-query tile, sequence, q head), laid
//                    out as the forward (queries as MFMA columns): walks the
//                    64-key tiles up to each wave's diagonal in ascending order.
// Both products of dS and P with Q, dO or K take their transposed operand
// from the transposing LDS read (ds_read_b64_tr_b16); all tiles move by
// direct-to-LDS loads with explicit wait counts, as in the forward.
#include <type_traits>

#include "uattn_internal.h"
#include "uattn_numerics.h"
#include "uattn_tile_io.h"

namespace uattn {
namespace {

// One [64 rows][D] bf16 tile in LDS, read two ways: row fragments
// (ds_read_b128, a 16-lane group reads 16 consecutive rows at one logical
// 16-byte piece) and transposing reads (ds_read_b64_tr_b16, a 16-lane group
// reads 4 consecutive rows x 2 adjacent pieces; 32 lanes share an LDS cycle).
// The 16-byte pieces of each row are XOR-swizzled by 2 * (row & 7).  For
// d = 128 this was measured with the LDS bank-conflict counter on gfx950: it
// leaves both patterns conflict-free, while swizzles that spread 16 rows over
// 16 distinct pieces conflict on one pattern or the other.  For d = 64, whose
// 128-byte rows pair up in a 256-byte bank line, the same permutation is
// applied to row pairs (2 * ((row >> 1) & 3)).
template <int D>
struct BwdTile {
  static constexpr int kPieces = D / 8;
  static constexpr int kElems = kTileKeys * D;
  __device__ __forceinline__ static int swz(int row) { return D == 128 ? 2 * (row & 7) : 2 * ((row >> 1) & 3); }
  __device__ __forceinline__ static int off(int row, int piece) { return row * D + 8 * (piece ^ swz(row)); }
};

// Issue this wave's RPW rows (RPW*wave .. RPW*wave + RPW-1) of two [64][D]
// matrices into `dst` (first matrix) and dst + kElems (second); rows r with
// r >= nvalid are filled from the zero block.
template <int D, int RPW>
__device__ __forceinline__ void load_pair_async(__bf16* dst, const __bf16* abase, const __bf16* bbase,
                                                int64_t row_stride, int nvalid, int wave, int lane) {
  using BT = BwdTile<D>;
  constexpr int kInstr = RPW * BT::kPieces / 64;
  static_assert(kInstr >= 1 && RPW * BT::kPieces == 64 * kInstr, "tile split");
  const __bf16* zero = reinterpret_cast<const __bf16*>(g_zero_rows) + 8 * (lane & 15);
  const uint32_t d0 = __builtin_amdgcn_readfirstlane(lds_addr(dst + wave * kInstr * 64 * 8));
  if (nvalid >= RPW) {
    // every row of this wave is in the sequence: uniform bases and per-lane
    // byte offsets that do not change from tile to tile
#pragma unroll
    for (int i = 0; i < kInstr; ++i) {
      const int slot = (wave * kInstr + i) * 64 + lane;
      const int row = slot / BT::kPieces, piece = slot % BT::kPieces;
      const int r = row - RPW * wave;
      const uint32_t o = static_cast<uint32_t>((r * row_stride + 8 * (piece ^ BT::swz(row))) * 2);
      dma_b128_based(abase, o, d0 + i * 1024);
      dma_b128_based(bbase, o, d0 + i * 1024 + BT::kElems * 2);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < kInstr; ++i) {
    const int slot = (wave * kInstr + i) * 64 + lane;  // 16-byte LDS piece of the tile
    const int row = slot / BT::kPieces, piece = slot % BT::kPieces;
    const int r = row - RPW * wave;
    const bool ok = r < nvalid;
    const int lp = piece ^ BT::swz(row);  // logical piece held by this LDS piece
    const __bf16* as = ok ? abase + r * row_stride + 8 * lp : zero;
    const __bf16* bs = ok ? bbase + r * row_stride + 8 * lp : zero;
    dma_b128(as, d0 + i * 1024);
    dma_b128(bs, d0 + i * 1024 + BT::kElems * 2);
  }
}

// Transposed operand of a product that contracts over the 64 rows of a tile:
// lane i of 16-lane group g gets column 16*db + i and, for step st, rows
// 32*st + 16*h + 4*g + k in element 4*h + k (the row order pack_rows uses).
template <int D>
__device__ __forceinline__ void read_tr_operand(const __bf16* tile, int db, int lane, bf16x8 (&a)[2]) {
  using BT = BwdTile<D>;
  const int g = lane >> 4, src = lane & 15;
  const int row = 4 * g + (src >> 2);  // + 32*st + 16*h: bits 4-5, which the swizzle ignores
  const int sub = src & 3;
  const int piece = (2 * db + (sub >> 1)) ^ BT::swz(row);
  const __bf16* base = tile + row * D + 8 * piece + 4 * (sub & 1);
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    const s16x4 lo = lds_read_tr16(base + (32 * st) * D);
    const s16x4 hi = lds_read_tr16(base + (32 * st + 16) * D);
    const s16x4 w[2] = {lo, hi};
    __builtin_memcpy(&a[st], w, sizeof(bf16x8));
  }
}

// Row-fragment operand: lane (g, i) gets row 16*blk + i, d = 32*st + 8*g .. +7.
template <int D>
__device__ __forceinline__ void read_row_operand(const __bf16* tile, int blk, int lane, bf16x8 (&a)[D / 32]) {
  using BT = BwdTile<D>;
  const int g = lane >> 4, row = 16 * blk + (lane & 15);
#pragma unroll
  for (int st = 0; st < D / 32; ++st) a[st] = *reinterpret_cast<const bf16x8*>(tile + BT::off(row, 4 * st + g));
}

// Values in the MFMA result layout of four 16-row blocks (x[blk][j] at row
// 16*blk + 4*g + j) -> the bf16 B operand of a product contracting over those
// 64 rows, in the order read_tr_operand delivers: step st, element e holds
// row 32*st + 16*(e/4) + 4*g + e%4.
__device__ __forceinline__ void pack_rows(const float (&x)[4][4], bf16x8 (&b)[2]) {
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int e = 0; e < 8; ++e) b[st][e] = to_bf16(x[2 * st + (e >> 2)][e & 3]);
}

struct BwdParams {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  const __bf16* out;
  const __bf16* dout;
  const float* lse;
  const int32_t* cu;
  float* ws_d;   // [Hq][T] D_i
  float* ws_l2;  // [Hq][T] lse_i * log2(e)
  __bf16* dq;
  __bf16* dk;
  __bf16* dv;
  int hq, hkv, group, total, num_seqs;
  XcdUnits kv_units, dq_units;  // of key tiles; of query tiles, counted from the end
  int kv_blocks;  // bwd_grads_kernel: the workgroups before the dQ ones
  int first;      // workgroups of the launches before this one
  float c, scale;
};

__device__ __forceinline__ void seq_range(const BwdParams& p, int seq, int& lo, int& L) {
  // clamp the (trusted) offsets so that a malformed table cannot index outside the tensors
  lo = min(max(p.cu[seq], 0), p.total);
  L = max(min(p.cu[seq + 1], p.total) - lo, 0);
}

// ---------------------------------------------------------------------------
// D_i = dO_i . O_i (fp32, lane-ordered partial sums then an xor butterfly) and
// lse_i * log2(e), for every (token, q head) row.  D/8 lanes per row.  Rows
// are enumerated head-major (r = h * T + t), the order of the two workspace
// planes, so consecutive rows write consecutive words (each row's out and
// dout reads are one 2*D-byte run either way).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void bwd_prep_kernel(BwdParams p) {
  constexpr int LPR = D / 8;
  constexpr int kRows = 256 / LPR;
  const int64_t rows = static_cast<int64_t>(p.total) * p.hq;
  const int64_t r = static_cast<int64_t>(p.first + blockIdx.x) * kRows + threadIdx.x / LPR;
  const int sub = threadIdx.x % LPR;
  int64_t row = 0;  // token-major index of (t, h) in out, dout and lse
  float acc = 0.f;
  if (r < rows) {
    const int h = static_cast<int>(r / p.total);
    const int64_t t = r % p.total;
    row = t * p.hq + h;
    const bf16x8 o = *reinterpret_cast<const bf16x8*>(p.out + row * D + 8 * sub);
    const bf16x8 d = *reinterpret_cast<const bf16x8*>(p.dout + row * D + 8 * sub);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = acc + static_cast<float>(o[e]) * static_cast<float>(d[e]);
  }
#pragma unroll
  for (int m = LPR / 2; m >= 1; m >>= 1) acc = acc + __shfl_xor(acc, m, LPR);
  if (r < rows && sub == 0) {
    p.ws_d[r] = acc;
    p.ws_l2[r] = p.lse[row] * 1.44269504088896340736f;
  }
}

// ---------------------------------------------------------------------------
// dK, dV
//
// 8 waves; waves w and w+4 share a SIMD (as in the forward) and the keys
// 32*(w%4) .. +31 of the workgroup's 128.  Wave w < 4 forms S and P and
// accumulates dV; wave w+4 forms dP and dS (from P, passed in fp32 through LDS)
// and accumulates dK.  One wave doing both needs the two accumulators (128
// registers), both key operands (64) and both score tiles (64), which leaves
// one wave on a SIMD and nothing to run beside its matrix instructions.
//
// Ping-pong, as the forward: a step of a wave is a matrix phase (the products
// of tile t-1's weights, then the scores of tile t) and a vector phase (the
// weights of tile t), each in a slot opened by a workgroup barrier, the waves
// 4-7 one slot behind:
//   slot 2t    waves 0-3: dV += dO(t-1)^T P(t-1), S(t)    waves 4-7: dS(t-1)
//   slot 2t+1  waves 0-3: P(t) -> registers and LDS       waves 4-7: dK += Q(t-1)^T dS(t-1), dP(t)
// so P(t) is written in slot 2t+1 and read in slot 2t+2.  Tiles t-1 and t are
// both read during a step, so the tiles move through a ring of three stages:
// waves 4-7, whose vector phase is the shorter one (no exponentials), load
// tile t+2 in slot 2t+2 over tile t-1, whose last readers ended in slot 2t+1,
// and wait for it before slot 2t+4, the first that reads it.
//
// Order: query tiles from the sequence's end down, the group's heads inside.
// Every key tile of a (sequence, kv head) starts at the same query tile and
// keeps step with the others, so the tiles that one of them brings into the
// XCD's L2 serve all: 20% of the L2 requests of the whole launch (dQ with it)
// miss on the pack below.  (With units that start at different tiles 24%, and 39%
// from the diagonal up with the heads outside, the backward 1-5% slower.)
//
// What bounds it: the matrix phases with the other wave's vector work beside
// them (matrix units busy 54% of the launch's cycles, dQ with it, on the pack
// below, 60% on 8 x 32K, 64/8 heads).  8 sequences of 512-8192 tokens, 32/8
// heads, d = 128 (2.8 TFLOP in these four products): 4.85 ms with one wave per
// SIMD and everything in it, 2.5-2.7 ms so (1.05-1.1 PFLOP/s).  Loads by waves
// 0-3 in their matrix phase 2.8, in their vector phase 2.6 ms; the next phase's
// first operands read before the barrier 2.7 ms.
// ---------------------------------------------------------------------------
constexpr int kKvPairs = 4;                        // wave pairs, each with its own keys
constexpr int kKvWaves = 2 * kKvPairs;
constexpr int kKeysPerPair = 32;
constexpr int kKeyTile = kKvPairs * kKeysPerPair;  // keys per workgroup
constexpr int kQTile = kTileKeys;                  // queries per step
// Key tiles to a work unit (see xcd_tile): they walk the same query tiles in
// step, so a unit's tiles come from its XCD's L2 (groups of 4, 16 and 32 were
// within 2% of 8).
constexpr int kKeyTileGroup = 8;
// From this many workgroups to a CU on.  Backward in single tiles / in eights, us:
// 16 of 200-2048 tokens, 32/8 heads, d = 128 (5.5 to a CU) 1106 / 956, 8 of 512-4096,
// 16/16 (12) 1194 / 1121, 16 of 1000, 32/8 (4.0) 573 / 576; d = 64, 24 of 1000, 16/4
// (3.0) 282 / 298.  (Ragged packs gain below the line too: 10 of 200-2048, 32/8 heads
// 511 / 484, 4 of 512-8192, 16/4, d = 64 1088 / 710.)
constexpr int kKeyTileRounds = 4;

// One matrix phase: acc[db][nb] += T^T w over the 64 rows of the tile at
// `tr_tile` (kPrev), then s[qb][nb] = R x over the rows of the tile at `row_tile`
// (kScores).  LDS reads run ahead of the products that use them, in a fixed
// order, so that one wave alone keeps the matrix unit fed.  A d block or K
// step enters the LDS address as a XOR of bits that the rest leaves clear
// (rows of 2*D bytes, even swizzle), so one register holds each base.
template <int D, bool kPrev, bool kScores>
__device__ __forceinline__ void dkdv_matrix_phase(uint32_t tr_tile, uint32_t row_tile, const bf16x8 (&w)[2][2],
                                                  const bf16x8 (&x)[2][D / 32], f32x4 (&acc)[D / 16][2],
                                                  f32x4 (&s)[4][2], int lane) {
  using BT = BwdTile<D>;
  constexpr int NDB = D / 16, NST = D / 32;
  constexpr int kAhead = 3;
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
  const int g = lane >> 4, src = lane & 15;
  const int trow = 4 * g + (src >> 2), sub = src & 3;
  uint32_t ta = tr_tile + trow * D * 2 + 16 * ((sub >> 1) ^ BT::swz(trow)) + 8 * (sub & 1);
  uint32_t ra = row_tile + src * D * 2 + 16 * (g ^ BT::swz(src));
  asm volatile("" : "+v"(ta), "+v"(ra));
  auto tread = [&](int db, bf16x8(&a)[2]) {
    lds_s16x4* tp = reinterpret_cast<lds_s16x4*>(static_cast<uintptr_t>(ta ^ (32u * db)));
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(tp + (32 * st) * D / 4);
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(tp + (32 * st + 16) * D / 4);
      const s16x4 v[2] = {lo, hi};
      __builtin_memcpy(&a[st], v, sizeof(bf16x8));
    }
  };
  auto rread = [&](int qb, bf16x8(&a)[NST]) {
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      const lds_bf16x8* rp = reinterpret_cast<const lds_bf16x8*>(static_cast<uintptr_t>(ra ^ (64u * st)));
      a[st] = rp[16 * qb * D / 8];
    }
  };
  bf16x8 ra_op[2][NST];
  if constexpr (kPrev) {
    bf16x8 tr_op[kAhead][2];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) tread(i, tr_op[i]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      bf16x8(&a)[2] = tr_op[db % kAhead];
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int st = 0; st < 2; ++st) acc[db][nb] = mfma16(a[st], w[nb][st], acc[db][nb]);
      if (db + kAhead < NDB) tread(db + kAhead, tr_op[db % kAhead]);
      if constexpr (kScores) {
        if (db == NDB - 3) rread(0, ra_op[0]);
        if (db == NDB - 1) rread(1, ra_op[1]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else if constexpr (kScores) {
    rread(0, ra_op[0]);
    rread(1, ra_op[1]);
  }
  if constexpr (kScores) {
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) {
      bf16x8(&a)[NST] = ra_op[qb & 1];
      f32x4 r[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int st = 0; st < NST; ++st) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) r[nb] = mfma16(a[st], x[nb][st], r[nb]);
        __builtin_amdgcn_sched_barrier(0);
      }
      s[qb][0] = r[0];
      s[qb][1] = r[1];
      if (qb + 2 < 4) rread(qb + 2, ra_op[qb & 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int D>
struct DkdvSmem {
  // a stage: the Q tile, the dO tile, then 64 D_i and 64 lse2 floats
  static constexpr int kStageElems = 2 * BwdTile<D>::kElems + 256;
  static constexpr int kStages = 3;
  __bf16 tiles[kStages * kStageElems];
  alignas(1024) f32x4 p[kKvPairs][8][64];  // P(t), in each lane's score layout
};

template <int D>
__device__ __forceinline__ void bwd_dkdv(const BwdParams& p, DkdvSmem<D>& sm, int pid) {
  using BT = BwdTile<D>;
  constexpr int NST = D / 32, NDB = D / 16;
  constexpr int kRpw = kQTile / kKvPairs;  // rows of a tile that each of the waves 4-7 loads
  constexpr int kStageElems = DkdvSmem<D>::kStageElems, kStages = DkdvSmem<D>::kStages;
  __bf16* const lds = sm.tiles;
  f32x4(*const pbuf)[8][64] = sm.p;

  const XcdTile at = xcd_tile(pid, p.kv_units);
  if (at.tile >= p.kv_units.ntiles) return;
  const int kt = at.tile, seq = at.seq, kvh = at.kvh;
  int lo, L;
  seq_range(p, seq, lo, L);
  const int k0 = kt * kKeyTile;
  if (k0 >= L) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int pair = wave & (kKvPairs - 1);
  const bool late = wave >= kKvPairs;                         // dP, dS, dK; one slot behind
  const int g = lane >> 4, col = lane & 15;
  const int kw0 = k0 + kKeysPerPair * pair;

  // B operands of this wave's keys (K, or V in the late waves):
  // xf[nb][st] = K[kw0 + 16*nb + col][32*st + 8*g .. +7]
  bf16x8 xf[2][NST];
  const __bf16* xsrc = late ? p.v : p.k;
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    const int kp = kw0 + 16 * nb + col;
    if (kp < L) {
      const int64_t off = (static_cast<int64_t>(lo + kp) * p.hkv + kvh) * D + 8 * g;
#pragma unroll
      for (int st = 0; st < NST; ++st) xf[nb][st] = *reinterpret_cast<const bf16x8*>(xsrc + off + 32 * st);
    } else {
#pragma unroll
      for (int st = 0; st < NST; ++st)
#pragma unroll
        for (int e = 0; e < 8; ++e) xf[nb][st][e] = static_cast<__bf16>(0.0f);
    }
  }

  const int nqt = (L + kQTile - 1) / kQTile;
  const int n = p.group * (nqt - k0 / kQTile);  // steps: >= 1 since k0 < L
  const int64_t qstride = static_cast<int64_t>(p.hq) * D;
  const float* zero_f = reinterpret_cast<const float*>(g_zero_rows) + lane;

  // the tile that is loaded next: head ih of the group, query tile iq
  int ih = 0, iq = nqt - 1;
  auto issue = [&](int stage) {  // waves 4-7 only
    const int head = kvh * p.group + ih;
    const int q0 = iq * kQTile;
    if (++ih == p.group) {
      ih = 0;
      --iq;
    }
    __bf16* st = lds + stage * kStageElems;
    const int pos = q0 + kRpw * pair;
    const int64_t off = (static_cast<int64_t>(lo + pos) * p.hq + head) * D;
    load_pair_async<D, kRpw>(st, p.q + off, p.dout + off, qstride, L - pos, pair, lane);
    if (pair < 2) {
      const float* plane = pair == 0 ? p.ws_d : p.ws_l2;
      const int qq = q0 + lane;
      const float* src = qq < L ? plane + static_cast<int64_t>(head) * p.total + lo + qq : zero_f;
      dma_b32(src, __builtin_amdgcn_readfirstlane(lds_addr(st + 2 * BT::kElems + 128 * pair)));
    }
  };

  f32x4 acc[NDB][2];  // dV^T, or dK^T in the late waves
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) acc[db][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 s[4][2];
  bf16x8 wb[2][2];  // P, or dS, of the last tile in the products' operand order
  const float c = p.c;
  const uint32_t lds0 = lds_addr(lds);
  // the early waves contract dO with P and score Q; the late ones Q with dS and dO
  const uint32_t tr_off = late ? 0 : BT::kElems * 2, row_off = late ? BT::kElems * 2 : 0;

  // weights of the tile in `stage` with its first query at q0
  auto vector_phase = [&](int stage, int q0) {
    const float* dvec = reinterpret_cast<const float*>(lds + stage * kStageElems + 2 * BT::kElems);
    float w[2][4][4];
    if (!late) {
      const float* lvec = dvec + 64;
      // P; keys after the query, and rows past the sequence, get P = 0
      const bool full = (q0 >= kw0 + kKeysPerPair - 1) && (q0 + kQTile <= L);  // wave-uniform
      auto weights = [&](auto masked) {
#pragma unroll
        for (int qb = 0; qb < 4; ++qb) {
          const f32x4 l2 = *reinterpret_cast<const f32x4*>(lvec + 16 * qb + 4 * g);
#pragma unroll
          for (int nb = 0; nb < 2; ++nb) {
            f32x4 pv;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              float x = hw_exp2(__builtin_fmaf(s[qb][nb][j], c, -l2[j]));
              if constexpr (decltype(masked)::value) {
                const int qp = q0 + 16 * qb + 4 * g + j;
                const int kp = kw0 + 16 * nb + col;
                x = (kp <= qp && qp < L) ? x : 0.f;
              }
              pv[j] = x;
              w[nb][qb][j] = x;
            }
            pbuf[pair][2 * qb + nb][lane] = pv;
          }
        }
      };
      if (full)
        weights(std::false_type{});
      else
        weights(std::true_type{});
    } else {
      // dS = P (dP - D)
#pragma unroll
      for (int qb = 0; qb < 4; ++qb) {
        const f32x4 dd = *reinterpret_cast<const f32x4*>(dvec + 16 * qb + 4 * g);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
          const f32x4 pv = pbuf[pair][2 * qb + nb][lane];
#pragma unroll
          for (int j = 0; j < 4; ++j) w[nb][qb][j] = pv[j] * (s[qb][nb][j] - dd[j]);
        }
      }
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) pack_rows(w[nb], wb[nb]);
  };

  if (late) {
    issue(0);
    if (n > 1) issue(1);
  }
  // the key operands (and stage 0) have landed; the compiler's own wait, so
  // that it does not keep those register loads pending into the loop
  wait_vmem_below<0>();
  if (late) __builtin_amdgcn_s_barrier();  // the late waves' extra slot (nothing is pending here)

  // step t: its tile in stage t % 3, the previous tile's in `prev`
  int cur = 0, prev = 2, vh = 0, vq = nqt - 1;  // vh, vq: head and query tile of step t
  auto step = [&](int t, auto prev_const, auto scores_const) {
    constexpr bool kPrev = decltype(prev_const)::value, kScores = decltype(scores_const)::value;
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_s_setprio(2);
    __builtin_amdgcn_sched_barrier(0);
    const int next = cur == kStages - 1 ? 0 : cur + 1;
    dkdv_matrix_phase<D, kPrev, kScores>(lds0 + prev * (kStageElems * 2) + tr_off,
                                         lds0 + cur * (kStageElems * 2) + row_off, wb, xf, acc, s, lane);
    if constexpr (kScores) {
      __builtin_amdgcn_sched_barrier(0);
      wait_vmem_below<0>();  // tile t+1, loaded a step ago (free in the early waves)
      lds_barrier();
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      if (late && t + 2 < n) issue(prev);
      vector_phase(cur, vq * kQTile);
      if (++vh == p.group) {
        vh = 0;
        --vq;
      }
      prev = cur;
      cur = next;
    }
  };
  step(0, std::false_type{}, std::true_type{});
#pragma unroll 1
  for (int t = 1; t < n; ++t) step(t, std::true_type{}, std::true_type{});
  step(n, std::true_type{}, std::false_type{});
  if (!late) lds_barrier();  // the early waves' matching slot

  // lane (g, col): key kw0 + 16*nb + col, d = 16*db + 4*g .. +3
  __bf16* dst = late ? p.dk : p.dv;
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    const int kp = kw0 + 16 * nb + col;
    if (kp < L) {
      const int64_t off = (static_cast<int64_t>(lo + kp) * p.hkv + kvh) * D + 4 * g;
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        bf16x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = to_bf16(late ? acc[db][nb][j] * p.scale : acc[db][nb][j]);
        *reinterpret_cast<bf16x4*>(dst + off + 16 * db) = o;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------
constexpr int kDqWaves = 8;
constexpr int kDqNB = 2;
constexpr int kDqWaveRows = kDqNB * kQCols;
constexpr int kDqRows = kDqWaves * kDqWaveRows;
constexpr int kDqTileGroup = 2;  // query tiles (of all the group's heads) to a work unit, see xcd_tile
// From this many workgroups to a CU on, as in the forward (kTileRounds).  Single / pairs,
// us: 8 of 1000 tokens, 16/16 heads, d = 64 (2 to a CU) 111 / 116, 24 of 1000, 16/4 (6)
// 280 / 285; d = 128, 8 of 512-4096, 32/32 (14) 2292 / 2259, 40/8 heads (16) 2628 /
// 2611.  Between 8 and 14 both are within 1%.
constexpr int kDqTileRounds = 8;

template <int D>
struct DqSmem {
  static constexpr int kStageElems = 2 * BwdTile<D>::kElems;  // K tile, V tile
  __bf16 tiles[2 * kStageElems];
};

template <int D>
__device__ __forceinline__ void bwd_dq(const BwdParams& p, DqSmem<D>& sm, int pid) {
  using BT = BwdTile<D>;
  constexpr int NST = D / 32, NDB = D / 16;
  constexpr int kRpw = kTileKeys / kDqWaves;
  constexpr int kStageElems = DqSmem<D>::kStageElems;
  __bf16* const lds = sm.tiles;

  const XcdTile at = xcd_tile(pid, p.dq_units);
  if (at.tile >= p.dq_units.ntiles) return;
  // query tiles counted from the end: longest work first
  const int zrev = at.tile, seq = at.seq, kvh = at.kvh;
  const int head = kvh * p.group + at.head;
  int lo, L;
  seq_range(p, seq, lo, L);
  const int nqt = (L + kDqRows - 1) / kDqRows;
  const int qt = nqt - 1 - zrev;
  if (qt < 0) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int g = lane >> 4, col = lane & 15;
  const int q0 = qt * kDqRows + wave * kDqWaveRows;
  const bool wave_on = q0 < L;
  const int last_q0 = min(qt * kDqRows + kDqRows - kDqWaveRows, ((L - 1) / kDqWaveRows) * kDqWaveRows);
  const int wg_last_tile = last_q0 / kTileKeys;
  const int my_last_tile = q0 / kTileKeys;

  // B operands of this lane's query columns: qf[nb][st] = Q[q0 + 16*nb + col][32*st + 8*g .. +7]
  bf16x8 qf[kDqNB][NST], df[kDqNB][NST];
  float ddv[kDqNB], l2v[kDqNB];
#pragma unroll
  for (int nb = 0; nb < kDqNB; ++nb) {
    const int qp = q0 + kQCols * nb + col;
    if (wave_on && qp < L) {
      const int64_t row = static_cast<int64_t>(lo + qp) * p.hq + head;
#pragma unroll
      for (int st = 0; st < NST; ++st) {
        qf[nb][st] = *reinterpret_cast<const bf16x8*>(p.q + row * D + 8 * g + 32 * st);
        df[nb][st] = *reinterpret_cast<const bf16x8*>(p.dout + row * D + 8 * g + 32 * st);
      }
      const int64_t w = static_cast<int64_t>(head) * p.total + lo + qp;
      ddv[nb] = p.ws_d[w];
      l2v[nb] = p.ws_l2[w];
    } else {
#pragma unroll
      for (int st = 0; st < NST; ++st)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          qf[nb][st][e] = static_cast<__bf16>(0.0f);
          df[nb][st][e] = static_cast<__bf16>(0.0f);
        }
      ddv[nb] = 0.f;
      l2v[nb] = 0.f;
    }
  }

  const int64_t kstride = static_cast<int64_t>(p.hkv) * D;
  auto issue = [&](int t) {
    const int pos = t * kTileKeys + kRpw * wave;
    const int64_t off = (static_cast<int64_t>(lo + pos) * p.hkv + kvh) * D;
    load_pair_async<D, kRpw>(lds + (t & 1) * kStageElems, p.k + off, p.v + off, kstride, L - pos, wave, lane);
  };

  f32x4 acc[kDqNB][NDB];
#pragma unroll
  for (int nb = 0; nb < kDqNB; ++nb)
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[nb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c = p.c;

  issue(0);
  // the Q/dO operands, D and lse (and stage 0) have landed; see bwd_dkdv
  wait_vmem_below<0>();
  auto tile_step = [&](int t, auto stage_const) {  // tile t, in stage SI = t % 2
    constexpr int SI = decltype(stage_const)::value;
    wait_barrier<0>();
    if (t + 1 <= wg_last_tile) issue(t + 1);
    if (wave_on && t <= my_last_tile) {
      const __bf16* ks = lds + SI * kStageElems;
      const __bf16* vs = ks + BT::kElems;
      // S^T = K Q^T and dP^T = V dO^T: rows = keys 16*kb + 4*g + j, column = query 16*nb + col
      f32x4 s[kDqNB][4], dp[kDqNB][4];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        bf16x8 a[NST], b[NST];
        read_row_operand<D>(ks, kb, lane, a);
        read_row_operand<D>(vs, kb, lane, b);
#pragma unroll
        for (int nb = 0; nb < kDqNB; ++nb) {
          f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int st = 0; st < NST; ++st) x = mfma16(a[st], qf[nb][st], x);
#pragma unroll
          for (int st = 0; st < NST; ++st) y = mfma16(b[st], df[nb][st], y);
          s[nb][kb] = x;
          dp[nb][kb] = y;
        }
      }
      bf16x8 sb[kDqNB][2];
      // only the diagonal tile holds keys after a query: their scores become
      // -inf there (a branch on the wave-uniform condition, not a select on
      // every tile), and exp2 turns them into P = +0, as the forward's mask
      if (t == my_last_tile) {
#pragma unroll
        for (int nb = 0; nb < kDqNB; ++nb) mask_scores(s[nb], t * kTileKeys, q0 + kQCols * nb + col, lane);
      }
#pragma unroll
      for (int nb = 0; nb < kDqNB; ++nb) {
        float dsv[4][4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float x = hw_exp2(__builtin_fmaf(s[nb][kb][j], c, -l2v[nb]));
            dsv[kb][j] = x * (dp[nb][kb][j] - ddv[nb]);
          }
        pack_rows(dsv, sb[nb]);
      }
      // dQ^T += K^T dS^T (contracting over the 64 keys)
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        bf16x8 kt[2];
        read_tr_operand<D>(ks, db, lane, kt);
#pragma unroll
        for (int nb = 0; nb < kDqNB; ++nb)
#pragma unroll
          for (int st = 0; st < 2; ++st) acc[nb][db] = mfma16(kt[st], sb[nb][st], acc[nb][db]);
      }
    }
  };
  // unrolled by the stage count: stage addresses are constant offsets
  for (int t = 0; t <= wg_last_tile; t += 2) {
    tile_step(t, std::integral_constant<int, 0>{});
    if (t + 1 <= wg_last_tile) tile_step(t + 1, std::integral_constant<int, 1>{});
  }

#pragma unroll
  for (int nb = 0; nb < kDqNB; ++nb) {
    const int qp = q0 + kQCols * nb + col;
    if (wave_on && qp < L) {
      __bf16* row = p.dq + (static_cast<int64_t>(lo + qp) * p.hq + head) * D + 4 * g;
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        bf16x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = to_bf16(acc[nb][db][j] * p.scale);
        *reinterpret_cast<bf16x4*>(row + 16 * db) = w;
      }
    }
  }
}

// One launch for both: each workgroup has a CU to itself either way (registers,
// LDS), and the dQ workgroups fill the CUs that dK/dV leaves idle, which
// are most of them where a call has few key tiles and at the end of any call.
// The dK/dV workgroups, whose walks are the longer ones, go first.
// 6 sequences of 64-700 tokens, 16/4 heads, d = 64: 41.7 + 13.3 us in two
// launches, 44.8 in one (forward and backward 72.2 -> 61.9); 8 of 512-8192,
// 32/8 heads, d = 128: 4.40 ms either way.
//
// Except at d = 64 with many dQ workgroups (kDqApart to a CU) of sequences that on
// average fill at most half of one: there a dQ workgroup alone has 32 KB of LDS and 163
// registers, so the next one starts as the waves without rows end; behind the 82 KB
// that dK/dV needs it cannot.  us in one launch and in two: 2048 sequences of 16
// tokens, 8/1 heads (64 to a CU) 297 / 241, 1024 of 40, 8/2 (32) 175 / 146, 256 of
// 128, 16/4 (16) 171 / 163; but 53 of 119-238, 40/5 (8) 153 / 164, 64 of 1-512, 16/4
// (6) 176 / 182 and 40 of 1000, 16/4 (10) 509 / 553.
constexpr int kDqApart = 8;
static_assert(kKvWaves == kDqWaves, "one block size");
template <int D>
__global__ __launch_bounds__(kKvWaves * 64, 1) void bwd_grads_kernel(BwdParams p) {
  union Smem {
    DkdvSmem<D> dkdv;
    DqSmem<D> dq;
  };
  __shared__ __attribute__((aligned(1024))) Smem sm;
  const int pid = p.first + blockIdx.x;
  if (pid < p.kv_blocks)
    bwd_dkdv<D>(p, sm.dkdv, pid);
  else
    bwd_dq<D>(p, sm.dq, pid - p.kv_blocks);  // kv_blocks is a multiple of the XCD count
}

template <int D>
__global__ __launch_bounds__(kDqWaves * 64, 1) void bwd_dq_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) DqSmem<D> sm;
  bwd_dq<D>(p, sm, p.first + blockIdx.x);
}

template <int D>
hipError_t launch_backward_d(const BwdParams& p0, int max_seqlen, hipStream_t stream) {
  const int64_t rows = static_cast<int64_t>(p0.total) * p0.hq;
  constexpr int kPrepRows = 256 / (D / 8);
  const int64_t nprep = (rows + kPrepRows - 1) / kPrepRows;
  BwdParams p = p0;
  const int64_t ktiles = (static_cast<int64_t>(max_seqlen) + kKeyTile - 1) / kKeyTile;
  const int64_t qtiles = (static_cast<int64_t>(max_seqlen) + kDqRows - 1) / kDqRows;
  const int64_t busy_kv = busy_workgroups(max_seqlen, p.num_seqs, p.total, kKeyTile, p.hkv);
  const int64_t busy_dq = busy_workgroups(max_seqlen, p.num_seqs, p.total, kDqRows, p.hq);
  // At d = 64 not for equal lengths (at least 5/6 of max_seqlen on average): half the
  // bytes to share, and the long walks no longer start first.  Single tiles / eights:
  // 40 of 1000, 16/4 heads 479 / 510, 32 of 2048 1267 / 1314, 30 of 1500-2048 (0.86)
  // 998 / 1030; 20 of 2000-3000 (0.83) 1312 / 1297, 24 of 300-4000 1459 / 1336.
  const bool equal = 6 * static_cast<int64_t>(p.total) >= 5 * static_cast<int64_t>(max_seqlen) * p.num_seqs;
  const int kt_group =
      D == 64 && equal ? 1 : unit_tiles(busy_kv, p.num_seqs, p.hkv, kKeyTileRounds, kKeyTileGroup);
  const int qt_group = unit_tiles(busy_dq, p.num_seqs, p.hq, kDqTileRounds, kDqTileGroup);
  // Over four units to a sequence the tiles of one cost nearly the same: rotated, 8
  // sequences of 512-8192 tokens, 32/8 heads, d = 128 lose about 1%.
  const bool rotate = busy_kv <= int64_t{4} * kt_group * p.num_seqs * p.hkv;
  p.kv_units = xcd_units(ktiles, kt_group, 1, p.num_seqs, p.hkv, rotate);
  p.dq_units = xcd_units(qtiles, qt_group, p.group, p.num_seqs, p.hkv);
  const int64_t nkv = xcd_grid(p.kv_units), ndq = xcd_grid(p.dq_units);
  if (nkv + ndq > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
  p.kv_blocks = static_cast<int>(nkv);
  hipError_t e = launch_parts(nprep, 256, [&](int first, unsigned n) {
    p.first = first;
    hipLaunchKernelGGL(bwd_prep_kernel<D>, dim3(n), dim3(256), 0, stream, p);
  });
  if (e != hipSuccess) return e;
  auto grads = [&](int first, unsigned n) {
    p.first = first;
    hipLaunchKernelGGL(bwd_grads_kernel<D>, dim3(n), dim3(kKvWaves * 64), 0, stream, p);
  };
  if constexpr (D == 64) {
    const bool short_seqs = 2 * static_cast<int64_t>(p.total) <= static_cast<int64_t>(p.num_seqs) * kDqRows;
    if (short_seqs && busy_dq > static_cast<int64_t>(kDqApart) * device_cus()) {
      e = launch_parts(nkv, kKvWaves * 64, grads);
      if (e != hipSuccess) return e;
      return launch_parts(ndq, kDqWaves * 64, [&](int first, unsigned n) {
        p.first = first;
        hipLaunchKernelGGL(bwd_dq_kernel<D>, dim3(n), dim3(kDqWaves * 64), 0, stream, p);
      });
    }
  }
  return launch_parts(nkv + ndq, kKvWaves * 64, grads);
}

}  // namespace

size_t backward_ws_bytes(int64_t total_tokens, int64_t num_q_heads) {
  return static_cast<size_t>(2 * total_tokens * num_q_heads) * sizeof(float);
}

hipError_t launch_backward(const BackwardLaunch& a, hipStream_t stream) {
  BwdParams p;
  p.q = static_cast<const __bf16*>(a.q);
  p.k = static_cast<const __bf16*>(a.k);
  p.v = static_cast<const __bf16*>(a.v);
  p.out = static_cast<const __bf16*>(a.out);
  p.dout = static_cast<const __bf16*>(a.dout);
  p.lse = a.lse;
  p.cu = a.cu_seqlens;
  p.ws_d = static_cast<float*>(a.workspace);
  p.ws_l2 = p.ws_d + static_cast<int64_t>(a.total_tokens) * a.num_q_heads;
  p.dq = static_cast<__bf16*>(a.dq);
  p.dk = static_cast<__bf16*>(a.dk);
  p.dv = static_cast<__bf16*>(a.dv);
  p.hq = a.num_q_heads;
  p.hkv = a.num_kv_heads;
  p.group = a.num_q_heads / a.num_kv_heads;
  p.total = a.total_tokens;
  p.num_seqs = a.num_seqs;
  p.c = a.c;
  p.scale = a.scale;
  return a.head_dim == 128 ? launch_backward_d<128>(p, a.max_seqlen, stream)
                           : launch_backward_d<64>(p, a.max_seqlen, stream);
}

}  // namespace uattn
