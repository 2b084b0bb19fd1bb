// Token staleness and the coverage-driven schedule.
//
// A token no anchor sees keeps its state and misses that step's denoising
// until the next full step (Sec. 3.2, invalid matches); regions few anchors
// observe rely on the full steps, which adaptive anchor selection and
// visibility-aware refresh would relieve (the paper's limitations section).
// The library's reading of those two policies:
//   staleness    per token, the consecutive steps without a fresh prediction
//                (its view an anchor, or a full step) or a transported
//                increment (an anchor of the step sees it), saturating at
//                254; background tokens hold 255 and never count;
//   selection    greedy weighted maximum coverage: view u covers (b, v, p)
//                when v = u or u sees it, an uncovered foreground token
//                weighs 1 + staleness; forced views first, then the largest
//                gain (ties: lower view), a views in all, sorted;
//   refresh      due when the fraction of foreground tokens with staleness
//                >= R exceeds tau (host, gc_schedule_refresh_due).
// Visibility comes from single-anchor pairs: whether anchor u alone sees
// token p of view v, one bit each, from the correspondence operator's own
// tap test (gc_geometry.h).  A set sees a token iff one of its anchors does,
// because each anchor is tested on its own.
//
// All counters are integers, so the reductions (wave ballots and shuffles,
// block sums in LDS, one atomic per block and counter) are deterministic.
#include "gc_common.h"
#include "gc_compact.h"
#include "gc_geometry.h"

namespace gc {
namespace {

constexpr int kBlock = 256;
constexpr uint8_t kBackground = 255;

// Unaligned vectors: the hardware reads and writes them at any byte, so a
// row's bytes move in wide accesses whatever H * W and the buffer's address.
typedef uint32_t u32x4_u __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x2_u __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32_u __attribute__((aligned(1)));
typedef uint16_t u16_u __attribute__((aligned(1)));

// Wave-wide sum and maximum, returned wave-uniform; every lane of the wave
// must be active.  Within each row of 16 lanes, DPP moves pair lane i with i
// xor 1, i xor 2, 7 - i (within 8) and 15 - i, so every lane ends with its
// row's total; the four row totals are then read into scalar registers.
constexpr int kDppXor1 = 0xb1;          // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4e;          // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfMirror = 0x141;   // row_half_mirror
constexpr int kDppMirror = 0x140;       // row_mirror

__device__ __forceinline__ uint32_t wave_add(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_mov_dpp(x, kDppXor1, 0xf, 0xf, false);
  x += __builtin_amdgcn_mov_dpp(x, kDppXor2, 0xf, 0xf, false);
  x += __builtin_amdgcn_mov_dpp(x, kDppHalfMirror, 0xf, 0xf, false);
  x += __builtin_amdgcn_mov_dpp(x, kDppMirror, 0xf, 0xf, false);
  return (uint32_t)__builtin_amdgcn_readlane(x, 0) + (uint32_t)__builtin_amdgcn_readlane(x, 16) +
         (uint32_t)__builtin_amdgcn_readlane(x, 32) + (uint32_t)__builtin_amdgcn_readlane(x, 48);
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor1, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppXor2, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppHalfMirror, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppMirror, 0xf, 0xf, false));
  return max(max((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 16)),
             max((uint32_t)__builtin_amdgcn_readlane((int)v, 32), (uint32_t)__builtin_amdgcn_readlane((int)v, 48)));
}

constexpr int kCompactTok = 256;   // tokens per chunk, and threads per block
constexpr int kCompactWaves = kCompactTok / 64;
// anchors whose tap loads a wave keeps in flight together (before the rotation
// 1: 45 us, 2 and 3: 35, 4: 39)
constexpr int kPairBatch = 2;

// Ballots m[q] of the lanes whose token P (live: one to look at) anchor u0 + q
// of asset b sees; u0 is wave-uniform, and an anchor past the last view repeats
// the last one, for the caller to drop.
__device__ __forceinline__ void pair_ballots(const float (&P)[3], bool live, const float* __restrict__ pos,
                                             const gc_camera* __restrict__ cams, int b, int N, int u0, int H, int W,
                                             float tol2, unsigned long long (&m)[kPairBatch]) {
  AnchorProj pj[kPairBatch];
  bool any = false;
#pragma unroll
  for (int q = 0; q < kPairBatch; ++q) {
    pj[q] = anchor_project(P, wave_camera(cams + (int64_t)b * N + min(u0 + q, N - 1)), H, W);
    any |= pj[q].ok;
    m[q] = 0ull;
  }
  if (__ballot(any & live)) {
    TapPos tp[kPairBatch];
#pragma unroll
    for (int q = 0; q < kPairBatch; ++q)
      tp[q] = anchor_tap_positions(pj[q], pos + ((int64_t)b * N + min(u0 + q, N - 1)) * H * W * 3, H, W);
#pragma unroll
    for (int q = 0; q < kPairBatch; ++q) m[q] = __ballot(live & anchor_sees(P, pj[q], tp[q], H, W, tol2));
  }
}

// One block per chunk of kCompactTok tokens of a view (grid: x = chunk,
// y = b * N + v), for every anchor u: the chunk's foreground tokens are
// compacted once, the waves take the (anchors, group of 64 of them) items in
// turn, each leaving one ballot per anchor, and the rows' bits are put
// together from the ballots by the tokens' ranks.  The anchor is the same for
// a whole wave, so its camera sits in scalar registers.
// Bound by vector-ALU issue (21 of 28 us; two IEEE divisions and four tap
// distances per pair).  8 assets x 12 views of 128 x 128: 78 -> 28 us against a
// lane per raster token and anchor, which also formed the unused weights.
__global__ __launch_bounds__(kCompactTok) void k_cov_pairs(const float* __restrict__ pos,
                                                           const gc_camera* __restrict__ cams,
                                                           const float* __restrict__ bbox, int B, int N, int H, int W,
                                                           int wpr, uint32_t* __restrict__ bits) {
  constexpr int kWords = kCompactTok / 32;         // words of bits per chunk and anchor
  __shared__ CompactLds<kCompactTok> s;
  __shared__ unsigned long long seen[GC_MAX_VIEWS][kCompactTok / 64];   // ballots: [anchor][group]
  static_assert(sizeof(s.q) >= GC_MAX_VIEWS * kWords * 4, "the words take the positions' place");
  uint32_t(*words)[kWords] = reinterpret_cast<uint32_t(*)[kWords]>(&s.q[0][0]);   // [anchor][word], after the last pair
  const int bv = blockIdx.y;
  const int b = bv / N, v = bv - b * N;
  const int HW = H * W;
  const int p0 = rotated_chunk() * kCompactTok;
  const int w0 = p0 / 32;
  int n_fg;
  const int rank = compact_foreground(pos + (int64_t)bv * HW * 3, HW, p0, s, &n_fg);
  if (n_fg == 0) {   // a chunk of background: nothing to evaluate
    for (int i = (int)threadIdx.x; i < N * kWords; i += kCompactTok) {
      const int u = i / kWords, w = i - u * kWords;
      if (w0 + w < wpr) bits[(((int64_t)u * B + b) * N + v) * wpr + w0 + w] = 0u;
    }
    return;
  }
  const int lane = __lane_id();
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int groups = (n_fg + 63) / 64;
  const float tol2 = bbox[(int64_t)b * 8 + 6];
  const int batches = (N + kPairBatch - 1) / kPairBatch;
  for (int it = wv; it < groups * batches; it += kCompactWaves) {
    const int ub = it / groups, g = it - ub * groups;   // uniform
    const int i = g * 64 + lane;
    const bool live = i < n_fg;
    const int j = live ? i : 0;
    const float P[3] = {s.q[0][j], s.q[1][j], s.q[2][j]};
    unsigned long long m[kPairBatch];
    pair_ballots(P, live, pos, cams, b, N, ub * kPairBatch, H, W, tol2, m);
#pragma unroll
    for (int q = 0; q < kPairBatch; ++q)
      if (lane == 0 && ub * kPairBatch + q < N) seen[ub * kPairBatch + q][g] = m[q];
  }
  __syncthreads();
  // a token's bit for anchor u is bit rank % 32 of word rank / 32 of u's
  // ballots; lane u of the wave collects the wave's two words for anchor u
  const uint32_t mine = rank >= 0 ? 1u << (rank & 31) : 0u;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(&seen[0][0]) + (rank >= 0 ? rank >> 5 : 0);
  uint32_t lo = 0u, hi = 0u;
  for (int u = 0; u < N; ++u) {
    const unsigned long long m = __ballot((src[u * kWords] & mine) != 0u);
    lo = lane == u ? (uint32_t)m : lo;
    hi = lane == u ? (uint32_t)(m >> 32) : hi;
  }
  if (lane < N) {
    words[lane][wv * 2] = lane == v ? 0u : lo;       // a view is no anchor of its own
    words[lane][wv * 2 + 1] = lane == v ? 0u : hi;
  }
  __syncthreads();
  for (int i = (int)threadIdx.x; i < N * kWords; i += kCompactTok) {
    const int u = i / kWords, w = i - u * kWords;
    if (w0 + w < wpr) bits[(((int64_t)u * B + b) * N + v) * wpr + w0 + w] = words[u][w];
  }
}

// Small launches: a lane per raster token and kPairBatch anchors per block
// (grid: x = chunk, y = b * N + v, z = batch of anchors).  Latency-bound there:
// no barriers, and the anchors side by side instead of one after another in a
// block.  One asset, per call: 6 views of 64 x 64 3.3 us (compacted 5.9), 12
// of 32 x 32 3.2 (8.3), 64 of 16 x 16 5.2 (14.6).
__global__ __launch_bounds__(kCompactTok) void k_cov_pairs_direct(const float* __restrict__ pos,
                                                                  const gc_camera* __restrict__ cams,
                                                                  const float* __restrict__ bbox, int B, int N, int H,
                                                                  int W, int wpr, uint32_t* __restrict__ bits) {
  const int bv = blockIdx.y;
  const int b = bv / N, v = bv - b * N;
  const int u0 = (int)blockIdx.z * kPairBatch;
  const int HW = H * W;
  const int p = (int)(blockIdx.x * kCompactTok + threadIdx.x);
  const float* pp = pos + ((int64_t)bv * HW + min(p, HW - 1)) * 3;
  const float P[3] = {pp[0], pp[1], pp[2]};
  const bool live = p < HW && finite_f(P[0]) && finite_f(P[1]) && finite_f(P[2]);
  unsigned long long m[kPairBatch];
  pair_ballots(P, live, pos, cams, b, N, u0, H, W, bbox[(int64_t)b * 8 + 6], m);
  const int lane = __lane_id();
  const int w = p >> 5;   // a wave's tokens are two words of the row
#pragma unroll
  for (int q = 0; q < kPairBatch; ++q)
    if ((lane & 31) == 0 && u0 + q < N && w < wpr)
      bits[(((int64_t)(u0 + q) * B + b) * N + v) * wpr + w] = u0 + q == v ? 0u : (uint32_t)(m[q] >> (lane & 32));
}

// The direct launch by its blocks and the compacted one's (its grid without
// the anchors).  Up to 2048 direct blocks everything is latency; above that
// the direct launch pays for the background's lanes, and is ahead only while
// the compacted one has too few blocks to hide their chains.  Direct /
// compacted in us: 2 views of 512 x 512 (2048 and 2048 blocks) 4.7 / 5.3, 12 of
// 128 x 128 (4608, 768) 8.5 / 9.9, 32 of 64 x 64 (8192, 512) 14.5 / 21.9, 8 x 4
// of 128 x 128 (4096, 2048) 8.0 / 7.3, 2 x 12 of 128 x 128 (9216, 1536)
// 14.3 / 11.9, 15 x 64 of 16 x 16 (30720, 960) 41.5 / 29.3, 64 of 64 x 64 (32768,
// 1024) 49.7 / 53.8.
bool pairs_direct(int64_t direct_blocks, int64_t compact_blocks) {
  return direct_blocks <= 2048 || (direct_blocks <= 16384 && compact_blocks <= 1024);
}

// Four tokens per thread: three 16-byte loads (positions are 4-byte aligned)
// and one 4-byte store; the last thread takes what is left one by one.
__global__ __launch_bounds__(kBlock) void k_cov_init(const float* __restrict__ pos, int64_t n_tok,
                                                     uint8_t* __restrict__ stale) {
  typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
  const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
  if (i >= n_tok) return;
  const auto value = [](float x, float y, float z) -> uint32_t {
    return finite_f(x) && finite_f(y) && finite_f(z) ? 0u : kBackground;
  };
  if (i + 4 <= n_tok) {
    const f32x4_u* P = reinterpret_cast<const f32x4_u*>(pos + i * 3);
    const f32x4_u a = P[0], b = P[1], c = P[2];
    *reinterpret_cast<u32_u*>(stale + i) = value(a.x, a.y, a.z) | value(a.w, b.x, b.y) << 8 |
                                           value(b.z, b.w, c.x) << 16 | value(c.y, c.z, c.w) << 24;
  } else {
    for (int64_t k = i; k < n_tok; ++k) stale[k] = (uint8_t)value(pos[3 * k], pos[3 * k + 1], pos[3 * k + 2]);
  }
}

// The token kernels give each lane one pair word: 32 consecutive tokens of
// a row, the staleness bytes of those tokens (two 16-byte loads at any
// address) and, per view, one coalesced uint32 of the pair bits.  The 64 lanes
// of a wave cover 2048 tokens of one (asset, view) row: an item.

__device__ __forceinline__ uint32_t pair_word(const uint32_t* __restrict__ bits, int B, int N, int wpr, int u, int b,
                                              int v, int wi) {
  return bits[(((int64_t)u * B + b) * N + v) * wpr + wi];
}

// Tokens of word wi of view v that the views in mask cover: all of them when
// v is in the set, else those some view of the set sees.
__device__ __forceinline__ uint32_t set_covers(const uint32_t* __restrict__ bits, int B, int N, int wpr,
                                               unsigned long long mask, int b, int v, int wi) {
  if ((mask >> v) & 1ull) return ~0u;
  uint32_t acc = 0u;
  for (; mask; mask &= mask - 1) acc |= pair_word(bits, B, N, wpr, __ffsll((long long)mask) - 1, b, v, wi);
  return acc;
}

// Bits of word wi that are tokens of the row (the last word may be partial).
__device__ __forceinline__ uint32_t valid_bits(int HW, int wi) {
  const int n = HW - wi * 32;
  return n >= 32 ? ~0u : (n <= 0 ? 0u : (1u << n) - 1u);
}

// Staleness bytes of tokens t0 .. t0 + 31 of a row, four per register (token
// t0 + 4k + j in byte j of d[k]); tokens past the row read as background.
// The row's end is read in one form that depends on HW alone, whose loads are
// all issued before any is looked at.  (A branch per four tokens there, each
// with loads of its own to wait for, took the step alone on 6 views of 60 x 60
// from 3.9 to 5.0 us.)
__device__ __forceinline__ void load_bytes(const uint8_t* __restrict__ row, int HW, int t0, uint32_t (&d)[8]) {
  if (t0 + 32 <= HW) {
    const u32x4_u lo = *reinterpret_cast<const u32x4_u*>(row + t0);
    const u32x4_u hi = *reinterpret_cast<const u32x4_u*>(row + t0 + 16);
    d[0] = lo.x; d[1] = lo.y; d[2] = lo.z; d[3] = lo.w;
    d[4] = hi.x; d[5] = hi.y; d[6] = hi.z; d[7] = hi.w;
  } else if (HW % 16 == 0) {   // the last word is half full (or past the row)
    const u32x4_u lo = *reinterpret_cast<const u32x4_u*>(row + min(t0, HW - 16));
    const uint32_t none = t0 < HW ? 0u : ~0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      d[k] = lo[k] | none;
      d[4 + k] = ~0u;
    }
  } else if (HW >= 32) {
    // the last 32 bytes of the row, of which those in front of t0 (other
    // tokens', perhaps being stepped meanwhile) are shifted out
    const u32x4_u lo = *reinterpret_cast<const u32x4_u*>(row + HW - 32);
    const u32x4_u hi = *reinterpret_cast<const u32x4_u*>(row + HW - 16);
    d[0] = lo.x; d[1] = lo.y; d[2] = lo.z; d[3] = lo.w;
    d[4] = hi.x; d[5] = hi.y; d[6] = hi.z; d[7] = hi.w;
    const int skip = t0 - (HW - 32);   // bytes; 32 and more: nothing of the row is left
    const int words = skip >> 2;
#pragma unroll
    for (int by = 4; by >= 1; by /= 2)
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t next = k + by < 8 ? d[k + by < 8 ? k + by : 0] : ~0u;
        d[k] = words & by ? next : d[k];
      }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t x = __builtin_amdgcn_alignbyte(k < 7 ? d[k < 7 ? k + 1 : 0] : ~0u, d[k], skip & 3);
      d[k] = words >= 8 ? ~0u : x;
    }
  } else {   // rows shorter than that: dwords, or the up to three bytes there are
    const int last = max(HW - 4, 0);
    uint32_t x[8];
    if (HW >= 4) {
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = *reinterpret_cast<const u32_u*>(row + min(t0 + 4 * k, last));
    } else {
      const uint32_t b0 = row[0], b1 = row[min(1, HW - 1)], b2 = row[min(2, HW - 1)];
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = (b0 | b1 << 8 | b2 << 16) | ~0u << (8 * HW);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int skip = t0 + 4 * k - min(t0 + 4 * k, last);
      const uint32_t y = __builtin_amdgcn_alignbyte(~0u, x[k], skip & 3);
      d[k] = skip >= 4 ? ~0u : y;
    }
  }
}

// The reverse; at the end of a row that the accesses straddle, the r tokens
// left go out in the powers of two that make up r, largest first.
__device__ __forceinline__ void store_bytes(uint8_t* __restrict__ row, int HW, int t0, const uint32_t (&d)[8]) {
  uint8_t* to = row + t0;
  const int r = HW - t0;
  if (r >= 32) {
    *reinterpret_cast<u32x4_u*>(to) = u32x4_u{d[0], d[1], d[2], d[3]};
    *reinterpret_cast<u32x4_u*>(to + 16) = u32x4_u{d[4], d[5], d[6], d[7]};
  } else if (r > 0) {
    if (r & 16) *reinterpret_cast<u32x4_u*>(to) = u32x4_u{d[0], d[1], d[2], d[3]};
    to += r & 16;
    // what is left, from its first token on (picked by masks: a choice between
    // elements would make the compiler index d, and move it to memory)
    const uint32_t m = r & 16 ? ~0u : 0u;
    uint32_t e0 = (d[4] & m) | (d[0] & ~m), e1 = (d[5] & m) | (d[1] & ~m);
    const uint32_t e2 = (d[6] & m) | (d[2] & ~m), e3 = (d[7] & m) | (d[3] & ~m);
    if (r & 8) {
      *reinterpret_cast<u32x2_u*>(to) = u32x2_u{e0, e1};
      e0 = e2;
      e1 = e3;
      to += 8;
    }
    if (r & 4) {
      *reinterpret_cast<u32_u*>(to) = e0;
      e0 = e1;
      to += 4;
    }
    if (r & 2) {
      *reinterpret_cast<u16_u*>(to) = (uint16_t)e0;
      e0 >>= 16;
      to += 2;
    }
    if (r & 1) *to = (uint8_t)e0;
  }
}

// The same for tokens t0 .. t0 + 7.
__device__ __forceinline__ void load_bytes(const uint8_t* __restrict__ row, int HW, int t0, uint32_t (&d)[2]) {
  if (t0 + 8 <= HW) {
    const u32x2_u q = *reinterpret_cast<const u32x2_u*>(row + t0);
    d[0] = q.x;
    d[1] = q.y;
  } else {   // the row's end
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int t = t0 + 4 * k;
      if (t + 4 <= HW) {
        d[k] = *reinterpret_cast<const u32_u*>(row + t);
      } else {
        uint32_t x = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) x |= (t + j < HW ? (uint32_t)row[t + j] : 0xffu) << (8 * j);
        d[k] = x;
      }
    }
  }
}

__device__ __forceinline__ void store_bytes(uint8_t* __restrict__ row, int HW, int t0, const uint32_t (&d)[2]) {
  if (t0 + 8 <= HW) {
    *reinterpret_cast<u32x2_u*>(row + t0) = u32x2_u{d[0], d[1]};
  } else {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int t = t0 + 4 * k;
      if (t + 4 <= HW) {
        *reinterpret_cast<u32_u*>(row + t) = d[k];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (t + j < HW) row[t + j] = (uint8_t)(d[k] >> (8 * j));
      }
    }
  }
}

// Bytewise (x + 1) mod 256: the token weight 1 + staleness, 0 for background.
__device__ __forceinline__ uint32_t bytes_plus_one(uint32_t x) {
  return ((x & 0x7f7f7f7fu) + 0x01010101u) ^ (x & 0x80808080u);
}

// 0x80 in each byte of x that is not zero, 0 elsewhere.
__device__ __forceinline__ uint32_t bytes_nonzero(uint32_t x) {
  return (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;
}

// Bits 4k .. 4k + 3 of sel as bytes 0 / 1 (nibble bit j moves to bit 8 j:
// the product's partial terms land on distinct bits, so nothing carries).
__device__ __forceinline__ uint32_t nibble_bytes(uint32_t sel, int k) {
  return (((sel >> (4 * k)) & 0xfu) * 0x00204081u) & 0x01010101u;
}

// The per-step staleness rule on four tokens' bytes s (token j in byte j):
// background (255) stays; a token whose byte of fresh_bytes is 0xff becomes
// 0; any other foreground token adds 1, saturating at 254.
__device__ __forceinline__ uint32_t stale_step(uint32_t s, uint32_t fresh_bytes) {
  const uint32_t fgm = (bytes_nonzero(~s) >> 7) * 0xffu;          // 0xff per foreground byte
  const uint32_t inc = bytes_nonzero(~(s | 0x01010101u)) >> 7;     // s < 254
  return (s + inc) & ~(fresh_bytes & fgm);
}

// The statistics of a row -- foreground tokens, tokens with staleness >= R,
// sum, max -- over the words its block's lanes add.
constexpr int kRowBlock = 512;

struct RowStats {
  uint32_t fg = 0, ge = 0, sum = 0, mx = 0;   // this lane's totals
  // d: a word's staleness bytes after the step (background 255, also past the row)
  __device__ __forceinline__ void add(const uint32_t (&d)[8], int R) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t on = bytes_nonzero(~d[k]);
      const uint32_t nf = d[k] & ((on >> 7) * 0xffu);   // background reads 0
      fg += (uint32_t)__popc(on);
      sum = __builtin_amdgcn_udot4(nf, 0x01010101u, sum, false);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t x = (nf >> (8 * j)) & 0xffu;
        ge += x >= (uint32_t)R ? 1u : 0u;
        mx = max(mx, x);
      }
    }
  }
  // every thread of a kRowBlock block calls it
  __device__ __forceinline__ void write(uint32_t* __restrict__ out) const {
    __shared__ uint32_t part[kRowBlock / 64][4];
    const uint32_t a = wave_add(fg), b = wave_add(ge), c = wave_add(sum), m = wave_max(mx);
    if (__lane_id() == 0) {
      uint32_t* p = part[threadIdx.x / 64];
      p[0] = a; p[1] = b; p[2] = c; p[3] = m;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
      const int k = (int)threadIdx.x;
      uint32_t acc = 0u;
      for (int q = 0; q < kRowBlock / 64; ++q) acc = k == 3 ? max(acc, part[q][k]) : acc + part[q][k];
      out[k] = acc;
    }
  }
};

// One step of a word's 32 tokens; fresh: the tokens some view of the set covers.
__device__ __forceinline__ void step_word(uint32_t (&d)[8], uint32_t fresh) {
#pragma unroll
  for (int k = 0; k < 8; ++k) d[k] = stale_step(d[k], nibble_bytes(fresh, k) * 0xffu);
}

// One block per (asset, view) row (blockIdx.x = b * N + v); its lanes
// stride over the row's pair words.  The statistics are reduced in the block
// and written once: no atomics, and no zeroing launch in front.
__global__ __launch_bounds__(kRowBlock) void k_cov_update(const uint32_t* __restrict__ bits, int B, int N, int HW,
                                                          int wpr, unsigned long long anchor_mask, int R,
                                                          uint8_t* __restrict__ stale, uint32_t* __restrict__ stats) {
  const int bv = blockIdx.x;
  const int b = bv / N, v = bv % N;
  uint8_t* row = stale + (int64_t)bv * HW;
  RowStats st;
  for (int wi = (int)threadIdx.x; wi < wpr; wi += kRowBlock) {
    const uint32_t fresh = set_covers(bits, B, N, wpr, anchor_mask, b, v, wi) & valid_bits(HW, wi);
    uint32_t d[8];
    load_bytes(row, HW, wi * 32, d);
    step_word(d, fresh);
    st.add(d, R);
    store_bytes(row, HW, wi * 32, d);
  }
  st.write(stats + (int64_t)bv * 4);
}

// ---------------------------------------------------------------------------
// Selection and scores through the coverage histogram (N <= kHistViews).
// Every foreground token has a cover mask: bit v for its own view v and bit
// u for every view u that sees it.  H[m], the summed weight 1 + staleness of
// the tokens whose mask is m, decides both: with Y[X] the sum of H[m] over
// the masks m that are subsets of X (the subset sums of H) and U all views,
//   gain(u | S) = Y[U \ S] - Y[U \ (S + u)]   (the uncovered weight u covers)
//   score(S)    = Y[U] - Y[U \ S]             (the weight S covers)
// as exact integer sums.  Two launches: H and a block counter are cleared,
// then one kernel makes the pass over the tokens -- each block builds its
// histogram in LDS and adds its non-zero bins to H with integer atomics --
// and its last block to finish (the counter's ticket) takes the subset sums
// and runs every greedy round, or scores every set, with two lookups per
// candidate.  No block waits for another.
constexpr int kHistViews = 12;
constexpr int kHistBins = 1 << kHistViews;
constexpr int kHistThreads = 1024;                // 4 lanes per pair word, 8 tokens each
constexpr int kHistBlocks = 256;                  // blocks of the token pass (more for huge inputs)
constexpr int64_t kHistMaxWords = 1 << 16;        // words per block: 2^21 tokens * 255 < 2^32 per LDS bin

constexpr int kWaitVm0 = 0x0f70;                  // s_waitcnt vmcnt(0), the other counters at their maxima

struct HistState {
  unsigned long long H[kHistBins];
  unsigned int ticket;                            // blocks of the token pass that have added their bins
};

// Clears H, the ticket and (the fused update) the statistics.
__global__ void k_hist_clear(HistState* __restrict__ hs, int nb, uint32_t* __restrict__ stats, int n_stats) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nb) hs->H[i] = 0ull;
  if (i < n_stats) stats[i] = 0u;
  if (i == 0) hs->ticket = 0u;
}

// Y = the subset sums of H, left in y (LDS, indexed by mask).  The calling
// block has acquired the other blocks' additions to H (the ticket), so plain
// loads see them.  256 threads each hold 16 masks that differ in four bits
// and add along those bits in registers: bits 0-3 (masks 16t .. 16t + 15),
// then, after a transpose through y, bits 4-7, then bits 8-11; the passes
// over bits at or above N are skipped (their masks are never read).
__device__ __forceinline__ void subset_sums(const HistState* __restrict__ hs, int N, unsigned long long* y) {
  const int nb = 1 << N;
  const int t = (int)threadIdx.x;
  unsigned long long r[16];
  auto sum4 = [&r]() {
#pragma unroll
    for (int bit = 0; bit < 4; ++bit)
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if ((j >> bit) & 1) r[j] += r[j ^ (1 << bit)];
  };
  if (t < kHistBins / 16) {
    const int m0 = 16 * t;
    if (m0 < nb) {   // nb >= 16 whenever N >= 4; a smaller nb fills one partial row
      const ulonglong2* src = reinterpret_cast<const ulonglong2*>(hs->H + m0);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const ulonglong2 q = 2 * j < nb - m0 ? src[j] : make_ulonglong2(0ull, 0ull);
        r[2 * j] = q.x;
        r[2 * j + 1] = 2 * j + 1 < nb - m0 ? q.y : 0ull;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) r[j] = 0ull;
    }
    sum4();
#pragma unroll
    for (int j = 0; j < 16; ++j) y[m0 + j] = r[j];
  }
  __syncthreads();
  for (int ph = 1; ph < 3 && 4 * ph < N; ++ph) {   // uniform
    const int sh = 4 * ph;                          // this pass's four bits: sh .. sh + 3
    const int low = t & ((1 << sh) - 1);            // bits below sh
    const int high = (t >> sh) << (sh + 4);         // bits above sh + 3
    if (t < kHistBins / 16) {
#pragma unroll
      for (int j = 0; j < 16; ++j) r[j] = y[high | (j << sh) | low];
      sum4();
#pragma unroll
      for (int j = 0; j < 16; ++j) y[high | (j << sh) | low] = r[j];
    }
    __syncthreads();
  }
}

// The views of mask in ascending order, by the first GC_MAX_VIEWS threads of a block.
__device__ __forceinline__ void write_set(unsigned long long mask, int32_t* out) {
  const int u = (int)threadIdx.x;
  if (u < GC_MAX_VIEWS && ((mask >> u) & 1ull)) out[__popcll(mask & ((1ull << u) - 1ull))] = u;
}

// Candidate sets as view masks.
constexpr int kMaxSets = 64;       // candidate sets per gc_coverage_score call
struct SetMasks {
  unsigned long long m[kMaxSets];
};

// The pass over the tokens (lane group of 4 per pair word, 8 tokens per
// lane; each wave takes 16 consecutive words per round, blocks stride over
// the words of every (asset, view) row), then in the last block: SCORE ==
// false, forced views first and a - n_forced greedy rounds, the set to out;
// SCORE == true, score[m] for the M sets.  UPDATE: the pass first applies
// one step of the staleness rule with the anchor set anchor_mask to the
// lane's tokens (stored back) and adds their statistics to stats (cleared
// by k_hist_clear) -- the per-row sums of one wave with one atomic each --
// so the histogram, and the selection or scores, are those of the updated
// staleness.
template <bool SCORE, bool UPDATE>
__global__ __launch_bounds__(kHistThreads) void k_cov_hist(const uint32_t* __restrict__ bits,
                                                           uint8_t* __restrict__ stale, int B, int N, int HW,
                                                           int wpr, int64_t n_words, HistState* __restrict__ hs, int a,
                                                           unsigned long long forced, int32_t* __restrict__ out,
                                                           SetMasks sets, int M, unsigned long long* __restrict__ score,
                                                           unsigned long long anchor_mask, int R,
                                                           uint32_t* __restrict__ stats) {
  __shared__ unsigned long long y[kHistBins];     // the last block's subset sums
  __shared__ uint32_t h[kHistBins];               // this block's histogram
  __shared__ int last;
  const int nb = 1 << N;
  for (int i = (int)threadIdx.x; i < nb; i += kHistThreads) h[i] = 0u;
  __syncthreads();
  const int lane = __lane_id();
  const int sub = lane & 3;                       // which 8 tokens of the word
  // the whole wave runs every round (a lane past the end only contributes
  // nothing), so the statistics' wave reductions see every lane
  for (int64_t base = ((int64_t)blockIdx.x * kHistThreads + (threadIdx.x & ~63)) >> 2; base < n_words;
       base += (int64_t)gridDim.x * (kHistThreads / 4)) {
    const int64_t wg = base + (lane >> 2);
    const bool active = wg < n_words;
    const int bv = active ? (int)(wg / wpr) : 0;
    const int wi = active ? (int)(wg - (int64_t)bv * wpr) : 0;
    const int b = bv / N, v = bv - b * N;
    uint32_t d[2] = {~0u, ~0u};   // staleness bytes of the lane's 8 tokens (background past the row)
    if (active) load_bytes(stale + (int64_t)bv * HW, HW, wi * 32 + 8 * sub, d);
    uint32_t pb[kHistViews];      // the other views' pair bits of these 8 tokens
#pragma unroll
    for (int u = 0; u < kHistViews; ++u)
      pb[u] = (active && u < N && u != v) ? (pair_word(bits, B, N, wpr, u, b, v, wi) >> (8 * sub)) & 0xffu : 0u;
    if constexpr (UPDATE) {
      uint32_t fresh = (anchor_mask >> v) & 1ull ? 0xffu : 0u;
#pragma unroll
      for (int u = 0; u < kHistViews; ++u) fresh |= (anchor_mask >> u) & 1ull ? pb[u] : 0u;
      fresh &= (valid_bits(HW, wi) >> (8 * sub)) & 0xffu;
      uint32_t c_fg = 0u, c_ge = 0u, c_sum = 0u, c_max = 0u;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t s0 = d[k];
        const uint32_t n = stale_step(s0, nibble_bytes(fresh, k) * 0xffu);
        d[k] = n;
        const uint32_t fgm = (bytes_nonzero(~s0) >> 7) * 0xffu;
        const uint32_t nf = n & fgm;                               // background reads 0
        c_fg += (uint32_t)__popc(bytes_nonzero(~s0));
        c_sum = __builtin_amdgcn_udot4(nf, 0x01010101u, c_sum, false);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t x = (nf >> (8 * j)) & 0xffu;
          c_ge += x >= (uint32_t)R ? 1u : 0u;
          c_max = max(c_max, x);
        }
      }
      if (active) store_bytes(stale + (int64_t)bv * HW, HW, wi * 32 + 8 * sub, d);
      // per-row statistics: one atomic per counter for a wave within one row
      const int bv0 = __builtin_amdgcn_readfirstlane(bv);   // lane 0 is always active
      if (__ballot(active && bv != bv0) == 0ull) {
        c_fg = wave_add(c_fg);
        c_ge = wave_add(c_ge);
        c_sum = wave_add(c_sum);
        c_max = wave_max(c_max);
        if (lane == 0) {
          uint32_t* st = stats + (int64_t)bv0 * 4;
          if (c_fg) atomicAdd(st + 0, c_fg);
          if (c_ge) atomicAdd(st + 1, c_ge);
          if (c_sum) atomicAdd(st + 2, c_sum);
          if (c_max) atomicMax(st + 3, c_max);
        }
      } else if (active) {
        uint32_t* st = stats + (int64_t)bv * 4;
        if (c_fg) atomicAdd(st + 0, c_fg);
        if (c_ge) atomicAdd(st + 1, c_ge);
        if (c_sum) atomicAdd(st + 2, c_sum);
        if (c_max) atomicMax(st + 3, c_max);
      }
    }
    const uint32_t w[2] = {bytes_plus_one(d[0]), bytes_plus_one(d[1])};   // weights 1 + staleness, 0: background
    if (!(w[0] | w[1])) continue;
    // neighbouring tokens mostly share a mask: runs of one mask go to LDS as one add
    uint32_t run_m = 0u, run_w = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t wt = (w[j >> 2] >> (8 * (j & 3))) & 0xffu;
      uint32_t m = 1u << v;
#pragma unroll
      for (int u = 0; u < kHistViews; ++u) m |= ((pb[u] >> j) & 1u) << u;
      if (wt) {
        if (m == run_m) {
          run_w += wt;
        } else {
          if (run_w) atomicAdd(&h[run_m], run_w);
          run_m = m;
          run_w = wt;
        }
      }
    }
    if (run_w) atomicAdd(&h[run_m], run_w);
  }
  __syncthreads();
  for (int i = (int)threadIdx.x; i < nb; i += kHistThreads)
    if (h[i]) atomicAdd(&hs->H[i], (unsigned long long)h[i]);
  // The last block to add its bins computes the result (no block waits).  A
  // barrier waits for no memory operation and the ticket's release only for
  // those of its own wave, so every wave lets its bin atomics complete before
  // the barrier; the block's acquire-release ticket (whose release covers the
  // XCD's L2 for all of them) then orders them before the last block's reads
  // of H.  A release fence per wave instead, each writing back L2, takes the
  // kernel from 18.7 to 39.8 us (8 x 12 views of 128 x 128).
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(&hs->ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  subset_sums(hs, N, y);
  const unsigned all = (1u << N) - 1u;
  if constexpr (SCORE) {
    if ((int)threadIdx.x < M) score[threadIdx.x] = y[all] - y[all & ~(unsigned)sets.m[threadIdx.x]];
  } else {
    // one thread runs the rounds; per round the N + 1 lookups are issued
    // together (a view outside [0, N) or already chosen looks up its own
    // mask and is no candidate); the larger gain wins, on equal gains the
    // lower view
    __shared__ unsigned result;
    if (threadIdx.x == 0) {
      unsigned chosen = (unsigned)forced;
      for (int n = __popc(chosen); n < a; ++n) {
        const unsigned free_views = all & ~chosen;
        unsigned long long rest[kHistViews];
#pragma unroll
        for (int u = 0; u < kHistViews; ++u) rest[u] = y[free_views & ~(1u << u)];
        const unsigned long long base = y[free_views];
        unsigned long long best_g = 0ull;
        int best = kHistViews;
#pragma unroll
        for (int u = 0; u < kHistViews; ++u) {
          const bool cand = u < N && !((chosen >> u) & 1u);
          const unsigned long long g = base - rest[u];
          const bool take = cand && (best == kHistViews || g > best_g);
          best_g = take ? g : best_g;
          best = take ? u : best;
        }
        chosen |= 1u << best;
      }
      result = chosen;
    }
    __syncthreads();
    write_set(result, out);
  }
}

// ---------------------------------------------------------------------------
// Selection and scores with more views than the histogram serves: one launch
// per greedy round (or one for all the sets), the staleness step in the first,
// and a last one that picks the last view, writes the result and recomputes
// the statistics row by row.  A round's blocks leave their partial sums in the
// workspace and every block of the next launch adds them up and picks the
// round's view itself: no launch in between, no atomics, nothing to clear.
//
// Bound by launches and latency.  Update + selection of 5 views at 2 assets x 20
// views of 95 x 97: 96 -> 33 us against an update and, per round, a pass of
// one-wave blocks and a pick; update + the scores of 20 sets 33 -> 10.4 us; 64
// views of 96 x 96 with 8 anchors 232 -> 105 us.
//
// A block's four waves share an item (64 pair words of one row, a word per
// lane); each takes every fourth view.  The weights are turned into bit
// planes, so that a view's sum over a word's 32 tokens is one masked popcount
// per plane that occurs (staleness is small: two or three of eight).
constexpr int kSelBlock = 256;
constexpr int kSelWaves = kSelBlock / 64;
// Partial sums per candidate and round that the workspace holds: twice what a
// round's launch uses, so that its size stays the one callers have been told
// (gc_coverage_workspace_bytes) whatever their views.
constexpr int kRedBlocks = 1024;
constexpr int kSelBlocks = 512;    // 8 x 16 views of 128 x 128 (1024 items): 256 / 512 blocks 40 / 38 us
static_assert(kSelWaves == 4, "k_score_pass deals every fourth view");
static_assert(kSelBlocks <= kRedBlocks, "the workspace holds the partial sums");
constexpr int kFlushItems = 4096;  // items whose sums fit a lane's and a wave's 32 bits (32 * 255 * 64 * 4096 < 2^32)

struct SelState {
  unsigned long long part[2][kRedBlocks * GC_MAX_VIEWS];  // of this and the previous round: [block][candidate]
  unsigned long long chosen[GC_MAX_ANCHORS + 1];          // views chosen before round r
};

// Blocks of a score pass: more of them where their partials stay few enough
// for the one block that adds them up, no more than of the largest selection (8
// assets x 16 views of 128 x 128, one set: 512 / 2048 blocks 7.5 / 6.6 us).
constexpr int kScoreBlocks = 2048;
int score_blocks(int64_t n_items, int M) {
  int64_t n = (int64_t)kSelBlocks * GC_MAX_VIEWS / M;
  if (n > kScoreBlocks) n = kScoreBlocks;
  return (int)(n_items < n ? n_items : n);
}

int sel_blocks(int64_t n_items) { return (int)(n_items < kSelBlocks ? n_items : kSelBlocks); }

// The sums over the blocks' partials of candidates 0 .. n - 1 to out (LDS);
// every thread of the block (a multiple of 64, at least GC_MAX_VIEWS) calls it,
// and it ends on a barrier.  A thread's stride is a multiple of n, so it adds
// one candidate's partials from coalesced loads that depend on nothing.  At most
// kSumThreads threads per candidate: their additions to out go to one address.
constexpr int kSumThreads = 128;
__device__ __forceinline__ void sum_partials(const unsigned long long* __restrict__ part, int n, int nblk,
                                             unsigned long long* out) {
  const int t = (int)threadIdx.x, T = min((int)blockDim.x / n, kSumThreads) * n;
  if (t < n) out[t] = 0ull;
  unsigned long long acc = 0ull;
  if (t < T) {
#pragma unroll 8
    for (int i = t; i < n * nblk; i += T) acc += part[i];
  }
  __syncthreads();
  if (t < T) atomicAdd(&out[t % n], acc);
  __syncthreads();
}

// The views chosen before round r (r >= 1): those before round r - 1 and the
// unchosen view with the largest gain of that round (ties: lower view).
__device__ __forceinline__ unsigned long long chosen_before(const SelState* st, int r, int N, int nblk,
                                                            unsigned long long* gain) {
  unsigned long long chosen = st->chosen[r - 1];
  sum_partials(st->part[(r - 1) & 1], N, nblk, gain);
  const int lane = __lane_id();
  const bool cand = lane < N && !((chosen >> lane) & 1ull);
  const unsigned long long g = cand ? gain[lane] : 0ull;
  const uint32_t hi = wave_max((uint32_t)(g >> 32));
  const bool top = cand && (uint32_t)(g >> 32) == hi;
  const uint32_t lo = wave_max(top ? (uint32_t)g : 0u);
  const unsigned long long best = __ballot(top && (uint32_t)g == lo);
  return best ? chosen | (best & (~best + 1ull)) : chosen;
}

// Bit planes of a word's weights: bit t of plane j is bit j of token t's byte.
__device__ __forceinline__ uint32_t weight_plane(const uint32_t (&w)[8], int j) {
  uint32_t p = 0u;
#pragma unroll
  for (int k = 0; k < 8; k += 2) {   // eight tokens: the byte's partial sums land on distinct bits
    uint32_t x = __builtin_amdgcn_udot4((w[k] >> j) & 0x01010101u, 0x08040201u, 0u, false);
    x = __builtin_amdgcn_udot4((w[k + 1] >> j) & 0x01010101u, 0x80402010u, x, false);
    p |= x << (4 * k);
  }
  return p;
}

// The bits that occur in some weight of the wave's live words.
__device__ __forceinline__ uint32_t wave_planes(const uint32_t (&w)[8]) {
  uint32_t x = ((w[0] | w[1]) | (w[2] | w[3])) | ((w[4] | w[5]) | (w[6] | w[7]));
  x |= x >> 16;
  x = (x | x >> 8) & 0xffu;
  uint32_t m = 0u;
#pragma unroll
  for (int j = 0; j < 8; ++j) m |= __ballot((x >> j) & 1u) ? 1u << j : 0u;
  return m;
}

// Gains of round r (r = 0: the forced views are chosen): per token weight
// 1 + staleness if no chosen view covers it, added to every candidate that
// does; items whose view is chosen are covered throughout and add nothing.
// UPDATE: the staleness step of anchor_mask is applied first (round 0).
// VPW: views per wave.
template <int VPW, bool UPDATE>
__global__ __launch_bounds__(kSelBlock) void k_sel_round(const uint32_t* __restrict__ bits, uint8_t* __restrict__ stale,
                                                         int B, int N, int HW, int wpr, SelState* st, int r, int nblk,
                                                         unsigned long long forced, unsigned long long anchor_mask) {
  __shared__ unsigned long long gain[GC_MAX_VIEWS];
  __shared__ uint32_t word[VPW * kSelWaves][64];   // the item's pair words of every view
  const int lane = __lane_id();
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int cpr = (wpr + 63) / 64;   // items per (asset, view)
  const int64_t n_items = (int64_t)B * N * cpr;
  uint32_t d[8], wd[VPW];
  int bv, wi;
  auto load = [&](int64_t it) {
    bv = (int)(it / cpr);
    wi = (int)(it - (int64_t)bv * cpr) * 64 + lane;
    const int b = bv / N, v = bv - b * N;
    load_bytes(stale + (int64_t)bv * HW, HW, wi * 32, d);
#pragma unroll
    for (int q = 0; q < VPW; ++q) {
      const int u = q * kSelWaves + wv;
      wd[q] = u >= N || wi >= wpr ? 0u : u == v ? ~0u : pair_word(bits, B, N, wpr, u, b, v, wi);
    }
  };
  if (blockIdx.x < n_items) load(blockIdx.x);   // in flight while the view of the last round is picked
  const unsigned long long chosen = r == 0 ? forced : chosen_before(st, r, N, nblk, gain);
  if (blockIdx.x == 0 && threadIdx.x == 0) st->chosen[r] = chosen;
  uint32_t acc[VPW] = {};
  unsigned long long total[VPW] = {};
  int left = kFlushItems;
  for (int64_t it = blockIdx.x; it < n_items; it += gridDim.x) {
#pragma unroll
    for (int q = 0; q < VPW; ++q) word[q * kSelWaves + wv][lane] = wd[q];
    __syncthreads();
    auto covered = [&](unsigned long long mask) {   // the word's tokens that the views in mask cover
      uint32_t c = 0u;
      for (; mask; mask &= mask - 1) c |= word[__ffsll((long long)mask) - 1][lane];
      return c;
    };
    const uint32_t live = wi < wpr ? valid_bits(HW, wi) & ~covered(chosen) : 0u;
    if constexpr (UPDATE) {   // after the barrier: every wave has read the old bytes
      step_word(d, wi < wpr ? covered(anchor_mask) & valid_bits(HW, wi) : 0u);
      if (wv == 0) store_bytes(stale + (int64_t)bv * HW, HW, wi * 32, d);
    }
    if (__ballot(live != 0u)) {
#pragma unroll
      for (int k = 0; k < 8; ++k) d[k] = bytes_plus_one(d[k]);
      const uint32_t planes = wave_planes(d);
      for (int j = 0; j < 8; ++j) {
        if (!((planes >> j) & 1u)) continue;   // uniform
        const uint32_t p = weight_plane(d, j) & live;
#pragma unroll
        for (int q = 0; q < VPW; ++q) acc[q] += (uint32_t)__popc(wd[q] & p) << j;
      }
    }
    if (it + gridDim.x < n_items) load(it + gridDim.x);
    if (--left == 0) {
      left = kFlushItems;
#pragma unroll
      for (int q = 0; q < VPW; ++q) {
        total[q] += wave_add(acc[q]);
        acc[q] = 0u;
      }
    }
    __syncthreads();   // the next item's words overwrite these
  }
#pragma unroll
  for (int q = 0; q < VPW; ++q) {
    const int u = q * kSelWaves + wv;
    total[q] += wave_add(acc[q]);
    if (u < N && lane == 0) st->part[r & 1][blockIdx.x * N + u] = total[q];
  }
}

// Partial scores of the M sets: 1 + staleness over the foreground tokens a set
// covers.  The item's pair words are put in LDS once, for every set: those of
// the views in need, which some set (or the step's anchor set) holds.
// 15 assets x 64 views of 64 x 64, one set of three views: 10.3 us; 26.7 with
// every view's words, one load after another.
template <bool UPDATE>
__global__ __launch_bounds__(kSelBlock) void k_score_pass(const uint32_t* __restrict__ bits,
                                                          uint8_t* __restrict__ stale, int B, int N, int HW, int wpr,
                                                          SelState* st, SetMasks sets, int M, unsigned long long need,
                                                          unsigned long long anchor_mask) {
  constexpr int kLoads = 4;
  __shared__ uint32_t word[GC_MAX_VIEWS][64];
  const int lane = __lane_id();
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int cpr = (wpr + 63) / 64;
  const int64_t n_items = (int64_t)B * N * cpr;
  unsigned long long mine = 0ull;   // lane m: set m's total
  for (int64_t it = blockIdx.x; it < n_items; it += gridDim.x) {
    const int bv = (int)(it / cpr);
    const int b = bv / N, v = bv - b * N;
    const int wi = (int)(it - (int64_t)bv * cpr) * 64 + lane;
    const bool in = wi < wpr;
    uint8_t* row = stale + (int64_t)bv * HW;
    uint32_t d[8];
    load_bytes(row, HW, wi * 32, d);
    // every fourth view for each wave; a view past the last repeats it
    for (unsigned long long m = need & (0x1111111111111111ull << wv); m;) {   // uniform
      int u[kLoads];
      uint32_t x[kLoads];
#pragma unroll
      for (int q = 0; q < kLoads; ++q) {
        u[q] = m ? __ffsll((long long)m) - 1 : u[q > 0 ? q - 1 : 0];
        m &= m - 1;
        x[q] = pair_word(bits, B, N, wpr, u[q], b, v, min(wi, wpr - 1));
      }
#pragma unroll
      for (int q = 0; q < kLoads; ++q) word[u[q]][lane] = !in ? 0u : u[q] == v ? ~0u : x[q];
    }
    if constexpr (UPDATE) __builtin_amdgcn_s_waitcnt(kWaitVm0);   // the old bytes, which wave 0 overwrites
    __syncthreads();
    const uint32_t live = in ? valid_bits(HW, wi) : 0u;
    if constexpr (UPDATE) {
      uint32_t fresh = 0u;
      for (unsigned long long m = anchor_mask; m; m &= m - 1) fresh |= word[__ffsll((long long)m) - 1][lane];
      step_word(d, fresh & live);
      if (wv == 0) store_bytes(row, HW, wi * 32, d);   // after the barrier: every wave has read the old bytes
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) d[k] = bytes_plus_one(d[k]);
    const uint32_t planes = wave_planes(d);
    uint32_t p[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = (planes >> j) & 1u ? weight_plane(d, j) & live : 0u;
    for (int s = wv; s < M; s += kSelWaves) {   // uniform
      uint32_t cov = 0u, sum = 0u;
      for (unsigned long long m = sets.m[s]; m; m &= m - 1) cov |= word[__ffsll((long long)m) - 1][lane];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if ((planes >> j) & 1u) sum += (uint32_t)__popc(cov & p[j]) << j;
      const uint32_t g = wave_add(sum);
      if (lane == s) mine += g;
    }
    __syncthreads();   // the next item's words overwrite these
  }
  // a wave's lanes hold its own sets' totals; the partials of set s sit with wave s % kSelWaves
  if (lane < M && lane % kSelWaves == wv) st->part[0][blockIdx.x * M + lane] = mine;
}

// The result (block 0) after `rounds` rounds of k_sel_round or one pass of
// k_score_pass, and, STATS, the statistics of row blockIdx.x.
template <bool SCORE, bool STATS>
__global__ __launch_bounds__(kRowBlock) void k_cov_final(const SelState* st, int N, int rounds, int nblk,
                                                         unsigned long long forced, int32_t* __restrict__ out, int M,
                                                         unsigned long long* __restrict__ score,
                                                         const uint8_t* __restrict__ stale, int HW, int wpr, int R,
                                                         uint32_t* __restrict__ stats) {
  if (blockIdx.x == 0) {
    __shared__ unsigned long long sum[kMaxSets];
    if constexpr (SCORE) {
      sum_partials(st->part[0], M, nblk, sum);
      if ((int)threadIdx.x < M) score[threadIdx.x] = sum[threadIdx.x];
    } else {
      write_set(rounds ? chosen_before(st, rounds, N, nblk, sum) : forced, out);
    }
  }
  if constexpr (STATS) {
    const uint8_t* row = stale + (int64_t)blockIdx.x * HW;
    RowStats rs;
    for (int wi = (int)threadIdx.x; wi < wpr; wi += kRowBlock) {
      uint32_t d[8];
      load_bytes(row, HW, wi * 32, d);
      rs.add(d, R);
    }
    rs.write(stats + (int64_t)blockIdx.x * 4);
  }
}

// The histogram path: clear H and the ticket (and the statistics), then the
// pass over the tokens with the last block's rounds (select) or scores
// (score); UPDATE applies the staleness step first (anchor_mask, R, stats).
template <bool SCORE, bool UPDATE>
void launch_hist(const uint32_t* bits, uint8_t* stale, int B, int N, size_t HW, HistState* hs, int a,
                 unsigned long long forced, int32_t* out, const SetMasks& sets, int M, unsigned long long* score,
                 unsigned long long anchor_mask, int R, uint32_t* stats, hipStream_t stream) {
  const int wpr = (int)((HW + 31) / 32);
  const int64_t n_words = (int64_t)B * N * wpr;
  int64_t nblk = (n_words * 4 + kHistThreads - 1) / kHistThreads;
  if (nblk > kHistBlocks) nblk = kHistBlocks;
  const int64_t need = (n_words + kHistMaxWords - 1) / kHistMaxWords;
  if (nblk < need) nblk = need;
  const int n_stats = UPDATE ? B * N * 4 : 0;   // B * N <= 65535 (check_grid)
  const int n_clear = (1 << N) > n_stats ? (1 << N) : n_stats;
  hipLaunchKernelGGL(k_hist_clear, dim3((unsigned)((n_clear + 255) / 256)), dim3(256), 0, stream, hs, 1 << N, stats,
                     n_stats);
  hipLaunchKernelGGL((k_cov_hist<SCORE, UPDATE>), dim3((unsigned)nblk), dim3(kHistThreads), 0, stream, bits, stale, B,
                     N, (int)HW, wpr, n_words, hs, a, forced, out, sets, M, score, anchor_mask, R, stats);
}

// The histogram path serves N <= kHistViews (its grid stays below 2^31 blocks for any legal size).
bool hist_path(int N) { return N <= kHistViews; }

int check_grid(int B, int N, int H, int W, const char* who) {
  if (B < 1 || N < 1 || H < 1 || W < 1) return fail(GC_ERR_SHAPE, "%s: bad shape B=%d N=%d H=%d W=%d", who, B, N, H, W);
  if (N > GC_MAX_VIEWS) return fail(GC_ERR_CAPACITY, "%s: N=%d exceeds %d", who, N, GC_MAX_VIEWS);
  if (H > GC_MAX_GRID || W > GC_MAX_GRID) return fail(GC_ERR_CAPACITY, "%s: grid %dx%d exceeds %d", who, H, W, GC_MAX_GRID);
  if ((int64_t)B * N * N > 65535) return fail(GC_ERR_CAPACITY, "%s: B*N*N exceeds 65535", who);
  return GC_OK;
}

}  // namespace
}  // namespace gc

using namespace gc;

extern "C" int64_t gc_coverage_pair_words(int B, int N, int H, int W) {
  if (B < 1 || N < 1 || H < 1 || W < 1) return 0;
  const int64_t wpr = ((int64_t)H * W + 31) / 32;
  return (int64_t)N * B * N * wpr;
}

extern "C" int gc_coverage_pairs(const float* pos, const gc_camera* cams, const float* bbox, int B, int N, int H,
                                 int W, uint32_t* pair_bits, hipStream_t stream) {
  clear_error();
  if (!pos || !cams || !bbox || !pair_bits) return fail(GC_ERR_ARG, "gc_coverage_pairs: null pointer");
  int rc = check_grid(B, N, H, W, "gc_coverage_pairs");
  if (rc) return rc;
  if (!aligned16(pos) || !aligned16(pair_bits)) return fail(GC_ERR_ALIGN, "gc_coverage_pairs: pos and pair_bits must be 16-byte aligned");
  const size_t HW = (size_t)H * W;
  const int wpr = (int)((HW + 31) / 32);
  const size_t nb = (size_t)gc_coverage_pair_words(B, N, H, W) * 4;
  if (overlaps(pair_bits, nb, pos, (size_t)B * N * HW * 12) || overlaps(pair_bits, nb, cams, (size_t)B * N * sizeof(gc_camera)) ||
      overlaps(pair_bits, nb, bbox, (size_t)B * 32))
    return fail(GC_ERR_ALIAS, "gc_coverage_pairs: pair_bits overlaps an input");
  const int64_t chunks = ((int64_t)HW + kCompactTok - 1) / kCompactTok, batches = (N + kPairBatch - 1) / kPairBatch;
  if (pairs_direct(chunks * B * N * batches, chunks * B * N))
    hipLaunchKernelGGL(k_cov_pairs_direct, dim3((unsigned)chunks, (unsigned)(B * N), (unsigned)batches),
                       dim3(kCompactTok), 0, stream, pos, cams, bbox, B, N, H, W, wpr, pair_bits);
  else
    hipLaunchKernelGGL(k_cov_pairs, dim3((unsigned)chunks, (unsigned)(B * N)), dim3(kCompactTok), 0, stream, pos, cams,
                       bbox, B, N, H, W, wpr, pair_bits);
  return after_launch(stream, "gc_coverage_pairs");
}

extern "C" int gc_coverage_init(const float* pos, int B, int N, int H, int W, uint8_t* stale, hipStream_t stream) {
  clear_error();
  if (!pos || !stale) return fail(GC_ERR_ARG, "gc_coverage_init: null pointer");
  int rc = check_grid(B, N, H, W, "gc_coverage_init");
  if (rc) return rc;
  const int64_t n_tok = (int64_t)B * N * H * W;
  if (overlaps(stale, (size_t)n_tok, pos, (size_t)n_tok * 12)) return fail(GC_ERR_ALIAS, "gc_coverage_init: stale overlaps pos");
  hipLaunchKernelGGL(k_cov_init, dim3((unsigned)((n_tok + 4 * kBlock - 1) / (4 * kBlock))), dim3(kBlock), 0, stream, pos, n_tok,
                     stale);
  return after_launch(stream, "gc_coverage_init");
}

namespace gc {
namespace {

// Argument checks of one staleness step; mask: the anchor set's views.
int check_update(const uint32_t* pair_bits, int B, int N, int H, int W, const int32_t* anchors, int a, int R,
                 const uint8_t* stale, const uint32_t* stats, const char* who, unsigned long long* mask) {
  if (!pair_bits || !anchors || !stale || !stats) return fail(GC_ERR_ARG, "%s: null pointer", who);
  int rc = check_grid(B, N, H, W, who);
  if (rc) return rc;
  if (a < 1 || a > N) return fail(GC_ERR_ARG, "%s: a=%d outside [1, N=%d]", who, a, N);
  if (R < 1) return fail(GC_ERR_ARG, "%s: R=%d must be >= 1", who, R);
  *mask = 0;
  for (int s = 0; s < a; ++s) {
    if (anchors[s] < 0 || anchors[s] >= N) return fail(GC_ERR_ARG, "%s: anchor %d outside [0, %d)", who, anchors[s], N);
    if ((*mask >> anchors[s]) & 1ull) return fail(GC_ERR_ARG, "%s: anchor %d listed twice", who, anchors[s]);
    *mask |= 1ull << anchors[s];
  }
  const size_t HW = (size_t)H * W;
  const size_t n_tok = (size_t)B * N * HW, nb = (size_t)gc_coverage_pair_words(B, N, H, W) * 4;
  if (overlaps(stats, (size_t)B * N * 16, stale, n_tok) || overlaps(stats, (size_t)B * N * 16, pair_bits, nb) ||
      overlaps(stale, n_tok, pair_bits, nb))
    return fail(GC_ERR_ALIAS, "%s: stale, stats and pair_bits must not overlap", who);
  if (!aligned16(pair_bits) || !aligned16(stats)) return fail(GC_ERR_ALIGN, "%s: pair_bits and stats must be 16-byte aligned", who);
  return GC_OK;
}

// Argument checks of a selection; mask: the forced views.
int check_select(const uint32_t* pair_bits, const uint8_t* stale, int B, int N, int H, int W, int a,
                 const int32_t* forced, int n_forced, const int32_t* anchors_out, const void* workspace,
                 size_t ws_bytes, const char* who, unsigned long long* mask) {
  if (!pair_bits || !stale || !anchors_out || !workspace) return fail(GC_ERR_ARG, "%s: null pointer", who);
  int rc = check_grid(B, N, H, W, who);
  if (rc) return rc;
  if (a < 1 || a > N) return fail(GC_ERR_ARG, "%s: a=%d outside [1, N=%d]", who, a, N);
  if (a > GC_MAX_ANCHORS) return fail(GC_ERR_CAPACITY, "%s: a=%d exceeds %d", who, a, GC_MAX_ANCHORS);
  if (n_forced < 0 || n_forced > a || (n_forced > 0 && !forced))
    return fail(GC_ERR_ARG, "%s: n_forced=%d outside [0, a=%d]", who, n_forced, a);
  if (ws_bytes < gc_coverage_workspace_bytes())
    return fail(GC_ERR_CAPACITY, "%s: workspace of %zu bytes, %zu needed", who, ws_bytes, gc_coverage_workspace_bytes());
  if (!aligned16(workspace) || !aligned16(pair_bits)) return fail(GC_ERR_ALIGN, "%s: workspace and pair_bits must be 16-byte aligned", who);
  *mask = 0;
  for (int j = 0; j < n_forced; ++j) {
    if (forced[j] < 0 || forced[j] >= N) return fail(GC_ERR_ARG, "%s: forced view %d outside [0, %d)", who, forced[j], N);
    if ((*mask >> forced[j]) & 1ull) return fail(GC_ERR_ARG, "%s: forced view %d listed twice", who, forced[j]);
    *mask |= 1ull << forced[j];
  }
  const size_t HW = (size_t)H * W;
  const size_t n_tok = (size_t)B * N * HW, nb = (size_t)gc_coverage_pair_words(B, N, H, W) * 4;
  const size_t ws = gc_coverage_workspace_bytes();
  if (overlaps(workspace, ws, pair_bits, nb) || overlaps(workspace, ws, stale, n_tok) ||
      overlaps(anchors_out, (size_t)a * 4, workspace, ws) || overlaps(anchors_out, (size_t)a * 4, pair_bits, nb) ||
      overlaps(anchors_out, (size_t)a * 4, stale, n_tok))
    return fail(GC_ERR_ALIAS, "%s: workspace / anchors_out overlap an input", who);
  return GC_OK;
}

// Argument checks of a scoring call; masks: the candidate sets as view masks.
int check_score(const uint32_t* pair_bits, const uint8_t* stale, int B, int N, int H, int W, const int32_t* sets,
                int M, int a, const uint64_t* scores, const void* workspace, size_t ws_bytes, const char* who,
                SetMasks* masks) {
  if (!pair_bits || !stale || !sets || !scores || !workspace) return fail(GC_ERR_ARG, "%s: null pointer", who);
  int rc = check_grid(B, N, H, W, who);
  if (rc) return rc;
  if (M < 1 || M > kMaxSets) return fail(GC_ERR_CAPACITY, "%s: M=%d outside [1, %d]", who, M, kMaxSets);
  if (a < 1 || a > N) return fail(GC_ERR_ARG, "%s: a=%d outside [1, N=%d]", who, a, N);
  std::memset(masks, 0, sizeof(*masks));
  for (int m = 0; m < M; ++m)
    for (int j = 0; j < a; ++j) {
      const int u = sets[m * a + j];
      if (u < 0 || u >= N) return fail(GC_ERR_ARG, "%s: view %d of set %d outside [0, %d)", who, u, m, N);
      masks->m[m] |= 1ull << u;
    }
  const size_t HW = (size_t)H * W;
  const size_t n_tok = (size_t)B * N * HW, nb = (size_t)gc_coverage_pair_words(B, N, H, W) * 4;
  if (ws_bytes < gc_coverage_workspace_bytes())
    return fail(GC_ERR_CAPACITY, "%s: workspace of %zu bytes, %zu needed", who, ws_bytes, gc_coverage_workspace_bytes());
  const size_t ws = gc_coverage_workspace_bytes();
  if (overlaps(scores, (size_t)M * 8, pair_bits, nb) || overlaps(scores, (size_t)M * 8, stale, n_tok) ||
      overlaps(workspace, ws, pair_bits, nb) || overlaps(workspace, ws, stale, n_tok) ||
      overlaps(workspace, ws, scores, (size_t)M * 8))
    return fail(GC_ERR_ALIAS, "%s: scores / workspace overlap an input or each other", who);
  if (!aligned16(pair_bits) || !aligned16(workspace) || ((uintptr_t)scores & 7u))
    return fail(GC_ERR_ALIGN, "%s: pair_bits and workspace 16-byte, scores 8-byte aligned", who);
  return GC_OK;
}

// The staleness step alone: one block per (asset, view) row, each writing its
// row's statistics.
void launch_update(const uint32_t* pair_bits, int B, int N, size_t HW, unsigned long long mask, int R, uint8_t* stale,
                   uint32_t* stats, hipStream_t stream) {
  hipLaunchKernelGGL(k_cov_update, dim3((unsigned)(B * N)), dim3(kRowBlock), 0, stream, pair_bits, B, N, (int)HW,
                     (int)((HW + 31) / 32), mask, R, stale, stats);
}

// The selection on the current staleness (after the optional step of
// mask_upd, R, stats, which the first pass over the tokens applies itself).
void launch_select(const uint32_t* pair_bits, uint8_t* stale, int B, int N, size_t HW, int a, unsigned long long forced,
                   int n_forced, int32_t* anchors_out, void* workspace, bool upd, unsigned long long mask_upd, int R,
                   uint32_t* stats, hipStream_t stream) {
  const int rounds = a - n_forced;
  if (hist_path(N) && rounds > 0) {
    SetMasks none;
    std::memset(&none, 0, sizeof(none));
    HistState* hs = static_cast<HistState*>(workspace);
    if (upd)
      launch_hist<false, true>(pair_bits, stale, B, N, HW, hs, a, forced, anchors_out, none, 0, nullptr, mask_upd, R,
                               stats, stream);
    else
      launch_hist<false, false>(pair_bits, stale, B, N, HW, hs, a, forced, anchors_out, none, 0, nullptr, 0ull, 1,
                                nullptr, stream);
    return;
  }
  SelState* st = static_cast<SelState*>(workspace);
  const int wpr = (int)((HW + 31) / 32);
  const int nblk = sel_blocks((int64_t)B * N * ((wpr + 63) / 64));
  if (rounds == 0 && upd) {   // the forced views are the whole set: the step alone
    launch_update(pair_bits, B, N, HW, mask_upd, R, stale, stats, stream);
    upd = false;
  }
#define GC_SEL_ROUND(VPW_, UPD_)                                                                               \
  hipLaunchKernelGGL((k_sel_round<VPW_, UPD_>), dim3((unsigned)nblk), dim3(kSelBlock), 0, stream, pair_bits, stale, B, N, \
                     (int)HW, wpr, st, r, nblk, forced, mask_upd)
  for (int r = 0; r < rounds; ++r) {
    const bool step = upd && r == 0;
    if (N <= 4 * kSelWaves) {
      if (step) GC_SEL_ROUND(4, true); else GC_SEL_ROUND(4, false);
    } else if (N <= 8 * kSelWaves) {
      if (step) GC_SEL_ROUND(8, true); else GC_SEL_ROUND(8, false);
    } else {
      if (step) GC_SEL_ROUND(16, true); else GC_SEL_ROUND(16, false);
    }
  }
#undef GC_SEL_ROUND
  if (upd)
    hipLaunchKernelGGL((k_cov_final<false, true>), dim3((unsigned)(B * N)), dim3(kRowBlock), 0, stream, st, N, rounds,
                       nblk, forced, anchors_out, 0, nullptr, stale, (int)HW, wpr, R, stats);
  else
    hipLaunchKernelGGL((k_cov_final<false, false>), dim3(1), dim3(kRowBlock), 0, stream, st, N, rounds, nblk, forced,
                       anchors_out, 0, nullptr, nullptr, 0, 0, 1, nullptr);
}

// The set scores on the current staleness (after the optional step, as above).
void launch_score(const uint32_t* pair_bits, uint8_t* stale, int B, int N, size_t HW, const SetMasks& masks, int M,
                  int a, uint64_t* scores, void* workspace, bool upd, unsigned long long mask_upd, int R,
                  uint32_t* stats, hipStream_t stream) {
  unsigned long long* out = reinterpret_cast<unsigned long long*>(scores);
  if (hist_path(N)) {
    HistState* hs = static_cast<HistState*>(workspace);
    if (upd)
      launch_hist<true, true>(pair_bits, stale, B, N, HW, hs, a, 0ull, nullptr, masks, M, out, mask_upd, R, stats,
                              stream);
    else
      launch_hist<true, false>(pair_bits, stale, B, N, HW, hs, a, 0ull, nullptr, masks, M, out, 0ull, 1, nullptr,
                               stream);
    return;
  }
  SelState* st = static_cast<SelState*>(workspace);
  const int wpr = (int)((HW + 31) / 32);
  const int nblk = score_blocks((int64_t)B * N * ((wpr + 63) / 64), M);
  unsigned long long need = upd ? mask_upd : 0ull;
  for (int m = 0; m < M; ++m) need |= masks.m[m];
  if (upd) {
    hipLaunchKernelGGL(k_score_pass<true>, dim3((unsigned)nblk), dim3(kSelBlock), 0, stream, pair_bits, stale, B, N,
                       (int)HW, wpr, st, masks, M, need, mask_upd);
    hipLaunchKernelGGL((k_cov_final<true, true>), dim3((unsigned)(B * N)), dim3(kRowBlock), 0, stream, st, N, 0, nblk,
                       0ull, nullptr, M, out, stale, (int)HW, wpr, R, stats);
  } else {
    hipLaunchKernelGGL(k_score_pass<false>, dim3((unsigned)nblk), dim3(kSelBlock), 0, stream, pair_bits, stale, B, N,
                       (int)HW, wpr, st, masks, M, need, 0ull);
    hipLaunchKernelGGL((k_cov_final<true, false>), dim3(1), dim3(kRowBlock), 0, stream, st, N, 0, nblk, 0ull, nullptr,
                       M, out, nullptr, 0, 0, 1, nullptr);
  }
}

}  // namespace
}  // namespace gc

extern "C" int gc_coverage_update(const uint32_t* pair_bits, int B, int N, int H, int W, const int32_t* anchors, int a,
                                  int R, uint8_t* stale, uint32_t* stats, hipStream_t stream) {
  clear_error();
  unsigned long long mask = 0;
  const int rc = check_update(pair_bits, B, N, H, W, anchors, a, R, stale, stats, "gc_coverage_update", &mask);
  if (rc) return rc;
  launch_update(pair_bits, B, N, (size_t)H * W, mask, R, stale, stats, stream);
  return after_launch(stream, "gc_coverage_update");
}

extern "C" size_t gc_coverage_workspace_bytes(void) {
  const size_t n = sizeof(SelState) > sizeof(HistState) ? sizeof(SelState) : sizeof(HistState);
  return (n + 255) / 256 * 256;
}

extern "C" int gc_coverage_select(const uint32_t* pair_bits, const uint8_t* stale, int B, int N, int H, int W, int a,
                                  const int32_t* forced, int n_forced, int32_t* anchors_out, void* workspace,
                                  size_t ws_bytes, hipStream_t stream) {
  clear_error();
  unsigned long long mask = 0;
  const int rc = check_select(pair_bits, stale, B, N, H, W, a, forced, n_forced, anchors_out, workspace, ws_bytes,
                              "gc_coverage_select", &mask);
  if (rc) return rc;
  // the pass reads the staleness only (no update): the cast is for the shared kernel
  launch_select(pair_bits, const_cast<uint8_t*>(stale), B, N, (size_t)H * W, a, mask, n_forced, anchors_out, workspace,
                false, 0ull, 1, nullptr, stream);
  return after_launch(stream, "gc_coverage_select");
}

extern "C" int gc_coverage_score(const uint32_t* pair_bits, const uint8_t* stale, int B, int N, int H, int W,
                                 const int32_t* sets, int M, int a, uint64_t* scores, void* workspace, size_t ws_bytes,
                                 hipStream_t stream) {
  clear_error();
  SetMasks masks;
  const int rc = check_score(pair_bits, stale, B, N, H, W, sets, M, a, scores, workspace, ws_bytes,
                             "gc_coverage_score", &masks);
  if (rc) return rc;
  launch_score(pair_bits, const_cast<uint8_t*>(stale), B, N, (size_t)H * W, masks, M, a, scores, workspace, false, 0ull,
               1, nullptr, stream);
  return after_launch(stream, "gc_coverage_score");
}

extern "C" int gc_coverage_update_select(const uint32_t* pair_bits, int B, int N, int H, int W, const int32_t* anchors,
                                         int a, int R, uint8_t* stale, uint32_t* stats, int a_next,
                                         const int32_t* forced, int n_forced, int32_t* anchors_out, void* workspace,
                                         size_t ws_bytes, hipStream_t stream) {
  clear_error();
  const char* who = "gc_coverage_update_select";
  unsigned long long mask_upd = 0, mask_forced = 0;
  int rc = check_update(pair_bits, B, N, H, W, anchors, a, R, stale, stats, who, &mask_upd);
  if (rc) return rc;
  rc = check_select(pair_bits, stale, B, N, H, W, a_next, forced, n_forced, anchors_out, workspace, ws_bytes, who,
                    &mask_forced);
  if (rc) return rc;
  const size_t ws = gc_coverage_workspace_bytes();
  if (overlaps(stats, (size_t)B * N * 16, workspace, ws) || overlaps(stats, (size_t)B * N * 16, anchors_out, (size_t)a_next * 4))
    return fail(GC_ERR_ALIAS, "%s: stats overlaps the workspace or anchors_out", who);
  launch_select(pair_bits, stale, B, N, (size_t)H * W, a_next, mask_forced, n_forced, anchors_out, workspace, true,
                mask_upd, R, stats, stream);
  return after_launch(stream, who);
}

extern "C" int gc_coverage_update_score(const uint32_t* pair_bits, int B, int N, int H, int W, const int32_t* anchors,
                                        int a, int R, uint8_t* stale, uint32_t* stats, const int32_t* sets, int M,
                                        int a_set, uint64_t* scores, void* workspace, size_t ws_bytes,
                                        hipStream_t stream) {
  clear_error();
  const char* who = "gc_coverage_update_score";
  unsigned long long mask_upd = 0;
  int rc = check_update(pair_bits, B, N, H, W, anchors, a, R, stale, stats, who, &mask_upd);
  if (rc) return rc;
  SetMasks masks;
  rc = check_score(pair_bits, stale, B, N, H, W, sets, M, a_set, scores, workspace, ws_bytes, who, &masks);
  if (rc) return rc;
  const size_t ws = gc_coverage_workspace_bytes();
  if (overlaps(stats, (size_t)B * N * 16, workspace, ws) || overlaps(stats, (size_t)B * N * 16, scores, (size_t)M * 8))
    return fail(GC_ERR_ALIAS, "%s: stats overlaps the workspace or scores", who);
  launch_score(pair_bits, stale, B, N, (size_t)H * W, masks, M, a_set, scores, workspace, true, mask_upd, R, stats,
               stream);
  return after_launch(stream, who);
}
