// Foreground compaction of a chunk of one view's tokens, for the kernels that
// evaluate the correspondence operator over every (token, anchor) pair.
//
// Only a token with a finite position can be seen by an anchor, and about a
// quarter of the tokens is foreground, so a lane per raster token leaves most
// lanes of the silhouette's waves idle and starts whole waves for nothing.
// A block loads kCompactTok consecutive tokens (coalesced), ranks the
// foreground ones in token order and puts their positions side by side in
// LDS; the operator then runs on full waves of them.
//
// Small chunks: with larger ones fewer groups of 64 are partly filled, but a
// dense block's chain of groups grows while its neighbours are empty (8 assets
// x 12 views of 128 x 128: visibility pairs with chunks of 256 / 512 / 1024
// tokens 28 / 30 / 37 us, builder with 128 / 256 17.9 / 19.6 us).  For the same
// reason launches of few chunks do without: both kernels have a direct form.
#pragma once

#include "gc_common.h"
#include "gc_geometry.h"

namespace gc {

// First chunk of the block (x, y): x rotated by three chunks per row y.  Views
// have their foreground in the same places, and blocks are dealt to XCDs and
// CUs round-robin: in plain order some CUs get the dense chunks of every view
// and others the empty ones, where the chunks per view and the CUs have a
// common factor (visibility pairs of 8 assets x 12 views of 128 x 128 32.3 us
// in plain order, 28.0 rotated; 6 x 16 views 40.0 and 33.8; builder 18.7 and
// 17.9; grids without such a factor, 75 x 101 or 160 x 160, the same within
// 3 %; rotations by 1, 7 and 11 in between).
__device__ __forceinline__ int rotated_chunk() { return (int)((blockIdx.x + blockIdx.y * 3u) % gridDim.x); }

// A chunk of TOK tokens: one per thread of a block of TOK.
template <int TOK> struct CompactLds {
  float q[3][TOK];              // positions of the chunk's foreground tokens, in token order
  uint16_t at[TOK];             // their tokens' offsets in the chunk
  int32_t count[TOK / 64];
};

// Rank among the chunk's foreground tokens of this thread's token p0 +
// threadIdx.x of the view map row [HW][3] (-1: background or past the view);
// n_fg: the chunk's foreground count.  Every thread of the block must call
// it; it ends on a barrier.
template <int TOK>
__device__ __forceinline__ int compact_foreground(const float* __restrict__ row, int HW, int p0, CompactLds<TOK>& s,
                                                  int* n_fg) {
  const int wv = (int)threadIdx.x / 64;
  const int p = p0 + (int)threadIdx.x;
  const float* pp = row + (int64_t)(p < HW ? p : HW - 1) * 3;
  const float P[3] = {pp[0], pp[1], pp[2]};
  const bool fg = p < HW && finite_f(P[0]) && finite_f(P[1]) && finite_f(P[2]);
  const unsigned long long m = __ballot(fg);
  if (__lane_id() == 0) s.count[wv] = __popcll(m);
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < TOK / 64; ++w) {
    const int c = s.count[w];
    before += w < wv ? c : 0;
    total += c;
  }
  int rank = -1;
  if (fg) {
    rank = before + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    s.q[0][rank] = P[0];
    s.q[1][rank] = P[1];
    s.q[2][rank] = P[2];
    s.at[rank] = (uint16_t)threadIdx.x;
  }
  __syncthreads();
  *n_fg = __builtin_amdgcn_readfirstlane(total);   // the same for every thread
  return rank;
}

}  // namespace gc
