// Correspondence builder: G_{A->v} for every non-anchor view of every asset,
// for one anchor set (once per asset and anchor set; the rotation has only a
// few distinct sets, so the host caches one build per set).
//
// Every float operation is written in a fixed order and the library is
// compiled without contraction, so the tap choice (an integer decision taken
// in float) is reproducible exactly.
//
// Visibility reductions use wavefront ballots: the anchors that see a token
// are counted by a ballot over its lane group, and each wave counts its
// visible pairs / tokens / taps with ballot + popcount before one lane adds
// them to the asset's counters.
#include "gc_common.h"
#include "gc_compact.h"
#include "gc_geometry.h"

namespace gc {
namespace {

// Launch size of the builder, in blocks per CU (256 CUs).  The coverage
// counters cost one device-scope atomic per block and counter, and atomics
// on one address serialise, so a build that counts uses fewer, longer
// blocks; one that does not uses enough blocks to hide its load latency.
constexpr int kBuildBlocksPerCU = 16;
constexpr int kBuildBlocksPerCUStats = 4;
// Tokens per chunk of a view.  Compacted chunks, a token per thread: groups of
// four lanes 128 (8 assets x 8 target views of 128 x 128 with 4 anchors 17.9 us;
// 256 19.6); with the counters, whose atomics grow with the blocks, 256 (21.6
// us; 192 25.5, 128 28.4), as with groups of eight lanes (3 assets x 10 target
// views of 75 x 101 with 6 anchors 12.0 us; 128 13.7, 64 15.4).
constexpr int build_threads(int group, bool count, bool compact) { return compact && group == 4 && !count ? 128 : 256; }
constexpr int build_tok(int group, bool count, bool compact) {
  return build_threads(group, count, compact) / (compact ? 1 : group);
}

// Target tokens up to which a build takes the direct launch.  Direct /
// compacted in us, one asset unless said: 5 target views of 64 x 64, 1 anchor
// 3.8 / 7.1; 4 of 64 x 64, 8 anchors 4.1 / 11.3; 8 assets x 8 of 128 x 128 (2^20
// tokens), 4 anchors 20.5 / 17.9; around the lines: 4 x 8 of 128 x 128 (2^19), 4
// anchors 12.3 / 13.4; 4 x 10 (655,360), 2 anchors 13.0 / 12.7; 8 x 6 (786,432), 6
// anchors 25.6 / 25.9; 8 x 7 (917,504), 5 anchors 28.2 / 26.5.  With the counters,
// whose few long blocks hide less of the chain: 12 of 64 x 64 (49,152), 4
// anchors 9.4 / 9.7; 2 x 8 of 64 x 64 (65,536) 10.7 / 9.8.
bool build_direct(int64_t tokens, int a, bool count) {
  return tokens <= (count ? 3 << 14 : a <= 4 ? 1 << 19 : 3 << 18);
}

struct BuildArgs {
  const float* pos;
  const gc_camera* cams;
  const float* bbox;
  int32_t* corr;
  float* weights;
  uint32_t* stats;
  int N, H, W, a, K, NT;
  int32_t anchor_view[GC_MAX_ANCHORS];
  int32_t target_view[GC_MAX_VIEWS];
};

__global__ void k_zero_u32(uint32_t* __restrict__ p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

__device__ __forceinline__ uint32_t wave_count(bool pred) {
  return (uint32_t)__popcll(__ballot(pred));
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o);
  return v;
}

// A block's visible pairs, visible tokens, foreground tokens and kept taps.
struct BuildCounts {
  uint32_t pairs = 0, pix = 0, fg = 0;   // wave totals (uniform across the wave)
  uint32_t taps_lane = 0;                // this lane's kept taps, summed over the wave at the end
};

// One (token, anchor slot s) per lane, a token's slots in G adjacent lanes:
// projection into the slot's anchor, the four footprint taps' tests, the K
// nearest and their normalised area weights; the number of anchors that see
// the token (n_vis) is a ballot over the lane group.  Words and weights of one
// token are adjacent, so a group writes them coalesced.  eval: the token is
// foreground and the slot an anchor's; store: the slot's word is written;
// row: the token's row of the operator.  Every lane of the wave calls it.
template <int G, bool COUNT>
__device__ __forceinline__ void build_pair(const BuildArgs& g, const float (&P)[3], const gc_camera& cam,
                                           const float* __restrict__ src, float tol2, int s, bool eval, bool store,
                                           int64_t row, BuildCounts& cnt) {
  AnchorProj pj = anchor_project(P, cam, g.H, g.W);
  pj.ok &= eval;
  AnchorTaps at;
  at.word = 0;
  at.mask = 0;
  if (__ballot(pj.ok)) {
    const TapPos tp = anchor_tap_positions(pj, src, g.H, g.W);
    at = anchor_select(P, pj, tp, g.H, g.W, g.K, tol2);
  }
  // n_vis: anchors of this token that see it -- a ballot over the lane group
  const unsigned long long seen = __ballot(at.word != 0);
  const int n_vis = __popcll((seen >> (__lane_id() & ~(G - 1))) & ((1ull << G) - 1));
  if (store) g.corr[row * g.a + s] = at.word;
  // weights only for pairs the anchor sees: the transport reads a pair's
  // weights only when its word is non-zero (most pairs' words are zero)
  if (at.word != 0) {
    float out[4] = {0.f, 0.f, 0.f, 0.f};
    const float inv = (float)n_vis;
    if (__ballot((n_vis & (n_vis - 1)) != 0)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) at.wk[k] = at.wk[k] / inv;
    } else {   // dividing by a power of two is multiplying by its exact reciprocal
      const float rcp = __builtin_ldexpf(1.0f, -__builtin_ctz((unsigned)n_vis));
#pragma unroll
      for (int k = 0; k < 4; ++k) at.wk[k] = at.wk[k] * rcp;
    }
#pragma unroll
    for (int k = 3; k >= 0; --k) {   // the kept taps in ascending order, zeros behind them
      const bool keep = at.mask & (1 << k);
      const float w = at.wk[k];
      out[3] = keep ? out[2] : out[3];
      out[2] = keep ? out[1] : out[2];
      out[1] = keep ? out[0] : out[1];
      out[0] = keep ? w : out[0];
    }
    float* ww = g.weights + (row * g.a + s) * g.K;
    if (g.K == 4) {   // 16-byte aligned: the weights base is, and each (token, slot) row is 16 bytes
      *reinterpret_cast<float4*>(ww) = make_float4(out[0], out[1], out[2], out[3]);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q < g.K) ww[q] = out[q];
    }
  }
  if (COUNT) {
    cnt.pairs += (uint32_t)__popcll(seen);
    cnt.pix += wave_count(s == 0 && n_vis > 0);
    cnt.taps_lane += (uint32_t)__popc(at.mask);
  }
}

// grid: y = b * NT + target slot; x = blocks that stride over the view's
// chunks.  The block's anchor cameras are staged in LDS.  A block counts its
// visible pairs / tokens / foreground tokens / taps over all its chunks and
// adds them to the asset's counters once: few blocks per asset keep the
// same-address atomics from serialising.
//
// COMPACT: a block compacts the foreground tokens of a chunk of one target
// view, writes the other tokens' zero words, and then gives each (compacted
// token, anchor slot) a lane: a group of G = 4 or 8 adjacent lanes serves one
// token (lanes with slot >= a idle).  Bound by vector-ALU issue (10 of 17.9 us)
// and by the chain of a block's loads: 8 assets x 8 target views of 128 x 128
// with 4 anchors 17.9 us, 21.5 with the counters, against 20.5 and 30.6
// without the compaction.
// Otherwise: a lane per (raster token, slot), for small launches, which last
// about as long as one block's chain: one group of tokens here, up to G of
// them, one after another, in a compacted chunk.
template <int G, bool COUNT, bool COMPACT>
__global__ __launch_bounds__(build_threads(G, COUNT, COMPACT)) void k_build(BuildArgs g) {
  constexpr int kThreads = build_threads(G, COUNT, COMPACT);
  constexpr int kTok = build_tok(G, COUNT, COMPACT);
  __shared__ CompactLds<COMPACT ? kTok : 64> list;
  __shared__ gc_camera cam_lds[GC_MAX_ANCHORS];
  __shared__ int32_t view_lds[GC_MAX_ANCHORS];   // a lane's own slot: from LDS, not a per-lane kernel-argument load
  const int HW = g.H * g.W;
  const int bt = blockIdx.y;
  const int b = bt / g.NT;
  const int ti = bt - b * g.NT;
  const float* view = g.pos + ((int64_t)b * g.N + g.target_view[ti]) * HW * 3;
  const int64_t row0 = ((int64_t)b * g.NT + ti) * HW;
  if (threadIdx.x < g.a) {
    view_lds[threadIdx.x] = g.anchor_view[threadIdx.x];
    cam_lds[threadIdx.x] = g.cams[(int64_t)b * g.N + g.anchor_view[threadIdx.x]];
  }
  const float tol2 = g.bbox[(int64_t)b * 8 + 6];
  const int s = (int)threadIdx.x & (G - 1);      // anchor slot of this lane
  const int sc = s < g.a ? s : 0;
  const int n_chunks = (HW + kTok - 1) / kTok;
  BuildCounts cnt;
  if constexpr (COMPACT) {
    for (int chunk = rotated_chunk(); chunk < n_chunks; chunk += gridDim.x) {
      const int p0 = chunk * kTok;
      int n_fg;
      const int rank = compact_foreground(view, HW, p0, list, &n_fg);   // its barriers also order the cameras
      const int p = p0 + (int)threadIdx.x;
      if (rank < 0 && p < HW) {   // a background token: no anchor sees it
        int32_t* cw = g.corr + (row0 + p) * g.a;
        if (G == 4 && g.a == 4) {
          *reinterpret_cast<int4*>(cw) = make_int4(0, 0, 0, 0);
        } else {
          for (int q = 0; q < g.a; ++q) cw[q] = 0;
        }
      }
      if (COUNT && threadIdx.x / 64 == 0) cnt.fg += (uint32_t)n_fg;
      for (int i0 = 0; i0 < n_fg; i0 += kThreads / G) {
        const int i = i0 + (int)threadIdx.x / G;
        const bool live = i < n_fg && s < g.a;
        const int ic = i < n_fg ? i : 0;
        const float P[3] = {list.q[0][ic], list.q[1][ic], list.q[2][ic]};
        build_pair<G, COUNT>(g, P, cam_lds[sc], g.pos + ((int64_t)b * g.N + view_lds[sc]) * HW * 3, tol2, s, live, live,
                             row0 + p0 + list.at[ic], cnt);
      }
      __syncthreads();   // the next chunk's compaction overwrites the list
    }
  } else {
    __syncthreads();
    for (int chunk = blockIdx.x; chunk < n_chunks; chunk += gridDim.x) {
      const int p = chunk * kTok + (int)threadIdx.x / G;
      const float* pp = view + (int64_t)min(p, HW - 1) * 3;
      const float P[3] = {pp[0], pp[1], pp[2]};
      const bool fg = p < HW && finite_f(P[0]) && finite_f(P[1]) && finite_f(P[2]);
      if (COUNT) cnt.fg += wave_count(s == 0 && fg);
      build_pair<G, COUNT>(g, P, cam_lds[sc], g.pos + ((int64_t)b * g.N + view_lds[sc]) * HW * 3, tol2, s,
                           fg && s < g.a, p < HW && s < g.a, row0 + p, cnt);
    }
  }

  if constexpr (COUNT) {
    // blocks never straddle assets (grid y is per asset and target): the
    // block sums its waves' totals in LDS, one thread per counter adds them
    // to the asset's counters
    __shared__ uint32_t part[kThreads / 64][4];
    const uint32_t c_taps = wave_sum(cnt.taps_lane);
    const int wv = (int)threadIdx.x / 64;
    if (__lane_id() == 0) {
      part[wv][0] = cnt.pairs;
      part[wv][1] = cnt.pix;
      part[wv][2] = cnt.fg;
      part[wv][3] = c_taps;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
      uint32_t sum = 0;
      for (int w = 0; w < kThreads / 64; ++w) sum += part[w][threadIdx.x];
      if (sum) atomicAdd(g.stats + (int64_t)b * 4 + threadIdx.x, sum);
    }
  }
}

}  // namespace
}  // namespace gc

using namespace gc;

extern "C" int gc_build_correspondence(const float* pos, const gc_camera* cams, int B, int N, int H, int W,
                                       const int32_t* anchors, int a, int K, const float* bbox, int32_t* corr,
                                       float* weights, uint32_t* stats, hipStream_t stream) {
  clear_error();
  if (!pos || !cams || !anchors || !bbox) return fail(GC_ERR_ARG, "build: null input pointer");
  if (B < 1 || N < 1 || H < 1 || W < 1) return fail(GC_ERR_SHAPE, "build: bad shape B=%d N=%d H=%d W=%d", B, N, H, W);
  if (N > GC_MAX_VIEWS) return fail(GC_ERR_CAPACITY, "build: N=%d exceeds %d", N, GC_MAX_VIEWS);
  if (H > GC_MAX_GRID || W > GC_MAX_GRID) return fail(GC_ERR_CAPACITY, "build: grid %dx%d exceeds %d", H, W, GC_MAX_GRID);
  if (a < 1 || a > N) return fail(GC_ERR_ARG, "build: a=%d outside [1, N=%d]", a, N);
  if (a > GC_MAX_ANCHORS) return fail(GC_ERR_CAPACITY, "build: a=%d exceeds %d", a, GC_MAX_ANCHORS);
  if (K < 1 || K > 4) return fail(GC_ERR_ARG, "build: K=%d outside [1, 4]", K);
  if ((int64_t)B * (N - a) > 65535) return fail(GC_ERR_CAPACITY, "build: B*(N-a) exceeds 65535");
  BuildArgs g{};
  bool is_anchor[GC_MAX_VIEWS] = {};
  for (int s = 0; s < a; ++s) {
    const int u = anchors[s];
    if (u < 0 || u >= N) return fail(GC_ERR_ARG, "build: anchor %d outside [0, %d)", u, N);
    if (is_anchor[u]) return fail(GC_ERR_ARG, "build: anchor %d listed twice", u);
    is_anchor[u] = true;
    g.anchor_view[s] = u;
  }
  const int NT = N - a;
  if (NT > 0 && (!corr || !weights)) return fail(GC_ERR_ARG, "build: null output pointer");
  if (!aligned16(pos) || (corr && !aligned16(corr)) || (weights && !aligned16(weights)))
    return fail(GC_ERR_ALIGN, "build: pos, corr and weights must be 16-byte aligned");
  const size_t HW = (size_t)H * W;
  const size_t n_corr = (size_t)B * NT * HW * a * 4, n_w = (size_t)B * NT * HW * a * K * 4;
  const size_t n_pos = (size_t)B * N * HW * 12;
  if (overlaps(corr, n_corr, pos, n_pos) || overlaps(weights, n_w, pos, n_pos) || overlaps(corr, n_corr, weights, n_w) ||
      overlaps(stats, (size_t)B * 16, corr, n_corr) || overlaps(stats, (size_t)B * 16, weights, n_w))
    return fail(GC_ERR_ALIAS, "build: outputs overlap each other or the position maps");
  int t = 0;
  for (int v = 0; v < N; ++v)
    if (!is_anchor[v]) g.target_view[t++] = v;
  g.pos = pos;
  g.cams = cams;
  g.bbox = bbox;
  g.corr = corr;
  g.weights = weights;
  g.stats = stats;
  g.N = N;
  g.H = H;
  g.W = W;
  g.a = a;
  g.K = K;
  g.NT = NT;
  if (stats) hipLaunchKernelGGL(k_zero_u32, dim3((4 * B + 255) / 256), dim3(256), 0, stream, stats, 4 * B);
  if (NT > 0) {
    // x-blocks per (asset, target), from the launch size above
#define GC_BUILD(G_, COUNT_, COMPACT_)                                                                        \
  do {                                                                                                        \
    constexpr int tok = build_tok(G_, COUNT_, COMPACT_);                                                      \
    const int64_t chunks = ((int64_t)HW + tok - 1) / tok;                                                     \
    const int64_t per_cu = COUNT_ ? kBuildBlocksPerCUStats : kBuildBlocksPerCU;                               \
    int64_t bx = (per_cu * 256 + (int64_t)B * NT - 1) / ((int64_t)B * NT);                                    \
    if (bx > chunks) bx = chunks;                                                                             \
    hipLaunchKernelGGL((k_build<G_, COUNT_, COMPACT_>), dim3((unsigned)bx, (unsigned)(B * NT)),               \
                       dim3(build_threads(G_, COUNT_, COMPACT_)), 0, stream, g);                              \
  } while (0)
#define GC_BUILD_G(G_)                                                              \
  do {                                                                              \
    if (stats) {                                                                    \
      if (direct) GC_BUILD(G_, true, false); else GC_BUILD(G_, true, true);         \
    } else {                                                                        \
      if (direct) GC_BUILD(G_, false, false); else GC_BUILD(G_, false, true);       \
    }                                                                               \
  } while (0)
    const bool direct = build_direct((int64_t)B * NT * (int64_t)HW, a, stats != nullptr);
    if (a <= 4) GC_BUILD_G(4); else GC_BUILD_G(8);
#undef GC_BUILD_G
#undef GC_BUILD
  }
  return after_launch(stream, "gc_build_correspondence");
}
