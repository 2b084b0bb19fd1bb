// Once-per-asset position-map kernels: area downsample to the latent grid and
// the per-asset bounding box / squared match tolerance.
//
// Both are HBM-streaming reductions (no contraction): each render sample is
// read once.  The downsample sums each block in double in the order of a
// plain row-major loop (rows of the block, then samples in a row), whichever
// kernel runs, so its float result does not depend on the launch shape.
#include "gc_common.h"

namespace gc {
namespace {

constexpr int kBlock = 256;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// One thread per latent pixel, reading its f x f block directly (any f).
__global__ __launch_bounds__(kBlock) void k_downsample(const float* __restrict__ hi, int64_t n_pix,
                                                       int Hr, int Wr, int f, int H, int W,
                                                       float* __restrict__ lo) {
  const int64_t gid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (gid >= n_pix) return;
  const int i = (int)(gid % W);
  const int64_t mj = gid / W;
  const int j = (int)(mj % H);
  const int64_t m = mj / H;
  int n_fg = 0;
  double sx = 0.0, sy = 0.0, sz = 0.0;
  for (int dy = 0; dy < f; ++dy) {
    const float* row = hi + ((m * Hr + (int64_t)j * f + dy) * Wr + (int64_t)i * f) * 3;
    for (int dx = 0; dx < f; ++dx) {
      const float x = row[3 * dx], y = row[3 * dx + 1], z = row[3 * dx + 2];
      if (finite_f(x) && finite_f(y) && finite_f(z)) {
        n_fg += 1;
        sx += (double)x;
        sy += (double)y;
        sz += (double)z;
      }
    }
  }
  float* o = lo + gid * 3;
  if (2 * n_fg < f * f) {
    const float qnan = __uint_as_float(0x7fc00000u);
    o[0] = qnan;
    o[1] = qnan;
    o[2] = qnan;
  } else {
    const double n = (double)n_fg;
    o[0] = (float)(sx / n);
    o[1] = (float)(sy / n);
    o[2] = (float)(sz / n);
  }
}

// Staged variant: a wave takes 64 consecutive latent pixels.  Its vectors and
// rows in flight are unrolled for the factor, so it exists for the factors that
// renders and latent grids of this library's workloads have between them (2, 3,
// 4, 6, 8, 16); every other one takes the direct kernel, at the cost of its
// strided loads: 10 maps to 96 x 96 by 5 10.4 us and by 10 53.8, 6 to 64 x 64 by
// 12 50.1 (by 16, staged, 19.7), 6 to 32 x 32 by 32 333.
// Per render row the pixels' segments (3F floats each) are read as aligned
// vectors in memory order, one per lane, so that every load instruction covers
// whole lines, and are handed to the pixels' lanes through the wave's own LDS
// (no barrier: LDS operations of one wave keep their order); the next rows'
// loads are in flight meanwhile.  Each lane folds its samples in the same
// row-major order as the direct kernel.
// HBM-bound: 8 x 12 renders of 1024 x 1024 by f = 8 take 198 us (6.2 TB/s;
// single-precision sums or no finiteness tests: 198), against 213 with plain
// loads, whether staged or 96 strided bytes per lane.  Against one thread per
// pixel reading its block sample by sample: f = 16 to 64 x 64 1847 -> 206 us,
// f = 6 to 128 x 128 290 -> 123 us, f = 3 to 101 x 75 21 -> 15 us.
template <int F> struct Stage {
  static constexpr int kV = F % 4 == 0 ? 4 : F % 2 == 0 ? 2 : 1;   // floats per vector (a segment starts on a multiple)
  static constexpr int kVec = 3 * F / kV;                          // vectors per segment
  static constexpr int kRows = F == 3 ? 3 : F == 4 ? 4 : F == 16 ? 1 : 2;   // rows loaded together
  static_assert(F % kRows == 0, "whole steps");
  typedef float Vec __attribute__((ext_vector_type(kV)));
};

template <int F>
__global__ __launch_bounds__(kBlock) void k_downsample_staged(const float* __restrict__ hi, int64_t n_pix, int Hr,
                                                              int Wr, int H, int W, float* __restrict__ lo) {
  using S = Stage<F>;
  using Vec = typename S::Vec;
  __shared__ Vec stage[kBlock / 64][S::kRows][64 * S::kVec];
  const int lane = __lane_id();
  Vec(*mine)[64 * S::kVec] = stage[threadIdx.x / 64];
  const int64_t gid0 = (int64_t)blockIdx.x * kBlock;
  const int64_t gid = gid0 + threadIdx.x;
  // this lane's pixel (the last one, where the block reaches past it): the
  // block's first pixel is the same for all lanes, the rest is 32-bit
  const int64_t mj0 = gid0 / W;
  const uint32_t i1 = (uint32_t)(gid0 - mj0 * W) + (uint32_t)(min(gid, n_pix - 1) - gid0);
  const int64_t m0 = mj0 / H;
  const uint32_t j1 = (uint32_t)(mj0 - m0 * H) + i1 / (uint32_t)W;
  const uint32_t i = i1 % (uint32_t)W, j = j1 % (uint32_t)H;
  const int64_t m = m0 + j1 / (uint32_t)H;
  const int64_t rs = (int64_t)Wr * 3 / S::kV;   // vectors per render row
  const int64_t base = (m * Hr + (int64_t)j * F) * rs + (int64_t)i * S::kVec;
  const int64_t base0 = __shfl(base, 0);        // the wave's first pixel
  const Vec* src = reinterpret_cast<const Vec*>(hi) + base0;
  const int32_t rel = (int32_t)(base - base0);
  int32_t off[S::kVec];                         // vector 64 c + lane of the wave's segments in memory order
#pragma unroll
  for (int c = 0; c < S::kVec; ++c) {
    const int q = c * 64 + lane, px = q / S::kVec;
    off[c] = __shfl(rel, px) + (q - px * S::kVec);
  }
  Vec buf[S::kRows][S::kVec];
  auto load = [&](int dy0) {
#pragma unroll
    for (int r = 0; r < S::kRows; ++r)
#pragma unroll
      for (int c = 0; c < S::kVec; ++c)
        buf[r][c] = __builtin_nontemporal_load(src + (int64_t)(dy0 + r) * rs + off[c]);
  };
  int n_fg = 0;
  double sx = 0.0, sy = 0.0, sz = 0.0;
  load(0);
  for (int dy0 = 0; dy0 < F; dy0 += S::kRows) {
#pragma unroll
    for (int r = 0; r < S::kRows; ++r)
#pragma unroll
      for (int c = 0; c < S::kVec; ++c) mine[r][c * 64 + lane] = buf[r][c];
    if (dy0 + S::kRows < F) load(dy0 + S::kRows);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int r = 0; r < S::kRows; ++r) {
      float seg[3 * F];
#pragma unroll
      for (int c = 0; c < S::kVec; ++c) {
        const Vec q = mine[r][lane * S::kVec + c];
#pragma unroll
        for (int e = 0; e < S::kV; ++e) seg[c * S::kV + e] = q[e];
      }
#pragma unroll
      for (int dx = 0; dx < F; ++dx) {
        const float x = seg[3 * dx], y = seg[3 * dx + 1], z = seg[3 * dx + 2];
        if (finite_f(x) && finite_f(y) && finite_f(z)) {
          n_fg += 1;
          sx += (double)x;
          sy += (double)y;
          sz += (double)z;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if (gid >= n_pix) return;
  float* o = lo + gid * 3;
  if (2 * n_fg < F * F) {
    const float qnan = __uint_as_float(0x7fc00000u);
    o[0] = qnan;
    o[1] = qnan;
    o[2] = qnan;
  } else {
    const double n = (double)n_fg;
    o[0] = (float)(sx / n);
    o[1] = (float)(sy / n);
    o[2] = (float)(sz / n);
  }
}

// Vector variant for f = 4 and 8 and small inputs: one thread per latent
// pixel, each of its F render rows read as 3F/4 aligned 16-byte vectors (the
// pixel's segment of a render row is 3F contiguous floats at a multiple of 48
// bytes), kRows rows in flight per step.  The strided vectors of one wave tile
// a contiguous run of the render row, so L2 serves the lines neighbouring
// lanes share (plain loads: a nontemporal hint makes those lines miss); without
// the staging's LDS round trip per step each thread folds its samples in the
// same row-major order as the direct kernel.
template <int F>
__global__ __launch_bounds__(kBlock) void k_downsample_vec(const float* __restrict__ hi, int64_t n_pix, int Hr,
                                                           int Wr, int H, int W, float* __restrict__ lo) {
  constexpr int kRow4 = 3 * F / 4;          // vectors per render-row segment
  constexpr int kRows = 4;                  // rows loaded together
  static_assert(F % 4 == 0, "F must be a multiple of 4");
  const int64_t gid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (gid >= n_pix) return;
  const int i = (int)(gid % W);
  const int64_t mj = gid / W;
  const int j = (int)(mj % H);
  const int64_t m = mj / H;
  const f32x4* src = reinterpret_cast<const f32x4*>(hi + ((m * Hr + (int64_t)j * F) * Wr + (int64_t)i * F) * 3);
  const int64_t rs = (int64_t)Wr * 3 / 4;   // vectors per render row
  int n_fg = 0;
  double sx = 0.0, sy = 0.0, sz = 0.0;
  for (int dy0 = 0; dy0 < F; dy0 += kRows) {
    float buf[kRows][3 * F];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
      for (int c = 0; c < kRow4; ++c) {
        const f32x4 q = src[(int64_t)(dy0 + r) * rs + c];
        buf[r][4 * c] = q.x;
        buf[r][4 * c + 1] = q.y;
        buf[r][4 * c + 2] = q.z;
        buf[r][4 * c + 3] = q.w;
      }
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
      for (int dx = 0; dx < F; ++dx) {
        const float x = buf[r][3 * dx], y = buf[r][3 * dx + 1], z = buf[r][3 * dx + 2];
        if (finite_f(x) && finite_f(y) && finite_f(z)) {
          n_fg += 1;
          sx += (double)x;
          sy += (double)y;
          sz += (double)z;
        }
      }
  }
  float* o = lo + gid * 3;
  if (2 * n_fg < F * F) {
    const float qnan = __uint_as_float(0x7fc00000u);
    o[0] = qnan;
    o[1] = qnan;
    o[2] = qnan;
  } else {
    const double n = (double)n_fg;
    o[0] = (float)(sx / n);
    o[1] = (float)(sy / n);
    o[2] = (float)(sz / n);
  }
}

// Input bytes up to which f = 4 and 8 take the vector variant, whose chain per
// block is shorter; above, the staged one's whole-line loads count.  Vector /
// staged in us, the same input again and again (a fresh one each time): f = 8,
// 4 maps to 32 x 32 5.5 / 6.8 (6.1 / 7.4), 6 to 64 x 64 (18.9 MB) 5.9 / 7.3 (8.0 /
// 7.9), 10 to 96 x 96 (70.8 MB) 13.3 / 13.3 (17.1 / 15.8); f = 4, 4 to 32 x 32 2.9 /
// 3.4 (2.9 / 3.4), 24 to 96 x 96 (42.5 MB) 8.0 / 8.4 (10.2 / 10.8), 48 to 128 x 128
// (151 MB) 24.2 / 25.7 (28.8 / 27.5), 96 to 128 x 128 51.5 / 51.1 (56.2 / 52.0).
constexpr int64_t kVecMaxBytes = 48ll << 20;

// Order-preserving float <-> uint32 encoding for integer atomics.
__device__ __forceinline__ uint32_t enc_ord(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float dec_ord(uint32_t e) {
  return __uint_as_float((e & 0x80000000u) ? (e & 0x7fffffffu) : ~e);
}

// bbox[b] is used as the accumulator while the reduction over several blocks
// runs: words 0..2 encoded min, 3..5 encoded max, 6 blocks done, 7 = 1 once a
// foreground sample is seen.
__global__ void k_bbox_init(uint32_t* __restrict__ acc, int B) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  uint32_t* a = acc + (int64_t)b * 8;
  const uint32_t pinf = 0xFF800000u, ninf = 0x007FFFFFu;  // enc(+inf), enc(-inf)
  a[0] = pinf; a[1] = pinf; a[2] = pinf;
  a[3] = ninf; a[4] = ninf; a[5] = ninf;
  a[6] = 0u; a[7] = 0u;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o));
  return v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
  return v;
}

// The asset's box and squared tolerance from the encoded extremes.
__device__ __forceinline__ void bbox_write(const uint32_t (&e)[6], bool seen, float tol_frac, float* o) {
  if (!seen) {
    for (int c = 0; c < 8; ++c) o[c] = 0.0f;
    return;
  }
  float mn[3], mx[3];
  for (int c = 0; c < 3; ++c) {
    mn[c] = dec_ord(e[c]);
    mx[c] = dec_ord(e[3 + c]);
  }
  const float ex = mx[0] - mn[0], ey = mx[1] - mn[1], ez = mx[2] - mn[2];
  const float d2 = (ex * ex + ey * ey) + ez * ez;
  const float tf2 = tol_frac * tol_frac;
  for (int c = 0; c < 3; ++c) {
    o[c] = mn[c];
    o[3 + c] = mx[c];
  }
  o[6] = tf2 * d2;
  o[7] = 0.0f;
}

// grid (chunks, B): every thread folds a strided slice of asset b's samples,
// kBoxUnroll in flight; waves reduce with cross-lane shuffles, the block
// through LDS.  One chunk: the block writes the result itself.  More: lanes of
// its first wave add the block's extremes to the accumulator, and the last
// block to finish turns them into the result (no block waits).
// Few, large blocks: the atomics on an asset's one accumulator line serialise.
// (48 blocks per asset of one load in flight per thread, and launches of their
// own for clearing and for the result, took 22 us for 8 assets x 196,608
// samples and 13.4 us for 6144.)
constexpr int kBoxBlock = 1024;
constexpr int kBoxUnroll = 4;   // samples a thread has in flight
// Measured with the calls' launches: 24,576 samples 7.9 us in one block, 10.6
// in several; 92,160 samples 17.9 and 10.6.  8 assets x 196,608 samples with
// 2048 / 4096 / 8192 / 16384 samples per block: 29 / 15.5 / 11.5 / 10.5 us.
constexpr int64_t kBoxSingle = 32768;
constexpr int64_t kBoxPerBlock = 16384;
constexpr int64_t kBoxMaxChunks = 64;
__global__ __launch_bounds__(kBoxBlock) void k_bbox_accum(const float* __restrict__ pos, int64_t per_asset,
                                                          float tol_frac, uint32_t* __restrict__ acc) {
  __shared__ uint32_t part[7][kBoxBlock / 64];
  __shared__ int last;
  const int b = blockIdx.y;
  const float* p = pos + (int64_t)b * per_asset * 3;
  uint32_t mn[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
  uint32_t mx[3] = {0u, 0u, 0u};
  bool any = false;
  const int64_t stride = (int64_t)gridDim.x * kBoxBlock;
  for (int64_t q0 = (int64_t)blockIdx.x * kBoxBlock + threadIdx.x; q0 < per_asset; q0 += kBoxUnroll * stride) {
    float v[kBoxUnroll][3];
#pragma unroll
    for (int u = 0; u < kBoxUnroll; ++u) {   // past the end: the last sample again
      const float* s = p + 3 * min(q0 + u * stride, per_asset - 1);
#pragma unroll
      for (int c = 0; c < 3; ++c) v[u][c] = s[c];
    }
#pragma unroll
    for (int u = 0; u < kBoxUnroll; ++u) {
      if (!(finite_f(v[u][0]) && finite_f(v[u][1]) && finite_f(v[u][2]))) continue;
      any = true;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const uint32_t e = enc_ord(v[u][c]);
        mn[c] = min(mn[c], e);
        mx[c] = max(mx[c], e);
      }
    }
  }
  const uint32_t seen = __ballot(any) ? 1u : 0u;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    mn[c] = wave_min_u32(mn[c]);
    mx[c] = wave_max_u32(mx[c]);
  }
  if (__lane_id() == 0) {
    const int wv = threadIdx.x / 64;
    for (int c = 0; c < 3; ++c) {
      part[c][wv] = mn[c];
      part[3 + c][wv] = mx[c];
    }
    part[6][wv] = seen;
  }
  __syncthreads();
  // lane c of the first wave folds quantity c of the waves
  uint32_t fold = 0u;
  if (threadIdx.x < 7) {
    fold = part[threadIdx.x][0];
    for (int w = 1; w < kBoxBlock / 64; ++w) {
      const uint32_t x = part[threadIdx.x][w];
      fold = threadIdx.x < 3 ? min(fold, x) : max(fold, x);
    }
  }
  uint32_t* a = acc + (int64_t)b * 8;
  if (gridDim.x > 1) {   // the ticket's release waits for its own wave, which is the one that adds
    if (threadIdx.x < 3) atomicMin(a + threadIdx.x, fold);
    else if (threadIdx.x < 6) atomicMax(a + threadIdx.x, fold);
    else if (threadIdx.x == 6) atomicOr(a + 7, fold);
    __syncthreads();
    if (threadIdx.x == 0)
      last = __hip_atomic_fetch_add(a + 6, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!last || threadIdx.x >= 7) return;
    fold = __hip_atomic_load(a + (threadIdx.x < 6 ? threadIdx.x : 7u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (threadIdx.x >= 7) {
    return;
  }
  uint32_t e[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) e[c] = (uint32_t)__shfl((int)fold, c);
  const bool on = __shfl((int)fold, 6) != 0;
  if (threadIdx.x == 0) bbox_write(e, on, tol_frac, reinterpret_cast<float*>(a));
}

}  // namespace
}  // namespace gc

using namespace gc;

extern "C" int gc_posmap_downsample(const float* pos_hi, int64_t n_maps, int Hr, int Wr, int f,
                                    float* pos_lat, hipStream_t stream) {
  clear_error();
  if (!pos_hi || !pos_lat) return fail(GC_ERR_ARG, "downsample: null pointer");
  if (n_maps < 0 || Hr < 1 || Wr < 1) return fail(GC_ERR_SHAPE, "downsample: bad shape n_maps=%lld Hr=%d Wr=%d",
                                                 (long long)n_maps, Hr, Wr);
  if (f < 1 || f > 64 || Hr % f || Wr % f)
    return fail(GC_ERR_SHAPE, "downsample: factor %d must be in [1, 64] and divide Hr=%d, Wr=%d", f, Hr, Wr);
  const int H = Hr / f, W = Wr / f;
  if (H > GC_MAX_GRID || W > GC_MAX_GRID)
    return fail(GC_ERR_CAPACITY, "downsample: latent grid %dx%d exceeds %d", H, W, GC_MAX_GRID);
  if (!aligned16(pos_hi) || !aligned16(pos_lat)) return fail(GC_ERR_ALIGN, "downsample: pointers must be 16-byte aligned");
  const size_t nin = (size_t)n_maps * Hr * Wr * 3 * 4, nout = (size_t)n_maps * H * W * 3 * 4;
  if (overlaps(pos_hi, nin, pos_lat, nout)) return fail(GC_ERR_ALIAS, "downsample: output overlaps input");
  const int64_t n_pix = n_maps * (int64_t)H * W;
  if (n_pix == 0) return GC_OK;
  const int64_t blocks = (n_pix + kBlock - 1) / kBlock;
  if (blocks > 0x7fffffff) return fail(GC_ERR_CAPACITY, "downsample: too many latent pixels");
  const dim3 grid((unsigned)blocks), block(kBlock);
#define GC_STAGED(F_)                                                                                     \
  case F_:                                                                                                \
    hipLaunchKernelGGL(k_downsample_staged<F_>, grid, block, 0, stream, pos_hi, n_pix, Hr, Wr, H, W, pos_lat); \
    break
  const bool vec = (int64_t)nin <= kVecMaxBytes;
  if (vec && f == 4)
    hipLaunchKernelGGL(k_downsample_vec<4>, grid, block, 0, stream, pos_hi, n_pix, Hr, Wr, H, W, pos_lat);
  else if (vec && f == 8)
    hipLaunchKernelGGL(k_downsample_vec<8>, grid, block, 0, stream, pos_hi, n_pix, Hr, Wr, H, W, pos_lat);
  else switch (f) {
    GC_STAGED(2);
    GC_STAGED(3);
    GC_STAGED(4);
    GC_STAGED(6);
    GC_STAGED(8);
    GC_STAGED(16);
    default:
      hipLaunchKernelGGL(k_downsample, grid, block, 0, stream, pos_hi, n_pix, Hr, Wr, f, H, W, pos_lat);
  }
#undef GC_STAGED
  return after_launch(stream, "gc_posmap_downsample");
}

extern "C" int gc_posmap_bbox(const float* pos, int B, int N, int H, int W, float tol_frac, float* bbox,
                              hipStream_t stream) {
  clear_error();
  if (!pos || !bbox) return fail(GC_ERR_ARG, "bbox: null pointer");
  if (B < 1 || N < 1 || H < 1 || W < 1) return fail(GC_ERR_SHAPE, "bbox: bad shape B=%d N=%d H=%d W=%d", B, N, H, W);
  if (B > 65535) return fail(GC_ERR_CAPACITY, "bbox: B=%d exceeds 65535", B);
  if (!(tol_frac > 0.0f && tol_frac <= 1.0f)) return fail(GC_ERR_ARG, "bbox: tol_frac %g outside (0, 1]", tol_frac);
  if (!aligned16(pos) || !aligned16(bbox)) return fail(GC_ERR_ALIGN, "bbox: pointers must be 16-byte aligned");
  const int64_t per = (int64_t)N * H * W;
  if (overlaps(pos, (size_t)B * per * 12, bbox, (size_t)B * 32)) return fail(GC_ERR_ALIAS, "bbox: output overlaps input");
  uint32_t* acc = reinterpret_cast<uint32_t*>(bbox);
  // one block reads an asset of up to kBoxSingle samples faster than several
  // blocks and the launch that clears their accumulator
  int64_t chunks = 1;
  if (per > kBoxSingle) {
    chunks = (per + kBoxPerBlock - 1) / kBoxPerBlock;
    if (chunks > kBoxMaxChunks) chunks = kBoxMaxChunks;
    hipLaunchKernelGGL(k_bbox_init, dim3((B + 63) / 64), dim3(64), 0, stream, acc, B);
  }
  hipLaunchKernelGGL(k_bbox_accum, dim3((unsigned)chunks, B), dim3(kBoxBlock), 0, stream, pos, per, tol_frac, acc);
  return after_launch(stream, "gc_posmap_bbox");
}
