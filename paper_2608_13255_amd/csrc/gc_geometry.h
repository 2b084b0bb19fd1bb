// Device code of the correspondence operator G_{A->v} for one (target token,
// anchor) pair (Sec. 3.2, correspondence operator): projection into the
// anchor camera, the 2x2 footprint around the projection, the per-tap
// tolerance test, the K nearest in-tolerance taps and their normalised area
// weights.  Shared by the builder (which stores the result) and the fused
// on-the-fly transport (which uses it at once), so both take every decision
// with the same float operations in the same order.
#pragma once

#include "gc_common.h"

namespace gc {

struct AnchorTaps {
  int32_t word;   // (x0+1) | (y0+1) << 12 | mask << 24, or 0 when the anchor contributes nothing
  int mask;       // kept taps, bit k for tap (x0 + (k & 1), y0 + (k >> 1))
  float wk[4];    // this anchor's normalised weight of tap k (before the division by n_vis)
};

// The operator for one pair runs in three steps so that callers can keep
// several anchors' tap loads in flight: anchor_project (arithmetic only),
// anchor_tap_positions (the four loads, all issued together) and
// anchor_select (the tests, the selection and the weights), or anchor_sees
// where only the visibility is wanted.

struct AnchorProj {
  bool ok;          // the projection lands within two pixels of the grid
  int x0, y0;       // the footprint's top-left tap
  float ax, ay;     // bilinear fractions
};

// P: the target token's 3D point (finite); cam: the anchor's camera.
// Without branches: the camera's words are then loaded together (behind a
// branch each would be a load of its own with its own wait), and an
// orthographic camera's unused quotient costs less than that.  A comparison
// with NaN is false, so the bounds of px and py reject what is not finite.
__device__ __forceinline__ AnchorProj anchor_project(const float (&P)[3], const gc_camera& cam, int H, int W) {
  const float* R = cam.R;
  const float xc = ((R[0] * P[0] + R[1] * P[1]) + R[2] * P[2]) + cam.t[0];
  const float yc = ((R[3] * P[0] + R[4] * P[1]) + R[5] * P[2]) + cam.t[1];
  const float zc = ((R[6] * P[0] + R[7] * P[1]) + R[8] * P[2]) + cam.t[2];
  const bool pinhole = cam.model == 0;
  const float qx = xc / zc, qy = yc / zc;
  const float px = cam.fx * (pinhole ? qx : xc) + cam.cx;
  const float py = cam.fy * (pinhole ? qy : yc) + cam.cy;
  AnchorProj o;
  o.ok = (pinhole ? zc > 0.0f : cam.model == 1) & (px >= -2.0f) & (px <= (float)W + 2.0f) & (py >= -2.0f) &
         (py <= (float)H + 2.0f);
  const float gx = o.ok ? px - 0.5f : 0.0f, gy = o.ok ? py - 0.5f : 0.0f;
  const float fx0 = floorf(gx), fy0 = floorf(gy);
  o.ax = gx - fx0;
  o.ay = gy - fy0;
  o.x0 = (int)fx0;
  o.y0 = (int)fy0;
  return o;
}

// A camera the whole wave uses, in scalar registers: all its words are loaded
// together here (left alone, the compiler sinks parts of the load behind the
// camera model's branch, each with a wait of its own).  Through the constant
// address space, since nothing writes cameras while a kernel runs.
__device__ __forceinline__ gc_camera wave_camera(const gc_camera* cam) {
  static_assert(sizeof(gc_camera) == 68, "17 words");
  typedef const __attribute__((address_space(4))) uint32_t* ConstWords;
  const ConstWords src = (ConstWords)(uintptr_t)cam;
  uint32_t w[17];
#pragma unroll
  for (int i = 0; i < 17; ++i) w[i] = src[i];
#pragma unroll
  for (int i = 0; i < 17; ++i) asm volatile("" : "+s"(w[i]));
  gc_camera c;
  __builtin_memcpy(&c, w, sizeof(c));
  return c;
}

// Positions of the four taps (x0 + (k & 1), y0 + (k >> 1)) of the anchor
// view's map src [H][W][3].  Every load reads a pixel clamped onto the grid,
// so all four are issued without a branch; anchor_select ignores the taps
// that are off the grid (and all of them when the projection failed).
struct TapPos {
  float q[4][3];
};

__device__ __forceinline__ TapPos anchor_tap_positions(const AnchorProj& pj, const float* src, int H, int W) {
  // grids have at most 4094 rows and columns: a row's byte offset is a product
  // of 24-bit factors, and every byte offset within the view is 32-bit
  const uint32_t row = 12u * (uint32_t)W;
  const uint32_t xa = 12u * (uint32_t)min(max(pj.x0, 0), W - 1), xb = 12u * (uint32_t)min(max(pj.x0 + 1, 0), W - 1);
  const uint32_t ra = __umul24((uint32_t)min(max(pj.y0, 0), H - 1), row);
  const uint32_t rb = __umul24((uint32_t)min(max(pj.y0 + 1, 0), H - 1), row);
  const uint32_t at[4] = {ra + xa, ra + xb, rb + xa, rb + xb};
  TapPos t;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float* Q = reinterpret_cast<const float*>(reinterpret_cast<const char*>(src) + at[k]);
    t.q[k][0] = Q[0];
    t.q[k][1] = Q[1];
    t.q[k][2] = Q[2];
  }
  return t;
}

// The per-tap tolerance test: valid[k] when tap k lies on the grid, is
// finite and at most sqrt(tol2) away from P; d2[k]: its squared distance
// (any value where it is not valid).  A NaN in the tap makes the distance NaN
// and an infinite one makes it infinite, so the comparison with a finite
// tolerance decides the tap's finiteness too: its components are looked at
// only when the tolerance itself overflowed to infinity.  pj.ok must hold.
__device__ __forceinline__ void taps_in_tolerance(const float (&P)[3], const AnchorProj& pj, const TapPos& tp, int H,
                                                  int W, float tol2, bool (&valid)[4], float (&d2)[4]) {
  const bool in_x[2] = {(uint32_t)pj.x0 < (uint32_t)W, (uint32_t)(pj.x0 + 1) < (uint32_t)W};
  const bool in_y[2] = {(uint32_t)pj.y0 < (uint32_t)H, (uint32_t)(pj.y0 + 1) < (uint32_t)H};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float dx = tp.q[k][0] - P[0], dy = tp.q[k][1] - P[1], dz = tp.q[k][2] - P[2];
    d2[k] = (dx * dx + dy * dy) + dz * dz;
    valid[k] = in_x[k & 1] & in_y[k >> 1] & (d2[k] <= tol2);
  }
  if (__ballot(!finite_f(tol2))) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      valid[k] = valid[k] && finite_f(tp.q[k][0]) && finite_f(tp.q[k][1]) && finite_f(tp.q[k][2]);
  }
}

// Whether the anchor sees P: some tap is valid (the word of anchor_select is
// non-zero exactly then).  A tap off the grid was read at the neighbouring
// pixel on it, which is the footprint's other tap of that row or column unless
// both are off, so with the footprint touching the grid the nearest of the
// four distances decides (a NaN is never the nearest).
__device__ __forceinline__ bool anchor_sees(const float (&P)[3], const AnchorProj& pj, const TapPos& tp, int H, int W,
                                            float tol2) {
  if (__ballot(!finite_f(tol2))) {
    bool valid[4];
    float d2[4];
    taps_in_tolerance(P, pj, tp, H, W, tol2, valid, d2);
    return pj.ok & (valid[0] | valid[1] | valid[2] | valid[3]);
  }
  float d2[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float dx = tp.q[k][0] - P[0], dy = tp.q[k][1] - P[1], dz = tp.q[k][2] - P[2];
    d2[k] = (dx * dx + dy * dy) + dz * dz;
  }
  const float nearest = __builtin_fminf(__builtin_fminf(d2[0], d2[1]), __builtin_fminf(d2[2], d2[3]));
  return pj.ok & ((uint32_t)(pj.x0 + 1) <= (uint32_t)W) & ((uint32_t)(pj.y0 + 1) <= (uint32_t)H) & (nearest <= tol2);
}

// The per-tap tolerance test, the K nearest valid taps and their normalised
// area weights; tol2: squared tolerance.
__device__ __forceinline__ AnchorTaps anchor_select(const float (&P)[3], const AnchorProj& pj, const TapPos& tp, int H,
                                                    int W, int K, float tol2) {
  AnchorTaps o;
  o.word = 0;
  o.mask = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) o.wk[k] = 0.0f;
  if (!pj.ok) return o;
  const int x0 = pj.x0, y0 = pj.y0;
  const float ax = pj.ax, ay = pj.ay;
  bool valid[4];
  float d2[4];
  taps_in_tolerance(P, pj, tp, H, W, tol2, valid, d2);
  int nvalid = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) nvalid += valid[k] ? 1 : 0;
  if (nvalid == 0) return o;
  bool sel[4] = {false, false, false, false};
  if (nvalid <= K) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sel[k] = valid[k];
  } else {
    for (int r = 0; r < K; ++r) {
      int best = -1;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (!valid[k] || sel[k]) continue;
        if (best < 0 || d2[k] < d2[best]) best = k;
      }
      sel[best] = true;
    }
  }
  const float wx[2] = {1.0f - ax, ax};
  const float wy[2] = {1.0f - ay, ay};
  float area[4];
  float S = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    area[k] = sel[k] ? wx[k & 1] * wy[k >> 1] : 0.0f;
    S = S + area[k];
  }
  if (S > 0.0f) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (sel[k] && area[k] > 0.0f) {
        o.wk[k] = area[k] / S;
        o.mask |= 1 << k;
      }
    }
  } else {
    int best = -1;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (sel[k] && (best < 0 || d2[k] < d2[best])) best = k;
#pragma unroll
    for (int k = 0; k < 4; ++k) o.wk[k] = k == best ? 1.0f : 0.0f;
    o.mask = 1 << best;
  }
  o.word = (int32_t)((uint32_t)(x0 + 1) | ((uint32_t)(y0 + 1) << 12) | ((uint32_t)o.mask << 24));
  return o;
}

}  // namespace gc
