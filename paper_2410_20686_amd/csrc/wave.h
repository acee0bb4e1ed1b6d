// Cross-lane helpers of the compositing kernels (64-wide CDNA wavefronts, gfx950 DPP and
// row-swap permutes) and the thread-to-pixel map of a tile.
#pragma once

#include "common.h"

namespace odgs {

template <int CTRL>
__device__ inline float dpp_read(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Exchange step of a multi-value butterfly: the lane keeps `lo` or `hi` (by `bit`) and adds the
// partner's copy of the same slot; the partner (reached with DPP control CTRL) has the opposite
// `bit` and holds the same slot meanings.
template <int CTRL>
__device__ inline float bfly(float lo, float hi, bool bit) {
  return (bit ? hi : lo) + dpp_read<CTRL>(bit ? lo : hi);
}

// Sum of a value over the four 16-lane rows of the wavefront, returned in every row: the gfx950
// row-swap permutes (lanes 32-63 <-> 0-31, then odd <-> even rows) need no LDS traffic.
__device__ inline float sum_rows(float x) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Flags of a staged entry in the one-wavefront compositors (above the quadrant mask).
constexpr int kEntryWrap = 1;   // some pixel centre of the tile may need the seam wrap
constexpr int kEntryClamp = 2;  // opacity above 0.99: alpha may be clamped (forward quadrant tasks: or the colour is
                                // infinite; reverse: or the colour is kLarge and more, see is_large)

// A uniform word the compiler cannot relate to its other uses, so that a test of it stays a scalar
// test beside its branch.
__device__ inline int opaque(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

// Lane `lane` (uniform) of `x` takes the uniform word `value`.
__device__ inline void set_lane(uint32_t& x, uint32_t value, int lane) {
  asm("s_mov_b32 m0, %2\n\tv_writelane_b32 %0, %1, m0" : "+v"(x) : "s"(value), "s"(lane) : "m0");
}

// Upstream gradients and colours below kLarge give the reverse steps finite values throughout: with both
// below 2^50 (and dL/dC . background below it), dL/dC . colour stays below 2^102, and so does the sum of such
// products times weights that add up to one; over 1 - alpha >= 0.01 below 2^109.  A value that is not finite
// counts as large.  Only where something is large does a step zero dL/dalpha by a select of its own for
// pixels that the Gaussian does not reach; elsewhere its product with alpha = 0 is zero.
constexpr float kLarge = 0x1p50f;
__device__ inline bool is_large(float sum_of_magnitudes) { return !(sum_of_magnitudes < kLarge); }
__device__ inline float magnitude(float a, float b, float c) { return fabsf(a) + fabsf(b) + fabsf(c); }

// Keeps a rarely taken uniform branch a branch: the value is not computed on the other path.
__device__ inline void keep_branch(float& x) { asm volatile("" : "+v"(x)); }

// Pixel of a thread inside a TILE x TILE tile: wavefront w owns quadrant w (row-major over the
// TILE/8 x TILE/8 quadrants), lane l the pixel (l % 8, l / 8) inside it.
template <int TILE>
__device__ inline void local_pixel(int t, int& lx, int& ly) {
  constexpr int QPR = TILE / 8;
  const int w = t >> 6, l = t & 63;
  lx = (w % QPR) * 8 + (l & 7);
  ly = (w / QPR) * 8 + (l >> 3);
}

}  // namespace odgs
