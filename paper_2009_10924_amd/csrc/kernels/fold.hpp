// The fold of column partial sums, shared by the fold kernels (gelu.hip) and by generated kernels that carry a program's folds
// along.  Embedded in the library as text like the headers that generated kernels are made of.
#pragma once
#include "device_utils.hpp"

namespace fsk {

constexpr int kFoldF32 = 0, kFoldF16 = 1, kFoldBf16 = 2;   // storage dtypes of the sums

// ---- fold of column partials: [n_rows, width] float32 (rows `stride` floats apart) -> [width] ---------
// Workgroup = Q column quads x G row groups (256 threads).  Each thread sums its rows in
// order with eight independent loads in flight, LDS folds the G groups in order.  Few
// partial rows: (Q,G) = (16,16); many: (4,64), so a thread still needs one batch of loads.
// What bounds it is the latency of its loads, one after the other if they are not issued together: with the last, partial
// batch issued row by row, 82 / 163 / 326 partial rows (6 / 3 / 6 of them per thread) made the two launches of a GELU
// backward of 3.5 MB take 8.9 / 7.4 / 8.5 us.  Issued together, over some 5400 timed plans with column sums: 65 to 128
// partial rows 0.8 us less, 129 to 256 0.3, 257 to 512 0.6, more 0.4, at most 16 level.
template <int Q, int G>
__device__ __forceinline__ void fold_tile(const float* __restrict__ partials, float* __restrict__ out0, float* __restrict__ out1,
                                          uint32_t n, uint32_t width, uint32_t stride, uint32_t split, uint32_t out_cols, uint32_t block,
                                          f32x4* __restrict__ sm, int out_dt) {
  const uint32_t q = threadIdx.x % Q, g = threadIdx.x / Q;
  const uint32_t col = (block * Q + q) * 4u;
  f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
  if (col < width) {
    uint32_t t = g;
    for (; t + 7 * G < n; t += 8 * G) {
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4*>(partials + (size_t)(t + u * G) * stride + col);
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    if (t < n) {   // the rest, at most eight rows: one batch as well (clamped to the last row, what is too many left out)
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4*>(partials + (size_t)min(t + u * G, n - 1u) * stride + col);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (t + u * G < n) s += v[u];
    }
  }
  sm[g * Q + q] = s;
  __syncthreads();
  // the G row groups fold through LDS four at a time (G = 16: two levels, G = 64: three; the same order every
  // run): a barrier costs more than three more LDS reads, and a serial walk over all G slots more than both
#pragma unroll
  for (int span = G / 4; span >= 1; span /= 4) {
    if ((int)g < span) sm[g * Q + q] += sm[(g + span) * Q + q] + sm[(g + 2 * span) * Q + q] + sm[(g + 3 * span) * Q + q];
    __syncthreads();
  }
  if (g == 0 && col < width) {
    const f32x4 v = sm[q];
    // the split is a multiple of 4, so a quad never straddles the two outputs; sums handed out in 16 bits are
    // rounded here, once
    float* const base = col < split ? out0 : out1;
    const uint32_t at = col < split ? col : col - split;
    const float quad[4] = {v.x, v.y, v.z, v.w};
    if (at + 4u > out_cols) {   // the last quad of a sum whose columns are no multiple of 4: the rest of it is padding
#pragma unroll
      for (uint32_t e = 0; e < 3u; ++e)
        if (at + e < out_cols) {
          if (out_dt == kFoldF32) base[at + e] = quad[e];
          else if (out_dt == kFoldBf16) store1(reinterpret_cast<bf16_t*>(base) + at + e, quad[e]);
          else store1(reinterpret_cast<f16_t*>(base) + at + e, quad[e]);
        }
    } else if (out_dt == kFoldF32) {
      *reinterpret_cast<f32x4*>(base + at) = v;
    } else {
      if (out_dt == kFoldBf16) StoreN<bf16_t, 4>::run(reinterpret_cast<bf16_t*>(base) + at, quad);
      else StoreN<f16_t, 4>::run(reinterpret_cast<f16_t*>(base) + at, quad);
    }
  }
}

}  // namespace fsk
