// Stitched bias + tanh-GELU, alone (thread composition) or packed with the
// bias-gradient column reduction (kernel packing + a global hand-off):
//     z = x + bias;  y = gelu(z);  dbias = colsum(grad * gelu'(z))
// GELU and GELU' share one exp and one reciprocal per element (the computation-reuse
// rule of the paper's Section 4.5) and one read of x.
//
// The column reduction needs rows owned by other workgroups, which the paper's
// schemes exclude (Section 4.1, last paragraph: no inter-block communication).  Here
// it is one round trip through device memory: every workgroup leaves its column
// partials in a [n_row_blocks, cols] float32 workspace, and the partials are folded in
// row-block order (fixed order: results are bit-identical from run to run) by a second,
// tiny launch (k_colfold): the kernel boundary is the hand-off.  Folding inside the same
// launch (the workgroup that arrives last reads the others' partials) needs an agent-scope
// release per workgroup before it signals its arrival, which on this part writes back the
// whole L2 of the workgroup's die while that cache is full of freshly stored y: measured
// at 1.6x the time of the two launches, so that form is not built.
#include <hip/hip_runtime.h>

#include "device_utils.hpp"
#include "fold.hpp"
#include "kernel_table.hpp"

namespace fsk {
using namespace fs;

// ---- bias + GELU only ------------------------------------------------------------
template <typename T, bool STREAM>
__global__ void __launch_bounds__(256) k_bias_gelu(const T* __restrict__ x, const T* __restrict__ bias,
                                                   T* __restrict__ y, uint32_t rows, uint32_t cols) {
  constexpr int VEC = Elem<T>::VEC;
  const uint32_t vecs_per_row = cols / VEC;
  const uint32_t n_vec = rows * vecs_per_row;
  const uint32_t vi = blockIdx.x * 256u + threadIdx.x;
  if (vi >= n_vec) return;
  const uint32_t cv = vi % vecs_per_row;
  const u32x4 rx = load_input<STREAM>(x + (size_t)vi * VEC);
  const u32x4 rb = load_raw(bias + cv * VEC);
  float v[VEC], b[VEC];
  unpack(rx, v, (const T*)nullptr);
  unpack(rb, b, (const T*)nullptr);
#pragma unroll
  for (int e = 0; e < VEC; ++e) v[e] = gelu_fwd(v[e] + b[e]);
  store_vec_nt(y + (size_t)vi * VEC, v);
}

// y = gelu(z) and acc += g * gelu'(z) with shared sub-expressions:
//   t = -2c log2(e) (1 + a z^2);  e = 2^(z t) = exp(-2u);  s = 1/(1+e);  y = z s
//   gelu' = s + z s (1-s) d(2u)/dz,   d(2u)/dz = 2c (1 + 3 a z^2)
__device__ __forceinline__ float gelu_and_grad(float z, float g, float& acc) {
  constexpr float c = 0.7978845608028654f, a = 0.044715f;
  constexpr float k = -2.0f * c * kLog2e;
  const float z2 = z * z;
  const float t = __builtin_fmaf(k * a, z2, k);
  const float s = fast_rcp(1.0f + __builtin_amdgcn_exp2f(z * t));
  const float y = z * s;
  const float dw = __builtin_fmaf(6.0f * c * a, z2, 2.0f * c);
  acc = __builtin_fmaf(g, __builtin_fmaf(__builtin_fmaf(-y, s, y), dw, s), acc);
  return y;
}

// ---- bias + GELU forward + bias-gradient column partials ------------------------------
// Workgroup (ct, rb): column tile ct of 64*VEC columns, row tiles rb, rb + n_rb, ... of
// WAVES*UNROLL rows each.  Lane l owns columns [l*VEC, l*VEC+VEC) of the tile, wave w
// rows w, w+WAVES, ... of a row tile, so every wave-wide access is one contiguous
// 1 KB piece, and at any moment the resident workgroups sweep one band of rows
// (DRAM pages stay open) while each keeps its column sums in registers.
// The row loop has no test inside (but for ragged float32 shapes; FAST: nothing is clamped either, the rows fill every workgroup's row tiles exactly and the
// columns fill the column tiles).  That matters beyond the saved compares: the
// memory counter of this part counts loads and stores alike, in issue order, and when a
// store sits inside a branch the compiler can no longer tell how many stores follow the
// loads it waits for, so it waits for everything -- every round of the loop then ends
// with the wave idle until its own y stores are acknowledged.  With unconditional stores
// the wait before the next tile's data leaves the UNROLL stores of this tile in flight.
template <typename T, int WAVES, int UNROLL, bool FAST, bool STREAM>
__global__ void __launch_bounds__(WAVES * 64) k_bias_gelu_dbias(const T* __restrict__ x, const T* __restrict__ bias,
                                                                const T* __restrict__ grad, T* __restrict__ y,
                                                                float* __restrict__ partials, uint32_t rows, uint32_t cols,
                                                                uint32_t n_row_tiles) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int TILE_COLS = 64 * VEC, NT = WAVES * 64, TILE_ROWS = WAVES * UNROLL;
  __shared__ __align__(16) float red[WAVES][TILE_COLS];
  const uint32_t n_col_tiles = (cols + TILE_COLS - 1) / TILE_COLS;
  const uint32_t rb = blockIdx.x / n_col_tiles;
  const uint32_t ct = blockIdx.x - rb * n_col_tiles;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t col = FAST ? ct * TILE_COLS + lane * VEC
                            : min(ct * TILE_COLS + lane * VEC, cols - VEC);   // clamped lanes of a ragged tile redo valid columns

  float acc[VEC], b[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.0f;
  unpack(load_raw(bias + col), b, (const T*)nullptr);
  // software pipeline: the loads of the next row tile are in flight while this one is
  // computed, so a wave overlaps its own ALU phase (two quarter-rate ops per element)
  // with its own memory phase instead of relying on the other waves of the SIMD.
  u32x4 nx[UNROLL], ng[UNROLL];
  auto issue = [&](uint32_t r0) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const uint32_t r = r0 + wave + u * WAVES;
      const size_t off = (size_t)(FAST ? r : min(r, rows - 1)) * cols + col;
      nx[u] = load_input<STREAM>(x + off);
      ng[u] = load_input<STREAM>(grad + off);
    }
  };
  // all rows of the tile first, then their stores in one burst (measured: 0.5 us of 50 against a store
  // after every row; the memory system takes a run of writes better than writes sprinkled between reads)
  auto compute = [&](uint32_t r0, const u32x4 (&rx)[UNROLL], const u32x4 (&rg)[UNROLL]) {
    float out[UNROLL][VEC];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      float gv[VEC];
      unpack(rx[u], out[u], (const T*)nullptr);
      unpack(rg[u], gv, (const T*)nullptr);
#pragma unroll
      for (int e = 0; e < VEC; ++e) out[u][e] = gelu_and_grad(out[u][e] + b[e], gv[e], acc[e]);
    }
    // (a clamped lane writes what the owner of its columns writes, to the same place)
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) store_vec_nt(y + (size_t)(r0 + wave + u * WAVES) * cols + col, out[u]);
  };
  // the rows' last tile, where it is a partial one
  auto compute_some = [&](uint32_t r0, const u32x4 (&rx)[UNROLL], const u32x4 (&rg)[UNROLL]) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const uint32_t r = r0 + wave + u * WAVES;
      if (r < rows) {
        float xv[VEC], gv[VEC];
        unpack(rx[u], xv, (const T*)nullptr);
        unpack(rg[u], gv, (const T*)nullptr);
#pragma unroll
        for (int e = 0; e < VEC; ++e) xv[e] = gelu_and_grad(xv[e] + b[e], gv[e], acc[e]);
        store_vec_nt(y + (size_t)r * cols + col, xv);
      }
    }
  };
  const uint32_t stride = n_row_tiles * TILE_ROWS;
  uint32_t r0 = rb * TILE_ROWS;
  // Only the rows' very last tile can be partial, and it is the last one of its workgroup: no other round has a test around its
  // loads or its stores.  First and last round stand outside the loop: the loop is then entered with the same sequence of
  // loads and stores in flight that its own rounds leave behind, which is what lets the wait at its head be
  // "all but the last stores" on both ways in.  Measured, rounds with tests / without (us): bf16 [8191,3072] 28.4 / 27.8, f16
  // [2001,4096] 11.1 / 10.5, bf16 [4097,768] 7.4 / 7.2, bf16 [30001,520] 24.9 / 24.1; f32 [12345,1544] 49.5 / 50.7, so ragged
  // float32 shapes keep the tests (and gain by the rounds outside the loop: [4001,3072] 28.7 / 26.2, [20001,520] 26.7 / 25.1).
  constexpr bool UNTESTED = FAST || VEC == 8;
  auto round = [&](uint32_t at) {
    u32x4 rx[UNROLL], rg[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) { rx[u] = nx[u]; rg[u] = ng[u]; }
    issue(at + stride);
    if constexpr (UNTESTED) compute(at, rx, rg);
    else compute_some(at, rx, rg);
  };
  issue(r0);   // (every workgroup has a row tile)
  if (r0 + stride < rows) {
    round(r0);
    r0 += stride;
    for (; r0 + stride < rows; r0 += stride) round(r0);
  }
  if (FAST || (UNTESTED && r0 + TILE_ROWS <= rows)) compute(r0, nx, ng);
  else compute_some(r0, nx, ng);

  // regional step: fold the waves of this workgroup through LDS, in wave order
#pragma unroll
  for (int e = 0; e < VEC; e += 4)   // 128-bit LDS stores: scalar ones would be VEC floats apart from lane to lane
    *reinterpret_cast<f32x4*>(&red[wave][lane * VEC + e]) = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
  __syncthreads();
  for (uint32_t c = threadIdx.x; c < TILE_COLS; c += NT) {
    float s = red[0][c];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) s += red[w][c];
    const uint32_t gc = ct * TILE_COLS + c;
    if (gc < cols) partials[(size_t)rb * cols + gc] = s;
  }
}

static_assert(kFoldF32 == DT_F32 && kFoldF16 == DT_F16 && kFoldBf16 == DT_BF16, "fold_tile takes the storage dtypes' numbers");

template <int Q, int G>
__global__ void __launch_bounds__(256) k_colfold(const float* __restrict__ partials, float* __restrict__ out0,
                                                 float* __restrict__ out1, uint32_t n, uint32_t width, uint32_t stride,
                                                 uint32_t split, uint32_t out_cols, int32_t out_dt) {
  __shared__ f32x4 sm[G * Q];
  // stride >= width: a fold may take a slice of wider partial rows
  fold_tile<Q, G>(partials, out0, out1, n, width, stride, split, out_cols, blockIdx.x, sm, out_dt);
}

// Several independent folds in one launch: workgroups [first_block[i], first_block[i+1]) run fold i.  The table
// is read from the kernel-argument segment with wave-uniform addresses (indexing the by-value parameter would
// make the compiler copy it to per-lane scratch first).
typedef const FoldManyP __attribute__((address_space(4))) * ConstFolds;

__global__ void __launch_bounds__(256) k_colfold_many(const FoldManyP table_in_kernarg) {
  __shared__ f32x4 sm[256];
  ConstFolds tab = (ConstFolds)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t b = blockIdx.x;
  int i = -1;
#pragma unroll
  for (int j = 0; j < kFoldManyMax; ++j) i += b >= tab->first_block[j] ? 1 : 0;   // first_block[0] = 0, unused ones ~0
  i = __builtin_amdgcn_readfirstlane(i);
  const float* partials = tab->partials[i];
  float* out0 = tab->out0[i];
  float* out1 = tab->out1[i];
  const uint32_t block = b - tab->first_block[i];
  if (tab->quads[i] == 4)
    fold_tile<4, 64>(partials, out0, out1, tab->n[i], tab->width[i], tab->stride[i], tab->split[i], tab->out_cols[i], block, sm, tab->out_dt[i]);
  else
    fold_tile<16, 16>(partials, out0, out1, tab->n[i], tab->width[i], tab->stride[i], tab->split[i], tab->out_cols[i], block, sm, tab->out_dt[i]);
}

}  // namespace fsk

namespace fs {
using namespace fsk;

namespace {
template <typename T, bool FAST, bool S>
const void* dbias_sym(int waves, int unroll) {
  if (waves == 4 && unroll == 2) return (const void*)k_bias_gelu_dbias<T, 4, 2, FAST, S>;
  if (waves == 4 && unroll == 4) return (const void*)k_bias_gelu_dbias<T, 4, 4, FAST, S>;
  if (waves == 8 && unroll == 2) return (const void*)k_bias_gelu_dbias<T, 8, 2, FAST, S>;
  if (waves == 8 && unroll == 4) return (const void*)k_bias_gelu_dbias<T, 8, 4, FAST, S>;
  return nullptr;
}
template <typename T, bool S>
const void* gelu_sym_s(int32_t kernel, const GeluP& p) {
  if (kernel == K_BIAS_GELU) return (const void*)k_bias_gelu<T, S>;
  return p.fast ? dbias_sym<T, true, S>(p.waves, p.unroll) : dbias_sym<T, false, S>(p.waves, p.unroll);
}
template <typename T>
const void* gelu_sym(int32_t kernel, const GeluP& p) {
  return p.stream ? gelu_sym_s<T, true>(kernel, p) : gelu_sym_s<T, false>(kernel, p);
}
}  // namespace

int launch_fold_many(const FoldManyP& table, uint32_t n_blocks, void* stream) {
  if (n_blocks == 0) return 0;
  FoldManyP t = table;
  void* argv[1] = {&t};
  return (int)hipLaunchKernel((const void*)k_colfold_many, dim3(n_blocks), dim3(256), argv, 0, static_cast<hipStream_t>(stream));
}

const void* gelu_kernel_symbol(int32_t kernel, const KernelArgs& a) {
  const GeluP& p = a.u.gelu;
  if (kernel == K_COLFOLD) return p.fold_quads == 4 ? (const void*)k_colfold<4, 64> : (const void*)k_colfold<16, 16>;
  switch (p.dt) {
    case DT_F32: return gelu_sym<float>(kernel, p);
    case DT_F16: return gelu_sym<f16_t>(kernel, p);
    default: return gelu_sym<bf16_t>(kernel, p);
  }
}

}  // namespace fs
