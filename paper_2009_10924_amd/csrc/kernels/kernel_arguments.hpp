// What the hand-written kernels take as arguments: the words that small numbers share, packed by the launcher and taken apart
// by the kernels, both here so that they can be checked against each other on the host.
#pragma once
#include <cstring>

#include "launch.hpp"

#if defined(__HIP__)
#define FS_SHARED __host__ __device__ __forceinline__
#else
#define FS_SHARED inline
#endif

namespace fs {
// Kernel arguments.  A kernel takes its pointers and the few values it needs, one by one and 64 bytes in all where that can
// be: the compiler preloads the first fourteen dwords into scalar registers (build.py; never a part of a by-value block, so
// there is none), a wavefront then issues its first loads without fetching anything, and the arguments are one line for the
// host to write and for the device to read.  Small numbers share a word with a row's columns.
// Measured against pointers and a parameter block of 44 to 100 bytes behind them (us per call, before / after): softmax f32
// [64,128] 3.8 / 3.4, attention scores f16 [32,12,128,128] 4.93 / 4.51, add + bias + LayerNorm f32 [8192,768] 10.9 / 9.8, f16
// [635,4608] 5.2 / 4.5, head split + normalisation f32 [64,512,12,64] 33.1 / 32.6, bias + GELU backward bf16 [108,1280] (two
// launches) 6.85 / 6.5.  With these values in front of the block and the block still there, a small call was no faster (4.0).

// columns (below 2^24) and the row's lanes: their log2 for a lane group, their number of wavefronts for a whole workgroup;
// `flags`: five more bits
inline uint32_t row_word(uint32_t cols, uint32_t lanes_code, uint32_t flags = 0) { return cols | lanes_code << 24 | flags << 27; }
// the same for a softmax (columns below 2^18) and its mask: whether it varies along the row, the shifts of two divisions
inline uint32_t softmax_word(uint32_t cols, uint32_t lanes_code, uint32_t mask_inner, uint32_t s1, uint32_t s2) {
  return cols | lanes_code << 18 | mask_inner << 21 | s1 << 22 | s2 << 27;
}
// head dimension (below 2^16), log2 of the lanes per row, the shifts of two divisions
inline uint32_t tchain_word(uint32_t D, uint32_t lanes_log2, uint32_t s_tiles, uint32_t s_h) { return D | lanes_log2 << 16 | s_tiles << 19 | s_h << 24; }
// columns (below 2^13), log2 of the lanes per row, workgroups in the grid (the grid's size from the hardware's own arguments
// would put 256 bytes of them behind the kernel's)
inline uint32_t lnbwd_word(uint32_t cols, uint32_t lanes_log2, uint32_t grid) { return cols | lanes_log2 << 13 | grid << 16; }
// a tiled transpose: the shifts of three divisions, walk_q, every_other
inline uint32_t transpose_word(const TransposeP& t) {
  return t.div[0].s | t.div[1].s << 5 | t.div[2].s << 10 | (t.walk_q ? 1u << 15 : 0u) | (t.every_other ? 1u << 16 : 0u);
}
inline bool transpose_two_batch_axes(const TransposeP& t) { return t.in_batch[0] != 0 || t.out_batch[0] != 0; }

// ---- what a kernel's arguments say: `block`: a whole workgroup per row -----------------------------------------------
FS_SHARED SoftmaxP softmax_params(bool block, uint32_t rows, uint32_t word, float scale, uint32_t d1, uint32_t m1, uint32_t d2, uint32_t m2,
                                  uint32_t ms0, uint32_t ms1, uint32_t ms2) {
  SoftmaxP p{};
  p.rows = rows;
  p.cols = word & 0x3FFFFu;
  p.lanes_log2 = (int32_t)((word >> 18) & 7u);
  p.lanes_per_row = block ? p.lanes_log2 * 64 : 1 << p.lanes_log2;
  p.mask_inner = (int32_t)((word >> 21) & 1u);
  p.scale = scale;
  p.od[1] = FastDiv{d1, m1, (word >> 22) & 31u};
  p.od[2] = FastDiv{d2, m2, word >> 27};
  p.ms[0] = ms0, p.ms[1] = ms1, p.ms[2] = ms2;
  return p;
}
FS_SHARED LayerNormP layernorm_params(bool block, uint32_t rows, uint32_t word, float eps, float inv_cols) {
  LayerNormP p{};
  p.rows = rows;
  p.cols = word & 0xFFFFFFu;
  p.lanes_log2 = (int32_t)((word >> 24) & 7u);
  p.lanes_per_row = block ? p.lanes_log2 * 64 : 1 << p.lanes_log2;
  p.has_res = (int32_t)((word >> 27) & 1u), p.has_bias = (int32_t)((word >> 28) & 1u), p.has_affine = (int32_t)((word >> 29) & 1u);
  p.eps = eps;
  p.inv_cols = inv_cols;
  return p;
}
FS_SHARED LnBwdP lnbwd_params(uint32_t rows, uint32_t word) {
  LnBwdP p{};
  p.rows = rows;
  p.cols = word & 0x1FFFu;
  p.lanes_log2 = (int32_t)((word >> 13) & 7u);
  p.lanes_per_row = 1 << p.lanes_log2;
  // as the host would round it: for whole numbers below 2^24 the quotient in float and the one in double, rounded, agree
  p.inv_cols = 1.0f / (float)p.cols;
  return p;
}
FS_SHARED uint32_t lnbwd_grid(uint32_t word) { return word >> 16; }
FS_SHARED RowP row_params(bool block, uint32_t rows, uint32_t word, float f0, float f1) {
  RowP p{};
  p.rows = rows;
  p.cols = word & 0xFFFFFFu;
  p.lanes_log2 = (int32_t)((word >> 24) & 7u);
  p.lanes_per_row = block ? p.lanes_log2 * 64 : 1 << p.lanes_log2;
  p.f[0] = f0, p.f[1] = f1;
  return p;
}
FS_SHARED TChainP tchain_params(uint32_t word, uint32_t S, uint32_t H, uint32_t s_tile, uint32_t tiles_d, uint32_t tiles_m, uint32_t h_m, float eps) {
  TChainP p{};
  p.S = S, p.H = H;
  p.D = word & 0xFFFFu;
  p.lanes_log2 = (int32_t)((word >> 16) & 7u);
  p.lanes_per_row = 1 << p.lanes_log2;
  p.s_tile = (int32_t)s_tile;
  p.div_s_tiles = FastDiv{tiles_d, tiles_m, (word >> 19) & 31u};
  p.div_h = FastDiv{H, h_m, (word >> 24) & 31u};
  p.eps = eps;
  return p;
}
// The numbers of tiles follow from the extents (TQ, TX: a tile's).
FS_SHARED TransposeP units_params(uint32_t TQ, uint32_t TX, uint32_t m0, uint32_t m1, uint32_t word, uint32_t nq, uint32_t nx, uint32_t in_row, uint32_t in_batch, uint32_t n_tiles,
                                  uint32_t out_row, uint32_t out_batch) {
  TransposeP p{};
  p.walk_q = (word >> 15) & 1u;
  p.every_other = (word >> 16) & 1u;
  const uint32_t tq = (nq + TQ - 1u) / TQ, tx = (nx + TX - 1u) / TX;
  p.div[0] = FastDiv{p.walk_q ? tq >> p.every_other : tx, m0, word & 31u};
  p.div[1] = FastDiv{p.walk_q ? tx : tq, m1, (word >> 5) & 31u};
  p.nq = nq, p.nx = nx, p.in_row = in_row, p.out_row = out_row;
  p.in_batch[1] = in_batch, p.out_batch[1] = out_batch;
  p.n_tiles = n_tiles;
  return p;
}
FS_SHARED void units_second_axis(TransposeP* p, uint32_t word, uint32_t d2, uint32_t m2, uint32_t in_batch0, uint32_t out_batch0) {
  p->div[2] = FastDiv{d2, m2, (word >> 10) & 31u};
  p->in_batch[0] = in_batch0, p->out_batch[0] = out_batch0;
}

// ---- the launcher's side -------------------------------------------------------------------------------------------
// Storage of one launch's arguments and their addresses, which is what hipLaunchKernel wants.
struct ArgList {
  alignas(8) char bytes[256];
  void* address[24];
  size_t n = 0, at = 0;
  template <typename T>
  void add(const T& v) {
    at = (at + alignof(T) - 1) & ~(alignof(T) - 1);
    memcpy(bytes + at, &v, sizeof v);
    address[n++] = bytes + at;
    at += sizeof v;
  }
  template <typename T, typename... Rest>
  void add(const T& v, const Rest&... rest) {
    add(v);
    add(rest...);
  }
};
// The arguments of `kernel`, as its definition lists them; false: a value that its word cannot hold (or a kernel that is not
// launched this way).
bool list_arguments(int32_t kernel, const KernelArgs& a, uint32_t grid, ArgList* l);

}  // namespace fs
