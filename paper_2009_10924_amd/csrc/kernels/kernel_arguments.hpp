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
static_assert(sizeof(TransposeP) + 2 * sizeof(void*) <= 256 && sizeof(BinaryP) + 3 * sizeof(void*) <= 256, "ArgList holds every kernel's arguments");
// The arguments of `kernel`, as its definition lists them; false: a value that its word cannot hold (or a kernel that is not
// launched this way).  Inlined into the launcher, where the list's places are constants.
__attribute__((always_inline)) inline bool list_arguments(int32_t kernel, const KernelArgs& a, uint32_t grid, ArgList* l) {
  void* const* p = a.p;
  const uint32_t cols24 = 1u << 24;
  switch (kernel) {
    case K_UNARY: case K_COPY: l->add(p[0], p[1], a.u.unary); return true;
    case K_BINARY: l->add(p[0], p[1], p[2], a.u.binary); return true;
    case K_REDUCE_ROW: case K_REDUCE_MID: l->add(p[0], p[1], a.u.reduce); return true;
    case K_TRANSPOSE_TILE: {
      const TransposeP& t = a.u.transpose;
      if (t.vec == 1) {   // 32x32 single elements
        l->add(p[0], p[1], t);
        return true;
      }
      l->add(p[0], p[1], t.div[0].m, t.div[1].m, transpose_word(t), t.nq, t.nx, t.in_row, t.in_batch[1], t.n_tiles, t.out_row, t.out_batch[1]);
      if (transpose_two_batch_axes(t)) l->add(t.div[2].d, t.div[2].m, t.in_batch[0], t.out_batch[0]);
      return true;
    }
    case K_TRANSPOSE_ROWS: {
      const TransposeP& t = a.u.transpose;
      l->add(p[0], p[1], t.n, t.vec, t.in_stride[0], t.in_stride[1], t.in_stride[2], t.out_ext[0], t.out_ext[1], t.out_ext[2]);
      return true;
    }
    case K_SOFTMAX_WAVE: case K_SOFTMAX_BLOCK: {
      const SoftmaxP& s = a.u.softmax;
      const bool any_length = s.vecs_per_lane == 0;   // k_softmax_generic: the columns travel in the place of the rows
      if (!any_length && s.cols >= (1u << 18)) return false;
      const uint32_t lanes = kernel == K_SOFTMAX_WAVE ? (uint32_t)s.lanes_log2 : (uint32_t)s.lanes_per_row / 64u;
      if (lanes > 7u) return false;
      l->add(p[0], s.has_mask ? p[1] : nullptr, p[2], any_length ? s.cols : s.rows,
             softmax_word(any_length ? 0u : s.cols, lanes, s.mask_inner != 0, s.od[1].s, s.od[2].s), s.scale, s.od[1].d, s.od[1].m, s.od[2].d, s.od[2].m,
             s.ms[0], s.ms[1], s.ms[2]);
      return true;
    }
    case K_LAYERNORM_WAVE: case K_LAYERNORM_BLOCK: {
      const LayerNormP& n = a.u.layernorm;
      const uint32_t lanes = kernel == K_LAYERNORM_WAVE ? (uint32_t)n.lanes_log2 : (uint32_t)n.lanes_per_row / 64u;
      if (n.cols >= cols24 || lanes > 7u) return false;
      const uint32_t flags = (n.has_res ? 1u : 0u) | (n.has_bias ? 2u : 0u) | (n.has_affine ? 4u : 0u);
      l->add(p[0], p[1], p[2], n.rows, row_word(n.cols, lanes, flags), p[3], p[4], p[5], n.eps, n.inv_cols);
      if (n.stats) l->add(p[6], p[7]);
      return true;
    }
    case K_LAYERNORM_BWD: {
      const LnBwdP& n = a.u.lnbwd;
      if (n.cols >= (1u << 13) || n.lanes_log2 > 6 || grid >= (1u << 16)) return false;
      l->add(p[0], p[1], p[2], p[3], p[4], n.rows, lnbwd_word(n.cols, (uint32_t)n.lanes_log2, grid), p[5], p[6]);
      return true;
    }
    case K_BIAS_GELU: l->add(p[0], p[1], p[2], a.u.gelu.rows, a.u.gelu.cols); return true;
    case K_BIAS_GELU_DBIAS: l->add(p[0], p[1], p[2], p[3], p[4], a.u.gelu.rows, a.u.gelu.cols, a.u.gelu.n_row_tiles); return true;
    case K_COLFOLD: {
      const GeluP& f = a.u.gelu;
      l->add(p[0], p[1], p[2], f.n_row_tiles, f.fold_cols, f.cols, f.fold_split, f.fold_out_cols, f.dt);
      return true;
    }
    case K_TCHAIN_WAVE: case K_TCHAIN_LDS: {
      const TChainP& t = a.u.tchain;
      if (t.D >= (1u << 16) || t.lanes_log2 > 6) return false;
      l->add(p[0], p[1], p[2], tchain_word(t.D, (uint32_t)t.lanes_log2, t.div_s_tiles.s, t.div_h.s), t.S, t.H, t.s_tile, t.div_s_tiles.d, t.div_s_tiles.m,
             t.div_h.m, t.eps);
      return true;
    }
    case K_ROW_WAVE: case K_ROW_BLOCK: {
      const RowP& r = a.u.row;
      const uint32_t lanes = kernel == K_ROW_WAVE ? (uint32_t)r.lanes_log2 : (uint32_t)r.lanes_per_row / 64u;
      if (r.cols >= cols24 || lanes > 7u) return false;
      l->add(p[0], p[1], p[2], r.rows, row_word(r.cols, lanes), p[4], r.f[0], r.f[1]);
      return true;
    }
    default: return false;
  }
}

}  // namespace fs
