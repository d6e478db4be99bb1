// The arguments that a hand-written kernel is launched with.  Host code only: the tests take them apart again with the kernels'
// own functions.
#include "kernels/kernel_arguments.hpp"

namespace fs {

static_assert(sizeof(TransposeP) + 2 * sizeof(void*) <= 256 && sizeof(BinaryP) + 3 * sizeof(void*) <= 256, "ArgList holds every kernel's arguments");

bool list_arguments(int32_t kernel, const KernelArgs& a, uint32_t grid, ArgList* l) {
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
