// Kernel dispatch: the symbol that serves a (kernel id, parameter block) and the arguments that it takes.
#include <hip/hip_runtime.h>

#include <cstring>

#include "kernel_table.hpp"

namespace fs {

namespace {
const char* const kNames[K_COUNT] = {
    "unary", "binary", "reduce_row", "reduce_mid", "transpose_rows", "transpose_tile", "copy", "softmax_wave", "softmax_block",
    "layernorm_wave", "layernorm_block", "bias_gelu", "bias_gelu_dbias", "colfold", "tchain_wave", "tchain_lds", "row_wave",
    "row_block", "row_program", "layernorm_bwd", "row_generated",
};

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

// The arguments of `kernel`, as its definition lists them (see kernel_table.hpp); false: a value that its word cannot hold,
// which no plan offers.
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
      l->add(p[0], p[1], p[2], p[3], r.rows, row_word(r.cols, lanes), p[4], r.f[0], r.f[1]);
      return true;
    }
    default: return false;
  }
}

const void* symbol_for(int32_t kernel, const KernelArgs& a) {
  switch (kernel) {
    case K_UNARY: case K_BINARY: case K_REDUCE_ROW: case K_REDUCE_MID:
    case K_TRANSPOSE_ROWS: case K_TRANSPOSE_TILE: case K_COPY:
      return unfused_kernel_symbol(kernel, a);
    case K_SOFTMAX_WAVE: case K_SOFTMAX_BLOCK:
      return softmax_kernel_symbol(kernel, a);
    case K_LAYERNORM_WAVE: case K_LAYERNORM_BLOCK: case K_LAYERNORM_BWD:
      return layernorm_kernel_symbol(kernel, a);
    case K_BIAS_GELU: case K_BIAS_GELU_DBIAS: case K_COLFOLD:
      return gelu_kernel_symbol(kernel, a);
    case K_TCHAIN_WAVE: case K_TCHAIN_LDS:
      return tchain_kernel_symbol(kernel, a);
    case K_ROW_WAVE: case K_ROW_BLOCK:
      return rowops_kernel_symbol(kernel, a);
    case K_ROW_PROGRAM:
      return rowprog_kernel_symbol(kernel, a);
    default:
      return nullptr;
  }
}
}  // namespace

const char* kernel_name(int32_t kernel) {
  return (kernel >= 0 && kernel < K_COUNT) ? kNames[kernel] : "?";
}

const char* hip_error_text(int err) { return hipGetErrorString(static_cast<hipError_t>(err)); }

int launch_kernel(int32_t kernel, const KernelArgs& args, const LaunchShape& s, void* stream) {
  if (kernel < 0 || kernel >= K_COUNT) return (int)hipErrorInvalidValue;
  const void* sym = symbol_for(kernel, args);
  if (!sym) return (int)hipErrorInvalidDeviceFunction;
  if (kernel == K_ROW_PROGRAM) {
    // one by-value argument: pointers by class, then the program
    ProgArgs pa;
    for (int i = 0; i < kProgMaxOperands; ++i) {
      pa.full[i] = args.p[kSlotFull + i];
      pa.col[i] = args.p[kSlotCol + i];
      pa.rscal[i] = args.p[kSlotRscal + i];
      pa.out[i] = args.p[kSlotOut + i];
      pa.rout[i] = args.p[kSlotRout + i];
    }
    pa.p = args.u.prog;
    if (s.lds_bytes > 64u * 1024u) {
      // more dynamic LDS than the default cap: the limit is a per-kernel attribute
      if (s.lds_bytes > (uint32_t)kProgMaxLdsBytes) return (int)hipErrorInvalidValue;
      const hipError_t e = hipFuncSetAttribute(sym, hipFuncAttributeMaxDynamicSharedMemorySize, (int)s.lds_bytes);
      if (e != hipSuccess) return (int)e;
    }
    void* one[1] = {&pa};
    return (int)hipLaunchKernel(sym, dim3(s.grid[0], s.grid[1], s.grid[2]), dim3(s.block[0], s.block[1], s.block[2]),
                                one, s.lds_bytes, static_cast<hipStream_t>(stream));
  }
  ArgList list;
  if (!list_arguments(kernel, args, s.grid[0], &list)) return (int)hipErrorInvalidValue;
  return (int)hipLaunchKernel(sym, dim3(s.grid[0], s.grid[1], s.grid[2]), dim3(s.block[0], s.block[1], s.block[2]),
                              list.address, s.lds_bytes, static_cast<hipStream_t>(stream));
}

KernelResources kernel_resources(int32_t kernel, const KernelArgs& args) {
  KernelResources r;
  const void* sym = (kernel >= 0 && kernel < K_COUNT) ? symbol_for(kernel, args) : nullptr;
  if (!sym) return r;
  hipFuncAttributes attr;
  if (hipFuncGetAttributes(&attr, sym) == hipSuccess) {
    r.vgprs = attr.numRegs;
    r.static_lds = (int32_t)attr.sharedSizeBytes;
    r.from_device = true;
  } else {
    (void)hipGetLastError();   // no device: the caller falls back to its own estimate
  }
  return r;
}

}  // namespace fs
