// Per-family lookup of the compiled kernel variant for a (kernel id, parameter block).
#pragma once
#include "launch.hpp"

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

const void* unfused_kernel_symbol(int32_t kernel, const KernelArgs& a);
const void* softmax_kernel_symbol(int32_t kernel, const KernelArgs& a);
const void* layernorm_kernel_symbol(int32_t kernel, const KernelArgs& a);
const void* gelu_kernel_symbol(int32_t kernel, const KernelArgs& a);
const void* tchain_kernel_symbol(int32_t kernel, const KernelArgs& a);
const void* rowops_kernel_symbol(int32_t kernel, const KernelArgs& a);
const void* rowprog_kernel_symbol(int32_t kernel, const KernelArgs& a);
}  // namespace fs
