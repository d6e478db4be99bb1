// Per-op baseline plan: one launch per op in graph order (two for a reduction over
// a non-innermost axis), float32 intermediates in the caller's workspace.
#include <algorithm>
#include <cstring>

#include "fs_internal.hpp"

namespace fs {

namespace {

constexpr int64_t kAlign = 256;
int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

// First-fit reuse of workspace blocks whose tenant is dead (lifetime = producer op
// to last consumer op).  A block is never handed to the op that still reads it.
struct Arena {
  struct Block { int64_t off, size; bool free; };
  std::vector<Block> blocks;
  int64_t top = 0;
  int64_t alloc(int64_t bytes) {
    bytes = round_up(bytes, kAlign);
    for (Block& b : blocks)
      if (b.free && b.size >= bytes) { b.free = false; return b.off; }
    blocks.push_back({top, bytes, false});
    top += bytes;
    return top - bytes;
  }
  void release(int64_t off) {
    for (Block& b : blocks)
      if (b.off == off) b.free = true;
  }
};

int pick_vec(int64_t inner) { return inner % 8 == 0 ? 8 : inner % 4 == 0 ? 4 : 1; }

// Units along q of the transpose's tile (256 units of vec x vec elements).  What a shape costs is the padded area, times
// what the ends of its runs waste where they fall inside 128-byte lines -- on the writing side more than on the reading
// one, and not where one tile spans the whole of a dense row.  Measured (us for 8 / 16 / 32 units): [64,197,768] bf16,
// rows of 197 written, 8.6 / 12.3 / 17.2; [16,1024,1000] bf16, rows of 1000 read, 16.9 / 12.8 / 12.9; [64,49,2048] bf16,
// area 5.2 / 2.6 / 1.3 times the tensor, 8.1 / 6.3 / 6.0; extents and rows of whole lines within 3 %.
uint32_t transpose_units_along_q(const TransposeP& p) {
  uint32_t best = 16;
  double best_cost = 0;
  for (uint32_t units : {16u, 8u, 32u}) {
    const uint32_t side_q = units * p.vec, side_x = 256 / units * p.vec;
    const uint32_t tq = (p.nq + side_q - 1) / side_q, tx = (p.nx + side_x - 1) / side_x;
    const auto waste = [&](uint32_t pitch, uint32_t extent, uint32_t tiles, uint32_t side) {
      if ((uint64_t)pitch * p.elem_bytes % 128 == 0 || (tiles == 1 && pitch == extent)) return 0.0;
      return 128.0 / ((double)side * p.elem_bytes);
    };
    const double area = (double)tq * side_q / p.nq * ((double)tx * side_x / p.nx);
    const double cost = area * (1.0 + 0.6 * waste(p.out_row, p.nx, tx, side_x) + 0.15 * waste(p.in_row, p.nq, tq, side_q));
    if (best_cost == 0 || cost < best_cost) { best = units; best_cost = cost; }
  }
  return best;
}

uint32_t pow2_at_least(uint32_t v) {
  uint32_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

}  // namespace

fs_status build_unfused(const fs_graph& g, Candidate* out) {
  const int n_t = (int)g.tensors.size();
  std::vector<BufRef> where(n_t);
  std::vector<int32_t> dt(n_t);          // dtype of the buffer that holds the tensor
  std::vector<int> last_use(n_t, -1);
  for (int t = 0; t < n_t; ++t)
    for (int c : g.tensors[t].consumers) last_use[t] = std::max(last_use[t], c);

  for (int t : g.inputs) {
    where[t].kind = BUF_INPUT;
    where[t].slot = g.tensors[t].input_slot;
    dt[t] = g.tensors[t].dtype;
  }

  Arena arena;
  int64_t moved = 0;
  std::vector<Launch>& L = out->launches;
  L.clear();

  auto add_launch = [&](int32_t kernel) -> Launch& {
    L.emplace_back();
    L.back().kernel = kernel;
    L.back().shape.block[0] = 256;
    return L.back();
  };
  auto grid1d = [](Launch& l, int64_t threads) { l.shape.grid[0] = (uint32_t)std::max<int64_t>(1, (threads + 255) / 256); };

  for (int oi = 0; oi < (int)g.ops.size(); ++oi) {
    const Op& op = g.ops[oi];
    const Tensor& r = g.tensors[op.out];
    const Tensor& a = g.tensors[op.in[0]];
    const int64_t n_out = r.numel();

    // where the result lives
    BufRef dst;
    int32_t dst_dt = r.dtype;
    bool extra_store = false;   // output with consumers and a narrower storage dtype
    if (r.output_slot >= 0 && (r.consumers.empty() || r.store_as == r.dtype)) {
      dst.kind = BUF_OUTPUT;
      dst.slot = r.output_slot;
      dst_dt = r.store_as;
    } else {
      dst.kind = BUF_WORKSPACE;
      dst.offset = arena.alloc(n_out * dtype_bytes(r.dtype));
      extra_store = r.output_slot >= 0;
    }
    where[op.out] = dst;
    dt[op.out] = dst_dt;

    const int32_t opc = op.opcode;
    if (opc <= FS_MAX || opc == FS_BROADCAST) {
      const int ib = opc == FS_BROADCAST ? op.in[0] : op.in[1];
      const Tensor& b = g.tensors[ib];
      // per-axis strides of both operands over the result, then collapse
      int64_t dims[FS_MAX_RANK], sa[FS_MAX_RANK], sb[FS_MAX_RANK];
      auto strides = [&](const Tensor& t, int64_t* s) {
        int64_t acc = 1;
        for (int k = r.rank - 1; k >= 0; --k) {
          const int kt = k - (r.rank - t.rank);
          const int64_t d = kt >= 0 ? t.dims[kt] : 1;
          s[k] = (d == 1) ? 0 : acc;
          acc *= d;
        }
      };
      strides(a, sa);
      strides(b, sb);
      for (int k = 0; k < r.rank; ++k) dims[k] = r.dims[k];
      int64_t cd[FS_MAX_RANK], ca[FS_MAX_RANK], cb[FS_MAX_RANK];
      int cr = 0;
      for (int k = 0; k < r.rank; ++k) {
        if (dims[k] == 1) continue;
        if (cr > 0 && ca[cr - 1] == sa[k] * dims[k] && cb[cr - 1] == sb[k] * dims[k]) {
          cd[cr - 1] *= dims[k];
          ca[cr - 1] = sa[k];
          cb[cr - 1] = sb[k];
        } else {
          cd[cr] = dims[k]; ca[cr] = sa[k]; cb[cr] = sb[k];
          ++cr;
        }
      }
      if (cr == 0) { cd[0] = 1; ca[0] = 0; cb[0] = 0; cr = 1; }
      Launch& l = add_launch(K_BINARY);
      BinaryP& p = l.args.u.binary;
      p = BinaryP{};
      p.op = opc == FS_BROADCAST ? B_FIRST : opc;   // B_ADD..B_MAX share the opcode numbering
      p.a_dt = dt[op.in[0]]; p.b_dt = dt[ib]; p.out_dt = dst_dt;
      p.rank = cr;
      p.n = (uint32_t)n_out;
      for (int k = 0; k < cr; ++k) { p.dims[k] = (uint32_t)cd[k]; p.sa[k] = (uint32_t)ca[k]; p.sb[k] = (uint32_t)cb[k]; }
      p.vec = pick_vec(cd[cr - 1]);
      l.ptr[0] = where[op.in[0]]; l.ptr[1] = where[ib]; l.ptr[2] = dst;
      grid1d(l, n_out / p.vec);
      moved += a.numel() * dtype_bytes(p.a_dt) + (opc == FS_BROADCAST ? 0 : b.numel() * dtype_bytes(p.b_dt)) + n_out * dtype_bytes(dst_dt);
    } else if (opc == FS_REDUCE_SUM || opc == FS_REDUCE_MAX || opc == FS_REDUCE_MEAN) {
      int64_t outer = 1, inner = 1;
      for (int k = 0; k < op.axis; ++k) outer *= a.dims[k];
      for (int k = op.axis + 1; k < a.rank; ++k) inner *= a.dims[k];
      const int64_t red = a.dims[op.axis];
      const int32_t rop = opc == FS_REDUCE_SUM ? R_SUM : opc == FS_REDUCE_MAX ? R_MAX : R_MEAN;
      const float mean_scale = rop == R_MEAN ? (float)(1.0 / (double)red) : 1.0f;
      if (inner == 1) {
        Launch& l = add_launch(K_REDUCE_ROW);
        ReduceP& p = l.args.u.reduce;
        p = ReduceP{};
        p.op = rop; p.in_dt = dt[op.in[0]]; p.out_dt = dst_dt;
        p.outer = (uint32_t)outer; p.red = (uint32_t)red; p.inner = 1;
        p.vec = pick_vec(red);
        p.lanes_per_row = std::min<uint32_t>(64, pow2_at_least((uint32_t)((red + p.vec - 1) / p.vec)));
        p.post_scale = mean_scale;
        l.ptr[0] = where[op.in[0]]; l.ptr[1] = dst;
        l.shape.grid[0] = (uint32_t)((outer + 256 / p.lanes_per_row - 1) / (256 / p.lanes_per_row));
      } else {
        const int vec = pick_vec(inner);
        const int64_t inner_blocks = (inner / vec + 255) / 256;
        int64_t nchunk = std::max<int64_t>(1, 2048 / std::max<int64_t>(1, outer * inner_blocks));
        nchunk = std::min<int64_t>(nchunk, std::max<int64_t>(1, red / 32));
        const int64_t chunk = (red + nchunk - 1) / nchunk;
        nchunk = (red + chunk - 1) / chunk;
        BufRef partial = dst;
        int32_t partial_dt = dst_dt;
        if (nchunk > 1) {
          partial.kind = BUF_WORKSPACE;
          partial.offset = arena.alloc(outer * nchunk * inner * 4);
          partial_dt = FS_F32;
        }
        {
          Launch& l = add_launch(K_REDUCE_MID);
          ReduceP& p = l.args.u.reduce;
          p = ReduceP{};
          p.op = rop; p.in_dt = dt[op.in[0]]; p.out_dt = partial_dt; p.vec = vec;
          p.outer = (uint32_t)outer; p.red = (uint32_t)red; p.inner = (uint32_t)inner;
          p.chunk = (uint32_t)chunk; p.nchunk = (uint32_t)nchunk;
          p.post_scale = nchunk > 1 ? 1.0f : mean_scale;
          l.ptr[0] = where[op.in[0]]; l.ptr[1] = partial;
          l.shape.grid[0] = (uint32_t)(inner_blocks * nchunk * outer);
        }
        if (nchunk > 1) {
          Launch& l = add_launch(K_REDUCE_MID);
          ReduceP& p = l.args.u.reduce;
          p = ReduceP{};
          p.op = rop == R_MEAN ? R_SUM : rop; p.in_dt = FS_F32; p.out_dt = dst_dt; p.vec = vec;
          p.outer = (uint32_t)outer; p.red = (uint32_t)nchunk; p.inner = (uint32_t)inner;
          p.chunk = (uint32_t)nchunk; p.nchunk = 1;
          p.post_scale = mean_scale;
          l.ptr[0] = partial; l.ptr[1] = dst;
          l.shape.grid[0] = (uint32_t)(inner_blocks * outer);
          arena.release(partial.offset);
          moved += 2 * outer * nchunk * inner * 4;
        }
      }
      moved += a.numel() * dtype_bytes(dt[op.in[0]]) + n_out * dtype_bytes(dst_dt);
    } else if (opc == FS_TRANSPOSE) {
      // the output's axes with their extents and input strides; extents of 1 dropped, axes that stay neighbours merged
      int64_t in_stride_axis[FS_MAX_RANK];   // contiguous strides of the input, by input axis
      {
        int64_t acc = 1;
        for (int k = a.rank - 1; k >= 0; --k) { in_stride_axis[k] = acc; acc *= a.dims[k]; }
      }
      int64_t ext[FS_MAX_RANK], from[FS_MAX_RANK];
      int m = 0;
      for (int k = 0; k < r.rank; ++k) {
        const int64_t stride = in_stride_axis[op.perm[k]];
        if (r.dims[k] == 1) continue;
        if (m > 0 && from[m - 1] == stride * r.dims[k]) {
          ext[m - 1] *= r.dims[k];
          from[m - 1] = stride;
        } else {
          ext[m] = r.dims[k];
          from[m++] = stride;
        }
      }
      if (m == 0) { ext[0] = 1; from[0] = 1; m = 1; }
      const bool keeps_inner = from[m - 1] == 1;
      Launch& l = add_launch(keeps_inner ? K_TRANSPOSE_ROWS : K_TRANSPOSE_TILE);
      TransposeP& p = l.args.u.transpose;
      p = TransposeP{};
      p.elem_bytes = dtype_bytes(a.dtype);
      p.n = (uint32_t)n_out;
      p.stream = streams_inputs(g) ? 1 : 0;
      l.ptr[0] = where[op.in[0]]; l.ptr[1] = dst;
      if (keeps_inner) {
        const int64_t inner = ext[m - 1];
        int vec = 16 / p.elem_bytes;
        while (vec > 1 && inner % vec != 0) vec >>= 1;
        p.vec = vec;
        uint32_t lead[3] = {1, 1, 1};
        for (int k = 0; k < m - 1; ++k) {
          lead[3 - (m - 1) + k] = (uint32_t)ext[k];
          p.in_stride[3 - (m - 1) + k] = (uint32_t)from[k];
        }
        p.out_ext[0] = lead[1];
        p.out_ext[1] = lead[2];
        p.out_ext[2] = (uint32_t)inner;
        grid1d(l, n_out / vec);
      } else {
        int q = 0;   // the output axis that the input's innermost axis has become
        for (int k = 0; k < m; ++k) if (from[k] == 1) q = k;
        p.nq = (uint32_t)ext[q];
        p.nx = (uint32_t)ext[m - 1];
        p.in_row = (uint32_t)from[m - 1];
        int64_t to[FS_MAX_RANK], acc = 1;
        for (int k = m - 1; k >= 0; --k) { to[k] = acc; acc *= ext[k]; }
        p.out_row = (uint32_t)to[q];
        uint32_t batch[2] = {1, 1};
        for (int k = m - 2, slot = 1; k >= 0; --k) {
          if (k == q) continue;
          batch[slot] = (uint32_t)ext[k];
          p.in_batch[slot] = (uint32_t)from[k];
          p.out_batch[slot] = (uint32_t)to[k];
          --slot;
        }
        const uint32_t v128 = 16 / p.elem_bytes;
        p.vec = p.nq >= v128 && p.nx >= v128 ? (int32_t)v128 : 1;
        // A small matrix per batch entry gets a wavefront's tile, not a workgroup's: with one in 256 threads and 16 to 32 KB of
        // LDS most threads idle and few matrices are in flight.  Measured (us, a workgroup each / a wavefront each / 32x32
        // single elements): [16384,30,30] bf16 27.2 / 15.7 / 31.9, [16384,20,20] f32 15.9 / 12.1 / 26.0, [4096,9,9]
        // bf16 5.9 / 4.6 / 4.9, [65536,8,8] f32 36.5 / 16.9 / 49.7; full tiles ([16384,64,64] bf16) 45.0 / 43.9 / 126.
        p.tile_units = p.nq <= 8u * p.vec && p.nx <= 8u * p.vec ? 64u : 256u;
        p.tile_uq = p.vec == 1 ? 0u : p.tile_units == 64u ? 8u : transpose_units_along_q(p);
        const uint32_t side_q = p.vec > 1 ? p.tile_uq * p.vec : 32, side_x = p.vec > 1 ? p.tile_units / p.tile_uq * p.vec : 32;
        const uint32_t tq = (p.nq + side_q - 1) / side_q, tx = (p.nx + side_x - 1) / side_x;
        // Neighbouring workgroups walk along q where that makes them read whole lines of one short contiguous span
        // ([64,512,12,64] -> [64,12,64,512] float32: 36.1 against 37.4 us); along x otherwise: long or unaligned input
        // rows lose more than that on the writing side (4096 x 4096 float32 25.2 against 29.3, 4001 x 3333 26.5 / 39.0).
        // Longer rows that are written out as rows of 1 to 2 KB take every other tile along q first, then the next x, then
        // the tiles in between (us along x / along q / every other one, float32 to [.., h*d, s]): s 512 of 4 KB rows 49.7 /
        // 48.8 / 46.5, of 8 KB rows 96.0 / 92.6 / 89.4, s 500 of 8 KB rows 61.5 / 54.2 / 51.0, s 256 25.3 / 24.4 / 23.9, s 384
        // level; outside that span it loses: s 256 of 4 KB rows in bf16 13.0 / 13.2 / 13.7, s 2048 23.9 / 24.8 / 24.4.
        const uint64_t read_row = (uint64_t)p.nq * p.elem_bytes, written_row = (uint64_t)p.out_row * p.elem_bytes;
        const bool whole_lines = (uint64_t)p.in_row * p.elem_bytes % 128 == 0;
        p.every_other = whole_lines && read_row > 3072 && tq % 2 == 0 && written_row >= 1024 && written_row <= 2048 ? 1 : 0;
        p.walk_q = whole_lines && (read_row <= 3072 || p.every_other) ? 1 : 0;
        p.div[0] = make_fastdiv(p.walk_q ? tq >> p.every_other : tx);
        p.div[1] = make_fastdiv(p.walk_q ? tx : tq);
        p.div[2] = make_fastdiv(batch[1]);
        for (const FastDiv& d : p.div)   // (both tile axes are at least 2 long, so none of these is near 2^31)
          if (d.d == 0) return fail(FS_ERR_SHAPE, "transpose: no exact division by one of its extents");
        const int64_t blocks = (int64_t)tq * tx * batch[0] * batch[1];
        if (blocks >= (int64_t(1) << 31)) return fail(FS_ERR_SHAPE, "transpose: too many tiles");
        p.n_tiles = (uint32_t)blocks;
        const int64_t per_workgroup = p.vec > 1 && p.tile_units == 64u ? 4 : 1;
        l.shape.grid[0] = (uint32_t)((blocks + per_workgroup - 1) / per_workgroup);
      }
      moved += 2 * n_out * p.elem_bytes;
    } else {
      // unary family, convert included
      Launch& l = add_launch(K_UNARY);
      UnaryP& p = l.args.u.unary;
      p = UnaryP{};
      switch (opc) {
        case FS_SCALE: p.op = U_SCALE; break;
        case FS_ADD_SCALAR: p.op = U_ADD_SCALAR; break;
        case FS_SQUARE: p.op = U_SQUARE; break;
        case FS_EXP: p.op = U_EXP; break;
        case FS_RSQRT: p.op = U_RSQRT; break;
        case FS_TANH: p.op = U_TANH; break;
        case FS_GELU_TANH: p.op = U_GELU; break;
        case FS_GELU_TANH_GRAD: p.op = U_GELU_GRAD; break;
        case FS_LOG: p.op = U_LOG; break;
        case FS_SIGMOID: p.op = U_SIGMOID; break;
        case FS_RELU: p.op = U_RELU; break;
        case FS_ABS: p.op = U_ABS; break;
        case FS_SQRT: p.op = U_SQRT; break;
        default: p.op = U_COPY; break;   // FS_CONVERT: the store does the rounding
      }
      p.in_dt = dt[op.in[0]]; p.out_dt = dst_dt;
      p.n = (uint32_t)n_out;
      p.vec = pick_vec(n_out);
      p.value = (float)op.scalar;
      l.ptr[0] = where[op.in[0]]; l.ptr[1] = dst;
      grid1d(l, n_out / p.vec);
      moved += n_out * (dtype_bytes(p.in_dt) + dtype_bytes(dst_dt));
    }

    if (extra_store) {
      Launch& l = add_launch(K_UNARY);
      UnaryP& p = l.args.u.unary;
      p = UnaryP{};
      p.op = U_COPY; p.in_dt = dst_dt; p.out_dt = r.store_as;
      p.n = (uint32_t)n_out; p.vec = pick_vec(n_out);
      l.ptr[0] = dst;
      l.ptr[1].kind = BUF_OUTPUT; l.ptr[1].slot = r.output_slot;
      grid1d(l, n_out / p.vec);
      moved += n_out * (dtype_bytes(dst_dt) + dtype_bytes(r.store_as));
    }

    // operands that die here give their workspace back
    for (int i = 0; i < op.n_in; ++i) {
      const int t = op.in[i];
      if (where[t].kind == BUF_WORKSPACE && last_use[t] == oi && !(i == 1 && op.in[0] == op.in[1])) arena.release(where[t].offset);
    }
  }

  fs_plan_info& info = out->info;
  memset(&info, 0, sizeof info);
  info.scheme = FS_SCHEME_UNFUSED;
  info.n_kernels = (int32_t)L.size();
  info.workspace_bytes = arena.top;
  info.bytes_min = graph_bytes_min(g);
  info.bytes_moved_model = moved;
  snprintf(info.pattern, sizeof info.pattern, "unfused");
  // dominant kernel = the launch with the most threads
  size_t dom = 0;
  for (size_t i = 1; i < L.size(); ++i)
    if ((uint64_t)L[i].shape.grid[0] > (uint64_t)L[dom].shape.grid[0]) dom = i;
  if (!L.empty()) {
    for (int k = 0; k < 3; ++k) { info.block[k] = (int32_t)L[dom].shape.block[k]; info.grid[k] = (int32_t)L[dom].shape.grid[k]; }
    snprintf(info.kernel, sizeof info.kernel, "%s", kernel_name(L[dom].kernel));
  }
  return FS_OK;
}

// Up to 96 MiB of inputs are read through the caches, more past them.  A hinted read takes no place in the 256 MB memory-side
// cache: a later read of the same tensor, by this kernel or another, goes to device memory again, and a read of lines that
// the kernel before has just written is slower too.  Measured (us, hinted / plain), inputs written by the kernel before:
// softmax f16 160 MB moved 30.4 / 26.6, LayerNorm f32 80 MB 20.4 / 16.7, its backward 120 MB 32.6 / 25.0, 24 MB of
// either level; three sets of buffers in turn: softmax f16 48 MB 7.8 / 7.6, 80 MB 15.0 / 13.0, LayerNorm bf16 48 MB 11.0 / 8.6,
// scores f16 120 MB 20.8 / 17.3, transpose bf16 24 MB 5.3 / 4.3, bias + GELU backward f32 80 MB 18.9 / 15.6.  Inputs that no
// cache can hold are better off without taking a place there: the same turns level out at 100 MB of inputs and lose 3 to 7 %
// from 130 MB on.  Where each pass reads other memory (900 MB of inputs in turn, 22 shapes of 4 to 96 MB in all families) the plain read
// loses 0.3 % on average and at most 6 % (transpose bf16 4096 x 4096 13.7 / 14.5, LayerNorm bf16 [8192,1024] 10.0 / 10.4, f32 [8192,768]
// 11.3 / 11.6); the same shapes over three sets of buffers gain 11 % on average and lose at most 0.3 %.
//
// The parts of a larger graph keep hinted reads: what one step hands to the next was stored past the caches, and the inputs of
// all steps together use up the place (block backward of 53 MB 29.4 / 30.1, of 201 MB 51.7 / 56.0).  A program of one pattern has no such
// steps: LayerNorm backward f32 [8192,768] 17.8 / 15.3, RMS norm bf16 [4096,4096] 12.5 / 10.2.
bool streams_inputs(const fs_graph& g) {
  int64_t b = 0;
  for (int t : g.inputs) b += g.tensors[t].numel() * dtype_bytes(g.tensors[t].dtype);
  return g.cut_out || b > (int64_t(96) << 20);
}

int64_t graph_bytes_min(const fs_graph& g) {
  int64_t b = 0;
  for (int t : g.inputs) b += g.tensors[t].numel() * dtype_bytes(g.tensors[t].dtype);
  for (int t : g.outputs) b += g.tensors[t].numel() * dtype_bytes(g.tensors[t].store_as);
  return b;
}

}  // namespace fs
