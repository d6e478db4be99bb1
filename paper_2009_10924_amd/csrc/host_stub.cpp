// TEST-ONLY stand-in for kernels/*.hip: lets the host core (graph, matcher, evaluator, planner, explorer, row-program
// compiler, code generator, executor) be built with the host compiler and its sanitizers and "executed" on a machine
// without a GPU.  Launches are checked (shape, pointers) and recorded, never run; device pointers are never
// dereferenced.  The product library is never built from this file.
#include <cstdlib>
#include <cstring>
#include <memory>
#include <string>

#include "fs_internal.hpp"
#include "kernels/kernel_arguments.hpp"

namespace fs {

namespace {
const char* const kNames[K_COUNT] = {"unary", "binary", "reduce_row", "reduce_mid", "transpose_rows", "transpose_tile", "copy",
                                     "softmax_wave", "softmax_block", "layernorm_wave", "layernorm_block", "bias_gelu",
                                     "bias_gelu_dbias", "colfold", "tchain_wave", "tchain_lds", "row_wave", "row_block",
                                     "row_program", "layernorm_bwd", "row_generated"};
long g_launches = 0;

// what any launch must satisfy whatever the kernel: returns a hipError-like code (1 = invalid value)
int check_shape(const LaunchShape& s) {
  const uint64_t threads = (uint64_t)s.block[0] * s.block[1] * s.block[2];
  const uint64_t groups = (uint64_t)s.grid[0] * s.grid[1] * s.grid[2];
  if (threads == 0 || threads > 1024 || groups == 0 || groups > 0x7fffffffull) return 1;
  if (s.lds_bytes > 160u * 1024u) return 1;
  return 0;
}
template <typename T>
T argument(const ArgList& l, size_t k) {
  T v;
  memcpy(&v, l.address[k], sizeof v);
  return v;
}
bool same(const FastDiv& a, const FastDiv& b) { return a.d == b.d && a.m == b.m && a.s == b.s; }

// The arguments of a launch, taken apart with the kernel's own functions, are what its parameter block says.
bool arguments_round_trip(int32_t kernel, const KernelArgs& a, uint32_t grid) {
  ArgList l;
  if (!list_arguments(kernel, a, grid, &l)) return false;
  auto u = [&](size_t k) { return argument<uint32_t>(l, k); };
  auto f = [&](size_t k) { return argument<float>(l, k); };
  switch (kernel) {
    case K_SOFTMAX_WAVE: case K_SOFTMAX_BLOCK: {
      const SoftmaxP& s = a.u.softmax;
      const bool block = kernel == K_SOFTMAX_BLOCK;
      const SoftmaxP q = softmax_params(block, u(3), u(4), f(5), u(6), u(7), u(8), u(9), u(10), u(11), u(12));
      if (s.vecs_per_lane == 0 ? u(3) != s.cols : (q.rows != s.rows || q.cols != s.cols || q.lanes_per_row != s.lanes_per_row)) return false;
      if (!block && q.lanes_log2 != s.lanes_log2) return false;
      return q.mask_inner == (s.mask_inner != 0) && q.scale == s.scale && same(q.od[1], s.od[1]) && same(q.od[2], s.od[2]) &&
             memcmp(q.ms, s.ms, sizeof q.ms) == 0 && (argument<void*>(l, 1) != nullptr) == (s.has_mask && a.p[1]);
    }
    case K_LAYERNORM_WAVE: case K_LAYERNORM_BLOCK: {
      const LayerNormP& n = a.u.layernorm;
      const LayerNormP q = layernorm_params(kernel == K_LAYERNORM_BLOCK, u(3), u(4), f(8), f(9));
      return q.rows == n.rows && q.cols == n.cols && q.lanes_per_row == n.lanes_per_row && !q.has_res == !n.has_res && !q.has_bias == !n.has_bias &&
             !q.has_affine == !n.has_affine && q.eps == n.eps && q.inv_cols == n.inv_cols && l.n == (n.stats ? 12u : 10u);
    }
    case K_LAYERNORM_BWD: {
      const LnBwdP& n = a.u.lnbwd;
      const LnBwdP q = lnbwd_params(u(5), u(6));
      return q.rows == n.rows && q.cols == n.cols && q.lanes_per_row == n.lanes_per_row && q.lanes_log2 == n.lanes_log2 && lnbwd_grid(u(6)) == grid &&
             q.inv_cols == (float)(1.0 / (double)n.cols);
    }
    case K_TCHAIN_WAVE: case K_TCHAIN_LDS: {
      const TChainP& t = a.u.tchain;
      const TChainP q = tchain_params(u(3), u(4), u(5), u(6), u(7), u(8), u(9), f(10));
      return q.D == t.D && q.S == t.S && q.H == t.H && q.s_tile == t.s_tile && q.lanes_log2 == t.lanes_log2 && q.lanes_per_row == t.lanes_per_row &&
             same(q.div_s_tiles, t.div_s_tiles) && same(q.div_h, t.div_h) && q.eps == t.eps;
    }
    case K_ROW_WAVE: case K_ROW_BLOCK: {
      const RowP& r = a.u.row;
      const RowP q = row_params(kernel == K_ROW_BLOCK, u(3), u(4), f(6), f(7));
      return q.rows == r.rows && q.cols == r.cols && q.lanes_per_row == r.lanes_per_row && q.f[0] == r.f[0] && q.f[1] == r.f[1];
    }
    case K_TRANSPOSE_TILE: {
      const TransposeP& t = a.u.transpose;
      if (t.vec == 1) return true;   // the block as it is
      const uint32_t uq = t.tile_units == 64 ? 8u : t.tile_uq, vec = (uint32_t)t.vec;
      TransposeP q = units_params(uq * vec, t.tile_units / uq * vec, u(2), u(3), u(4), u(5), u(6), u(7), u(8), u(9), u(10), u(11));
      if (transpose_two_batch_axes(t)) {
        units_second_axis(&q, u(4), u(12), u(13), u(14), u(15));
        if (!same(q.div[2], t.div[2])) return false;
      }
      return same(q.div[0], t.div[0]) && same(q.div[1], t.div[1]) && q.nq == t.nq && q.nx == t.nx && q.in_row == t.in_row && q.out_row == t.out_row &&
             q.in_batch[0] == t.in_batch[0] && q.in_batch[1] == t.in_batch[1] && q.out_batch[0] == t.out_batch[0] &&
             q.out_batch[1] == t.out_batch[1] && !q.walk_q == !t.walk_q && q.every_other == t.every_other && q.n_tiles == t.n_tiles;
    }
    default: return true;
  }
}

// Every field of the words at its limits comes back, and one beyond is refused: number of checks that failed.
int check_words() {
  int bad = 0;
  const FastDiv divs[] = {{1, 0, 0}, {3, 0xAAAAAAABu, 1}, {0x7fffffffu, 0xffffffffu, 30}};
  auto expect = [&](int32_t kernel, const KernelArgs& a, uint32_t grid, bool fits) {
    ArgList l;
    bad += fits ? !arguments_round_trip(kernel, a, grid) : list_arguments(kernel, a, grid, &l);
  };
  for (int block = 0; block < 2; ++block)
    for (int lanes = 0; lanes <= (block ? 7 : 6); ++lanes)
      for (const FastDiv& d : divs)
        for (uint32_t cols : {1u, 197u, (1u << 18) - 1u, 1u << 18, (1u << 24) - 1u, 1u << 24}) {
          const int32_t per_row = block ? 64 * lanes : 1 << lanes;
          KernelArgs a{};
          for (int mask = 0; mask < 4; ++mask) {
            a = KernelArgs{};
            a.p[1] = &a;
            SoftmaxP& s = a.u.softmax;
            s.has_mask = mask & 1, s.mask_inner = mask >> 1, s.rows = 0x7fffffffu, s.cols = cols, s.lanes_per_row = per_row, s.lanes_log2 = lanes;
            s.vecs_per_lane = 1, s.scale = 0.125f, s.od[1] = d, s.od[2] = divs[2], s.ms[0] = 0xffffffffu, s.ms[2] = 1;
            expect(block ? K_SOFTMAX_BLOCK : K_SOFTMAX_WAVE, a, 1, cols < (1u << 18));
          }
          for (int flags = 0; flags < 16; ++flags) {
            a = KernelArgs{};
            LayerNormP& n = a.u.layernorm;
            n.has_res = flags & 1, n.has_bias = (flags >> 1) & 1, n.has_affine = (flags >> 2) & 1, n.stats = flags >> 3, n.rows = 0x7fffffffu;
            n.cols = cols, n.eps = 1e-5f, n.inv_cols = 1.0f / (float)cols, n.lanes_per_row = per_row, n.lanes_log2 = lanes;
            expect(block ? K_LAYERNORM_BLOCK : K_LAYERNORM_WAVE, a, 1, cols < (1u << 24));
          }
          a = KernelArgs{};
          RowP& r = a.u.row;
          r.rows = 0x7fffffffu, r.cols = cols, r.lanes_per_row = per_row, r.lanes_log2 = lanes, r.f[0] = 1e-6f, r.f[1] = 0.5f;
          expect(block ? K_ROW_BLOCK : K_ROW_WAVE, a, 1, cols < (1u << 24));
          if (block) continue;
          for (uint32_t grid : {1u, 65535u, 65536u})
            for (uint32_t c : {1u, 8191u, 8192u}) {
              a = KernelArgs{};
              LnBwdP& b = a.u.lnbwd;
              b.rows = 0x7fffffffu, b.cols = c, b.lanes_per_row = per_row, b.lanes_log2 = lanes;
              expect(K_LAYERNORM_BWD, a, grid, grid < 65536u && c < 8192u);
            }
          for (uint32_t dim : {1u, 65535u, 65536u}) {
            a = KernelArgs{};
            TChainP& t = a.u.tchain;
            t.D = dim, t.S = 0x7fffffffu, t.H = d.d, t.s_tile = 16, t.lanes_per_row = per_row, t.lanes_log2 = lanes, t.div_s_tiles = divs[2], t.div_h = d;
            t.eps = 1e-6f;
            expect(K_TCHAIN_WAVE, a, 1, dim < 65536u);
          }
        }
  KernelArgs a{};   // more lanes than a code can say
  a.u.softmax.vecs_per_lane = 1, a.u.softmax.cols = 64, a.u.softmax.lanes_per_row = 512;
  expect(K_SOFTMAX_BLOCK, a, 1, false);
  return bad;
}
}  // namespace

int launch_kernel(int32_t kernel, const KernelArgs& args, const LaunchShape& shape, void*) {
  if (kernel < 0 || kernel >= K_COUNT || kernel == K_ROW_GENERATED) return 1;
  if (check_shape(shape)) return 1;
  if (!args.p[0] && kernel != K_ROW_PROGRAM) return 1;   // every compiled-in kernel reads its first pointer
  if (kernel != K_ROW_PROGRAM && !arguments_round_trip(kernel, args, shape.grid[0])) return 1;
  ++g_launches;
  return 0;
}
int launch_pack(const PackTable& table, void*) {
  if (table.n <= 0 || table.n > kPackMaxMembers || table.total_blocks == 0) return 1;
  for (int i = 0; i < table.n; ++i)
    if (!table.e[i].in[0] || !table.e[i].out) return 1;
  ++g_launches;
  return 0;
}
int launch_fold_many(const FoldManyP& table, uint32_t n_blocks, void*) {
  if (n_blocks == 0) return 0;
  if (table.first_block[0] != 0 || !table.partials[0] || !table.out0[0]) return 1;
  ++g_launches;
  return 0;
}
KernelResources kernel_resources(int32_t, const KernelArgs&) { return KernelResources(); }
KernelResources pack_kernel_resources() { return KernelResources(); }
const char* kernel_name(int32_t k) { return (k >= 0 && k < K_COUNT) ? kNames[k] : "?"; }
const char* hip_error_text(int) { return "launch refused by the host stub"; }

// "compilation" of generated kernels: succeeds when FS_STUB_COMPILE_OK is set (the source is kept, so that identical
// sources share a kernel as in the product), otherwise fails like a missing run-time compiler would
struct GenKernel {
  std::string source;
  bool loaded = false;
};
namespace {
bool g_device = true, g_capturing = false;   // what fs_stub_state() says of the machine
}
bool gen_available() { return true; }
int gen_compile(const std::string& src, const char* entry, std::shared_ptr<GenKernel>* out, std::string* log) {
  if (getenv("FS_STUB_COMPILE_OK") && entry && src.find(entry) != std::string::npos) {
    *out = std::make_shared<GenKernel>();
    (*out)->source = src;
    return 0;
  }
  if (log) *log = "host stub: no compiler (" + std::to_string(src.size()) + " bytes of source)";
  return 1;
}
void gen_compile_together(const std::vector<GenSource>&) {}
GenResources gen_resources(const GenKernel*) { return GenResources(); }
int gen_preload(GenKernel* k) {
  k->loaded = k->loaded || g_device;
  return 0;
}
bool gen_ready(GenKernel* k, void*) {
  k->loaded = k->loaded || (g_device && !g_capturing);
  return k->loaded;
}
int gen_launch(GenKernel* k, const void* args, size_t args_bytes, const LaunchShape& shape, void*) {
  if (!k || !args || args_bytes == 0 || args_bytes % sizeof(void*) != 0 || check_shape(shape)) return 1;
  if (!k->loaded && (g_capturing || !g_device)) return 1;   // nothing can be loaded now
  k->loaded = true;
  ++g_launches;
  return 0;
}

}  // namespace fs

// the entry points that live in .hip files in the product
extern "C" fs_status fs_execute_static(const fs_plan* p, const void* const* inputs, void* const* outputs, void* hip_stream) {
  fs::clear_error();
  const fs_status s = fs::check_execute_args(p, inputs, outputs, "fs_execute_static");
  if (s != FS_OK) return s;
  const fs::Candidate& c = p->candidates[p->chosen];
  if (c.info.workspace_bytes > (int64_t)FS_STATIC_SCRATCH_BYTES)
    return fs::fail(FS_ERR_WORKSPACE, "fs_execute_static: the plan needs %lld bytes of scratch, the static array holds %lld",
                    (long long)c.info.workspace_bytes, (long long)FS_STATIC_SCRATCH_BYTES);
  return fs::run_launches(p, inputs, outputs, reinterpret_cast<void*>(0x7000000), hip_stream, c.launches.size());
}
extern "C" fs_status fs_stream_probe(void*, const void*, size_t, size_t, int32_t, int32_t, int32_t, void*) {
  return fs::fail(FS_ERR_HIP, "fs_stream_probe: not part of the host stub");
}
extern "C" long fs_stub_launch_count(void) { return fs::g_launches; }
extern "C" void fs_stub_state(int device, int capturing) { fs::g_device = device != 0, fs::g_capturing = capturing != 0; }
extern "C" int fs_stub_check_argument_words(void) { return fs::check_words(); }
