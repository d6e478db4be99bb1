// Per-op baseline: one kernel per op of the subgraph, every intermediate through
// HBM as float32.  This is what the stitched kernels are measured against
// (the paper's un-stitched execution, Section 2.2: one launch and one round trip
// through off-chip memory per op).  Each kernel still uses 128-bit accesses where
// the shape allows, so the baseline is an honest one.
#include <hip/hip_runtime.h>

#include "device_utils.hpp"
#include "kernel_table.hpp"

namespace fsk {
using namespace fs;

// ---- run-time-dtype vector access (dtype is wave-uniform, branches are scalar) ----
template <int V>
__device__ __forceinline__ void load_rt(const void* base, int dt, uint32_t off, float (&v)[V]) {
  if constexpr (V == 1) {
    if (dt == DT_F32) v[0] = load1(reinterpret_cast<const float*>(base) + off);
    else if (dt == DT_F16) v[0] = load1(reinterpret_cast<const f16_t*>(base) + off);
    else v[0] = load1(reinterpret_cast<const bf16_t*>(base) + off);
  } else if constexpr (V == 4) {
    if (dt == DT_F32) load_vec4(reinterpret_cast<const float*>(base) + off, v);
    else if (dt == DT_F16) load_vec4(reinterpret_cast<const f16_t*>(base) + off, v);
    else load_vec4(reinterpret_cast<const bf16_t*>(base) + off, v);
  } else {
    static_assert(V == 8, "vector width");
    if (dt == DT_F32) {
      float a[4], b[4];
      load_vec(reinterpret_cast<const float*>(base) + off, a);
      load_vec(reinterpret_cast<const float*>(base) + off + 4, b);
#pragma unroll
      for (int i = 0; i < 4; ++i) { v[i] = a[i]; v[4 + i] = b[i]; }
    } else if (dt == DT_F16) {
      load_vec(reinterpret_cast<const f16_t*>(base) + off, v);
    } else {
      load_vec(reinterpret_cast<const bf16_t*>(base) + off, v);
    }
  }
}

template <int V>
__device__ __forceinline__ void store_rt(void* base, int dt, uint32_t off, const float (&v)[V]) {
  if constexpr (V == 1) {
    if (dt == DT_F32) store1(reinterpret_cast<float*>(base) + off, v[0]);
    else if (dt == DT_F16) store1(reinterpret_cast<f16_t*>(base) + off, v[0]);
    else store1(reinterpret_cast<bf16_t*>(base) + off, v[0]);
  } else if constexpr (V == 4) {
    if (dt == DT_F32) store_vec4(reinterpret_cast<float*>(base) + off, v);
    else if (dt == DT_F16) store_vec4(reinterpret_cast<f16_t*>(base) + off, v);
    else store_vec4(reinterpret_cast<bf16_t*>(base) + off, v);
  } else {
    if (dt == DT_F32) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = v[i]; b[i] = v[4 + i]; }
      store_vec(reinterpret_cast<float*>(base) + off, a);
      store_vec(reinterpret_cast<float*>(base) + off + 4, b);
    } else if (dt == DT_F16) {
      store_vec(reinterpret_cast<f16_t*>(base) + off, v);
    } else {
      store_vec(reinterpret_cast<bf16_t*>(base) + off, v);
    }
  }
}

__device__ __forceinline__ float load_rt1(const void* base, int dt, uint32_t off) {
  float v[1];
  load_rt<1>(base, dt, off, v);
  return v[0];
}

// ---- unary ----------------------------------------------------------------------
__device__ __forceinline__ float unary_apply(int op, float x, float value) {
  switch (op) {
    case U_SCALE: return x * value;
    case U_ADD_SCALAR: return x + value;
    case U_SQUARE: return x * x;
    case U_EXP: return fast_exp(x);
    case U_RSQRT: return fast_rsqrt(x);
    case U_TANH: return tanhf(x);
    case U_GELU: return gelu_fwd(x);
    case U_GELU_GRAD: return gelu_grad(x);
    case U_LOG: return full_log(x);
    case U_SIGMOID: return fast_sigmoid(x);
    case U_RELU: return fmaxf(x, 0.0f);
    case U_ABS: return __builtin_fabsf(x);
    case U_SQRT: return full_sqrt(x);
    default: return x;
  }
}

template <int V>
__global__ void __launch_bounds__(256) k_unary(const void* in, void* out, UnaryP p) {
  const uint32_t i = (blockIdx.x * 256u + threadIdx.x) * V;
  if (i >= p.n) return;
  float v[V];
  load_rt<V>(in, p.in_dt, i, v);
#pragma unroll
  for (int k = 0; k < V; ++k) v[k] = unary_apply(p.op, v[k], p.value);
  store_rt<V>(out, p.out_dt, i, v);
}

// ---- binary with broadcasting ---------------------------------------------------
__device__ __forceinline__ float binary_apply(int op, float a, float b) {
  switch (op) {
    case B_ADD: return a + b;
    case B_SUB: return a - b;
    case B_MUL: return a * b;
    case B_DIV: return a / b;
    case B_MAX: return fmaxf(a, b);
    default: return a;
  }
}

template <int V>
__global__ void __launch_bounds__(256) k_binary(const void* a, const void* b, void* out, BinaryP p) {
  const uint32_t e = (blockIdx.x * 256u + threadIdx.x) * V;
  if (e >= p.n) return;
  // coordinates of element e in the collapsed output, innermost first
  uint32_t rest = e, oa = 0, ob = 0;
  uint32_t inner_sa = p.sa[p.rank - 1], inner_sb = p.sb[p.rank - 1];
  for (int k = p.rank - 1; k >= 0; --k) {
    uint32_t c;
    if (k == 0) { c = rest; }
    else { c = rest % p.dims[k]; rest = rest / p.dims[k]; }
    oa += c * p.sa[k];
    ob += c * p.sb[k];
  }
  float va[V], vb[V];
  if (inner_sa == 1 || V == 1) load_rt<V>(a, p.a_dt, oa, va);
  else { float s = load_rt1(a, p.a_dt, oa);
#pragma unroll
         for (int k = 0; k < V; ++k) va[k] = s; }
  if (inner_sb == 1 || V == 1) load_rt<V>(b, p.b_dt, ob, vb);
  else { float s = load_rt1(b, p.b_dt, ob);
#pragma unroll
         for (int k = 0; k < V; ++k) vb[k] = s; }
#pragma unroll
  for (int k = 0; k < V; ++k) va[k] = binary_apply(p.op, va[k], vb[k]);
  store_rt<V>(out, p.out_dt, e, va);
}

// ---- row reduction: [rows, cols] -> [rows] --------------------------------------
__device__ __forceinline__ float red_identity(int op) { return op == R_MAX ? -INFINITY : 0.0f; }
__device__ __forceinline__ float red_apply(int op, float a, float b) { return op == R_MAX ? fmaxf(a, b) : a + b; }

template <int V>
__global__ void __launch_bounds__(256) k_reduce_row(const void* in, void* out, ReduceP p) {
  const uint32_t L = p.lanes_per_row;
  const uint32_t rows_per_block = 256u / L;
  const uint32_t row = blockIdx.x * rows_per_block + threadIdx.x / L;
  const uint32_t lane = threadIdx.x % L;
  float acc = red_identity(p.op);
  if (row < p.outer) {
    const uint32_t base = row * p.red;
    for (uint32_t c = lane * V; c < p.red; c += L * V) {
      float v[V];
      load_rt<V>(in, p.in_dt, base + c, v);
#pragma unroll
      for (int k = 0; k < V; ++k) acc = red_apply(p.op, acc, v[k]);
    }
  }
  acc = (p.op == R_MAX) ? group_allreduce<OpMax>(acc, L) : group_allreduce<OpSum>(acc, L);
  if (row < p.outer && lane == 0) {
    float r[1] = {acc * p.post_scale};
    store_rt<1>(out, p.out_dt, row, r);
  }
}

// ---- reduction over a middle axis: [outer, red, inner] -> [outer, nchunk, inner] --
// Each lane owns V adjacent inner positions and walks `chunk` rows of the reduced
// axis; lanes of a wave read adjacent addresses.  A second launch of the same
// kernel folds the chunks.
template <int V>
__global__ void __launch_bounds__(256) k_reduce_mid(const void* in, void* out, ReduceP p) {
  const uint32_t inner_vecs = p.inner / V;
  const uint32_t n_inner_blocks = (inner_vecs + 255u) / 256u;
  uint32_t bid = blockIdx.x;
  const uint32_t ib = bid % n_inner_blocks; bid /= n_inner_blocks;
  const uint32_t ch = bid % p.nchunk;
  const uint32_t o = bid / p.nchunk;
  const uint32_t iv = ib * 256u + threadIdx.x;
  if (iv >= inner_vecs) return;
  const uint32_t r0 = ch * p.chunk;
  const uint32_t r1 = min(r0 + p.chunk, p.red);
  float acc[V];
#pragma unroll
  for (int k = 0; k < V; ++k) acc[k] = red_identity(p.op);
  uint32_t off = (o * p.red + r0) * p.inner + iv * V;
  for (uint32_t r = r0; r < r1; ++r, off += p.inner) {
    float v[V];
    load_rt<V>(in, p.in_dt, off, v);
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = red_apply(p.op, acc[k], v[k]);
  }
#pragma unroll
  for (int k = 0; k < V; ++k) acc[k] *= p.post_scale;
  store_rt<V>(out, p.out_dt, (o * p.nchunk + ch) * p.inner + iv * V, acc);
}

// ---- transpose, innermost axis kept: rows of contiguous elements are re-ordered ----
template <typename VT>
__global__ void __launch_bounds__(256) k_transpose_rows(const void* in, void* out, uint32_t n, uint32_t vec, uint32_t is0, uint32_t is1,
                                                        uint32_t is2, uint32_t oe0, uint32_t oe1, uint32_t oe2) {
  const uint32_t vi = blockIdx.x * 256u + threadIdx.x;   // vector index in the output
  const uint32_t e = vi * vec;
  if (e >= n) return;
  // Plain divisions, measured: multiply-high ones are slower here ([64,512,12,64] -> [64,12,512,64] float32 34.6 against
  // 35.5 us, the wavefronts then reach their loads closer together), four vectors per thread slower still (36.1).
  uint32_t rest = e;
  const uint32_t c3 = rest % oe2; rest /= oe2;
  const uint32_t c2 = rest % oe1; rest /= oe1;
  const uint32_t c1 = rest % oe0, c0 = rest / oe0;
  const uint32_t src = c0 * is0 + c1 * is1 + c2 * is2 + c3;
  reinterpret_cast<VT*>(out)[vi] = reinterpret_cast<const VT*>(in)[src / vec];
}

// Tile `index` of a transpose, and where its batch entry starts in the input and in the output.  TWO: there are two axes
// outside the tile (with one, it is the second of TransposeP's).
template <bool TWO>
struct TileAt {
  uint32_t bq, bx;
  size_t in_base, out_base;
  __device__ __forceinline__ TileAt(const TransposeP& p, uint32_t index) {
    uint32_t rest = index;
    uint32_t r = fast_div(rest, p.div[0]);
    const uint32_t inner = rest - r * p.div[0].d;
    rest = r;
    r = fast_div(rest, p.div[1]);
    const uint32_t outer = rest - r * p.div[1].d;
    const uint32_t phase = r & p.every_other;
    r >>= p.every_other;
    uint32_t b0 = 0, b1 = r;
    if constexpr (TWO) {
      b0 = fast_div(r, p.div[2]);
      b1 = r - b0 * p.div[2].d;
    }
    bq = p.walk_q ? (inner << p.every_other) + phase : outer;
    bx = p.walk_q ? outer : inner;
    in_base = (size_t)b1 * p.in_batch[1];
    out_base = (size_t)b1 * p.out_batch[1];
    if constexpr (TWO) {
      in_base += (size_t)b0 * p.in_batch[0];
      out_base += (size_t)b0 * p.out_batch[0];
    }
  }
};

// ---- transpose, innermost axis moves: 32x32 tile through padded LDS ---------------
// For tile axes shorter than a 128-bit access.  Reads are contiguous along the input's innermost axis, writes along the
// output's; the 33-word pitch keeps both LDS phases free of bank conflicts.
template <typename T>
__global__ void __launch_bounds__(256) k_transpose_tile(const T* __restrict__ in, T* __restrict__ out, TransposeP p) {
  __shared__ T tile[32][33];
  const TileAt<true> t(p, blockIdx.x);
  const uint32_t tx = threadIdx.x & 31u, ty = threadIdx.x >> 5;
  for (uint32_t j = ty; j < 32u; j += 8u) {
    const uint32_t cq = t.bq * 32u + tx, cx = t.bx * 32u + j;
    if (cq < p.nq && cx < p.nx) tile[j][tx] = in[t.in_base + cq + (size_t)cx * p.in_row];
  }
  __syncthreads();
  for (uint32_t i = ty; i < 32u; i += 8u) {
    const uint32_t cq = t.bq * 32u + i, cx = t.bx * 32u + tx;
    if (cq < p.nq && cx < p.nx) out[t.out_base + (size_t)cq * p.out_row + cx] = tile[tx][i];
  }
}

// ---- transpose, innermost axis moves: 128-bit accesses on both HBM sides AND both LDS sides ----------------
// The tile is UQ x UX units of VEC x VEC elements (UQ * UX = UNITS threads, one unit each; VEC = elements in 16
// bytes), TQ = UQ * VEC along the input's innermost axis q by TX = UX * VEC along the output's innermost axis x.
// A thread loads its unit as VEC rows of 16 bytes (a wave reads runs of UQ * 16 bytes), transposes it in
// registers (32-bit elements: a renaming; 16-bit elements: one byte-permute per pair), and parks it in LDS as VEC
// 16-byte pieces, one per tile column, each holding VEC consecutive elements of x.
// After the barrier a thread reads one 16-byte piece per pass and stores it: a wave writes runs of UX * 16 bytes
// (or several full columns).  LDS is [TQ columns][UX pieces] of 16 bytes, unpadded; piece u of column c sits at
// position u ^ (c / VEC mod 8): any eight neighbouring lanes -- the lanes one LDS cycle serves for a 128-bit
// access -- then hit eight different 16-byte bank groups, writing (same row unit, eight column units) and
// reading (same column, eight neighbouring pieces) alike, where a padded tile with scalar accesses ran at two
// lanes per bank (measured: conflict cycles half of the LDS-active cycles).
// Extents that are no multiple of VEC: the last unit along an axis slides back to end where the axis ends, so it moves
// some elements that the unit before it moves as well (the same bits to the same place), and rows start at any element;
// the memory pipeline takes 128-bit accesses at any element address.  [64,197,768] -> [64,768,197] bfloat16 (39 MB, cold)
// 8.5 us, 25.7 as 32x32 tiles of single elements; 4001 x 3333 float32 (107 MB) 26.3 against 41.1; extents of whole units
// as before (4096 x 4096 bfloat16 13.8 us).
// UNITS = 64, for matrices of at most 8 x 8 units: a tile per wavefront, four batch entries per workgroup.
template <typename T, int UQ, bool STREAM, int UNITS, bool TWO>
__device__ __forceinline__ void transpose_units(const T* __restrict__ in, T* __restrict__ out, const TransposeP& p) {
  constexpr uint32_t VEC = 16 / sizeof(T), UX = UNITS / UQ, TQ = UQ * VEC, TX = UX * VEC;
  typedef typename AtAlignment<u32x4, (int)sizeof(T)>::type Unaligned;
  __shared__ u32x4 tiles[256 / UNITS][TQ * UX];
  const uint32_t part = UNITS == 256 ? 0u : threadIdx.x / UNITS, tid = UNITS == 256 ? threadIdx.x : threadIdx.x % UNITS;
  u32x4* const tile = tiles[part];
  const uint32_t index = blockIdx.x * (256u / UNITS) + part;
  const bool there = UNITS == 256 || index < p.n_tiles;
  const TileAt<TWO> t(p, there ? index : 0u);
  const uint32_t uq = tid % UQ, ux = tid / UQ;
  if (there && t.bq * TQ + uq * VEC < p.nq && t.bx * TX + ux * VEC < p.nx) {
    const uint32_t cq = min(t.bq * TQ + uq * VEC, p.nq - VEC), cx = min(t.bx * TX + ux * VEC, p.nx - VEC);
    u32x4 row[VEC];
#pragma unroll
    for (uint32_t s = 0; s < VEC; ++s) {
      const Unaligned* const at = reinterpret_cast<const Unaligned*>(in + t.in_base + cq + (size_t)(cx + s) * p.in_row);
      row[s] = STREAM ? __builtin_nontemporal_load(at) : *at;
    }
    // transpose in registers: col[e] = elements e of rows 0..VEC-1
    u32x4 col[VEC];
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) col[e] = u32x4{row[0][e], row[1][e], row[2][e], row[3][e]};
    } else {
      // 2x2 blocks of 16-bit elements first: for rows (2m, 2m+1) and dword k, lo = [r0.lo16, r1.lo16] is column 2k,
      // hi = [r0.hi16, r1.hi16] column 2k+1, each holding rows 2m, 2m+1; the rest is a renaming
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        uint32_t lo[4], hi[4];
#pragma unroll
        for (uint32_t m = 0; m < 4; ++m) {
          lo[m] = __builtin_amdgcn_perm(row[2 * m + 1][k], row[2 * m][k], 0x05040100u);   // [r0.lo, r1.lo]
          hi[m] = __builtin_amdgcn_perm(row[2 * m + 1][k], row[2 * m][k], 0x07060302u);   // [r0.hi, r1.hi]
        }
        col[2 * k] = u32x4{lo[0], lo[1], lo[2], lo[3]};
        col[2 * k + 1] = u32x4{hi[0], hi[1], hi[2], hi[3]};
      }
    }
#pragma unroll
    for (uint32_t e = 0; e < VEC; ++e) tile[(uq * VEC + e) * UX + (ux ^ (uq & 7u))] = col[e];
  }
  __syncthreads();
  // store: piece u of column c -> 16 bytes of the column's output row
  const uint32_t u = tid % UX, c_first = tid / UX;
  const uint32_t x0 = t.bx * TX + u * VEC, cx = min(x0, p.nx - VEC);
#pragma unroll
  for (uint32_t s = 0; s < TQ / UQ; ++s) {
    const uint32_t c = c_first + s * UQ, unit = c / VEC, q0 = t.bq * TQ + unit * VEC;
    const u32x4 v = tile[c * UX + (u ^ (unit & 7u))];
    if (there && q0 < p.nq && x0 < p.nx)
      __builtin_nontemporal_store(v, reinterpret_cast<Unaligned*>(out + t.out_base + (size_t)(min(q0, p.nq - VEC) + c % VEC) * p.out_row + cx));
  }
}

// (what they say: units_params)
// Measured against a by-value block of 128 bytes (us, before / after): [64,197,768] -> [64,768,197] bf16 7.2 / 6.9, [8,64,792] ->
// [8,792,64] bf16 4.1 / 3.6, [59,220,8,64] -> [59,8,64,220] f16 5.1 / 4.8.
#define UNITS_PARAMS uint32_t m0, uint32_t m1, uint32_t word, uint32_t nq, uint32_t nx, uint32_t in_row, uint32_t in_batch, uint32_t n_tiles, \
                     uint32_t out_row, uint32_t out_batch
#define UNITS_ARGS m0, m1, word, nq, nx, in_row, in_batch, n_tiles, out_row, out_batch
template <typename T, int UQ, bool STREAM, int UNITS = 256>
__global__ void __launch_bounds__(256) k_transpose_units(const T* __restrict__ in, T* __restrict__ out, UNITS_PARAMS) {
  constexpr uint32_t VEC = 16 / sizeof(T);
  const TransposeP p = units_params(UQ * VEC, UNITS / UQ * VEC, UNITS_ARGS);
  transpose_units<T, UQ, STREAM, UNITS, false>(in, out, p);
}
// two axes outside the tile
template <typename T, int UQ, bool STREAM, int UNITS = 256>
__global__ void __launch_bounds__(256) k_transpose_units2(const T* __restrict__ in, T* __restrict__ out, UNITS_PARAMS, uint32_t d2, uint32_t m2,
                                                          uint32_t in_batch0, uint32_t out_batch0) {
  constexpr uint32_t VEC = 16 / sizeof(T);
  TransposeP p = units_params(UQ * VEC, UNITS / UQ * VEC, UNITS_ARGS);
  units_second_axis(&p, word, d2, m2, in_batch0, out_batch0);
  transpose_units<T, UQ, STREAM, UNITS, true>(in, out, p);
}

// ---- streaming copy (the measured HBM ceiling) ------------------------------------
__global__ void __launch_bounds__(256) k_copy(const u32x4* __restrict__ src, u32x4* __restrict__ dst, UnaryP p) {
  const uint32_t n_vec = p.n;   // 128-bit vectors
  uint32_t i = blockIdx.x * 1024u + threadIdx.x;
  u32x4 v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) if (i + k * 256u < n_vec) v[k] = __builtin_nontemporal_load(src + i + k * 256u);
#pragma unroll
  for (int k = 0; k < 4; ++k) if (i + k * 256u < n_vec) __builtin_nontemporal_store(v[k], dst + i + k * 256u);
}

}  // namespace fsk

// ---- host launchers ----------------------------------------------------------------
namespace fs {
using namespace fsk;

namespace {
template <typename T, bool STREAM>
const void* units_symbol(const TransposeP& p) {
  const bool two = transpose_two_batch_axes(p);
  if (p.tile_units == 64) return two ? (const void*)k_transpose_units2<T, 8, STREAM, 64> : (const void*)k_transpose_units<T, 8, STREAM, 64>;
  switch (p.tile_uq) {
    case 8: return two ? (const void*)k_transpose_units2<T, 8, STREAM> : (const void*)k_transpose_units<T, 8, STREAM>;
    case 32: return two ? (const void*)k_transpose_units2<T, 32, STREAM> : (const void*)k_transpose_units<T, 32, STREAM>;
    default: return two ? (const void*)k_transpose_units2<T, 16, STREAM> : (const void*)k_transpose_units<T, 16, STREAM>;
  }
}
}  // namespace

const void* unfused_kernel_symbol(int32_t kernel, const KernelArgs& a) {
  switch (kernel) {
    case K_UNARY:
      return a.u.unary.vec == 8 ? (const void*)k_unary<8> : a.u.unary.vec == 4 ? (const void*)k_unary<4> : (const void*)k_unary<1>;
    case K_BINARY:
      return a.u.binary.vec == 8 ? (const void*)k_binary<8> : a.u.binary.vec == 4 ? (const void*)k_binary<4> : (const void*)k_binary<1>;
    case K_REDUCE_ROW:
      return a.u.reduce.vec == 8 ? (const void*)k_reduce_row<8> : a.u.reduce.vec == 4 ? (const void*)k_reduce_row<4> : (const void*)k_reduce_row<1>;
    case K_REDUCE_MID:
      return a.u.reduce.vec == 8 ? (const void*)k_reduce_mid<8> : a.u.reduce.vec == 4 ? (const void*)k_reduce_mid<4> : (const void*)k_reduce_mid<1>;
    case K_TRANSPOSE_ROWS: {
      const int vb = a.u.transpose.vec * a.u.transpose.elem_bytes;
      return vb == 16 ? (const void*)k_transpose_rows<u32x4> : vb == 8 ? (const void*)k_transpose_rows<u32x2>
           : vb == 4 ? (const void*)k_transpose_rows<uint32_t> : (const void*)k_transpose_rows<uint16_t>;
    }
    case K_TRANSPOSE_TILE:
      if (a.u.transpose.vec > 1) {
        const bool wide = a.u.transpose.elem_bytes == 4;
        if (a.u.transpose.stream) return wide ? units_symbol<uint32_t, true>(a.u.transpose) : units_symbol<uint16_t, true>(a.u.transpose);
        return wide ? units_symbol<uint32_t, false>(a.u.transpose) : units_symbol<uint16_t, false>(a.u.transpose);
      }
      return a.u.transpose.elem_bytes == 4 ? (const void*)k_transpose_tile<uint32_t> : (const void*)k_transpose_tile<uint16_t>;
    case K_COPY:
      return (const void*)k_copy;
    default:
      return nullptr;
  }
}

}  // namespace fs
