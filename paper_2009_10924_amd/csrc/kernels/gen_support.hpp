// Support code of the generated row kernels (paper Section 4: the code generator takes a
// fusion pattern and produces one kernel).  A generated kernel is straight-line code over
// named per-lane values; what every such kernel shares -- the geometry of a row over a lane
// group or a workgroup, the 128-bit loads issued up front at clamped addresses, unpacking,
// the streaming store and the row reductions -- lives here, with every extent a template
// constant so that index arithmetic, padding tests and loops fold away at compile time.
// This header is embedded in the library as text and handed to the run-time compiler in
// front of the generated kernel; the library's own build also compiles it (a fixed sample
// kernel instantiates it) so that a mistake shows at build time.
#pragma once
#include "device_utils.hpp"

namespace fsk {

// Pointer block of a generated kernel, one by-value argument (slots as in K_ROW_PROGRAM).
struct GenArgs {
  const void* full[8];
  const void* col[8];
  const void* rscal[8];
  void* out[8];
  void* rout[8];
  void* ws;   // partial column sums, one row per workgroup (patterns with column sums), else null
};

// Compile-time switches handed to generic lambdas of a generated kernel (`if constexpr (decltype(tag)::value)`).
struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

// value of `v` in lane (own lane ^ mask) of the wavefront
__device__ __forceinline__ float xor_lane(float v, uint32_t mask) {
  const int addr = (int)(((threadIdx.x ^ mask) & 63u) << 2);
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr, __builtin_bit_cast(int, v)));
}

// value + the value 32 lanes further / in the other one of two neighbouring 16-lane rows: the swap instructions leave one
// half in both halves of the one register and the other half in the other.  (The elements are copied out first:
// bit-casting a vector element is miscompiled into a read of element 0, see unpack().)
__device__ __forceinline__ float add_other_half(float v) {
  const uint32_t b = __builtin_bit_cast(uint32_t, v);
  const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  const uint32_t one = r[0], other = r[1];
  return __builtin_bit_cast(float, one) + __builtin_bit_cast(float, other);
}
__device__ __forceinline__ float add_other_row(float v) {
  const uint32_t b = __builtin_bit_cast(uint32_t, v);
  const auto r = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  const uint32_t one = r[0], other = r[1];
  return __builtin_bit_cast(float, one) + __builtin_bit_cast(float, other);
}

// One step of one lane in storage form: VEC elements of 2 or 4 bytes are 2, 4, 8, 16 or 32 bytes.  VEC is 8 or 4, and
// 1 for rows shorter than 4 elements.  EA: the alignment the address is known to have, in bytes -- that of a whole step, 16
// at most, where the row length is a multiple of VEC elements, that of one element otherwise (a row then starts anywhere).  The
// memory pipeline takes 64- and 128-bit accesses at any element address: a copy of 64 MB each way through 128-bit
// accesses that all start 2 bytes off runs at 5.18 TB/s, 4 or 8 bytes off at 5.53, aligned at 5.75, and element by
// element at 4.97 with eight times the instructions and one register per element.
template <int BYTES, int EA> struct StepBits;
template <int EA> struct StepBits<32, EA> {
  static_assert(EA <= 16, "callers' pointers are aligned to 16 bytes, and the second half starts 16 behind the first");
  u32x4 lo, hi;
  template <bool STREAM, typename T>
  __device__ __forceinline__ static StepBits load(const T* p) {
    StepBits r;
    const typename AtAlignment<u32x4, EA>::type* q = reinterpret_cast<const typename AtAlignment<u32x4, EA>::type*>(p);
    r.lo = STREAM ? __builtin_nontemporal_load(q) : q[0];
    r.hi = STREAM ? __builtin_nontemporal_load(q + 1) : q[1];
    return r;
  }
};
template <typename V, int EA> struct OneAccess {
  template <bool STREAM, typename T>
  __device__ __forceinline__ static V get(const T* p) {
    const typename AtAlignment<V, EA>::type* q = reinterpret_cast<const typename AtAlignment<V, EA>::type*>(p);
    return STREAM ? __builtin_nontemporal_load(q) : *q;
  }
};
#define FSK_STEP_BITS(BYTES, V)                                        \
  template <int EA> struct StepBits<BYTES, EA> {                       \
    V w;                                                               \
    template <bool STREAM, typename T>                                 \
    __device__ __forceinline__ static StepBits load(const T* p) {      \
      StepBits r;                                                      \
      r.w = OneAccess<V, EA>::template get<STREAM>(p);                 \
      return r;                                                        \
    }                                                                  \
  };
FSK_STEP_BITS(16, u32x4)
FSK_STEP_BITS(8, u32x2)
FSK_STEP_BITS(4, uint32_t)
FSK_STEP_BITS(2, uint16_t)
#undef FSK_STEP_BITS

// Registers that hold a step in storage form across several passes: after this the compiler no longer knows what is
// in them, so it cannot carry the unpacked float32 form (twice the registers of a 16-bit step) from one pass to the
// next instead.  No instruction is emitted.
template <int EA>
__device__ __forceinline__ void forget_contents(StepBits<32, EA>& s) { asm volatile("" : "+v"(s.lo), "+v"(s.hi)); }
template <int EA>
__device__ __forceinline__ void forget_contents(StepBits<16, EA>& s) { asm volatile("" : "+v"(s.w)); }
template <int EA>
__device__ __forceinline__ void forget_contents(StepBits<8, EA>& s) { asm volatile("" : "+v"(s.w)); }
template <int EA>
__device__ __forceinline__ void forget_contents(StepBits<4, EA>& s) { asm volatile("" : "+v"(s.w)); }
template <int EA>
__device__ __forceinline__ void forget_contents(StepBits<2, EA>& s) {
  uint32_t t = s.w;
  asm volatile("" : "+v"(t));
  s.w = (uint16_t)t;
}

template <int EA>
__device__ __forceinline__ void unpack_step(const StepBits<32, EA>& r, float (&v)[8], const float*) {
  float a[4], b[4];
  unpack(r.lo, a, (const float*)nullptr);
  unpack(r.hi, b, (const float*)nullptr);
#pragma unroll
  for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
}
template <int EA>
__device__ __forceinline__ void unpack_step(const StepBits<16, EA>& r, float (&v)[4], const float*) { unpack(r.w, v, (const float*)nullptr); }
template <int EA, typename T>
__device__ __forceinline__ void unpack_step(const StepBits<16, EA>& r, float (&v)[8], const T*) { unpack(r.w, v, (const T*)nullptr); }
template <int EA>
__device__ __forceinline__ void unpack_step(const StepBits<8, EA>& r, float (&v)[4], const bf16_t*) {
  v[0] = __builtin_bit_cast(float, r.w.x << 16); v[1] = __builtin_bit_cast(float, r.w.x & 0xFFFF0000u);
  v[2] = __builtin_bit_cast(float, r.w.y << 16); v[3] = __builtin_bit_cast(float, r.w.y & 0xFFFF0000u);
}
template <int EA>
__device__ __forceinline__ void unpack_step(const StepBits<8, EA>& r, float (&v)[4], const f16_t*) {
  unpack_f16(r.w.x, v[0], v[1]);
  unpack_f16(r.w.y, v[2], v[3]);
}
template <int EA>
__device__ __forceinline__ void unpack_step(const StepBits<4, EA>& r, float (&v)[1], const float*) { v[0] = __builtin_bit_cast(float, r.w); }
template <int EA>
__device__ __forceinline__ void unpack_step(const StepBits<2, EA>& r, float (&v)[1], const bf16_t*) { v[0] = bf16_bits_to_f32(r.w); }
template <int EA>
__device__ __forceinline__ void unpack_step(const StepBits<2, EA>& r, float (&v)[1], const f16_t*) {
  v[0] = (float)__builtin_bit_cast(_Float16, r.w);
}

// Stores N float32 values as TO at an address known to be aligned to EA bytes, past the caches (see StoreN).
template <typename TO, int N, int EA>
__device__ __forceinline__ void store_elements(TO* p, const float (&v)[N]) {
  if constexpr (EA >= 16 || EA >= (int)sizeof(TO) * N || N == 1) {
    StoreN<TO, N>::run(p, v);
  } else if constexpr (sizeof(TO) == 4) {
    if constexpr (N == 2) {
      const u32x2 w = {__builtin_bit_cast(uint32_t, v[0]), __builtin_bit_cast(uint32_t, v[1])};
      __builtin_nontemporal_store(w, reinterpret_cast<typename AtAlignment<u32x2, EA>::type*>(p));
    } else {
#pragma unroll
      for (int e = 0; e < N; e += 4) {
        const f32x4 w = {v[e], v[e + 1], v[e + 2], v[e + 3]};
        __builtin_nontemporal_store(w, reinterpret_cast<typename AtAlignment<f32x4, EA>::type*>(p + e));
      }
    }
  } else {
    uint32_t w[N / 2];
#pragma unroll
    for (int e = 0; e < N; e += 2) w[e / 2] = pack2(v[e], v[e + 1], (const TO*)nullptr);
    if constexpr (N == 8) __builtin_nontemporal_store(u32x4{w[0], w[1], w[2], w[3]}, reinterpret_cast<typename AtAlignment<u32x4, EA>::type*>(p));
    else if constexpr (N == 4) __builtin_nontemporal_store(u32x2{w[0], w[1]}, reinterpret_cast<typename AtAlignment<u32x2, EA>::type*>(p));
    else __builtin_nontemporal_store(w[0], reinterpret_cast<typename AtAlignment<uint32_t, EA>::type*>(p));
  }
}

// ROWS x COLS row space; VEC elements per lane and step; K steps per lane; L lanes per row: a lane group of one
// wavefront in a 256-thread workgroup, or, when BLOCK, the whole workgroup of L = 256, 512 or 1024 threads.
// R: rows each lane group works through, one after the other (the kernel body runs R times with virtual
// workgroup indices it * (workgroups over the rows, a constant) + its own, so that at any moment the resident workgroups sweep one band of rows).
// ROW_STRIDE > COLS: the pattern's rows are ROW_STRIDE elements long and the kernel works on column tiles of COLS
// elements (patterns without row reductions only: nothing ties the tiles of a row together); `tile` picks the tile.
// TILES: their number, where the last one may be shorter than the others (1: all of COLS elements).
// PAST_CACHES: operands that are read once carry the streaming hint (inputs too large for the caches, see streams_inputs()).
//
// Row lengths that are no multiple of VEC: the row's last step slides back so that it ends where the row ends, and
// reads some elements that the step before it holds as well (BACK of them).  Every load is then one whole access
// inside the row.  The repeated elements count once: reductions and column sums leave them out of the last step.  Its
// store either writes only the TAIL elements the step owns, in at most three pieces, or (AGAIN) the whole step, the
// repeated elements a second time with the value their owner gives them: one access instead of three more (rows of 197
// 16-bit elements, 29.8 MB: 7.6 against 8.9 us for the bare copy, 7.0 with rows padded to whole steps).
//
// EDGES != 0 (such rows again, stored AGAIN): the steps lie on the multiples of VEC elements of the whole tensor instead of
// the row's, so every access but a row's first and last is aligned; these two slide inwards, the first to where the row starts,
// the last to where it ends, and the elements that a neighbour holds too count once.  What a row then takes is at most one
// step more.  EDGE_FIRST / EDGE_LAST: the object may hold the row's first / last step (a chunk between them neither).
constexpr int EDGE_FIRST = 1, EDGE_LAST = 2, EDGE_INNER = 4;
template <uint32_t ROWS, uint32_t COLS, int VEC, int K, uint32_t L, bool BLOCK, uint32_t R = 1, uint32_t ROW_STRIDE = COLS, uint32_t TILES = 1,
          bool PAST_CACHES = false, int EDGES = 0>
struct GenRow {
  static constexpr bool ON_GRID = EDGES != 0;   // of the tensor's steps
  static constexpr bool SHORT_LAST = TILES > 1 && TILES * COLS != ROW_STRIDE;
  static constexpr uint32_t LAST_COLS = SHORT_LAST ? ROW_STRIDE - (TILES - 1u) * COLS : COLS;
  static constexpr uint32_t NVEC = (COLS + VEC - 1) / VEC, LAST_NVEC = (LAST_COLS + VEC - 1) / VEC;
  static constexpr int TAIL = (int)(LAST_COLS % VEC), BACK = TAIL != 0 ? VEC - TAIL : 0;
  static_assert(!SHORT_LAST || COLS % VEC == 0, "only the last tile ends inside a step");
  static constexpr uint32_t LANES = L;
  static constexpr uint32_t ROWS_PER_WG = BLOCK ? 1u : 256u / L;
  // the row fills its lanes (and no element is held twice) / the rows fill the workgroups: no clamp, no padding test
  static constexpr bool FULL_COLS = !ON_GRID && NVEC == LANES * K && TAIL == 0 && !SHORT_LAST;
  static constexpr bool FULL_ROWS = ROWS % (ROWS_PER_WG * R) == 0;
  static constexpr int KV = K * VEC;
  static constexpr uint32_t PADDED_COLS = LANES * K * VEC;   // columns the lanes of a row cover, padding included
  static_assert(TAIL == 0 || ROW_STRIDE >= (uint32_t)VEC, "a row holds at least one step");
  template <typename T> static constexpr int alignment() {
    constexpr int step = (int)sizeof(T) * (ROW_STRIDE % VEC == 0 ? VEC : 1);
    return step < 16 ? step : 16;
  }

  uint32_t lane, row, row_c, col0;
  bool row_ok, last;   // last: the tile that may be shorter than the others
  int lead;            // ON_GRID: elements between the start of the row's first step and the row's own start

  __device__ __forceinline__ explicit GenRow(uint32_t vblock, uint32_t tile = 0) {
    const uint32_t tid = threadIdx.x;
    col0 = tile * COLS;
    last = tile == TILES - 1u;
    lane = BLOCK ? tid : (tid & (L - 1u));
    row = BLOCK ? vblock : vblock * ROWS_PER_WG + tid / L;
    row_ok = FULL_ROWS || row < ROWS;
    row_c = FULL_ROWS ? row : min(row, ROWS - 1u);
    lead = ON_GRID ? (int)((row_c * (ROW_STRIDE % VEC)) % VEC) : 0;
  }
  // a chunk of a long row: COLS columns from column `first_col` on (the row itself is ROW_STRIDE elements long)
  __device__ __forceinline__ GenRow(uint32_t vblock, uint32_t tile, uint32_t first_col) : GenRow(vblock, tile) { col0 = first_col; }
  // only a lane's last step can be padding or the row's last one (K is the smallest that covers the row)
  static constexpr __device__ __forceinline__ bool inner(int k) {
    if constexpr (ON_GRID) return before_last(k) && behind_first(k);
    return FULL_COLS || (!SHORT_LAST && (uint32_t)k < (NVEC - 1u) / LANES);
  }
  // ON_GRID: no lane's step k can be the row's last one (or padding) / its first one
  static constexpr __device__ __forceinline__ bool before_last(int k) { return (EDGES & EDGE_LAST) == 0 || ((uint32_t)k + 1u) * LANES * VEC <= COLS; }
  static constexpr __device__ __forceinline__ bool behind_first(int k) { return (EDGES & EDGE_FIRST) == 0 || k > 0; }
  // ON_GRID: the row's column at which step k lies on the grid (the first one's may be negative), and where it is read and written
  __device__ __forceinline__ int grid_col(int k) const { return (int)col0 + (int)(lane + k * LANES) * VEC - lead; }
  __device__ __forceinline__ int edge_col(int k) const {
    int c = grid_col(k);
    if (!behind_first(k)) c = max(c, 0);
    if (!before_last(k)) c = min(c, (int)ROW_STRIDE - VEC);
    return c;
  }
  // steps and columns of the row (of this tile of it), and the steps that hold no repeated element
  __device__ __forceinline__ uint32_t n_steps() const { return SHORT_LAST && last ? LAST_NVEC : NVEC; }
  __device__ __forceinline__ uint32_t n_cols() const { return SHORT_LAST && last ? LAST_COLS : COLS; }
  __device__ __forceinline__ uint32_t n_whole() const { return SHORT_LAST && !last ? NVEC : LAST_NVEC - (TAIL != 0 ? 1u : 0u); }
  __device__ __forceinline__ bool valid(int k) const {
    if constexpr (ON_GRID) return before_last(k) || grid_col(k) < (int)ROW_STRIDE;
    return inner(k) || lane + k * LANES < n_steps();
  }
  // element e of step k is the lane's own: neither padding nor a repetition of the step before
  __device__ __forceinline__ bool own(int k, int e) const {
    if constexpr (ON_GRID) {   // a step that slid by n elements: its first n (slid back) or its last -n (slid forward) are a neighbour's
      const int n = grid_col(k) - edge_col(k);
      return (before_last(k) || e >= n) && (behind_first(k) || e < VEC + n);
    }
    return inner(k) || lane + k * LANES < (e < BACK ? n_whole() : n_steps());
  }
  // first column of step k (the last step's slides back; padding steps stay on the last step).  Signed: the last chunk
  // of a long row may be shorter than a step, which then starts in the chunk before.
  __device__ __forceinline__ int first_of(int k) const {
    if constexpr (ON_GRID) return edge_col(k) - (int)col0;
    if (inner(k)) return (int)(lane + k * LANES) * VEC;
    if constexpr (TAIL != 0) return min((int)(lane + k * LANES) * VEC, (int)n_cols() - VEC);
    return (int)min(lane + k * LANES, n_steps() - 1u) * VEC;
  }

  // the lane's K steps of row `at_row` of a [.., COLS] tensor, in storage form; STREAM: read once, so the loads may
  // carry the streaming hint and then do not displace the operands that every row re-reads from cache
  template <typename T> using Step = StepBits<VEC * (int)sizeof(T), alignment<T>()>;
  template <typename T>
  struct Raw {
    Step<T> w[K];
    // (a lane's own places in LDS: nobody else reads or writes them)
    __device__ __forceinline__ void park(Step<T> (&lds)[K][L]) const {
#pragma unroll
      for (int k = 0; k < K; ++k) lds[k][threadIdx.x] = w[k];
    }
    __device__ __forceinline__ void fetch(const Step<T> (&lds)[K][L]) {
#pragma unroll
      for (int k = 0; k < K; ++k) w[k] = lds[k][threadIdx.x];
    }
    __device__ __forceinline__ void forget_contents() {
#pragma unroll
      for (int k = 0; k < K; ++k) fsk::forget_contents(w[k]);
    }
  };
  template <typename T, bool STREAM>
  __device__ __forceinline__ Raw<T> load(const void* p, size_t at_row) const {
    Raw<T> r;
    const T* base = static_cast<const T*>(p) + at_row * ROW_STRIDE + col0;
#pragma unroll
    for (int k = 0; k < K; ++k) r.w[k] = Step<T>::template load<STREAM && PAST_CACHES>(base + first_of(k));
    return r;
  }

  template <typename T>
  __device__ __forceinline__ void unpack_to(const Raw<T>& r, float (&v)[KV]) const {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float part[VEC];
      unpack_step(r.w[k], part, (const T*)nullptr);
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[k * VEC + e] = part[e];
    }
  }

  template <typename TO, bool AGAIN = false>
  __device__ __forceinline__ void store(void* p, const float (&v)[KV]) const { store_at<TO, AGAIN>(p, (size_t)row, v); }

  // N of the last step's own elements, from its element FROM on
  template <typename TO, int FROM, int N>
  __device__ __forceinline__ static void store_piece(TO* step, const float (&part)[VEC]) {
    float w[N];
#pragma unroll
    for (int e = 0; e < N; ++e) w[e] = part[FROM + e];
    store_elements<TO, N, (int)sizeof(TO)>(step + FROM, w);
  }
  // the row's values to row `at_row` of the output (its own row, or the place a folded transpose gives it)
  template <typename TO, bool AGAIN = false>
  __device__ __forceinline__ void store_at(void* p, size_t at_row, const float (&v)[KV]) const {
    TO* base = static_cast<TO*>(p) + at_row * ROW_STRIDE + col0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float part[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) part[e] = v[k * VEC + e];
      static_assert(!ON_GRID || AGAIN, "a step that slid is written whole");
      if constexpr (TAIL == 0 && !ON_GRID) {
        if (row_ok && valid(k)) store_elements<TO, VEC, alignment<TO>()>(base + (size_t)(lane + k * LANES) * VEC, part);
      } else if constexpr (AGAIN) {
        if (row_ok && valid(k)) store_elements<TO, VEC, alignment<TO>()>(base + first_of(k), part);
      } else {
        if (row_ok && own(k, 0)) store_elements<TO, VEC, alignment<TO>()>(base + (size_t)(lane + k * LANES) * VEC, part);
        if (!inner(k) && row_ok && (!SHORT_LAST || last) && lane + k * LANES == LAST_NVEC - 1u) {
          TO* const step = base + ((int)LAST_COLS - VEC);
          if constexpr (TAIL >= 4) store_piece<TO, BACK, 4>(step, part);
          if constexpr ((TAIL & 2) != 0) store_piece<TO, BACK + (TAIL & 4), 2>(step, part);
          if constexpr ((TAIL & 1) != 0) store_piece<TO, VEC - 1, 1>(step, part);
        }
      }
    }
  }

  template <typename TO>
  __device__ __forceinline__ void store_scalar(void* p, float v) const {
    if (row_ok && lane == 0) store1(static_cast<TO*>(p) + row, v);
  }

  // all-reduce over the row: every lane of the row ends with the same value.  SQUARE: of the squared
  // elements.  slot: one float per wavefront of the workgroup, LDS private to this reduction (BLOCK only).
  template <typename OP, bool IS_MAX, bool SQUARE>
  __device__ __forceinline__ float reduce(const float (&v)[KV], float* slot) const {
    return finish<OP>(partial<OP, IS_MAX, SQUARE>(v), slot);
  }
  // the two halves of reduce(): the lane's own elements folded to one value (rows worked through in chunks fold
  // their chunks' values lane by lane first), and the all-reduce of the lanes' values over the row
  template <typename OP, bool IS_MAX, bool SQUARE>
  __device__ __forceinline__ float partial(const float (&v)[KV]) const {
    // the lane's own elements are combined pairwise (a tree, not a chain): log2(KV) dependent steps instead of
    // KV, and a float32 sum whose rounding error grows with the depth of the tree
    float t[KV];
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float x = SQUARE ? v[k * VEC + e] * v[k * VEC + e] : v[k * VEC + e];
        t[k * VEC + e] = own(k, e) ? x : (IS_MAX ? -__builtin_huge_valf() : 0.0f);
      }
    }
#pragma unroll
    for (int n = KV; n > 1; n = (n + 1) / 2) {
#pragma unroll
      for (int i = 0; i < n / 2; ++i) t[i] = OP::apply(t[2 * i], t[2 * i + 1]);
      if (n & 1) t[n / 2] = t[n - 1];
    }
    return t[0];
  }
  template <typename OP>
  __device__ __forceinline__ static float finish(float r, float* slot) {
    if constexpr (BLOCK) return block_allreduce<OP>(r, slot, (int)(L / 64u));
    else return group_allreduce<OP>(r, (int)L);
  }

  // ---- column sums over all rows (lane-group rows only) ----------------------------------------------------
  // the row's values join the lane's running sums; padding lanes, repeated elements and rows beyond the last add nothing
  __device__ __forceinline__ void colsum_add(const float (&v)[KV], float (&sum)[KV]) const {
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) sum[k * VEC + e] += row_ok && own(k, e) ? v[k * VEC + e] : 0.0f;
    }
  }
  // Lane-group rows: the workgroup's lane groups hold sums of the same columns: first the groups of a wavefront are folded
  // lane to lane (every lane of the first group ends with the wavefront's sum), then the four wavefronts through `lds`
  // (4 * PADDED_COLS floats, used by this sum only), and one row of COLS partial sums goes to `dst`.  Fixed order
  // throughout, so the result is the same from run to run.  In LDS a wavefront's sums lie step after step, so a lane
  // writes 128-bit vectors (single floats, VEC apart from lane to lane, meet in the same banks).  colsum_park and
  // colsum_flush have a barrier between them, one for all the sums of a pattern.
  __device__ __forceinline__ void colsum_park(const float (&sum)[KV], float* lds) const {
    if constexpr (BLOCK) return;
    float v[KV];
#pragma unroll
    for (int j = 0; j < KV; ++j) v[j] = sum[j];
    if constexpr (L <= 1u) {
#pragma unroll
      for (int j = 0; j < KV; ++j) v[j] += xor_lane(v[j], 1u);
    }
    if constexpr (L <= 2u) {
#pragma unroll
      for (int j = 0; j < KV; ++j) v[j] += xor_lane(v[j], 2u);
    }
    if constexpr (L <= 4u) {
#pragma unroll
      for (int j = 0; j < KV; ++j) v[j] += xor_lane(v[j], 4u);
    }
    if constexpr (L <= 8u) {   // row_ror:8 : the other half of the 16 lanes
#pragma unroll
      for (int j = 0; j < KV; ++j) v[j] += dpp_move<0x128>(v[j]);
    }
    if constexpr (L <= 16u) {
#pragma unroll
      for (int j = 0; j < KV; ++j) v[j] = add_other_row(v[j]);
    }
    if constexpr (L <= 32u) {
#pragma unroll
      for (int j = 0; j < KV; ++j) v[j] = add_other_half(v[j]);
    }
    const uint32_t tid = threadIdx.x;
    if ((tid & 63u) < L) {
      float* mine = lds + (tid >> 6) * PADDED_COLS + lane * VEC;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if constexpr (VEC >= 4) {
#pragma unroll
          for (int e = 0; e < VEC; e += 4)
            *reinterpret_cast<f32x4*>(mine + k * L * VEC + e) = f32x4{v[k * VEC + e], v[k * VEC + e + 1], v[k * VEC + e + 2], v[k * VEC + e + 3]};
        } else {
          mine[k * L] = v[k];
        }
      }
    }
  }
  // The same where the workgroup has seen all rows: its sums are final, in their own dtype.
  template <typename TO>
  __device__ __forceinline__ void colsum_finish(const float* lds, void* out) const {
    static_assert(!BLOCK, "");
    for (uint32_t c = threadIdx.x; c < n_cols(); c += 256u) {
      const uint32_t at = c < n_whole() * VEC ? c : c + BACK;
      store1(static_cast<TO*>(out) + col0 + c, ((lds[at] + lds[PADDED_COLS + at]) + lds[2u * PADDED_COLS + at]) + lds[3u * PADDED_COLS + at]);
    }
  }
  __device__ __forceinline__ void colsum_flush(const float (&sum)[KV], const float* lds, float* dst) const {
    if constexpr (BLOCK) {
      // a workgroup per row: every lane owns its columns alone, the sums over the workgroup's rows are complete
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int at = first_of(k);
        if (own(k, 0)) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) dst[at + e] = sum[k * VEC + e];
        } else if (TAIL != 0 && own(k, VEC - 1)) {
#pragma unroll
          for (int e = BACK; e < VEC; ++e) dst[at + e] = sum[k * VEC + e];
        }
      }
      return;
    }
    // where column c lies in LDS: the last step's own columns are the last ones of its vector
    const auto fold4 = [&](uint32_t at) {
      return ((lds[at] + lds[PADDED_COLS + at]) + lds[2u * PADDED_COLS + at]) + lds[3u * PADDED_COLS + at];
    };
    if constexpr (TAIL == 0 && VEC >= 4) {
      for (uint32_t c = threadIdx.x * 4u; c < n_cols(); c += 1024u) {
        const f32x4* at = reinterpret_cast<const f32x4*>(lds + c);
        const f32x4 s = ((at[0] + at[PADDED_COLS / 4u]) + at[PADDED_COLS / 2u]) + at[PADDED_COLS / 4u * 3u];
        *reinterpret_cast<f32x4*>(dst + c) = s;
      }
    } else {
      for (uint32_t c = threadIdx.x; c < n_cols(); c += 256u) dst[c] = fold4(c < n_whole() * VEC ? c : c + BACK);
    }
  }
};

// A mid-pattern `convert`: the float32 value rounded to the storage dtype (nearest even) and widened again.  The value
// is pinned in a register first (an empty asm the compiler cannot see through): otherwise the compiler may fuse the
// multiplication that produced it with the conversion into one mixed-precision instruction (v_fma_mixlo_f16), which
// rounds the exact product once -- while another use of the same value (the store) rounds the float32 product.  The
// two differ by one 16-bit ulp where the float32 product is a tie, and a column sum of the rounded values would no
// longer be the sum of what is stored.
template <int DT> __device__ __forceinline__ float gen_round(float v) { return v; }
template <> __device__ __forceinline__ float gen_round<1>(float v) {
  asm volatile("" : "+v"(v));
  return (float)(_Float16)v;
}
template <> __device__ __forceinline__ float gen_round<2>(float v) {
  asm volatile("" : "+v"(v));
  return bf16_bits_to_f32(pack_bf16(v, 0.0f) & 0xFFFFu);
}

}  // namespace fsk
