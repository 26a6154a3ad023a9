// Neighbour aggregation on the partition graph (the AGG of the layer definition in Section 3)
// and its transpose for backward (the per-edge factor 1/D(v_j[i]) in the proof of Theorem 3).
//
// The edge weights of both the mean and the GCN normalisation factor into a per-source and a
// per-destination vector, so the kernels walk a pattern-only CSR:
//     Y[v] = out_scale[v] * ( self * in_scale[v] * X[v] + sum_{u in N(v)} in_scale[u] * X[u] )
// Because the (masked) partition graph is symmetric, the transposed product is the same pull
// with the roles of the two scale vectors exchanged - no atomics, fixed summation order.
// Rows are stored as float32 or bfloat16; sums are always float32.
//
// Three kernels.  Every graph carries its rows sorted by descending degree:
//  * aggregate_kernel: rows by teams of lanes - long rows a workgroup each, middling ones a wavefront each, short ones
//    a group of 16 to 64 lanes - in one launch, longest rows first.
//  * aggregate_hub_kernel (hub rows, AGG_HUB_MIN neighbours and more - the nodes that keep a high degree after
//    the cut, Theorem 2): a workgroup of sixteen wavefronts per (row, column panel); every wavefront sums a
//    strided share of the neighbours, the sixteen partial rows are staged in LDS and added in wavefront order.
//    A launch of its own over the head of the order, when the graph has such rows.
//  * aggregate_sliced_kernel (high average degree): a team of lanes per row or per (row, column slice), slices bound to XCDs.
// Which wavefront sums which neighbours is fixed by the launch shape, so results are run-to-run identical.
#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "common.h"

namespace cofree {

// ---- typed row access: VEC consecutive elements <-> float registers ---------------------------
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));

template <typename T>
struct RowIO;

// Raw / load_raw / keep_if / fma_raw: the gather loops load a batch of neighbour segments unconditionally -
// a slot without a neighbour re-reads the batch's first neighbour and is zeroed by keep_if, a lane past the
// end of the row re-reads the row's last window - and only then add them up.  A load under a per-lane
// condition is a branch to the compiler, which then waited for each load before issuing the next one
// (bfloat16 launches of 128-byte rows took twice as long as float32 launches of the same bytes).
template <>
struct RowIO<float> {
  static constexpr int WIDE = 4;  // elements per 16-byte access
  typedef f32x4u Raw;
  __device__ static Raw zero_raw() { return Raw{0.f, 0.f, 0.f, 0.f}; }
  __device__ static Raw load_raw(const float* p) { return *reinterpret_cast<const f32x4u*>(p); }
  __device__ static Raw keep_if(bool ok, const Raw& r) { return Raw{ok ? r[0] : 0.f, ok ? r[1] : 0.f, ok ? r[2] : 0.f, ok ? r[3] : 0.f}; }
  __device__ static void fma_raw(float (&acc)[4], float s, const Raw& r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = fmaf(s, r[i], acc[i]);
  }
  __device__ static void unpack(const Raw& r, float (&v)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = r[i];
  }
  __device__ static void load_wide(const float* p, float (&v)[4]) {
    const f32x4u t = *reinterpret_cast<const f32x4u*>(p);
    v[0] = t[0];
    v[1] = t[1];
    v[2] = t[2];
    v[3] = t[3];
  }
  __device__ static void store_wide(float* p, const float (&v)[4], bool stream = false) {
    f32x4u t;
    t[0] = v[0];
    t[1] = v[1];
    t[2] = v[2];
    t[3] = v[3];
    COFREE_STORE_PIECE(reinterpret_cast<f32x4u*>(p), t, stream);
  }
  __device__ static float load1(const float* p) { return *p; }
  __device__ static void store1(float* p, float x) { *p = x; }
};

template <>
struct RowIO<bf16_t> {
  static constexpr int WIDE = 8;
  typedef u32x4u Raw;
  __device__ static Raw zero_raw() { return Raw{0u, 0u, 0u, 0u}; }
  __device__ static Raw load_raw(const bf16_t* p) { return *reinterpret_cast<const u32x4u*>(p); }
  __device__ static Raw keep_if(bool ok, const Raw& r) { return Raw{ok ? r[0] : 0u, ok ? r[1] : 0u, ok ? r[2] : 0u, ok ? r[3] : 0u}; }
  __device__ static void fma_raw(float (&acc)[8], float s, const Raw& r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[2 * i] = fmaf(s, __uint_as_float(r[i] << 16), acc[2 * i]);
      acc[2 * i + 1] = fmaf(s, __uint_as_float(r[i] & 0xffff0000u), acc[2 * i + 1]);
    }
  }
  __device__ static void unpack(const Raw& r, float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(r[i] << 16);
      v[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u);
    }
  }
  __device__ static void load_wide(const bf16_t* p, float (&v)[8]) {
    const u32x4u t = *reinterpret_cast<const u32x4u*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(t[i] << 16);
      v[2 * i + 1] = __uint_as_float(t[i] & 0xffff0000u);
    }
  }
  __device__ static void store_wide(bf16_t* p, const float (&v)[8], bool stream = false) {
    u32x4u t;
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    COFREE_STORE_PIECE(reinterpret_cast<u32x4u*>(p), t, stream);
  }
  __device__ static float load1(const bf16_t* p) { return bf16_to_f32(*p); }
  __device__ static void store1(bf16_t* p, float x) { *p = f32_to_bf16(x); }
};

// VEC elements starting at p, of which only the first `avail` exist (avail >= VEC: one wide access)
template <typename T, int VEC>
__device__ inline void load_elems(const T* p, int avail, float (&v)[VEC]) {
  if (avail >= VEC) {
    RowIO<T>::load_wide(p, v);
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = i < avail ? RowIO<T>::load1(p + i) : 0.f;
  }
}
template <typename T, int VEC>
__device__ inline void store_elems(T* p, int avail, const float (&v)[VEC]) {
  if (avail >= VEC) {
    RowIO<T>::store_wide(p, v);
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i)
      if (i < avail) RowIO<T>::store1(p + i, v[i]);
  }
}

template <typename T>
struct AggK {
  const int64_t* rowptr;
  const int32_t* col;
  const T* X;
  uint32_t ldx;
  T* Y;
  uint32_t ldy;
  int width;  // columns of this launch
  int64_t n;
  const int32_t* order;  // the i-th team works on row order[slot0 + i] (null: row i)
  int32_t n_block, n_wave;  // row kernel: the first n_block rows get a workgroup each, the next n_wave a wavefront each
  int32_t slot0;      // first entry of `order` this launch covers (its bucket); n counts the entries from there
  // row kernel on the processing-order copy of the graph: rowptr, col and in_vals are that copy's, indexed by
  // slot, and the row's own factors come per slot too (null: none, or read by row id from in_scale / out_scale)
  int by_slot;
  const float* in_scale_slot;
  const float* out_scale_slot;
  const float* in_scale;  // per node
  const float* in_vals;   // the same factor per adjacency entry (in_vals[e] = in_scale[col[e]]), or null
  const float* out_scale;
  int self_loop;
  const T* relu_src;  // the row's other operand: gates the result, or is added to it (add_src)
  uint32_t ld_relu;
  int add_src;
  float gate_scale;  // factor on the elements that pass relu_src
  // output epilogue (after out_scale): + bias, ReLU
  const float* bias;
  int relu_out;
  int col0;  // first column of this launch in the full matrix (bias index)
  int stream_out;  // the result goes past the caches
  DropoutK drop;  // after everything else (DROP instances; ldy is the width of the full matrix there)
};

// Row numbers and strides have 32 bits, so that the offset of a row is one multiplication.
template <typename T>
__device__ inline T* row_at(T* base, uint32_t row, uint32_t ld) {
  return base + (uint64_t)row * ld;
}

// A lane owns VEC consecutive columns starting at a multiple of VEC.  When the last lane's columns
// would cross the end of a row of at least VEC columns, its window is moved left to end with the row,
// so that every access stays one wide access; the leading columns of the window are then also those of the lane before
// it, and both lanes store the same sums (left out, they cost a store for each of the last lane's own
// columns: 1.88M rows of 47 bfloat16 381 -> 363 us).  In rows of at least VEC columns a lane therefore has either a
// full window or none (avail <= 0).  Only rows narrower than VEC (the TINY kernel instances) use
// element accesses.
struct LaneCols {
  int c0;     // first column of the window
  int avail;  // columns of the window that exist (>= VEC unless the whole row is narrower than VEC)
};
template <int VEC>
__device__ inline LaneCols lane_cols(int width, int start) {
  LaneCols l;
  l.c0 = start;
  l.avail = width - start;
  if (l.avail > 0 && l.avail < VEC && width >= VEC) {
    l.c0 = width - VEC;
    l.avail = VEC;
  }
  return l;
}

// Shared tail of the kernels: self term, destination scale, gate or added row, bias, ReLU, store.
// The operands of the tail that depend on the row alone - its own X row, its gate row, its two scales -
// are requested together as soon as the row is known (RowTail::request, all loads back to back, nothing
// uses them yet) and applied after the neighbour sum: fetched one after the other at the end, each with
// its own wait, they added up to three memory round trips to the life of every lane group.
template <typename T, int VEC, bool TINY>
struct RowTail {
  typename RowIO<T>::Raw xs, g;
  float ss, so;
  // cread: first column of the lane's read window (valid memory also for lanes that own nothing); s: the row's
  // slot (used by the launches on the processing-order copy)
  __device__ void request(const AggK<T>& p, uint32_t row, uint32_t s, int cread) {
    ss = 1.f;
    so = 1.f;
    xs = RowIO<T>::zero_raw();
    g = RowIO<T>::zero_raw();
    if constexpr (!TINY) {
      if (p.out_scale_slot) so = p.out_scale_slot[s];
      else if (p.out_scale) so = p.out_scale[row];
      if (p.self_loop) {
        if (p.in_scale_slot) ss = p.in_scale_slot[s];
        else if (p.in_scale) ss = p.in_scale[row];
        xs = RowIO<T>::load_raw(row_at(p.X, row, p.ldx) + cread);
      }
      if (p.relu_src) g = RowIO<T>::load_raw(row_at(p.relu_src, row, p.ld_relu) + cread);
    }
  }
};

// DROP: dropout of the finished row, 1 in rows of a multiple of four columns (100k rows of 128 bfloat16: a launch of its own took
// 15 us), 2 in any, where lanes begin inside draws and have one draw more (20k rows of 33 float32: 5 us; one instance for both
// cost the former 3 us of 30).
template <typename T, int VEC, bool TINY, int DROP>
__device__ inline void finish_row(const AggK<T>& p, uint32_t row, int c0, int avail, float (&acc)[VEC],
                                  const RowTail<T, VEC, TINY>& t) {
  constexpr bool ADDS = sizeof(T) == 4;  // bfloat16 rows are only gated (with this branch 172 columns of 2.35M rows took 1 % longer)
  float other[VEC];                      // the row's other operand
  if constexpr (TINY) {
    if (p.self_loop) {
      const float ss = p.in_scale ? p.in_scale[row] : 1.f;
      float xs[VEC];
      load_elems<T, VEC>(row_at(p.X, row, p.ldx) + c0, avail, xs);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = fmaf(ss, xs[i], acc[i]);
    }
    const float so = p.out_scale ? p.out_scale[row] : 1.f;
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] *= so;
    if (p.relu_src) load_elems<T, VEC>(row_at(p.relu_src, row, p.ld_relu) + c0, avail, other);
  } else {
    if (p.self_loop) RowIO<T>::fma_raw(acc, t.ss, t.xs);
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] *= t.so;
    if (p.relu_src) RowIO<T>::unpack(t.g, other);
  }
  // A window of a row that is not TINY exists whole, so its biases are wide loads without a condition: eight
  // conditional ones, each with its own wait, held a launch back by half (2.35M rows of 172 bfloat16 1615 -> 1222 us,
  // 100k rows of 128 43.8 -> 27.0).
  auto add_bias = [&](float (&x)[VEC]) __attribute__((always_inline)) {
    const float* const b = p.bias + (p.col0 + c0);
    if constexpr (TINY) {
#pragma unroll
      for (int i = 0; i < VEC; ++i)
        if (i < avail) x[i] += b[i];
    } else {
#pragma unroll
      for (int q = 0; q < VEC / 4; ++q) {
        const f32x4u t = reinterpret_cast<const f32x4u*>(b)[q];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[4 * q + i] += t[i];
      }
    }
  };
  if (ADDS && p.add_src) {
    // (other + bias) + the scaled sum, each rounded: the bits of a product with its bias that is added to the sum.  Another
    // order opens or closes the ReLU of elements within rounding of zero, and Adam's first steps make whole steps of that.
#pragma clang fp contract(off)
    if (p.bias) add_bias(other);
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = other[i] + acc[i];
  } else {
    if (p.relu_src) {
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] = other[i] > 0.f ? acc[i] * p.gate_scale : 0.f;
    }
    if (p.bias) add_bias(acc);
  }
  if (p.relu_out) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = fmaxf(acc[i], 0.f);
  }
  if constexpr (DROP) {
    const uint64_t first = (uint64_t)row * p.ldy + (uint32_t)(p.col0 + c0);
    if constexpr (DROP == 2) {
      drop_span<VEC>(p.drop, first, acc);
    } else {
#pragma unroll
      for (int q = 0; q < VEC; q += 4) drop4(p.drop, first + q, acc + q);
    }
  }
  // A window that was moved left stores the columns that it shares with the lane before as well: both have the same sums.
  if constexpr (TINY) store_elems<T, VEC>(row_at(p.Y, row, p.ldy) + c0, avail, acc);
  else RowIO<T>::store_wide(row_at(p.Y, row, p.ldy) + c0, acc, p.stream_out);
}

// ---- rows by teams of lanes -----------------------------------------------------------------------
// A row belongs to a team: TL lanes of a wavefront (short rows), a whole wavefront, or a workgroup (long rows).
// Inside a team LPS lanes hold the row's columns (NCH pieces of 16 bytes each) and the team's NG = lanes / LPS
// neighbour groups fetch different neighbours in the same load instruction; the groups are added in a fixed butterfly
// order at the end, a workgroup's four wavefronts in ascending order through LDS.  Neighbour ids (and factors) are
// fetched one per team lane with one coalesced load and handed out by cross-lane reads.
// Rows come in descending degree: the workgroups of the grid's front take the n_block longest rows, then come n_wave
// rows of a wavefront each, then the short rows, 64 / TL per wavefront.  A short team walks a row at 0.115 us per
// neighbour (four in flight), so without the larger teams one row outlasted everything else on graphs of up to a few
// million entries: 100k nodes, 600k entries, 128-wide bfloat16 80 -> 30 us a launch; 600k nodes, 4M entries, 100-wide
// float32 470 -> 350 us.  It is one launch because launches of their own for the long rows cost more than they saved.
// The lines (32 and 128 neighbours, common.h) are flat: 16 to 64 and 64 to 512 measured within 4 % on every workload,
// the smaller workgroup line ahead on 20k nodes (14 -> 11 us a launch).  At most 64 registers in float32 and 72 in
// bfloat16 (64 where a row takes a whole wavefront's lanes) are what the occupancy of the gather needs: 73, 76 and 66 cost
// 3-8 % of every large launch; fewer in bfloat16 go to scratch memory (30 % slower).
template <int LANES>
__device__ inline int team_read_i(int x, int j) {
  if constexpr (LANES == 64) return __builtin_amdgcn_readlane(x, j);
  else return __shfl(x, j, 64);
}
template <int LANES>
__device__ inline float team_read_f(float x, int j) {
  return __int_as_float(team_read_i<LANES>(__float_as_int(x), j));
}

// Adds the neighbours of a short row: col and vals point at its first entry (vals null: factors per node, or none).  The
// groups read their neighbours' ids themselves.  A row has few neighbours, so a batch is one, two or four neighbours a group,
// whichever covers the longest row of the wavefront (rows come in descending degree: mostly all of them); slots past a
// row's end repeat its last neighbour (see RowIO) and are left out, by selects where any lane has one.  Launches of
// rows of up to 64 bfloat16 take as long as their instructions: with batches of four throughout, 64-bit indices and the row's
// offsets waiting for its number they had 230 vector ones a wavefront, half of the time (1.88M rows, 3.9M entries, 47
// bfloat16 363 -> 311 us, 3 bfloat16 258 -> 214; from 128 on, bound by memory, 0-3 %).
template <typename T, int TL, int LPS, int TINY>
__device__ inline void gather_short(const AggK<T>& p, const int32_t* __restrict__ col, const float* __restrict__ vals, int cnt,
                                    int lane, int cread, float (&acc)[RowIO<T>::WIDE]) {
  constexpr int VEC = RowIO<T>::WIDE, NG = TL / LPS;
  const T* __restrict__ X = p.X + (TINY ? 0 : cread);
  const float* __restrict__ in_scale = p.in_scale;
  const int grp = lane % TL / LPS, last = cnt > 0 ? cnt - 1 : 0;
  // one group a row: its ids are fetched one per lane and handed out by cross-lane reads, so that a batch does not wait for
  // its own ids (20k rows of 128 bfloat16 9.7 -> 8.0 us)
  int my_col = 0;
  float my_s = 1.f;
  auto fetch = [&](int j) {
    if (NG > 1 || j % TL != 0) return;
    const int q = j + lane % TL, qc = q < last ? q : last;
    my_col = col[qc];
    if (vals) my_s = vals[qc];
    else if (in_scale) my_s = in_scale[my_col];
  };
  auto batch = [&](int j, auto size) {
    constexpr int B = decltype(size)::value;
    uint32_t u[B];
    float s[B];
#pragma unroll
    for (int t = 0; t < B; ++t) {
      const int q = j + t * NG + grp, qc = q < last ? q : last;
      if constexpr (NG == 1) {
        const int from = lane - lane % TL + qc % TL;
        u[t] = (uint32_t)__shfl(my_col, from, 64);
        s[t] = __shfl(my_s, from, 64);
      } else {
        u[t] = (uint32_t)col[qc];
        s[t] = vals ? vals[qc] : 1.f;
      }
    }
    if (NG > 1 && !vals && in_scale) {
#pragma unroll
      for (int t = 0; t < B; ++t) s[t] = in_scale[u[t]];
    }
    const bool whole = __all(j + B * NG <= cnt);
    if constexpr (TINY) {
      float v[B][TINY];
#pragma unroll
      for (int t = 0; t < B; ++t)
#pragma unroll
        for (int i = 0; i < TINY; ++i) v[t][i] = RowIO<T>::load1(row_at(X, u[t], p.ldx) + i);
#pragma unroll
      for (int t = 0; t < B; ++t)
#pragma unroll
        for (int i = 0; i < TINY; ++i) acc[i] = j + t * NG + grp < cnt ? fmaf(s[t], v[t][i], acc[i]) : acc[i];
    } else {
      typename RowIO<T>::Raw v[B];
#pragma unroll
      for (int t = 0; t < B; ++t) v[t] = RowIO<T>::load_raw(row_at(X, u[t], p.ldx));
      if (whole) {
#pragma unroll
        for (int t = 0; t < B; ++t) RowIO<T>::fma_raw(acc, s[t], v[t]);
      } else {
#pragma unroll
        for (int t = 0; t < B; ++t) RowIO<T>::fma_raw(acc, s[t], RowIO<T>::keep_if(j + t * NG + grp < cnt, v[t]));
      }
    }
  };
  for (int j = 0; __any(j < cnt);) {
    fetch(j);
    if (__any(j + 2 * NG < cnt)) {
      batch(j, std::integral_constant<int, 4>{});
      j += 4 * NG;
    } else if (__any(j + NG < cnt)) {
      batch(j, std::integral_constant<int, 2>{});
      j += 2 * NG;
    } else {
      batch(j, std::integral_constant<int, 1>{});
      j += NG;
    }
  }
#pragma unroll
  for (int off = LPS; off < TL; off <<= 1) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] += __shfl_xor(acc[i], off, 64);
  }
}

// Adds the neighbours of a row that fall to this wavefront (entries first .. of every `stride`, 64 of them at a time): ids are
// fetched one per lane and handed out by cross-lane reads.
template <typename T, int LPS, int NCH>
__device__ inline void gather_row(const AggK<T>& p, const int32_t* __restrict__ col, const float* __restrict__ vals, int cnt_row,
                                  int first, int stride, int lane, const int (&cread)[NCH], float (&acc)[NCH][RowIO<T>::WIDE]) {
  constexpr int VEC = RowIO<T>::WIDE, NG = 64 / LPS;
  constexpr int UNR = 4;
  const T* __restrict__ X = p.X;
  const float* __restrict__ in_scale = p.in_scale;
  const int grp = lane / LPS;
  for (int e0 = first; e0 < cnt_row; e0 += stride) {
    const int e = e0 + lane < cnt_row ? e0 + lane : cnt_row - 1;
    const int my_col = col[e];
    float my_s = 1.f;
    if (vals) my_s = vals[e];
    else if (in_scale) my_s = in_scale[my_col];
    const int cnt = cnt_row - e0 < 64 ? cnt_row - e0 : 64;
    for (int j = 0; j < cnt; j += UNR * NG) {
      uint32_t u[UNR];
      float s[UNR];
      bool ok[UNR];
#pragma unroll
      for (int t = 0; t < UNR; ++t) {
        // slot of this group; a slot past the row's end repeats the last neighbour (see RowIO) and is left out
        const int q = j + t * NG + (NG == 1 ? 0 : grp);
        ok[t] = q < cnt;
        const int qc = ok[t] ? q : cnt - 1;
        u[t] = (uint32_t)team_read_i<LPS>(my_col, qc);
        s[t] = team_read_f<LPS>(my_s, qc);
      }
      typename RowIO<T>::Raw v[UNR][NCH];
#pragma unroll
      for (int t = 0; t < UNR; ++t) {
        const T* const src = row_at(X, u[t], p.ldx);
#pragma unroll
        for (int c = 0; c < NCH; ++c) v[t][c] = RowIO<T>::load_raw(src + cread[c]);
      }
#pragma unroll
      for (int t = 0; t < UNR; ++t)
#pragma unroll
        for (int c = 0; c < NCH; ++c) RowIO<T>::fma_raw(acc[c], s[t], RowIO<T>::keep_if(ok[t], v[t][c]));
    }
  }
#pragma unroll
  for (int off = LPS; off < 64; off <<= 1) {
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[c][i] += __shfl_xor(acc[c][i], off, 64);
  }
}

// The same for a whole wavefront of at least eight neighbour groups (narrow rows), `wave` of `waves` that share the row: the
// groups read their neighbours' ids themselves, which are consecutive.  Ids handed out 64 at a time leave most loads of so
// many groups without a neighbour.  Rows of less than one access have an instance for every width: element loads under a
// condition on the width wait for each other (3 bfloat16 columns: 230k nodes, 14M entries 302 -> 108 us, 30k nodes 162 -> 44).
template <typename T, int LPS, int TINY>
__device__ inline void gather_narrow(const AggK<T>& p, const int32_t* __restrict__ col, const float* __restrict__ in_vals, int cnt,
                                     int wave, int waves, int lane, int cread, float (&acc)[RowIO<T>::WIDE]) {
  constexpr int VEC = RowIO<T>::WIDE, NG = 64 / LPS;
  constexpr int UNR = 4;
  const float* __restrict__ in_scale = p.in_scale;
  const T* __restrict__ X = p.X + (TINY ? 0 : cread);
  const int last = cnt - 1, e0 = wave * (NG * UNR) + lane / LPS, step = waves * (NG * UNR);
  // scale_mode: 0 no per-source factor, 1 gathered from the per-node vector, 2 per entry
  auto gather = [&](auto scale_mode) {
    constexpr int MODE = decltype(scale_mode)::value;
    for (int e = e0; e < cnt; e += step) {
      uint32_t u[UNR];
      float s[UNR];
      if constexpr (TINY) {
        // 64 neighbours a slot: the element loads of slots that no lane has are passed over
        float v[UNR][TINY];
#pragma unroll
        for (int t = 0; t < UNR; ++t) u[t] = e + t * NG < cnt ? (uint32_t)col[e + t * NG] : ~0u;
#pragma unroll
        for (int t = 0; t < UNR; ++t) {
          s[t] = 1.f;
#pragma unroll
          for (int i = 0; i < TINY; ++i) v[t][i] = 0.f;
          if (u[t] != ~0u) {
            if constexpr (MODE == 2) s[t] = in_vals[e + t * NG];
            if constexpr (MODE == 1) s[t] = in_scale[u[t]];
#pragma unroll
            for (int i = 0; i < TINY; ++i) v[t][i] = RowIO<T>::load1(row_at(X, u[t], p.ldx) + i);
          }
        }
#pragma unroll
        for (int t = 0; t < UNR; ++t)
#pragma unroll
          for (int i = 0; i < TINY; ++i) acc[i] = fmaf(s[t], v[t][i], acc[i]);
      } else {
        typename RowIO<T>::Raw v[UNR];
#pragma unroll
        for (int t = 0; t < UNR; ++t) {
          const int ec = e + t * NG < last ? e + t * NG : last;  // past the end: the last one, left out (see RowIO)
          u[t] = (uint32_t)col[ec];
          if constexpr (MODE == 2) s[t] = in_vals[ec];
        }
#pragma unroll
        for (int t = 0; t < UNR; ++t) {
          if constexpr (MODE == 1) s[t] = in_scale[u[t]];
          if constexpr (MODE == 0) s[t] = 1.f;
          v[t] = RowIO<T>::load_raw(row_at(X, u[t], p.ldx));
        }
#pragma unroll
        for (int t = 0; t < UNR; ++t) RowIO<T>::fma_raw(acc, s[t], RowIO<T>::keep_if(e + t * NG < cnt, v[t]));
      }
    }
  };
  if (in_vals) gather(std::integral_constant<int, 2>{});
  else if (in_scale) gather(std::integral_constant<int, 1>{});
  else gather(std::integral_constant<int, 0>{});
#pragma unroll
  for (int off = LPS; off < 64; off <<= 1) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] += __shfl_xor(acc[i], off, 64);
  }
}

// TINY: the columns of rows narrower than one 16-byte access (element accesses; LPS = 1), else 0.
// Rows need only element alignment (see LaneCols for the ragged end of a row).
template <typename T, int TL, int LPS, int NCH, int TINY, int DROP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NCH > 1 ? 4 : (sizeof(T) == 4 || TL == 64 ? 8 : 7)))) void aggregate_kernel(const AggK<T> p) {
  constexpr int VEC = RowIO<T>::WIDE;
  constexpr int RPW = 64 / TL;  // short rows per wavefront
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPS;
  const uint32_t b = blockIdx.x, n_block = p.n_block, n_wave = p.n_wave;
  const uint32_t wave_blocks = (n_wave + 3) / 4;
  int team;  // 0 short rows, 1 a wavefront per row, 2 a workgroup per row (uniform over the block)
  uint32_t slot, limit;
  if (b < n_block) {
    team = 2;
    slot = b;
    limit = n_block;
  } else if (b < n_block + wave_blocks) {
    team = 1;
    slot = n_block + (b - n_block) * 4 + wave;
    limit = n_block + n_wave;
  } else {
    team = 0;
    slot = n_block + n_wave + ((b - n_block - wave_blocks) * 4 + wave) * RPW + lane / TL;
    limit = (uint32_t)p.n;
  }
  if (slot >= limit) return;  // never in a workgroup that shares a row
  const uint32_t s = (uint32_t)p.slot0 + slot;
  uint32_t row = slot;
  int64_t beg, end;
  if (p.by_slot) {  // the row's number is not needed for its offsets: both are on their way together
    row = (uint32_t)p.order[s];
    beg = p.rowptr[s], end = p.rowptr[s + 1];
  } else {
    if (p.order) row = (uint32_t)p.order[s];
    beg = p.rowptr[row], end = p.rowptr[row + 1];
  }
  const int cnt = (int)(end - beg);
  // a row without neighbours beside one that has some reads the graph's first entry
  const int64_t at = cnt > 0 ? beg : 0;
  const int32_t* const col = p.col + at;
  const float* const vals = p.in_vals ? p.in_vals + at : nullptr;

  float acc[NCH][VEC];
  LaneCols lc[NCH];
  int cread[NCH];  // first column a lane reads (lanes past the end: the row's last window)
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    lc[c] = lane_cols<VEC>(p.width, (sub + c * LPS) * VEC);
    cread[c] = lc[c].avail > 0 ? lc[c].c0 : (p.width >= VEC ? p.width - VEC : 0);
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[c][i] = 0.f;
  }
  RowTail<T, VEC, TINY != 0> tail[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) tail[c].request(p, row, s, cread[c]);

  bool short_row = false;
  if constexpr (TL < 64) short_row = team == 0;
  if (short_row) {
    if constexpr (TL < 64) gather_short<T, TL, LPS, TINY>(p, col, vals, cnt, lane, cread[0], acc[0]);
  } else {
    if constexpr (LPS <= 8) gather_narrow<T, LPS, TINY>(p, col, vals, cnt, team == 2 ? wave : 0, team == 2 ? 4 : 1, lane, cread[0], acc[0]);
    else gather_row<T, LPS, NCH>(p, col, vals, cnt, team == 2 ? wave * 64 : 0, team == 2 ? 256 : 64, lane, cread, acc);
    if (team == 2) {
      __shared__ float partial[3][NCH * LPS * VEC];
      if (wave > 0 && lane < LPS) {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
          for (int i = 0; i < VEC; ++i) partial[wave - 1][(c * VEC + i) * LPS + sub] = acc[c][i];
      }
      __syncthreads();
      if (wave > 0) return;
#pragma unroll
      for (int w = 0; w < 3; ++w)
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
          for (int i = 0; i < VEC; ++i) acc[c][i] += partial[w][(c * VEC + i) * LPS + sub];
    }
  }
  if ((lane % (team == 0 ? TL : 64)) >= LPS) return;  // the first neighbour group of the team writes
#pragma unroll
  for (int c = 0; c < NCH; ++c)
    if (lc[c].avail > 0) finish_row<T, VEC, TINY != 0, DROP>(p, row, lc[c].c0, lc[c].avail, acc[c], tail[c]);
}

// ---- XCD-affine column slices ---------------------------------------------------------------------
// For graphs of high average degree whose matrix is far larger than one XCD's 4 MB L2.  Workgroups are dealt round-robin to
// the 8 XCDs, so workgroup b works on column slice b % 8 (with fewer slices on slice b % slices, where the XCDs of a slice
// share its rows), and each XCD's L2 only ever holds that part of every row - as many more (hot) rows.
// Rows of up to AGG_BLOCK_MIN neighbours belong to LPS lanes each, so that a wavefront works on 64 / LPS rows of nearly equal
// degree (processing order) without adding groups up at the end: a wavefront for every row and slice spent about half of its
// instructions outside the gather (256 float32: 115k nodes, 3.5M entries 510 -> 342 us, 230k nodes, 14M entries 1645 -> 1515,
// 9.4 TB/s of gathered rows; 256 bfloat16, which had no slices: 230k nodes 875 -> 690, 600k nodes, 15M entries 1026 -> 952).
// Longer rows take a wavefront, in which a neighbour has as many lanes as a row has pieces, or a slice, and float32 has a sum for
// every load in flight: eight lanes whatever the row and one sum were up to 2.1 times as far from float64 as the row kernel is
// (230k nodes, 14M entries, 4 float32: relative error of a mean over hubs 9.0e-8, now 4.4e-8, row kernel 4.4e-8) and slower where
// most rows are long (60k nodes, 9M entries, 8 bfloat16 68 -> 48 us; 230k nodes 101 -> 86).
// Rows that are no whole lines, or narrow ones, take the same teams without slices.

// lane n of each team of LPS lanes, to all of the team (n < 8)
template <int LPS, int N>
__device__ inline int team_share(int x) {
  return __builtin_amdgcn_ds_swizzle(x, (N << 5) | (LPS < 32 ? 32 - LPS : 0));
}

// Adds the neighbours of the team's row, eight at a time: a lane holds the id (and factor) of one.  In float32 each of the
// eight has a sum of its own, added pairwise at the end, so that sums are rounded as often as with a wavefront per row (one sum
// per two: 2-4 % faster, 2-3 % further from float64).  bfloat16 results are rounded to 2^-9 anyway and registers are dearer.
template <typename T, int LPS, int MODE>
__device__ inline void gather_teams(const AggK<T>& p, const T* __restrict__ X, const int32_t* __restrict__ col,
                                    const float* __restrict__ vals, int cnt, int lane, float (&out)[RowIO<T>::WIDE]) {
  constexpr int VEC = RowIO<T>::WIDE, UNR = 8, SUMS = VEC == 4 ? 8 : 2;
  const int most = __builtin_amdgcn_readlane(cnt, 0), least = __builtin_amdgcn_readlane(cnt, 63);  // descending degree
  const int last = cnt > 0 ? cnt - 1 : 0, k = lane & 7;
  float acc[SUMS][VEC];
#pragma unroll
  for (int t = 0; t < SUMS; ++t)
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[t][i] = out[i] = 0.f;
  if (most == 0) return;  // the graph may have no entry to read
  int id = col[k < last ? k : last];
  float f = 1.f;
  if constexpr (MODE == 2) f = vals[k < last ? k : last];
  for (int e = 0; e < most; e += UNR) {
    if constexpr (MODE == 1) f = p.in_scale[id];
    uint32_t u[UNR];
    u[0] = team_share<LPS, 0>(id), u[1] = team_share<LPS, 1>(id), u[2] = team_share<LPS, 2>(id), u[3] = team_share<LPS, 3>(id);
    u[4] = team_share<LPS, 4>(id), u[5] = team_share<LPS, 5>(id), u[6] = team_share<LPS, 6>(id), u[7] = team_share<LPS, 7>(id);
    float w[UNR];
    if constexpr (MODE != 0) {
      const int fi = __float_as_int(f);
      w[0] = __int_as_float(team_share<LPS, 0>(fi)), w[1] = __int_as_float(team_share<LPS, 1>(fi));
      w[2] = __int_as_float(team_share<LPS, 2>(fi)), w[3] = __int_as_float(team_share<LPS, 3>(fi));
      w[4] = __int_as_float(team_share<LPS, 4>(fi)), w[5] = __int_as_float(team_share<LPS, 5>(fi));
      w[6] = __int_as_float(team_share<LPS, 6>(fi)), w[7] = __int_as_float(team_share<LPS, 7>(fi));
    }
    typename RowIO<T>::Raw v[UNR];
#pragma unroll
    for (int t = 0; t < UNR; ++t) v[t] = RowIO<T>::load_raw(row_at(X, u[t], p.ldx));
    const int n = e + UNR + k < last ? e + UNR + k : last;  // the next batch's
    id = col[n];
    if constexpr (MODE == 2) f = vals[n];
    if (e + UNR > least) {
#pragma unroll
      for (int t = 0; t < UNR; ++t) v[t] = RowIO<T>::keep_if(e + t < cnt, v[t]);
    }
#pragma unroll
    for (int t = 0; t < SUMS; ++t) {
      if constexpr (SUMS == UNR) {
        RowIO<T>::fma_raw(acc[t], MODE == 0 ? 1.f : w[t], v[t]);
      } else {
        float x[VEC] = {};
#pragma unroll
        for (int q = t; q < UNR; q += SUMS) RowIO<T>::fma_raw(x, MODE == 0 ? 1.f : w[q], v[q]);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[t][i] += x[i];
      }
    }
  }
#pragma unroll
  for (int d = SUMS / 2; d > 0; d >>= 1)
#pragma unroll
    for (int t = 0; t < d; ++t)
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[t][i] += acc[t + d][i];
#pragma unroll
  for (int i = 0; i < VEC; ++i) out[i] = acc[0][i];
}

template <typename T, int LPS, int DROP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 5))) void aggregate_sliced_kernel(
    const AggK<T> p, int slice_bits, uint32_t long_units, int long_bits) {
  constexpr int VEC = RowIO<T>::WIDE;
  constexpr int NG = 64 / LPS;
  constexpr int UNR = 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t xcd = blockIdx.x & 7u, unit = ((blockIdx.x >> 3) << (3 - slice_bits)) + (xcd >> slice_bits);
  const bool is_long = unit < long_units;  // uniform over the block
  const int bits = is_long ? long_bits : LPS == 8 ? 3 : LPS == 16 ? 4 : LPS == 32 ? 5 : 6;  // 2^bits lanes share a neighbour
  const int sub = lane & ((1 << bits) - 1), grp = lane >> bits;
  // a lane's columns: whole lines of a slice, or any row that is not cut (the last window moved, lanes past the end idle)
  const LaneCols lc = lane_cols<VEC>(p.width, ((int)(xcd & ((1u << slice_bits) - 1u)) * LPS + sub) * VEC);
  const int c0 = lc.avail > 0 ? lc.c0 : p.width - VEC;
  const T* __restrict__ X = p.X + c0;
  const uint32_t limit = is_long ? (uint32_t)p.n_wave : (uint32_t)p.n;
  const uint32_t first = is_long ? unit * 4 + wave : (uint32_t)p.n_wave + ((unit - long_units) * 4 + wave) * NG;
  if (first >= limit) return;
  const uint32_t slot = is_long ? first : first + grp;
  const bool has = slot < limit;
  const uint32_t s = (uint32_t)p.slot0 + (has ? slot : limit - 1);
  const uint32_t row = (uint32_t)p.order[s];
  const uint32_t at = p.by_slot ? s : row;
  const int64_t beg = p.rowptr[at];
  const int cnt = has ? (int)(p.rowptr[at + 1] - beg) : 0;
  const int32_t* __restrict__ col = p.col + (cnt > 0 ? beg : 0);
  const float* __restrict__ vals = p.in_vals ? p.in_vals + (cnt > 0 ? beg : 0) : nullptr;
  RowTail<T, VEC, false> tail;
  tail.request(p, row, s, c0);
  float acc[VEC];
  if (!is_long) {
    if (vals) gather_teams<T, LPS, 2>(p, X, col, vals, cnt, lane, acc);
    else if (p.in_scale) gather_teams<T, LPS, 1>(p, X, col, vals, cnt, lane, acc);
    else gather_teams<T, LPS, 0>(p, X, col, vals, cnt, lane, acc);
    if (!has || lc.avail <= 0) return;
  } else {
    constexpr int SUMS = VEC == 4 ? UNR : 1;
    float part[SUMS][VEC];
#pragma unroll
    for (int t = 0; t < SUMS; ++t)
#pragma unroll
      for (int i = 0; i < VEC; ++i) part[t][i] = 0.f;
    // every load of the loop is unconditional (see RowIO): ids past the end of the row repeat its last id and are
    // zeroed after the load
    const int ng = 64 >> bits;
    for (int e = grp; e < cnt; e += ng * UNR) {
      uint32_t u[UNR];
      float f[UNR];
      typename RowIO<T>::Raw v[UNR];
#pragma unroll
      for (int t = 0; t < UNR; ++t) {
        const int ec = e + t * ng < cnt ? e + t * ng : cnt - 1;
        u[t] = (uint32_t)col[ec];
        f[t] = 1.f;
        if (vals) f[t] = vals[ec];
      }
#pragma unroll
      for (int t = 0; t < UNR; ++t) {
        if (!vals && p.in_scale) f[t] = p.in_scale[u[t]];
        v[t] = RowIO<T>::load_raw(row_at(X, u[t], p.ldx));
      }
#pragma unroll
      for (int t = 0; t < UNR; ++t) RowIO<T>::fma_raw(part[t % SUMS], f[t], RowIO<T>::keep_if(e + t * ng < cnt, v[t]));
    }
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      if constexpr (SUMS == 4) acc[i] = (part[0][i] + part[1][i]) + (part[2][i] + part[3][i]);
      else acc[i] = part[0][i];
    }
    for (int off = 1 << bits; off < 64; off <<= 1) {
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] += __shfl_xor(acc[i], off, 64);
    }
    if (grp != 0 || lc.avail <= 0) return;
  }
  finish_row<T, VEC, false, DROP>(p, row, c0, VEC, acc, tail);
}

// ---- hub rows -----------------------------------------------------------------------------------
// One workgroup of HUB_WAVES wavefronts per (row, column panel of LPS lanes x 16 bytes).  Inside a wavefront the
// lanes form 64/LPS neighbour groups as in the long-row kernel; neighbour j of the row goes to wavefront
// (j / NG) % HUB_WAVES, group j % NG, so that consecutive ids - one coalesced read - feed one wavefront's load
// instruction.  The groups of a wavefront are added by the same butterfly, then wavefront w > 0 writes its
// partial panel to LDS and wavefront 0 adds the partials in ascending w: a fixed order.
constexpr int HUB_WAVES = 16;
template <typename T, int LPS, int DROP>
__global__ __launch_bounds__(HUB_WAVES * 64) void aggregate_hub_kernel(const AggK<T> p) {
  constexpr int VEC = RowIO<T>::WIDE;
  constexpr int NG = 64 / LPS;
  constexpr int UNR = 4;
  __shared__ float partial[HUB_WAVES - 1][LPS * VEC];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPS, grp = lane / LPS;
  const uint32_t row = (uint32_t)p.order[p.slot0 + blockIdx.x];
  const LaneCols lc = lane_cols<VEC>(p.width, (int)blockIdx.y * (LPS * VEC) + sub * VEC);
  const int c0 = lc.c0, avail = lc.avail;
  const int cread = avail > 0 ? c0 : p.width - VEC;  // the launcher sends only rows of at least VEC columns here
  const int32_t* __restrict__ col = p.col;
  const float* __restrict__ in_scale = p.in_scale;
  const float* __restrict__ in_vals = p.in_vals;
  const T* __restrict__ Xread = p.X + cread;
  const int64_t beg = p.rowptr[row], end = p.rowptr[row + 1];
  float acc[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
  RowTail<T, VEC, false> tail;
  if (wave == 0) tail.request(p, row, 0, cread);
  if (end > beg) {
    const int64_t last = end - 1;
    // step of one wavefront: NG neighbours; of the workgroup: NG * HUB_WAVES; UNR steps in flight
    for (int64_t e = beg + (int64_t)wave * NG + grp; e < end; e += (int64_t)NG * HUB_WAVES * UNR) {
      uint32_t u[UNR];
      float sc[UNR];
      typename RowIO<T>::Raw v[UNR];
#pragma unroll
      for (int t = 0; t < UNR; ++t) {
        const int64_t ee = e + (int64_t)t * NG * HUB_WAVES;
        const int64_t ec = ee < last ? ee : last;
        u[t] = (uint32_t)col[ec];
        sc[t] = in_vals ? in_vals[ec] : 1.f;
      }
#pragma unroll
      for (int t = 0; t < UNR; ++t) {
        if (!in_vals && in_scale) sc[t] = in_scale[u[t]];
        v[t] = RowIO<T>::load_raw(row_at(Xread, u[t], p.ldx));
      }
#pragma unroll
      for (int t = 0; t < UNR; ++t)
        RowIO<T>::fma_raw(acc, sc[t], RowIO<T>::keep_if(e + (int64_t)t * NG * HUB_WAVES < end, v[t]));
    }
  }
#pragma unroll
  for (int off = LPS; off < 64; off <<= 1) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] += __shfl_xor(acc[i], off, 64);
  }
  if (wave > 0 && grp == 0) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) partial[wave - 1][sub * VEC + i] = acc[i];
  }
  __syncthreads();
  if (wave != 0 || grp != 0 || avail <= 0) return;
  for (int w = 0; w < HUB_WAVES - 1; ++w) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] += partial[w][sub * VEC + i];
  }
  finish_row<T, VEC, false, DROP>(p, row, c0, avail, acc, tail);
}

// ---- host side ------------------------------------------------------------------------------------
template <typename T>
static const char* type_name() {
  return sizeof(T) == 4 ? "float" : "bf16";
}

// One launch = one timing record, named by the kernel's template instance and the launch's shape.  Algorithmic
// traffic of a launch over `rows` rows with `nnz` adjacency entries: every source row read once and every output
// row written once (`rows` each: the sources of a bucket's rows are as many again at this graph's symmetry only on
// average, so the bucket is charged its own row count), 4 bytes per entry, 8 per row offset, the per-node scale
// vectors and the gate matrix once.
template <typename T>
struct LaunchCost {
  const AggArgs& a;
  const T* R;
  double bytes(int64_t rows, int64_t nnz) const {
    return 2.0 * (double)rows * a.width * sizeof(T) + 4.0 * (double)nnz + 8.0 * (double)(rows + 1) +
           4.0 * (double)rows * ((a.in_scale ? 1 : 0) + (a.out_scale ? 1 : 0)) +
           (R ? (double)rows * a.width * sizeof(T) : 0.0);
  }
  double flops(int64_t nnz) const { return 2.0 * (double)nnz * a.width; }
};

// One launch of the row kernel: k.n rows, of which the first k.n_block take a workgroup and the next k.n_wave a
// wavefront each.  Column lanes: the smallest power of two that covers the row in 16-byte pieces.  Short rows come
// four to a wavefront, where the columns leave that many lanes: with more rows, narrow rows measured slower (8 rows
// of 6 pieces: 0.50 ms, 4 rows 0.41 ms on 1.9M rows of 47 bfloat16); lanes that the columns leave free fetch further
// neighbours of the row.
template <typename T, int WIDTH = RowIO<T>::WIDE - 1>
static void launch_tiny(const AggK<T>& k, dim3 grid, hipStream_t stream) {
  if (k.width == WIDTH) {
    aggregate_kernel<T, 16, 1, 1, WIDTH, 0><<<grid, 256, 0, stream>>>(k);
  } else {
    if constexpr (WIDTH > 1) launch_tiny<T, WIDTH - 1>(k, grid, stream);
  }
}

constexpr int ROW_PIECES = 128;  // wider rows take several launches
template <typename T, int DROP>
static int32_t launch_rows(const AggK<T>& k, hipStream_t stream, const LaunchCost<T>& cost, int64_t nnz) {
  constexpr int WIDE = RowIO<T>::WIDE;
  const int chunks = (k.width + WIDE - 1) / WIDE;
  const bool tiny = k.width < WIDE;
  if (DROP && tiny) return fail(COFREE_EINVAL, "internal: no dropout in rows of less than one access");
  int lps = 1;
  while (lps < chunks && lps < 64) lps *= 2;
  const int tl = lps < 16 ? 16 : lps;
  const int nch = chunks > 64 ? 2 : 1;
  const int64_t short_rows = k.n - k.n_block - k.n_wave, per_block = 4 * (64 / tl);
  const int64_t blocks = k.n_block + ((int64_t)k.n_wave + 3) / 4 + (short_rows + per_block - 1) / per_block;
  COFREE_REQUIRE(blocks < ((int64_t)1 << 31), "aggregate: grid too large");
  char pname[96] = "";
  if (profiling()) snprintf(pname, sizeof(pname), "aggregate_kernel<%s,%d,%d,%d,%d,%d> width=%d", type_name<T>(), tl, lps, nch,
           tiny ? (int)k.width : 0, DROP, (int)cost.a.width);
  ProfScope prof(pname, stream, cost.bytes(k.n, nnz), cost.flops(nnz));
  const dim3 grid((unsigned)blocks);
  if (tiny) launch_tiny<T>(k, grid, stream);
  else if (lps == 1) aggregate_kernel<T, 16, 1, 1, 0, DROP><<<grid, 256, 0, stream>>>(k);
  else if (lps == 2) aggregate_kernel<T, 16, 2, 1, 0, DROP><<<grid, 256, 0, stream>>>(k);
  else if (lps == 4) aggregate_kernel<T, 16, 4, 1, 0, DROP><<<grid, 256, 0, stream>>>(k);
  else if (lps == 8) aggregate_kernel<T, 16, 8, 1, 0, DROP><<<grid, 256, 0, stream>>>(k);
  else if (lps == 16) aggregate_kernel<T, 16, 16, 1, 0, DROP><<<grid, 256, 0, stream>>>(k);
  else if (lps == 32) aggregate_kernel<T, 32, 32, 1, 0, DROP><<<grid, 256, 0, stream>>>(k);
  else if (nch == 1) aggregate_kernel<T, 64, 64, 1, 0, DROP><<<grid, 256, 0, stream>>>(k);
  else aggregate_kernel<T, 64, 64, 2, 0, DROP><<<grid, 256, 0, stream>>>(k);
  return COFREE_OK;
}

template <typename T, int DROP>
static int32_t launch_sliced(const AggK<T>& k, int lps, int long_bits, int slice_bits, hipStream_t stream, const LaunchCost<T>& cost, int64_t nnz) {
  const int64_t long_units = (k.n_wave + 3) / 4, rows = 4 * (64 / lps), parts = 8 >> slice_bits;
  const int64_t units = long_units + (k.n - k.n_wave + rows - 1) / rows;
  const int64_t blocks = (units + parts - 1) / parts * 8;
  COFREE_REQUIRE(blocks < ((int64_t)1 << 31), "aggregate: grid too large");
  const dim3 grid((unsigned)blocks);
  char pname[96] = "";
  if (profiling()) snprintf(pname, sizeof(pname), "aggregate_sliced_kernel<%s,%d,%d> width=%d", type_name<T>(), lps, DROP,
           (int)cost.a.width);
  ProfScope prof(pname, stream, cost.bytes(k.n, nnz), cost.flops(nnz));
  switch (lps) {
    case 8: aggregate_sliced_kernel<T, 8, DROP><<<grid, 256, 0, stream>>>(k, slice_bits, (uint32_t)long_units, long_bits); break;
    case 16: aggregate_sliced_kernel<T, 16, DROP><<<grid, 256, 0, stream>>>(k, slice_bits, (uint32_t)long_units, long_bits); break;
    case 32: aggregate_sliced_kernel<T, 32, DROP><<<grid, 256, 0, stream>>>(k, slice_bits, (uint32_t)long_units, long_bits); break;
    case 64: aggregate_sliced_kernel<T, 64, DROP><<<grid, 256, 0, stream>>>(k, slice_bits, (uint32_t)long_units, long_bits); break;
    default: return fail(COFREE_EINVAL, "internal: bad lanes-per-slice");
  }
  return COFREE_OK;
}

// hub rows: order[0 .. n_hub), one workgroup per (row, panel of lps lanes x 16 bytes)
template <typename T, int DROP>
static int32_t launch_hub(const AggK<T>& k, hipStream_t stream, const LaunchCost<T>& cost, int64_t nnz) {
  constexpr int WIDE = RowIO<T>::WIDE;
  int lps = 1;
  while (lps < 64 && lps * WIDE < k.width) lps *= 2;
  const int panels = (k.width + lps * WIDE - 1) / (lps * WIDE);
  COFREE_REQUIRE(k.n < ((int64_t)1 << 31) && panels < 65536, "aggregate: hub grid too large");
  const dim3 grid((unsigned)k.n, (unsigned)panels);
  char pname[96] = "";
  if (profiling()) snprintf(pname, sizeof(pname), "aggregate_hub_kernel<%s,%d,%d> width=%d", type_name<T>(), lps, DROP,
           (int)cost.a.width);
  ProfScope prof(pname, stream, cost.bytes(k.n, nnz), cost.flops(nnz));
  switch (lps) {
    case 1: aggregate_hub_kernel<T, 1, DROP><<<grid, HUB_WAVES * 64, 0, stream>>>(k); break;
    case 2: aggregate_hub_kernel<T, 2, DROP><<<grid, HUB_WAVES * 64, 0, stream>>>(k); break;
    case 4: aggregate_hub_kernel<T, 4, DROP><<<grid, HUB_WAVES * 64, 0, stream>>>(k); break;
    case 8: aggregate_hub_kernel<T, 8, DROP><<<grid, HUB_WAVES * 64, 0, stream>>>(k); break;
    case 16: aggregate_hub_kernel<T, 16, DROP><<<grid, HUB_WAVES * 64, 0, stream>>>(k); break;
    case 32: aggregate_hub_kernel<T, 32, DROP><<<grid, HUB_WAVES * 64, 0, stream>>>(k); break;
    default: aggregate_hub_kernel<T, 64, DROP><<<grid, HUB_WAVES * 64, 0, stream>>>(k); break;
  }
  return COFREE_OK;
}

template <typename T, int DROP>
static int32_t launch_typed(const AggArgs& a, hipStream_t stream) {
  constexpr int WIDE = RowIO<T>::WIDE;
  const T* X = (const T*)a.X;
  T* Y = (T*)a.Y;
  const T* R = (const T*)(a.add ? a.add : a.relu_src);
  AggK<T> k{};
  k.rowptr = a.g.rowptr;
  k.col = a.g.col;
  k.ldx = (uint32_t)a.ldx;
  k.ldy = (uint32_t)a.ldy;
  k.in_scale = a.in_scale;
  k.out_scale = a.out_scale;
  k.self_loop = a.self_loop;
  k.ld_relu = (uint32_t)(a.add ? a.ld_add : a.ld_relu);
  k.add_src = a.add != nullptr;
  k.gate_scale = a.gate_scale;
  k.bias = a.bias;
  k.relu_out = a.relu_out;
  k.drop = dropout_k(a.dropout);
  k.width = a.width;
  k.col0 = 0;
  // Results of 160 MB and more go past the caches (stream_result): the memory-side cache of 256 MB then keeps rows that are
  // gathered again.  Time with / without, plain mean and GCN form, rows whose result the next launch gathers from, ten shapes of 3 to
  // 30 neighbours a node: 230 MB 0.89 to 0.97, 180 MB 0.89 to 1.00, 140 MB 0.94 to 1.04, 110 MB 0.94 to 1.10, 50 MB 0.98 to 1.25; where
  // the result is read once, in order, 0.90 to 0.99 at 230 MB, 0.93 to 1.01 at 110 MB.  1.88M rows of 47 bfloat16 290 -> 229 us,
  // 470k of 100 float32 154 -> 104, 230k of 256 float32 (14M entries) 1336 -> 1279, 2.35M of 256 bfloat16 1070 -> 1049.
  k.stream_out = stream_result((double)a.g.n * a.width * sizeof(T));
  k.X = X;
  k.Y = Y;
  k.relu_src = R;
  const LaunchCost<T> cost{a, R};

  // Hub rows (the head of the sorted row order) get a launch of their own.  COFREE_AGG_BUCKETS = 0 leaves them - and
  // all other long rows - to the teams of the row kernel that take every other row.
  bool buckets = a.g.order != nullptr;
  if (const char* env = getenv("COFREE_AGG_BUCKETS")) buckets = buckets && atoi(env) != 0;
  const int64_t n_hub = buckets && a.width >= WIDE ? a.g.n_hub : 0;
  const int64_t hub_nnz = n_hub > 0 ? a.g.nnz_hub : 0;

  // High average degree: teams of lanes per row in wavefronts of rows of nearly equal degree (aggregate_sliced_kernel), cut into
  // up to 8 XCD-affine column slices of whole 128-byte lines, two at least; else a wavefront for every row.
  //  * Slices, of rows of four lines and more from a matrix of one XCD's 4 MB L2 on (8k nodes, 300k entries, 256 float32 30 -> 21 us;
  //    115k nodes, 3.5M entries 472 -> 344; 230k nodes, 14M entries 1805 -> 1455), of two lines from 12 MB on (60k nodes, 2.2M entries,
  //    128 bfloat16 59 -> 52; 8 MB 36 -> 38).  Up to 420 MB in float32, 500 MB in bfloat16: the rows that are gathered most stay in
  //    the memory-side cache of 256 MB, beyond that pieces of one line cost more than the hits are worth (20 to 40 entries a node;
  //    128 float32 358 MB 1.00 and 0.98 of the time of a wavefront for every row, 410 MB 1.00 and 0.97, 435 MB 1.02 and 0.99, 512 MB
  //    1.03 and 1.00; 256 bfloat16 410 MB 0.95 and 0.91, 512 MB 0.96 and 0.93; 512 bfloat16 410 MB 0.89 and 0.90, 461 MB 0.97 and
  //    1.01, 614 MB 1.07 and 1.03, 1024 MB 1.16 and 1.13; GCN and mean).
  //  * float32 rows of eight lines and more are cut whatever their number: a wavefront for every row sums all of a neighbour
  //    list in one chain, up to 6.8 times as far from float64 (600k nodes, 15M entries, 256 float32: relative error of a mean over
  //    hubs 6.1e-7 and 0.9e-7).  256 float32 461 MB 1.02 of the time, 614 MB 1.12, 1024 MB 1.16; 512 float32, in slices of two
  //    lines, 471 MB 0.76, 1229 MB 0.92, 1638 MB 1.00, 2048 MB 1.08.
  //  * Without slices, rows of up to 16 pieces of 16 bytes that are no whole lines or lie beyond that: a team walks a row alone, so
  //    a launch has to outlast 128 neighbours - up to four pieces from 2^21 entries on (60k nodes, 2.2M entries, 16 float32 36 -> 28
  //    us; 115k nodes, 3.5M entries, 8 bfloat16 72 -> 31; 600k nodes, 15M entries 337 -> 149), up to eight from 3 * 2^20 on (115k
  //    nodes, 3.5M entries, 47 bfloat16 104 -> 78, 40 bfloat16 77 -> 67; 60k nodes, 2.2M entries 47 -> 50), wider rows from 2^23
  //    on (230k nodes, 14M entries, 41 float32 435 -> 397; 300k nodes, 9M entries 330 -> 312; 115k nodes, 7M entries 175 -> 180), and
  //    where no factors are read beside the ids, below an average of 48 neighbours (33 float32: 300k nodes, 9M entries 232 -> 228;
  //    230k nodes, 14M entries 299 -> 308; 60k nodes, 9M entries 136 -> 147).  Wider still, a wavefront has two rows and gains nothing
  //    (100 float32: 230k nodes, 14M entries 865 -> 803, 300k nodes, 9M entries 628 -> 643).
  // Below an average of 16 neighbours neither is faster than the row kernel (600k nodes, 7M entries: 1.00 to 1.15 of its time).
  const bool dense_rows = a.g.nnz / a.g.n >= AGG_LONG_MIN;
  const int64_t row_bytes = a.width * (int64_t)sizeof(T), lines = row_bytes / 128;
  const double matrix = (double)a.g.n * row_bytes;
  const int pieces = (a.width + WIDE - 1) / WIDE;
  const bool sliceable = a.g.order != nullptr && lines * 128 == row_bytes && lines >= 2 && lines <= 64 && (lines & (lines - 1)) == 0;
  const bool teamable = a.g.order != nullptr && a.width >= WIDE && pieces <= 32;
  bool waves = dense_rows;
  bool sliced = dense_rows && sliceable && matrix >= (lines >= 4 ? 4e6 : 12e6) &&
                (sizeof(T) == 4 ? lines >= 8 || matrix <= 420e6 : matrix <= 500e6);
  bool teams = dense_rows && teamable && !sliced && pieces <= 16 && a.g.nnz >= (pieces <= 4 ? 1 << 21 : pieces <= 8 ? 3 << 20 : 1 << 23) &&
               (pieces <= 8 || a.in_scale || a.g.nnz / a.g.n < 48);
  if (const char* env = getenv("COFREE_AGG_SLICES")) {  // 0 = by degree, 1 = a wavefront per row, 2 = teams, 8 = sliced
    const int v = atoi(env);
    if (v == 0 || v == 1) waves = v == 1, sliced = teams = false;
    if (v == 2) sliced = false, teams = teamable;
    if (v == 8) sliced = sliceable, teams = false;
  }
  int slice_bits = lines >= 8 ? 3 : lines == 4 ? 2 : 1, team_lanes = (int)(lines * 8 >> slice_bits);
  if (teams) {
    slice_bits = 0, team_lanes = 8;
    while (team_lanes < pieces) team_lanes *= 2;
  }
  int long_bits = 0;  // a neighbour of a long row takes as many lanes as the row has pieces, but a whole slice
  while ((1 << long_bits) < (teams ? pieces : team_lanes)) ++long_bits;

  // Per-source factors of a large graph are read per entry: the per-node vector no longer stays in L2 there, and
  // every neighbour's factor would cost a memory access of its own beside the row it scales (28M-node partition,
  // 256-wide bfloat16 launch: 16.7 ms with the per-node gather, 15.9 ms with the per-entry stream; no difference
  // at 1.9M nodes), and so are those of teams, which read them with the ids, and of slices, each of which would gather them again
  // (115k nodes, 3.5M entries, 256-wide float32: with the gather a four-layer training step took 5.36 ms, with the stream 5.07).  COFREE_AGG_ENTRY_SCALE = 0 / 1 forces one or the other.
  k.in_vals = nullptr;
  if (a.in_scale) {
    bool per_entry = sliced || teams || a.g.n >= AGG_ENTRY_SCALE_MIN_NODES;
    if (const char* env = getenv("COFREE_AGG_ENTRY_SCALE")) per_entry = atoi(env) != 0;
    if (per_entry && a.in_scale == a.g.inv_deg) k.in_vals = a.g.val_inv_deg;
    if (per_entry && a.in_scale == a.g.gcn_norm) k.in_vals = a.g.val_gcn_norm;
  }

  // 1. hub rows
  if (n_hub > 0) {
    k.order = a.g.order;
    k.slot0 = 0;
    k.n = n_hub;
    COFREE_TRY((launch_hub<T, DROP>(k, stream, cost, a.g.nnz_hub)));
  }
  // 2b. every other row, order[n_hub ..)
  if (n_hub == a.g.n) {
    COFREE_HIP_CHECK(hipGetLastError());
    return COFREE_OK;
  }
  k.order = a.g.order;
  k.slot0 = (int32_t)n_hub;
  k.n = a.g.n - n_hub;
  // Graphs of high average degree leave their long rows to a wavefront each where the rows are narrow, so that four
  // wavefronts would find too little to share (115k nodes, 7M entries, 8 bfloat16 columns 1.10 -> 0.99 of the time with a
  // wavefront for every row), and from eight million entries on, where a launch outlasts a row of 4095 neighbours anyway
  // (230k nodes, 14M entries, 41 float32 columns: shared 437 us, a wavefront each 409; 30k nodes, 14M entries, 300 columns 1.09
  // -> 1.00).  Elsewhere the shared rows are what a launch waits for (60k nodes, 2M entries, 128 bfloat16 columns 0.61
  // of that time, 0.81 without; 115k nodes, 7M entries, 41 float32 columns 0.77 and 0.86).
  // (A launch has less than 2^32 work-items: eight million long rows do not need a workgroup each either.)
  const bool share = a.g.n_block < (1 << 23) && (!waves || (a.width > 8 * WIDE && a.g.nnz < (1 << 23)));
  k.n_block = buckets && share ? (int32_t)(a.g.n_block - n_hub) : 0;
  k.n_wave = waves ? (int32_t)(k.n - k.n_block) : (buckets ? (int32_t)(a.g.n_wave - n_hub) - k.n_block : 0);
  // The row kernel walks the processing-order copy of the graph (1.9M-node partition, 512-wide float32: 3.00 ms
  // by row id, 2.8 ms in natural order with its worse balance).  COFREE_AGG_SLOTS = 0 reads by row id.
  bool slots = a.g.order != nullptr && a.g.s_rowptr != nullptr;
  if (const char* env = getenv("COFREE_AGG_SLOTS")) slots = slots && atoi(env) != 0;
  if (slots) {
    k.by_slot = 1;
    k.rowptr = a.g.s_rowptr;
    k.col = a.g.s_col;
    if (k.in_vals) k.in_vals = a.in_scale == a.g.inv_deg ? a.g.s_val_inv_deg : a.g.s_val_gcn_norm;
    if (a.in_scale == a.g.inv_deg) k.in_scale_slot = a.g.s_inv_deg;
    if (a.in_scale == a.g.gcn_norm) k.in_scale_slot = a.g.s_gcn_norm;
    if (a.out_scale == a.g.inv_deg) k.out_scale_slot = a.g.s_inv_deg;
    if (a.out_scale == a.g.gcn_norm) k.out_scale_slot = a.g.s_gcn_norm;
  }
  if (sliced || teams) {
    k.n_block = 0;
    k.n_wave = (int32_t)(std::max(a.g.n_block, n_hub) - n_hub);  // longer rows are never left to a team
    COFREE_TRY((launch_sliced<T, DROP>(k, team_lanes, long_bits, slice_bits, stream, cost, a.g.nnz - hub_nnz)));
    COFREE_HIP_CHECK(hipGetLastError());
    return COFREE_OK;
  }
  // Rows of 65 to 96 pieces leave a quarter to a half of a wavefront's second access without columns.  Where such rows are short and
  // their matrix is beyond the caches, so that a launch waits for its bytes and not for the graph, 64 pieces and the others are two
  // launches: 500k rows of 300 float32, 3 entries each 554 -> 480 us, 250k of 260 (2 entries) 197 -> 163, 250k of 530 bfloat16 (4) 270 ->
  // 230, 500k of 768 (7) 953 -> 851.  From 4 (bfloat16: 8) entries a row on 0.98 to 1.09 (0.85 to 1.03), below 250 (200) MB up to 1.06
  // (150k of 300 float32, 4 entries), on 30k rows 1.07 to 1.23; of 97 to 125 pieces 1.01 to 1.10.
  const bool halves = pieces > 64 && pieces <= 96 && a.width >= 65 * WIDE && a.g.nnz < a.g.n * (sizeof(T) == 4 ? 4 : 8) &&
                      matrix >= (sizeof(T) == 4 ? 250e6 : 200e6);
  const int panel = (halves ? 64 : ROW_PIECES) * WIDE;  // columns one launch covers
  for (int c0 = 0; c0 < a.width; c0 += panel) {
    k.width = a.width - c0 < panel ? a.width - c0 : panel;
    k.col0 = c0;
    k.X = X + c0;
    k.Y = Y + c0;
    k.relu_src = R ? R + c0 : nullptr;
    COFREE_TRY((launch_rows<T, DROP>(k, stream, cost, a.g.nnz - hub_nnz)));
  }
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

// contiguous rows of at least one wide access in every launch (1028 bfloat16 columns leave four to the second)
// Narrow rows of a width that is no multiple of four over many nodes: their lanes, with windows that overlap and a draw more
// each, take longer than a launch that draws once an element (GCN forward, q = 0.3, there / here: bfloat16 10 columns over 400k nodes 99 / 117 us, 18
// over 100k 38 / 42, 23 over 400k 0.99; float32 5 over 400k 76 / 81, 9 0.97; over 20k nodes 0.94 and 0.96).
bool aggregate_drops(const AggArgs& a) {
  if (a.width % 4 != 0 && a.g.n >= 1 << 16 && a.width < (a.dtype == COFREE_F32 ? 8 : 23)) return false;
  const int wide = a.dtype == COFREE_F32 ? RowIO<float>::WIDE : RowIO<bf16_t>::WIDE;
  const int last = a.width % (ROW_PIECES * wide);
  return a.width >= wide && a.ldy == a.width && (last == 0 || last >= wide);
}

int32_t launch_aggregate(const AggArgs& a, hipStream_t stream) {
  COFREE_REQUIRE(a.dtype == COFREE_F32 || a.dtype == COFREE_BF16, "aggregate: unknown dtype");
  COFREE_REQUIRE(a.width >= 1, "aggregate: width must be >= 1");
  COFREE_REQUIRE(a.X && a.Y && a.X != a.Y, "aggregate: X and Y must be distinct non-NULL buffers");
  COFREE_REQUIRE(a.ldx >= a.width && a.ldy >= a.width, "aggregate: leading dimension smaller than width");
  COFREE_REQUIRE(a.g.n < ((int64_t)1 << 31), "aggregate: too many rows");
  COFREE_REQUIRE(!a.add || (!a.relu_src && a.dtype == COFREE_F32), "aggregate: added to in float32, not gated as well");
  COFREE_REQUIRE((a.ldx | a.ldy | a.ld_relu | a.ld_add) < ((int64_t)1 << 32), "aggregate: leading dimension too large");
  if (a.g.n == 0) return COFREE_OK;
  auto typed = [&](auto drop) {
    return a.dtype == COFREE_F32 ? launch_typed<float, decltype(drop)::value>(a, stream) : launch_typed<bf16_t, decltype(drop)::value>(a, stream);
  };
  if (!(a.dropout.q > 0.f)) return typed(std::integral_constant<int, 0>{});
  return a.width % 4 == 0 ? typed(std::integral_constant<int, 1>{}) : typed(std::integral_constant<int, 2>{});
}

}  // namespace cofree

using namespace cofree;

extern "C" int32_t cofree_aggregate(const cofree_partition* part, const cofree_masks* masks, int32_t mask_id,
                                    int32_t mode, const void* X, void* Y, int32_t width, int32_t dtype,
                                    void* stream) {
  AggArgs a;
  COFREE_TRY(select_graph(part, masks, mask_id, &a.g));
  a.X = X;
  a.Y = Y;
  a.width = width;
  a.ldx = a.ldy = width;
  a.dtype = dtype;
  switch (mode) {
    case COFREE_AGG_MEAN: a.out_scale = a.g.inv_deg; break;
    case COFREE_AGG_MEAN_T: a.in_scale = a.g.inv_deg; break;
    case COFREE_AGG_GCN:
      a.in_scale = a.g.gcn_norm;
      a.out_scale = a.g.gcn_norm;
      a.self_loop = 1;
      break;
    default: return fail(COFREE_EINVAL, "aggregate: unknown mode");
  }
  return launch_aggregate(a, (hipStream_t)stream);
}
