// Float32 products with a narrow side on the float32 matrix cores of gfx950: results of at most 64 columns, and weight
// gradients of at most 64 rows or columns.  They read one wide operand once and do little with it, so memory bounds them
// (at 48 columns the matrix units take four fifths of the time that the wide operand takes to arrive; at 64 as long).
//
// Both kernels take operands from memory to the matrix instruction's registers with 16-byte loads and no LDS in between,
// because nothing says which k a lane's element must be as long as both operands agree, nor which column:
//  * C = A op(B)^T: v_mfma_f32_16x16x4 wants element k = lane / 16 of row lane % 16.  A lane loads the four k from
//    4 * (lane / 16) on of its row, and element c of all lanes is one instruction.  Parameters lie in LDS in the order that
//    the instructions read them.  They are the instruction's first operand, which leaves a lane four neighbouring columns
//    of one row of the result: one 16-byte store, no staging.
//    Two products of one matrix are the blocks of columns of one.
//  * C = A^T B over nodes: a lane loads four neighbouring columns of node lane / 16, and element b of all lanes is the
//    operand for the columns 4 i + b; the narrow side likewise, with as many columns per lane as it has blocks of 16.
// Where the last lane's columns would cross the end of a row, its window is moved left to end with the row; the columns
// that it shares with the lane before are computed twice, with the same result.
//
// Before, these shapes went through LDS in tiles of 128 x 128, of which a narrow product used half, with two steps of 16 k in
// flight (gemm.hip).  470k x 47 x 512: 326 -> 254 us (4.1 TB/s), weight gradient 327 -> 274; 300k x 41 x 256: 107 -> 82 and 106 -> 84;
// 20,000 x 33 x 500: 28 -> 20 and 25 -> 22; 64 x 64 over 20,000 nodes 18 -> 12; 2,000 x 16 x 64: 6.6 -> 3.6.
#include <algorithm>
#include <climits>
#include <cstdio>

#include "colsum.h"
#include "common.h"

namespace cofree {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));

constexpr int CUS = 256, LDS_BYTES = 160 * 1024;

// ---- C = epilogue(A1 op(B1)^T + A2 op(B2)^T), at most 64 columns ------------------------------------------------
struct NarrowK {
  const float *A1, *A2, *B1, *B2;
  int64_t lda1, lda2, ldb1, ldb2;
  int32_t K1, K2;  // K2 = 0: one segment
  float* C;
  int64_t ldc, M;
  int32_t N;
  int64_t tiles;      // of 16 rows
  int32_t rounds;     // tiles per wavefront
  int32_t col_waves;  // wavefronts that share a tile, NB blocks of columns each
  int32_t part_steps; // steps of 16 k whose parameters LDS holds
  const float* bias;
  int32_t relu;
  const float* row_scale;
  const float* gate;
  int64_t ldg;
  int32_t accumulate, relu_last, gate_last;
  float gate_scale;
  const float* B_second;  // TWO: the second result, of the blocks of columns from `half` on
  float* C_second;
  int32_t half;
};

// Steps of 16 k that a wavefront has in flight (DEPTH of the kernel): eight, or about as many as the product has, because a
// ring that is too long repeats the last step (33,000 rows x 64 x 64: 9.4 -> 8.1 us with four, 60,000 x 48 x 8 10.7 -> 6.1 with
// two).  Sixteen, and loads of four steps issued together, were no faster.  One says that a segment has fewer than 4 k and is
// read element by element.

// A step's k: segment and first k.  A lane has the four from 4 g on, g its group of 16; where they would cross the end of the
// segment, its last four, of which those that the group before has are zero.
template <bool ELEMENTS>
struct Step {
  bool second;
  int32_t start, len;
  __device__ Step(int t, int n1, int32_t K1, int32_t K2) {
    second = t >= n1;
    start = (second ? t - n1 : t) * 16;
    len = second ? K2 : K1;
  }
  __device__ bool whole() const { return start + 16 <= len; }
  __device__ int32_t first(int g) const {
    const int32_t k = start + 4 * g;
    return ELEMENTS || k < len - 4 ? k : len - 4;
  }
  __device__ bool has(int g, int c) const { return ELEMENTS ? start + 4 * g + c < len : first(g) + c >= start + 4 * g; }
  __device__ int32_t at(int g, int c) const { return ELEMENTS && start + 4 * g + c > len - 1 ? len - 1 : first(g) + c; }
};

// A wavefront computes NB blocks of 16 columns of a tile of 16 rows; several may share a tile (SHARE).  A workgroup keeps
// all parameters in LDS where they fit and walks the row tiles; where they do not, it walks the parts of k for every round
// of tiles.  TWO: two results (an instance of its own: deciding by block cost every product of few rows 0.5 us, 4 % of a small layer).
template <int NB, bool SHARE, bool B_KMAJOR, int DEPTH, bool EXTRAS, bool TWO>
__global__ __launch_bounds__(1024) void narrow_gemm_kernel(const NarrowK p) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  constexpr bool ELEMENTS = DEPTH == 1;
  const int col_waves = SHARE ? p.col_waves : 1, nb = NB * col_waves;
  float* const bias = lds;              // [nb][16], in the order of `column`
  float* const params = lds + nb * 16;  // [step][nb][lane][4]
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b0 = wave % col_waves * NB;  // the wavefront's blocks, all of one result
  const bool second_result = TWO && b0 >= p.half;
  const int own_b0 = second_result ? b0 - p.half : b0;
  float* const C = second_result ? p.C_second : p.C;
  const int row_wave = wave / col_waves, row_waves = (int)(blockDim.x >> 6) / col_waves;
  const int n1 = (p.K1 + 15) / 16, n = n1 + (p.K2 + 15) / 16;

  struct Rows {
    const float *a1, *a2;
  };
  auto tile_of = [&](int round) { return ((int64_t)round * row_waves + row_wave) * gridDim.x + blockIdx.x; };
  auto rows_of = [&](int round) {
    int64_t i = tile_of(round) * 16 + r;
    if (i > p.M - 1) i = p.M - 1;
    return Rows{p.A1 + i * p.lda1, p.K2 ? p.A2 + i * p.lda2 : nullptr};
  };
  auto load = [&](const Rows& rows, int t, float4u& x) {
    const Step<ELEMENTS> s(t < n ? t : n - 1, n1, p.K1, p.K2);
    const float* const a = s.second ? rows.a2 : rows.a1;
    if constexpr (ELEMENTS) {
#pragma unroll
      for (int c = 0; c < 4; ++c) x[c] = a[s.at(g, c)];
    } else {
      x = *reinterpret_cast<const float4u*>(a + s.first(g));
    }
  };
  // output column of row i of the instruction's first operand in block b
  auto column = [&](int b, int i) {
    if (p.N < 4) return i < p.N ? i : p.N - 1;
    const int first = 16 * b + (i & ~3);
    return (first < p.N - 4 ? first : p.N - 4) + (i & 3);
  };
  auto fill = [&](int t0, int t1) {  // parameters of steps t0 .. t1 - 1; a wavefront takes steps of one block of columns
    const int b = wave % nb, every = (int)(blockDim.x >> 6) / nb;
    const bool of_second = TWO && b >= p.half;
    const int64_t j = column(of_second ? b - p.half : b, r);
    const float* const only_B = of_second ? p.B_second : p.B1;  // (two results: of one segment)
    constexpr int BATCH = DEPTH;
    for (int base = t0 + wave / nb; base < t1 && wave < every * nb; base += BATCH * every) {
      float4u v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int t = base + u * every;
        const Step<ELEMENTS> s(t < t1 ? t : t1 - 1, n1, p.K1, p.K2);
        const float* const B = TWO ? only_B : s.second ? p.B2 : p.B1;
        const int64_t ldb = !TWO && s.second ? p.ldb2 : p.ldb1;
        if constexpr (!B_KMAJOR && !ELEMENTS) {
          v[u] = *reinterpret_cast<const float4u*>(B + j * ldb + s.first(g));
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) v[u][c] = B[B_KMAJOR ? s.at(g, c) * ldb + j : j * ldb + s.at(g, c)];
        }
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int t = base + u * every;
        if (t >= t1) break;
        const Step<ELEMENTS> s(t, n1, p.K1, p.K2);
        float4 w;
        w.x = s.has(g, 0) ? v[u][0] : 0.f, w.y = s.has(g, 1) ? v[u][1] : 0.f;
        w.z = s.has(g, 2) ? v[u][2] : 0.f, w.w = s.has(g, 3) ? v[u][3] : 0.f;
        *reinterpret_cast<float4*>(params + (((t - t0) * nb + b) * 64 + lane) * 4) = w;
      }
    }
  };

  // this lane's columns of the result: windows of four, of which the first own[b] belong to the lane before
  int32_t col[NB], own[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int first = 16 * (own_b0 + b) + 4 * g;
    col[b] = p.N < 4 || first < p.N - 4 ? first : p.N - 4;
    own[b] = first - col[b];
  }

  float4u ring[DEPTH];
  Rows rows = rows_of(0);
#pragma unroll
  for (int s = 0; s < DEPTH; ++s) {
    load(rows, s, ring[s]);
    __builtin_amdgcn_sched_barrier(0);  // issued in the order of their use, as the loop assumes where it waits
  }
  floatx4 acc[NB];
  if (tid < nb * 16) bias[tid] = p.bias ? p.bias[column(tid >> 4, tid & 15)] : 0.f;

  // one chunk of DEPTH steps from t0 on; its slots are refilled with the steps from t_next on of rows `next`
  auto chunk = [&](int t0, int part0, const Rows next, int t_next) {
    asm("" : "+s"(t_next));  // or the places of all eight loads are kept in scalar registers across tiles, and spilled
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      const int t = t0 + s;
      float4u& x = ring[s];
      if (t < n) {  // uniform
        const Step<ELEMENTS> st(t, n1, p.K1, p.K2);
        if (!st.whole()) {
#pragma unroll
          for (int c = 0; c < 4; ++c) x[c] = st.has(g, c) ? x[c] : 0.f;
        }
        const float4* const b = reinterpret_cast<const float4*>(params) + ((t - part0) * nb + b0) * 64 + lane;
        float4 w[NB];
#pragma unroll
        for (int q = 0; q < NB; ++q) w[q] = b[64 * q];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int q = 0; q < NB; ++q)
            acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(c == 0 ? w[q].x : c == 1 ? w[q].y : c == 2 ? w[q].z : w[q].w, x[c],
                                                          acc[q], 0, 0, 0);
      }
      load(next, t_next + s, x);  // into the registers just used: anywhere else they would be moved here, and waited for
    }
  };

  bool filled = false;
  for (int round = 0; round < p.rounds; ++round) {
    const int64_t i = tile_of(round) * 16 + r;
    // after the last round the loads go on, from one row for all lanes (left out by a condition, every chunk waits longer: 45,000 rows
    // x 64 x 300 24.6 -> 29.0 us)
    const Rows next = round + 1 < p.rounds ? rows_of(round + 1) : Rows{p.A1, p.A2};
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int part0 = 0; part0 < n; part0 += p.part_steps) {
      const int part1 = part0 + p.part_steps < n ? part0 + p.part_steps : n;
      if (!filled || p.part_steps < n) {  // uniform over the workgroup
        if (filled) __syncthreads();      // the part before is no longer read
        fill(part0, part1);
        // All loads are waited for here (0x0f70: vmcnt(0)).  Left to itself the compiler assumes that some of a batch that was
        // not stored may be outstanding, and waits for everything at the first step of every chunk.
        __builtin_amdgcn_s_waitcnt(0x0f70);
        __syncthreads();
        filled = true;
      }
      if (p.part_steps >= n && tile_of(round) >= p.tiles) return;  // no barrier follows
#pragma nounroll
      for (int t0 = part0; t0 < part1; t0 += DEPTH) {
        const bool last = t0 + DEPTH >= n;
        chunk(t0, part0, Rows{last ? next.a1 : rows.a1, last ? next.a2 : rows.a2}, last ? 0 : t0 + DEPTH);
      }
    }
    rows = next;
    if (i >= p.M) continue;
    // a window of a row of N elements
    auto read = [&](const float* row, int b) {
      if (p.N >= 4) return *reinterpret_cast<const float4u*>(row + col[b]);
      float4u x;
#pragma unroll
      for (int c = 0; c < 4; ++c) x[c] = row[c < p.N ? c : p.N - 1];
      return x;
    };
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (16 * (own_b0 + b) + 4 * g >= p.N) continue;
      floatx4 y = acc[b] + *reinterpret_cast<const floatx4*>(bias + 16 * (b0 + b) + 4 * g);
      if (p.relu) {
#pragma unroll
        for (int c = 0; c < 4; ++c) y[c] = fmaxf(y[c], 0.f);
      }
      if constexpr (EXTRAS) {
        float4u gate = {1.f, 1.f, 1.f, 1.f}, sum = {0.f, 0.f, 0.f, 0.f};
        if (p.gate) gate = read(p.gate + i * p.ldg, b);
        if (p.accumulate) sum = read(C + i * p.ldc, b);
        const float rs = p.row_scale ? p.row_scale[i] : 1.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float x = y[c] * rs;
          const bool shut = !(gate[c] > 0.f);
          if (!p.gate_last) x = shut ? 0.f : x * p.gate_scale;
          x += sum[c];
          if (p.gate_last) x = shut ? 0.f : x * p.gate_scale;
          y[c] = p.relu_last ? fmaxf(x, 0.f) : x;
        }
      }
      float* const dst = C + i * p.ldc + col[b];
      // An element that the launch reads too (accumulated, or its own gate) is written by one lane only.
      if (p.N >= 4 && (own[b] == 0 || !EXTRAS)) {
        *reinterpret_cast<float4u*>(dst) = float4u{y[0], y[1], y[2], y[3]};
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c >= own[b] && col[b] + c < p.N) dst[c] = y[c];
      }
    }
  }
}

struct NarrowShape {
  int nb;            // blocks of 16 columns
  int64_t steps;     // of 16 k
  int64_t most;      // steps whose parameters LDS holds
  int64_t cu_tiles;  // row tiles of a CU
};
static NarrowShape narrow_shape(const GemmArgs& a) {
  NarrowShape s;
  s.nb = (a.N + 15) / 16 * (a.C_second ? 2 : 1);
  s.steps = ((int64_t)a.K1 + 15) / 16 + ((int64_t)a.K2 + 15) / 16;
  s.most = (LDS_BYTES - s.nb * 64) / (s.nb * 1024);
  s.cu_tiles = (a.M + 16 * CUS - 1) / (16 * CUS);
  return s;
}

// At most 64 columns, except, in the tiles of gemm.hip,
//  * parameters beyond LDS by several rounds of row tiles, each of which reads them again: more than 48 columns (90,000 x 64 x 1433
//    222 us here, 185 there; 150,000 332 and 304; in one round, 60,000, 118 and 123), and 33 to 48 in two rounds (90,000 x 41 x 900
//    120 and 111; 150,000 179 and 184)
//  * 49 to 64 columns by 113 to 320 k in one round or little more, where filling LDS and multiplying follow one another
//    (60,000 x 64 x 256 28.4 and 25.5, x 128 17.7 and 16.3; 45,000 x 256 22.8 and 24.9; 150,000 54.2 and 52.5)
bool gemm_narrow_fits(const GemmArgs& a) {
  if (a.N > 64) return false;
  const NarrowShape s = narrow_shape(a);
  if (s.steps > s.most && s.cu_tiles > 16 && (s.nb == 4 || (s.nb == 3 && s.cu_tiles <= 32))) return false;
  return !(s.nb == 4 && s.cu_tiles >= 14 && s.cu_tiles <= 24 && s.steps >= 8 && s.steps <= 20);
}

template <int NB, bool SHARE, bool B_KMAJOR, int DEPTH, bool EXTRAS, bool TWO>
static int32_t launch_narrow(const NarrowK& p, int64_t blocks, int threads, size_t lds, hipStream_t stream) {
  const auto kernel = narrow_gemm_kernel<NB, SHARE, B_KMAJOR, DEPTH, EXTRAS, TWO>;
  if (lds > 64 * 1024)
    COFREE_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                         LDS_BYTES));
  kernel<<<dim3((unsigned)blocks), threads, lds, stream>>>(p);
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

int32_t launch_gemm_narrow(const GemmArgs& a, hipStream_t stream) {
  NarrowK p{};
  p.A1 = (const float*)a.A1;
  p.lda1 = a.lda1;
  p.K1 = a.K1;
  p.A2 = (const float*)a.A2;
  p.lda2 = a.lda2;
  p.K2 = a.K2;
  p.B1 = a.B;
  p.ldb1 = a.ldb;
  if (a.K2 > 0) {
    p.B2 = a.B2 ? a.B2 : a.B + (a.b_kmajor ? (int64_t)a.K1 * a.ldb : (int64_t)a.K1);
    p.ldb2 = a.B2 ? a.ldb2 : a.ldb;
  }
  p.C = (float*)a.C;
  p.ldc = a.ldc;
  p.M = a.M;
  p.N = a.N;
  p.bias = a.bias;
  p.relu = a.relu;
  p.row_scale = a.row_scale;
  p.gate = (const float*)a.gate;
  p.ldg = a.ldg;
  p.accumulate = a.accumulate;
  p.relu_last = a.relu_last;
  p.gate_last = a.gate_last;
  p.gate_scale = a.gate ? a.gate_scale : 1.f;
  p.B_second = a.B_second;
  p.C_second = (float*)a.C_second;
  p.tiles = (a.M + 15) / 16;
  const auto [nb, steps, most, cu_tiles] = narrow_shape(a);
  p.half = nb / 2;
  const int depth = a.K1 < 4 || (a.K2 > 0 && a.K2 < 4) ? 1 : steps <= 2 ? 2 : steps <= 4 ? 4 : 8;
  p.part_steps = (int32_t)(steps <= most ? steps : most / depth * depth);
  const size_t lds = (size_t)p.part_steps * nb * 1024 + nb * 64;
  // A wavefront takes all columns of a row tile, workgroups as many row tiles as their CU has, up to 16.  With so few tiles that
  // every block of columns can have a wavefront of its own it gets one: the chain of matrix instructions on one tile is what
  // the launch waits for.  Five and six tiles of four blocks, which would lie unevenly on four SIMDs, are cut in two (20,000 x 64 x
  // 602: 38 us in five wavefronts, 30 in ten).  Always 16 tiles left CUs without a workgroup (33,000 x 48 x 64 11.7 -> 8.3 us).
  // Two results are two wavefronts' at least.
  p.col_waves = cu_tiles * nb <= 16 ? nb : a.C_second || (nb == 4 && cu_tiles <= 6 && depth == 8) ? 2 : 1;
  const int cols = nb / p.col_waves;  // blocks of columns a wavefront
  const int row_waves = (int)std::min<int64_t>(std::max<int64_t>(cu_tiles, (3 + p.col_waves) / p.col_waves), 16 / p.col_waves);
  const int waves = row_waves * p.col_waves;
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(16 / waves, (int64_t)(LDS_BYTES / lds)));
  const int64_t blocks = std::min<int64_t>((p.tiles + row_waves - 1) / row_waves, CUS * per_cu);
  const int64_t rounds = (p.tiles + blocks * row_waves - 1) / (blocks * row_waves);
  COFREE_REQUIRE(rounds < INT_MAX, "dense: too many rows");
  p.rounds = (int32_t)rounds;
  const bool extras = a.gate || a.accumulate || a.row_scale || a.relu_last;
  const double K = (double)a.K1 + a.K2, results = a.C_second ? 2.0 : 1.0;
  char pname[96] = "";  // the template instance launched below, then the shape
  if (profiling()) snprintf(pname, sizeof(pname), "narrow_gemm_kernel<%d,%s,%s,%d,%s,%s> N=%d K=%lld", cols, cols == 1 || p.col_waves > 1 ? "true" : "false", a.b_kmajor ? "true" : "false",
                            depth, extras ? "true" : "false", a.C_second ? "true" : "false", (int)a.N, (long long)K);
  ProfScope prof(pname, stream, 4.0 * ((double)a.M * K + results * ((double)a.N * K + (double)a.M * a.N * (a.accumulate ? 2 : 1))),
                 2.0 * results * (double)a.M * a.N * K);
  auto by_depth = [&](auto n, auto share, auto kmajor) {
    constexpr int NB = decltype(n)::value;
    constexpr bool SHARE = decltype(share)::value, KMAJOR = decltype(kmajor)::value;
    auto go = [&](auto d) {
      constexpr int DEPTH = decltype(d)::value;
      if constexpr (SHARE && !KMAJOR)
        if (a.C_second) return launch_narrow<NB, SHARE, KMAJOR, DEPTH, false, true>(p, blocks, 64 * waves, lds, stream);
      if constexpr (NB == 2 && SHARE && DEPTH < 8) return fail(COFREE_EINVAL, "internal: no narrow product of this shape");
      else
        return extras ? launch_narrow<NB, SHARE, KMAJOR, DEPTH, true, false>(p, blocks, 64 * waves, lds, stream)
                      : launch_narrow<NB, SHARE, KMAJOR, DEPTH, false, false>(p, blocks, 64 * waves, lds, stream);
    };
    if constexpr (NB == 2 && SHARE && KMAJOR) {
      return go(std::integral_constant<int, 8>{});
    } else {
      switch (depth) {
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 4: return go(std::integral_constant<int, 4>{});
        default: return go(std::integral_constant<int, 8>{});
      }
    }
  };
  auto by_order = [&](auto n, auto share) {
    return a.b_kmajor ? by_depth(n, share, std::true_type{}) : by_depth(n, share, std::false_type{});
  };
  const std::true_type shared{};
  const std::false_type alone{};
  switch (cols) {
    case 1: return by_order(std::integral_constant<int, 1>{}, shared);
    case 2: return p.col_waves == 2 ? by_order(std::integral_constant<int, 2>{}, shared) : by_order(std::integral_constant<int, 2>{}, alone);
    case 3: return by_order(std::integral_constant<int, 3>{}, alone);
    default: return by_order(std::integral_constant<int, 4>{}, alone);
  }
}

// ---- C = A^T [B | B2] over nodes, at most 64 rows or columns -----------------------------------------------------
struct NarrowWgradK {
  const float *wide1, *wide2, *narrow;  // columns of the wide side: n_wide1 of wide1, then n_wide2 of wide2
  int64_t ldw1, ldw2, ldn;
  int32_t n_wide1, n_wide2, n_narrow;
  int32_t panels1, panels;  // of 16 * NA columns, of wide1 and in all
  int64_t M, chunk;         // nodes, nodes per chunk
  int64_t n_chunks;
  int32_t rows_narrow;      // the narrow side is the rows of the result (operand A)
  float* part;              // [chunks][N1][N2]
  float* colsum_part;       // [chunks][N1] column sums of operand A, or null
  ColsumK extra;
};

// Two weight gradients of one kernel instance in one launch, the second's workgroups behind the first's: a launch less, and the
// first's last round is filled (19,717 nodes, two of 33 x 500: 43 -> 37 us, two of 3 x 33 9.5 -> 6.0; 230k nodes, two of 41 x
// 256: 139 -> 127).
struct NarrowPairK {
  NarrowWgradK job[2];
  uint32_t first_blocks;
};

template <int N>
struct Cols {
  float v[N];
};
template <int N>
__device__ inline void load_cols(const float* s, Cols<N>& x) {
  if constexpr (N == 4) {
    const float4u t = *reinterpret_cast<const float4u*>(s);
#pragma unroll
    for (int c = 0; c < 4; ++c) x.v[c] = t[c];
  } else if constexpr (N == 2) {
    const float2u t = *reinterpret_cast<const float2u*>(s);
    x.v[0] = t[0], x.v[1] = t[1];
  } else {
#pragma unroll
    for (int c = 0; c < N; ++c) x.v[c] = s[c];
  }
}
// first column of lane i's window of N in a row of n columns from `first` on, and which lane and element hold a column
template <int N>
__device__ inline int window(int first, int i, int n) {
  const int c = first + N * i;
  return c < n - N ? c : n - N;
}

// A workgroup of four wavefronts sums one chunk of nodes for one panel of the wide side: 16 * NA of its columns by all of the
// narrow side, 16 * NB at most.  Wavefronts take groups of 32 nodes in turn, eight steps of four nodes in flight, and their
// sums are added in wavefront order through LDS.
constexpr int WSTEPS = 8, WGROUP = 4 * WSTEPS;
template <int NA, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NB == 4 ? 2 : 3))) void narrow_wgrad_kernel(const NarrowPairK two) {
  // padded: lanes read down a column of it, with 16 * NB from as few as one bank (64 x 64 over 2,000 nodes 16.6 -> 10.3 us)
  constexpr int LD = 16 * NB + 4;
  __shared__ __attribute__((aligned(16))) float sums[4][NA * 16 * LD];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int which = blockIdx.x >= two.first_blocks;
  const NarrowWgradK& p = two.job[which];
  const int64_t L = blockIdx.x - (which ? two.first_blocks : 0u), 
                blocks = which ? gridDim.x - two.first_blocks : two.first_blocks;
  if (L >= blocks - p.extra.blocks) {
    colsum_block<float>(p.extra, L - (blocks - p.extra.blocks), &sums[0][0], tid);
    return;
  }
  // the panels of a chunk are neighbours on one XCD (ids congruent mod 8), whose L2 then holds the narrow side's rows
  const int64_t z = L / (8 * p.panels) * 8 + (L & 7);
  if (z >= p.n_chunks) return;
  const int panel = (int)((L >> 3) % p.panels);
  const bool second = panel >= p.panels1;
  const int c0 = (second ? panel - p.panels1 : panel) * (16 * NA);  // first column of the panel
  const int n_wide = second ? p.n_wide2 : p.n_wide1;
  const int64_t k_beg = z * p.chunk, k_end = k_beg + p.chunk < p.M ? k_beg + p.chunk : p.M;
  const int len = (int)(k_end - k_beg);
  const int64_t ldw = second ? p.ldw2 : p.ldw1;
  const float* const wide = (second ? p.wide2 : p.wide1) + k_beg * ldw + window<NA>(c0, r, n_wide);
  const float* const narrow = p.narrow + k_beg * p.ldn + window<NB>(0, r, p.n_narrow);

  floatx4 acc[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int CS = NA > NB ? NA : NB;
  float csum[CS] = {};
  const bool do_colsum = p.colsum_part != nullptr && (!p.rows_narrow || panel == 0);
  Cols<NA> w[WSTEPS];
  Cols<NB> x[WSTEPS];
  auto load = [&](int k0, int s) {  // nodes past the chunk repeat its last one
    int k = k0 + 4 * s + g;
    if (k > len - 1) k = len - 1;
    load_cols<NA>(wide + (int64_t)k * ldw, w[s]);
    load_cols<NB>(narrow + (int64_t)k * p.ldn, x[s]);
  };
  int k0 = wave * WGROUP;
  if (k0 < len) {
#pragma unroll
    for (int s = 0; s < WSTEPS; ++s) {
      load(k0, s);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (; k0 < len; k0 += 4 * WGROUP) {
      float group[CS] = {};  // column sums of this group, so that csum is rounded once for it
#pragma unroll
      for (int s = 0; s < WSTEPS; ++s) {
        Cols<NA>& u = w[s];
        Cols<NB>& v = x[s];
        if (k0 + WGROUP > len) {
          const bool in = k0 + 4 * s + g < len;
#pragma unroll
          for (int a = 0; a < NA; ++a) u.v[a] = in ? u.v[a] : 0.f;
#pragma unroll
          for (int b = 0; b < NB; ++b) v.v[b] = in ? v.v[b] : 0.f;
        }
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(u.v[a], v.v[b], acc[a][b], 0, 0, 0);
        if (do_colsum) {
          if (p.rows_narrow) {
#pragma unroll
            for (int b = 0; b < NB; ++b) group[b] += v.v[b];
          } else {
#pragma unroll
            for (int a = 0; a < NA; ++a) group[a] += u.v[a];
          }
        }
        load(k0 + 4 * WGROUP, s);  // into the registers just used
      }
#pragma unroll
      for (int c = 0; c < CS; ++c) csum[c] += group[c];
    }
  }
  // register v of lane (g, r) is row 4 g + v, column r of its block
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) sums[wave][((4 * g + v) * NA + a) * LD + r * NB + b] = acc[a][b][v];
  __syncthreads();
  // the column that element `place` of the windows holds, or -1 where the lane before has it
  auto column = [](int n, int first, int place, int N) {
    const int own = first + place / N * N, c = (own < n - N ? own : n - N) + place % N;
    return c >= own ? c : -1;
  };
  const int n_all = p.n_wide1 + p.n_wide2, at = second ? p.n_wide1 : 0;
  float* const part = p.part + z * (int64_t)n_all * p.n_narrow;
  // The partial sums of the four wavefronts, by lanes along the rows of the result.
  if (p.rows_narrow) {
    const int cw = lane < 16 * NA ? column(n_wide, c0, lane, NA) : -1;
    if (cw >= 0) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int e = 4 * (4 * j + wave);
        floatx4 t = *reinterpret_cast<const floatx4*>(&sums[0][lane * LD + e]);
#pragma unroll
        for (int s = 1; s < 4; ++s) t += *reinterpret_cast<const floatx4*>(&sums[s][lane * LD + e]);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int cn = column(p.n_narrow, 0, e + c, NB);
          if (cn >= 0) part[(int64_t)cn * n_all + at + cw] = t[c];
        }
      }
    }
  } else {
    constexpr int ROWS = 64 / (16 * NB);  // of the result, a wavefront at a time
    const int cn = lane < ROWS * 16 * NB ? column(p.n_narrow, 0, lane % (16 * NB), NB) : -1;
    if (cn >= 0) {
#pragma unroll
      for (int j = 0; j < 16 * NA / (4 * ROWS); ++j) {
        const int o = (4 * j + wave) * ROWS + lane / (16 * NB), e = o * LD + lane % (16 * NB);
        const int cw = column(n_wide, c0, o, NA);
        if (cw >= 0) part[(int64_t)(at + cw) * p.n_narrow + cn] = ((sums[0][e] + sums[1][e]) + sums[2][e]) + sums[3][e];
      }
    }
  }
  if (do_colsum) {
    __syncthreads();
    const int N = p.rows_narrow ? NB : NA;
    float* const lds = &sums[0][0];  // [wave][g][column]
#pragma unroll
    for (int c = 0; c < CS; ++c)
      if (c < N) lds[(wave * 4 + g) * 16 * N + r * N + c] = csum[c];
    __syncthreads();
    const int N_all = 16 * N;
    if (tid < N_all) {
      const int c = p.rows_narrow ? column(p.n_narrow, 0, tid, NB) : column(n_wide, c0, tid, NA);
      float t = 0.f;
      for (int s = 0; s < 16; ++s) t += lds[s * N_all + tid];
      if (c >= 0) p.colsum_part[z * (p.rows_narrow ? p.n_narrow : n_all) + (p.rows_narrow ? c : at + c)] = t;
    }
  }
}

bool wgrad_narrow_fits(int32_t N1, int32_t first, int32_t N2b) { return N1 <= 64 || (N2b == 0 && first <= 64); }

struct NarrowPlan {
  bool rows_narrow;
  int na, nb, panels1, panels;
  int64_t chunk, chunks;
};
static NarrowPlan plan_narrow(int32_t N1, int32_t first, int32_t N2b, int64_t M) {
  NarrowPlan q;
  q.rows_narrow = N2b > 0 || N1 <= first;
  const int narrow = q.rows_narrow ? N1 : first, wide = q.rows_narrow ? first : N1;
  q.na = wide < 4 || (N2b > 0 && N2b < 4) ? 1 : 4;
  q.nb = (narrow + 15) / 16;
  q.panels1 = (wide + 16 * q.na - 1) / (16 * q.na);
  q.panels = q.panels1 + (N2b + 16 * q.na - 1) / (16 * q.na);
  // One round of the workgroups that the chip holds, at least a group of nodes for every wavefront.  Panels that read the same
  // narrow rows drift apart on a long walk and read them again: with four blocks of columns and more than four panels, chunks of
  // more than 768 nodes are cut up to four times (64 x 602 over 150,000 nodes 163 -> 134 us, 64 x 300 88 -> 68; not where chunks are
  // short, 64 x 602 over 20,000 29 -> 32, nor with three blocks, 33 x 500 over 300,000 167 -> 179), and long reductions get more chunks.
  const int64_t resident = CUS * (q.nb == 4 ? 2 : 3), one = std::max<int64_t>(1, resident / q.panels);
  const int64_t rounds = q.nb == 4 && q.panels > 4 ? std::min<int64_t>(std::max<int64_t>((M + 768 * one - 1) / (768 * one), 1), 4) : 1;
  const int64_t s = std::max<int64_t>(std::max<int64_t>(1, resident * rounds / q.panels), std::min<int64_t>(M / 16384, 2048));
  const int64_t whole = 4 * WGROUP;
  q.chunk = std::max<int64_t>(1, ((M + s - 1) / s + whole - 1) / whole) * whole;
  q.chunks = std::max<int64_t>(1, (M + q.chunk - 1) / q.chunk);
  return q;
}

size_t wgrad_narrow_workspace_floats(int32_t N1, int32_t first, int32_t N2b, int64_t M) {
  if (!wgrad_narrow_fits(N1, first, N2b)) return 0;
  return (size_t)plan_narrow(N1, first, N2b, M).chunks * ((size_t)N1 * ((size_t)first + N2b) + N1);
}

template <int NA, int NB>
static int32_t launch_narrow_wgrad(const NarrowPairK& p, int64_t blocks, hipStream_t stream) {
  narrow_wgrad_kernel<NA, NB><<<dim3((unsigned)blocks), 256, 0, stream>>>(p);
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

static int32_t fill_narrow(const WgradArgs& a, const NarrowPlan& q, NarrowWgradK* job, int64_t* blocks, SplitSums* sums) {
  const int32_t N2b = a.B2 ? a.N2b : 0, N1 = a.N1, N2 = a.N2 + N2b;
  NarrowWgradK p{};
  p.rows_narrow = q.rows_narrow;
  p.narrow = (const float*)(q.rows_narrow ? a.A : a.B);
  p.ldn = q.rows_narrow ? a.lda : a.ldb;
  p.n_narrow = q.rows_narrow ? N1 : a.N2;
  p.wide1 = (const float*)(q.rows_narrow ? a.B : a.A);
  p.ldw1 = q.rows_narrow ? a.ldb : a.lda;
  p.n_wide1 = q.rows_narrow ? a.N2 : N1;
  p.wide2 = (const float*)a.B2;
  p.ldw2 = a.ldb2;
  p.n_wide2 = N2b;
  p.panels1 = q.panels1;
  p.panels = q.panels;
  p.M = a.M;
  p.chunk = q.chunk;
  p.n_chunks = q.chunks;
  p.part = a.workspace;
  float* const colsum_part = a.workspace + (size_t)q.chunks * N1 * N2;
  p.colsum_part = a.colsum_out && !a.colsum_src ? colsum_part : nullptr;
  COFREE_TRY(plan_colsum(a, &p.extra, sums));
  *blocks = (q.chunks + 7) / 8 * 8 * q.panels + p.extra.blocks;
  COFREE_REQUIRE(q.chunk < INT_MAX - WGROUP * 8 && *blocks < INT_MAX / 2, "wgrad: too many rows");
  *job = p;
  COFREE_TRY(add_split_sum(sums, a.workspace, (int64_t)N1 * N2, (int32_t)q.chunks, a.C, a.ldc, N1, N2));
  if (p.colsum_part) COFREE_TRY(add_split_sum(sums, colsum_part, N1, (int32_t)q.chunks, a.colsum_out, N1, 1, N1));
  return COFREE_OK;
}

static bool narrow_wgrad(const WgradArgs& a) {
  return a.dtype == COFREE_F32 && wgrad_narrow_fits(a.N1, a.N2, a.B2 ? a.N2b : 0);
}
bool wgrads_pair(const WgradArgs& a, const WgradArgs& b) {
  if (!narrow_wgrad(a) || !narrow_wgrad(b) || a.M != b.M) return false;
  const NarrowPlan q = plan_narrow(a.N1, a.N2, a.B2 ? a.N2b : 0, a.M), r = plan_narrow(b.N1, b.N2, b.B2 ? b.N2b : 0, b.M);
  return q.na == r.na && q.nb == r.nb;
}

int32_t launch_wgrad_narrow(const WgradArgs& a, const WgradArgs* b, SplitSums* sums, hipStream_t stream) {
  const NarrowPlan q = plan_narrow(a.N1, a.N2, a.B2 ? a.N2b : 0, a.M);
  NarrowPairK p{};
  int64_t first = 0, second = 0;
  COFREE_TRY(fill_narrow(a, q, &p.job[0], &first, sums));
  if (b) COFREE_TRY(fill_narrow(*b, plan_narrow(b->N1, b->N2, b->B2 ? b->N2b : 0, b->M), &p.job[1], &second, sums));
  p.first_blocks = (uint32_t)first;
  const int64_t blocks = first + second;
  auto bytes = [](const WgradArgs& w, const NarrowWgradK& j) {
    const double N1 = w.N1, N2 = (double)w.N2 + (w.B2 ? w.N2b : 0), M = (double)w.M;
    return 4.0 * (M * N1 * (j.extra.X ? 2 : 1) + M * N2 + N1 * N2);
  };
  auto flops = [](const WgradArgs& w) { return 2.0 * (double)w.M * w.N1 * ((double)w.N2 + (w.B2 ? w.N2b : 0)); };
  char pname[96] = "";
  if (profiling()) snprintf(pname, sizeof(pname), "narrow_wgrad_kernel<%d,%d> N=%dx%d%s", q.na, q.nb, (int)a.N1,
                            (int)(a.N2 + (a.B2 ? a.N2b : 0)), b ? " and another" : "");
  ProfScope prof(pname, stream, bytes(a, p.job[0]) + (b ? bytes(*b, p.job[1]) : 0.0), flops(a) + (b ? flops(*b) : 0.0));
  switch (q.na * 8 + q.nb) {
    case 9: return launch_narrow_wgrad<1, 1>(p, blocks, stream);
    case 10: return launch_narrow_wgrad<1, 2>(p, blocks, stream);
    case 11: return launch_narrow_wgrad<1, 3>(p, blocks, stream);
    case 12: return launch_narrow_wgrad<1, 4>(p, blocks, stream);
    case 33: return launch_narrow_wgrad<4, 1>(p, blocks, stream);
    case 34: return launch_narrow_wgrad<4, 2>(p, blocks, stream);
    case 35: return launch_narrow_wgrad<4, 3>(p, blocks, stream);
    default: return launch_narrow_wgrad<4, 4>(p, blocks, stream);
  }
}

}  // namespace cofree
