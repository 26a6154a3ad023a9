// Float32 products of the layers on the bfloat16 matrix cores, with float32 operands, sums and results.
//
// A float32 has 24 significant bits and a bfloat16 eight, so a float32 is the sum of three bfloat16: x = h + m + l with
// h = bf16(x), m = bf16(x - h), l = x - h - m (both differences are exact in float32, and the second has at most eight
// bits left).  A product of two float32 is then nine products of bfloat16, each exact in float32; the six that reach
// 2^-24 of it (l h, h l, m m, m h, h m, h h) are summed in float32 - the three-way split of Henry, Tang and Heinecke
// ("Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations", ARITH 2019).  What is
// left out is below 2^-23 of a product at worst and around 2^-27 of it on average, less than the rounding of the
// running sum.
//
// Which shapes: results of more than 64 columns (weight gradients: more than 64 rows and columns) and ranges of at
// least eight k; two products or weight gradients of one matrix as the columns or rows of one (TWO).  Narrower ones are bound by their
// bytes and stay on the float32 instructions (gemm_narrow.hip).
//
// Rounding: every matrix instruction rounds its accumulator once.  h h has one of its own and the five products below it
// another, which is about 2^-8 of the first, so that its rounding does not show; the two are added at the end.  The sum
// is then rounded once per 16 k, where the float32 instructions round it once per pair of k - but only for pairs that
// are not zero: features and gated gradients may be sparse, and with all six products in one accumulator results came
// out up to twice as far from float64 as with float32 instructions.  Error against float64 relative to the result,
// float32 instructions / one accumulator / two: 88k x 512 x 512 4.0e-7 / 3.4e-7 / 1.3e-7, with half of operand A zero
// 2.9e-7 / 3.3e-7 / 9.8e-8, with nine tenths zero 1.3e-7 / 2.3e-7 / 5.2e-8; weight gradients of the same operands
// 4.6e-7 / 4.1e-7 / 1.8e-7, 2.4e-7 / 3.6e-7 / 1.3e-7 and 1.1e-7 / 1.4e-7 / 1.0e-7.
//
// What bounds it: a 32x32x16 bfloat16 matrix instruction takes 32 cycles, eight 32x32x2 float32 ones 512, so six of
// the former could be 2.7 times as fast; but a loop of nothing but matrix instructions on random data already lowers
// the shader clock from 2.4 to 1.7 GHz (1,760 TFLOP/s in bfloat16, 1,500 with the vector instructions of a split in
// between): for such a loop power, not issue slots, is the limit.  Here matrix units are busy 58 % of the cycles at 1.77 GHz in A B^T, 56 % at
// 1.86 in weight gradients, 47 % at 1.91 in gated A B (512 x 512 over 1.87M rows): the clock is lowered, but matrix instructions take 1.03,
// 1.04 and 0.90 of its 1.7 GHz, so something else is waited for too, most of all in A B.  Candidates, not measured apart: the first
// steps and the end of a tile (A B asks for its gates there), 12 LDS reads for 24 matrix instructions, and the left operand's
// split, which every column tile repeats.  In TFLOP/s of the product, float32
// instructions / the steps read from LDS behind each barrier / now: 470k x 512 x 512 127 / 169 / 189 (A B^T), 529k x 512 x 1024
// 134 / 187 / 200, 230k x 256 x 602 118 / 131 / 152; weight gradients 512 x 512 over 470k nodes - / 165 / 186.
//
// Tiling: 128x128 of the result per workgroup, four wavefronts 2x2 of 64x64 each (128 accumulators: two sets of four
// 32x32 blocks), two workgroups per CU; see run_split for the pipeline.  One set of accumulators leaves room for
// 128x256 tiles, but rounds more often; two sets in such tiles were no faster with one wavefront per SIMD or with eight
// wavefronts in one workgroup.  Nor were 512 workgroups that take tiles in turn and request the next one's first step before
// they write the last (470k x 512 x 512 1285 -> 1400 us), nor a second step of a row operand in flight (0.97 to 1.09 of the time).
// Results of few tiles: gemm_split_few_kernel.
//
// LDS plane of an operand of 128 rows: [k-group of 8][row][8 bfloat16].  A matrix operand - 8 consecutive k of 32
// consecutive rows per half wavefront - is then 512 contiguous bytes.  Neighbouring rows are swapped in every other
// group of eight and the second k-group is 64 bytes further than its rows take, so that all ways of filling a plane
// (eight lanes = four rows of both k-groups, every row or every other row of one) write 128 distinct bytes: no bank
// conflicts by the counter.
//
// Non-finite values: an infinity (or a magnitude that rounds to one in bfloat16) makes x - h, and with it every
// result it reaches, NaN.  A wavefront that finds a non-finite result in a 32x32 block computes the block again with
// float32 matrix instructions, which treat infinities and NaN as IEEE arithmetic does.
// Small values: bfloat16 ends at 2^-133, so a float32 below 2^-110 is not the sum of three.  What is lost is below 2^-134
// and does not matter beside larger values; a workgroup that finds a row of an operand all below 2^-95 (in a thread's
// share of it), and not zero, computes its whole tile again.
// Both cost time where they happen: 230k x 256 x 602 0.57 ms in turn with others of its kind, with a NaN in one column of
// B 1.13, with one in every tile of A 1.18 (float32 instructions 0.68 and 0.77).  Looking for small rows costs 1-2 %.
#include <climits>
#include <cstdio>
#include <type_traits>

#include "colsum.h"
#include "common.h"

namespace cofree {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t uint32x4 __attribute__((ext_vector_type(4)));

constexpr int SBK = 16;  // k per step: one matrix instruction deep

struct SplitK {
  const float* A1;
  const float* A2;
  const float* B1;
  const float* B2;
  int64_t lda1, lda2, ldb1, ldb2;
  int64_t K1, K2;  // lengths of the two k-segments (K2 = 0: one); weight gradients: K1 = all nodes
  float* C;
  int64_t ldc;
  int64_t M;
  int32_t N;
  int64_t k_chunk;         // weight gradients: nodes per chunk
  int64_t c_split_stride;  // weight gradients: floats between the chunks' partials
  int32_t tiles_m, tiles_n;
  int64_t n_groups;
  int32_t n_split;     // weight gradients: columns n_split .. of the result come from B2 (0: all from B1)
  float* colsum_part;  // weight gradients: [chunks][M] partial column sums of operand A, or null
  int32_t colsum_f64;  // ... in float64 inside a chunk
  ColsumK extra;       // weight gradients: workgroups behind the others that sum columns of another matrix
  const float* bias;
  int32_t relu;
  const float* row_scale;
  const float* gate;
  int64_t ldg;
  int32_t accumulate, relu_last, gate_last;
  float gate_scale;
  DropoutK drop;
  const unsigned char* planes;  // parameters split beforehand: [column tile][step][STEP_IMAGE]
  const uint32_t* small_params; // [column tile][step]: they are to be computed again (see below)
  // second result (TWO): the columns from `half` on are those of A B_second^T, B1 = B_second + b_offset, stored at C_second;
  // second weight gradient: the rows from `half` on are those of A2^T B
  const float* B_second;
  float* C_second;
  int64_t b_offset;
  int32_t half;
};

constexpr int TILE = 128;                 // rows and columns of a workgroup's result
constexpr int PLANE_KG = TILE * 16 + 64;  // bytes of a k-group
constexpr int PLANE = 2 * PLANE_KG;       // bytes of a plane (16 k)
constexpr int OPERAND = 3 * PLANE;        // the three planes of an operand
constexpr int STAGE = 2 * OPERAND;        // a step of both operands
constexpr int STEP_IMAGE = 3 * TILE * 32;  // a step of parameters split beforehand: three planes of [k-group][row][8]
__device__ inline int plane_row(int row) { return (row ^ ((row >> 3) & 1)) * 16; }

// x0, x1 -> their high, middle and low parts, packed (x0 in the low half of each dword)
__device__ inline void split_pair(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = pack_bf16x2(x0, x1);
  const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
  m = pack_bf16x2(r0, r1);
  const float s0 = r0 - __uint_as_float(m << 16), s1 = r1 - __uint_as_float(m & 0xffff0000u);
  l = pack_bf16x2(s0, s1);
}

// Eight consecutive k of one row, split: a thread's share of a step on its way to LDS.
struct Group {
  uint32x4 h, m, l;
  __device__ void pair(int q, float x0, float x1) {
    uint32_t a, b, c;
    split_pair(x0, x1, a, b, c);
    h[q] = a, m[q] = b, l[q] = c;
  }
  __device__ void write(unsigned char* d, int plane) const {
    *reinterpret_cast<uint32x4*>(d) = h;
    *reinterpret_cast<uint32x4*>(d + plane) = m;
    *reinterpret_cast<uint32x4*>(d + 2 * plane) = l;
  }
};

// ---- operand movers: 128 rows x 16 k of an operand from memory to registers to LDS -----------------------------
// A thread's share is eight consecutive k of one row.  Loads are unconditional vector loads at a block-uniform base plus a
// constant 32-bit offset per thread.  Rows past the matrix edge repeat its last row (they feed results that are never
// stored).  A range that is not whole steps ends with the window of its last 16 k, of which the ones that the step before
// had are zero on the way to LDS (ONLY_PART).  In a range of less than one step the second group of eight is the range's last
// eight, of which the ones that the first group has are zero; fewer than eight k are read at clamped places.

// Of the eight places from kq on that a thread has in a step's window, those that count: lo <= place < hi.  start: the k of
// place 0, but in short ranges the thread's places start at short_first.
struct Window {
  int start, lo, hi;
};
__device__ inline Window window_of(int t, int k_len, int kq) {
  const int k0 = t * SBK, last = k_len - SBK;
  if (last < 0) return k_len < 8 ? Window{0, 0, k_len} : Window{0, kq == 0 ? 0 : 24 - k_len, SBK};
  const int start = k0 < last ? k0 : last;
  return Window{start, k0 - start, SBK};
}
__device__ inline int short_first(int k_len, int kq) { return k_len >= 8 && kq > k_len - 8 ? k_len - 8 : kq; }

// the bits that are set in any of four values
__device__ inline uint32_t any_bit(float a, float b, float c, float d) {
  return __float_as_uint(a) | __float_as_uint(b) | __float_as_uint(c) | __float_as_uint(d);
}
// From the bits set in any of them: values that are below 2^-95, all of them, and not all zero (2^-95 has the lowest
// exponent with one of its three upper bits set).
__device__ inline bool all_small(uint32_t bits) { return (bits & 0x70000000u) == 0u && (bits & 0x7fffffffu) != 0u; }

// k-contiguous source: thread t holds k-group t%2 of row t/2
struct SplitKContig {
  struct Raw {
    float4u x[2];
  };
  const char* base;
  uint32_t off;  // bytes to the thread's group of the first step
  int kq, k_len;
  __device__ void init(const float* P, int64_t ld, int64_t extent, int64_t i0, int64_t k_len_, int tid) {
    base = reinterpret_cast<const char*>(P + i0 * ld);
    kq = (tid & 1) * 8;
    k_len = (int)k_len_;
    const int64_t last = extent - 1 - i0, r = tid >> 1;
    off = (uint32_t)(r < last ? r : last) * (uint32_t)ld * 4u + (k_len < SBK ? 0u : (uint32_t)kq * 4u);
  }
  // rows of two matrices: the first `half` begin at P + offset, the others at P
  __device__ void init_two(const float* P, int64_t offset, int32_t half, int64_t ld, int64_t extent, int64_t i0, int64_t k_len_, int tid) {
    base = reinterpret_cast<const char*>(P);
    kq = (tid & 1) * 8;
    k_len = (int)k_len_;
    const int64_t last = extent - 1, r = i0 + (tid >> 1) < last ? i0 + (tid >> 1) : last;
    off = (uint32_t)((r < half ? offset + r * ld : (r - half) * ld) * 4) + (k_len < SBK ? 0u : (uint32_t)kq * 4u);
  }
  __device__ void load(int t, Raw& w) const {
    const char* const p = base + (int64_t)window_of(t, k_len, 0).start * 4;
    w.x[0] = *reinterpret_cast<const float4u*>(p + off);
    w.x[1] = *reinterpret_cast<const float4u*>(p + off + 16u);
  }
  __device__ void load_short(Raw& w) const {  // 8 <= k_len < 16
    const char* const p = base + (off + (uint32_t)short_first(k_len, kq) * 4u);
    w.x[0] = *reinterpret_cast<const float4u*>(p);
    w.x[1] = *reinterpret_cast<const float4u*>(p + 16);
  }
  __device__ float value(const Window& in, int c, const Raw& w) const {
    return kq + c >= in.lo && kq + c < in.hi ? w.x[c >> 2][c & 3] : 0.f;
  }
  // the q-th pair of the share; ODD: with the other sign in odd rows
  template <bool ODD, bool ONLY_PART>
  __device__ void pair(int q, int tid, int t, const Raw& w, uint32_t, Group& g) const {
    const uint32_t flip = ODD ? (uint32_t)tid << 30 & 0x80000000u : 0u;
    const Window in = window_of(t, k_len, kq);
    float e[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = 2 * q + i;
      e[i] = __uint_as_float(__float_as_uint(ONLY_PART ? value(in, c, w) : w.x[c >> 2][c & 3]) ^ flip);
    }
    g.pair(q, e[0], e[1]);
  }
  __device__ static void write(unsigned char* lds, int tid, const Raw&, const Group& g) {
    g.write(lds + (tid & 1) * PLANE_KG + plane_row(tid >> 1), PLANE);
  }
  __device__ static uint32_t bits(const Raw& w) {
    return any_bit(w.x[0][0], w.x[0][1], w.x[0][2], w.x[0][3]) | any_bit(w.x[1][0], w.x[1][1], w.x[1][2], w.x[1][3]);
  }
};

// k-major source (element (i, k) at P[k ld + i]): thread t holds column t%128 of the eight k of group t/128 (the same for
// a whole wavefront, so rows are addressed with scalars).  TWO: columns of two matrices.
template <bool TWO>
struct SplitKMajorOf {
  static constexpr bool OF_TWO = TWO;
  struct Raw {
    float x[8];
  };
  const float* base;
  int64_t ld;
  uint32_t off;   // bytes to the thread's column
  int kq, k_len;  // kq: first k of the thread's group
  __device__ void init(const float* P, int64_t ld_, int64_t extent, int64_t i0, int64_t k_len_, int tid) {
    base = P;
    ld = ld_;
    kq = __builtin_amdgcn_readfirstlane((tid / TILE) * 8);
    k_len = (int)k_len_;
    const int64_t i = i0 + tid % TILE;
    off = (uint32_t)(i < extent - 1 ? i : extent - 1) * 4u;
  }
  // the first `half` columns are those of P, the others of P2
  __device__ void init_two(const float* P, const float* P2, int32_t half, int64_t ld_, int64_t extent, int64_t i0, int64_t k_len_, int tid) {
    init(P, ld_, extent, i0, k_len_, tid);
    const int64_t i = off / 4u;
    base = i < half ? P + i : P2 + (i - half);
    off = 0;
  }
  __device__ void load(int t, Raw& w) const {
    const float* row = base + (int64_t)(window_of(t, k_len, 0).start + kq) * ld;
#pragma unroll
    for (int c = 0; c < 8; ++c, row += ld) w.x[c] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + off);
  }
  __device__ void load_short(Raw& w) const {  // k_len < 16
    const int first = short_first(k_len, kq);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const float* const row = base + (int64_t)(first + c < k_len ? first + c : k_len - 1) * ld;
      w.x[c] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + off);
    }
  }
  __device__ float value(const Window& in, int c, const Raw& w) const { return kq + c >= in.lo && kq + c < in.hi ? w.x[c] : 0.f; }
  // sign: 0 or the sign bit, on every element
  template <bool, bool ONLY_PART>
  __device__ void pair(int q, int, int t, const Raw& w, uint32_t sign, Group& g) const {
    const Window in = window_of(t, k_len, kq);
    float e[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = 2 * q + i;
      e[i] = __uint_as_float(__float_as_uint(ONLY_PART ? value(in, c, w) : w.x[c]) ^ sign);
    }
    g.pair(q, e[0], e[1]);
  }
  __device__ static void write(unsigned char* lds, int tid, const Raw&, const Group& g) {
    g.write(lds + (tid / TILE) * PLANE_KG + plane_row(tid % TILE), PLANE);
  }
  // sum of the thread's eight k (weight gradients: column sums of operand A)
  template <bool ONLY_PART>
  __device__ float sum(int t, const Raw& w) const {
    const Window in = window_of(t, k_len, kq);
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) s += ONLY_PART ? value(in, c, w) : w.x[c];
    return s;
  }
  __device__ static uint32_t bits(const Raw& w) {
    return any_bit(w.x[0], w.x[1], w.x[2], w.x[3]) | any_bit(w.x[4], w.x[5], w.x[6], w.x[7]);
  }
};

typedef SplitKMajorOf<false> SplitKMajor;

// Parameters that split_params_kernel has split: the three planes of a step, 16 bytes (eight k of a row) after another
struct SplitPlanes {
  struct Raw {
    uint32x4 x[3];
  };
  const unsigned char* base;  // the column tile's first step
  uint32_t off;
  __device__ void init(const unsigned char* P, int tid) {
    base = P;
    off = (uint32_t)tid * 16u;
  }
  __device__ void load(int t, Raw& w) const {
    const unsigned char* const p = base + (int64_t)t * STEP_IMAGE;
#pragma unroll
    for (int q = 0; q < 3; ++q) w.x[q] = *reinterpret_cast<const uint32x4*>(p + q * (STEP_IMAGE / 3) + off);
  }
  __device__ void load_short(Raw& w) const { load(0, w); }
  template <bool, bool>
  __device__ void pair(int, int, int, const Raw&, uint32_t, Group&) const {}
  __device__ static void write(unsigned char* lds, int tid, const Raw& w, const Group&) {
    unsigned char* const d = lds + (tid / TILE) * PLANE_KG + plane_row(tid % TILE);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint32x4*>(d + q * PLANE) = w.x[q];
  }
  __device__ static uint32_t bits(const Raw&) { return 0u; }
};

// The accumulators of a wavefront's 2x2 blocks of 32x32: of h h, and of the five smaller products.
struct Sums {
  floatx16 hh[2][2], rest[2][2];
};

// A wavefront's operands of a step: planes h, m, l of two row blocks of A and two column blocks of B.
struct Operands {
  bf16x8 a[3][2], b[2][3];
  __device__ void read_a(const unsigned char* as, int p) {
#pragma unroll
    for (int m = 0; m < 2; ++m) a[p][m] = *reinterpret_cast<const bf16x8*>(as + p * PLANE + m * 512);
  }
  __device__ void read_b(const unsigned char* bs, int o) {
#pragma unroll
    for (int p = 0; p < 3; ++p) b[o][p] = *reinterpret_cast<const bf16x8*>(bs + p * PLANE + o * 512);
  }
};

// 16 k of a wavefront's blocks: 24 matrix instructions, in twelve slots of two with work(slot) in front of each.  Nothing
// moves from one slot to another: left alone, the compiler gathers the LDS reads in front of the barrier.  The operands that
// the first slots need (planes m and l of A, the first column block of B) were read during the step before, and here those
// of the step after (NEXT, at as_next and bs_next) as soon as their registers are free: read behind the barrier, they had
// the matrix units wait for LDS in every step (half of the time, by the counters).
constexpr int SLOTS = 12;
template <bool NEXT, typename F>
__device__ inline void multiply_step(const unsigned char* as, const unsigned char* bs, const unsigned char* as_next,
                                     const unsigned char* bs_next, Operands& x, Sums& acc, F work) {
  constexpr int PA[6] = {2, 1, 1, 0, 0, 0}, PB[6] = {0, 1, 0, 2, 1, 0};
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int o = s / 6, pa = PA[s % 6], pb = PB[s % 6];
    if (s == 0) x.read_a(as, 0);
    if (s == 1) x.read_b(bs, 1);
    if (NEXT && s == 6) x.read_b(bs_next, 0);
    if (NEXT && s == 7) x.read_a(as_next, 2);
    if (NEXT && s == 9) x.read_a(as_next, 1);
    work(s);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      floatx16& c = pa + pb > 0 ? acc.rest[m][o] : acc.hh[m][o];
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.a[pa][m], x.b[o][pb], c, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A thread's share of a column sum, in float64 where a narrow matrix is (TWO, see launch_wgrad_split)
struct ColumnSum {
  float sum = 0.f;
  double sum64 = 0.0;
  bool f64 = false;
};

// One k-range of length k_len >= 1.  csum: column sums of operand A (only where the caller wants them).  small: set where
// the thread's share of either operand is all small.
//
// LDS holds three steps, one barrier per step: while step t is multiplied, step t+2 is split and written in between the
// matrix instructions (a wavefront's vector instructions issue while its matrix instructions run), step t+3 is requested
// from memory into the registers that this frees, and the operands of step t+1 are read.
//
// The matrix instructions cut off (towards minus infinity) what of a small product lies far below the running sum.  In
// one result that is little, but it does not average out where results are added up: over neighbours, over all nodes in
// a bias gradient, over the chunks of a weight gradient (115k nodes, 256 wide: bias gradients three layers down were
// 4.7e-7 off, with float32 instructions 7.4e-8).  So half of the sums are formed with the other sign, and what is cut off
// cancels: results in odd rows of a product (on operand A, taken back when they are written); in weight gradients every
// FLIP_STEPS steps of a sum (FLIP, on operand B), starting with the other sign in odd chunks (phase).
constexpr int FLIP_STEPS = 16;
template <bool FLIP, typename MA, typename MB>
__device__ inline void run_split(const MA& ma, const MB& mb, int k_len, unsigned char* smem, int a_off, int b_off,
                                 Sums& acc, int tid, int phase, bool colsum, ColumnSum& csum, bool& small) {
  const int n = (k_len + SBK - 1) / SBK;
  typename MA::Raw ra;
  typename MB::Raw rb;
  Group ga, gb;
  uint32_t bits_a = 0, bits_b = 0;
  // the thread's share of step t: four pairs, then (q = 4) on to LDS
  auto put_a = [&](int q, int t, unsigned char* d, auto part) {
    if (q < 4) return ma.template pair<!FLIP, decltype(part)::value>(q, tid, t, ra, 0u, ga);
    bits_a |= MA::bits(ra);
    ma.write(d, tid, ra, ga);
  };
  auto put_b = [&](int q, int t, unsigned char* d, auto part) {
    const uint32_t sign = FLIP && (t / FLIP_STEPS + phase) % 2 ? 0x80000000u : 0u;
    if (q < 4) return mb.template pair<false, decltype(part)::value>(q, tid, t, rb, sign, gb);
    bits_b |= MB::bits(rb);
    mb.write(d + OPERAND, tid, rb, gb);
  };
  auto put = [&](int t, unsigned char* d, auto part) {
#pragma unroll
    for (int q = 0; q < 5; ++q) put_a(q, t, d, part), put_b(q, t, d, part);
  };
  auto add_csum = [&](int t, auto part) {
    if constexpr (FLIP) {
      if (colsum) {
        const float s = ma.template sum<decltype(part)::value>(t, ra);
        if (MA::OF_TWO && csum.f64) csum.sum64 += (double)s;
        else csum.sum += s;
      }
    }
  };
  auto flip = [&](int t) {
    if (!FLIP || t == 0 || t % FLIP_STEPS != 0) return;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc.hh[m][q][v] = -acc.hh[m][q][v], acc.rest[m][q][v] = -acc.rest[m][q][v];
  };
  const std::true_type part{};
  const std::false_type whole{};
  typename MA::Raw ra1;
  typename MB::Raw rb1;
  if (k_len < SBK) {
    ma.load_short(ra);
    mb.load_short(rb);
    ra1 = ra, rb1 = rb;
  } else {
    const int t = n > 1 ? 1 : 0;  // the only step twice: under a condition, step 0 would wait for step 1 (gradients 1-2 % slower)
    ma.load(0, ra);
    mb.load(0, rb);
    ma.load(t, ra1);
    mb.load(t, rb1);
  }
  __syncthreads();  // whoever used the LDS before is done
  unsigned char *d0 = smem, *d1 = smem + STAGE, *d2 = smem + 2 * STAGE;  // steps t, t + 1, t + 2
  add_csum(0, part);
  put(0, d0, part);
  if (n > 1) {
    ra = ra1, rb = rb1;
    add_csum(1, part);
    put(1, d1, part);
  }
  if (n > 2) {
    ma.load(2, ra);
    mb.load(2, rb);
  }
  __syncthreads();
  Operands x;
  x.read_a(d0 + a_off, 2);
  x.read_a(d0 + a_off, 1);
  x.read_b(d0 + OPERAND + b_off, 0);
  int t = 0;
#pragma nounroll
  for (; t + 3 < n; ++t) {
    add_csum(t + 2, whole);
    flip(t);
    multiply_step<true>(d0 + a_off, d0 + OPERAND + b_off, d1 + a_off, d1 + OPERAND + b_off, x, acc, [&](int s) {
      if (s >= 1 && s < 6) put_a(s - 1, t + 2, d2, whole);
      if (s == 5) ma.load(t + 3, ra);
      if (s >= 6 && s < 11) put_b(s - 6, t + 2, d2, whole);
      if (s == 10) mb.load(t + 3, rb);
    });
    __syncthreads();
    unsigned char* const d = d0;
    d0 = d1;
    d1 = d2;
    d2 = d;
  }
  if (n > 2) {  // the last step to be written
    add_csum(t + 2, part);
    flip(t);
    multiply_step<true>(d0 + a_off, d0 + OPERAND + b_off, d1 + a_off, d1 + OPERAND + b_off, x, acc, [&](int s) {
      if (s >= 1 && s < 6) put_a(s - 1, t + 2, d2, part);
      if (s >= 6 && s < 11) put_b(s - 6, t + 2, d2, part);
    });
    __syncthreads();
    unsigned char* const d = d0;
    d0 = d1;
    d1 = d2;
    d2 = d;
    ++t;
  }
  if (n > 1) {
    flip(t);
    multiply_step<true>(d0 + a_off, d0 + OPERAND + b_off, d1 + a_off, d1 + OPERAND + b_off, x, acc, [](int) {});
    d0 = d1;
    ++t;
  }
  flip(t);
  multiply_step<false>(d0 + a_off, d0 + OPERAND + b_off, d0, d0, x, acc, [](int) {});
  if (FLIP && ((n - 1) / FLIP_STEPS + phase) % 2) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc.hh[m][q][v] = -acc.hh[m][q][v], acc.rest[m][q][v] = -acc.rest[m][q][v];
  }
  small |= all_small(bits_a) || all_small(bits_b);
}

// The float32 parameters of a product, split for SplitPlanes: a workgroup writes the image of one step of one column tile
// and says in flags whether a row's eight k are all small (see above).
struct SplitParamsK {
  const float* B[2];
  int64_t ldb[2];
  int32_t k_len[2], steps[2];
  int32_t N, k_major;
  const float* B_second;  // rows from `half` on (see SplitK)
  int32_t half;
  unsigned char* image;
  uint32_t* flags;
};
__global__ __launch_bounds__(256) void split_params_kernel(const SplitParamsK p) {
  const int tid = threadIdx.x, steps = p.steps[0] + p.steps[1];
  const int tile = (int)blockIdx.x / steps, step = (int)blockIdx.x % steps;
  const int seg = step >= p.steps[0], t = step - (seg ? p.steps[0] : 0);
  // k-contiguous sources: neighbouring threads read the two halves of a row
  const int kg = p.k_major ? tid / TILE : tid & 1, row = p.k_major ? tid % TILE : tid >> 1;
  const int k_len = p.k_len[seg];
  const Window in = window_of(t, k_len, kg * 8);
  const int first = k_len < SBK ? short_first(k_len, kg * 8) : in.start + kg * 8;
  const int64_t j = (int64_t)tile * TILE + row, ldb = p.ldb[seg];
  const bool of_second = j >= p.half;
  const float* const B = of_second ? p.B_second - p.half * ldb : p.B[seg];
  float e[8];
  uint32_t bits = 0;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const int k = first + c, place = kg * 8 + c;
    e[c] = j < p.N && place >= in.lo && place < in.hi ? (p.k_major ? B[k * ldb + j] : B[j * ldb + k]) : 0.f;
    bits |= __float_as_uint(e[c]);
  }
  Group g;
#pragma unroll
  for (int q = 0; q < 4; ++q) g.pair(q, e[2 * q], e[2 * q + 1]);
  g.write(p.image + (int64_t)blockIdx.x * STEP_IMAGE + (kg * TILE + row) * 16, STEP_IMAGE / 3);
  const int any = __syncthreads_or(all_small(bits));
  if (tid == 0) p.flags[blockIdx.x] = any ? 1u : 0u;
}

// One 32x32 block of the result over the same range on the float32 matrix instructions, operands straight from memory.
// Element k of the lane's row of an operand is at P[k sk]; half wavefront g takes the g-th eight of 16 k, the next of
// which are requested while one is multiplied.
__device__ inline void run_plain(const float* A, int64_t ska, const float* B, int64_t skb, int64_t k_len, int g, floatx16& acc) {
  struct Eight {
    float a[8], b[8];
  } now, next;
  auto load = [&](int64_t k0, Eight& w) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int64_t k = k0 + 8 * g + s < k_len ? k0 + 8 * g + s : k_len - 1;
      w.a[s] = A[k * ska];
      w.b[s] = B[k * skb];
    }
  };
  if (k_len <= 0) return;
  load(0, now);
#pragma nounroll
  for (int64_t k0 = 0; k0 < k_len; k0 += 16) {
    load(k0 + 16, next);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const bool in = k0 + 8 * g + s < k_len;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? now.a[s] : 0.f, in ? now.b[s] : 0.f, acc, 0, 0, 0);
    }
    now = next;
  }
}

// A_KMAJOR: weight gradient C = A^T B over graph nodes, float32 partials per chunk; else C = sum of segments A op(B).
// DROP: dropout of the result, in rows of a multiple of four contiguous columns (529k x 512 with K = 1024: a pass of its own
// took 353 us, a training step with three of them is 760 us shorter without).  Its generator runs beside the matrix
// instructions of the CU's other workgroup, where a pass of its own reads and writes the result once more.
// TWO: two results of one matrix A, whose columns follow one another and are stored apart, without an epilogue; two weight
// gradients of one matrix B, whose rows follow one another.
template <bool A_KMAJOR, bool B_KMAJOR, bool PLANES, bool DROP, bool TWO = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void gemm_split_kernel(
    const SplitK p) {
  constexpr int STAGE_LD = 68, STAGE_WAVE = 32 * STAGE_LD;  // result staging: floats
  __shared__ __attribute__((aligned(128))) unsigned char smem[3 * STAGE];
  static_assert(3 * STAGE >= 4 * STAGE_WAVE * 4, "results are staged where the operands were");
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int g = lane >> 5, r = lane & 31;
  // XCD-aware linear id -> (group, member): the tiles that share an operand panel are adjacent on one XCD
  int64_t i0, j0, z = 0;
  {
    const int64_t L = blockIdx.x;
    if constexpr (A_KMAJOR) {
      if (L >= (int64_t)gridDim.x - p.extra.blocks) {
        colsum_block<float>(p.extra, L - ((int64_t)gridDim.x - p.extra.blocks), reinterpret_cast<float*>(smem), threadIdx.x);
        return;
      }
    }
    const int64_t per_group = A_KMAJOR ? p.tiles_m * p.tiles_n : p.tiles_n;
    const int64_t group = (L / (8 * per_group)) * 8 + (L & 7);
    const int64_t member = (L >> 3) % per_group;
    if (group >= p.n_groups) return;  // padding of the last group octet (uniform over the block)
    if constexpr (A_KMAJOR) {
      z = group;
      i0 = (member / p.tiles_n) * TILE;
      j0 = (member % p.tiles_n) * TILE;
    } else {
      i0 = group * TILE;
      j0 = member * TILE;
    }
  }
  const int a_off = g * PLANE_KG + wm * 1024 + plane_row(r);
  const int b_off = g * PLANE_KG + wn * 1024 + plane_row(r);
  Sums sums;
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int v = 0; v < 16; ++v) sums.hh[m][n][v] = sums.rest[m][n][v] = 0.f;

  // weight gradients: this block's chunk of nodes and its matrix of operand B
  int64_t k_beg = 0, k_len = 0;
  const float* Bw = p.B1;
  int64_t ldbw = p.ldb1, extent_b = p.N, jw = j0;
  if constexpr (A_KMAJOR) {
    k_beg = z * p.k_chunk;
    const int64_t k_end = k_beg + p.k_chunk < p.K1 ? k_beg + p.k_chunk : p.K1;
    k_len = k_end > k_beg ? k_end - k_beg : 0;
    if (p.n_split > 0) extent_b = p.n_split;
    if (p.n_split > 0 && j0 >= p.n_split) {  // a column tile of the second matrix
      Bw = p.B2;
      ldbw = p.ldb2;
      extent_b = p.N - p.n_split;
      jw = j0 - p.n_split;
    }
  }
  const int n_seg = !A_KMAJOR && p.K2 > 0 ? 2 : 1;
  ColumnSum csum;
  if constexpr (A_KMAJOR && TWO) csum.f64 = p.colsum_f64;
  bool small = false;
  if constexpr (A_KMAJOR) {
    if (k_len > 0) {
      SplitKMajorOf<TWO> ma;
      SplitKMajor mb;
      if constexpr (TWO) ma.init_two(p.A1 + k_beg * p.lda1, p.A2 + k_beg * p.lda1, p.half, p.lda1, p.M, i0, k_len, tid);
      else ma.init(p.A1 + k_beg * p.lda1, p.lda1, p.M, i0, k_len, tid);
      mb.init(Bw + k_beg * ldbw, ldbw, extent_b, jw, k_len, tid);
      run_split<true>(ma, mb, (int)k_len, smem, a_off, b_off, sums, tid, (int)(z & 1), p.colsum_part != nullptr && j0 == 0, csum,
                      small);
    }
  } else {
    // one loop body for both segments (two inlined copies would each claim their own accumulators)
#pragma nounroll
    for (int seg = 0; seg < n_seg; ++seg) {
      const int k_seg = (int)(seg ? p.K2 : p.K1);
      SplitKContig ma;
      ma.init(seg ? p.A2 : p.A1, seg ? p.lda2 : p.lda1, p.M, i0, k_seg, tid);
      if constexpr (PLANES) {
        const int steps1 = (int)((p.K1 + SBK - 1) / SBK), steps = steps1 + (int)((p.K2 + SBK - 1) / SBK);
        const int64_t first = (j0 / TILE) * steps + (seg ? steps1 : 0);
        SplitPlanes mb;
        mb.init(p.planes + first * STEP_IMAGE, tid);
        const int n = (k_seg + SBK - 1) / SBK;
        uint32_t again = p.small_params[first + (tid < n ? tid : 0)];
        for (int t = tid + 256; t < n; t += 256) again |= p.small_params[first + t];
        run_split<false>(ma, mb, k_seg, smem, a_off, b_off, sums, tid, 0, false, csum, small);
        small |= again != 0u;
      } else if constexpr (B_KMAJOR) {
        SplitKMajor mb;
        mb.init(seg ? p.B2 : p.B1, seg ? p.ldb2 : p.ldb1, p.N, j0, k_seg, tid);
        run_split<false>(ma, mb, k_seg, smem, a_off, b_off, sums, tid, 0, false, csum, small);
      } else {
        SplitKContig mb;
        if constexpr (TWO) mb.init_two(p.B_second, p.b_offset, p.half, p.ldb1, p.N, j0, k_seg, tid);
        else mb.init(seg ? p.B2 : p.B1, seg ? p.ldb2 : p.ldb1, p.N, j0, k_seg, tid);
        run_split<false>(ma, mb, k_seg, smem, a_off, b_off, sums, tid, 0, false, csum, small);
      }
    }
  }
  floatx16(&acc)[2][2] = sums.hh;
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[m][n][v] += sums.rest[m][n][v];
  // blocks that the split does not get right (see above) are computed again
  int again = __syncthreads_or(small) ? 15 : 0;
#pragma unroll
  for (int blk = 0; blk < 4; ++blk) {
    float bad = 0.f;  // stays zero while every result is finite
#pragma unroll
    for (int v = 0; v < 16; ++v) bad = fmaf(acc[blk / 2][blk % 2][v], 0.f, bad);
    if (__any(!(bad == 0.f))) again |= 1 << blk;
  }
#pragma nounroll
  for (int blk = 0; again >> blk != 0; ++blk) {
    if (!(again >> blk & 1)) continue;
    const int64_t ib = i0 + wm * 64 + blk / 2 * 32 + r, jb = jw + wn * 64 + blk % 2 * 32 + r;
    const int64_t ia = ib < p.M ? ib : p.M - 1, ja = jb < extent_b ? jb : extent_b - 1;
    floatx16 c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = 0.f;
    if constexpr (A_KMAJOR) {
      const float* const A = TWO && ia >= p.half ? p.A2 + (ia - p.half) : p.A1 + ia;
      run_plain(A + k_beg * p.lda1, p.lda1, Bw + k_beg * ldbw + ja, ldbw, k_len, g, c);
    } else {
#pragma nounroll
      for (int seg = 0; seg < n_seg; ++seg) {
        const int64_t ldb = seg ? p.ldb2 : p.ldb1;
        const float* B = (seg ? p.B2 : p.B1) + ja * (B_KMAJOR ? 1 : ldb);
        if (TWO && ja >= p.half) B = p.B_second + (ja - p.half) * ldb;
        run_plain((seg ? p.A2 : p.A1) + ia * (seg ? p.lda2 : p.lda1), 1, B,
                  B_KMAJOR ? ldb : 1, seg ? p.K2 : p.K1, g, c);
      }
#pragma unroll
      for (int v = 1; v < 16; v += 2) c[v] = -c[v];  // odd rows with the other sign, as the split leaves them
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if (b == blk) acc[b / 2][b % 2] = c;
  }

  // accumulator register v of lane (g, r) is element [8 (v/4) + 4 g + v%4][r] of its 32x32 block
  if constexpr (A_KMAJOR) {
    float* Cz = p.C + z * p.c_split_stride;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int64_t j = j0 + wn * 64 + n * 32 + r;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int64_t i = i0 + wm * 64 + m * 32 + 8 * (v >> 2) + 4 * g + (v & 3);
          if (j < p.N && i < p.M) Cz[i * p.ldc + j] = acc[m][n][v];
        }
      }
    }
    if (p.colsum_part != nullptr && j0 == 0) {
      // the two k-groups of a column are added in order through LDS
      float* const red = reinterpret_cast<float*>(smem);
      __syncthreads();
      red[tid] = csum.f64 ? (float)csum.sum64 : csum.sum;
      __syncthreads();
      if (tid < TILE && i0 + tid < p.M) p.colsum_part[z * p.M + i0 + tid] = red[tid] + red[TILE + tid];
    }
  } else {
    // Each wavefront passes its result through LDS in 32-row blocks, after which a lane holds four consecutive
    // columns of one row: gate and accumulate operands are read, and the result is written, 16 bytes at a time.
    // Those operands and the row scales do not depend on the product, so they are requested for four passes at a
    // time, unconditionally at clamped addresses, the first four of a block before its staging barriers.
    constexpr int LPR = 16;           // lanes per staged row
    constexpr int RPP = 64 / LPR;     // rows per pass
    constexpr int PASSES = 32 / RPP;  // passes per 32-row block
    float* const st = reinterpret_cast<float*>(smem) + wave * STAGE_WAVE;
    const int er = lane / LPR, ec = (lane % LPR) * 4;
    const int64_t jv = j0 + wn * 64 + ec;
    const bool wide_lane = jv + 4 <= p.N;   // the lane's four columns all exist
    const int64_t jl = wide_lane ? jv : 0;  // where its 16-byte operand loads go (in range: N >= 4)
    const bool extras = p.gate || p.accumulate || p.row_scale;  // uniform over the launch
    struct Extra {
      float4u g, c;
      float rs;
    };
    if constexpr (TWO) {
      const bool whole = i0 + TILE <= p.M;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int64_t j = j0 + wn * 64 + n * 32 + r;
        if (j < p.N) {
          float* const dst = (j < p.half ? p.C + j : p.C_second + (j - p.half)) + (i0 + wm * 64 + 4 * g) * p.ldc;
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              const int row = m * 32 + 8 * (v >> 2) + (v & 3);
              if (whole || i0 + wm * 64 + 4 * g + row < p.M) dst[(int64_t)row * p.ldc] = v & 1 ? -acc[m][n][v] : acc[m][n][v];
            }
        }
      }
      return;
    }
    if constexpr (!DROP) {
      if (!extras && !p.relu_last && i0 + TILE <= p.M) {
        // Nothing but bias and ReLU: a register of a block is two rows of a whole line of 128 bytes and is stored as it lies
        // (470k x 512 x 512 1330 -> 1281 us, 60k x 256 x 256 58 -> 53; with gates or row factors, element by element like
        // this, products took up to 11 % longer than through LDS).
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const int64_t j = j0 + wn * 64 + n * 32 + r;
          if (j < p.N) {
            const float bj = p.bias ? p.bias[j] : 0.f;
            float* const dst = p.C + (i0 + wm * 64 + 4 * g) * p.ldc + j;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                float x = (v & 1 ? -acc[m][n][v] : acc[m][n][v]) + bj;  // odd rows were summed with the other sign
                if (p.relu) x = fmaxf(x, 0.f);
                dst[(int64_t)(m * 32 + 8 * (v >> 2) + (v & 3)) * p.ldc] = x;
              }
          }
        }
        return;
      }
    }
    auto request = [&](int m, int s, Extra& e) {
      int64_t il = i0 + wm * 64 + m * 32 + s * RPP + er;
      if (il > p.M - 1) il = p.M - 1;
      e.g = float4u{1.f, 1.f, 1.f, 1.f};
      e.c = float4u{0.f, 0.f, 0.f, 0.f};
      e.rs = 1.f;
      if (p.gate) e.g = *reinterpret_cast<const float4u*>(p.gate + il * p.ldg + jl);
      if (p.accumulate) e.c = *reinterpret_cast<const float4u*>(p.C + il * p.ldc + jl);
      if (p.row_scale) e.rs = p.row_scale[il];
    };
    auto pass = [&](int m, int s, bool have, const Extra& e) {
      const int row = s * RPP + er;
      const int64_t i = i0 + wm * 64 + m * 32 + row;
      if (i < p.M && jv < p.N) {
        const float4 t = *reinterpret_cast<const float4*>(st + row * STAGE_LD + ec);
        float x[4] = {t.x, t.y, t.z, t.w};
        float* dst = p.C + i * p.ldc + jv;
        if (wide_lane) {
          if (have) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              float y = x[c] * e.rs;
              const bool shut = !(e.g[c] > 0.f);
              if (!p.gate_last) y = shut ? 0.f : y * p.gate_scale;
              y += e.c[c];
              if (p.gate_last) y = shut ? 0.f : y * p.gate_scale;
              x[c] = y;
            }
          }
          if (p.relu_last) {
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = fmaxf(x[c], 0.f);
          }
          if constexpr (DROP) drop4(p.drop, (uint64_t)i * (uint32_t)p.N + (uint32_t)jv, x);
          float4u out;
#pragma unroll
          for (int c = 0; c < 4; ++c) out[c] = x[c];
          *reinterpret_cast<float4u*>(dst) = out;
        } else {
          const float sc = p.row_scale ? p.row_scale[i] : 1.f;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if (jv + c < p.N) {
              float y = x[c] * sc;
              const bool shut = p.gate && !(p.gate[i * p.ldg + jv + c] > 0.f);
              if (!p.gate_last) y = shut ? 0.f : y * p.gate_scale;
              if (p.accumulate) y += dst[c];
              if (p.gate_last) y = shut ? 0.f : y * p.gate_scale;
              if (p.relu_last) y = fmaxf(y, 0.f);
              dst[c] = y;
            }
          }
        }
      }
    };
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      Extra e[4] = {};
      if (extras) {
#pragma unroll
        for (int q = 0; q < 4; ++q) request(m, q, e[q]);
      }
      __syncthreads();  // operand planes (m = 0) / previous block no longer read
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int64_t j = j0 + wn * 64 + n * 32 + r;
        const float bj = (p.bias && j < p.N) ? p.bias[j] : 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          float x = (v & 1 ? -acc[m][n][v] : acc[m][n][v]) + bj;  // odd rows were summed with the other sign
          if (p.relu) x = fmaxf(x, 0.f);
          st[(8 * (v >> 2) + 4 * g + (v & 3)) * STAGE_LD + n * 32 + r] = x;
        }
      }
      __syncthreads();
      if (extras) {
#pragma nounroll
        for (int q0 = 0; q0 < PASSES; q0 += 4) {
          if (q0 > 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) request(m, q0 + q, e[q]);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) pass(m, q0 + q, true, e[q]);
        }
      } else {
#pragma nounroll
        for (int q0 = 0; q0 < PASSES; q0 += 4)
#pragma unroll
          for (int q = 0; q < 4; ++q) pass(m, q0 + q, false, e[0]);
      }
    }
  }
}

// ---- few rows ---------------------------------------------------------------------------------------------------
// The same product in 64x64 tiles of the result, 32x32 a wavefront, for results of so few 128x128 tiles that most CUs would have no
// workgroup.  There the time is the chain of one workgroup's steps: here a step has a quarter of the matrix instructions, and
// four steps of loads are in flight.  Wavefronts 0 and 1 move operand A, the others B.  Sums are formed in the same order, so
// results are those of the large tiles bit for bit.  No dropout: its four columns a draw lie in four lanes here.
constexpr int FEW_TILE = 64, FEW_KG = FEW_TILE * 16 + 64, FEW_PLANE = 2 * FEW_KG, FEW_OPERAND = 3 * FEW_PLANE, FEW_STAGE = 2 * FEW_OPERAND;
constexpr int FEW_RING = 4;
template <bool B_KMAJOR, bool TWO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void gemm_split_few_kernel(const SplitK p) {
  __shared__ __attribute__((aligned(128))) unsigned char smem[3 * FEW_STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, g = lane >> 5, r = lane & 31;
  const bool of_b = wave >= 2;
  // the column tiles of a row panel are neighbours on one XCD
  const int64_t L = blockIdx.x, group = (L / (8 * p.tiles_n)) * 8 + (L & 7), member = (L >> 3) % p.tiles_n;
  if (group >= p.n_groups) return;
  const int64_t i0 = group * FEW_TILE, j0 = member * FEW_TILE;

  // the thread's share of a step: eight k of one row, or (parameters [k][column]) of one column
  const int lt = tid & 127;
  const bool by_column = B_KMAJOR && of_b;  // uniform over the wavefront
  const int row = by_column ? lt & 63 : lt >> 1, kq = by_column ? (wave & 1) * 8 : (lt & 1) * 8;
  const int n1 = (int)((p.K1 + SBK - 1) / SBK), n = n1 + (int)((p.K2 + SBK - 1) / SBK);
  const float *s1, *s2 = nullptr;  // element k of the row at s[k sk]
  int64_t sk1 = 1, sk2 = 1;
  if (of_b) {
    const int64_t j = j0 + row < p.N - 1 ? j0 + row : p.N - 1;
    if (TWO && j >= p.half) s1 = p.B_second + (j - p.half) * p.ldb1;
    else s1 = p.B1 + (B_KMAJOR ? j : j * p.ldb1);
    if (p.K2 > 0) s2 = p.B2 + (B_KMAJOR ? j : j * p.ldb2);
    if (B_KMAJOR) sk1 = p.ldb1, sk2 = p.ldb2;
  } else {
    const int64_t i = i0 + row < p.M - 1 ? i0 + row : p.M - 1;
    s1 = p.A1 + i * p.lda1;
    if (p.K2 > 0) s2 = p.A2 + i * p.lda2;
  }
  const uint32_t flip = !of_b ? (uint32_t)row << 31 : 0u;  // odd rows are summed with the other sign

  struct Raw {
    float x[8];
  } ring[FEW_RING];
  auto load = [&](int q, Raw& w) __attribute__((always_inline)) {
    if (q > n - 1) q = n - 1;
    const bool second = q >= n1;
    const int k_len = (int)(second ? p.K2 : p.K1), t = second ? q - n1 : q;
    const int first = k_len < SBK ? short_first(k_len, kq) : window_of(t, k_len, kq).start + kq;
    const float* const s = second ? s2 : s1;
    if (by_column) {
      const int64_t sk = second ? sk2 : sk1;
#pragma unroll
      for (int c = 0; c < 8; ++c) w.x[c] = s[(first + c) * sk];
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float4u v = *reinterpret_cast<const float4u*>(s + first + 4 * h);
#pragma unroll
        for (int c = 0; c < 4; ++c) w.x[4 * h + c] = v[c];
      }
    }
  };
  bool small = false;
  uint32_t bits = 0;
  auto put = [&](int q, const Raw& w, unsigned char* stage) __attribute__((always_inline)) {
    const bool second = q >= n1;
    const int k_len = (int)(second ? p.K2 : p.K1), t = second ? q - n1 : q;
    if (q == n1) small |= all_small(bits), bits = 0;
    bits |= any_bit(w.x[0], w.x[1], w.x[2], w.x[3]) | any_bit(w.x[4], w.x[5], w.x[6], w.x[7]);
    float e[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) e[c] = __uint_as_float(__float_as_uint(w.x[c]) ^ flip);
    if ((t + 1) * SBK > k_len) {  // uniform: the last step of a segment that is not whole steps
      const Window in = window_of(t, k_len, kq);
#pragma unroll
      for (int c = 0; c < 8; ++c) e[c] = kq + c >= in.lo && kq + c < in.hi ? e[c] : 0.f;
    }
    Group o;
#pragma unroll
    for (int c = 0; c < 4; ++c) o.pair(c, e[2 * c], e[2 * c + 1]);
    o.write(stage + (of_b ? FEW_OPERAND : 0) + (kq >> 3) * FEW_KG + plane_row(row), FEW_PLANE);
  };
  struct Planes {
    bf16x8 a[3], b[3];
  };
  const int a_off = g * FEW_KG + wm * 512 + plane_row(r), b_off = FEW_OPERAND + g * FEW_KG + wn * 512 + plane_row(r);
  auto take = [&](const unsigned char* stage, Planes& x) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      x.a[q] = *reinterpret_cast<const bf16x8*>(stage + a_off + q * FEW_PLANE);
      x.b[q] = *reinterpret_cast<const bf16x8*>(stage + b_off + q * FEW_PLANE);
    }
  };
  floatx16 hh, rest;
#pragma unroll
  for (int v = 0; v < 16; ++v) hh[v] = rest[v] = 0.f;
  auto multiply = [&](const Planes& x) __attribute__((always_inline)) {
    constexpr int PA[6] = {2, 1, 1, 0, 0, 0}, PB[6] = {0, 1, 0, 2, 1, 0};
#pragma unroll
    for (int s = 0; s < 6; ++s) {
      floatx16& c = s < 5 ? rest : hh;
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.a[PA[s]], x.b[PB[s]], c, 0, 0, 0);
    }
  };

#pragma unroll
  for (int q = 0; q < FEW_RING; ++q) load(q, ring[q]);
  unsigned char *d0 = smem, *d1 = smem + FEW_STAGE, *d2 = smem + 2 * FEW_STAGE;  // steps t, t + 1, t + 2
  put(0, ring[0], d0);
  load(FEW_RING, ring[0]);
  if (n > 1) put(1, ring[1], d1);
  load(FEW_RING + 1, ring[1]);
  __syncthreads();
  // step t is multiplied, t + 2 written, t + 2 + FEW_RING requested
#pragma nounroll
  for (int t0 = 0; t0 < n; t0 += FEW_RING) {
#pragma unroll
    for (int s = 0; s < FEW_RING; ++s) {
      const int t = t0 + s;
      if (t < n) {  // uniform over the workgroup
        Planes x;
        take(d0, x);
        Raw& w = ring[(s + 2) % FEW_RING];
        if (t + 2 < n) put(t + 2, w, d2);
        load(t + 2 + FEW_RING, w);
        multiply(x);
        __syncthreads();
        unsigned char* const d = d0;
        d0 = d1;
        d1 = d2;
        d2 = d;
      }
    }
  }
  small |= all_small(bits);
#pragma unroll
  for (int v = 0; v < 16; ++v) hh[v] += rest[v];
  // blocks that the split does not get right are computed again (see gemm_split_kernel)
  bool again = __syncthreads_or(small);
  float bad = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) bad = fmaf(hh[v], 0.f, bad);
  again |= __any(!(bad == 0.f)) != 0;
  const int64_t jb = j0 + wn * 32 + r;
  if (again) {
    const int64_t ib = i0 + wm * 32 + r, ia = ib < p.M ? ib : p.M - 1, ja = jb < p.N ? jb : p.N - 1;
#pragma unroll
    for (int v = 0; v < 16; ++v) hh[v] = 0.f;
#pragma nounroll
    for (int seg = 0; seg < (p.K2 > 0 ? 2 : 1); ++seg) {
      const int64_t ldb = seg ? p.ldb2 : p.ldb1;
      const float* B = (seg ? p.B2 : p.B1) + ja * (B_KMAJOR ? 1 : ldb);
      if (TWO && ja >= p.half) B = p.B_second + (ja - p.half) * ldb;
      run_plain((seg ? p.A2 : p.A1) + ia * (seg ? p.lda2 : p.lda1), 1, B, B_KMAJOR ? ldb : 1, seg ? p.K2 : p.K1, g, hh);
    }
#pragma unroll
    for (int v = 1; v < 16; v += 2) hh[v] = -hh[v];
  }
  // register v of lane (g, r) is element [8 (v / 4) + 4 g + v % 4][r] of the block: a register is two rows of a whole line
  if (jb >= p.N) return;
  const int64_t first = i0 + wm * 32 + 4 * g;
  float* const C = TWO && jb >= p.half ? p.C_second + (jb - p.half) : p.C + jb;
  const float bj = !TWO && p.bias ? p.bias[jb] : 0.f;
  float gate[16], sum[16], rs[16];
  if constexpr (!TWO) {
    auto at = [&](int v) {
      const int64_t i = first + 8 * (v >> 2) + (v & 3);
      return i < p.M ? i : p.M - 1;
    };
    if (p.gate) {
#pragma unroll
      for (int v = 0; v < 16; ++v) gate[v] = p.gate[at(v) * p.ldg + jb];
    }
    if (p.accumulate) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[v] = C[at(v) * p.ldc];
    }
    if (p.row_scale) {
#pragma unroll
      for (int v = 0; v < 16; ++v) rs[v] = p.row_scale[at(v)];
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int64_t i = first + 8 * (v >> 2) + (v & 3);
    float x = (v & 1 ? -hh[v] : hh[v]) + bj;
    if constexpr (!TWO) {
      if (p.relu) x = fmaxf(x, 0.f);
      if (p.row_scale) x *= rs[v];
      if (p.gate && !p.gate_last) x = gate[v] > 0.f ? x * p.gate_scale : 0.f;
      if (p.accumulate) x += sum[v];
      if (p.gate && p.gate_last) x = gate[v] > 0.f ? x * p.gate_scale : 0.f;
      if (p.relu_last) x = fmaxf(x, 0.f);
    }
    if (i < p.M) C[i * p.ldc] = x;
  }
}

// 32-bit element offsets inside a tile: 128 rows of a k-contiguous operand
static bool split_strides_ok(int64_t lda, int64_t ldb) { return lda < ((int64_t)1 << 22) && ldb < ((int64_t)1 << 22); }

bool gemm_split_fits(const GemmArgs& a) {
  return a.dtype == COFREE_F32 && a.N > 64 && a.K1 >= 8 && (a.K2 == 0 || a.K2 >= 8) && split_strides_ok(a.lda1, a.ldb) &&
         (a.K2 == 0 || split_strides_ok(a.lda2, a.B2 ? a.ldb2 : 0));
}

// The parameters are split by a launch of their own, of 6 us, where every workgroup would split them again: from 20 billion
// operand pairs on (230k x 256 x 256: 231 -> 225 us and the launch; 230k x 256 x 602 496 -> 467, 470k x 512 x 512 1374 -> 1330, gated
// 1465 -> 1359; 60k x 256 x 256 59.7 -> 58.1).
size_t split_param_bytes(int64_t M, int32_t N, int64_t K1, int64_t K2) {
  if (N <= 64 || (double)M * N * ((double)K1 + K2) < 2e10) return 0;
  const size_t images = (size_t)((N + TILE - 1) / TILE) * (size_t)((K1 + SBK - 1) / SBK + (K2 + SBK - 1) / SBK);
  return images * (STEP_IMAGE + 4);
}

static bool split_params_first(const GemmArgs& a) {
  const size_t bytes = split_param_bytes(a.M, a.C_second ? 2 * a.N : a.N, a.K1, a.K2);
  return bytes > 0 && a.param_scratch && a.param_scratch_bytes >= bytes;
}

// Results of at most 64 tiles of 128x128 are computed in tiles of a quarter of that: the line is where those are one for each CU.
// Microseconds, large tiles / small ones: 4 tiles (500 x 128 x 512) 24.7 / 19.9, 16 (2k x 66 x 500) 26.5 / 20.0, 40 (5k x 128 x 512)
// 24.0 / 20.4, 64 (2k x 512 x 512) 25.1 / 20.9; above, 79 (10k x 128 x 512) 24.1 / 24.2, 158 (10k x 256 x 256) 16.2 / 19.3.
// But not A B of up to three steps and more than 80 columns, where nothing but the ends of a tile is left (backward of 128 -> 8 over 4,000 nodes
// 22.4 / 23.5, 256 -> 32 25.6 / 26.4, 200 -> 48 28.2 / 29.1; 66 -> 8 over 2,000 0.93 of the time in small ones, A B^T of 8 k 0.95).
static bool few_tiles(const GemmArgs& a, int64_t K, int64_t large_tiles) {
  return large_tiles <= 64 && !(a.b_kmajor && K <= 48 && a.N > 80);
}

int32_t launch_gemm_split(const GemmArgs& a, hipStream_t stream) {
  SplitK p{};
  p.A1 = (const float*)a.A1;
  p.lda1 = a.lda1;
  p.K1 = a.K1;
  p.A2 = (const float*)a.A2;
  p.lda2 = a.lda2;
  p.K2 = a.K2;
  p.B1 = a.B;
  p.ldb1 = a.ldb;
  p.B2 = a.B2 ? a.B2 : a.B + (a.b_kmajor ? (int64_t)a.K1 * a.ldb : (int64_t)a.K1);
  p.ldb2 = a.B2 ? a.ldb2 : a.ldb;
  p.C = (float*)a.C;
  p.ldc = a.ldc;
  p.M = a.M;
  const int32_t N = a.C_second ? 2 * a.N : a.N;
  p.N = N;
  p.B_second = a.B_second;
  p.C_second = (float*)a.C_second;
  p.b_offset = a.C_second ? a.B - a.B_second : 0;
  p.half = a.C_second ? a.N : INT_MAX;
  p.bias = a.bias;
  p.relu = a.relu;
  p.row_scale = a.row_scale;
  p.gate = (const float*)a.gate;
  p.ldg = a.ldg;
  p.accumulate = a.accumulate;
  p.relu_last = a.relu_last;
  p.gate_last = a.gate_last;
  p.gate_scale = a.gate ? a.gate_scale : 1.f;
  p.drop = dropout_k(a.dropout);
  const int64_t K = (int64_t)a.K1 + a.K2;
  p.n_groups = (a.M + TILE - 1) / TILE;
  p.tiles_n = (N + TILE - 1) / TILE;
  const int64_t blocks = ((p.n_groups + 7) / 8) * 8 * p.tiles_n;
  COFREE_REQUIRE(blocks > 0 && blocks < ((int64_t)1 << 31), "dense: grid too large");
  const bool drop = p.drop.scale != 0.f;  // forward products only
  const bool planes = split_params_first(a);
  if (!planes && !drop && few_tiles(a, K, p.n_groups * p.tiles_n)) {
    p.n_groups = (a.M + FEW_TILE - 1) / FEW_TILE;
    p.tiles_n = (N + FEW_TILE - 1) / FEW_TILE;
    const int64_t few = (p.n_groups + 7) / 8 * 8 * p.tiles_n;
    char pname[96] = "";
    if (profiling()) snprintf(pname, sizeof(pname), "gemm_split_few_kernel<%s,%s> N=%d K=%d", a.b_kmajor ? "true" : "false",
             a.C_second ? "true" : "false", (int)N, (int)K);
    ProfScope prof(pname, stream, 4.0 * ((double)a.M * K + (double)N * K + (double)a.M * N * (a.accumulate ? 2 : 1)),
                   2.0 * (double)a.M * N * (double)K);
    if (a.C_second) gemm_split_few_kernel<false, true><<<dim3((unsigned)few), 256, 0, stream>>>(p);
    else if (a.b_kmajor) gemm_split_few_kernel<true, false><<<dim3((unsigned)few), 256, 0, stream>>>(p);
    else gemm_split_few_kernel<false, false><<<dim3((unsigned)few), 256, 0, stream>>>(p);
    COFREE_HIP_CHECK(hipGetLastError());
    return COFREE_OK;
  }
  if (planes) {
    SplitParamsK q{};
    q.B[0] = p.B1, q.B[1] = p.B2;
    q.ldb[0] = p.ldb1, q.ldb[1] = p.ldb2;
    q.k_len[0] = a.K1, q.k_len[1] = a.K2;
    q.steps[0] = (a.K1 + SBK - 1) / SBK, q.steps[1] = (a.K2 + SBK - 1) / SBK;
    q.N = N, q.k_major = a.b_kmajor;
    q.B_second = a.B_second, q.half = p.half;
    const int steps = q.steps[0] + q.steps[1];
    q.image = (unsigned char*)a.param_scratch;
    q.flags = (uint32_t*)(q.image + (size_t)p.tiles_n * steps * STEP_IMAGE);
    ProfScope prof("split_params_kernel", stream, 10.0 * (double)N * K, 0.0);
    split_params_kernel<<<dim3((unsigned)(p.tiles_n * steps)), 256, 0, stream>>>(q);
    p.planes = q.image;
    p.small_params = q.flags;
  }
  char pname[96] = "";
  if (profiling()) snprintf(pname, sizeof(pname), "gemm_split_kernel<false,%s,%s,%s,%s> N=%d K=%d", a.b_kmajor ? "true" : "false",
           planes ? "true" : "false", drop && !a.b_kmajor ? "true" : "false", a.C_second ? "true" : "false", (int)N, (int)K);
  ProfScope prof(pname, stream, 4.0 * ((double)a.M * K + (double)N * K + (double)a.M * N * (a.accumulate ? 2 : 1)),
                 2.0 * (double)a.M * N * (double)K);
  const dim3 grid((unsigned)blocks);
  if (a.C_second && planes) gemm_split_kernel<false, false, true, false, true><<<grid, 256, 0, stream>>>(p);
  else if (a.C_second) gemm_split_kernel<false, false, false, false, true><<<grid, 256, 0, stream>>>(p);
  else if (planes && a.b_kmajor) gemm_split_kernel<false, true, true, false><<<grid, 256, 0, stream>>>(p);
  else if (planes && drop) gemm_split_kernel<false, false, true, true><<<grid, 256, 0, stream>>>(p);
  else if (planes) gemm_split_kernel<false, false, true, false><<<grid, 256, 0, stream>>>(p);
  else if (a.b_kmajor) gemm_split_kernel<false, true, false, false><<<grid, 256, 0, stream>>>(p);
  else if (drop) gemm_split_kernel<false, false, false, true><<<grid, 256, 0, stream>>>(p);
  else gemm_split_kernel<false, false, false, false><<<grid, 256, 0, stream>>>(p);
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

bool wgrad_split_fits(const WgradArgs& a) {
  return a.N1 > 64 && a.N2 > 64 && (!a.B2 || a.N2b >= 4) && split_strides_ok(a.lda, a.ldb) &&
         split_strides_ok(0, a.B2 ? a.ldb2 : 0);
}

int32_t launch_wgrad_split(const WgradArgs& a, SplitSums* sums, hipStream_t stream) {
  const int32_t N1 = a.A2 ? 2 * a.N1 : a.N1, N2 = a.N2 + (a.B2 ? a.N2b : 0);
  const int32_t S = wgrad_splits(a.N1, N2, a.M, WGRAD_RESIDENT_SPLIT);  // also of two gradients, see wgrad_two_fits()
  SplitK p{};
  p.A1 = (const float*)a.A;
  p.lda1 = a.lda;
  p.A2 = (const float*)a.A2;
  p.half = a.A2 ? a.N1 : INT_MAX;
  p.B1 = (const float*)a.B;
  p.ldb1 = a.ldb;
  p.B2 = (const float*)a.B2;
  p.ldb2 = a.ldb2;
  p.n_split = a.B2 ? a.N2 : 0;
  p.K1 = a.M;
  p.C = a.workspace;
  p.ldc = N2;
  p.M = N1;
  p.N = N2;
  int64_t chunk = (a.M + S - 1) / S;
  p.k_chunk = ((chunk + SBK - 1) / SBK) * SBK;
  if (p.k_chunk < SBK) p.k_chunk = SBK;
  p.c_split_stride = (int64_t)N1 * N2;
  p.tiles_m = (N1 + TILE - 1) / TILE;
  p.tiles_n = (N2 + TILE - 1) / TILE;
  p.n_groups = S;
  float* colsum_part = a.workspace + (size_t)S * N1 * N2;
  p.colsum_part = a.colsum_out && !a.colsum_src ? colsum_part : nullptr;
  // Two gradients of up to 64 rows each would be a pair in gemm_narrow.hip, whose chunks are other ones and whose column sums are rounded once
  // a group of 32 nodes.  So column sums are formed in float64 inside a chunk, and the chunks' partials are added in float64: against
  // float64, errors of gradients over 17,000 to 1,000,000 nodes, 66 to 602 -> 33 to 64, are 0.47 to 0.68 of the pair's and of bias gradients 0.43 to
  // 0.76, where float32 sums had up to 1.11 and 1.41.  602 -> 64 over 300k nodes 395 -> 395 us, 256 -> 41 over 115k 71 -> 72.
  const bool narrow = a.A2 && a.N1 <= 64;
  p.colsum_f64 = narrow;
  COFREE_TRY(plan_colsum(a, &p.extra, sums));
  const int64_t blocks = (int64_t)((S + 7) / 8) * 8 * p.tiles_m * p.tiles_n + p.extra.blocks;
  COFREE_REQUIRE(blocks > 0 && blocks < ((int64_t)1 << 31), "wgrad: grid too large");
  {
    char pname[96] = "";
    if (profiling()) snprintf(pname, sizeof(pname), "gemm_split_kernel<true,true,false,false,%s> N=%dx%d", a.A2 ? "true" : "false", (int)N1, (int)N2);
    ProfScope prof(pname, stream, 4.0 * ((double)a.M * N1 * (p.extra.X ? 2 : 1) + (double)a.M * N2 + (double)N1 * N2),
                   2.0 * (double)a.M * N1 * N2);
    if (a.A2) gemm_split_kernel<true, true, false, false, true><<<dim3((unsigned)blocks), 256, 0, stream>>>(p);
    else gemm_split_kernel<true, true, false, false><<<dim3((unsigned)blocks), 256, 0, stream>>>(p);
  }
  COFREE_HIP_CHECK(hipGetLastError());
  COFREE_TRY(add_split_sum(sums, a.workspace, p.c_split_stride, S, a.C, a.ldc, a.N1, N2, narrow));
  if (a.A2) COFREE_TRY(add_split_sum(sums, a.workspace + (size_t)a.N1 * N2, p.c_split_stride, S, a.C2, a.ldc, a.N1, N2, narrow));
  if (p.colsum_part) COFREE_TRY(add_split_sum(sums, colsum_part, N1, S, a.colsum_out, a.N1, 1, a.N1, narrow));
  return COFREE_OK;
}

}  // namespace cofree
