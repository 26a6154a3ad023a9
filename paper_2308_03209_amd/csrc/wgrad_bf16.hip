// Weight gradients of bfloat16 activations, C[N1, N2 + N2b] = A^T [B | B2] over the graph nodes, float32 partials per
// chunk of nodes.
//
// Bound by the bytes of A and B, so on large graphs the tile of the result is as large as a CU's registers hold - 256 x 256
// in eight wavefronts, 128 accumulators each - and every operand row is read once per launch where the result fits a tile
// (wgrad_tile has the rule for smaller ones).
// A workgroup per CU streams its chunk in steps of 32 or 64 nodes: 16-byte pieces of rows go through a ring of registers
// (80 to 96 KB in flight per CU) into LDS as they lie in memory, [node][column], double-buffered with one barrier per
// step.  The matrix instructions want eight consecutive nodes of one column per lane: the transposing LDS read
// (ds_read_b64_tr_b16: the sixteen lanes of a group read four rows of sixteen columns and receive a column each)
// delivers four at a time.  Rows are 64 bytes apart modulo 256, so that the four rows and both column halves that
// thirty-two lanes read lie in different banks.
//
// Measured against 128 x 128 tiles of four wavefronts (each operand read once per tile, scattered into LDS by the
// writer): 2.35M nodes, 256 x 256 725 -> 438 us (5.5 TB/s), 172 x 256 with the column sums of a third matrix 691 -> 518;
// 1.88M nodes, 256 x (256 + 256) 759 -> 536, 47 x 256 263 -> 229; 100k nodes, 47 x 128 23 -> 17.
#include <algorithm>
#include <cstdio>

#include "colsum.h"
#include "common.h"

namespace cofree {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));

constexpr int WG_WAVES = 8, WG_CUS = 256;

struct WgradK {
  const bf16_t* A;
  const bf16_t* B;
  const bf16_t* B2;
  int64_t lda, ldb, ldb2;
  int32_t N1, N2, N2b;  // columns of the three matrices (N2b = 0: no second one)
  int64_t M, chunk;
  float* C;  // partials: [chunks][N1 (two: + N1b)][N2 + N2b]
  int32_t tiles_m, tiles_n;
  int64_t n_chunks;
  float* colsum_part;  // [chunks][N1] partial column sums of A, or null
  ColsumK extra;
  const bf16_t* A2;  // TWO: a second matrix like A, of N1b columns
  int32_t N1b;
};

// Places of operand columns: pieces of eight, the last piece of a matrix moved left to end with its rows (the columns it
// shares with the piece before are computed twice and stored once), the pieces of a second matrix behind those of the first.
struct Piece {
  int32_t col;    // first column inside its matrix
  int32_t first;  // columns of it that belong to the piece before
  bool second;    // a piece of the second matrix
  bool exists;
};
__device__ inline Piece piece_of(int q, int32_t N, int32_t Nb) {
  const int own = (N + 7) >> 3, all = own + ((Nb + 7) >> 3);
  Piece x;
  x.exists = q < all;
  if (q >= all) q = all - 1;
  x.second = q >= own;
  const int32_t c = 8 * (x.second ? q - own : q), end = x.second ? Nb : N;
  x.col = c < end - 8 ? c : end - 8;
  x.first = c - x.col;
  return x;
}

// TM x TN: tile of the result; SN: nodes per step; D: steps in flight; WM x WN: wavefronts over the tile.
// PARTS: of a thread's column sums - two where two matrices A share a tile of twice the rows that one of them would take, in which a
// thread has twice the nodes of a column.  TWO: of two matrices A (instances of their own: looking for the second one in every launch cost
// 0.3 to 1.5 us: backward of 602 -> 33 over 20k nodes 45.7 -> 47.2, of 1000 -> 24 over 6,000 39.2 -> 40.3).
template <int TM, int TN, int SN, int D, int WM, int WN, int PARTS, bool TWO>
__global__ __launch_bounds__(64 * WG_WAVES) __attribute__((amdgpu_waves_per_eu(2))) void wgrad_bf16_kernel(
    const WgradK p) {
  static_assert(WM * WN == WG_WAVES, "eight wavefronts");
  constexpr int T = 64 * WG_WAVES;
  constexpr int PA = TM * 2 + 64, PB = TN * 2 + 64;  // bytes between rows in LDS
  constexpr int STEP = SN * (PA + PB);
  constexpr int QA = TM / 8, QB = TN / 8;                // pieces of a row
  constexpr int JA = SN * QA / T, JB = SN * QB / T;      // pieces of a step that a thread moves
  static_assert(JA * T == SN * QA && JB * T == SN * QB, "whole pieces");
  constexpr int RM = TM / WM / 32, RN = TN / WN / 32;  // 32 x 32 blocks of a wavefront
  static_assert(PARTS == 1 || JA == 2 || (JA == 1 && D % 2 == 0), "a part is a thread's piece of a step, or every other step");
  constexpr int RED = PARTS * (T / QA) * TM * 4;       // column sums: one row of the tile per thread group and part
  __shared__ __attribute__((aligned(128))) unsigned char smem[2 * STEP > RED ? 2 * STEP : RED];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int64_t L = blockIdx.x;
  const int per_chunk = p.tiles_m * p.tiles_n;
  // the tiles of a chunk read the same rows: they lie next to each other on one XCD
  const int64_t own = ((p.n_chunks + 7) / 8) * 8 * per_chunk;
  if (L >= own) {  // one workgroup of colsum_block's 256 threads in each half
    const int64_t b = (L - own) * 2 + (tid >> 8);
    // (the last workgroup's second half repeats the last block: both halves meet its barrier)
    colsum_block<bf16_t>(p.extra, b < p.extra.blocks ? b : p.extra.blocks - 1, reinterpret_cast<float*>(smem) + (tid >> 8) * 1024,
                         tid & 255);
    return;
  }
  const int64_t z = (L / (8 * per_chunk)) * 8 + (L & 7);
  const int member = (int)((L >> 3) % per_chunk);
  if (z >= p.n_chunks) return;  // padding of the last octet (uniform over the block)
  const int32_t N1b = TWO ? p.N1b : 0;
  const int qm = (member / p.tiles_n) * QA, qn = (member % p.tiles_n) * QB;  // first pieces of the tile
  const int64_t k_beg = z * p.chunk;
  const int64_t k_end = k_beg + p.chunk < p.M ? k_beg + p.chunk : p.M;
  const int k_len = (int)(k_end > k_beg ? k_end - k_beg : 0);

  floatx16 acc[RM][RN];
#pragma unroll
  for (int m = 0; m < RM; ++m)
#pragma unroll
    for (int n = 0; n < RN; ++n)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[m][n][v] = 0.f;
  float csum[PARTS][8] = {};
  const bool colsum = p.colsum_part != nullptr && qn == 0;

  // thread t moves piece t % Q of rows t / Q + (T / Q) j of a step; rows past the chunk repeat its last one (and become
  // zero on the way to LDS)
  const int ra = tid / QA, rb = tid / QB;
  const Piece xa = piece_of(qm + tid % QA, p.N1, N1b), xb = piece_of(qn + tid % QB, p.N2, p.N2b);
  const int64_t ldb = xb.second ? p.ldb2 : p.ldb;
  const bf16_t* const pa = (TWO && xa.second ? p.A2 : p.A) + k_beg * p.lda + xa.col;
  const bf16_t* const pb = (xb.second ? p.B2 : p.B) + k_beg * ldb + xb.col;
  struct Raw {
    u32x4u a[JA], b[JB];
  } ring[D];
  auto load = [&](int k0, Raw& w) {
#pragma unroll
    for (int j = 0; j < JA; ++j) {
      const int k = k0 + ra + (T / QA) * j;
      w.a[j] = *reinterpret_cast<const u32x4u*>(pa + (int64_t)(k < k_len ? k : k_len - 1) * p.lda);
    }
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int k = k0 + rb + (T / QB) * j;
      w.b[j] = *reinterpret_cast<const u32x4u*>(pb + (int64_t)(k < k_len ? k : k_len - 1) * ldb);
    }
  };
  const int to_a = ra * PA + (tid % QA) * 16, to_b = SN * PA + rb * PB + (tid % QB) * 16;
  auto store = [&](int k0, unsigned char* d, Raw& w, int s) __attribute__((always_inline)) {
    if (k0 + SN > k_len) {  // uniform: the chunk ends inside this step
#pragma unroll
      for (int j = 0; j < JA; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) w.a[j][c] = k0 + ra + (T / QA) * j < k_len ? w.a[j][c] : 0u;
#pragma unroll
      for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) w.b[j][c] = k0 + rb + (T / QB) * j < k_len ? w.b[j][c] : 0u;
    }
#pragma unroll
    for (int j = 0; j < JA; ++j) {
      *reinterpret_cast<uint4*>(d + to_a + (T / QA) * j * PA) = make_uint4(w.a[j][0], w.a[j][1], w.a[j][2], w.a[j][3]);
      if (colsum) {
        float (&sum)[8] = csum[PARTS == 2 && (JA == 2 ? j : s & 1) == 1 ? PARTS - 1 : 0];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          sum[2 * c] += __uint_as_float(w.a[j][c] << 16);
          sum[2 * c + 1] += __uint_as_float(w.a[j][c] & 0xffff0000u);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < JB; ++j)
      *reinterpret_cast<uint4*>(d + to_b + (T / QB) * j * PB) = make_uint4(w.b[j][0], w.b[j][1], w.b[j][2], w.b[j][3]);
  };
  // transposing read: lane l asks for four columns 16 (l / 16 % 2) + 4 (l % 4) of row 8 (l / 32) + l / 4 % 4 and receives
  // rows 8 (l / 32) .. + 3 of column l % 32
  const int tr = 8 * (lane >> 5) + ((lane >> 2) & 3), tc = (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
  const int from_a = tr * PA + tc + wm * RM * 64, from_b = SN * PA + tr * PB + tc + wn * RN * 64;
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  auto operand = [&](const unsigned char* at, int pitch) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + 4 * pitch));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto multiply = [&](const unsigned char* d) {
#pragma unroll
    for (int s = 0; s < SN / 16; ++s) {
      bf16x8 b[RN];
#pragma unroll
      for (int n = 0; n < RN; ++n) b[n] = operand(d + from_b + s * 16 * PB + n * 64, PB);
#pragma unroll
      for (int m = 0; m < RM; ++m) {
        const bf16x8 a = operand(d + from_a + s * 16 * PA + m * 64, PA);
#pragma unroll
        for (int n = 0; n < RN; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[n], acc[m][n], 0, 0, 0);
      }
    }
  };

  const int n = (k_len + SN - 1) / SN;
  if (n > 0) {
    // loads past the end repeat the last step, which keeps the count of loads in flight the same on every path
    auto step = [&](int t, int s, bool refill) {
      unsigned char* const d = smem + (t & 1) * STEP;
      store(t * SN, d, ring[s], s);
      if (refill) load((t + D < n ? t + D : n - 1) * SN, ring[s]);
      __syncthreads();
      multiply(d);
    };
#pragma unroll
    for (int s = 0; s < D; ++s) load((s < n ? s : n - 1) * SN, ring[s]);
    int t0 = 0;
#pragma nounroll
    for (; t0 + D <= n; t0 += D) {
#pragma unroll
      for (int s = 0; s < D; ++s) step(t0 + s, s, true);
    }
#pragma unroll
    for (int s = 0; s < D - 1; ++s)
      if (t0 + s < n) step(t0 + s, s, false);
  }

  // accumulator register v of lane (g, r) is element [8 (v / 4) + 4 g + v % 4][r] of its 32 x 32 block
  const int g = lane >> 5, r = lane & 31;
  const int64_t ldc = (int64_t)p.N2 + p.N2b;
  float* const Cz = p.C + z * (p.N1 + N1b) * ldc;
#pragma unroll
  for (int q = 0; q < RN; ++q) {
    const int place = (wn * RN + q) * 32 + r;
    const Piece xc = piece_of(qn + (place >> 3), p.N2, p.N2b);
    if (!xc.exists || (place & 7) < xc.first) continue;
    const int64_t j = (xc.second ? p.N2 : 0) + xc.col + (place & 7);
#pragma unroll
    for (int m = 0; m < RM; ++m)
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const Piece xr = piece_of(qm + (wm * RM + m) * 4 + h, p.N1, N1b);
        const int32_t row = (TWO && xr.second ? p.N1 : 0) + xr.col + 4 * g;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (xr.exists && 4 * g + v >= xr.first) Cz[(int64_t)(row + v) * ldc + j] = acc[m][q][4 * h + v];
      }
  }
  if (colsum) {
    // the threads that hold the same piece are added in order
    float* const red = reinterpret_cast<float*>(smem);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PARTS; ++q)
#pragma unroll
      for (int c = 0; c < 8; ++c) red[(q * (T / QA) + ra) * TM + (tid % QA) * 8 + c] = csum[q][c];
    __syncthreads();
    if (tid < TM) {
      float t = 0.f;
      for (int h = 0; h < PARTS * (T / QA); ++h) t += red[h * TM + tid];
      const Piece xr = piece_of(qm + (tid >> 3), p.N1, N1b);
      if (xr.exists && !(TWO && xr.second) && (tid & 7) >= xr.first) p.colsum_part[z * p.N1 + xr.col + (tid & 7)] = t;
    }
  }
}

static int32_t pieces_of(int32_t N) { return (N + 7) / 8; }

// Tile of the result (rows x columns, and how many).  The larger it is the less is read, but a workgroup per CU then means
// more and shorter chunks, each with a ramp, a barrier per step that no other workgroup hides and a partial result of its
// own (256 x 256 over 20k nodes: 256 chunks of 78 nodes and 64 MB of partials).  So small graphs take 128 x 128, as long as
// the operands are not read too often for it, and results of up to 256 x 256 over middling ones 128 x 256.  Measured in
// us of the layer's two launches, 128 x 128 / 128 x 256 / 256 x 256 (and 128 x 128 of four wavefronts, gemm_bf16.hip):
// 256 x 256 over 20k nodes 19 / 21 / 30 (21), 100k 30 / 33 / 41 (36), 400k 92 / 92 / 109 (102), 800k 182 / 163 / 175 (186),
// 1.6M 353 / 316 / 307 (375); 512 x 300 over 20k 30 / 28 / 31 (38), 50k 54 / 44 / 44 (57), 100k 94 / 74 / 69 (89).
struct WgradTile {
  int32_t h, w, m, n;
};
// rows, columns: in whole pieces
static WgradTile wgrad_tile(int32_t rows, int32_t columns, int64_t M) {
  const int32_t small = ((rows + 127) / 128) * ((columns + 127) / 128);  // tiles of 128 x 128
  const bool narrow = M < (1 << 17) && (small <= 10 || M < (1 << 15)), middling = small <= 4 && M < (1 << 20);
  WgradTile t;
  t.h = rows <= 64 ? 64 : (rows <= 128 || narrow || middling ? 128 : 256);
  t.w = columns <= 128 || narrow ? 128 : 256;
  t.m = (rows + t.h - 1) / t.h;
  t.n = (columns + t.w - 1) / t.w;
  return t;
}

// Chunks of nodes: a whole number of rounds of a workgroup per CU, enough of them for walks of at most about 16k nodes
// (over longer ones the tiles of a chunk drift apart and each fetches its rows from memory), chunks of at least 64.
// A chunk's tiles are on one XCD, which has 32 CUs: three tiles and 85 chunks were 33 workgroups on some.
static int32_t wgrad_chunks(int32_t tiles, int64_t M) {
  const int64_t per_round = tiles <= WG_CUS / 8 ? 8 * (WG_CUS / 8 / tiles) : std::max(1, WG_CUS / tiles);
  const int64_t walks = std::min<int64_t>((M + 16383) / 16384, 2048);
  int64_t s = per_round * std::max<int64_t>(1, (walks + per_round - 1) / per_round);
  s = std::min<int64_t>(s, (M + 63) / 64);
  return (int32_t)std::max<int64_t>(1, s);
}

bool wgrad_bf16_fits(int32_t N1, int32_t N2, int32_t N2b) { return N1 >= 8 && N2 >= 8 && (N2b == 0 || N2b >= 8); }

// Tile and chunks of the gradient of one matrix A.  A launch of two has larger tiles but the same chunks (see wgrad_two_fits()).
static WgradTile tile_of_one(int32_t N1, int32_t N2, int32_t N2b, int64_t M) {
  return wgrad_tile(8 * pieces_of(N1), 8 * (pieces_of(N2) + pieces_of(N2b)), M);
}

size_t wgrad_bf16_workspace_floats(int32_t N1, int32_t N2, int32_t N2b, int64_t M) {
  const WgradTile t = tile_of_one(N1, N2, N2b, M);
  return (size_t)wgrad_chunks(t.m * t.n, M) * ((size_t)N1 * ((size_t)N2 + N2b) + (size_t)N1);
}

template <int PARTS, bool TWO>
static void launch_tile(int32_t th, int32_t tw, unsigned blocks, const WgradK& p, hipStream_t stream) {
  const dim3 grid(blocks);
  if (tw == 256 && th == 256) wgrad_bf16_kernel<256, 256, 32, 3, 2, 4, PARTS, TWO><<<grid, 64 * WG_WAVES, 0, stream>>>(p);
  else if (tw == 256 && th == 128) wgrad_bf16_kernel<128, 256, 32, 4, 2, 4, PARTS, TWO><<<grid, 64 * WG_WAVES, 0, stream>>>(p);
  else if (th == 256) wgrad_bf16_kernel<256, 128, 32, 4, 4, 2, PARTS, TWO><<<grid, 64 * WG_WAVES, 0, stream>>>(p);
  else if (th == 128) wgrad_bf16_kernel<128, 128, 32, 6, 2, 4, PARTS, TWO><<<grid, 64 * WG_WAVES, 0, stream>>>(p);
  else if (tw == 256) wgrad_bf16_kernel<64, 256, 64, 2, 1, 8, 1, TWO><<<grid, 64 * WG_WAVES, 0, stream>>>(p);
  else wgrad_bf16_kernel<64, 128, 64, 4, 2, 4, 1, TWO><<<grid, 64 * WG_WAVES, 0, stream>>>(p);
}

int32_t launch_wgrad_bf16_rows(const WgradArgs& a, SplitSums* sums, hipStream_t stream) {
  WgradK p{};
  p.A = (const bf16_t*)a.A;
  p.lda = a.lda;
  p.B = (const bf16_t*)a.B;
  p.ldb = a.ldb;
  p.B2 = (const bf16_t*)a.B2;
  p.ldb2 = a.ldb2;
  p.N1 = a.N1;
  p.A2 = (const bf16_t*)a.A2;
  p.N1b = a.A2 ? a.N1 : 0;
  p.N2 = a.N2;
  p.N2b = a.B2 ? a.N2b : 0;
  p.M = a.M;
  const int32_t N2 = p.N2 + p.N2b;
  const int32_t rows = 8 * (pieces_of(p.N1) + pieces_of(p.N1b));
  WgradTile tile = wgrad_tile(rows, 8 * (pieces_of(p.N2) + pieces_of(p.N2b)), a.M);
  // With the chunks of one gradient a tile of both is no workgroup more: 100 x 256 over 300,000 nodes 120 us in two tiles of 128 rows, 109 in
  // one of 256 (but over 2,000, 16 chunks a tile, 15 and 17).
  if (a.A2 && rows > 128 && a.M >= 1 << 17) tile.h = 256, tile.m = 1;
  p.tiles_m = tile.m;
  p.tiles_n = tile.n;
  const WgradTile one = tile_of_one(p.N1, p.N2, p.N2b, a.M);
  const bool apart = one.h < tile.h;
  const int32_t S = wgrad_chunks(one.m * one.n, a.M);
  p.n_chunks = S;
  p.chunk = std::max<int64_t>(1, (((a.M + S - 1) / S) + 31) / 32 * 32);
  p.C = a.workspace;
  const int32_t N1 = p.N1 + p.N1b;
  float* const colsum_part = a.workspace + (size_t)S * N1 * N2;
  p.colsum_part = a.colsum_out && !a.colsum_src ? colsum_part : nullptr;
  COFREE_TRY(plan_colsum(a, &p.extra, sums));
  const int64_t blocks = ((p.n_chunks + 7) / 8) * 8 * p.tiles_m * p.tiles_n + (p.extra.blocks + 1) / 2;
  COFREE_REQUIRE(blocks > 0 && blocks < ((int64_t)1 << 31) && p.chunk < ((int64_t)1 << 31), "wgrad: grid too large");
  const int32_t th = tile.h, tw = tile.w;
  {
    char pname[96] = "";
    const char* rest = tw == 256 ? (th == 256 ? "32,3,2,4" : (th == 128 ? "32,4,2,4" : "64,2,1,8"))
                                 : (th == 256 ? "32,4,4,2" : (th == 128 ? "32,6,2,4" : "64,4,2,4"));
    if (profiling()) snprintf(pname, sizeof(pname), "wgrad_bf16_kernel<%d,%d,%s,%d,%s> N=%dx%d", (int)th, (int)tw, rest, apart ? 2 : 1, a.A2 ? "true" : "false", (int)N1, (int)N2);
    ProfScope prof(pname, stream, 2.0 * ((double)a.M * N1 * (p.extra.X ? 2 : 1) + (double)a.M * N2) + 4.0 * (double)N1 * N2,
                   2.0 * (double)a.M * N1 * N2);
    if (apart) launch_tile<2, true>(th, tw, (unsigned)blocks, p, stream);
    else if (a.A2) launch_tile<1, true>(th, tw, (unsigned)blocks, p, stream);
    else launch_tile<1, false>(th, tw, (unsigned)blocks, p, stream);
  }
  COFREE_HIP_CHECK(hipGetLastError());
  COFREE_TRY(add_split_sum(sums, a.workspace, (int64_t)N1 * N2, S, a.C, a.ldc, a.N1, N2));
  if (a.A2) COFREE_TRY(add_split_sum(sums, a.workspace + (size_t)a.N1 * N2, (int64_t)N1 * N2, S, a.C2, a.ldc, a.N1, N2));
  if (p.colsum_part) COFREE_TRY(add_split_sum(sums, colsum_part, a.N1, S, a.colsum_out, a.N1, 1, a.N1));
  return COFREE_OK;
}

}  // namespace cofree
