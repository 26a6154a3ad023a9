// Launch of the products whose parameters fit LDS, and their instances for at most 128 columns.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "gemm_bf16_resident.h"

namespace cofree {

bool launch_resident_narrow(int nb, int nch, int end, dim3 grid, hipStream_t stream, const ResidentK& p) {
  switch (nb) {
    case 2: return launch_resident_pieces<2, 8>(nch, end, grid, stream, p);
    case 3: return launch_resident_pieces<3, 8>(nch, end, grid, stream, p);
    case 4: return launch_resident_pieces<4, 8>(nch, end, grid, stream, p);
    default: return false;
  }
}

static int pieces(int32_t K) { return (K + 63) / 64; }
static int col_blocks(int32_t N) { return N <= 64 ? 2 : (N <= 256 ? (N + 31) / 32 : 0); }

// Column parts of at most 128 KB of parameters each: the fewest, up to four (0: they do not fit).
static int column_parts(int32_t N, int nch) {
  for (int parts = 1; parts <= 4; ++parts) {
    const int nb = col_blocks((N + parts - 1) / parts);
    if (nb > 0 && nb * nch <= 32) return parts;
  }
  return 0;
}

// Rows from which the resident kernel is the faster one.  Every workgroup first converts its parameters, row by row the
// slower (A B^T), while the tiled kernel (gemm_bf16.hip) has 128 or 256 columns in a tile, empty or not, and where a result has few of them 64,
// with parameters as they are: eight pieces of parameters (of 32 columns x 64 k) and more then take longer than the chain of a tile.  us of a
// GCN layer, tiled / resident: forward 300 -> 64 over 500 rows 11.7 / 13.5, 60k 26.0 / 28.6, 400 -> 40 over 30k 16.6 / 21.9; backward 256 -> 64 over 2,000
// 18.6 / 21.9, 30k 40.8 / 42.5, 128 -> 128 over 30k 35.4 / 36.4; fewer pieces: forward 64 -> 64 over 2,000 9.6 / 8.9, backward 90 -> 90 over 30k 36.0 / 35.1;
// more tiles: backward 300 -> 64 over 60k 60.9 / 54.5.  us of a launch
// and the aggregation beside it, tiled / resident: A B^T of 256 x 256 (columns x k) over 20k rows 23 / 36, 100k 57 / 69, 200k 127 / 123,
// 800k 452 / 431; 128 x 128 20k 15 / 17, 100k 34 / 34, 200k 54 / 51; 128 x 400 200k 88 / 90, 400k 195 / 183; 172 x 256 20k 28 / 31,
// 50k 46 / 42, 200k 137 / 101; 47 x 256 2k 16 / 12, 100k 45 / 40; 512 k everywhere slower: 512 x 512 200k 281 / 284, 1.6M
// 2012 / 2074; 380 x 276 140k 98 / 61.  A B (with the launches of the weight gradient): 128 x 128 20k 35 / 32, 100k 56 / 50; 172 x 256 20k 54 / 52, 100k
// 105 / 93; 256 x 256 20k 54 / 58, 100k 106 / 104, 200k 229 / 203; 256 x 172 100k 99 / 103, 200k 190 / 180; 512 x 512 20k 74 / 80, 100k
// 231 / 225; 130 x 129, where a quarter of the k is padding, 100k 110 / 116, 200k 184 / 176.  Dropout would be a pass of its own
// beside the tiled kernel (100k x 128: 15 us).
static int64_t resident_min_rows(int32_t N, int32_t K, int nch, bool kmajor, bool drop) {
  const int param = (N + 31) / 32 * nch;  // of 32 columns x 64 k
  const bool tiles_empty = N <= 64 || 4 * (int64_t)((N + 127) / 128 * 128) >= 5 * (int64_t)N;
  if (kmajor) return param <= 8 || (tiles_empty && 4 * 64 * nch <= 5 * K) ? 0 : 1 << 17;
  if (drop) return param <= 8 ? 0 : 1 << 15;
  if (nch >= 8) return INT64_MAX;
  if (tiles_empty) return N <= 64 ? 0 : 1 << 15;
  return param <= 24 || (nch == 5 && N > 256 && N <= 384) ? 1 << 17 : 1 << 18;
}

// Where the rows are few, though, and there are eight pieces and more: tiles store the ragged end of a row element by element, and read
// parameters [k][column] in single floats; the resident kernel reads rows of odd length slowly, which many rows show.  Layers, tiled / resident:
// A B of up to 64 columns GCN backward 33 -> 200 over 2,000 25.4 / 24.2, 64 -> 200 over 20k 34.1 / 33.4, 64 -> 193 over 20k 0.87, 45 -> 500 over 2,000 32.2 / 30.1,
// 63 -> 300 over 20k 41.3 / 39.7;
// A B^T of 45 columns and 251 k over 2,000 1.22 (33 columns 1.01, 64 1.04, 45 over 20k 1.01), of 63 and 224 over 20k 20.8 / 19.4, conventional GraphSAGE 256 -> 45 over 2,000 forward 24.9 / 23.2;
// A B of 65 to 128 GCN backward 77 -> 181 over 2,000 30.1 / 27.8, 86 -> 300 over 7,000 37.6 / 36.1, 117 -> 117 over 2,000 28.6 / 26.9 (96 -> 184 0.99, 104 -> 117
// 0.98), conventional GraphSAGE 93 -> 181 over 7,000 49.6 / 45.1.
static bool few_resident(const GemmArgs& a, int nch) {
  const bool ragged = a.N % 8 > 1;
  if (a.N > 64) return a.b_kmajor && ragged && nch <= (a.N <= 96 ? 6 : a.N <= 128 ? 3 : 0);
  const bool few = a.M < 1 << 14, even = (a.K1 | a.K2) % 2 == 0;
  if (!a.b_kmajor) return ragged && nch <= 4 && (few || even);
  return few ? ragged || nch <= 4 : even && nch <= (ragged ? 5 : 4);
}

// At most 512 k, segments of at least eight, parameters of at most four column parts, and rows as above.
// COFREE_BF16_TILE = 0 takes every product that fits, any other none.
static bool resident_fits(const GemmArgs& a, bool drop) {
  const int nch = pieces(a.K1) + (a.K2 > 0 ? pieces(a.K2) : 0);
  const int64_t strides = a.lda1 | a.lda2 | a.ldc | a.ldg;  // 32-bit offsets inside a tile of 32 rows
  int64_t rows = resident_min_rows(a.N, a.K1 + a.K2, nch, a.b_kmajor != 0, drop);
  if (!drop && (a.N + 31) / 32 * nch >= 8 && gemm_bf16_few(a.M, a.N) && !few_resident(a, nch)) rows = INT64_MAX;
  if (const char* e = getenv("COFREE_BF16_TILE")) {
    if (atoi(e) != 0) return false;
    rows = 0;
  }
  return a.N >= 32 && a.M >= 32 && a.M >= rows && strides < ((int64_t)1 << 26) && a.K1 >= 8 && (a.K2 == 0 || a.K2 >= 8) && nch <= 8 &&
         column_parts(a.N, nch) > 0;
}
bool gemm_resident_fits(const GemmArgs& a) { return resident_fits(a, a.dropout.q > 0.f); }

// Dropout needs a lane's eight columns to start at a whole draw in every part, and a product that only writes.
bool gemm_resident_drops(const GemmArgs& a) {
  if (!resident_fits(a, true) || a.gate || a.accumulate) return false;
  return a.N % (4 * column_parts(a.N, pieces(a.K1) + (a.K2 > 0 ? pieces(a.K2) : 0))) == 0;
}

int32_t launch_gemm_resident(const GemmArgs& a, hipStream_t stream) {
  ResidentK p{};
  p.A1 = (const bf16_t*)a.A1;
  p.lda1 = a.lda1;
  p.K1 = a.K1;
  p.A2 = (const bf16_t*)a.A2;
  p.lda2 = a.lda2;
  p.K2 = a.K2;
  p.nch1 = pieces(a.K1);
  p.W1 = a.B;
  p.ldw1 = a.ldb;
  p.W2 = a.B2 ? a.B2 : a.B + (a.b_kmajor ? (int64_t)a.K1 * a.ldb : (int64_t)a.K1);
  p.ldw2 = a.B2 ? a.ldb2 : a.ldb;
  p.kmajor = a.b_kmajor;
  p.C = (bf16_t*)a.C;
  p.ldc = a.ldc;
  p.M = a.M;
  p.N = a.N;
  p.bias = a.bias;
  p.relu = a.relu;
  p.row_scale = a.row_scale;
  p.gate = (const bf16_t*)a.gate;
  p.ldg = a.ldg;
  p.accumulate = a.accumulate;
  p.relu_last = a.relu_last;
  p.gate_last = a.gate_last;
  p.gate_scale = a.gate ? a.gate_scale : 1.f;
  p.drop = dropout_k(a.dropout);
  const int nch = pieces(a.K1) + (a.K2 > 0 ? pieces(a.K2) : 0);
  const int64_t K = (int64_t)a.K1 + a.K2, tiles = (a.M + 31) / 32;
  p.parts = column_parts(a.N, nch);
  const int nb = col_blocks((a.N + p.parts - 1) / p.parts);
  // a workgroup per CU; with several parts the teams come eight at a time, one on each XCD
  p.teams = tiles < RES_CUS ? tiles : RES_CUS;
  if (p.parts > 1) p.teams = 8 * std::min<int64_t>((tiles + 7) / 8, RES_CUS / 8 / p.parts);
  const dim3 grid((unsigned)(p.teams * p.parts));
  const int end = a.gate || a.accumulate ? RES_EXTRAS : (p.drop.scale != 0.f ? RES_DROP : RES_PLAIN);
  char pname[96] = "";
  if (profiling()) snprintf(pname, sizeof(pname), "gemm_bf16_resident_kernel<%d,%d,%d> N=%d K=%d", nb, nch, end, (int)a.N, (int)K);
  ProfScope prof(pname, stream, 2.0 * ((double)a.M * K + (double)a.N * K + (double)a.M * a.N * (a.accumulate ? 2 : 1)),
                 2.0 * (double)a.M * a.N * (double)K);
  const bool ok = nb <= 4 ? launch_resident_narrow(nb, nch, end, grid, stream, p) : launch_resident_wide(nb, nch, end, grid, stream, p);
  if (!ok) return fail(COFREE_EINVAL, "internal: no resident product of this shape");
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

}  // namespace cofree
