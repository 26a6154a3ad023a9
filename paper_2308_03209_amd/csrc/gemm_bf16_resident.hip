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

// COFREE_BF16_TILE sends every product to the tiled kernel.
// At most 512 k, segments of at least eight, and parameters of at most four column parts.
bool gemm_resident_fits(const GemmArgs& a) {
  const int nch = pieces(a.K1) + (a.K2 > 0 ? pieces(a.K2) : 0);
  const int64_t strides = a.lda1 | a.lda2 | a.ldc | a.ldg;  // 32-bit offsets inside a tile of 32 rows
  return !getenv("COFREE_BF16_TILE") && a.N >= 32 && a.M >= 32 && strides < ((int64_t)1 << 26) && a.K1 >= 8 && (a.K2 == 0 || a.K2 >= 8) && nch <= 8 &&
         column_parts(a.N, nch) > 0;
}

// Dropout needs a lane's eight columns to start at a whole draw in every part, and a product that only writes.
bool gemm_resident_drops(const GemmArgs& a) {
  if (!gemm_resident_fits(a) || a.gate || a.accumulate) return false;
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
