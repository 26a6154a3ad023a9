// Launch of the products whose parameters fit LDS, and their instances for at most 128 columns.
#include <cstdio>

#include "gemm_bf16_resident.h"

namespace cofree {

bool launch_resident_narrow(int nb, int nch, bool extras, dim3 grid, hipStream_t stream, const ResidentK& p) {
  switch (nb) {
    case 2: return launch_resident_pieces<2, 8>(nch, extras, grid, stream, p);
    case 3: return launch_resident_pieces<3, 8>(nch, extras, grid, stream, p);
    case 4: return launch_resident_pieces<4, 8>(nch, extras, grid, stream, p);
    default: return false;
  }
}

static int pieces(int32_t K) { return (K + 63) / 64; }
static int col_blocks(int32_t N) { return N <= 64 ? 2 : (N <= 256 ? (N + 31) / 32 : 0); }

// Parameters of at most 128 KB in LDS (and at most 512 k), segments of at least eight k.
bool gemm_resident_fits(const GemmArgs& a) {
  const int nb = col_blocks(a.N), nch = pieces(a.K1) + (a.K2 > 0 ? pieces(a.K2) : 0);
  const int64_t strides = a.lda1 | a.lda2 | a.ldc | a.ldg;  // 32-bit offsets inside a tile of 32 rows
  return nb > 0 && a.N >= 32 && a.M >= 32 && strides < ((int64_t)1 << 26) && a.K1 >= 8 && (a.K2 == 0 || a.K2 >= 8) && nch <= 8 && nb * nch <= 32;
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
  const int nb = col_blocks(a.N), nch = pieces(a.K1) + (a.K2 > 0 ? pieces(a.K2) : 0);
  const int64_t K = (int64_t)a.K1 + a.K2, tiles = (a.M + 31) / 32;
  const dim3 grid((unsigned)(tiles < RES_CUS ? tiles : RES_CUS));
  char pname[96] = "";
  if (profiling()) snprintf(pname, sizeof(pname), "gemm_bf16_resident_kernel<%d,%d> N=%d K=%d", nb, nch, (int)a.N, (int)K);
  ProfScope prof(pname, stream, 2.0 * ((double)a.M * K + (double)a.N * K + (double)a.M * a.N * (a.accumulate ? 2 : 1)),
                 2.0 * (double)a.M * a.N * (double)K);
  const bool extras = a.gate || a.accumulate;
  const bool ok = nb <= 4 ? launch_resident_narrow(nb, nch, extras, grid, stream, p) : launch_resident_wide(nb, nch, extras, grid, stream, p);
  if (!ok) return fail(COFREE_EINVAL, "internal: no resident product of this shape");
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

}  // namespace cofree
