// Partial column sums (bias gradients whose operand no weight gradient of the layer reads): a workgroup of 256
// threads sums one chunk of rows of one panel of 256 columns.  Run by extra workgroups at the end of a weight-gradient
// launch (see WgradArgs::colsum_src): they fill its last, partly empty round (470k x 47 float32: the launch 328 -> 336 us
// where the two launches for the sums took 70; at its front they held up the others, 443 us).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace cofree {

struct ColsumK {
  const void* X;  // [M, N] (ld), or null: no extra workgroups
  int64_t ld, M;
  int32_t N;
  int32_t splits, panels;
  int32_t blocks;  // splits * panels
  int64_t rows_per_split;
  float* partial;  // [splits][N]
};

__device__ inline void colsum_ld4(const float* p, float (&v)[4]) {
  typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
  const f32x4 t = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = t[i];
}
__device__ inline void colsum_ld4(const bf16_t* p, float (&v)[4]) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(2)));
  const u32x2 t = *reinterpret_cast<const u32x2*>(p);
  v[0] = __uint_as_float(t[0] << 16), v[1] = __uint_as_float(t[0] & 0xffff0000u);
  v[2] = __uint_as_float(t[1] << 16), v[3] = __uint_as_float(t[1] & 0xffff0000u);
}
__device__ inline float colsum_ld1(const float* p) { return *p; }
__device__ inline float colsum_ld1(const bf16_t* p) { return bf16_to_f32(*p); }

// LPR lanes share a row - 16 for at most 64 columns, 32 for 128, else 64 - each owning four columns of the panel; the
// 4 * 64 / LPR row groups of the workgroup take rows in turn, eight requested before the first is added (one dependent
// load per iteration leaves the loop waiting on memory), and are added in order through LDS (sm: 1024 floats).
template <typename T>
__device__ inline void colsum_block(const ColsumK& p, int64_t b, float* sm, int tid) {
  const int lpr = p.N <= 64 ? 16 : (p.N <= 128 ? 32 : 64), groups = 256 / lpr;
  const int quad = tid % lpr, grp = tid / lpr;
  const int64_t split = b / p.panels;
  const int32_t c0 = (int32_t)(b % p.panels) * 256;
  const int64_t r0 = split * p.rows_per_split;
  const int64_t r1 = r0 + p.rows_per_split < p.M ? r0 + p.rows_per_split : p.M;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  const int avail = p.N - (c0 + 4 * quad);
  if (avail > 0) {
    const T* src = (const T*)p.X + c0 + 4 * quad;
    int64_t r = r0 + grp;
    if (avail >= 4) {
      for (; r + 7 * groups < r1; r += 8 * groups) {
        float v[8][4];
#pragma unroll
        for (int u = 0; u < 8; ++u) colsum_ld4(src + (r + u * groups) * p.ld, v[u]);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[q] += v[u][q];
      }
    }
    for (; r < r1; r += groups) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q < avail) acc[q] += colsum_ld1(src + r * p.ld + q);
    }
  }
  *reinterpret_cast<float4*>(sm + (grp * lpr + quad) * 4) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  __syncthreads();
  const int c = tid;
  if (c < 4 * lpr && c0 + c < p.N) {
    float t = sm[c];
    for (int g = 1; g < groups; ++g) t += sm[g * lpr * 4 + c];
    p.partial[split * p.N + c0 + c] = t;
  }
}

}  // namespace cofree
