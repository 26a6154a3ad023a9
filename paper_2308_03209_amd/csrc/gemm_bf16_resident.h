// Products of bfloat16 activations with parameters, C = sum of segments A op(W), for parameters that fit LDS.
//
// These products are bound by the bytes of A and C (1.9M rows x 256 x 256: 1.9 GB moved for 0.25 TFLOP).  So every CU
// keeps one workgroup of eight wavefronts for the whole launch, which converts the parameters to bfloat16 into LDS
// once (up to 128 KB; no launch of its own for the conversion), and the wavefronts then stream rows past them, each
// on its own and without a barrier: a wavefront multiplies 32 rows by all columns, its rows of A come from memory
// straight into the registers the matrix instructions read them from, and the registers of a piece of 64 k are
// refilled with the next 32 rows' piece as soon as its instructions are issued, so that about 16 KB per wavefront are
// always in flight - also while results are written.
//
// Measured against the tiled kernel (gemm_bf16.hip), counted bytes over the time of a launch: 1.88M rows, N x K = 256 x 256
// 3.6-3.8 -> 4.9 TB/s, 256 x 128 4.3 -> 5.1, 47 x 256 3.7 -> 4.8, 128 x 94 2.6 -> 3.2, 172 x 256 2.6 -> 3.8; a copy of
// rows by the same access pattern reaches 5.3.  What it took: waiting for the next rows with the count of stores issued
// behind them, so that the stores are not waited for (8 waves do not hide that); whole 128-byte lines of C per store
// instruction; a row factor that arrives with the rows; no register spilled (a scratch frame costs 20 %).
//
// Parameters beyond 128 KB are cut by columns into two to four parts, each resident in its own workgroups.  The workgroups
// of one group of rows lie next to each other on one XCD and walk the rows alike, so the rows come from memory once and
// from that XCD's L2 for the others.  Measured, 1.88M rows to 256 columns, against the tiled
// kernel: K = 356 684 -> 598 us, 303 649 -> 481, 512 717 -> 711.  Over many rows parameters of more than 256 k now lie in registers
// (gemm_bf16_pinned.hip: 479, 427 and 587); parts remain for more than 256 columns of fewer k, fewer rows, and sums in place.

// The first matrix operand is the parameter block, the second the rows: a lane then holds four consecutive columns of
// one row at a time, and passes 32 x 32 results through 4 KB of LDS of its wavefront (float32, 16-byte pieces permuted
// by row so that both directions are free of bank conflicts) to hold eight consecutive columns.
#pragma once

#include "common.h"

namespace cofree {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));

constexpr int RES_WAVES = 8, RES_CUS = 256;

struct ResidentK {
  const bf16_t* A1;
  const bf16_t* A2;
  int64_t lda1, lda2;
  int32_t K1, K2;  // lengths of the segments (K2 = 0: one)
  int32_t nch1;    // pieces of 64 k of the first segment
  const float* W1;
  const float* W2;
  int64_t ldw1, ldw2;
  int32_t kmajor;  // element (column n, k) of W at W[k ld + n] instead of W[n ld + k]
  bf16_t* C;
  int64_t ldc, M;
  int32_t N;
  int32_t parts;  // column parts
  int64_t teams;  // groups of `parts` workgroups that share their rows
  const float* bias;
  int32_t relu;
  const float* row_scale;
  const bf16_t* gate;
  int64_t ldg;
  int32_t accumulate, relu_last, gate_last;
  float gate_scale;
  DropoutK drop;
};

// 128-bit value >> 16 * halves (0 .. 8), without branches
__device__ inline u32x4u shift_halves(const u32x4u& w, int halves) {
  const uint64_t lo = (uint64_t)w[0] | ((uint64_t)w[1] << 32), hi = (uint64_t)w[2] | ((uint64_t)w[3] << 32);
  const int bits = 16 * halves, b = bits & 63;
  const uint64_t spill = b ? hi << (64 - b) : 0;
  const uint64_t l1 = (lo >> b) | spill, h1 = hi >> b;
  const uint64_t rl = bits >= 128 ? 0 : (bits >= 64 ? h1 : l1), rh = bits >= 64 ? 0 : h1;
  return u32x4u{(uint32_t)rl, (uint32_t)(rl >> 32), (uint32_t)rh, (uint32_t)(rh >> 32)};
}

// NB: 32-column blocks of a part, 32 (NB - 1) <= its columns <= 32 NB (two for 32 columns); NCH: pieces of 64 k over both segments.
// LDS parameters: [k-group of 8][column][8 bfloat16]: a matrix operand is 512 contiguous bytes per half wavefront.
// END: RES_EXTRAS - the result is gated by another matrix or accumulated; RES_DROP - dropout of the result
// (1.88M x 128: the pass of its own took 203 us, a step with two of them is 300 us shorter without).
constexpr int RES_PLAIN = 0, RES_EXTRAS = 1, RES_DROP = 2;
template <int NB, int NCH, int END>
__global__ __launch_bounds__(64 * RES_WAVES) __attribute__((amdgpu_waves_per_eu(2))) void gemm_bf16_resident_kernel(
    const ResidentK p) {
  constexpr bool EXTRAS = END == RES_EXTRAS;
  constexpr int COLS = 32 * NB;
  constexpr int B_BYTES = NCH * 8 * COLS * 16;
  constexpr int STORES = 2 * NB;  // of one tile
  __shared__ __attribute__((aligned(128))) unsigned char smem[B_BYTES + RES_WAVES * 4096];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 5, r = lane & 31;

  // the workgroup's columns n0 .. n1 - 1 and its group of rows (uniform over the block)
  int team = blockIdx.x, n0 = 0, n1 = p.N;
  if (p.parts > 1) {
    const int on_xcd = blockIdx.x >> 3, part = on_xcd % p.parts;
    team = (on_xcd / p.parts) * 8 + (blockIdx.x & 7);
    n0 = part * p.N / p.parts;
    n1 = (part + 1) * p.N / p.parts;
  }
  // Block b of 32 result columns starts at column n0 + 32 b, the last one at n1 - 32: where the columns are no
  // multiple of 32 those that two blocks share are computed twice, alike, so that every lane writes eight
  // existing columns.  column_of: the column at place m of the parameters in LDS.
  const auto block_col = [&](int b) { return n0 + 32 * b < n1 - 32 ? n0 + 32 * b : n1 - 32; };
  const auto column_of = [&](int m) { return (int64_t)(block_col(m >> 5) + (m & 31)); };

  // ---- parameters: 8 columns x 8 k-groups per wavefront and step, four steps requested at a time
  {
    constexpr int UNITS = NCH * (COLS / 8), BATCH = 4;  // a unit = one piece of 64 k of eight columns
    const int nl = lane & 7, kl = lane >> 3;
#pragma nounroll
    for (int u0 = wave; u0 < UNITS; u0 += RES_WAVES * BATCH) {
      float x[BATCH][8];
#pragma unroll
      for (int q = 0; q < BATCH; ++q) {
        const int u = u0 + q * RES_WAVES;
        const int c = u < UNITS ? u / (COLS / 8) : 0, n = (u % (COLS / 8)) * 8 + nl;
        const bool second = c >= p.nch1;
        const int k = ((second ? c - p.nch1 : c) * 8 + kl) * 8, K = second ? p.K2 : p.K1;
        const float* const W = second ? p.W2 : p.W1;
        const int64_t ld = second ? p.ldw2 : p.ldw1;
        // clamped and unconditional, so that a batch's 32 loads are in flight together
        const int64_t nc = column_of(n) * (p.kmajor ? 1 : ld), kd = p.kmajor ? ld : 1;
#pragma unroll
        for (int i = 0; i < 8; ++i) x[q][i] = W[nc + (k + i < K ? k + i : K - 1) * kd];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[q][i] = k + i < K ? x[q][i] : 0.f;
      }
#pragma unroll
      for (int q = 0; q < BATCH; ++q) {
        const int u = u0 + q * RES_WAVES;
        if (u < UNITS) {
          const int c = u / (COLS / 8), n = (u % (COLS / 8)) * 8 + nl;
          *reinterpret_cast<uint4*>(smem + ((c * 8 + kl) * COLS + n) * 16) =
              make_uint4(pack_bf16x2(x[q][0], x[q][1]), pack_bf16x2(x[q][2], x[q][3]), pack_bf16x2(x[q][4], x[q][5]),
                         pack_bf16x2(x[q][6], x[q][7]));
        }
      }
    }
  }
  __syncthreads();

  // ---- rows: wavefront w of team b takes the 32-row tiles w * teams + b, then every 8 * teams-th.
  // The last tile ends with the matrix: the rows it shares with the tile before are computed twice, alike (not where
  // results are added to C, see below).
  const int64_t tiles = (p.M + 31) / 32, stride = (int64_t)RES_WAVES * p.teams;
  int64_t t = (int64_t)__builtin_amdgcn_readfirstlane(wave) * p.teams + team;
  if (t >= tiles) return;
  const unsigned char* const bs = smem + (g * COLS + r) * 16;
  float* const st = reinterpret_cast<float*>(smem + B_BYTES + wave * 4096);
  const auto first_row = [&](int64_t tt) { return tt * 32 < p.M - 32 ? tt * 32 : p.M - 32; };

  float bias[4];  // biases of the columns at places 4 lane .. + 3 of the parameters
#pragma unroll
  for (int i = 0; i < 4; ++i) bias[i] = p.bias && 4 * lane < COLS ? p.bias[column_of(4 * lane + i)] : 0.f;
  u32x4u a[NCH][4];
  // piece c of the tile that starts at row i0, lane (r, g): k = 16 s + 8 g .. + 7 of row r; past the end of the
  // segment the eight that end with it are read (and moved into place before they are used)
  auto load = [&](int64_t i0, int r_, int k8, int c) {
    const bool second = c >= p.nch1;  // uniform
    const int K = second ? p.K2 : p.K1, k0 = (second ? c - p.nch1 : c) * 64;
    const bf16_t* const base = (second ? p.A2 + i0 * p.lda2 : p.A1 + i0 * p.lda1) + k0;
    const uint32_t row = (uint32_t)r_ * (uint32_t)(second ? p.lda2 : p.lda1);
    if (k0 + 64 <= K) {  // uniform
#pragma unroll
      for (int s = 0; s < 4; ++s) a[c][s] = *reinterpret_cast<const u32x4u*>(base + 16 * s + (row + (uint32_t)k8));
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = 16 * s + k8 < K - 8 - k0 ? 16 * s + k8 : K - 8 - k0;  // negative where K < k0 + 8
        a[c][s] = *reinterpret_cast<const u32x4u*>(base + ((int64_t)row + k));
      }
    }
  };
#pragma unroll
  for (int c = 0; c < NCH; ++c) load(first_row(t), r, 8 * g, c);

  // the row factor of the lane's row r travels with the rows (without row factors: any float that is there)
  const float* const row_scale = p.row_scale ? p.row_scale : reinterpret_cast<const float*>(p.A1);
  float rs_next = row_scale[first_row(t) + r];
  if constexpr (!EXTRAS) __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
#pragma nounroll
  for (; t < tiles; t += stride) {
    const int64_t i0 = first_row(t), next = first_row(t + stride < tiles ? t + stride : t);
    // the lane's places as values the compiler cannot compute ahead of the loop (it kept every sum with them in a
    // register of its own, and accumulators in memory instead)
    int rr = r, k8 = 8 * g, er = lane >> 2, ec = (lane & 3) * 8;
    asm volatile("" : "+v"(rr), "+v"(k8), "+v"(er), "+v"(ec));
    const float rs_r = rs_next;
    rs_next = row_scale[next + rr];
    floatx16 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const bool second = c >= p.nch1;
      const int K = second ? p.K2 : p.K1, k0 = (second ? c - p.nch1 : c) * 64;
      if (k0 + 64 > K) {  // uniform: the segment ends inside this piece
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int past = k0 + 16 * s + k8 - (K - 8);
          a[c][s] = shift_halves(a[c][s], past < 0 ? 0 : (past > 8 ? 8 : past));
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bf16x8 rows = __builtin_bit_cast(bf16x8, a[c][s]);
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              *reinterpret_cast<const bf16x8*>(bs + (c * 4 + s) * 2 * COLS * 16 + b * 512), rows, acc[b], 0, 0, 0);
      }
      load(next, rr, k8, c);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- results: a lane's registers 4 q .. 4 q + 3 of block b are columns 8 q + 4 g .. + 3 of the block in row r.
    // Without EXTRAS every tile writes without a condition, so that the number of stores behind the loads of the next
    // tile is known and waiting for those does not wait for the stores.
    struct Extra {
      u32x4u g[2], c[2];
    } e, e_next;
    float rs[2];  // row factors of rows er and 16 + er
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float x = __int_as_float(__builtin_amdgcn_ds_bpermute((16 * h + er) * 4, __float_as_int(rs_r)));
      rs[h] = p.row_scale ? x : 1.f;
    }
    auto request = [&](int b, Extra& x) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        x.g[h] = u32x4u{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};  // ones: everything passes
        x.c[h] = u32x4u{0u, 0u, 0u, 0u};
        const uint32_t row = (uint32_t)(16 * h + er);
        if (p.gate) x.g[h] = *reinterpret_cast<const u32x4u*>(p.gate + i0 * p.ldg + block_col(b) + (row * (uint32_t)p.ldg + (uint32_t)ec));
        if (p.accumulate) x.c[h] = *reinterpret_cast<const u32x4u*>(p.C + i0 * p.ldc + block_col(b) + (row * (uint32_t)p.ldc + (uint32_t)ec));
      }
    };
    if constexpr (EXTRAS) request(0, e);
    u32x4u packed[2][2];  // results of two neighbouring blocks, [block % 2][row half]
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(st + rr * 32 + (((2 * q + (k8 >> 3)) ^ (rr & 7)) * 4)) =
            make_float4(acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]);
      // what the next block adds to is read before this one is written: they may share columns
      if constexpr (EXTRAS)
        if (b + 1 < NB) request(b + 1, e_next);
      float bj[8];  // biases of the lane's eight columns, from the lanes that hold them
#pragma unroll
      for (int c = 0; c < 8; ++c)
        bj[c] = __int_as_float(__builtin_amdgcn_ds_bpermute((8 * b + (ec >> 2) + (c >> 2)) * 4, __float_as_int(bias[c & 3])));
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int row = 16 * h + er;
        const float4 lo = *reinterpret_cast<const float4*>(st + row * 32 + (((ec >> 2) ^ (row & 7)) * 4));
        const float4 hi = *reinterpret_cast<const float4*>(st + row * 32 + ((((ec >> 2) + 1) ^ (row & 7)) * 4));
        float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          x[c] += bj[c];
          if (p.relu) x[c] = fmaxf(x[c], 0.f);
          x[c] *= rs[h];
          if constexpr (EXTRAS) {
            const float gv = bf16_to_f32((bf16_t)(c & 1 ? e.g[h][c >> 1] >> 16 : e.g[h][c >> 1] & 0xffffu));
            const float cv = bf16_to_f32((bf16_t)(c & 1 ? e.c[h][c >> 1] >> 16 : e.c[h][c >> 1] & 0xffffu));
            float y = x[c];
            const bool shut = !(gv > 0.f);
            if (!p.gate_last) y = shut ? 0.f : y * p.gate_scale;
            y += cv;
            if (p.gate_last) y = shut ? 0.f : y * p.gate_scale;
            x[c] = y;
          }
          if (p.relu_last) x[c] = fmaxf(x[c], 0.f);
        }
        if constexpr (END == RES_DROP) {
          const uint64_t first = (uint64_t)(i0 + row) * (uint32_t)p.N + (uint32_t)(block_col(b) + ec);
          drop4(p.drop, first, x);
          drop4(p.drop, first + 4, x + 4);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) packed[b & 1][h][c] = pack_bf16x2(x[2 * c], x[2 * c + 1]);
      }
      // rows that an earlier tile has (or will have) added to are left alone
      const auto mine = [&](int row) { return !EXTRAS || !p.accumulate || i0 + row >= t * 32; };
      const auto at = [&](int row, int col) {
        return reinterpret_cast<u32x4u*>(p.C + i0 * p.ldc + ((uint32_t)row * (uint32_t)p.ldc + (uint32_t)col));
      };
      if (b % 2 == 0) {
        if (b + 1 == NB) {
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (mine(16 * h + er)) *at(16 * h + er, block_col(b) + ec) = packed[0][h];
        }
      } else {
        // two blocks side by side: once more through LDS, after which eight lanes write a whole 128-byte line of C
        // (64-byte pieces reach 4.7 instead of 5.3 TB/s in a copy of the same rows)
#pragma unroll
        for (int w = 0; w < 2; ++w)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int row = 16 * h + er, piece = w * 4 + (ec >> 3);
            *reinterpret_cast<uint4*>(st + row * 32 + ((piece ^ (row & 7)) * 4)) =
                make_uint4(packed[w][h][0], packed[w][h][1], packed[w][h][2], packed[w][h][3]);
          }
        const int lr = (er * 4 + (ec >> 3)) >> 3, piece = (er * 4 + (ec >> 3)) & 7;  // lane / 8, lane % 8
        const int col = (piece < 4 ? block_col(b - 1) : block_col(b)) + (piece & 3) * 8;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int row = 8 * w + lr;
          const uint4 v = *reinterpret_cast<const uint4*>(st + row * 32 + ((piece ^ (row & 7)) * 4));
          if (mine(row)) *at(row, col) = u32x4u{v.x, v.y, v.z, v.w};
        }
      }
      if constexpr (EXTRAS) e = e_next;
      __builtin_amdgcn_sched_barrier(0);  // block by block: mixed, they need more registers than there are
    }
    // the next tile's rows have arrived once no more is outstanding than this tile's stores
    if constexpr (!EXTRAS) __builtin_amdgcn_s_waitcnt((STORES & 15) | (7 << 4) | (15 << 8) | ((STORES >> 4) << 14));
  }
}

// Launches the instance for NB column blocks and nch pieces; false if there is none.
bool launch_resident_narrow(int nb, int nch, int end, dim3 grid, hipStream_t stream, const ResidentK& p);  // 2 .. 4
bool launch_resident_wide(int nb, int nch, int end, dim3 grid, hipStream_t stream, const ResidentK& p);    // 5 .. 8

template <int NB, int NCH>
inline bool launch_resident_instance(int end, dim3 grid, hipStream_t stream, const ResidentK& p) {
  if (end == RES_EXTRAS) gemm_bf16_resident_kernel<NB, NCH, RES_EXTRAS><<<grid, 64 * RES_WAVES, 0, stream>>>(p);
  else if (end == RES_DROP) gemm_bf16_resident_kernel<NB, NCH, RES_DROP><<<grid, 64 * RES_WAVES, 0, stream>>>(p);
  else gemm_bf16_resident_kernel<NB, NCH, RES_PLAIN><<<grid, 64 * RES_WAVES, 0, stream>>>(p);
  return true;
}
// nch counted down from the most that 128 KB of parameters allow
template <int NB, int NCH>
inline bool launch_resident_pieces(int nch, int end, dim3 grid, hipStream_t stream, const ResidentK& p) {
  if (nch == NCH) return launch_resident_instance<NB, NCH>(end, grid, stream, p);
  if constexpr (NCH > 1) return launch_resident_pieces<NB, NCH - 1>(nch, end, grid, stream, p);
  return false;
}

}  // namespace cofree
