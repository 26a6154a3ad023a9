// Products of bfloat16 activations with parameters of more than 128 KB, C = sum of segments A op(W), parameters in registers.
//
// Bound by the bytes of A and C like the products of gemm_bf16_resident.h, but LDS holds only 160 KB, and cut into column parts
// the rows were fetched 1.35 times (the workgroups that share them drift apart).  A CU's registers hold 512 KB: a workgroup of
// four wavefronts, one per SIMD, keeps up to 256 columns x 512 k there for the whole launch, 64 columns a wavefront (256 of its
// 512 registers), and streams 32-row tiles past them.  A tile comes from memory in whole 128-byte lines, two or three tiles
// in flight in registers, passes through one of two LDS buffers, and every wavefront multiplies all of it by its columns; one barrier a
// tile.  16-byte pieces of a row lie at places permuted by the row, so that both directions are free of bank conflicts.
// 1.88M rows, 256 columns x 512 k: 717 us in tiles, 708 in column parts, 587 here (4.9 TB/s of rows and results).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "gemm_bf16_resident.h"

namespace cofree {

typedef uint32_t uint32x4v __attribute__((ext_vector_type(4)));

constexpr int PIN_WAVES = 4, PIN_COLS = 256;

template <int NCH, int END>
__global__ __launch_bounds__(64 * PIN_WAVES) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_bf16_pinned_kernel(
    const ResidentK p, const bf16_t* __restrict__ Wb, int64_t ldwb) {
  constexpr bool GATED = END == RES_EXTRAS;
  constexpr int RING = NCH == 8 || (GATED && NCH == 7) ? 2 : 3;  // tiles in flight: what the registers leave
  constexpr int STAGING = 8192;  // two blocks of 32 x 32 sums
  constexpr int TILE_BYTES = NCH * 4096;  // 32 rows, 128 bytes of each per piece
  __shared__ __attribute__((aligned(128))) unsigned char smem[2 * TILE_BYTES + PIN_WAVES * STAGING];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, r = lane & 31;

  // the workgroup's columns n0 .. n1 - 1 and its group of rows (uniform over the block)
  int team = blockIdx.x, n0 = 0, n1 = p.N;
  if (p.parts > 1) {
    const int on_xcd = blockIdx.x >> 3, part = on_xcd % p.parts;
    team = (on_xcd / p.parts) * 8 + (blockIdx.x & 7);
    n0 = part * PIN_COLS;
    n1 = n0 + PIN_COLS < p.N ? n0 + PIN_COLS : p.N;
  }
  const int64_t tiles = (p.M + 31) / 32, stride = p.teams;
  int64_t t = team;
  if (t >= tiles) return;
  // The wavefront's two blocks of 32 columns; a block that would cross the end is moved left to end with the columns, and those
  // it shares with another are computed twice, alike; a wavefront without columns of its own does the last ones again.
  const auto block_col = [&](int b) { return n0 + 64 * wave + 32 * b < n1 - 32 ? n0 + 64 * wave + 32 * b : n1 - 32; };

  // piece c: its segment, and the first k of it
  const auto second = [&](int c) { return c >= p.nch1; };
  const auto seg_len = [&](int c) { return second(c) ? p.K2 : p.K1; };
  const auto seg_k0 = [&](int c) { return (second(c) ? c - p.nch1 : c) * 64; };

  // ---- parameters: lane (r, g) holds k = 16 s + 8 g .. + 7 of column r of a block; past the end of a segment zeros.  Sixteen
  // loads are in flight together.
  bf16x8 w[NCH][4][2];
#pragma unroll
  for (int c0 = 0; c0 < NCH; c0 += 2) {
    u32x4u x[2][4][2];
    const auto k_of = [&](int c, int s) { return seg_k0(c) + 16 * s + 8 * g - (seg_len(c) - 8); };  // against the last eight
#pragma unroll
    for (int c = c0; c < c0 + 2 && c < NCH; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int past = k_of(c, s);
          x[c - c0][s][b] = *reinterpret_cast<const u32x4u*>(Wb + (int64_t)(block_col(b) + r) * ldwb + (second(c) ? p.K1 : 0) +
                                                            (seg_len(c) - 8 + (past < 0 ? past : 0)));
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = c0; c < c0 + 2 && c < NCH; ++c)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int past = k_of(c, s);
          uint32x4v v = shift_halves(x[c - c0][s][b], past < 0 ? 0 : (past > 8 ? 8 : past));
          asm volatile("" : "+a"(v));  // accumulation registers, where the matrix instructions can read them; not moved per use
          w[c][s][b] = __builtin_bit_cast(bf16x8, v);
        }
  }

  const auto first_row = [&](int64_t tt) { return tt * 32 < p.M - 32 ? tt * 32 : p.M - 32; };
  const int er = lane >> 2, ec = (lane & 3) * 8;  // results: a lane finishes eight columns of rows er and 16 + er of a block
  float bias[2][8];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int c = 0; c < 8; ++c) bias[b][c] = p.bias ? p.bias[block_col(b) + ec + c] : 0.f;

  // rows: wavefront w moves rows 8 w .. + 7 of a tile, eight lanes a line; lane / 8 its row, lane % 8 its piece of eight k
  const int mr = 8 * wave + (lane >> 3), mk = (lane & 7) * 8;
  u32x4u ring[RING][NCH];
  const auto load = [&](int64_t tt, u32x4u& x, int c) __attribute__((always_inline)) {
    const int64_t lda = second(c) ? p.lda2 : p.lda1;
    const bf16_t* const base = (second(c) ? p.A2 : p.A1) + first_row(tt < tiles ? tt : tiles - 1) * lda;
    const int k = seg_k0(c) + mk, end = seg_len(c) - 8;
    x = *reinterpret_cast<const u32x4u*>(base + ((int64_t)((uint32_t)mr * (uint32_t)lda) + (k < end ? k : end)));
  };
  const int put_at = mr * 128 + (((lane & 7) ^ (mr & 7)) * 16);
  const auto put = [&](const u32x4u& x, unsigned char* stage, int c) __attribute__((always_inline)) {
    u32x4u v = x;
    if (seg_k0(c) + 64 > seg_len(c)) {  // uniform: the segment ends inside this piece
      const int past = seg_k0(c) + mk - (seg_len(c) - 8);
      v = shift_halves(v, past < 0 ? 0 : (past > 8 ? 8 : past));
    }
    *reinterpret_cast<uint4*>(stage + c * 4096 + put_at) = make_uint4(v[0], v[1], v[2], v[3]);
  };
  int take_at[4];  // lane (r, g): k = 16 s + 8 g .. + 7 of row r
#pragma unroll
  for (int s = 0; s < 4; ++s) take_at[s] = r * 128 + (((2 * s + g) ^ (r & 7)) * 16);

  const float* const row_scale = p.row_scale ? p.row_scale : reinterpret_cast<const float*>(p.A1);
  float* const st = reinterpret_cast<float*>(smem + 2 * TILE_BYTES + wave * STAGING);
#pragma unroll
  for (int q = 0; q < RING; ++q)
#pragma unroll
    for (int c = 0; c < NCH; ++c) load(t + q * stride, ring[q][c], c);
  float rs_next = row_scale[first_row(t) + r];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    put(ring[0][c], smem, c);
    load(t + RING * stride, ring[0][c], c);
  }
  __syncthreads();

  // The tile before, whose sums are in `st`, is finished between the matrix instructions of this one: work(0) .. work(11), in
  // order (one wavefront a SIMD: behind one another they took 3.1 us a tile of 512 k, 2.3 of which its bytes need).
  int64_t done_i0 = 0;
  float done_rs = 0.f;
  u32x4u gate[2][2];  // [block][row half]
  float4 lo[2], hi[2];
  u32x4u packed[2][2], line[4];
  const auto request = [&](int64_t i0) __attribute__((always_inline)) {  // what the tile at i0 is gated by
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        gate[b][h] = *reinterpret_cast<const u32x4u*>(p.gate + i0 * p.ldg + block_col(b) + ((uint32_t)(16 * h + er) * (uint32_t)p.ldg + (uint32_t)ec));
  };
  const auto take_sums = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float* const row = st + b * 1024 + (16 * h + er) * 32;
      lo[h] = *reinterpret_cast<const float4*>(row + (((ec >> 2) ^ (er & 7)) * 4));
      hi[h] = *reinterpret_cast<const float4*>(row + ((((ec >> 2) + 1) ^ (er & 7)) * 4));
    }
  };
  const auto finish = [&](int b) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float y[8] = {lo[h].x, lo[h].y, lo[h].z, lo[h].w, hi[h].x, hi[h].y, hi[h].z, hi[h].w};
      const float f = __int_as_float(__builtin_amdgcn_ds_bpermute((16 * h + er) * 4, __float_as_int(done_rs)));
      const float rs = p.row_scale ? f : 1.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        y[c] += bias[b][c];
        if (p.relu) y[c] = fmaxf(y[c], 0.f);
        y[c] *= rs;
        if constexpr (GATED) {
          const uint32_t gw = gate[b][h][c >> 1];
          y[c] = __uint_as_float(c & 1 ? gw & 0xffff0000u : gw << 16) > 0.f ? y[c] * p.gate_scale : 0.f;
        }
        if (p.relu_last) y[c] = fmaxf(y[c], 0.f);
      }
      if constexpr (END == RES_DROP) {
        const uint64_t first = (uint64_t)(done_i0 + 16 * h + er) * (uint32_t)p.N + (uint32_t)(block_col(b) + ec);
        drop4(p.drop, first, y);
        drop4(p.drop, first + 4, y + 4);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) packed[b][h][c] = pack_bf16x2(y[2 * c], y[2 * c + 1]);
    }
  };
  const auto work = [&](int q) __attribute__((always_inline)) {
    if (q == 0) take_sums(0);
    if (q == 2) finish(0);
    if (q == 3) take_sums(1);
    if (q == 5) finish(1);
    if (q == 6) {  // once more through LDS, after which eight lanes write a whole 128-byte line of C
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int row = 16 * h + er, piece = b * 4 + (ec >> 3);
          *reinterpret_cast<uint4*>(st + row * 32 + ((piece ^ (row & 7)) * 4)) =
              make_uint4(packed[b][h][0], packed[b][h][1], packed[b][h][2], packed[b][h][3]);
        }
    }
    const int lr = lane >> 3, piece = lane & 7;
    if (q == 8) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint4 v = *reinterpret_cast<const uint4*>(st + (8 * u + lr) * 32 + ((piece ^ lr) * 4));
        line[u] = u32x4u{v.x, v.y, v.z, v.w};
      }
    }
    if (q == 10) {
      const int col = block_col(piece >> 2) + (piece & 3) * 8;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = 8 * u + lr;
        *reinterpret_cast<u32x4u*>(p.C + done_i0 * p.ldc + ((uint32_t)row * (uint32_t)p.ldc + (uint32_t)col)) = line[u];
      }
    }
  };

  constexpr int AHEAD = GATED && NCH == 8 ? 3 : 4;
  // one tile out of `stage`; x: the registers of the next one, which goes to the other buffer
  constexpr int WORK = 12;
  static_assert(WORK + NCH <= 4 * NCH, "a slot for everything");
  const auto step = [&](auto before, unsigned char* stage, unsigned char* other, u32x4u (&x)[NCH]) __attribute__((always_inline)) {
    const int64_t i0 = first_row(t), next = first_row(t + stride < tiles ? t + stride : t);
    const float rs = rs_next;
    rs_next = row_scale[next + r];
    const auto move = [&](int c) __attribute__((always_inline)) {
      put(x[c], other, c);
      load(t + (RING + 1) * stride, x[c], c);
    };
    floatx16 acc[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
    bf16x8 rows[AHEAD];  // read that many steps ahead; in order, or the compiler waits for every read at its use
    const auto take = [&](int k) __attribute__((always_inline)) {
      rows[k % AHEAD] = *reinterpret_cast<const bf16x8*>(stage + k / 4 * 4096 + take_at[k % 4]);
    };
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) take(k);
#pragma unroll
    for (int k = 0; k < 4 * NCH; ++k) {
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[k / 4][k % 4][b], rows[k % AHEAD], acc[b], 0, 0, 0);
      if (k + AHEAD < 4 * NCH) take(k + AHEAD);
      if (decltype(before)::value && k < WORK) work(k);
      if (GATED && k == WORK - 1) request(i0);
      if (k >= WORK && k < WORK + NCH) move(k - WORK);
      __builtin_amdgcn_sched_barrier(0);
    }
    // a lane's registers 4 q .. + 3 of block b are columns 8 q + 4 g .. + 3 of the block in row r
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(st + b * 1024 + r * 32 + (((2 * q + g) ^ (r & 7)) * 4)) =
            make_float4(acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]);
    done_i0 = i0;
    done_rs = rs;
    __syncthreads();
    t += stride;
  };
  unsigned char *now = smem, *other = smem + TILE_BYTES;
  const auto last = [&](auto before, u32x4u (&x)[NCH]) __attribute__((always_inline)) {
    step(before, now, other, x);
    unsigned char* const used = now;
    now = other;
    other = used;
    return t >= tiles;
  };
  const std::true_type has{};
  if (!last(std::false_type{}, ring[1])) {
#pragma nounroll
    while (true) {
      if constexpr (RING == 3)
        if (last(has, ring[2])) break;
      if (last(has, ring[0])) break;
      if (last(has, ring[1])) break;
    }
  }
#pragma unroll
  for (int q = 0; q < WORK; ++q) work(q);
}

static int pinned_pieces(const GemmArgs& a) { return (a.K1 + 63) / 64 + (a.K2 + 63) / 64; }

// Which products.  us of a launch, resident or tiled kernel / this one; t: both need the launch of 6 us that converts parameters,
// else only this one does:
//  * 257 to 512 k, 129 to 512 columns, from 131072 rows on (256 columns x 512 k: 1.88M rows 717 t, 708 / 587, 400k 180 t, 167 / 139, 150k
//    72 t, 78 / 62, 110k 50 t / 50, 50k 30 t / 34; 256 x 428 150k 73 / 60; 256 x 356 1.88M 579 / 479; 256 x 303 1.88M 472 / 427; 130 x
//    320 400k 109 / 101, 150k 49 / 46), of more than 448 k and more than 256 columns, or columns that leave tiles empty, from 65536
//    on (500 x 500 75k 81 t / 59, 50k 60 t / 45; 140 x 512 75k 43 t / 38; but 300 x 400 75k 56 / 53, 400 x 300 47 / 44).
//    A second workgroup for few of the columns costs what a whole one does, so up to 307 columns only from 385 k on, up to 384 from 321 on, and
//    fewer than 196608 rows not of 385 to 448 k by up to 307 columns, nor A B of up to 384 columns or of these least k (276 columns x 276 k 276k 115 / 128, 800k 302 / 347; 300 x 350 800k 373 / 388; 276 x 448 800k
//    448 / 418, 140k 93 / 91, A B 276 x 420 78 / 92, 276k 167 / 161; 380 x 276 800k 342 / 350; 330 x 350 276k 168 / 144, A B 350 x 330 140k 81 / 84; 420 x 276
//    276k 160 / 129; layers of 135,000 rows: GCN 400 -> 260 forward 195 / 213, 290 -> 500 backward 387 / 407).
//    Nor does it pay where two of the wavefronts have few columns or none: up to 160 columns only from 385 k on, and up to 192 columns of up to 448 k from
//    262144 rows on (layers: conventional GraphSAGE 130 -> 130 over 200k forward 159 / 173, 400k 305 / 334; 150 -> 150 200k backward 299 / 310; GCN 130 -> 360 200k
//    backward 308 / 328; 172 -> 360 200k 348 / 366, 400k 0.95, 900k 0.95).
//  * 193 to 256 k (not fewer, in two segments: 182 columns x 71 + 71 k over 200k 50 / 62) of more than 160 columns that are no multiple of 64, from 131072 rows on (200 x 256 150k 57 / 41, 1.88M 441 / 359; 172 x
//    256 150k 49 / 41, 400k 99 / 88, 1.88M 420 / 366; 160 x 256 400k 90 / 92; 256 x 256 1.88M 372 / 366), of whole ones where the
//    tiled kernel would be taken (256 x 256 150k 55 t / 43, 200k 69 t / 53).
// Up to 128 columns half of the wavefronts would have none (128 x 256 1.88M 265 / 351).
// COFREE_BF16_TILE = 1 takes every product that fits, any other value none.
bool gemm_pinned_fits(const GemmArgs& a) {
  const int nch = pinned_pieces(a);
  const int64_t strides = a.lda1 | a.lda2 | a.ldc | a.ldg;  // 32-bit offsets inside a tile of 32 rows
  if (a.accumulate || a.N <= 128 || a.N > 512 || a.M < 32 || strides >= ((int64_t)1 << 26) || a.K1 < 8 || (a.K2 > 0 && a.K2 < 8) ||
      nch < 4 || nch > 8)
    return false;
  if (const char* e = getenv("COFREE_BF16_TILE")) return atoi(e) == 1;
  if (nch == 4) {
    if (a.N <= 160 || a.N > 256 || a.M < 1 << 17 || a.K1 + a.K2 <= 192) return false;
    return a.N % 64 != 0 || (!a.b_kmajor && a.dropout.q == 0.f && a.M < 1 << 18);
  }
  const bool tiles_empty = 4 * (int64_t)((a.N + 127) / 128 * 128) >= 5 * (int64_t)a.N;
  int64_t rows = nch == 8 && (a.N > 256 || tiles_empty) ? 1 << 16 : 1 << 17;
  if (a.N <= 192 && nch < 8) {
    if (a.N <= 160 && nch < 7) return false;
    rows = 1 << 18;
  }
  if (a.N > 256) {
    const int least = tiles_empty ? 7 : a.N <= 384 ? 6 : 5;
    if (nch < least) return false;
    if ((nch == least && (a.b_kmajor || tiles_empty)) || (a.b_kmajor && a.N <= 384)) rows = 3 << 16;
  }
  return a.M >= rows;
}
bool gemm_pinned_drops(const GemmArgs& a) { return gemm_pinned_fits(a) && !a.gate && !a.accumulate && a.N % 4 == 0; }

template <int NCH>
static void launch_pinned(int end, dim3 grid, hipStream_t stream, const ResidentK& p, const bf16_t* Wb, int64_t ldwb) {
  if (end == RES_EXTRAS) gemm_bf16_pinned_kernel<NCH, RES_EXTRAS><<<grid, 64 * PIN_WAVES, 0, stream>>>(p, Wb, ldwb);
  else if (end == RES_DROP) gemm_bf16_pinned_kernel<NCH, RES_DROP><<<grid, 64 * PIN_WAVES, 0, stream>>>(p, Wb, ldwb);
  else gemm_bf16_pinned_kernel<NCH, RES_PLAIN><<<grid, 64 * PIN_WAVES, 0, stream>>>(p, Wb, ldwb);
}

int32_t launch_gemm_pinned(const GemmArgs& a, const bf16_t* Wb, int64_t ldwb, hipStream_t stream) {
  ResidentK p{};
  p.A1 = (const bf16_t*)a.A1, p.lda1 = a.lda1, p.K1 = a.K1;
  p.A2 = (const bf16_t*)a.A2, p.lda2 = a.lda2, p.K2 = a.K2;
  p.nch1 = (a.K1 + 63) / 64;
  p.C = (bf16_t*)a.C, p.ldc = a.ldc, p.M = a.M, p.N = a.N;
  p.bias = a.bias, p.relu = a.relu, p.row_scale = a.row_scale;
  p.gate = (const bf16_t*)a.gate, p.ldg = a.ldg;
  p.relu_last = a.relu_last;
  p.gate_scale = a.gate ? a.gate_scale : 1.f;
  p.drop = dropout_k(a.dropout);
  const int nch = pinned_pieces(a);
  const int64_t K = (int64_t)a.K1 + a.K2, tiles = (a.M + 31) / 32;
  p.parts = (a.N + PIN_COLS - 1) / PIN_COLS;
  p.teams = std::min<int64_t>(tiles, RES_CUS);
  if (p.parts > 1) p.teams = 8 * std::min<int64_t>((tiles + 7) / 8, std::max(1, RES_CUS / 8 / p.parts));
  const dim3 grid((unsigned)(p.teams * p.parts));
  const int end = a.gate ? RES_EXTRAS : (p.drop.scale != 0.f ? RES_DROP : RES_PLAIN);
  char pname[96] = "";
  if (profiling()) snprintf(pname, sizeof(pname), "gemm_bf16_pinned_kernel<%d,%d> N=%d K=%d", nch, end, (int)a.N, (int)K);
  ProfScope prof(pname, stream, 2.0 * ((double)a.M * K + (double)a.N * K + (double)a.M * a.N),
                 2.0 * (double)a.M * a.N * (double)K);
  switch (nch) {
    case 4: launch_pinned<4>(end, grid, stream, p, Wb, ldwb); break;
    case 5: launch_pinned<5>(end, grid, stream, p, Wb, ldwb); break;
    case 6: launch_pinned<6>(end, grid, stream, p, Wb, ldwb); break;
    case 7: launch_pinned<7>(end, grid, stream, p, Wb, ldwb); break;
    case 8: launch_pinned<8>(end, grid, stream, p, Wb, ldwb); break;
    default: return fail(COFREE_EINVAL, "internal: no pinned product of this shape");
  }
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

}  // namespace cofree
