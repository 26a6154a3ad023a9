// Reweighted loss (Eq. 3), parameter update (Algorithm 1 line 11) and the small streaming
// kernels of backward (bias gradients, activation / dropout gates).
#include <cmath>
#include <mutex>

#include "common.h"

namespace cofree {

__device__ inline float ld_elem(const float* p) { return *p; }
__device__ inline float ld_elem(const bf16_t* p) { return bf16_to_f32(*p); }
__device__ inline void st_elem(float* p, float x) { *p = x; }
__device__ inline void st_elem(bf16_t* p, float x) { *p = f32_to_bf16(x); }

// four consecutive elements (contiguous matrices whose base is 16-byte aligned: quad q starts at 4q)
__device__ inline void ld_quad(const float* p, float (&v)[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
}
__device__ inline void ld_quad(const bf16_t* p, float (&v)[4]) {
  const uint2 t = *reinterpret_cast<const uint2*>(p);
  v[0] = __uint_as_float(t.x << 16), v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16), v[3] = __uint_as_float(t.y & 0xffff0000u);
}
__device__ inline void st_quad(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline void st_quad(bf16_t* p, const float (&v)[4]) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}

// four consecutive elements at any element-aligned address, of which only the first `avail` exist:
// one 16-byte (float32) / 8-byte (bfloat16) access when all four do
typedef float f32x4e __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2e __attribute__((ext_vector_type(2), aligned(2)));
__device__ inline void ld4(const float* p, int avail, float (&v)[4], float fill) {
  if (avail >= 4) {
    const f32x4e t = *reinterpret_cast<const f32x4e*>(p);
    v[0] = t[0], v[1] = t[1], v[2] = t[2], v[3] = t[3];
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = i < avail ? p[i] : fill;
  }
}
__device__ inline void ld4(const bf16_t* p, int avail, float (&v)[4], float fill) {
  if (avail >= 4) {
    const u32x2e t = *reinterpret_cast<const u32x2e*>(p);
    v[0] = __uint_as_float(t[0] << 16), v[1] = __uint_as_float(t[0] & 0xffff0000u);
    v[2] = __uint_as_float(t[1] << 16), v[3] = __uint_as_float(t[1] & 0xffff0000u);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = i < avail ? bf16_to_f32(p[i]) : fill;
  }
}
__device__ inline void ld4(const uint8_t* p, int avail, uint32_t (&v)[4]) {
  typedef uint32_t u32e __attribute__((aligned(1)));
  if (avail >= 4) {
    const uint32_t t = *reinterpret_cast<const u32e*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (t >> (8 * i)) & 0xffu;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = i < avail ? p[i] : 0u;
  }
}
__device__ inline void st4(float* p, int avail, const float (&v)[4]) {
  if (avail >= 4) {
    f32x4e t;
    t[0] = v[0], t[1] = v[1], t[2] = v[2], t[3] = v[3];
    *reinterpret_cast<f32x4e*>(p) = t;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < avail) p[i] = v[i];
  }
}
__device__ inline void st4(bf16_t* p, int avail, const float (&v)[4]) {
  if (avail >= 4) {
    u32x2e t;
    t[0] = pack_bf16x2(v[0], v[1]);
    t[1] = pack_bf16x2(v[2], v[3]);
    *reinterpret_cast<u32x2e*>(p) = t;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < avail) p[i] = f32_to_bf16(v[i]);
  }
}

// the same for eight bfloat16 elements (one 16-byte access when all eight exist)
typedef uint32_t u32x4e __attribute__((ext_vector_type(4), aligned(2)));
__device__ inline void ld_n(const float* p, int avail, float (&v)[4], float fill) { ld4(p, avail, v, fill); }
__device__ inline void st_n(float* p, int avail, const float (&v)[4]) { st4(p, avail, v); }
__device__ inline void ld_n(const bf16_t* p, int avail, float (&v)[8], float fill) {
  if (avail >= 8) {
    const u32x4e t = *reinterpret_cast<const u32x4e*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(t[i] << 16);
      v[2 * i + 1] = __uint_as_float(t[i] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = i < avail ? bf16_to_f32(p[i]) : fill;
  }
}
__device__ inline void st_n(bf16_t* p, int avail, const float (&v)[8]) {
  if (avail >= 8) {
    u32x4e t;
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    *reinterpret_cast<u32x4e*>(p) = t;
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (i < avail) p[i] = f32_to_bf16(v[i]);
  }
}

constexpr int LOSS_BLOCKS = 2048;  // workgroups, and partial sums, at most
// of loss_group_kernel: five a CU are resident in every bfloat16 instance of rows of several pieces (83 to 94 VGPRs), and a sixth would
// run behind them (2.4M x 172: 1,280 workgroups 378 us, 1,536 457, 2,048 395).  Float32 instances (38 to 75) would hold six and
// more, which was not measured.
constexpr int GROUP_BLOCKS = 5 * 256;

// Partial sums of cofree_loss_weighted_static: device memory that exists from the moment the library is loaded
// (one copy per GPU, 8 KiB, held until the process ends), so that the call never allocates.  In host code this
// name is only a handle for hipGetSymbolAddress; kernels receive the address that call returns.
static __device__ __align__(256) float scratch[LOSS_BLOCKS];

__device__ inline float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ inline float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// A workgroup's loss: its lanes' in a fixed order
__device__ inline void store_partial(float my_loss, float* __restrict__ partial) {
  __shared__ float wave_loss[4];
  my_loss = wave_sum(my_loss);
  if ((threadIdx.x & 63) == 0) wave_loss[threadIdx.x >> 6] = my_loss;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = (wave_loss[0] + wave_loss[1]) + (wave_loss[2] + wave_loss[3]);
}

// One wavefront per node: softmax over its C logits (lanes stride over classes), cross-entropy
// against the label, times c * w_j; dlogits = c * w_j * (softmax - onehot).  Each block adds up
// its wavefronts' losses in a fixed order into partial[blockIdx.x].
template <typename T>
__global__ __launch_bounds__(256) void loss_kernel(const T* __restrict__ logits,
                                                   const int32_t* __restrict__ labels,
                                                   const float* __restrict__ w,
                                                   const uint8_t* __restrict__ train_mask, int64_t n, int32_t C,
                                                   float scale_c, T* __restrict__ dlogits,
                                                   float* __restrict__ partial) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float my_loss = 0.f;
  for (int64_t row = (int64_t)blockIdx.x * 4 + wave; row < n; row += (int64_t)gridDim.x * 4) {
    const T* z = logits + row * C;
    float m = -INFINITY;
    for (int c = lane; c < C; c += 64) m = fmaxf(m, ld_elem(z + c));
    m = wave_max(m);
    float se = 0.f;
    for (int c = lane; c < C; c += 64) se += expf(ld_elem(z + c) - m);
    se = wave_sum(se);
    float wj = w ? w[row] : 1.f;
    if (train_mask && train_mask[row] == 0) wj = 0.f;
    int32_t y = labels[row];
    if ((uint32_t)y >= (uint32_t)C) {  // label outside [0, C): the node does not contribute
      y = 0;
      wj = 0.f;
    }
    const float coef = scale_c * wj;
    const float inv = 1.f / se;
    T* dz = dlogits + row * C;
    for (int c = lane; c < C; c += 64) {
      const float pr = expf(ld_elem(z + c) - m) * inv;
      st_elem(dz + c, coef * (pr - (c == y ? 1.f : 0.f)));
    }
    if (lane == 0) my_loss += coef * (m + logf(se) - ld_elem(z + y));
  }
  store_partial(my_loss, partial);
}

// e^x for x <= 0.  bfloat16 logits: the hardware's 2^x on x log2(e) (relative error about |x| 2^-24, far below
// the 2^-9 of the stored gradient); the library routine's range handling made the kernel issue-bound (172
// classes: 8.4 ms a launch over 28M nodes at 8 bytes per lane, 6.9 ms at 16 bytes, 5.5 ms with this).
// float32 logits keep expf.
template <typename T>
__device__ inline float softmax_exp(float x) {
  if constexpr (sizeof(T) == 2) return __builtin_amdgcn_exp2f(x * 1.44269504088896341f);
  else return expf(x);
}

// Same computation with a group of LANES lanes per node, C <= LANES * PIECES * PER (LANES a power of two dividing 64): lane l
// owns the PER consecutive classes - 16 bytes of them, four float32 or eight bfloat16 - from PER l on and, with two pieces, as
// many from PER (LANES + l) on, each read and written with one wide access; a wavefront works on 64/LANES nodes at once and on
// two of them per group and iteration, so that the loads of independent rows overlap.
// WIDE (C >= PER): a last piece that would cross the end of the row - or lie past it - is the window that ends with the row
// instead, with the `skip` leading classes that belong to the piece before left out of the sum, so that every lane issues the
// same unconditional wide loads and stores (a per-lane width branch around the loads made the loop wait for each row in turn);
// the overlapped classes are written twice with identical values.
// What bounds it: vector instructions (about 120 for eight classes of a row, a third of them for the row as a whole: reductions, 1 / sum,
// logarithm), hence two pieces a lane wherever the row has them, and no more lanes than it needs.  Microseconds with one piece
// and at least eight lanes, the label's logit fetched from its lane, and now: 2.4M x 172 bfloat16 501 / 378 (4.4 TB/s), 2.4M x 47
// bfloat16 148 / 120, 1.2M x 47 float32 119 / 108, 500k x 600 bfloat16 (then a wavefront a node) 946 / 291, 500k x 5 float32 25 / 9.
template <typename T, int LANES, int PIECES>
__global__ __launch_bounds__(256) void loss_group_kernel(const T* __restrict__ logits,
                                                         const int32_t* __restrict__ labels,
                                                         const float* __restrict__ w,
                                                         const uint8_t* __restrict__ train_mask, int64_t n, int32_t C,
                                                         float scale_c, T* __restrict__ dlogits,
                                                         float* __restrict__ partial) {
  constexpr int GROUPS = 256 / LANES, R = 2, PER = 16 / (int)sizeof(T), LAST = PIECES - 1;
  constexpr bool WIDE = LANES > 1 || PIECES > 1;
  const int gl = threadIdx.x % LANES, grp = threadIdx.x / LANES;
  int c0[PIECES], skip = 0;  // the pieces' first classes
#pragma unroll
  for (int q = 0; q < PIECES; ++q) c0[q] = (q * LANES + gl) * PER;
  const int last = c0[LAST], avail = C - last;
  if (WIDE && avail < PER) {
    skip = avail > 0 ? PER - avail : PER;
    c0[LAST] = C - PER;
  }
  float own[PER];  // 0 for a class that the piece before adds to the sum
#pragma unroll
  for (int k = 0; k < PER; ++k) own[k] = k >= skip ? 1.f : 0.f;
  // a workgroup owns one contiguous run of rows and walks it front to back, GROUPS * R consecutive rows per
  // iteration, so that rows sharing a cache line at their ends (rows are C elements long, any C) are handled
  // by the same workgroup close in time (timing equal to a grid-strided walk at 28M rows of 172 bfloat16)
  const int64_t per_block = (n + gridDim.x - 1) / gridDim.x, b0 = (int64_t)blockIdx.x * per_block;
  const int count = (int)(n - b0 < per_block ? n - b0 : per_block);
  // the run's rows by 32-bit offsets: its elements take less than 4 GiB (a GPU's memory over LOSS_BLOCKS)
  logits += b0 * C, dlogits += b0 * C, labels += b0;
  if (w) w += b0;
  if (train_mask) train_mask += b0;
  float my_loss = 0.f;
  for (int row0 = grp; row0 < count; row0 += R * GROUPS) {
    float v[R][PIECES][PER];
    bool valid[R];
    uint32_t at[R];
    float coefs[R];
    int32_t ys[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      valid[r] = row0 + r * GROUPS < count;
      const uint32_t row = valid[r] ? row0 + r * GROUPS : row0;  // a row past the end is computed on row0 and not stored
      at[r] = row * (uint32_t)C;
      // label and weight are requested with the logits, not after the reductions
      coefs[r] = w ? w[row] : 1.f;
      if (train_mask && train_mask[row] == 0) coefs[r] = 0.f;
      ys[r] = labels[row];
#pragma unroll
      for (int q = 0; q < PIECES; ++q) ld_n(logits + (at[r] + c0[q]), WIDE ? PER : C, v[r][q], -INFINITY);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float m = v[r][0][0];
#pragma unroll
      for (int k = 1; k < PIECES * PER; ++k) m = fmaxf(m, v[r][k / PER][k % PER]);
#pragma unroll
      for (int o = LANES / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
      // e of a skipped class is the value that its owner computes (same logit, same maximum); it only
      // stays out of this piece's share of the sum
      float e[PIECES][PER], se = 0.f;
#pragma unroll
      for (int q = 0; q < PIECES; ++q) {
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          e[q][k] = softmax_exp<T>(v[r][q][k] - m);
          if (WIDE) sum = q == LAST ? fmaf(e[q][k], own[k], sum) : sum + e[q][k];
          else if (k < C) sum += e[q][k];
        }
        se += sum;
      }
#pragma unroll
      for (int o = LANES / 2; o > 0; o >>= 1) se += __shfl_xor(se, o, 64);
      const bool known = (uint32_t)ys[r] < (uint32_t)C;  // label outside [0, C): the node does not contribute
      const int y = known ? ys[r] : 0;
      const float coef = scale_c * (known ? coefs[r] : 0.f);
      const float inv = 1.f / se;
      float zy = v[r][0][0];
#pragma unroll
      for (int q = 0; q < PIECES; ++q) {
        float g[PER];
        const int mine = y - c0[q];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          const bool hit = k == mine;
          g[k] = coef * (e[q][k] * inv - (hit ? 1.f : 0.f));
          zy = hit ? v[r][q][k] : zy;
        }
        if (valid[r]) st_n(dlogits + (at[r] + c0[q]), WIDE ? PER : C, g);
      }
      if (valid[r] && y / PER % LANES == gl) my_loss += coef * (m + logf(se) - zy);  // the lane that owns class y
    }
  }
  store_partial(my_loss, partial);
}

// Multi-label loss (the sigmoid + binary cross-entropy of Theorem 3): a thread takes four consecutive elements of the matrix
// as one list, grid-stride.  loss element = softplus(z) - y z with softplus(z) = max(z, 0) + log1p(e^-|z|);
// dlogits = c w_j (sigmoid(z) - y).  Per-thread sums in index order, then the fixed wavefront / block tree.
// log1p(e) = log(u) + (e - (u - 1)) / u with u = 1 + e rounded (u - 1 is exact): what the rounding of u left out, to
// first order.
// What bounds it: vector instructions, 65 an element; one element a thread with its row by division and log1pf took 230.
// 717k x 100 float32 292 -> 174 us, bfloat16 294 -> 162.
template <typename T>
__global__ __launch_bounds__(256) void bce_kernel(const T* __restrict__ logits, const uint8_t* __restrict__ targets,
                                                  const float* __restrict__ w,
                                                  const uint8_t* __restrict__ train_mask, int64_t n, int32_t C,
                                                  float scale_c, T* __restrict__ dlogits,
                                                  float* __restrict__ partial) {
  const int64_t total = n * C, step = (int64_t)gridDim.x * 1024, step_rows = step / C;
  const int32_t step_cols = (int32_t)(step - step_rows * C);
  int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4, row = i / C;
  int32_t col = (int32_t)(i - row * C);
  float my_loss = 0.f;
  auto weight = [&](int64_t r) {
    const float x = w ? w[r] : 1.f;
    return scale_c * (train_mask && train_mask[r] == 0 ? 0.f : x);
  };
  for (; i < total; i += step) {
    const int avail = total - i < 4 ? (int)(total - i) : 4;
    float z[4], g[4], coef[4];
    uint32_t t[4];
    ld4(logits + i, avail, z, 0.f);
    ld4(targets + i, avail, t);
    if (C >= 3) {  // two rows at most
      const float first = weight(row), next = weight(row + 1 < n ? row + 1 : row);
#pragma unroll
      for (int k = 0; k < 4; ++k) coef[k] = col + k < C ? first : next;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t r = row + ((col + k) >> (C - 1));
        coef[k] = weight(r < n ? r : n - 1);
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float y = t[k] != 0 ? 1.f : 0.f;
      const float e = expf(-fabsf(z[k])), u = 1.f + e;
      g[k] = coef[k] * ((z[k] >= 0.f ? 1.f : e) / u - y);
      const float log1p_e = logf(u) + (e - (u - 1.f)) / u;
      if (k < avail) my_loss += coef[k] * (fmaxf(z[k], 0.f) + log1p_e - y * z[k]);
    }
    st4(dlogits + i, avail, g);
    row += step_rows;
    col += step_cols;
    if (col >= C) col -= C, ++row;
  }
  store_partial(my_loss, partial);
}

// One workgroup: eight partial sums at most a thread, requested together
__global__ __launch_bounds__(256) void loss_reduce_kernel(const float* __restrict__ partial, int32_t count,
                                                          float* __restrict__ out) {
  static_assert(LOSS_BLOCKS == 8 * 256, "eight a thread");
  __shared__ float s[4];
  float x[8], acc = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int i = threadIdx.x + 256 * k;
    x[k] = partial[i < count ? i : 0];
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) acc += (int)threadIdx.x + 256 * k < count ? x[k] : 0.f;
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) *out = (s[0] + s[1]) + (s[2] + s[3]);
}

// partial[2b], partial[2b+1] = this block's sums of (a-b)^2 and a^2 (grid-stride, fixed order)
__global__ __launch_bounds__(256) void grad_gap_kernel(const float* __restrict__ a, const float* __restrict__ b,
                                                       int64_t n, float* __restrict__ partial) {
  __shared__ float wd[4], wr[4];
  float d2 = 0.f, r2 = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float x = a[i], d = x - b[i];
    d2 = fmaf(d, d, d2);
    r2 = fmaf(x, x, r2);
  }
  d2 = wave_sum(d2);
  r2 = wave_sum(r2);
  if ((threadIdx.x & 63) == 0) {
    wd[threadIdx.x >> 6] = d2;
    wr[threadIdx.x >> 6] = r2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = (wd[0] + wd[1]) + (wd[2] + wd[3]);
    partial[2 * blockIdx.x + 1] = (wr[0] + wr[1]) + (wr[2] + wr[3]);
  }
}

// out[j] = sqrt(sum over blocks of partial[2b + j]), j = 0, 1
__global__ __launch_bounds__(256) void grad_gap_finish_kernel(const float* __restrict__ partial, int32_t blocks,
                                                              float* __restrict__ out) {
  __shared__ float s[2][256];
  float acc0 = 0.f, acc1 = 0.f;
  for (int i = threadIdx.x; i < blocks; i += 256) {
    acc0 += partial[2 * i];
    acc1 += partial[2 * i + 1];
  }
  s[0][threadIdx.x] = acc0;
  s[1][threadIdx.x] = acc1;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      s[0][threadIdx.x] += s[0][threadIdx.x + o];
      s[1][threadIdx.x] += s[1][threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = sqrtf(s[0][0]);
    out[1] = sqrtf(s[1][0]);
  }
}

__global__ __launch_bounds__(256) void sgd_kernel(float* __restrict__ theta, const float* __restrict__ grad,
                                                  int64_t n, float lr) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) theta[i] -= lr * grad[i];
}

__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ theta, const float* __restrict__ grad,
                                                   float* __restrict__ m, float* __restrict__ v, int64_t n,
                                                   float lr, float b1, float b2, float eps, float inv_c1,
                                                   float inv_c2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float g = grad[i];
  const float mi = b1 * m[i] + (1.f - b1) * g;
  const float vi = b2 * v[i] + (1.f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  theta[i] -= lr * (mi * inv_c1) / (sqrtf(vi * inv_c2) + eps);
}

// ---- gradient gates: ReLU of the forward output and/or the dropout keep mask ----------------
template <typename T>
__global__ __launch_bounds__(256) void mask_grad_kernel(const T* src, const T* __restrict__ gate, T* dst,
                                                        int64_t total, float dropout_scale, uint32_t thr,
                                                        uint64_t seed, uint32_t epoch, uint32_t layer_stream) {
  // one thread per quad of four consecutive elements = one generator call
  const int64_t quad = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t base = quad * 4;
  if (base >= total) return;
  uint32_t words[4] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
  if (dropout_scale != 0.f) {
    const u32x4 w = draw4(seed, layer_stream, (uint64_t)quad, epoch);
    words[0] = w.x;
    words[1] = w.y;
    words[2] = w.z;
    words[3] = w.w;
  }
  if (base + 4 <= total) {  // whole quad: one 16-byte (float32) / 8-byte (bfloat16) access per operand
    float x[4], g[4] = {1.f, 1.f, 1.f, 1.f};
    ld_quad(src + base, x);
    if (gate) ld_quad(gate + base, g);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (!(g[c] > 0.f)) x[c] = 0.f;
      if (dropout_scale != 0.f) x[c] = words[c] >= thr ? x[c] * dropout_scale : 0.f;
    }
    st_quad(dst + base, x);
    return;
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int64_t i = base + c;
    if (i < total) {
      float x = ld_elem(src + i);
      if (gate && !(ld_elem(gate + i) > 0.f)) x = 0.f;
      if (dropout_scale != 0.f) x = words[c] >= thr ? x * dropout_scale : 0.f;
      st_elem(dst + i, x);
    }
  }
}

int32_t launch_mask_grad(int32_t dtype, const void* src, const void* gate, void* dst, int64_t M, int32_t N,
                         const DropoutArgs& d, hipStream_t stream) {
  COFREE_REQUIRE(src && dst, "mask_grad: NULL argument");
  COFREE_REQUIRE((((uintptr_t)src | (uintptr_t)dst | (uintptr_t)gate) & 15u) == 0, "mask_grad: buffers must be 16-byte aligned");
  COFREE_REQUIRE(dtype == COFREE_F32 || dtype == COFREE_BF16, "mask_grad: unknown dtype");
  const int64_t total = M * (int64_t)N;
  if (total == 0) return COFREE_OK;
  const int64_t quads = (total + 3) / 4;
  const int64_t blocks = (quads + 255) / 256;
  COFREE_REQUIRE(blocks < ((int64_t)1 << 31), "mask_grad: grid too large");
  float scale = 0.f;
  uint32_t thr = 0;
  if (d.q > 0.f) {
    scale = 1.0f / (1.0f - d.q);
    thr = prob_threshold((double)d.q);
  }
  ProfScope prof("mask_grad_kernel", stream, (dtype == COFREE_F32 ? 4.0 : 2.0) * (double)total * (gate ? 3 : 2),
                 (double)total);
  const uint32_t ls = STREAM_DROPOUT + 256u * d.layer_id;
  if (dtype == COFREE_F32)
    mask_grad_kernel<float><<<dim3((unsigned)blocks), 256, 0, stream>>>((const float*)src, (const float*)gate,
                                                                        (float*)dst, total, scale, thr, d.seed,
                                                                        d.epoch, ls);
  else
    mask_grad_kernel<bf16_t><<<dim3((unsigned)blocks), 256, 0, stream>>>((const bf16_t*)src, (const bf16_t*)gate,
                                                                         (bf16_t*)dst, total, scale, thr, d.seed,
                                                                         d.epoch, ls);
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

}  // namespace cofree

using namespace cofree;

extern "C" {

size_t cofree_loss_workspace_bytes(void) { return LOSS_BLOCKS * sizeof(float); }

// argument checks and weight vector shared by the two loss entry points
static int32_t loss_setup(const cofree_partition* part, int32_t weight_kind, const float* custom_w, const void* logits,
                          int32_t dtype, const void* labels, int32_t n_classes, const float* loss_out,
                          const void* dlogits, const void* workspace, size_t workspace_bytes, const float** w) {
  COFREE_REQUIRE(part != nullptr, "loss: partition is NULL");
  if (!part->on_device) return fail(COFREE_ESTATE, "loss: partition has no device copy");
  COFREE_REQUIRE(dtype == COFREE_F32 || dtype == COFREE_BF16, "loss: unknown dtype");
  COFREE_REQUIRE(logits && labels && loss_out && dlogits && workspace, "loss: NULL argument");
  COFREE_REQUIRE(n_classes >= 1, "loss: n_classes must be >= 1");
  if (workspace_bytes < cofree_loss_workspace_bytes()) return fail(COFREE_ENOMEM, "loss: workspace too small");
  switch (weight_kind) {
    case COFREE_W_DAR: *w = part->d_dar_weight; break;
    case COFREE_W_NONE: *w = nullptr; break;
    case COFREE_W_INV_RF:
      if (!part->d_inv_rf) return fail(COFREE_ESTATE, "loss: partition was built without COFREE_WITH_RF");
      *w = part->d_inv_rf;
      break;
    case COFREE_W_CUSTOM:
      COFREE_REQUIRE(custom_w != nullptr, "loss: custom_w is NULL");
      *w = custom_w;
      break;
    default: return fail(COFREE_EINVAL, "loss: unknown weight_kind");
  }
  return COFREE_OK;
}

// Workgroups of a loss over `items`, `each` of which a workgroup takes at a time: no more than there is work for, and `most`
static int loss_blocks(int64_t items, int64_t each, int most) {
  const int64_t b = (items + each - 1) / each;
  return b < 1 ? 1 : b < most ? (int)b : most;
}

// launches shared by cofree_loss_weighted and cofree_loss_weighted_static: `partial` holds LOSS_BLOCKS floats
static int32_t enqueue_softmax_loss(const cofree_partition* part, const float* w, const void* logits, int32_t dtype,
                                    const int32_t* labels, const uint8_t* train_mask, int32_t n_classes,
                                    float scale_c, float* loss_out, void* dlogits, float* partial, hipStream_t s) {
  const double es = dtype == COFREE_F32 ? 4.0 : 2.0;
  ProfScope prof("loss_kernels", s, (double)part->n_nodes * (2.0 * es * n_classes + 12.0),
                 8.0 * (double)part->n_nodes * n_classes);
#define COFREE_LOSS_ARGS(T) \
  (const T*)logits, labels, w, train_mask, part->n_nodes, n_classes, scale_c, (T*)dlogits, partial
  const bool f32 = dtype == COFREE_F32;
  const int pieces = (n_classes + (f32 ? 3 : 7)) / (f32 ? 4 : 8);  // of 16 bytes
  int blocks = 0;
#define COFREE_LOSS_GROUP(L, Q)                                                                \
  do {                                                                                         \
    blocks = loss_blocks(part->n_nodes, 2 * 256 / L, GROUP_BLOCKS);                            \
    if (f32) loss_group_kernel<float, L, Q><<<blocks, 256, 0, s>>>(COFREE_LOSS_ARGS(float));   \
    else loss_group_kernel<bf16_t, L, Q><<<blocks, 256, 0, s>>>(COFREE_LOSS_ARGS(bf16_t));     \
  } while (0)
  if (pieces <= 1) COFREE_LOSS_GROUP(1, 1);
  else if (pieces <= 2) COFREE_LOSS_GROUP(1, 2);
  else if (pieces <= 4) COFREE_LOSS_GROUP(2, 2);
  else if (pieces <= 8) COFREE_LOSS_GROUP(4, 2);
  else if (pieces <= 16) COFREE_LOSS_GROUP(8, 2);
  else if (pieces <= 32) COFREE_LOSS_GROUP(16, 2);
  else if (pieces <= 64) COFREE_LOSS_GROUP(32, 2);
  else if (pieces <= 128) COFREE_LOSS_GROUP(64, 2);
  else {
    blocks = loss_blocks(part->n_nodes, 4, LOSS_BLOCKS);
    if (f32) loss_kernel<float><<<blocks, 256, 0, s>>>(COFREE_LOSS_ARGS(float));
    else loss_kernel<bf16_t><<<blocks, 256, 0, s>>>(COFREE_LOSS_ARGS(bf16_t));
  }
#undef COFREE_LOSS_GROUP
#undef COFREE_LOSS_ARGS
  loss_reduce_kernel<<<1, 256, 0, s>>>(partial, blocks, loss_out);
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

int32_t cofree_loss_weighted(const cofree_partition* part, int32_t weight_kind, const float* custom_w,
                             const void* logits, int32_t dtype, const int32_t* labels, const uint8_t* train_mask,
                             int32_t n_classes, float scale_c, float* loss_out, void* dlogits, void* workspace,
                             size_t workspace_bytes, void* stream) {
  const float* w = nullptr;
  COFREE_TRY(loss_setup(part, weight_kind, custom_w, logits, dtype, labels, n_classes, loss_out, dlogits, workspace,
                        workspace_bytes, &w));
  return enqueue_softmax_loss(part, w, logits, dtype, labels, train_mask, n_classes, scale_c, loss_out, dlogits,
                              (float*)workspace, (hipStream_t)stream);
}

// Device address of `scratch` on the current GPU.  Looked up once per device, with that device current (every
// GPU holds its own copy of the array at its own address), and kept.
static int32_t static_scratch(float** out) {
  static std::mutex mu;
  static float* per_device[COFREE_STATIC_MAX_DEVICES] = {};
  int dev = -1;
  COFREE_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= COFREE_STATIC_MAX_DEVICES) return fail(COFREE_EINVAL, "loss_static: device index out of range");
  std::lock_guard<std::mutex> lk(mu);
  if (!per_device[dev]) {
    float* p = nullptr;
    COFREE_HIP_CHECK(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(COFREE_EHIP, "loss_static: hipGetSymbolAddress returned NULL");
    per_device[dev] = p;
  }
  *out = per_device[dev];
  return COFREE_OK;
}

int32_t cofree_loss_weighted_static(const cofree_partition* part, int32_t weight_kind, const float* custom_w,
                                    const void* logits, int32_t dtype, const int32_t* labels,
                                    const uint8_t* train_mask, int32_t n_classes, float scale_c, float* loss_out,
                                    void* dlogits, void* stream) {
  COFREE_REQUIRE(part != nullptr, "loss_static: partition is NULL");
  COFREE_REQUIRE(n_classes <= COFREE_LOSS_STATIC_MAX_CLASSES,
                 "loss_static: n_classes exceeds COFREE_LOSS_STATIC_MAX_CLASSES");
  COFREE_REQUIRE(part->n_nodes <= COFREE_LOSS_STATIC_MAX_NODES,
                 "loss_static: the partition has more nodes than COFREE_LOSS_STATIC_MAX_NODES");
  float* partial = nullptr;
  COFREE_TRY(static_scratch(&partial));
  const float* w = nullptr;
  COFREE_TRY(loss_setup(part, weight_kind, custom_w, logits, dtype, labels, n_classes, loss_out, dlogits, partial,
                        cofree_loss_workspace_bytes(), &w));
  // every partial sum that the reduction reads is written by its workgroup (a workgroup without rows writes 0)
  // before the reduction reads it, so nothing of an earlier call's contents survives into this one
  return enqueue_softmax_loss(part, w, logits, dtype, labels, train_mask, n_classes, scale_c, loss_out, dlogits,
                              partial, (hipStream_t)stream);
}

int32_t cofree_loss_bce_weighted(const cofree_partition* part, int32_t weight_kind, const float* custom_w,
                                 const void* logits, int32_t dtype, const uint8_t* targets, const uint8_t* train_mask,
                                 int32_t n_classes, float scale_c, float* loss_out, void* dlogits, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  const float* w = nullptr;
  COFREE_TRY(loss_setup(part, weight_kind, custom_w, logits, dtype, targets, n_classes, loss_out, dlogits, workspace,
                        workspace_bytes, &w));
  hipStream_t s = (hipStream_t)stream;
  float* partial = (float*)workspace;
  const double es = dtype == COFREE_F32 ? 4.0 : 2.0;
  ProfScope prof("loss_kernels", s, (double)part->n_nodes * ((2.0 * es + 1.0) * n_classes + 4.0),
                 12.0 * (double)part->n_nodes * n_classes);
  const int blocks = loss_blocks(part->n_nodes * n_classes, 4 * 256, LOSS_BLOCKS);
  if (dtype == COFREE_F32)
    bce_kernel<float><<<blocks, 256, 0, s>>>((const float*)logits, targets, w, train_mask, part->n_nodes,
                                                  n_classes, scale_c, (float*)dlogits, partial);
  else
    bce_kernel<bf16_t><<<blocks, 256, 0, s>>>((const bf16_t*)logits, targets, w, train_mask, part->n_nodes,
                                                   n_classes, scale_c, (bf16_t*)dlogits, partial);
  loss_reduce_kernel<<<1, 256, 0, s>>>(partial, blocks, loss_out);
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

int32_t cofree_grad_gap(int64_t n, const float* g_full, const float* g_sum, float* out, void* workspace,
                        size_t workspace_bytes, void* stream) {
  COFREE_REQUIRE(n >= 0, "grad_gap: n is negative");
  COFREE_REQUIRE((n == 0 || (g_full && g_sum)) && out && workspace, "grad_gap: NULL argument");
  if (workspace_bytes < cofree_loss_workspace_bytes()) return fail(COFREE_ENOMEM, "grad_gap: workspace too small");
  hipStream_t s = (hipStream_t)stream;
  constexpr int GAP_BLOCKS = LOSS_BLOCKS / 2;  // two partials per block
  float* partial = (float*)workspace;
  grad_gap_kernel<<<GAP_BLOCKS, 256, 0, s>>>(g_full, g_sum, n, partial);
  grad_gap_finish_kernel<<<1, 256, 0, s>>>(partial, GAP_BLOCKS, out);
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

int32_t cofree_step(int32_t kind, int64_t n, float* theta, const float* grad, float* m, float* v, float lr,
                    float b1, float b2, float eps, int64_t t, void* stream) {
  COFREE_REQUIRE(n >= 0, "step: n is negative");
  if (n == 0) return COFREE_OK;
  COFREE_REQUIRE(theta && grad, "step: NULL argument");
  const int64_t blocks = (n + 255) / 256;
  COFREE_REQUIRE(blocks < ((int64_t)1 << 31), "step: too many elements");
  hipStream_t s = (hipStream_t)stream;
  ProfScope prof("step_kernel", s, (kind == COFREE_SGD ? 12.0 : 28.0) * (double)n, 2.0 * (double)n);
  if (kind == COFREE_SGD) {
    sgd_kernel<<<dim3((unsigned)blocks), 256, 0, s>>>(theta, grad, n, lr);
  } else if (kind == COFREE_ADAM) {
    COFREE_REQUIRE(m && v, "step: Adam needs m and v");
    COFREE_REQUIRE(t >= 1, "step: Adam step count t must be >= 1");
    COFREE_REQUIRE(b1 >= 0.f && b1 < 1.f && b2 >= 0.f && b2 < 1.f, "step: betas must be in [0, 1)");
    const float inv_c1 = (float)(1.0 / (1.0 - std::pow((double)b1, (double)t)));
    const float inv_c2 = (float)(1.0 / (1.0 - std::pow((double)b2, (double)t)));
    adam_kernel<<<dim3((unsigned)blocks), 256, 0, s>>>(theta, grad, m, v, n, lr, b1, b2, eps, inv_c1, inv_c2);
  } else {
    return fail(COFREE_EINVAL, "step: unknown kind");
  }
  COFREE_HIP_CHECK(hipGetLastError());
  return COFREE_OK;
}

}  // extern "C"
