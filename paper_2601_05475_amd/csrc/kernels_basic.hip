// Plain-ALU kernels: embedding, residual + RMSNorm, RoPE + KV page write, a generic
// tiled linear layer, a generic attention kernel, sampling, reward scoring.
// They serve every dtype and shape; the bf16 MFMA kernels in kernels_mfma.hip take over
// the large contractions when the shape allows.
#include <stddef.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace mc {

// ------------------------------------------------------------------ block reductions
__device__ inline float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ inline double wave_sum_d(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// sum over a block of up to 1024 threads; every thread gets the result; fixed order
template <typename F>
__device__ inline F block_sum(F v, F *scratch /* >= 16 */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  F t = 0;
  for (int w = 0; w < nw; ++w) t += scratch[w];
  return t;
}
__device__ inline float block_max(float v, float *scratch) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  v = wave_max(v);
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  float t = scratch[0];
  for (int w = 1; w < nw; ++w) t = fmaxf(t, scratch[w]);
  return t;
}

// ------------------------------------------------------------------ embedding gather
template <typename T>
__global__ void embed_kernel(int d, const int32_t *__restrict__ tok, const T *__restrict__ table,
                             float *__restrict__ x) {
  const int r = blockIdx.x;
  const T *src = table + (size_t)tok[r] * d;
  float *dst = x + (size_t)r * d;
  if (sizeof(T) == 2 && d % 8 == 0) {
    // bf16 rows in 16-byte pieces (rows start on a multiple of 16 bytes: d % 8 == 0)
    for (int i = 8 * threadIdx.x; i < d; i += 8 * blockDim.x) {
      const uint4 e = *(const uint4 *)((const bf16_t *)src + i);
      *(float4 *)(dst + i) = make_float4(bf16_to_f32((bf16_t)(e.x & 0xFFFF)), bf16_to_f32((bf16_t)(e.x >> 16)),
                                         bf16_to_f32((bf16_t)(e.y & 0xFFFF)), bf16_to_f32((bf16_t)(e.y >> 16)));
      *(float4 *)(dst + i + 4) = make_float4(bf16_to_f32((bf16_t)(e.z & 0xFFFF)), bf16_to_f32((bf16_t)(e.z >> 16)),
                                             bf16_to_f32((bf16_t)(e.w & 0xFFFF)), bf16_to_f32((bf16_t)(e.w >> 16)));
    }
    return;
  }
  for (int i = threadIdx.x; i < d; i += blockDim.x) dst[i] = Cvt<T>::to_f32(src[i]);
}

int launch_embed(hipStream_t st, int dtype, int rows, int d, const int32_t *tokens,
                 const void *table, float *x) {
  if (rows <= 0) return MC_OK;
  if (dtype == MC_F32)
    embed_kernel<float><<<rows, 256, 0, st>>>(d, tokens, (const float *)table, x);
  else
    embed_kernel<bf16_t><<<rows, 256, 0, st>>>(d, tokens, (const bf16_t *)table, x);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// ------------------------------------------------------------------ residual + RMSNorm
// x[r] += sum_s partials[s][r];  h[r] = x[r] * gain / sqrt(mean(x[r]^2) + eps)
template <typename T>
__global__ __launch_bounds__(256) void add_rmsnorm_kernel(
    int rows, int d, float *__restrict__ x, const float *__restrict__ partials, int n_partials,
    size_t pstride, const T *__restrict__ gain, float eps, T *__restrict__ h, int h_tiled) {
  __shared__ float scratch[16];
  const int r = blockIdx.x;
  if (r >= rows) {                              // TILED_ZERO: a padding row
    for (int i = threadIdx.x; i < d; i += 256) h[tiled_offset(r, i, d)] = Cvt<T>::from_f32(0.f);
    return;
  }
  const size_t row = (size_t)blockIdx.x * d;
  float ss = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) {
    float v = x[row + i];
    for (int s = 0; s < n_partials; ++s) v += partials[s * pstride + row + i];
    if (n_partials) x[row + i] = v;
    ss += v * v;
  }
  ss = block_sum<float>(ss, scratch);
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  for (int i = threadIdx.x; i < d; i += 256) {
    const size_t at = h_tiled ? tiled_offset(r, i, d) : row + i;
    h[at] = Cvt<T>::from_f32(x[row + i] * inv * Cvt<T>::to_f32(gain[i]));
  }
}

// The same, four elements per thread and the row kept in registers between the two phases
// (d % 4 == 0, d <= 4 * VEC * blockDim).  bf16 output goes out as 8-byte stores; in the tiled
// layout four consecutive k stay inside one 16-byte chunk.
// rows_per_xcd > 0 (many rows): workgroups are dealt round-robin to the 8 XCDs, so block b works
// on row (b % 8) * rows_per_xcd + b / 8 and every XCD gets a contiguous range of rows.  In the
// tiled layout the 16-byte pieces of 8 consecutive rows share a 128-byte line; written from one
// L2 they leave as whole lines instead of eight partial ones.
// Written out, so that a row's sum has the same bits in every kernel that takes it (VEC fixes the order of the first two)
template <int VEC>
__device__ __forceinline__ float sum_squares(const float4 &v) {
  const float a = VEC == 1 ? v.x : v.y, b = VEC == 1 ? v.y : v.x;
  return fmaf(v.w, v.w, fmaf(v.z, v.z, fmaf(b, b, a * a)));
}

// false: a padding row (zeroed here where asked for) or no row at all
template <typename T>
__device__ __forceinline__ bool norm_row(int rows, int rows_per_xcd, int d, T *__restrict__ h, int h_tiled, int &r) {
  r = rows_per_xcd > 0 ? (int)(blockIdx.x & 7) * rows_per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  if (r < rows) return true;
  if (h_tiled == TILED_ZERO && r < padded_rows(rows))
    for (int i = 4 * threadIdx.x; i < d; i += 4 * blockDim.x) *(uint2 *)(h + tiled_offset(r, i, d)) = make_uint2(0u, 0u);    // tiled: bf16
  return false;
}

// v: the row's quads, ss: this thread's sum of their squares
template <typename T, int VEC>
__device__ __forceinline__ void norm_store(const float4 (&v)[VEC], float ss, int r, int d, const T *__restrict__ gain, float eps,
                                           T *__restrict__ h, int h_tiled, float *scratch) {
  const int nt = blockDim.x;
  const size_t row = (size_t)r * d;
  ss = block_sum<float>(ss, scratch);
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
  for (int j = 0; j < VEC; ++j) {
    const int i = 4 * (threadIdx.x + j * nt);
    if (i < d) {
      const size_t at = h_tiled ? tiled_offset(r, i, d) : row + i;
      const float o0 = v[j].x * inv * Cvt<T>::to_f32(gain[i]), o1 = v[j].y * inv * Cvt<T>::to_f32(gain[i + 1]),
                  o2 = v[j].z * inv * Cvt<T>::to_f32(gain[i + 2]), o3 = v[j].w * inv * Cvt<T>::to_f32(gain[i + 3]);
      if (sizeof(T) == 2) {
        uint2 pk;
        pk.x = (uint32_t)f32_to_bf16(o0) | ((uint32_t)f32_to_bf16(o1) << 16);
        pk.y = (uint32_t)f32_to_bf16(o2) | ((uint32_t)f32_to_bf16(o3) << 16);
        *(uint2 *)(h + at) = pk;
      } else {
        *(float4 *)(h + at) = make_float4(o0, o1, o2, o3);
      }
    }
  }
}

template <typename T, int VEC>
__global__ __launch_bounds__(1024) void add_rmsnorm_vec_kernel(
    int rows, int rows_per_xcd, int d, float *__restrict__ x, const float *__restrict__ partials, int n_partials,
    size_t pstride, const T *__restrict__ gain, float eps, T *__restrict__ h, int h_tiled) {
  __shared__ float scratch[16];
  const int nt = blockDim.x;
  int r;
  if (!norm_row(rows, rows_per_xcd, d, h, h_tiled, r)) return;
  const size_t row = (size_t)r * d;
  float4 v[VEC];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < VEC; ++j) {
    const int i = 4 * (threadIdx.x + j * nt);
    v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < d) {
      v[j] = *(const float4 *)(x + row + i);
      for (int s = 0; s < n_partials; ++s) {
        const float4 p = *(const float4 *)(partials + s * pstride + row + i);
        v[j].x += p.x; v[j].y += p.y; v[j].z += p.z; v[j].w += p.w;
      }
      if (n_partials) *(float4 *)(x + row + i) = v[j];
      ss += sum_squares<VEC>(v[j]);
    }
  }
  norm_store<T, VEC>(v, ss, r, d, gain, eps, h, h_tiled, scratch);
}

// Rows of a pass whose tokens, positions and KV slots are on the device
struct TokenRows {
  const int32_t *tok;
  __device__ int token(int r) const { return tok[r]; }
  __device__ void publish(int) const {}
};

// The first normalisation of a pass with the embedding gather in front of it, and for a decode step the rows' metadata
// beside it: a workgroup past the rows stores that, so no row waits for it.  Each of these is a few KB per row, so a
// decode step pays for the launches alone: metadata, gather and norm took 1.6 + 2.6 + 4.0 us at 8 rows of 2048.  The
// steps of a two-layer model of that width took 151 us so, 147 us with one launch.
template <typename T, int VEC, typename ROWS>
__global__ __launch_bounds__(1024) void embed_rmsnorm_kernel(int rows, int rows_per_xcd, int n_row_blocks, int d, ROWS src, const T *__restrict__ table,
                                                             float *__restrict__ x, const T *__restrict__ gain, float eps,
                                                             T *__restrict__ h, int h_tiled) {
  __shared__ float scratch[16];
  const int nt = blockDim.x;
  if ((int)blockIdx.x == n_row_blocks) {
    for (int i = threadIdx.x; i < rows; i += nt) src.publish(i);
    return;
  }
  int r;
  if (!norm_row(rows, rows_per_xcd, d, h, h_tiled, r)) return;
  const T *e = table + (size_t)src.token(r) * d;
  float *xr = x + (size_t)r * d;
  float4 v[VEC];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < VEC; ++j) {
    const int i = 4 * (threadIdx.x + j * nt);
    v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < d) {
      if (sizeof(T) == 2) {
        const uint2 p = *(const uint2 *)(e + i);
        v[j] = make_float4(bf16_to_f32((bf16_t)(p.x & 0xFFFF)), bf16_to_f32((bf16_t)(p.x >> 16)),
                           bf16_to_f32((bf16_t)(p.y & 0xFFFF)), bf16_to_f32((bf16_t)(p.y >> 16)));
      } else {
        v[j] = *(const float4 *)(e + i);
      }
      *(float4 *)(xr + i) = v[j];
      ss += sum_squares<VEC>(v[j]);
    }
  }
  norm_store<T, VEC>(v, ss, r, d, gain, eps, h, h_tiled, scratch);
}

__global__ void decode_rows_kernel(int rows, StepRows src, int32_t *__restrict__ tok) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  src.publish(r);
  tok[r] = src.token(r);
}

int launch_decode_rows(hipStream_t st, int rows, const StepRows &src, int32_t *tok) {
  decode_rows_kernel<<<(rows + 63) / 64, 64, 0, st>>>(rows, src, tok);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// Launch shape of the norms that take four elements per thread (norm_vec_ok)
struct NormShape {
  int nt, vec, rpx, grid;
};
bool norm_vec_ok(int d) { return d % 4 == 0 && d <= 16384; }
static NormShape norm_shape(int rows, int d, int h_tiled, int like_rows) {
  // enough threads for one float4 each where possible; at least one wave
  const int quads = d / 4, all_rows = h_tiled == TILED_ZERO ? padded_rows(rows) : rows;
  // many rows: 512 threads with two loads each in flight were measured faster than 1024 x 1
  const int nt_max = (like_rows >= 2048 && quads <= 4 * 512) ? 512 : 1024;
  NormShape n;
  n.nt = 64;
  while (n.nt < nt_max && n.nt < quads) n.nt *= 2;
  n.vec = (quads + n.nt - 1) / n.nt;
  // many rows into the tiled layout: a contiguous range of rows per XCD
  n.rpx = (h_tiled && rows >= 256) ? ((all_rows + 7) / 8 + 7) / 8 * 8 : 0;
  n.grid = n.rpx > 0 ? 8 * n.rpx : all_rows;
  return n;
}

template <typename T>
static void launch_add_rmsnorm_t(hipStream_t st, int rows, int d, float *x, const float *partials,
                                 int n_partials, size_t ps, const T *gain, float eps, T *h, int h_tiled, int like_rows) {
  if (norm_vec_ok(d)) {
    const NormShape n = norm_shape(rows, d, h_tiled, like_rows);
    if (n.vec <= 1) add_rmsnorm_vec_kernel<T, 1><<<n.grid, n.nt, 0, st>>>(rows, n.rpx, d, x, partials, n_partials, ps, gain, eps, h, h_tiled);
    else if (n.vec <= 2) add_rmsnorm_vec_kernel<T, 2><<<n.grid, n.nt, 0, st>>>(rows, n.rpx, d, x, partials, n_partials, ps, gain, eps, h, h_tiled);
    else add_rmsnorm_vec_kernel<T, 4><<<n.grid, n.nt, 0, st>>>(rows, n.rpx, d, x, partials, n_partials, ps, gain, eps, h, h_tiled);
  } else {
    const int all_rows = h_tiled == TILED_ZERO ? padded_rows(rows) : rows;
    add_rmsnorm_kernel<T><<<all_rows, 256, 0, st>>>(rows, d, x, partials, n_partials, ps, gain, eps, h, h_tiled);
  }
}

template <typename T, typename ROWS>
static void launch_embed_rmsnorm_t(hipStream_t st, int rows, int d, const ROWS &src, const T *table, float *x, const T *gain, float eps,
                                   T *h, int h_tiled) {
  const NormShape n = norm_shape(rows, d, h_tiled, rows);
  const int grid = n.grid + (std::is_same<ROWS, StepRows>::value ? 1 : 0);
  if (n.vec <= 1) embed_rmsnorm_kernel<T, 1, ROWS><<<grid, n.nt, 0, st>>>(rows, n.rpx, n.grid, d, src, table, x, gain, eps, h, h_tiled);
  else if (n.vec <= 2) embed_rmsnorm_kernel<T, 2, ROWS><<<grid, n.nt, 0, st>>>(rows, n.rpx, n.grid, d, src, table, x, gain, eps, h, h_tiled);
  else embed_rmsnorm_kernel<T, 4, ROWS><<<grid, n.nt, 0, st>>>(rows, n.rpx, n.grid, d, src, table, x, gain, eps, h, h_tiled);
}

int launch_embed_rmsnorm(hipStream_t st, int dtype, int rows, int d, const int32_t *tokens, const StepRows *step, const void *table,
                         float *x, const void *gain, float eps, void *h_out, int h_tiled) {
  if (rows <= 0) return MC_OK;
  if (!norm_vec_ok(d)) MC_FAIL(MC_ERR_UNSUPPORTED, "embedding with norm: d %% 4 == 0 and d <= 16384 (d = %d)", d);
  auto go = [&](const auto &src) {
    if (dtype == MC_F32) launch_embed_rmsnorm_t<float>(st, rows, d, src, (const float *)table, x, (const float *)gain, eps, (float *)h_out, h_tiled);
    else launch_embed_rmsnorm_t<bf16_t>(st, rows, d, src, (const bf16_t *)table, x, (const bf16_t *)gain, eps, (bf16_t *)h_out, h_tiled);
  };
  if (step) go(*step);
  else go(TokenRows{tokens});
  MC_HIP(hipGetLastError());
  return MC_OK;
}

int launch_add_rmsnorm(hipStream_t st, int dtype, int rows, int d, float *x, const float *partials,
                       int n_partials, const void *gain, float eps, void *h_out, int h_tiled, int like_rows) {
  if (rows <= 0) return MC_OK;
  if (like_rows <= 0) like_rows = rows;
  const size_t ps = (size_t)rows * d;
  if (dtype == MC_F32)
    launch_add_rmsnorm_t<float>(st, rows, d, x, partials, n_partials, ps, (const float *)gain, eps, (float *)h_out, h_tiled, like_rows);
  else
    launch_add_rmsnorm_t<bf16_t>(st, rows, d, x, partials, n_partials, ps, (const bf16_t *)gain, eps, (bf16_t *)h_out, h_tiled, like_rows);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

__global__ void gather_rows_kernel(int d, const float *__restrict__ x,
                                   const int32_t *__restrict__ idx, float *__restrict__ out) {
  const float *src = x + (size_t)idx[blockIdx.x] * d;
  float *dst = out + (size_t)blockIdx.x * d;
  for (int i = threadIdx.x; i < d; i += blockDim.x) dst[i] = src[i];
}

int launch_gather_rows(hipStream_t st, int rows, int d, const float *x, const int32_t *idx,
                       float *out) {
  if (rows <= 0) return MC_OK;
  gather_rows_kernel<<<rows, 256, 0, st>>>(d, x, idx, out);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// 4 to 10 KB of x and as much of t per row, one workgroup each: the launch is what it costs
__global__ __launch_bounds__(256) void gather_last_kernel(int d, int K, const float *__restrict__ x, const bf16_t *__restrict__ t,
                                                          const int32_t *__restrict__ idx, float *__restrict__ x_out,
                                                          bf16_t *__restrict__ t_out) {
  const int r = blockIdx.x, from = idx[r];
  for (int i = 4 * threadIdx.x; i < d; i += 4 * 256) *(float4 *)(x_out + (size_t)r * d + i) = *(const float4 *)(x + (size_t)from * d + i);
  for (int k = 8 * threadIdx.x; k < K; k += 8 * 256) *(uint4 *)(t_out + tiled_offset(r, k, K)) = *(const uint4 *)(t + tiled_offset(from, k, K));
}

int launch_gather_last(hipStream_t st, int rows, int d, int K, const float *x, const void *t, const int32_t *idx, float *x_out, void *t_out) {
  if (rows <= 0) return MC_OK;
  if (d % 4 || K % 64) MC_FAIL(MC_ERR_UNSUPPORTED, "gathered rows: d %% 4 == 0 and K %% 64 == 0 (d = %d, K = %d)", d, K);
  gather_last_kernel<<<rows, 256, 0, st>>>(d, K, x, (const bf16_t *)t, idx, x_out, (bf16_t *)t_out);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// ------------------------------------------------------------------ generic linear layer
// out[s][m][n] = sum_{k in split s} a[m][k] * w[n][k]; 64x64 tile, 16-deep slabs, 4x4 per thread.
// SWIGLU: two weight matrices, out[m][n] = silu(a.wg[n]) * (a.wu[n]) in the model dtype.
template <typename T, bool SWIGLU>
__global__ __launch_bounds__(256) void linear_generic_kernel(
    int M, int N, int K, int k_per_split, const T *__restrict__ a, const T *__restrict__ w,
    const T *__restrict__ w2, float *__restrict__ out, T *__restrict__ out_t) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 4];
  __shared__ float Ws[BK][BN + 4];
  __shared__ float Us[SWIGLU ? BK : 1][BN + 4];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN, split = blockIdx.z;
  const int k_begin = split * k_per_split;
  const int k_end = min(K, k_begin + k_per_split);
  float acc[4][4] = {}, acc2[4][4] = {};
  const int lr = tid >> 2, lk = (tid & 3) * 4;   // each thread stages 4 consecutive k of one row
  for (int k0 = k_begin; k0 < k_end; k0 += BK) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + lk + j;
      const bool kin = k < k_end;
      As[lk + j][lr] = (kin && m0 + lr < M) ? Cvt<T>::to_f32(a[(size_t)(m0 + lr) * K + k]) : 0.f;
      Ws[lk + j][lr] = (kin && n0 + lr < N) ? Cvt<T>::to_f32(w[(size_t)(n0 + lr) * K + k]) : 0.f;
      if (SWIGLU)
        Us[lk + j][lr] = (kin && n0 + lr < N) ? Cvt<T>::to_f32(w2[(size_t)(n0 + lr) * K + k]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float av[4], wv[4], uv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        av[i] = As[kk][ty * 4 + i];
        wv[i] = Ws[kk][tx * 4 + i];
        if (SWIGLU) uv[i] = Us[kk][tx * 4 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[i][j] += av[i] * wv[j];
          if (SWIGLU) acc2[i][j] += av[i] * uv[j];
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= N) continue;
      if (SWIGLU) {
        const float g = acc[i][j];
        out_t[(size_t)m * N + n] = Cvt<T>::from_f32(g / (1.0f + expf(-g)) * acc2[i][j]);
      } else {
        out[((size_t)split * M + m) * N + n] = acc[i][j];
      }
    }
  }
}

// The same for few rows (decode steps of fp32 models and of shapes the tiled kernels do not cover).
// With 64 x 64 tiles a 4 x 256 x 688 product is four workgroups that walk K in barriered slabs of 16,
// 34 us for 0.7 MB; here every wave takes one output column: its lanes stride over K with 16-byte
// loads, keep MR rows' sums and meet by shuffles.  What bounds it is the launch and one trip to memory
// (4 x 256 x 688: 34 -> 3.2 us, SwiGLU 4 x 688 x 256: 54 -> 4.0 us, LM head 4 x 4096 x 256: 26 -> 3.7 us).
template <typename T> struct Vec16;              // 16 bytes of T as floats
template <> struct Vec16<float> {
  static constexpr int N = 4;
  __device__ static void load(const float *p, float *v) {
    const float4 t = *(const float4 *)p;
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
};
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  __device__ static void load(const bf16_t *p, float *v) {
    const uint4 t = *(const uint4 *)p;
    const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = bf16_to_f32((bf16_t)(w[i] & 0xFFFF));
      v[2 * i + 1] = bf16_to_f32((bf16_t)(w[i] >> 16));
    }
  }
};

template <typename T, bool SWIGLU, int MR>
__global__ __launch_bounds__(256) void linear_few_rows_kernel(
    int M, int N, int K, int k_per_split, const T *__restrict__ a, const T *__restrict__ w,
    const T *__restrict__ w2, float *__restrict__ out, T *__restrict__ out_t) {
  constexpr int V = Vec16<T>::N;
  const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int m0 = blockIdx.y * MR, split = blockIdx.z;
  if (n >= N) return;
  const int k_begin = split * k_per_split, k_end = min(K, k_begin + k_per_split);
  float acc[MR] = {}, acc2[MR] = {};
  for (int k = k_begin + lane * V; k < k_end; k += 64 * V) {
    float wv[V], uv[V];
    Vec16<T>::load(w + (size_t)n * K + k, wv);
    if (SWIGLU) Vec16<T>::load(w2 + (size_t)n * K + k, uv);
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      float av[V];
      Vec16<T>::load(a + (size_t)min(m0 + m, M - 1) * K + k, av);
#pragma unroll
      for (int j = 0; j < V; ++j) {
        acc[m] += av[j] * wv[j];
        if (SWIGLU) acc2[m] += av[j] * uv[j];
      }
    }
  }
#pragma unroll
  for (int m = 0; m < MR; ++m) {
    acc[m] = wave_sum(acc[m]);
    if (SWIGLU) acc2[m] = wave_sum(acc2[m]);
  }
#pragma unroll
  for (int m = 0; m < MR; ++m)
    if (lane == m && m0 + m < M) {
      const float g = acc[m];
      if (SWIGLU) out_t[(size_t)(m0 + m) * N + n] = Cvt<T>::from_f32(g / (1.0f + expf(-g)) * acc2[m]);
      else out[((size_t)split * M + m0 + m) * N + n] = g;
    }
}

// Up to 32 rows, K in whole 16-byte pieces and pointers that allow them, and where it is the faster of the two
// by these estimates (us).  Here a wave pays for its start, for its sums' way across the lanes and for every
// 64 pieces of K it passes, full or not; the tiled kernel walks slabs of 16, 1.6 us each up to one workgroup per
// compute unit and more as they pile up.  Many rows, wide N and short or split K go to the tiles.  Fitted (what it
// chooses is at most 15 % off the better one) to
// fp32 and bf16, 4 to 32 rows, N 256 to 65536, K 256 to 4096, 1 to 16 splits; us tiles / here:
//   fp32:  4 x 256 x 688 34 / 3.2; 32 x 4096 x 4096 418 / 83, in 4 splits 110 / 77, in 16 57 / 128;
//          32 x 4096 x 256 in 4 splits 9 / 36; 16 x 14336 x 4096 403 / 140; 24 x 32000 x 1024 134 / 116, 32 rows 140 / 155
//   bf16:  32 x 32000 x 4096 548 / 401, in 4 splits of K 2048 175 / 264; SwiGLU 32 x 14336 x 4096 801 / 241,
//          32 x 65536 x 512 174 / 262
static bool few_rows_ok(int dtype, int M, int N, int K, int kps, int n_splits, const void *a, const void *w, const void *w2) {
  const int v = dtype == MC_F32 ? 4 : 8;
  if (M > 32 || K % v || (((uintptr_t)a | (uintptr_t)w | (uintptr_t)w2) & 15)) return false;
  const bool swiglu = w2 != nullptr;
  const double waves = (double)((M + 7) / 8) * N * n_splits * (M <= 4 ? 0.6 : 1.0), passes = (kps + 64 * v - 1) / (64 * v);
  const double here = waves * (swiglu ? 4.0e-4 + 4.0e-4 * passes : 2.3e-4 + 3.0e-4 * passes);
  const double slab = std::max(1.6, 0.95 + 0.0024 * ((N + 63) / 64) * n_splits) * (swiglu ? 1.9 : 1.0);
  return here <= kps / 16.0 * slab;
}

template <typename T, bool SWIGLU>
static void launch_few_rows(hipStream_t st, int M, int N, int K, int kps, int n_splits, const void *a, const void *w,
                            const void *w2, float *out, void *out_t) {
  const int mr = M <= 4 ? 4 : 8;
  const dim3 grid((N + 3) / 4, (M + mr - 1) / mr, n_splits);
  const T *A = (const T *)a, *W = (const T *)w, *W2 = (const T *)w2;
  if (mr == 4) linear_few_rows_kernel<T, SWIGLU, 4><<<grid, 256, 0, st>>>(M, N, K, kps, A, W, W2, out, (T *)out_t);
  else linear_few_rows_kernel<T, SWIGLU, 8><<<grid, 256, 0, st>>>(M, N, K, kps, A, W, W2, out, (T *)out_t);
}

// Whole layers of up to eight rows: the norm inside the product behind it, the QKV layer with rotation and stores, products that add to the
// residual stream.  A layer is then five launches (norm + QKV + rotary, attention, output projection, norm + SwiGLU, down projection) where it was
// eight.  As above a wave takes an output column (two for SwiGLU and for a rotary pair), with P pieces of 16 bytes of K per lane, all asked for at
// once.  NORM: a is fp32 x, and the operand is x * gain / sqrt(mean(x^2) + eps) rounded to the model's type; every wave takes the mean itself:
// rows of this path are a few KB, whose sum is a wave's shuffles away, where a norm launch takes 2.5 us and the gap before it.  What bounds the
// kernels is the launch and one trip to memory.
// A step of the two-layer fp32 model (4 candidates, d 256, F 688, vocabulary 4096): 19 launches -> 13, 61.6 -> 56.0 us.  Two loads deep over K in place
// of all at once: 16 steps 1480 against 1460 us.
// FEW_ROPE: a wave takes the members i and i + hd / 2 of a query or key head, or two coordinates of a value head.
enum { FEW_STORE = 0, FEW_SWIGLU = 1, FEW_ROPE = 2, FEW_ACCUM = 3 };
template <typename T, int MODE, bool NORM, int MR, int P>
__global__ __launch_bounds__(256) void few_rows_fused_kernel(int M, int N, int K, const void *__restrict__ a, const T *__restrict__ gain, float eps,
                                                             const T *__restrict__ w, const T *__restrict__ w2, float *__restrict__ out,
                                                             T *__restrict__ out_t, RopeOut ro) {
  constexpr int V = Vec16<T>::N;
  constexpr bool TWO = MODE == FEW_SWIGLU || MODE == FEW_ROPE;           // two weight rows per wave
  const int lane = threadIdx.x & 63, n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= (MODE == FEW_ROPE ? N / 2 : N)) return;
  const T *wr = w + (size_t)n * K, *ur = TWO ? w2 + (size_t)n * K : nullptr;
  int head = 0, i = 0, slot = 0, page = 0;
  double2 turn = {1.0, 0.0};
  if (MODE == FEW_ROPE) {
    const int half = ro.hd >> 1, row = min(lane & (MR - 1), M - 1);      // the row that this lane will store
    head = n / half;
    i = n % half;
    const bool turned = head < ro.Hq + ro.Hkv;
    wr = w + ((size_t)head * ro.hd + (turned ? i : 2 * i)) * K;
    ur = wr + (size_t)(turned ? half : 1) * K;
    slot = ro.row_off[row];
    page = ro.row_page[row];
    if (turned) turn = ro.table[(size_t)ro.row_pos[row] * half + i];
  }
  // pieces past K: the last one again, left out of the sums
  float av[MR][P][V], wv[P][V], uv[P][V], gv[P][V];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int k = min((p * 64 + lane) * V, K - V);
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      const size_t at = (size_t)min(m, M - 1) * K + k;
      if (NORM) {
#pragma unroll
        for (int j = 0; j < V; j += 4) Vec16<float>::load((const float *)a + at + j, av[m][p] + j);
      } else {
        Vec16<T>::load((const T *)a + at, av[m][p]);
      }
    }
    Vec16<T>::load(wr + k, wv[p]);
    if (TWO) Vec16<T>::load(ur + k, uv[p]);
    if (NORM) Vec16<T>::load(gain + k, gv[p]);
  }
  if (NORM) {
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      float ss = 0.f;
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int j = 0; j < V; ++j) ss = (p * 64 + lane) * V < K ? fmaf(av[m][p][j], av[m][p][j], ss) : ss;
      const float inv = 1.0f / sqrtf(wave_sum(ss) / (float)K + eps);
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int j = 0; j < V; ++j) av[m][p][j] = Cvt<T>::to_f32(Cvt<T>::from_f32(av[m][p][j] * inv * gv[p][j]));
    }
  }
  float acc[MR] = {}, acc2[MR] = {};
#pragma unroll
  for (int p = 0; p < P; ++p)
    if ((p * 64 + lane) * V < K)
#pragma unroll
      for (int m = 0; m < MR; ++m) {
        float s = 0.f, s2 = 0.f;                 // a piece by itself: short chains round less (K is not split over workgroups here)
#pragma unroll
        for (int j = 0; j < V; ++j) {
          s += av[m][p][j] * wv[p][j];
          if (TWO) s2 += av[m][p][j] * uv[p][j];
        }
        acc[m] += s;
        if (TWO) acc2[m] += s2;
      }
#pragma unroll
  for (int m = 0; m < MR; ++m) {
    acc[m] = wave_sum(acc[m]);
    if (TWO) acc2[m] = wave_sum(acc2[m]);
  }
#pragma unroll
  for (int m = 0; m < MR; ++m) {
    if (lane != m || m >= M) continue;
    const float g = acc[m];
    if (MODE == FEW_SWIGLU) {
      out_t[(size_t)m * N + n] = Cvt<T>::from_f32(g / (1.0f + expf(-g)) * acc2[m]);
    } else if (MODE == FEW_ACCUM) {
      out[(size_t)m * N + n] += g;
    } else if (MODE == FEW_STORE) {
      out[(size_t)m * N + n] = g;
    } else {
      const int hd = ro.hd, half = hd >> 1;
      const size_t at = (size_t)page * ro.Hkv * hd * ro.pg;
      const double lo = g, hi = acc2[m];
      if (head < ro.Hq + ro.Hkv) {
        const bool query = head < ro.Hq;
        T *dst = query ? (T *)ro.q_out + ((size_t)m * ro.Hq + head) * hd : (T *)ro.k_pages + at + (size_t)(head - ro.Hq) * ro.pg * hd;
        dst[query ? (size_t)i : k_elem_offset(slot, i, ro.pg, hd)] = Cvt<T>::from_f32((float)(lo * turn.x - hi * turn.y));
        dst[query ? (size_t)(i + half) : k_elem_offset(slot, i + half, ro.pg, hd)] = Cvt<T>::from_f32((float)(hi * turn.x + lo * turn.y));
      } else {
        T *dst = (T *)ro.v_pages + at + (size_t)(head - ro.Hq - ro.Hkv) * ro.pg * hd;
        dst[v_elem_offset(slot, 2 * i, ro.pg, hd)] = Cvt<T>::from_f32(g);
        dst[v_elem_offset(slot, 2 * i + 1, ro.pg, hd)] = Cvt<T>::from_f32(acc2[m]);
      }
    }
  }
}

// Where every product of the model goes by columns as it stands, K is at most 1024 (above, a K that is not split over workgroups costs more)
// and the rows are at most eight: every wave reads all its rows and takes their means, which 16 rows or a wide output pay for once per column.
// us per step, separate launches / this, two layers: d 256, F 688 58.7 / 52.5 for one row, 61.6 / 57.0 for 4, 74.3 / 72.0 for 8; d 512, F 1024
// 66.3 / 58.7, 69.0 / 63.6, 86.9 / 80.3; d 1024, F 1024 91.9 / 80.3, 98.3 / 86.0, 124 / 106; bf16, d 504 63.5 / 60.4, 67.7 / 65.6, 94.1 / 89.9;
// d 20 72.7 / 64.3, 73.7 / 69.6, 84.5 / 89.6.  With 16 rows
// and the LM head so too d 768 190 / 350, with 32 rows bf16 d 1016 255 / 629.
constexpr int kFusedMostK = 1024, kFusedMostRows = 8;
bool few_rows_fused_ok(int dtype, int rows, int d, int n_qkv, int qd, int F, int vocab, int head_dim) {
  if (rows > (d < 64 ? 4 : kFusedMostRows) || head_dim % 2 || std::max(d, std::max(qd, F)) > kFusedMostK) return false;
  // (the operands are rows of the model's and the session's arenas, aligned for 16-byte loads)
  auto ok = [&](int N, int K, bool swiglu) { return few_rows_ok(dtype, rows, N, K, K, 1, nullptr, nullptr, swiglu ? (const void *)16 : nullptr); };
  return ok(n_qkv, d, false) && ok(d, qd, false) && ok(F, d, true) && ok(d, F, false) && ok(vocab, d, false);
}
// The LM head with the final norm inside: fp32, up to four rows and a vocabulary of 4096.  us per step, norm and LM head apart / together, d 256: vocabulary
// 4096 57.0 / 56.0 for 4 rows, 72.0 / 72.2 for 8, 8192 58.1 / 58.3, 16384 60.6 / 63.1, 32000 67.1 / 74.0 and for 8 rows 88.4 / 102.8; bf16, d 504, vocabulary
// 4096 65.6 / 67.1.
bool few_rows_lm_head_ok(int dtype, int rows, int vocab) { return dtype == MC_F32 && rows <= 4 && vocab <= 4096; }

template <typename T, int MODE, bool NORM>
static void launch_few_fused_t(hipStream_t st, int M, int N, int K, const void *a, const void *gain, float eps, const void *w, const void *w2,
                               float *out, void *out_t, const RopeOut &ro) {
  const int columns = MODE == FEW_ROPE ? N / 2 : N, pieces = (K + 64 * Vec16<T>::N - 1) / (64 * Vec16<T>::N), grid = (columns + 3) / 4;
  auto go = [&](auto p) {
    constexpr int P = decltype(p)::value;
    if (M <= 4)
      few_rows_fused_kernel<T, MODE, NORM, 4, P><<<grid, 256, 0, st>>>(M, N, K, a, (const T *)gain, eps, (const T *)w, (const T *)w2, out, (T *)out_t, ro);
    else if constexpr (MODE != FEW_STORE)
      few_rows_fused_kernel<T, MODE, NORM, 8, P><<<grid, 256, 0, st>>>(M, N, K, a, (const T *)gain, eps, (const T *)w, (const T *)w2, out, (T *)out_t, ro);
  };
  if (pieces <= 1) go(std::integral_constant<int, 1>{});
  else if (pieces <= 2) go(std::integral_constant<int, 2>{});
  else if constexpr (sizeof(T) == 4) go(std::integral_constant<int, kFusedMostK / 256>{});
}

template <int MODE, bool NORM>
static int launch_few_fused(hipStream_t st, int dtype, int M, int N, int K, const void *a, const void *gain, float eps, const void *w,
                            const void *w2, float *out, void *out_t, const RopeOut &ro) {
  const bool lm_head = MODE == FEW_STORE;
  if (K > kFusedMostK || M > (lm_head ? 4 : kFusedMostRows) || (lm_head && dtype != MC_F32))
    MC_FAIL(MC_ERR_UNSUPPORTED, "fused layers of few rows: %d rows, K = %d", M, K);
  if (dtype == MC_F32) launch_few_fused_t<float, MODE, NORM>(st, M, N, K, a, gain, eps, w, w2, out, out_t, ro);
  else if constexpr (MODE != FEW_STORE) launch_few_fused_t<bf16_t, MODE, NORM>(st, M, N, K, a, gain, eps, w, w2, out, out_t, ro);
  MC_HIP(hipGetLastError());
  return MC_OK;
}
int launch_norm_qkv_rope_few(hipStream_t st, int dtype, int M, int N, int K, const float *x, const void *gain, float eps, const void *w, const RopeOut &ro) {
  return launch_few_fused<FEW_ROPE, true>(st, dtype, M, N, K, x, gain, eps, w, nullptr, nullptr, nullptr, ro);
}
int launch_norm_swiglu_few(hipStream_t st, int dtype, int M, int N, int K, const float *x, const void *gain, float eps, const void *wg, const void *wu, void *out) {
  return launch_few_fused<FEW_SWIGLU, true>(st, dtype, M, N, K, x, gain, eps, wg, wu, nullptr, out, RopeOut{});
}
int launch_norm_linear_few(hipStream_t st, int dtype, int M, int N, int K, const float *x, const void *gain, float eps, const void *w, float *out) {
  return launch_few_fused<FEW_STORE, true>(st, dtype, M, N, K, x, gain, eps, w, nullptr, out, nullptr, RopeOut{});
}
int launch_accumulate_few(hipStream_t st, int dtype, int M, int N, int K, const void *a, const void *w, float *x) {
  return launch_few_fused<FEW_ACCUM, false>(st, dtype, M, N, K, a, nullptr, 0.f, w, nullptr, x, nullptr, RopeOut{});
}

int launch_linear_generic(hipStream_t st, int dtype, int M, int N, int K, const void *a,
                          const void *w, float *out, int n_splits) {
  if (M <= 0 || N <= 0) return MC_OK;
  int kps = (K + n_splits - 1) / n_splits;
  kps = (kps + 15) / 16 * 16;
  if (few_rows_ok(dtype, M, N, K, kps, n_splits, a, w, nullptr)) {
    if (dtype == MC_F32) launch_few_rows<float, false>(st, M, N, K, kps, n_splits, a, w, nullptr, out, nullptr);
    else launch_few_rows<bf16_t, false>(st, M, N, K, kps, n_splits, a, w, nullptr, out, nullptr);
    MC_HIP(hipGetLastError());
    return MC_OK;
  }
  dim3 grid((N + 63) / 64, (M + 63) / 64, n_splits);
  if (dtype == MC_F32)
    linear_generic_kernel<float, false><<<grid, 256, 0, st>>>(
        M, N, K, kps, (const float *)a, (const float *)w, nullptr, out, nullptr);
  else
    linear_generic_kernel<bf16_t, false><<<grid, 256, 0, st>>>(
        M, N, K, kps, (const bf16_t *)a, (const bf16_t *)w, nullptr, out, nullptr);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

int launch_linear_swiglu_generic(hipStream_t st, int dtype, int M, int N, int K, const void *a,
                                 const void *wg, const void *wu, void *out) {
  if (M <= 0 || N <= 0) return MC_OK;
  if (few_rows_ok(dtype, M, N, K, K, 1, a, wg, wu)) {
    if (dtype == MC_F32) launch_few_rows<float, true>(st, M, N, K, K, 1, a, wg, wu, nullptr, out);
    else launch_few_rows<bf16_t, true>(st, M, N, K, K, 1, a, wg, wu, nullptr, out);
    MC_HIP(hipGetLastError());
    return MC_OK;
  }
  dim3 grid((N + 63) / 64, (M + 63) / 64, 1);
  if (dtype == MC_F32)
    linear_generic_kernel<float, true><<<grid, 256, 0, st>>>(
        M, N, K, (K + 15) / 16 * 16, (const float *)a, (const float *)wg, (const float *)wu,
        nullptr, (float *)out);
  else
    linear_generic_kernel<bf16_t, true><<<grid, 256, 0, st>>>(
        M, N, K, (K + 15) / 16 * 16, (const bf16_t *)a, (const bf16_t *)wg, (const bf16_t *)wu,
        nullptr, (bf16_t *)out);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// ------------------------------------------------------------------ RoPE + KV page write
__global__ void rope_table_kernel(int n_pos, int half, int hd, double rope_base, double2 *__restrict__ table) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)n_pos * half) return;
  const int pos = (int)(e / half), i = (int)(e % half);
  double sn, cs;
  sincos((double)pos * pow(rope_base, -2.0 * (double)i / (double)hd), &sn, &cs);
  table[e] = make_double2(cs, sn);
}

int launch_rope_table(hipStream_t st, int n_pos, int hd, double rope_base, double2 *table) {
  const size_t n = (size_t)n_pos * (hd / 2);
  if (n == 0) return MC_OK;
  rope_table_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(n_pos, hd / 2, hd, rope_base, table);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// One block per (row, head).  Heads 0..Hq-1 are queries, then Hkv key heads, then Hkv value
// heads.  The angle pos * base^(-2i/hd) and its sine/cosine are taken in double (from the table
// of the same expressions when one is given).  qk_interleaved: coordinate i of a query / key head
// sits at 2i and coordinate i + hd/2 at 2i + 1 of the input row (see launch_pack_tiled).
template <typename T>
__global__ __launch_bounds__(64) void rope_kv_kernel(
    int rows, int Hq, int Hkv, int hd, int pg, double rope_base,
    const float *__restrict__ qkv, int n_splits, const int32_t *__restrict__ row_pos,
    const int32_t *__restrict__ row_page, const int32_t *__restrict__ row_off,
    T *__restrict__ q_out, T *__restrict__ k_pages, T *__restrict__ v_pages,
    const double2 *__restrict__ table, int qk_interleaved) {
  const int r = blockIdx.x, h = blockIdx.y;
  const int nqkv = (Hq + 2 * Hkv) * hd, half = hd >> 1;
  const size_t sstride = (size_t)rows * nqkv;
  const float *src = qkv + (size_t)r * nqkv + (size_t)h * hd;
  const size_t pelems = (size_t)Hkv * hd * pg;
  if (h < Hq + Hkv) {
    const double pos = (double)row_pos[r];
    // queries go out row-major; a key goes to its slot of the page, in the page's layout
    T *dst = (h < Hq) ? q_out + ((size_t)r * Hq + h) * hd
                      : k_pages + (size_t)row_page[r] * pelems + (size_t)(h - Hq) * pg * hd;
    const int key = row_off[r];
    for (int i = threadIdx.x; i < half; i += 64) {
      float lo = 0.f, hi = 0.f;
      const int at_l = qk_interleaved ? 2 * i : i, at_h = qk_interleaved ? 2 * i + 1 : i + half;
      for (int s = 0; s < n_splits; ++s) {
        lo += src[s * sstride + at_l];
        hi += src[s * sstride + at_h];
      }
      double sn, cs;
      if (table) {
        const double2 t = table[(size_t)row_pos[r] * half + i];
        cs = t.x; sn = t.y;
      } else {
        sincos(pos * pow(rope_base, -2.0 * (double)i / (double)hd), &sn, &cs);
      }
      const size_t at_lo = (h < Hq) ? (size_t)i : k_elem_offset(key, i, pg, hd);
      const size_t at_hi = (h < Hq) ? (size_t)(i + half) : k_elem_offset(key, i + half, pg, hd);
      dst[at_lo] = Cvt<T>::from_f32((float)((double)lo * cs - (double)hi * sn));
      dst[at_hi] = Cvt<T>::from_f32((float)((double)hi * cs + (double)lo * sn));
    }
  } else {
    const int kvh = h - Hq - Hkv;
    T *dst = v_pages + (size_t)row_page[r] * pelems + (size_t)kvh * hd * pg;
    const int key = row_off[r];
    for (int i = threadIdx.x; i < hd; i += 64) {
      float v = 0.f;
      for (int s = 0; s < n_splits; ++s) v += src[s * sstride + i];
      dst[v_elem_offset(key, i, pg, hd)] = Cvt<T>::from_f32(v);
    }
  }
}

int launch_rope_kv(hipStream_t st, int dtype, int rows, int Hq, int Hkv, int hd, int page_tokens,
                   double rope_base, const float *qkv, int n_splits, const int32_t *row_pos,
                   const int32_t *row_page, const int32_t *row_off, void *q_out, void *k_pages,
                   void *v_pages, const double2 *table, int qk_interleaved) {
  if (rows <= 0) return MC_OK;
  dim3 grid(rows, Hq + 2 * Hkv);
  if (dtype == MC_F32)
    rope_kv_kernel<float><<<grid, 64, 0, st>>>(rows, Hq, Hkv, hd, page_tokens, rope_base, qkv,
                                               n_splits, row_pos, row_page, row_off,
                                               (float *)q_out, (float *)k_pages, (float *)v_pages,
                                               table, qk_interleaved);
  else
    rope_kv_kernel<bf16_t><<<grid, 64, 0, st>>>(rows, Hq, Hkv, hd, page_tokens, rope_base, qkv,
                                                n_splits, row_pos, row_page, row_off,
                                                (bf16_t *)q_out, (bf16_t *)k_pages,
                                                (bf16_t *)v_pages, table, qk_interleaved);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// ------------------------------------------------------------------ generic attention
// One workgroup per (query row, query head); its four waves take 64-key blocks in turn, first of the
// prefix keys the row sees, then of its own suffix keys, each with a running (max, sum, weighted
// value) state, and meet in LDS at the end.  Inside a block lane j scores key j (its row of K in
// pieces of four coordinates), then lane d accumulates coordinates d, d + 64, ... of the value sum,
// four consecutive keys per load: both page layouts keep them together, and a page holds whole
// quads of keys unless page_tokens is 1 or 2, when keys are taken one by one.
// At the tiny fp32 shape (16 workgroups, 136 keys) the time is the latency of a few rounds of loads:
// 23 us with one wave per workgroup and 4-byte loads, 9 us so.
template <typename T> __device__ inline float4 load4(const T *p);
template <> __device__ inline float4 load4<float>(const float *p) { return *(const float4 *)p; }
template <> __device__ inline float4 load4<bf16_t>(const bf16_t *p) {
  const uint2 t = *(const uint2 *)p;
  return make_float4(bf16_to_f32((bf16_t)(t.x & 0xFFFF)), bf16_to_f32((bf16_t)(t.x >> 16)),
                     bf16_to_f32((bf16_t)(t.y & 0xFFFF)), bf16_to_f32((bf16_t)(t.y >> 16)));
}

constexpr int kAttnWaves = 4;

// x of lane t, t uniform: by way of scalar registers, no trip through LDS
__device__ inline uint32_t of_lane(uint32_t x, int t) { return __builtin_amdgcn_readlane(x, t); }
__device__ inline unsigned long long of_lane(unsigned long long x, int t) {
  return ((unsigned long long)of_lane((uint32_t)(x >> 32), t) << 32) | of_lane((uint32_t)x, t);
}

// K4: head_dim is a multiple of 4 and the pools are aligned for loads of four elements (a key's coordinates lie
// together by fours in both layouts); V4: page_tokens is one as well (quads of keys).  With K by single
// loads, 64 rows x 16 heads of 64, 220 keys in pages of 2 took 53 us, by fours 28.
template <typename T, bool K4, bool V4>
__global__ __launch_bounds__(64 * kAttnWaves) void attention_generic_kernel(AttnArgs a) {
  constexpr int MAXD = 4;   // head_dim <= 256
  __shared__ __attribute__((aligned(16))) float qs[256];
  __shared__ __attribute__((aligned(16))) float ps[kAttnWaves][64];
  __shared__ float sm[kAttnWaves], sl[kAttnWaves], so[kAttnWaves][256];
  const int r = blockIdx.x, qh = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int hd = a.head_dim, pg = a.page_tokens, Hkv = a.n_kv_heads;
  const int kvh = qh / (a.n_q_heads / Hkv);
  int pos, tab_row = 0;
  if (a.row_pos) {
    pos = a.row_pos[r];
    if (a.page_table) tab_row = a.row_tab[r];
  } else {                                   // a decode step: one row per candidate, its last key is its own
    const int len = (a.row_len && a.suffix_len) ? min(max(a.row_len[r], 1), a.suffix_len) : a.suffix_len;
    pos = a.prefix_len + len - 1;
    tab_row = a.row_cand ? a.row_cand[r] : r;
  }
  const int n_keys = pos + 1, n_pre = min(n_keys, a.prefix_len);
  const size_t pelems = (size_t)Hkv * hd * pg, head_off = (size_t)kvh * hd * pg;
  const T *q = (const T *)a.q + ((size_t)r * a.n_q_heads + qh) * hd;
  for (int i = threadIdx.x; i < hd; i += 64 * kAttnWaves) qs[i] = Cvt<T>::to_f32(q[i]);
  const int32_t *tab = a.page_table ? a.page_table + (size_t)tab_row * a.table_stride : nullptr;
  const float scale = 1.0f / sqrtf((float)hd);
  float m = -INFINITY, l = 0.f, o[MAXD] = {0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  const int blocks_pre = (n_pre + 63) / 64, blocks_all = blocks_pre + (n_keys - n_pre + 63) / 64;
  for (int blk = wave; blk < blocks_all; blk += kAttnWaves) {
    const bool in_prefix = blk < blocks_pre;
    const int j0 = 64 * (in_prefix ? blk : blk - blocks_pre), n_seg = in_prefix ? n_pre : n_keys - n_pre;
    const int nblk = min(64, n_seg - j0), j = j0 + min(lane, nblk - 1);   // lanes past the end look at its last key
    const int page = in_prefix ? j / pg : tab[j / pg], off = j % pg;
    const size_t base = (size_t)page * pelems + head_off;
    const T *kp = (const T *)(in_prefix ? a.k_prefix : a.k_suffix) + base;
    const T *vpool = (const T *)(in_prefix ? a.v_prefix : a.v_suffix);
    float dot = 0.f;
    if (K4) {
#pragma unroll 4
      for (int i = 0; i < hd; i += 4) {
        const float4 k4 = load4<T>(kp + k_elem_offset(off, i, pg, hd)), q4 = *(const float4 *)(qs + i);
        dot += q4.x * k4.x; dot += q4.y * k4.y; dot += q4.z * k4.z; dot += q4.w * k4.w;
      }
    } else if (!kv_fragment_layout(pg, hd)) {
      const T *kr = kp + (size_t)off * hd;
      for (int i = 0; i < hd; ++i) dot += qs[i] * Cvt<T>::to_f32(kr[i]);
    } else {
      for (int i = 0; i < hd; ++i) dot += qs[i] * Cvt<T>::to_f32(kp[k_elem_offset(off, i, pg, hd)]);
    }
    const float s = lane < nblk ? dot * scale : -INFINITY;
    const float m_new = fmaxf(m, wave_max(s));
    const float p = lane < nblk ? expf(s - m_new) : 0.f;
    const float corr = expf(m - m_new);      // m = -inf on the first block: exp(-inf) = 0
    l = l * corr + wave_sum(p);
    ps[wave][lane] = p;                      // read by this wave only, in order behind the write
    m = m_new;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int c = 0; c < MAXD; ++c) {
      const int d = lane + 64 * c;
      if (64 * c >= hd) break;               // uniform
      float acc = o[c] * corr;
      if (V4) {
        // the last quad may reach past the sequence's end: its page holds the bytes, their weight is
        // not taken
#pragma unroll 4
        for (int t = 0; t < nblk; t += 4) {
          const size_t vb = of_lane((unsigned long long)base, t);
          const int vo = of_lane((uint32_t)off, t);
          const float4 w4 = *(const float4 *)(&ps[wave][t]);
          if (d < hd) {
            const float4 v4 = load4<T>(vpool + vb + v_elem_offset(vo, d, pg, hd));
            acc += w4.x * v4.x;
            if (t + 1 < nblk) acc += w4.y * v4.y;
            if (t + 2 < nblk) acc += w4.z * v4.z;
            if (t + 3 < nblk) acc += w4.w * v4.w;
          }
        }
      } else {
#pragma unroll 4
        for (int t = 0; t < nblk; ++t) {
          const size_t vb = of_lane((unsigned long long)base, t);
          const int vo = of_lane((uint32_t)off, t);
          if (d < hd) acc += ps[wave][t] * Cvt<T>::to_f32(vpool[vb + v_elem_offset(vo, d, pg, hd)]);
        }
      }
      o[c] = acc;
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (lane == 0) { sm[wave] = m; sl[wave] = l; }
#pragma unroll
  for (int c = 0; c < MAXD; ++c)
    if (lane + 64 * c < hd) so[wave][lane + 64 * c] = o[c];
  __syncthreads();
  float M = sm[0];
  for (int w = 1; w < kAttnWaves; ++w) M = fmaxf(M, sm[w]);
  float f[kAttnWaves], den = 0.f;
  for (int w = 0; w < kAttnWaves; ++w) {
    f[w] = sm[w] == -INFINITY ? 0.f : expf(sm[w] - M);    // a wave that saw no key has no weight
    den += f[w] * sl[w];
  }
  T *out = (T *)a.out;
  for (int d = threadIdx.x; d < hd; d += 64 * kAttnWaves) {
    float num = 0.f;
    for (int w = 0; w < kAttnWaves; ++w) num += f[w] * so[w][d];
    const size_t at = a.out_tiled ? tiled_offset(r, qh * hd + d, a.n_q_heads * hd)
                                  : ((size_t)r * a.n_q_heads + qh) * hd + d;
    out[at] = Cvt<T>::from_f32(num / den);
    if (a.out_tiled == TILED_ZERO)               // row r answers for padding rows rows + r, 2 rows + r, ...
      for (int z = a.rows + r; z < padded_rows(a.rows); z += a.rows) out[tiled_offset(z, qh * hd + d, a.n_q_heads * hd)] = Cvt<T>::from_f32(0.f);
  }
}

template <typename T>
static void launch_attention_generic_t(hipStream_t st, const AttnArgs &a) {
  const uintptr_t pools = (uintptr_t)a.k_prefix | (uintptr_t)a.v_prefix | (uintptr_t)a.k_suffix | (uintptr_t)a.v_suffix;
  const bool k4 = a.head_dim % 4 == 0 && pools % (4 * sizeof(T)) == 0;
  const dim3 grid(a.rows, a.n_q_heads);
  if (k4 && a.page_tokens % 4 == 0) attention_generic_kernel<T, true, true><<<grid, 64 * kAttnWaves, 0, st>>>(a);
  else if (k4) attention_generic_kernel<T, true, false><<<grid, 64 * kAttnWaves, 0, st>>>(a);
  else attention_generic_kernel<T, false, false><<<grid, 64 * kAttnWaves, 0, st>>>(a);
}

int launch_attention_generic(hipStream_t st, int dtype, const AttnArgs &a) {
  if (a.rows <= 0) return MC_OK;
  if (a.head_dim > 256) MC_FAIL(MC_ERR_UNSUPPORTED, "head_dim %d > 256", a.head_dim);
  if (dtype == MC_F32) launch_attention_generic_t<float>(st, a);
  else launch_attention_generic_t<bf16_t>(st, a);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// ------------------------------------------------------------------ sampling
// Order-preserving map of a float to an unsigned integer (larger float -> larger integer).
__device__ inline uint32_t float_order_bits(float f) {
  const uint32_t b = __float_as_uint(f + 0.0f);       // -0 -> +0
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float float_from_order_bits(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}
// 64-bit key whose descending order is (z descending, id ascending)
__device__ inline unsigned long long sample_key(float z, int id) {
  return ((unsigned long long)float_order_bits(z) << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)id);
}

__device__ inline unsigned long long block_max_u64(unsigned long long v, unsigned long long *scratch) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  for (int o = 32; o > 0; o >>= 1) {
    unsigned long long t = __shfl_xor(v, o, 64);
    v = t > v ? t : v;
  }
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  unsigned long long t = scratch[0];
  for (int w = 1; w < nw; ++w) t = scratch[w] > t ? scratch[w] : t;
  return t;
}

__device__ inline unsigned int block_reduce_u32(unsigned int v, bool take_max, unsigned int *scratch) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned int t = __shfl_xor(v, o, 64);
    v = take_max ? max(v, t) : min(v, t);
  }
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  unsigned int t = scratch[0];
  for (int w = 1; w < nw; ++w) t = take_max ? max(t, scratch[w]) : min(t, scratch[w]);
  return t;
}

// Slot in a shared list for every lane with `want` set: one atomic per wave, not per lane.
__device__ inline unsigned int wave_claim(bool want, unsigned int *counter) {
  const unsigned long long m = __ballot(want);
  if (m == 0) return 0;
  const int leader = __ffsll((long long)m) - 1;
  unsigned int base = 0;
  if ((int)(threadIdx.x & 63) == leader) base = atomicAdd(counter, (unsigned int)__popcll(m));
  base = __shfl(base, leader, 64);
  return base + (unsigned int)__popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull));
}

// Walk one row with all 1024 threads: f(valid, logit, index) is called the same number of times
// by every thread (so f may use wave-wide operations).  Loads go out in batches of eight 16-byte
// vectors per thread; a loop of single dependent-looking loads would pay the memory latency
// once per element.
template <typename F>
__device__ inline void scan_row(const float *row, int V, F f) {
  constexpr int NB = 8;
  const int tid = threadIdx.x;
  const int V4 = (((uintptr_t)row & 15) == 0) ? V / 4 : 0;
  const float4 *row4 = (const float4 *)row;
  for (int g0 = 0; g0 < V4; g0 += NB * 1024) {
    float4 z[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int g = g0 + j * 1024 + tid;
      z[j] = (g < V4) ? row4[g] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int g = g0 + j * 1024 + tid;
      const bool ok = g < V4;
      f(ok, z[j].x, 4 * g);
      f(ok, z[j].y, 4 * g + 1);
      f(ok, z[j].z, 4 * g + 2);
      f(ok, z[j].w, 4 * g + 3);
    }
  }
  for (int v0 = 4 * V4; v0 < V; v0 += 1024) {
    const int v = v0 + tid;
    const bool ok = v < V;
    f(ok, ok ? row[v] : 0.f, v);
  }
}

// LDS of the sampling kernel
struct SampleShared {
  unsigned long long sel[MC_MAX_TOP_K];
  float ev[MC_MAX_TOP_K];
  alignas(16) unsigned int hist[2048];
  unsigned long long scratch64[16];
  unsigned int scratch32[16];
  unsigned int s_bin, s_above, s_cnt, s_cnt2;
};
// group_select reads the groups' maxima four at a time
static_assert(alignof(SampleShared) >= 16 && offsetof(SampleShared, hist) % 16 == 0, "hist is read by 16-byte loads");

// Threshold selection of the k largest keys of the elements `scan` walks (224 < k <= 1024, at least
// 4096 elements, every thread sees some and no two threads see the same): pass 1 takes every
// thread's largest value; the threads form n_g >= k groups (n_g the next power of two), and the
// smallest of the n_g group maxima, L, is a lower bound of the k-th largest value (n_g >= k
// distinct elements are >= L); M is the overall maximum.  Pass 2 looks only at elements >= L (a
// fraction of a percent of a row for k = 50): they are kept in an LDS list and counted in a
// histogram over (M - value) in order-preserving integer units, 2047 bins.  The bin B in which the
// count reaches k bounds the top k from below, the list is cut down to bins <= B (k plus a few).
// Returns the number of keys left in sh.sel (>= k, the top k among them), or 0 if the list or the
// cut overflowed (many equal values).  Division by T > 0, correctly rounded, never reverses an
// order, so maxima are taken on the values themselves and only candidates are divided.
template <typename Scan>
__device__ inline int threshold_select(Scan scan, float temperature, int k, SampleShared &sh) {
  const int tid = threadIdx.x;
  unsigned int mine = 0;
  scan([&](bool ok, float z, int) {
    if (ok) mine = max(mine, float_order_bits(z));
  });
  const unsigned int M = float_order_bits(
      __fdiv_rn(float_from_order_bits(block_reduce_u32(mine, true, sh.scratch32)), temperature));
  int n_g = 1;
  while (n_g < k) n_g <<= 1;
  sh.hist[tid] = mine;
  __syncthreads();
  unsigned int gmax = 0xFFFFFFFFu;
  if (tid < n_g) {
    const int per = 1024 / n_g;
    gmax = 0;
    for (int i = 0; i < per; ++i) gmax = max(gmax, sh.hist[tid * per + i]);
  }
  const float z_l = float_from_order_bits(block_reduce_u32(gmax, false, sh.scratch32));
  const unsigned int L = float_order_bits(__fdiv_rn(z_l, temperature));
  // a value below z_low cannot reach L after the division (its quotient is smaller by dozens of
  // ulps): a cheap test that spares the division for nearly every element
  const float z_low = z_l - fabsf(z_l) * 3.8147e-06f - 1e-30f;
  const unsigned int range = M - L;
  int shift = 0;
  while ((range >> shift) > 2046u) ++shift;
  for (int i = tid; i < 2048; i += 1024) sh.hist[i] = 0;
  if (tid == 0) { sh.s_cnt = 0; sh.s_cnt2 = 0; }
  __syncthreads();
  scan([&](bool ok, float z, int v) {
    const bool maybe = ok && z >= z_low;
    if (__ballot(maybe) == 0) return;             // wave-uniform: most batches hold no candidate
    const unsigned int ob = maybe ? float_order_bits(__fdiv_rn(z, temperature)) : 0u;
    const bool keep = maybe && ob >= L;
    const unsigned int slot = wave_claim(keep, &sh.s_cnt);
    if (keep) {
      atomicAdd(&sh.hist[(M - ob) >> shift], 1u);
      if (slot < MC_MAX_TOP_K) sh.sel[slot] = ((unsigned long long)ob << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)v);
    }
  });
  __syncthreads();
  const unsigned int n_cand = sh.s_cnt;
  if (tid < 64) {
    // lane L owns bins [32L, 32L + 32): find the bin in which the running count reaches k
    unsigned int own = 0;
    for (int i = 0; i < 32; ++i) own += sh.hist[32 * tid + i];
    unsigned int incl = own;
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned int t = __shfl_up(incl, o, 64);
      if (tid >= o) incl += t;
    }
    const unsigned int excl = incl - own;
    if (excl < (unsigned int)k && incl >= (unsigned int)k) {   // exactly one lane (count >= n_g >= k)
      unsigned int run = excl;
      for (int i = 0; i < 32; ++i) {
        run += sh.hist[32 * tid + i];
        if (run >= (unsigned int)k) {
          sh.s_bin = (unsigned int)(32 * tid + i);
          sh.s_above = run;                          // elements in bins <= s_bin
          break;
        }
      }
    }
  }
  __syncthreads();
  const unsigned int B = sh.s_bin, G = sh.s_above;
  int n_sel = 0;
  if (n_cand <= MC_MAX_TOP_K && G <= MC_MAX_TOP_K) {
    // cut the list down to bins <= B: read everything, then write the survivors back
    unsigned long long mykeys[MC_MAX_TOP_K / 1024];
#pragma unroll
    for (int j = 0; j < MC_MAX_TOP_K / 1024; ++j) {
      const unsigned int i = tid + 1024 * j;
      mykeys[j] = (i < n_cand) ? sh.sel[i] : 0ull;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < MC_MAX_TOP_K / 1024; ++j) {
      const unsigned int i = tid + 1024 * j;
      const bool keep = i < n_cand && ((M - (unsigned int)(mykeys[j] >> 32)) >> shift) <= B;
      const unsigned int slot = wave_claim(keep, &sh.s_cnt2);
      if (keep) sh.sel[slot] = mykeys[j];
    }
    __syncthreads();
    n_sel = (int)sh.s_cnt2;                           // == G
  }
  __syncthreads();
  return n_sel;
}

// Radix selection of the k largest keys of a row: up to six passes on the 64-bit key (11/11/10-bit
// digits), exact for any input and any k.  Leaves exactly k keys in sh.sel.
__device__ inline int radix_select(const float *row, int V, float temperature, int k, SampleShared &sh) {
  const int tid = threadIdx.x;
  unsigned long long prefix = 0, pmask = 0;
  unsigned int need = (unsigned int)k;
  const int shifts[6] = {53, 42, 32, 21, 10, 0};
  const int nbits[6] = {11, 11, 10, 11, 11, 10};
  for (int pass = 0; pass < 6; ++pass) {
    const int shift = shifts[pass];
    const unsigned int bmask = (1u << nbits[pass]) - 1u;
    for (int i = tid; i < 2048; i += 1024) sh.hist[i] = 0;
    __syncthreads();
    for (int v = tid; v < V; v += 1024) {
      const unsigned long long key = sample_key(__fdiv_rn(row[v], temperature), v);
      if ((key & pmask) == prefix) atomicAdd(&sh.hist[(unsigned int)(key >> shift) & bmask], 1u);
    }
    __syncthreads();
    if (tid < 64) {
      // lane L owns bins [2048-32(L+1), 2048-32L): walk from the top bin down
      const int hi = 2048 - 32 * tid;
      unsigned int mine = 0;
      for (int i = 1; i <= 32; ++i) mine += sh.hist[hi - i];
      unsigned int incl = mine;                   // inclusive scan over lanes 0..L
      for (int o = 1; o < 64; o <<= 1) {
        const unsigned int t = __shfl_up(incl, o, 64);
        if (tid >= o) incl += t;
      }
      const unsigned int excl = incl - mine;
      if (excl < need && incl >= need) {          // exactly one lane
        unsigned int above = excl;
        for (int i = 1; i <= 32; ++i) {
          const unsigned int c = sh.hist[hi - i];
          if (above + c >= need) {
            sh.s_bin = (unsigned int)(hi - i);
            sh.s_above = above;
            sh.s_cnt = c;
            break;
          }
          above += c;
        }
      }
    }
    __syncthreads();
    prefix |= (unsigned long long)sh.s_bin << shift;
    pmask |= (unsigned long long)bmask << shift;
    need -= sh.s_above;
    const bool done = (sh.s_cnt == need);            // the whole bin belongs to the top k
    __syncthreads();
    if (done) break;
  }
  // every key >= prefix (low bits zero) is selected: exactly k of them
  if (tid == 0) sh.s_cnt = 0;
  __syncthreads();
  for (int v = tid; v < V; v += 1024) {
    const unsigned long long key = sample_key(__fdiv_rn(row[v], temperature), v);
    if (key >= prefix) {
      const unsigned int slot = atomicAdd(&sh.s_cnt, 1u);
      if (slot < MC_MAX_TOP_K) sh.sel[slot] = key;
    }
  }
  return k;
}

// Bitonic sort of sh.sel[0 .. n_sel), descending: the first k entries are the top k in order.
__device__ inline void sort_selected(int n_sel, SampleShared &sh) {
  const int tid = threadIdx.x;
  int kp = 1;
  while (kp < n_sel) kp <<= 1;
  __syncthreads();
  for (int i = n_sel + tid; i < kp; i += 1024) sh.sel[i] = 0ull;
  __syncthreads();
  for (int size = 2; size <= kp; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = tid; i < kp; i += 1024) {
        const int j = i ^ stride;
        if (j > i) {
          const unsigned long long x = sh.sel[i], y = sh.sel[j];
          const bool desc = ((i & size) == 0);
          if ((x < y) == desc) { sh.sel[i] = y; sh.sel[j] = x; }
        }
      }
      __syncthreads();
    }
  }
}

// An undivided value and its id (kEndsGroup: the last entry of a group's top list) for group_select
constexpr uint32_t kEndsGroup = 0x80000000u;
__device__ inline void list_candidate(SampleShared &sh, unsigned int at, float z, uint32_t id) {
  if (at < MC_MAX_TOP_K) sh.sel[at] = ((unsigned long long)__float_as_uint(z) << 32) | id;
}

// Two walks over one row for group_select: the largest value of this thread's elements, then a list
// of all elements >= z_low.  Rows of up to 4 * NB * 1024 values (32768) stay in registers between the two;
// longer ones are read again, from L2.  Rows that are not 16-byte aligned go element by element.
struct RowScan {
  static constexpr int NB = 8;
  const float *row;
  int V, V4;
  float4 z[NB];
  __device__ RowScan(const float *r, int v) : row(r), V(v), V4((((uintptr_t)r & 15) == 0) ? v / 4 : 0) {}
  __device__ inline void load(int g0) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int g = g0 + j * 1024 + (int)threadIdx.x;
      z[j] = (g < V4) ? ((const float4 *)row)[g] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    }
  }
  __device__ inline float largest() {
    float m = -INFINITY;
    for (int g0 = 0; g0 < V4; g0 += NB * 1024) {
      load(g0);
#pragma unroll
      for (int j = 0; j < NB; ++j) m = fmaxf(fmaxf(fmaxf(m, z[j].x), fmaxf(z[j].y, z[j].z)), z[j].w);
    }
    for (int v = 4 * V4 + (int)threadIdx.x; v < V; v += 1024) m = fmaxf(m, row[v]);
    return m;
  }
  __device__ inline void above(float z_low, SampleShared &sh) {
    for (int g0 = 0; g0 < V4; g0 += NB * 1024) {
      if (V4 > NB * 1024) load(g0);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int g = g0 + j * 1024 + (int)threadIdx.x;
        if (!(fmaxf(fmaxf(z[j].x, z[j].y), fmaxf(z[j].z, z[j].w)) >= z_low) || g >= V4) continue;
        const bool wx = z[j].x >= z_low, wy = z[j].y >= z_low, wz = z[j].z >= z_low, ww = z[j].w >= z_low;
        unsigned int at = atomicAdd(&sh.s_cnt, (unsigned int)(wx + wy + wz + ww));
        if (wx) list_candidate(sh, at++, z[j].x, 4 * g);
        if (wy) list_candidate(sh, at++, z[j].y, 4 * g + 1);
        if (wz) list_candidate(sh, at++, z[j].z, 4 * g + 2);
        if (ww) list_candidate(sh, at, z[j].w, 4 * g + 3);
      }
    }
    for (int v = 4 * V4 + (int)threadIdx.x; v < V; v += 1024) {
      const float x = row[v];
      if (x >= z_low) list_candidate(sh, atomicAdd(&sh.s_cnt, 1u), x, v);
    }
  }
};

// The same over the (value bits, id) pairs the LM head leaves beside the logits, four per group of
// 64 ids: lists of up to 2 * NB * 1024 pairs (a vocabulary of 262144) stay in registers.
struct ListScan {
  static constexpr int NB = 8;
  const uint4 *l4;
  int n2;
  uint4 e[NB];
  __device__ ListScan(const uint2 *list, int n) : l4((const uint4 *)list), n2(n / 2) {}
  __device__ inline void load(int g0) {
    const uint32_t none = __float_as_uint(-INFINITY);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int g = g0 + j * 1024 + (int)threadIdx.x;
      e[j] = (g < n2) ? l4[g] : make_uint4(none, 0u, none, 0u);
    }
  }
  __device__ inline float largest() {
    float m = -INFINITY;
    for (int g0 = 0; g0 < n2; g0 += NB * 1024) {
      load(g0);
#pragma unroll
      for (int j = 0; j < NB; ++j) m = fmaxf(fmaxf(m, __uint_as_float(e[j].x)), __uint_as_float(e[j].z));
    }
    return m;
  }
  __device__ inline void above(float z_low, SampleShared &sh) {
    for (int g0 = 0; g0 < n2; g0 += NB * 1024) {
      if (n2 > NB * 1024) load(g0);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int g = g0 + j * 1024 + (int)threadIdx.x;
        const float x = __uint_as_float(e[j].x), y = __uint_as_float(e[j].z);
        const bool wx = x >= z_low, wy = y >= z_low;
        if (!(wx || wy) || g >= n2) continue;
        unsigned int at = atomicAdd(&sh.s_cnt, (unsigned int)(wx + wy));
        if (wx) list_candidate(sh, at++, x, e[j].y);
        if (wy) list_candidate(sh, at, y, e[j].w | ((g & 1) ? kEndsGroup : 0u));
      }
    }
  }
};

// Cuts a list of n keys (256 <= n <= MC_MAX_TOP_K) down to those that can be among the k <= 224 largest: the first
// step of group_select once more, on the list, where the k-th largest of the maxima of 256 groups bounds the
// k-th largest key from below.  Rows whose largest values lie together (in neighbouring threads, so in few
// groups) leave up to 4096 keys here, and sorting them is what that would cost: top 50 of 8 x 32000 rising
// values 36 us sorted, 12.7 cut; top 200 of 64 x 32000 random ones, 389 keys on average, 23.7 either way.
// Returns how many are left in sh.sel.
__device__ inline int cut_list(int n, int k, SampleShared &sh) {
  const int tid = threadIdx.x;
  constexpr int PER = MC_MAX_TOP_K / 1024;
  unsigned long long mine[PER];
  unsigned int top = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    mine[j] = tid + 1024 * j < n ? sh.sel[tid + 1024 * j] : 0ull;
    top = max(top, (unsigned int)(mine[j] >> 32));
  }
  sh.hist[tid] = top;
  if (tid == 0) { sh.s_cnt = 0; sh.s_bin = 0xFFFFFFFFu; }
  __syncthreads();
  // neighbours in the list, which may be neighbours in the row, fall into different groups
  if (tid < 256) sh.hist[1024 + tid] = max(max(sh.hist[tid], sh.hist[tid + 256]), max(sh.hist[tid + 512], sh.hist[tid + 768]));
  __syncthreads();
  const unsigned int v = sh.hist[1024 + (tid >> 2)];
  int gt = 0;
#pragma unroll 4
  for (int j = 0; j < 16; ++j) {
    const uint4 u = *(const uint4 *)&sh.hist[1024 + (4 * j + (tid & 3)) * 4];
    gt += (u.x > v) + (u.y > v) + (u.z > v) + (u.w > v);
  }
  gt += __shfl_xor(gt, 1, 64);
  gt += __shfl_xor(gt, 2, 64);
  if ((tid & 3) == 0 && gt < k) atomicMin(&sh.s_bin, v);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (mine[j] != 0 && (unsigned int)(mine[j] >> 32) >= sh.s_bin) sh.sel[atomicAdd(&sh.s_cnt, 1u)] = mine[j];
  __syncthreads();
  return (int)sh.s_cnt;
}

// Selection of the k <= kGroupSelectMaxK largest keys, in order: the threads form n_g = 128 groups of
// eight (k <= 64) or 256 of four, and the k-th largest of the groups' maxima, L, is a lower bound of
// the k-th largest value (k distinct elements are >= L), a tight one: with the largest values spread at
// random n_g ln(n_g / (n_g - k)) elements of a row are >= L, 63 for k = 50 and 389 for k = 200.  Those go to a
// list in LDS (more than 384 are cut down by cut_list), and every one's rank is the number of larger keys in it
// (keys are distinct, the id is part of them), counted by 16 lanes per key.  Five barriers, and one pass over
// memory for rows of up to 32768 values; longer ones are read a second time.  Returns
// where the k sorted keys lie, or nullptr where L is no bound (fewer than k groups with a
// value) or the list overflowed (thousands of equal values).  NaN is passed over, as by the
// threshold selection.
// last_ob: largest order bits, after the division, of this thread's listed elements that end a
// group's list (0: none).
constexpr int kGroupSelectMaxK = 224, kRankMax = 384;
template <typename Scan>
__device__ inline const unsigned long long *group_select(Scan scan, float temperature, int k, SampleShared &sh,
                                                         unsigned int &last_ob) {
  const int tid = threadIdx.x;
  float m = scan.largest();
  const int gs = k <= 64 ? 3 : 2, sub = tid & ((1 << gs) - 1);   // log2 of a group's threads; index in the group
  m = fmaxf(m, __shfl_xor(m, 1, 64));
  m = fmaxf(m, __shfl_xor(m, 2, 64));
  if (gs == 3) m = fmaxf(m, __shfl_xor(m, 4, 64));
  if (sub == 0) sh.hist[tid >> gs] = float_order_bits(m);
  if (tid == 0) { sh.s_cnt = 0; sh.s_bin = 0xFFFFFFFFu; }
  __syncthreads();
  {
    const unsigned int v = sh.hist[tid >> gs];     // a group's threads count the maxima above its own
    int gt = 0;
#pragma unroll 4
    for (int j = 0; j < (gs == 3 ? 4 : 16); ++j) {
      const uint4 u = *(const uint4 *)&sh.hist[((j << gs) + sub) * 4];
      gt += (u.x > v) + (u.y > v) + (u.z > v) + (u.w > v);
    }
    gt += __shfl_xor(gt, 1, 64);
    gt += __shfl_xor(gt, 2, 64);
    if (gs == 3) gt += __shfl_xor(gt, 4, 64);
    if (sub == 0 && gt < k) atomicMin(&sh.s_bin, v);
  }
  __syncthreads();
  const float z_l = float_from_order_bits(sh.s_bin);
  if (!(z_l > -INFINITY)) return nullptr;
  // a value below this cannot reach L after the division, as in threshold_select
  scan.above(z_l - fabsf(z_l) * 3.8147e-06f - 1e-30f, sh);
  __syncthreads();
  int n = (int)sh.s_cnt;
  if (n < k || n > MC_MAX_TOP_K) return nullptr;
  last_ob = 0;
  for (int i = tid; i < n; i += 1024) {            // listed values become keys
    const unsigned long long c = sh.sel[i];
    const uint32_t id = (uint32_t)c;
    const unsigned long long key = sample_key(__fdiv_rn(__uint_as_float((uint32_t)(c >> 32)), temperature), (int)(id & ~kEndsGroup));
    if (id & kEndsGroup) last_ob = max(last_ob, (unsigned int)(key >> 32));
    sh.sel[i] = key;
  }
  __syncthreads();
  if (n > kRankMax) n = cut_list(n, k, sh);
  if (n > kRankMax) {
    sort_selected(n, sh);
    return sh.sel;
  }
  unsigned long long *sorted = (unsigned long long *)sh.hist;   // the maxima are no longer read
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int i = i0 + (tid >> 4);
    const unsigned long long key = i < n ? sh.sel[i] : ~0ull;
    int ahead = 0;
    for (int j = tid & 15; j < n; j += 16) ahead += sh.sel[j] > key;
    for (int o = 1; o < 16; o <<= 1) ahead += __shfl_xor(ahead, o, 64);
    if ((tid & 15) == 0 && i < n && ahead < k) sorted[ahead] = key;
  }
  __syncthreads();
  return sorted;
}

// One block of 1024 threads per candidate: exact top-k of z / T under the order (value
// descending, id ascending), then the softmax and the cumulative walk, whose additions run left
// to right as the rule demands.
//
// Where the LM head left per-group top lists beside the logits (top != nullptr: for every group
// of 64 consecutive ids its kTopListLen largest (value, id) pairs in order) and k <= kTopListMaxK,
// the selection runs on those lists, 1 / 16 of a row.  The result is the row's top k provided
// no group's last listed entry reaches the k-th selected value after the division (then an
// unlisted element of that group could belong to the top k, or tie with its last member): that
// is checked, and such a row is selected from the whole row instead, so the ids are the rule's
// in every case.  Selection from a row: group_select for k <= 224, threshold selection for k <= 1024
// (two passes over the row), radix selection for the rest and where those two give up.  A launch has as
// many blocks as rows, a few of the 256 CUs, and what bounds it is one block's chain of launch, memory
// and LDS round trips and barriers, so the steps of that chain were taken out: a second pass over
// a short row, a histogram, a bitonic sort, two serial walks over LDS by one thread.  Top 50 of 8 x 32000:
// 25.6 -> 10.1 us, 4 x 4096: 20 -> 8.2 us, 32 x 128256 from lists: 24 -> 10 us, from whole rows (wall
// time) 39 -> 17 us; top 200 of 64 x 152064: 87 -> 37 us; arg max of 64 x 152064: 54 -> 16 us.
constexpr int kTopListLen = 4, kTopListMaxK = 64;
__global__ __launch_bounds__(1024) void sample_kernel(
    int V, const float *__restrict__ logits, size_t row_stride, const uint2 *__restrict__ top,
    size_t top_stride, int n_groups, float temperature, int top_k,
    const float *__restrict__ uniforms, RowWords host_uniforms, int32_t *__restrict__ out_tokens,
    int32_t *__restrict__ host_tokens, int32_t *__restrict__ out_topk) {
  __shared__ SampleShared sh;
  const int b = blockIdx.x, tid = threadIdx.x;
  const float *row = logits + (size_t)b * row_stride;
  const uint2 *list = top ? top + (size_t)b * top_stride : nullptr;

  if (temperature <= 0.f || top_k == 1) {
    unsigned long long best = 0;
    if (list) {                                    // the arg max is the best of the groups' first entries
      for (int g = tid; g < n_groups; g += 1024) {
        const uint2 e = list[(size_t)g * kTopListLen];
        const unsigned long long key = sample_key(__uint_as_float(e.x), (int)e.y);
        best = key > best ? key : best;
      }
    } else {
      // 16-byte loads, eight in flight, past the end the last vector again (the same keys); single loads for the
      // rest and for rows that are not 16-byte aligned, where scan_row's would go one at a time
      constexpr int NB = 8;
      const int V4 = (((uintptr_t)row & 15) == 0) ? V / 4 : 0;
      auto take = [&](float z, int v) {
        const unsigned long long key = sample_key(z, v);
        best = key > best ? key : best;
      };
      for (int g0 = 0; g0 < V4; g0 += NB * 1024) {
        float4 z[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j)
          if (g0 + j * 1024 < V4) z[j] = ((const float4 *)row)[min(g0 + j * 1024 + tid, V4 - 1)];
#pragma unroll
        for (int j = 0; j < NB; ++j)
          if (g0 + j * 1024 < V4) {
            const int v = 4 * min(g0 + j * 1024 + tid, V4 - 1);
            take(z[j].x, v);
            take(z[j].y, v + 1);
            take(z[j].z, v + 2);
            take(z[j].w, v + 3);
          }
      }
      for (int v = 4 * V4 + tid; v < V; v += 1024) take(row[v], v);
    }
    best = block_max_u64(best, sh.scratch64);
    if (tid == 0) {
      const int tok = (int)(0xFFFFFFFFu - (uint32_t)(best & 0xFFFFFFFFull));
      out_tokens[b] = tok;
      if (host_tokens) host_tokens[b] = tok;
      if (out_topk) out_topk[b] = tok;
    }
    return;
  }
  const int k = (top_k <= 0 || top_k >= V) ? V : top_k;
  const float u = uniforms ? uniforms[b] : __uint_as_float(host_uniforms.v[b]);
  const unsigned long long *sorted = nullptr;      // the top k keys in order, in LDS
  unsigned int last_ob = 0;

  if (list && k <= kTopListMaxK && n_groups * kTopListLen >= 4096) {
    sorted = group_select(ListScan(list, n_groups * kTopListLen), temperature, k, sh, last_ob);
    // conclusive only if every group's last listed entry stays below the k-th selected value
    // (an entry that did not reach the list is below it)
    if (sorted && __syncthreads_or(last_ob >= (unsigned int)(sorted[k - 1] >> 32))) sorted = nullptr;
  }
  if (!sorted && k <= kGroupSelectMaxK && V >= 4096) {
    __syncthreads();
    sorted = group_select(RowScan(row, V), temperature, k, sh, last_ob);
  }
  if (!sorted) {
    __syncthreads();
    int n_sel = 0;                                 // keys in sel[] (>= k; the top k are among them)
    if (k > kGroupSelectMaxK && k <= 1024 && V >= 4096)
      n_sel = threshold_select([&](auto f) { scan_row(row, V, f); }, temperature, k, sh);
    if (n_sel == 0) n_sel = radix_select(row, V, temperature, k, sh);
    sort_selected(n_sel, sh);
    sorted = sh.sel;
  }
  const float z0 = float_from_order_bits((uint32_t)(sorted[0] >> 32));
  if (out_topk)
    for (int i = tid; i < k; i += 1024)
      out_topk[(size_t)b * k + i] = (int)(0xFFFFFFFFu - (uint32_t)(sorted[i] & 0xFFFFFFFFull));
  auto weight = [&](int i) { return i < k ? expf(float_from_order_bits((uint32_t)(sorted[i] >> 32)) - z0) : 0.f; };
  if (k > 64)
    for (int i = tid; i < k; i += 1024) sh.ev[i] = weight(i);
  __syncthreads();
  if (tid >= 64) return;
  // One wave.  The running sum takes 64 weights at a time out of the lanes' registers, in order, and lane i
  // keeps its value after entry i (past the last entry 0 is added); the walk ends with the first 64 that hold
  // the token.  The total of more than 64 is summed from LDS first, which is quicker (top 2000 of a row of 128256:
  // 163 us; 184 with all of it out of the registers).
  float total = 0.f, run = 0.f;
  if (k > 64)
    for (int i = 0; i < k; ++i) total += sh.ev[i];
  int pick = k - 1;
  for (int i0 = 0; i0 < k; i0 += 64) {
    const int i = i0 + tid;
    const float e = k > 64 ? (i < k ? sh.ev[i] : 0.f) : weight(i);
    float after = 0.f;
#pragma unroll
    for (int j = 0; j < 64; ++j) {
      run += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(e), j));
      after = tid == j ? run : after;
    }
    if (k <= 64) total = run;
    const unsigned long long hit = __ballot(i < k && __fdiv_rn(after, total) > u);
    if (hit) {
      pick = i0 + __ffsll((long long)hit) - 1;
      break;
    }
  }
  if (tid == 0) {
    const int tok = (int)(0xFFFFFFFFu - (uint32_t)(sorted[pick] & 0xFFFFFFFFull));
    out_tokens[b] = tok;
    if (host_tokens) host_tokens[b] = tok;
  }
}

int launch_sample(hipStream_t st, int n_cands, int vocab, const float *logits, size_t row_stride,
                  float temperature, int top_k, const float *uniforms, int32_t *out_tokens,
                  int32_t *out_topk, const void *top_lists, size_t top_stride, int n_groups, const RowWords *host_uniforms, int32_t *host_tokens) {
  if (n_cands <= 0) return MC_OK;
  sample_kernel<<<n_cands, 1024, 0, st>>>(vocab, logits, row_stride, (const uint2 *)top_lists, top_stride, n_groups,
                                          temperature, top_k, host_uniforms ? nullptr : uniforms, host_uniforms ? *host_uniforms : RowWords{}, out_tokens,
                                          host_tokens, out_topk);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

// ------------------------------------------------------------------ reward scoring
// log-softmax over the whole vocabulary read at the reward tokens (sums kept in double)
__global__ __launch_bounds__(1024) void reward_logprob_kernel(
    int V, const float *__restrict__ logits, const int32_t *__restrict__ ids, int R,
    float *__restrict__ out_lp) {
  __shared__ float scr_f[16];
  __shared__ double scr_d[16];
  const float *row = logits + (size_t)blockIdx.x * V;
  float m = -INFINITY;
  for (int v = threadIdx.x; v < V; v += 1024) m = fmaxf(m, row[v]);
  m = block_max(m, scr_f);
  double s = 0.0;
  for (int v = threadIdx.x; v < V; v += 1024) s += exp((double)row[v] - (double)m);
  s = block_sum<double>(s, scr_d);
  const double lse = (double)m + log(s);
  for (int r = threadIdx.x; r < R; r += 1024)
    out_lp[(size_t)blockIdx.x * R + r] = (float)((double)row[ids[r]] - lse);
}

// score_b = sum_r w_r softmax_r(lp_r / Ts); rank by (score descending, index ascending)
__global__ __launch_bounds__(1024) void score_rank_kernel(
    int B, int R, const float *__restrict__ lp, const float *__restrict__ w, float ts,
    float *__restrict__ scores, int32_t *__restrict__ rank) {
  extern __shared__ float sc[];
  for (int b = threadIdx.x; b < B; b += 1024) {
    const float *p = lp + (size_t)b * R;
    double mx = -1e300;
    for (int r = 0; r < R; ++r) mx = fmax(mx, (double)p[r] / (double)ts);
    double den = 0.0, num = 0.0;
    for (int r = 0; r < R; ++r) {
      const double e = exp((double)p[r] / (double)ts - mx);
      den += e;
      num += e * (double)w[r];
    }
    const float v = (float)(num / den);
    sc[b] = v;
    if (scores) scores[b] = v;
  }
  __syncthreads();
  if (rank)
    for (int b = threadIdx.x; b < B; b += 1024) {
      const float mine = sc[b];
      int ahead = 0;
      for (int c = 0; c < B; ++c) ahead += (sc[c] > mine) || (sc[c] == mine && c < b);
      rank[ahead] = b;
    }
}

int launch_reward_score(hipStream_t st, int n_cands, int vocab, const float *logits,
                        const int32_t *reward_ids, const float *reward_values, int n_reward,
                        float score_temperature, float *out_logprobs, float *out_scores,
                        int32_t *out_rank) {
  if (n_cands <= 0) return MC_OK;
  reward_logprob_kernel<<<n_cands, 1024, 0, st>>>(vocab, logits, reward_ids, n_reward,
                                                  out_logprobs);
  MC_HIP(hipGetLastError());
  score_rank_kernel<<<1, 1024, (size_t)n_cands * sizeof(float), st>>>(
      n_cands, n_reward, out_logprobs, reward_values, score_temperature, out_scores, out_rank);
  MC_HIP(hipGetLastError());
  return MC_OK;
}

}  // namespace mc
