// Row-wise and integer kernels of the tree-verify step, plus dtype-generic reference-grade
// products and attention used by the fp32 model path (the bf16 hot path uses the MFMA kernels).
#include "ht_common.h"
#include <type_traits>

namespace ht {

#define HT_DISPATCH_DTYPE(dtype, ...)                       \
  if ((dtype) == 0) { typedef float T; __VA_ARGS__ }        \
  else { typedef bf16_t T; __VA_ARGS__ }

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ inline float wave_max_dpp(float x) {
  // quads, half rows and rows by data-parallel-primitive moves, then rows and halves of the wave by lane swaps
  x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xf, 0xf, true)));    // lanes 1 0 3 2
  x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xf, 0xf, true)));    // lanes 2 3 0 1
  x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xf, 0xf, true)));   // half row mirrored
  x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xf, 0xf, true)));   // row mirrored
  unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  u = __float_as_uint(x);
  auto r2 = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r2[0]), __uint_as_float(r2[1]));
}
__device__ inline int wave_min_dpp(int x) {
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true));
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, true));
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true));
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, true));
  auto r = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
  x = min((int)r[0], (int)r[1]);
  auto r2 = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
  return min((int)r2[0], (int)r2[1]);
}

// block-wide sum for 256-thread blocks; `red` is __shared__ float[4]
__device__ inline float block_sum_256(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}
__device__ inline float block_max_256(float v, float* red) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

__global__ void copy_rows_kernel(const float* __restrict__ src, float* __restrict__ dst, size_t count) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = src[i];
}
hipError_t launch_load_rows(const float* src, float* x, int M, int d, hipStream_t s) {
  size_t count = (size_t)M * d;
  hipLaunchKernelGGL(copy_rows_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, src, x, count);
  return hipGetLastError();
}

template <typename T>
__global__ void convert_to_f32_kernel(const T* __restrict__ src, float* __restrict__ dst, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = Conv<T>::load(src + i);
}
hipError_t launch_convert_to_f32(int dtype, const void* src, float* dst, int n, hipStream_t s) {
  HT_DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(convert_to_f32_kernel<T>, dim3((n + 255) / 256), dim3(256), 0, s,
                                              (const T*)src, dst, n);)
  return hipGetLastError();
}

// dst[i] = bf16(src[i]), four elements per thread (count a multiple of 4)
__global__ void convert_to_bf16_kernel(const float* __restrict__ src, bf16_t* __restrict__ dst, size_t quads) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= quads) return;
  const float4 v = *(const float4*)(src + i * 4);
  *(uint2*)(dst + i * 4) = pack4_bf16(v.x, v.y, v.z, v.w);
}
hipError_t launch_convert_to_bf16(const float* src, void* dst, size_t count, hipStream_t s) {
  if (count % 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(convert_to_bf16_kernel, dim3((unsigned)((count / 4 + 255) / 256)), dim3(256), 0, s, src, (bf16_t*)dst,
                     count / 4);
  return hipGetLastError();
}

// Two passes over L2-sized data: bound by the latency of one round trip, so all splits of an element are requested before
// the first is added, 16 bytes a lane where `out` is aligned (33 rows of 5120 in six splits: 4.3 us with 4-byte loads one
// after the other), and no more than there are (128 rows of 5120 in two splits: 2.9 us with eight loads whatever the number).
template <typename V, int NS>
__global__ __launch_bounds__(256) void reduce_splits_kernel(const V* __restrict__ part, size_t stride, V* __restrict__ out) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= stride) return;
  V p[NS];
#pragma unroll
  for (int sp = 0; sp < NS; ++sp) p[sp] = part[sp * stride + i];
  V v = p[0];
#pragma unroll
  for (int sp = 1; sp < NS; ++sp) v += p[sp];
  out[i] = v;
}
template <typename V>
hipError_t launch_reduce_as(const float* part, int nsplit, size_t stride, float* out, hipStream_t s) {
  stride = stride * sizeof(float) / sizeof(V);
#define HT_REDUCE(NS)                                                                                                           \
  case NS:                                                                                                                      \
    hipLaunchKernelGGL((reduce_splits_kernel<V, NS>), dim3((unsigned)((stride + 255) / 256)), dim3(256), 0, s, (const V*)part,  \
                       stride, (V*)out);                                                                                        \
    break;
  switch (nsplit) {
    HT_REDUCE(1) HT_REDUCE(2) HT_REDUCE(3) HT_REDUCE(4) HT_REDUCE(5) HT_REDUCE(6) HT_REDUCE(7) HT_REDUCE(8)
    default: return hipErrorInvalidValue;
  }
#undef HT_REDUCE
  return hipGetLastError();
}
hipError_t launch_reduce_splits(const float* part, int nsplit, size_t stride, float* out, hipStream_t s) {
  typedef float float4v __attribute__((ext_vector_type(4)));
  const bool vec = stride % 4 == 0 && !((uintptr_t)out & 15) && !((uintptr_t)part & 15);
  return vec ? launch_reduce_as<float4v>(part, nsplit, stride, out, s) : launch_reduce_as<float>(part, nsplit, stride, out, s);
}

// ------------------------------------------------------------------------------------------------ residual + RMSNorm
// x[m] += sum over split-K partials of the previous projection (fixed order: deterministic), the
// updated residual is optionally saved (layer-t hidden states), then u[m] = x[m] * rsqrt(mean(x^2)+eps) * gain.
// One block of NT threads per row, four consecutive columns per thread and pass, every load of a pass
// issued before the first add so a row costs one memory round trip.
__device__ inline float block_sum_any(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = 0.f;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;
}

template <int NS>
__global__ void add_norm_kernel(float* __restrict__ x, const float* __restrict__ part, size_t part_stride,
                                const bf16_t* __restrict__ gain, bf16_t* __restrict__ u, float* __restrict__ save_h, int d,
                                float eps) {
  __shared__ float red[16];
  const int m = blockIdx.x;
  float* xr = x + (size_t)m * d;
  const float* pr = part + (size_t)m * d;
  float ss = 0.f;
  constexpr int MAXP = 4;                       // d <= MAXP * 4 * blockDim.x (checked by the launcher)
  float4 keep[MAXP];
#pragma unroll
  for (int p = 0; p < MAXP; ++p) {
    const int c = (p * blockDim.x + threadIdx.x) * 4;
    if (c < d) {
      float4 v = *(const float4*)(xr + c);
      float4 pv[NS > 0 ? NS : 1];
#pragma unroll
      for (int sp = 0; sp < NS; ++sp) pv[sp] = *(const float4*)(pr + sp * part_stride + c);
#pragma unroll
      for (int sp = 0; sp < NS; ++sp) { v.x += pv[sp].x; v.y += pv[sp].y; v.z += pv[sp].z; v.w += pv[sp].w; }
      if (NS) *(float4*)(xr + c) = v;
      if (save_h) *(float4*)(save_h + (size_t)m * d + c) = v;
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
      keep[p] = v;
    }
  }
  ss = block_sum_any(ss, red);
  const float scale = 1.0f / sqrtf(ss / (float)d + eps);
  if (u) {
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
      const int c = (p * blockDim.x + threadIdx.x) * 4;
      if (c < d) {
        const float4 v = keep[p];
        bf16_t* dst = u + (size_t)m * d + c;
        Conv<bf16_t>::store(dst + 0, v.x * scale * Conv<bf16_t>::load(gain + c + 0));
        Conv<bf16_t>::store(dst + 1, v.y * scale * Conv<bf16_t>::load(gain + c + 1));
        Conv<bf16_t>::store(dst + 2, v.z * scale * Conv<bf16_t>::load(gain + c + 2));
        Conv<bf16_t>::store(dst + 3, v.w * scale * Conv<bf16_t>::load(gain + c + 3));
      }
    }
  }
}
// kNormParts blocks per row: block (m, q) owns columns q dq .. (q + 1) dq - 1, dq = d / kNormParts.
template <int NS>
__global__ void add_norm_parts_kernel(float* __restrict__ x, const float* __restrict__ part, size_t part_stride,
                                      const bf16_t* __restrict__ gain, bf16_t* __restrict__ u,
                                      float* __restrict__ save_h, float* __restrict__ ss_out, int d) {
  __shared__ float red[16];
  const int m = blockIdx.x, dq = d / kNormParts, c0 = blockIdx.y * dq;
  float* xr = x + (size_t)m * d;
  const float* pr = part + (size_t)m * d;
  float ss = 0.f;
  constexpr int MAXP = 4;                       // dq <= MAXP * 4 * blockDim.x (checked by the launcher)
#pragma unroll
  for (int p = 0; p < MAXP; ++p) {
    const int cl = (p * blockDim.x + threadIdx.x) * 4;
    if (cl < dq) {
      const int c = c0 + cl;
      float4 v = *(const float4*)(xr + c);
      float4 pv[NS > 0 ? NS : 1];
#pragma unroll
      for (int sp = 0; sp < NS; ++sp) pv[sp] = *(const float4*)(pr + sp * part_stride + c);
#pragma unroll
      for (int sp = 0; sp < NS; ++sp) { v.x += pv[sp].x; v.y += pv[sp].y; v.z += pv[sp].z; v.w += pv[sp].w; }
      if (NS) *(float4*)(xr + c) = v;
      if (save_h) *(float4*)(save_h + (size_t)m * d + c) = v;
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
      if (u) {
        const uint2 g4 = *(const uint2*)(gain + c);
        *(uint2*)(u + (size_t)m * d + c) =
            pack4_bf16(v.x * __uint_as_float(g4.x << 16), v.y * __uint_as_float(g4.x & 0xffff0000u),
                       v.z * __uint_as_float(g4.y << 16), v.w * __uint_as_float(g4.y & 0xffff0000u));
      }
    }
  }
  ss = block_sum_any(ss, red);
  if (threadIdx.x == 0 && ss_out) ss_out[(size_t)m * kNormParts + blockIdx.y] = ss;
}
hipError_t launch_add_norm_parts(float* x, const float* part, int nsplit, size_t part_stride, const void* gain, void* u,
                                 float* save_h, float* ss, int M, int d, hipStream_t s) {
  if (d % (4 * kNormParts) || nsplit < 0 || nsplit > kMaxSplitK) return hipErrorInvalidValue;
  const int dq = d / kNormParts;
  int nt = 64;
  while (nt < 1024 && nt * 4 < dq) nt *= 2;
  if (dq > 16 * nt) return hipErrorInvalidValue;
#define HT_ADD_NORM_PARTS(NS)                                                                                      \
  case NS:                                                                                                         \
    hipLaunchKernelGGL((add_norm_parts_kernel<NS>), dim3(M, kNormParts), dim3(nt), 0, s, x, part, part_stride,     \
                       (const bf16_t*)gain, (bf16_t*)u, save_h, ss, d);                                            \
    break;
  switch (nsplit) {
    HT_ADD_NORM_PARTS(0) HT_ADD_NORM_PARTS(1) HT_ADD_NORM_PARTS(2) HT_ADD_NORM_PARTS(3) HT_ADD_NORM_PARTS(4)
    HT_ADD_NORM_PARTS(5) HT_ADD_NORM_PARTS(6) HT_ADD_NORM_PARTS(7) HT_ADD_NORM_PARTS(8)
  }
#undef HT_ADD_NORM_PARTS
  return hipGetLastError();
}

hipError_t launch_add_norm(float* x, const float* part, int nsplit, size_t part_stride, const void* gain,
                           void* u, float* save_h, int M, int d, float eps, hipStream_t s) {
  if (d % 4 || nsplit < 0 || nsplit > 1) return hipErrorInvalidValue;      // products that do not pack do not split K
  int nt = 64;
  while (nt < 1024 && nt * 4 < d) nt *= 2;
  if (d > 16 * nt) return hipErrorInvalidValue;
#define HT_ADD_NORM(NS)                                                                                         \
  case NS:                                                                                                      \
    hipLaunchKernelGGL((add_norm_kernel<NS>), dim3(M), dim3(nt), 0, s, x, part, part_stride, (const bf16_t*)gain, \
                       (bf16_t*)u, save_h, d, eps);                                                               \
    break;
  switch (nsplit) { HT_ADD_NORM(0) HT_ADD_NORM(1) }
#undef HT_ADD_NORM
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ rotary
// cs[m][j]: the factors of row m at position n + depth[m]
__global__ void rope_table_kernel(float2* __restrict__ cs, const int32_t* __restrict__ depth, int n, int half,
                                  double2 step, const int32_t* __restrict__ n_dev) {
  n = cache_len(n, n_dev);
  const int m = blockIdx.x;
  const int j = threadIdx.x;
  if (j >= half) return;
  cs[(size_t)m * half + j] = rope_factor(n + (depth ? depth[m] : m), rope_turns(j, step));   // no depth table: position n + m
}
hipError_t launch_rope_table(float* cs, const int32_t* depth, int n, int M, int hd, float base, hipStream_t s,
                             const int32_t* n_dev) {
  hipLaunchKernelGGL(rope_table_kernel, dim3(M), dim3(hd / 2), 0, s, (float2*)cs, depth, n, hd / 2, rope_step(base, hd / 2), n_dev);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ start of a pass
// The rows of a pass that are there when it starts, from the embedding table (by token) or from a buffer of fp32 rows, and
// the rotary factors of all rows it will end with, in one launch: workgroups 0 .. rows * shares - 1 copy, the others work
// out factors (they do not depend on one another; a launch of its own for each was two latencies in a row).  The tokens of a
// tree are put together here too (a launch, or a copy of the caller's, in front of this one took some 3 us), and with
// norm.gain the rows are normalised for the first block, kNormParts workgroups to a row as add_norm_parts_kernel does it: the
// launch behind this one that did it took 2 to 3 us (a step of four 7B-wide blocks 528 -> 526, of 70B-wide ones 887 -> 884).
template <typename T>
__global__ __launch_bounds__(1024) void start_pass_kernel(const T* __restrict__ emb, TokenSource tokens,
                                                         const float* __restrict__ rows_in, float* __restrict__ x, int rows,
                                                         int shares, int d, float2* __restrict__ cs, const int32_t* __restrict__ depth,
                                                         int n, int cs_rows, int half, double2 step, const int32_t* __restrict__ n_dev,
                                                         FirstNorm norm) {
  const int wg = blockIdx.x;
  if (wg < rows * shares) {
    const int m = wg / shares, part = wg % shares;          // part: which share of the row's columns
    const T* row = nullptr;
    if (!rows_in) {
      const int tok = !tokens.cand ? tokens.tok[m]
                      : m == 0     ? tokens.st->root
                                   : tokens.cand[(tokens.depth[m] - 1) * kMaxTopK + tokens.rank[m]];
      if (tokens.keep && part == 0 && threadIdx.x == 0) tokens.keep[m] = tok;
      row = emb + (size_t)tok * d;
    }
    if constexpr (sizeof(T) == 2) {
      if (norm.gain) {                                        // uniform; shares == kNormParts
        __shared__ float red[16];
        const int dq = d / kNormParts;
        float ss = 0.f;
        for (int c = part * dq + threadIdx.x * 4; c < (part + 1) * dq; c += blockDim.x * 4) {
          float4 v;
          if (row) {
            const uint2 r = *(const uint2*)(row + c);
            v = make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u), __uint_as_float(r.y << 16),
                            __uint_as_float(r.y & 0xffff0000u));
          } else {
            v = *(const float4*)(rows_in + (size_t)m * d + c);
          }
          *(float4*)(x + (size_t)m * d + c) = v;
          ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
          const uint2 g4 = *(const uint2*)(norm.gain + c);
          *(uint2*)(norm.u + (size_t)m * d + c) =
              pack4_bf16(v.x * __uint_as_float(g4.x << 16), v.y * __uint_as_float(g4.x & 0xffff0000u), v.z * __uint_as_float(g4.y << 16),
                         v.w * __uint_as_float(g4.y & 0xffff0000u));
        }
        ss = block_sum_any(ss, red);
        if (threadIdx.x == 0) norm.ss[(size_t)m * kNormParts + part] = ss;
        return;
      }
    }
    if (row) {
      for (int c = part * blockDim.x + threadIdx.x; c < d; c += shares * blockDim.x) x[(size_t)m * d + c] = Conv<T>::load(row + c);
    } else {
      for (int c = part * blockDim.x + threadIdx.x; c < d; c += shares * blockDim.x) x[(size_t)m * d + c] = rows_in[(size_t)m * d + c];
    }
    return;
  }
  n = cache_len(n, n_dev);
  const int i = (wg - rows * shares) * blockDim.x + threadIdx.x;
  if (i >= cs_rows * half) return;
  const int m = i / half, j = i % half;
  cs[i] = rope_factor(n + (depth ? depth[m] : m), rope_turns(j, step));
}
hipError_t launch_start_pass(int dtype, const void* emb, TokenSource tokens, const float* rows_in, float* x, int rows, int d,
                             float* cs, const int32_t* depth, int n, int cs_rows, int hd, float base, hipStream_t s,
                             const int32_t* n_dev, FirstNorm norm) {
  if (norm.gain && (dtype == 0 || d % (4 * kNormParts) || ((uintptr_t)emb & 7) || ((uintptr_t)norm.gain & 7))) return hipErrorInvalidValue;
  const int shares = norm.gain ? kNormParts : d >= 2048 ? 4 : 1;         // a few workgroups per row: a row is one dependent round trip per pass
  int nt = 256;
  while (norm.gain && nt < 1024 && nt * 4 * kNormParts < d) nt *= 2;     // the sum of squares in the order of the norm's own launch
  const int groups = rows * shares + (cs_rows * (hd / 2) + nt - 1) / nt;
  if (!groups) return hipSuccess;
  HT_DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(start_pass_kernel<T>, dim3(groups), dim3(nt), 0, s, (const T*)emb, tokens, rows_in, x,
                                              rows, shares, d, (float2*)cs, depth, n, cs_rows, hd / 2, rope_step(base, hd / 2), n_dev, norm);)
  return hipGetLastError();
}

// Rotates q and k of row m at its tree position and appends k, v to cache slot n+m.
// Layouts: q[M][Hq][hd]; K cache [cap][Hkv][hd]; V cache [Hkv][hd][cap] (key index contiguous).
// The inputs may come as `nsplit` split-K partial sums `split_stride` elements apart (added in index order).
template <typename T, typename TIN>
__global__ void rope_append_kernel(const TIN* __restrict__ q_in, int q_stride, const TIN* __restrict__ k_in,
                                   int k_stride, const TIN* __restrict__ v_in, int v_stride, int nsplit,
                                   size_t split_stride, const float2* __restrict__ cs, T* __restrict__ q,
                                   T* __restrict__ kc, T* __restrict__ vc, int n, int Hq, int Hkv, int hd, int cap,
                                   int paired, const int32_t* __restrict__ n_dev) {
  n = cache_len(n, n_dev);
  const int m = blockIdx.x, hh = blockIdx.y, j = threadIdx.x, half = hd / 2;
  if (j >= half) return;
  const float2 c = cs[(size_t)m * half + j];
  if (hh < Hq + Hkv) {
    const TIN* src = hh < Hq ? q_in + (size_t)m * q_stride + (size_t)hh * hd
                             : k_in + (size_t)m * k_stride + (size_t)(hh - Hq) * hd;
    // paired: the q and k columns of a head come in the packed projection's order, every run of 8 features
    // followed by the run of their rotary partners
    const int ja = paired ? 16 * (j >> 3) + (j & 7) : j, jb = paired ? ja + 8 : j + half;
    float a = Conv<TIN>::load(src + ja), b = Conv<TIN>::load(src + jb);
    for (int sp = 1; sp < nsplit; ++sp) {
      a += Conv<TIN>::load(src + sp * split_stride + ja);
      b += Conv<TIN>::load(src + sp * split_stride + jb);
    }
    const float ra = rope_low(a, b, c), rb = rope_high(a, b, c);
    T* dst = hh < Hq ? q + ((size_t)m * Hq + hh) * hd : kc + ((size_t)(n + m) * Hkv + (hh - Hq)) * hd;
    Conv<T>::store(dst + j, ra);
    Conv<T>::store(dst + j + half, rb);
  } else {
    const int h = hh - Hq - Hkv;
    const TIN* src = v_in + (size_t)m * v_stride + (size_t)h * hd;
    float a = Conv<TIN>::load(src + j), b = Conv<TIN>::load(src + j + half);
    for (int sp = 1; sp < nsplit; ++sp) {
      a += Conv<TIN>::load(src + sp * split_stride + j);
      b += Conv<TIN>::load(src + sp * split_stride + j + half);
    }
    Conv<T>::store(vc + ((size_t)h * hd + j) * cap + n + m, a);
    Conv<T>::store(vc + ((size_t)h * hd + j + half) * cap + n + m, b);
  }
}
// The same, four feature pairs per thread (hd % 8 == 0): 16-byte loads of the partial sums, 8-byte stores of q
// and k.  blockIdx.x = row, 256 threads cover 256 / (hd / 8) heads.
template <typename TIN> __device__ inline void load4(const TIN* p, float (&v)[4]);
template <> __device__ inline void load4<float>(const float* p, float (&v)[4]) {
  const float4 t = *(const float4*)p;
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
template <> __device__ inline void load4<bf16_t>(const bf16_t* p, float (&v)[4]) {
  const uint2 t = *(const uint2*)p;
  const bf16_t* h = (const bf16_t*)&t;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = bf16_to_float(h[i]);
}
template <typename T> __device__ inline void store4(T* p, const float (&v)[4]);
template <> __device__ inline void store4<float>(float* p, const float (&v)[4]) {
  *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
}
template <> __device__ inline void store4<bf16_t>(bf16_t* p, const float (&v)[4]) {
  *(uint2*)p = pack4_bf16(v[0], v[1], v[2], v[3]);
}

// One workgroup per (block of RB rows, head).  FRESH: it works the rotary factors of its rows out for itself, into LDS (one
// launch instead of two where a call has no other use for the table).  q and k heads: four feature pairs per thread and item, 16-byte loads,
// 8-byte stores.  v heads: the value cache is stored key-contiguous ([head][feature][slot]), so the rows go through LDS
// and every wavefront stores one feature of up to 64 consecutive rows at a time (a 2-byte store per row and feature
// straight from the row-major input touches a cache line of its own each).
template <typename T, typename TIN, bool FRESH = false>
__global__ __launch_bounds__(256) void rope_append_rows_kernel(
    const TIN* __restrict__ q_in, int q_stride, const TIN* __restrict__ k_in, int k_stride, const TIN* __restrict__ v_in,
    int v_stride, int nsplit, size_t split_stride, const float* __restrict__ cs, T* __restrict__ q, T* __restrict__ kc,
    T* __restrict__ vc, int n, int M, int RB, int Hq, int Hkv, int hd, int cap, int paired,
    const int32_t* __restrict__ n_dev, const int32_t* __restrict__ depth, double2 step) {
  extern __shared__ __attribute__((aligned(16))) unsigned char rows_lds[];
  n = cache_len(n, n_dev);
  const int m0 = blockIdx.x * RB, hh = blockIdx.y, half = hd / 2;
  const int rows = M - m0 < RB ? M - m0 : RB;
  float2* table = (float2*)rows_lds;                        // FRESH: [RB][half] (a v head's workgroup has no use for it)
  if (FRESH && hh < Hq + Hkv) {
    if (256 % half == 0) {                                  // a thread keeps its j
      const int j = threadIdx.x % half;
      const double2 turns = rope_turns(j, step);
      for (int r = threadIdx.x / half; r < rows; r += 256 / half) table[r * half + j] = rope_factor(n + depth[m0 + r], turns);
    } else {
      for (int i = threadIdx.x; i < rows * half; i += 256)
        table[i] = rope_factor(n + depth[m0 + i / half], rope_turns(i % half, step));
    }
    __syncthreads();
  }
  if (hh < Hq + Hkv) {
    const int per_row = half / 4;                          // items of four feature pairs
    for (int item = threadIdx.x; item < rows * per_row; item += 256) {
      const int m = m0 + item / per_row, j = (item % per_row) * 4;
      const TIN* src = hh < Hq ? q_in + (size_t)m * q_stride + (size_t)hh * hd
                               : k_in + (size_t)m * k_stride + (size_t)(hh - Hq) * hd;
      // paired: the q and k columns of a head come in the packed projection's order, every run of 8 features
      // followed by the run of their rotary partners
      const int ja = paired ? 16 * (j >> 3) + (j & 7) : j, jb = paired ? ja + 8 : j + half;
      float a[4], b[4];
      load4<TIN>(src + ja, a);
      load4<TIN>(src + jb, b);
      for (int sp = 1; sp < nsplit; ++sp) {
        float a2[4], b2[4];
        load4<TIN>(src + sp * split_stride + ja, a2);
        load4<TIN>(src + sp * split_stride + jb, b2);
#pragma unroll
        for (int i = 0; i < 4; ++i) { a[i] += a2[i]; b[i] += b2[i]; }
      }
      const float* cr = FRESH ? (const float*)(table + (m - m0) * half + j) : cs + ((size_t)m * half + j) * 2;
      const float4 c01 = *(const float4*)cr, c23 = *(const float4*)(cr + 4);
      const float2 c[4] = {make_float2(c01.x, c01.y), make_float2(c01.z, c01.w), make_float2(c23.x, c23.y), make_float2(c23.z, c23.w)};
      float ra[4], rb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { ra[i] = rope_low(a[i], b[i], c[i]); rb[i] = rope_high(a[i], b[i], c[i]); }
      T* dst = hh < Hq ? q + ((size_t)m * Hq + hh) * hd : kc + ((size_t)(n + m) * Hkv + (hh - Hq)) * hd;
      store4<T>(dst + j, ra);
      store4<T>(dst + j + half, rb);
    }
    return;
  }
  // v head: rows into LDS (row stride hd + 2 elements: the column reads below fall on consecutive banks)
  const int h = hh - Hq - Hkv, ldr = hd + 2;
  T* tile = (T*)rows_lds;
  const int per_row = hd / 4;
  for (int item = threadIdx.x; item < rows * per_row; item += 256) {
    const int r = item / per_row, j = (item % per_row) * 4;
    const TIN* src = v_in + (size_t)(m0 + r) * v_stride + (size_t)h * hd + j;
    float a[4];
    load4<TIN>(src, a);
    for (int sp = 1; sp < nsplit; ++sp) {
      float a2[4];
      load4<TIN>(src + sp * split_stride, a2);
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] += a2[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) Conv<T>::store(tile + r * ldr + j + i, a[i]);
  }
  __syncthreads();
  // RB is 16, 32 or 64: a wavefront stores 64 / RB features of RB consecutive rows at a time
  const int r = threadIdx.x % RB, per_pass = 256 / RB;
  for (int e = threadIdx.x / RB; e < hd; e += per_pass)
    if (r < rows) vc[((size_t)h * hd + e) * cap + n + m0 + r] = tile[r * ldr + e];
}

// rows per workgroup of rope_append_rows_kernel: 16 (measured: blocks of 64 rows leave too few workgroups for passes of
// 64 - 128 rows, which are latency bound)
constexpr int kRopeRows = 16;

hipError_t launch_rope_append(const float* qkv, int nsplit, const float* cs, void* q, void* kc, void* vc,
                              int n, int M, int Hq, int Hkv, int hd, int cap, bool paired, hipStream_t s,
                              const int32_t* n_dev) {
  const int stride = (Hq + 2 * Hkv) * hd;
  const float *k_in = qkv + (size_t)Hq * hd, *v_in = k_in + (size_t)Hkv * hd;
  bf16_t *qp = (bf16_t*)q, *kp = (bf16_t*)kc, *vp = (bf16_t*)vc;
  if (hd % 8 == 0) {
    const int RB = kRopeRows;
    hipLaunchKernelGGL((rope_append_rows_kernel<bf16_t, float>), dim3((M + RB - 1) / RB, Hq + 2 * Hkv), dim3(256),
                       (size_t)RB * (hd + 2) * sizeof(bf16_t), s, qkv, stride, k_in, stride, v_in, stride, nsplit,
                       (size_t)M * stride, cs, qp, kp, vp, n, M, RB, Hq, Hkv, hd, cap, paired ? 1 : 0, n_dev, nullptr, double2{});
    return hipGetLastError();
  }
  hipLaunchKernelGGL((rope_append_kernel<bf16_t, float>), dim3(M, Hq + 2 * Hkv), dim3(hd / 2), 0, s, qkv, stride, k_in, stride,
                     v_in, stride, nsplit, (size_t)M * stride, (const float2*)cs, qp, kp, vp, n, Hq, Hkv, hd, cap, paired ? 1 : 0,
                     n_dev);
  return hipGetLastError();
}
hipError_t launch_rope_append_split(int dtype, const void* q_in, const void* k_in, const void* v_in, const int32_t* depth,
                                    float base, float* cs, void* q, void* kc, void* vc, int n, int M, int Hq, int Hkv, int hd,
                                    int cap, hipStream_t s) {
  const int RB = kRopeRows, row_blocks = (M + RB - 1) / RB;
  const dim3 grid(row_blocks, Hq + 2 * Hkv);
#define HT_ROPE_ARGS                                                                                                        \
  (const T*)q_in, Hq * hd, (const T*)k_in, Hkv * hd, (const T*)v_in, Hkv * hd, 1, (size_t)0, cs, (T*)q, (T*)kc, (T*)vc, n, M, \
      RB, Hq, Hkv, hd, cap, 0, nullptr, depth, rope_step(base, hd / 2)
  const size_t values = (size_t)RB * (hd + 2) * (dtype == 0 ? 4 : 2), factors = (size_t)RB * (hd / 2) * sizeof(float2);
  // Factors worked out by every workgroup for itself as long as all of them together work out no more than a million (8 hd
  // each): a factor costs as many instructions every time, a launch for the table 1.5 us once.  Table and append in two
  // launches / in one, us, by workgroups.  As many k heads as q heads, heads of 128: 128 5.0 / 3.5, 512 6.2 / 5.0, 576 6.6 / 5.7,
  // 1024 7.4 / 7.2, 1152 7.9 / 8.0, 2048 10.3 / 11.4; heads of 64: 512 5.3 / 3.8, 1024 6.0 / 5.0, 2048 7.6 / 7.6, 2304 8.2 / 8.5.
  // A k head to four q heads, heads of 128: 640 6.0 / 5.0, 1280 7.0 / 7.2; heads of 64: 1440 6.1 / 5.6, 2560 7.1 / 7.8.
  if (hd % 8 == 0 && (size_t)row_blocks * (Hq + Hkv) * hd <= 131072) {
    HT_DISPATCH_DTYPE(dtype, hipLaunchKernelGGL((rope_append_rows_kernel<T, T, true>), grid, dim3(256),
                                                values > factors ? values : factors, s, HT_ROPE_ARGS);)
    return hipGetLastError();
  }
  const hipError_t e = launch_rope_table(cs, depth, n, M, hd, base, s);
  if (e != hipSuccess) return e;
  if (hd % 8 == 0) {
    HT_DISPATCH_DTYPE(dtype, hipLaunchKernelGGL((rope_append_rows_kernel<T, T>), grid, dim3(256), values, s, HT_ROPE_ARGS);)
    return hipGetLastError();
  }
#undef HT_ROPE_ARGS
  HT_DISPATCH_DTYPE(dtype, hipLaunchKernelGGL((rope_append_kernel<T, T>), dim3(M, Hq + 2 * Hkv), dim3(hd / 2), 0, s,
                                              (const T*)q_in, Hq * hd, (const T*)k_in, Hkv * hd, (const T*)v_in,
                                              Hkv * hd, 1, (size_t)0, (const float2*)cs, (T*)q, (T*)kc, (T*)vc, n, Hq, Hkv, hd,
                                              cap, 0, nullptr);)
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ SwiGLU gate
__global__ void silu_mul_kernel(const float* __restrict__ gu, bf16_t* __restrict__ act, int f) {
  const int m = blockIdx.y;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= f) return;
  const float g = gu[(size_t)m * 2 * f + j], up = gu[(size_t)m * 2 * f + f + j];
  Conv<bf16_t>::store(act + (size_t)m * f + j, g / (1.0f + expf(-g)) * up);
}
hipError_t launch_silu_mul(const float* gu, void* act, int M, int f, hipStream_t s) {
  hipLaunchKernelGGL(silu_mul_kernel, dim3((f + 255) / 256, M), dim3(256), 0, s, gu, (bf16_t*)act, f);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ argmax / top-k
// (value, id) order: larger value first, lower id first on equal values.  NaN never wins.
__device__ inline bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

// block-wide best for any block size that is a multiple of 64 (<= 1024); sv/si hold 16 entries
__device__ inline void block_best_any(float& v, int& i, float* sv, int* si) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    float ov = __shfl_xor(v, o, 64);
    int oi = __shfl_xor(i, o, 64);
    if (better(ov, oi, v, i)) { v = ov; i = oi; }
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = v; si[threadIdx.x >> 6] = i; }
  __syncthreads();
  v = sv[0]; i = si[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
    if (better(sv[w], si[w], v, i)) { v = sv[w]; i = si[w]; }
}

// g[row] = arg-max of a logit row, lowest id on ties.  1024 threads per row, 16-byte loads.  Few rows: bound by what one
// compute unit takes in, so rows of up to 32768 floats (AHEAD) are requested whole before the first comparison (one row of
// 32000: 7.0 -> 5.2 us).
constexpr int kArgmaxAhead = 8;               // 16-byte pieces per thread
template <bool AHEAD>
__device__ __forceinline__ void argmax_row(const float* __restrict__ z, int32_t* __restrict__ g, int V, int vec, int at) {
  __shared__ float sv[16];
  __shared__ int si[16];
  const float* row = z + (size_t)at * V;
  float bv = -INFINITY;
  int bi = 0x7fffffff;
  auto four = [&](const float4& q, int j) {
    if (better(q.x, j, bv, bi)) { bv = q.x; bi = j; }
    if (better(q.y, j + 1, bv, bi)) { bv = q.y; bi = j + 1; }
    if (better(q.z, j + 2, bv, bi)) { bv = q.z; bi = j + 2; }
    if (better(q.w, j + 3, bv, bi)) { bv = q.w; bi = j + 3; }
  };
  if (AHEAD) {
    float4 p[kArgmaxAhead];
#pragma unroll
    for (int i = 0; i < kArgmaxAhead; ++i) {
      const int j = (i * 1024 + threadIdx.x) * 4;
      p[i] = *(const float4*)(row + (j < V ? j : 0));
    }
#pragma unroll
    for (int i = 0; i < kArgmaxAhead; ++i) {
      const int j = (i * 1024 + threadIdx.x) * 4;
      if (j < V) four(p[i], j);
    }
  } else {
    const int v4 = vec ? (V & ~3) : 0;          // vec: rows are 16-byte aligned
    for (int j = threadIdx.x * 4; j < v4; j += blockDim.x * 4) four(*(const float4*)(row + j), j);
    for (int j = v4 + threadIdx.x; j < V; j += blockDim.x)
      if (better(row[j], j, bv, bi)) { bv = row[j]; bi = j; }
  }
  block_best_any(bv, bi, sv, si);
  if (threadIdx.x == 0) g[at] = bi == 0x7fffffff ? 0 : bi;
}
template <bool AHEAD>
__global__ __launch_bounds__(1024) void argmax_kernel(const float* __restrict__ z, int32_t* __restrict__ g, int V, int vec) {
  argmax_row<AHEAD>(z, g, V, vec, blockIdx.x);
}
// rows on 16 bytes; below three pieces per thread the eight fixed requests cost more than they hide (1000: 3.5 and 4.0 us,
// 8192: 4.0 and 4.35, 16384: 4.5 both, 32000: 5.6 and 5.0)
int argmax_vec(const float* z, int V) { return !((uintptr_t)z & 15) && !(V & 3); }
bool argmax_ahead(int vec, int V) { return vec && V > 12288 && V <= 4096 * kArgmaxAhead; }
hipError_t launch_argmax(const float* z, int32_t* g, int M, int V, hipStream_t s) {
  const int vec = argmax_vec(z, V);
  if (argmax_ahead(vec, V)) hipLaunchKernelGGL(argmax_kernel<true>, dim3(M), dim3(1024), 0, s, z, g, V, vec);
  else hipLaunchKernelGGL(argmax_kernel<false>, dim3(M), dim3(1024), 0, s, z, g, V, vec);
  return hipGetLastError();
}

// cand[i][r], r < width[i+1]: the r-th entry of logit row i in (value desc, id asc) order.
// Two stages of the same selection: repeated block-wide arg-best over the entries that come strictly after
// the previous pick in that order.  Stage 1 runs it on kTopkSlices slices of the row in parallel and leaves
// each slice's best b entries in scratch (any of the row's top b is among its slice's top b); stage 2 runs
// it once more over those kTopkSlices * b survivors.
constexpr int kTopkSlices = 32;

template <bool FINAL>
__global__ __launch_bounds__(256) void topk_kernel(const float* __restrict__ d, const float* __restrict__ sv_in,
                                                   const int32_t* __restrict__ si_in, float* __restrict__ sv_out,
                                                   int32_t* __restrict__ si_out, int32_t* __restrict__ cand,
                                                   const int32_t* __restrict__ width, int period, const int32_t* __restrict__ src_row,
                                                   int V) {
  __shared__ float sv[16];
  __shared__ int si[16];
  const int i = blockIdx.x, slice = blockIdx.y;
  const int b = width[i % period + 1];      // row i drafts the tree level i % period + 1
  // element range of this block: a slice of the logit row, or the survivors of all slices
  int lo, hi;
  if (FINAL) { lo = 0; hi = kTopkSlices * b; }
  else {
    const int per = (V + kTopkSlices - 1) / kTopkSlices;
    lo = slice * per;
    hi = lo + per < V ? lo + per : V;
  }
  float pv = INFINITY;
  int pi = -1;
  for (int r = 0; r < b; ++r) {
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int j = lo + threadIdx.x; j < hi; j += 256) {
      float v;
      int id;
      if (FINAL) { v = sv_in[(size_t)i * kTopkSlices * kMaxTopK + j]; id = si_in[(size_t)i * kTopkSlices * kMaxTopK + j]; }
      else { v = d[(size_t)(src_row ? src_row[i] : i) * V + j]; id = j; }
      const bool after = r == 0 || v < pv || (v == pv && id > pi);
      if (after && better(v, id, bv, bi)) { bv = v; bi = id; }
    }
    block_best_any(bv, bi, sv, si);
    if (threadIdx.x == 0) {
      if (FINAL) cand[i * kMaxTopK + r] = bi == 0x7fffffff ? 0 : bi;
      else {
        sv_out[(size_t)i * kTopkSlices * kMaxTopK + slice * b + r] = bi == 0x7fffffff ? -INFINITY : bv;
        si_out[(size_t)i * kTopkSlices * kMaxTopK + slice * b + r] = bi;
      }
    }
    pv = bv; pi = bi;
    __syncthreads();
  }
}
// The same two stages with the selection done by wavefronts on register-resident entries: every wavefront of a block
// takes a quarter of the block's entries (E per lane), picks its best b one by one (a wave-wide maximum by DPP moves,
// a ballot, the lowest id among equal values), the four lists meet in LDS and the first wavefront picks the best b
// of them the same way.  No block-wide barrier inside the rounds and no re-reading of the row.  The order is the
// total order (value descending, id ascending), so the result is that of `topk_kernel` bit for bit.
constexpr int kNoEntry = 0x7fffffff;       // id of an empty slot: loses against every real entry of the same value

template <int E>
__device__ inline void wave_select(float (&v)[E], int (&id)[E], int b, float* out_v, int* out_i) {
  const int lane = threadIdx.x & 63;
  for (int r = 0; r < b; ++r) {
    float bv = v[0];
    int bi = id[0];
#pragma unroll
    for (int e = 1; e < E; ++e)
      if (better(v[e], id[e], bv, bi)) { bv = v[e]; bi = id[e]; }
    const float top = wave_max_dpp(bv);
    const bool tie = bv == top;
    const uint64_t mask = __ballot(tie);
    int pick;
    if (mask & (mask - 1)) pick = wave_min_dpp(tie ? bi : kNoEntry);
    else pick = __builtin_amdgcn_readlane(bi, __builtin_amdgcn_readfirstlane(__builtin_ctzll(mask)));
    if (lane == 0) { out_v[r] = top; out_i[r] = pick; }
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (id[e] == pick) { v[e] = -INFINITY; id[e] = kNoEntry; }
  }
}

// WHOLE: one stage over a row of up to 2048 entries (rows that short are over before a second launch has started).
enum TopkStage { SLICE, FINAL, WHOLE };
template <int E, int STAGE>
__device__ __forceinline__ void topk_block(const float* __restrict__ d, const float* __restrict__ sv_in, const int32_t* __restrict__ si_in,
                                           float* __restrict__ sv_out, int32_t* __restrict__ si_out, int32_t* __restrict__ cand,
                                           const int32_t* __restrict__ width, int period, const int32_t* __restrict__ src_row, int V,
                                           int i, int slice, int wave, float (*list_v)[kMaxTopK], int (*list_i)[kMaxTopK]) {
  const int lane = threadIdx.x & 63;
  const int b = width[i % period + 1];      // row i drafts the tree level i % period + 1
  if (b <= 0) return;                       // uniform over the workgroup
  int lo, hi;
  if (STAGE == FINAL) { lo = 0; hi = kTopkSlices * b; }
  else if (STAGE == WHOLE) { lo = 0; hi = V; }
  else {
    const int per = (V + kTopkSlices - 1) / kTopkSlices;
    lo = slice * per;
    hi = lo + per < V ? lo + per : V;
  }
  const int quarter = (hi - lo + 3) / 4;
  const int w0 = lo + wave * quarter, w1 = w0 + quarter < hi ? w0 + quarter : hi;
  const size_t base = STAGE == FINAL ? (size_t)i * kTopkSlices * kMaxTopK : (size_t)(src_row ? src_row[i] : i) * V;
  float v[E];
  int id[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int j = w0 + lane + 64 * e;
    v[e] = -INFINITY;
    id[e] = kNoEntry;
    if (j < w1) {
      const float x = STAGE == FINAL ? sv_in[base + j] : d[base + j];
      const int xi = STAGE == FINAL ? si_in[base + j] : j;
      if (x == x && xi != kNoEntry) { v[e] = x; id[e] = xi; }      // NaN never wins
    }
  }
  wave_select<E>(v, id, b, list_v[wave], list_i[wave]);
  __syncthreads();
  if (wave) return;
  float v2[4];
  int id2[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v2[e] = lane < b ? list_v[e][lane] : -INFINITY;
    id2[e] = lane < b ? list_i[e][lane] : kNoEntry;
  }
  wave_select<4>(v2, id2, b, list_v[4], list_i[4]);
  if (lane < b) {                           // one wavefront: its LDS writes are ordered before these reads
    if (STAGE != SLICE) cand[i * kMaxTopK + lane] = list_i[4][lane] == kNoEntry ? 0 : list_i[4][lane];
    else {
      sv_out[(size_t)i * kTopkSlices * kMaxTopK + slice * b + lane] = list_v[4][lane];
      si_out[(size_t)i * kTopkSlices * kMaxTopK + slice * b + lane] = list_i[4][lane];
    }
  }
}

template <int E, int STAGE>
__global__ __launch_bounds__(256) void topk_wave_kernel(const float* __restrict__ d, const float* __restrict__ sv_in,
                                                        const int32_t* __restrict__ si_in, float* __restrict__ sv_out,
                                                        int32_t* __restrict__ si_out, int32_t* __restrict__ cand,
                                                        const int32_t* __restrict__ width, int period,
                                                        const int32_t* __restrict__ src_row, int V) {
  __shared__ float list_v[5][kMaxTopK];
  __shared__ int list_i[5][kMaxTopK];
  topk_block<E, STAGE>(d, sv_in, si_in, sv_out, si_out, cand, width, period, src_row, V, blockIdx.x, blockIdx.y, threadIdx.x >> 6,
                       list_v, list_i);
}

// The arg-max of T rows and the first stage of the selection over others in one launch (both read what one product has
// written): workgroups 0 .. T - 1 a row each, the others four slices of a row.  Where there is room on the chip (joint_selection
// says where) that saves a launch and hides one under the other.  Together with the launch that starts a pass
// putting its tokens together and the head storing the caller's rows itself, a step of 64 nodes on four 7B-wide blocks 549 -> 538
// us with 12 draft rows, 903 -> 892 on two of 70B width with 16.
template <bool AHEAD, int E>
__global__ __launch_bounds__(1024) void argmax_topk_kernel(const float* __restrict__ z, int32_t* __restrict__ g, int vec, int T,
                                                           const float* __restrict__ d, float* __restrict__ sv_out,
                                                           int32_t* __restrict__ si_out, const int32_t* __restrict__ width, int period,
                                                           const int32_t* __restrict__ src_row, int V) {
  if ((int)blockIdx.x < T) {
    argmax_row<AHEAD>(z, g, V, vec, blockIdx.x);
    return;
  }
  __shared__ float list_v[4][5][kMaxTopK];
  __shared__ int list_i[4][5][kMaxTopK];
  const int at = (blockIdx.x - T) * 4, quad = threadIdx.x >> 8;
  topk_block<E, SLICE>(d, nullptr, nullptr, sv_out, si_out, nullptr, width, period, src_row, V, at / kTopkSlices,
                       at % kTopkSlices + quad, (threadIdx.x >> 6) & 3, list_v[quad], list_i[quad]);
}

// Whether the joint launch is the faster one for draft rows of which the widest level takes b candidates.  Its workgroups hold four
// slices each, so four selecting wavefronts share a SIMD where workgroups of one slice have one, and up to 32 rows they are one
// workgroup a compute unit; beyond that a second one waits for sixteen free places at once.  What it saves (a launch, and the
// arg-max beside the selection) is 2.5 to 4 us, more for long rows; what it costs grows with b, and with the rows beyond 32.  Us, both
// stages and the arg-max of 64 rows, joint / separate, V = 32000: 12 rows of 4 candidates 11.5 / 15.3, of 10 21.4 / 23.5, of 40 70.8 /
// 64.4; 64 rows of 4 17.1 / 17.8, of 10 30.4 / 29.4; 192 of 2 22.2 / 22.4, of 4 31.5 / 28.6, of 10 60.0 / 48.7.  V = 4096: 64 of 4 15.5 /
// 16.1, 96 of 4 18.5 / 18.0.  V = 40000 (slices of sixteen entries a lane): 8 of 8 0.3 more, of 10 1.4 more, 40 of 4 0.8 less, of 8 3.2
// more.  V = 65536: 24 of 10 29.8 / 33.4, 80 of 6 38.4 / 42.4, 40 of 8 1.6 more.  V = 128000: 12 of 10 34.3 / 46.0, 24 of 16 49.0 /
// 61.3, 64 of 12 60.8 / 67.8, 128 of 10 79.9 / 84.2, of 40 247 / 239.
bool joint_selection(int rows, int b, int V) {
  if (V > 98304) return b <= (rows <= 32 ? 16 : 12);
  if (V > 49152) return b <= (rows <= 32 ? 10 : 6);
  if (V > 32768) return b <= (rows <= 32 ? 8 : 4);
  return rows <= 32 ? b <= 10 : b <= 4 && rows * b <= 256;
}
// scratch: float[rows][kTopkSlices][kMaxTopK] followed by int32 of the same shape
size_t topk_scratch_bytes(int rows) { return (size_t)rows * kTopkSlices * kMaxTopK * 8; }
hipError_t launch_topk(const float* d, int32_t* cand, const int32_t* width, void* scratch, int rows, int period,
                       const int32_t* src_row, int V, hipStream_t s, const float* z, int32_t* g, int T, int widest) {
  float* sv = (float*)scratch;
  int32_t* si = (int32_t*)(sv + (size_t)rows * kTopkSlices * kMaxTopK);
  // entries per lane of the first stage: a quarter of a slice over 64 lanes; of the second: a quarter of
  // kTopkSlices * b <= 2048 survivors
  const int per_lane = (((V + kTopkSlices - 1) / kTopkSlices + 3) / 4 + 63) / 64;
  const dim3 g1(rows, kTopkSlices), g2(rows, 1);
#define HT_TOPK_ARGS(in_v, in_i, out_v, out_i) d, in_v, in_i, out_v, out_i, cand, width, period, src_row, V
  if (g && (V <= 2048 || per_lane > 16 || !joint_selection(rows, widest, V))) {
    const hipError_t e = launch_argmax(z, g, T, V, s);
    if (e != hipSuccess) return e;
    g = nullptr;
  }
  if (V <= 2048) {
    hipLaunchKernelGGL((topk_wave_kernel<8, WHOLE>), g2, dim3(256), 0, s, HT_TOPK_ARGS(nullptr, nullptr, nullptr, nullptr));
    return hipGetLastError();
  }
  static_assert(kTopkSlices % 4 == 0, "the four slices of a workgroup are of one row");
  if (g) {
    const int vec = argmax_vec(z, V);
    const dim3 both(T + rows * (kTopkSlices / 4));
#define HT_BOTH(AHEAD, E) \
  hipLaunchKernelGGL((argmax_topk_kernel<AHEAD, E>), both, dim3(1024), 0, s, z, g, vec, T, d, sv, si, width, period, src_row, V)
    if (argmax_ahead(vec, V)) {
      if (per_lane <= 4) HT_BOTH(true, 4);
      else HT_BOTH(true, 16);
    } else {
      if (per_lane <= 4) HT_BOTH(false, 4);
      else HT_BOTH(false, 16);
    }
#undef HT_BOTH
  } else if (per_lane <= 4)
    hipLaunchKernelGGL((topk_wave_kernel<4, SLICE>), g1, dim3(256), 0, s, HT_TOPK_ARGS(nullptr, nullptr, sv, si));
  else if (per_lane <= 16)
    hipLaunchKernelGGL((topk_wave_kernel<16, SLICE>), g1, dim3(256), 0, s, HT_TOPK_ARGS(nullptr, nullptr, sv, si));
  else          // very large vocabularies: block-wide selection, any row length
    hipLaunchKernelGGL(topk_kernel<false>, g1, dim3(256), 0, s, HT_TOPK_ARGS(nullptr, nullptr, sv, si));
  hipLaunchKernelGGL((topk_wave_kernel<8, FINAL>), g2, dim3(256), 0, s, HT_TOPK_ARGS(sv, si, nullptr, nullptr));
#undef HT_TOPK_ARGS
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ tree choice / accept / compact
// ---- tree chosen from the draft distributions
// lp[i][r] = log-softmax value of candidate r of draft row i:  z - (max + log(sum exp(z - max))) over the whole row.
// One block of 1024 threads per row, few rows: bound by what one compute unit takes in (50 GB/s) and by the reductions
// behind it.  A thread brings in up to 32 floats at a time, all requested before the first is used (16 bytes each where the rows
// lie on 16 bytes), and keeps a sum against its own maximum, so a row is read once and maxima and sums meet once at the
// end.  Three rows, us, with two walks over the row (or a block-wide maximum in the middle) and now: 1000 3.3 and 3.2, 5000 3.6
// and 3.6, 8000 4.0 and 3.6, 32000 6.8 and 6.1, 128000 20.4 and 16.3; of odd length 1003 3.2 and 3.1, 8193 5.1 and 4.4, 32001
// 11.2 and 7.5, 127999 36 and 22.
// e^x for x <= 0 (NaN stays NaN, -inf gives 0): 2^(k + f), k the integer next to x log2 e and f the rest of that product, made
// in two parts and rounded once.  At most 0.86 units in the last place (0.26 in the mean) over x > -87 and 0.9 of the smallest
// denormal below, both as expf, whose range checks three rows of 1000 floats notice (3.5 us instead of 3.4), 32000 more so (6.8, 6.2).
__device__ inline float exp_below(float x) {
#pragma clang fp contract(off)
  x = x < -150.f ? -150.f : x;
  const float t = x * 1.44269504f, k = rintf(t);
  return ldexpf(__builtin_amdgcn_exp2f((t - k) + fmaf(x, 1.92596299e-8f, fmaf(x, 1.44269504f, -t))), (int)k);
}
template <int VEC, int PIECES>
__global__ __launch_bounds__(1024) void cand_logprob_kernel(const float* __restrict__ d, const int32_t* __restrict__ cand,
                                                            int b, int V, float* __restrict__ lp) {
  __shared__ float2 wave_red[16];
  constexpr int STEP = 1024 * VEC;
  const float* row = d + (size_t)blockIdx.x * V;
  // the candidates' own values are on their way while the row is summed up
  const float own = (int)threadIdx.x < b ? row[cand[blockIdx.x * kMaxTopK + threadIdx.x]] : 0.f;
  float peak = -INFINITY, sum = 0.f;
  for (int base = 0; base < V; base += PIECES * STEP) {
    float v[PIECES][VEC];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int j = base + i * STEP + threadIdx.x * VEC;
#pragma unroll
      for (int u = 0; u < VEC; ++u) v[i][u] = -INFINITY;
      if (base + i * STEP >= V) continue;                      // uniform
      if (j < V) {
        if (VEC == 4) {
          const float4 q = *(const float4*)(row + j);
          v[i][0] = q.x, v[i][VEC / 4] = q.y, v[i][VEC / 2] = q.z, v[i][VEC - 1] = q.w;
        } else {
          v[i][0] = row[j];
        }
      }
    }
    float high = peak;
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
      if (base + i * STEP < V) {
#pragma unroll
        for (int u = 0; u < VEC; ++u) high = fmaxf(high, v[i][u]);
      }
    const float ref = high == -INFINITY ? 0.f : high;          // (nothing but -inf so far: sums of zeros)
    sum *= exp_below(peak - ref);
    peak = high;
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      if (base + i * STEP < V) {
        float part = 0.f;
#pragma unroll
        for (int u = 0; u < VEC; ++u) part += exp_below(v[i][u] - ref);
        sum += part;
      }
    }
  }
  const float top = wave_max_dpp(peak);
  sum = wave_sum(sum * exp_below(peak - (top == -INFINITY ? 0.f : top)));
  if ((threadIdx.x & 63) == 0) wave_red[threadIdx.x >> 6] = make_float2(top, sum);
  __syncthreads();
  peak = wave_red[0].x;
#pragma unroll
  for (int w = 1; w < 16; ++w) peak = fmaxf(peak, wave_red[w].x);
  sum = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) sum += wave_red[w].y * exp_below(wave_red[w].x - peak);
  const float lse = peak + logf(sum);
  if ((int)threadIdx.x < b) lp[blockIdx.x * kMaxTopK + threadIdx.x] = own - lse;
}
hipError_t launch_cand_logprob(const float* d, const int32_t* cand, int rows, int b, int V, float* lp, hipStream_t s) {
  // As many pieces as the row has, up to eight of 16 bytes: loads that are not there are checked for all the same (5000 floats
  // in eight 3.9 us, in two 3.6; 16384 in eight 4.53, in four 4.48, in two 4.50).  Single floats four at a time up to 24576,
  // where the rounds cost less than the checks (8193: in 32 5.8, in four 4.35; 20001 6.6 and 5.95; 32001 7.5 and 8.0).
  if (!((uintptr_t)d & 15) && !(V & 3)) {
    if (V <= 4096) hipLaunchKernelGGL((cand_logprob_kernel<4, 1>), dim3(rows), dim3(1024), 0, s, d, cand, b, V, lp);
    else if (V <= 8192) hipLaunchKernelGGL((cand_logprob_kernel<4, 2>), dim3(rows), dim3(1024), 0, s, d, cand, b, V, lp);
    else if (V <= 16384) hipLaunchKernelGGL((cand_logprob_kernel<4, 4>), dim3(rows), dim3(1024), 0, s, d, cand, b, V, lp);
    else hipLaunchKernelGGL((cand_logprob_kernel<4, 8>), dim3(rows), dim3(1024), 0, s, d, cand, b, V, lp);
  } else if (V <= 24576) {
    hipLaunchKernelGGL((cand_logprob_kernel<1, 4>), dim3(rows), dim3(1024), 0, s, d, cand, b, V, lp);
  } else {
    hipLaunchKernelGGL((cand_logprob_kernel<1, 32>), dim3(rows), dim3(1024), 0, s, d, cand, b, V, lp);
  }
  return hipGetLastError();
}

// The T - 1 best nodes of the complete b-ary candidate tree of depth k in the order (score descending, depth
// ascending, rank path ascending), score = sum of lp along the path accumulated in float from the root down.
// Two ways lead there.  tree_walk takes one node at a time; tree_levels takes a level at a time with eight wavefronts
// and needs rows in order (best first, none above zero), as every softmax gives them.  A table that is not in order has no
// such order of nodes: there the walk is the definition.  tree_dynamic_kernel looks at the table and decides.
struct TreeScratch {
  float lp[kMaxTransfer * kMaxTopK];
  int cand[kMaxTransfer * kMaxTopK];
  int parent[kMaxTree], depth[kMaxTree], rank[kMaxTree];
};
__device__ inline float not_nan(float v) { return v == v ? v : -INFINITY; }

// (depth, path) order of two frontier entries with equal scores
__device__ inline bool tie_first(int depth_a, uint64_t path_a, int depth_b, uint64_t path_b) {
  return depth_a != depth_b ? depth_a < depth_b : path_a < path_b;
}

// A node never scores above its parent or its previous sibling, and each of the two comes first in that order, so
// the order is produced by a best-first walk: the frontier holds, for every node taken so far, its next sibling
// and (once) its first child; the best frontier entry becomes the next node.  The frontier never holds more than
// T <= 128 entries: slot j lives in the registers of lane j % 64 (one slot per lane in the first 63 rounds, two from then
// on), a round is one wave-wide maximum of the lanes' best scores, a ballot that names the winner (a second reduction over
// depth and path only when several lanes hold the best score), and register updates in two lanes.  What bounds it is the
// chain of dependent instructions from one round to the next, 0.3 us, so nothing on it waits for memory: the score of every
// entry's next sibling is at hand before the entry wins (its table read has until the entry wins again), and the best
// candidate of every level, which a first child adds, sits in a register of the lane of that number.
// One wavefront; rows of `t` that it does not reach keep what they hold.
template <int SLOTS>
__device__ __forceinline__ void tree_walk(TreeScratch& t, int k, int b, int T) {
  const int lane = threadIdx.x & 63;
  const float first = lane < k ? t.lp[lane * kMaxTopK] : 0.f;         // lane e: the best candidate of level e + 1
  // frontier slot: score, score of its next sibling, score of the parent, depth (0: empty), parent node,
  // path = ranks from the root down, 6 bits each, the last rank in the lowest digit
  float fs[SLOTS], fn[SLOTS], fb[SLOTS];
  int fd[SLOTS], fp[SLOTS];
  uint64_t fq[SLOTS];
#pragma unroll
  for (int i = 0; i < SLOTS; ++i) {
    fs[i] = fn[i] = -INFINITY;
    fb[i] = 0.f;
    fd[i] = fp[i] = 0;
    fq[i] = 0;
  }
  const float top_lp = t.lp[0], next_lp = t.lp[1];
  if (lane == 0) { fs[0] = top_lp; fn[0] = next_lp; fd[0] = 1; }      // first candidate of the first level, under the root
  int count = 1;
  auto round = [&](int v, auto both) __attribute__((always_inline)) -> bool {
    constexpr int N = decltype(both)::value ? 2 : 1;                // slots in use
    const bool second = N == 2 && fd[SLOTS - 1] != 0 &&
                        (fd[0] == 0 || fs[SLOTS - 1] > fs[0] ||
                         (fs[SLOTS - 1] == fs[0] && tie_first(fd[SLOTS - 1], fq[SLOTS - 1], fd[0], fq[0])));
    const float s = second ? fs[SLOTS - 1] : fs[0];
    const int d = second ? fd[SLOTS - 1] : fd[0];
    const uint64_t q = second ? fq[SLOTS - 1] : fq[0];
    const int par_l = second ? fp[SLOTS - 1] : fp[0];
    const float best = wave_max_dpp(d ? s : -INFINITY);
    const bool top = d != 0 && s == best;
    uint64_t tied = __ballot(top);
    if (tied == 0) return false;                   // frontier exhausted: uniform
    if (tied & (tied - 1)) {                       // several lanes hold the best score: depth, then path decide
      uint64_t key = top ? ((uint64_t)d << 48 | q) : ~0ull;
      uint64_t low = key;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const uint64_t other = __shfl_xor((unsigned long long)low, o, 64);
        low = other < low ? other : low;
      }
      tied = __ballot(key == low);
    }
    const int win = __builtin_amdgcn_readfirstlane(__builtin_ctzll(tied));
    const int depth = __builtin_amdgcn_readlane(d, win);
    const int par = __builtin_amdgcn_readlane(par_l, win);
    const uint64_t path = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(q >> 32), win) << 32 |
                          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)q, win);
    const int r = (int)(path & 63);
    if (lane == win) {                             // the next sibling takes the slot over
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (N == 1 || second == (i == 1)) {
          fs[i] = fn[i];
          fq[i] += 1;
          fd[i] = r + 1 < b ? depth : 0;
          if (r + 2 < b) fn[i] = fb[i] + t.lp[(depth - 1) * kMaxTopK + r + 2];
        }
      t.parent[v] = par;
      t.depth[v] = depth;
      t.rank[v] = r;
    }
    if (depth < k) {                               // the first child goes to a new slot
      // (read here, where all lanes are active: in the one-lane branch the lane of that number would not be)
      const float child = best + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(first), depth));
      if (lane == (count & 63)) {
#pragma unroll
        for (int i = 0; i < N; ++i)
          if (N == 1 || (count >> 6) == i) {
            fs[i] = child;
            fb[i] = best;
            fd[i] = depth + 1;
            fp[i] = v;
            fq[i] = path << 6;
            fn[i] = best + t.lp[depth * kMaxTopK + 1];
          }
      }
      ++count;
    }
    return true;
  };
  // before round v no more than v entries exist: the second slots stay empty until round 64
  bool more = true;
  const int alone = SLOTS == 1 || T < 64 ? T : 64;
  for (int v = 1; v < alone; ++v) {
    more = round(v, std::false_type{});
    if (!more) break;
  }
  if (SLOTS == 2 && more)
    for (int v = 64; v < T; ++v)
      if (!round(v, std::integral_constant<bool, SLOTS == 2>{})) break;
}

// Level by level: `ranked` holds the T - 1 best nodes of the levels so far, in order.  A round appends the children of the
// last level's nodes among them, counts for every entry how many come before it, and keeps the first T - 1; a node that
// drops out takes nothing with it that could still get in, because its children come after it.
//  - The order of the array is the order of ties: older levels first, a level in path order (children are appended parent
//    by parent in path order, so the same holds for the next level).  So entry j comes before entry i if its score is
//    higher, or equal and j < i.
//  - A node (a_1 .. a_e) of ranks a_i - 1 comes after every node of the same or a smaller depth whose ranks are nowhere
//    larger: sum over f <= e of a_1 .. a_f nodes with itself.  Only nodes with a sum of at most T - 1 are appended, and, once
//    T - 1 nodes are known, only those that beat the last: at most kLevelRoom a round (2806 for eight levels of 64
//    candidates and 128 nodes, 10 + 84 + about 100 for three levels of 10 and 64 nodes).
// Bound: a handful of LDS round trips and barriers a level, and the counting, 2 instructions for every pair of entries.
constexpr int kTreeWaves = 8;
static_assert(kMaxTransfer % kTreeWaves == 0, "a wavefront brings in whole levels of the table");
constexpr int kLevelRoom = 2816;
constexpr int kLevelMany = 256, kLevelBuckets = 256;
constexpr int kCountStep = 4;                                  // 16-byte reads of entries in flight while they are compared
struct LevelScratch {
  alignas(16) uint32_t key[2][kMaxTree + kLevelRoom + 4 * kCountStep];      // scores as integers in the same order: ranked, then appended
  uint16_t id[2][kMaxTree];                                   // node ids of the ranked entries
  uint16_t from[kLevelRoom];                                  // appended entry: index of its parent in the level, rank
  alignas(16) int place[kMaxTree + kLevelRoom];               // entries that come before it
  float score[2][kMaxTree];                                   // last level's ranked nodes in path order: score,
  int prod[2][kMaxTree], sum[2][kMaxTree];                    // a_1 .. a_e and the sum above,
  uint16_t node[2][kMaxTree];                                 // id
  uint16_t parent[1 + kMaxTransfer * kMaxTree];               // by id (0: the root): parent's id, rank, depth, place in the tree
  uint8_t rank[1 + kMaxTransfer * kMaxTree], depth[1 + kMaxTransfer * kMaxTree], at[1 + kMaxTransfer * kMaxTree];
  int count[2][kTreeWaves];
};

__device__ inline uint32_t ordered_bits(float v) {             // larger float, larger integer; never 0 for a number
  const uint32_t u = __float_as_uint(v + 0.0f);                // (-0 and 0 are equal)
  return u & 0x80000000u ? ~u : u | 0x80000000u;
}

__device__ inline float from_ordered_bits(uint32_t k) { return __uint_as_float(k & 0x80000000u ? k & 0x7fffffffu : ~k); }

__device__ __forceinline__ void tree_levels(TreeScratch& t, LevelScratch& l, int k, int b, int T) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const uint64_t below = (1ull << lane) - 1;
  const float inv_b = 1.0f / (float)b;
  if (tid == 0) {
    l.score[0][0] = 0.f;
    l.prod[0][0] = 1;
    l.sum[0][0] = 0;
    l.node[0][0] = 0;
    l.at[0] = 0;
  }
  __syncthreads();
  int m = 0, level = 1, ids = 1;                               // ranked entries, nodes of the last level, ids given out
  for (int e = 0; e < k && level > 0; ++e) {
    uint32_t* const key = l.key[e & 1];
    const int cur = e & 1, nxt = cur ^ 1;
    const int grid = level * b;                                // child slots, parent by parent
    const int per_wave = (grid + 64 * kTreeWaves - 1) / (64 * kTreeWaves) * 64, g0 = wave * per_wave;
    const uint32_t last = m == T - 1 ? key[m - 1] : 0;         // what an appended entry has to beat
    auto child = [&](int g, uint32_t& score_bits, int& from) __attribute__((always_inline)) -> bool {
      const int p = (int)(((float)g + 0.5f) * inv_b), r = g - p * b;      // g < 8192: exact
      if (g >= grid) return false;
      from = p << 6 | r;
      score_bits = ordered_bits(l.score[cur][p] + t.lp[e * kMaxTopK + r]);
      return l.sum[cur][p] + l.prod[cur][p] * (r + 1) <= T - 1 && score_bits > last;
    };
    uint32_t bits = 0;
    int from = 0, mine = 0;
    bool yes = false;
    uint64_t all = 0;
    for (int g = g0; g < g0 + per_wave && g < grid; g += 64) {
      yes = child(g + lane, bits, from);
      all = __ballot(yes);
      mine += __popcll(all);
    }
    if (lane == 0) l.count[0][wave] = mine;
    __syncthreads();
    int at = m, added = 0;
    auto take_counts = [&](const int* counts, int& upto, int& total) __attribute__((always_inline)) {
#pragma unroll
      for (int w = 0; w < kTreeWaves; ++w) {
        const int c = counts[w];
        upto += w < wave ? c : 0;
        total += c;
      }
    };
    take_counts(l.count[0], at, added);
    if (m > 0 && m + added > kLevelMany) {
      // So many that counting would take long: a histogram of how far entries are behind the first (kLevelBuckets of 1/16,
      // the last one without end) says which buckets the first T - 1 lie in; the others are left out.
      for (int i = tid; i < kLevelBuckets; i += 64 * kTreeWaves) l.place[i] = 0;
      __syncthreads();
      const float top = from_ordered_bits(key[0]);
      auto bucket = [&](uint32_t score_bits) __attribute__((always_inline)) {
        return (int)fminf((top - from_ordered_bits(score_bits)) * 16.f, (float)(kLevelBuckets - 1));
      };
      for (int i = tid; i < m; i += 64 * kTreeWaves) atomicAdd(&l.place[bucket(key[i])], 1);
      for (int g = g0; g < g0 + per_wave && g < grid; g += 64)
        if (child(g + lane, bits, from)) atomicAdd(&l.place[bucket(bits)], 1);
      __syncthreads();
      static_assert(kLevelBuckets == 256, "four buckets to a lane");
      const int4 h = *(const int4*)(l.place + lane * 4);
      int sum = h.x + h.y + h.z + h.w;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int other = __shfl_up(sum, o, 64);
        sum += lane >= o ? other : 0;
      }
      const uint64_t enough = __ballot(sum >= T - 1);
      const int limit = enough ? __builtin_ctzll(enough) * 4 + 3 : kLevelBuckets;       // to four buckets
      auto close = [&](int g) __attribute__((always_inline)) { return child(g, bits, from) && bucket(bits) <= limit; };
      mine = 0;
      for (int g = g0; g < g0 + per_wave && g < grid; g += 64) {
        yes = close(g + lane);
        all = __ballot(yes);
        mine += __popcll(all);
      }
      if (lane == 0) l.count[1][wave] = mine;
      __syncthreads();
      at = m;
      added = 0;
      take_counts(l.count[1], at, added);
      for (int g = g0; g < g0 + per_wave && g < grid; g += 64) {
        if (per_wave > 64) {
          yes = close(g + lane);
          all = __ballot(yes);
        }
        if (yes) {
          const int i = at + __popcll(all & below);
          key[i] = bits;
          l.from[i - m] = (uint16_t)from;
        }
        at += __popcll(all);
      }
    } else {
      for (int g = g0; g < g0 + per_wave && g < grid; g += 64) {
        if (per_wave > 64) {                                   // (with one turn everything is still in registers)
          yes = child(g + lane, bits, from);
          all = __ballot(yes);
        }
        if (yes) {
          const int i = at + __popcll(all & below);
          key[i] = bits;
          l.from[i - m] = (uint16_t)from;
        }
        at += __popcll(all);
      }
    }
    const int entries = m + added;
    if (tid < 4 * kCountStep) key[entries + tid] = 0;          // never before anything: the counts go by so many
    // 64 entries to a wavefront; where that leaves wavefronts over, 2^lg of them share the entries these are compared with
    const int blocks = (entries + 63) / 64, lg = blocks == 1 ? 3 : blocks == 2 ? 2 : blocks <= 4 ? 1 : 0;
    const int steps = (entries + 4 * kCountStep - 1) / (4 * kCountStep), share = (steps + (1 << lg) - 1) >> lg;
    if (lg)
      for (int i = tid; i < entries; i += 64 * kTreeWaves) l.place[i] = 0;
    __syncthreads();
    for (int block = wave >> lg; block < blocks; block += kTreeWaves) {
      const int i0 = block * 64, i = i0 + lane, s0 = (wave & ((1 << lg) - 1)) * share, s1 = s0 + share < steps ? s0 + share : steps;
      const uint32_t own = i < entries ? key[i] : 0, less = own - 1;
      int before = 0;
      for (int j0 = s0 * 4 * kCountStep; j0 < s1 * 4 * kCountStep; j0 += 4 * kCountStep) {
        uint4 v[kCountStep];
#pragma unroll
        for (int u = 0; u < kCountStep; ++u) v[u] = *(const uint4*)(key + j0 + u * 4);
        if (j0 < i0 || j0 >= i0 + 64) {            // all of them in front of this wavefront's entries, or behind
          const uint32_t bar = j0 < i0 ? less : own;
#pragma unroll
          for (int u = 0; u < kCountStep; ++u) before += (v[u].x > bar) + (v[u].y > bar) + (v[u].z > bar) + (v[u].w > bar);
        } else {
#pragma unroll
          for (int u = 0; u < kCountStep; ++u) {
            const int j = j0 + u * 4;
            before += (v[u].x > (j < i ? less : own)) + (v[u].y > (j + 1 < i ? less : own)) + (v[u].z > (j + 2 < i ? less : own)) +
                      (v[u].w > (j + 3 < i ? less : own));
          }
        }
      }
      if (i < entries) {
        if (lg) atomicAdd(&l.place[i], before);
        else l.place[i] = before;
      }
    }
    __syncthreads();
    const int per = (added + 64 * kTreeWaves - 1) / (64 * kTreeWaves) * 64, a0 = wave * per;
    mine = 0;
    for (int a = a0; a < a0 + per && a < added; a += 64)
      mine += __popcll(__ballot(a + lane < added && l.place[m + a + lane] < T - 1));
    if (lane == 0) l.count[0][wave] = mine;
    for (int i = tid; i < m; i += 64 * kTreeWaves) {           // older entries move down
      const int to = l.place[i];
      if (to < T - 1) {
        l.key[nxt][to] = key[i];
        l.id[nxt][to] = l.id[cur][i];
      }
    }
    __syncthreads();
    int pos = 0, kept = 0;
    take_counts(l.count[0], pos, kept);
    for (int a = a0; a < a0 + per && a < added; a += 64) {
      const int i = m + a + lane;
      const int to = a + lane < added ? l.place[i] : T;
      const bool keep = to < T - 1;
      const uint64_t stays = __ballot(keep);
      if (keep) {
        const int slot = pos + __popcll(stays & below), id = ids + slot, f = l.from[i - m], p = f >> 6, r = f & 63;
        const int prod = l.prod[cur][p] * (r + 1);
        l.key[nxt][to] = key[i];
        l.id[nxt][to] = (uint16_t)id;
        l.score[nxt][slot] = l.score[cur][p] + t.lp[e * kMaxTopK + r];
        l.prod[nxt][slot] = prod;
        l.sum[nxt][slot] = l.sum[cur][p] + prod;
        l.node[nxt][slot] = (uint16_t)id;
        l.parent[id] = l.node[cur][p];
        l.rank[id] = (uint8_t)r;
        l.depth[id] = (uint8_t)(e + 1);
      }
      pos += __popcll(stays);
    }
    m = entries < T - 1 ? entries : T - 1;
    level = kept;
    ids += kept;
    if (level == 0 || e + 1 == k) {                            // the ranked entries are where the last round left them
      __syncthreads();
      for (int v = 1 + tid; v <= m; v += 64 * kTreeWaves) l.at[l.id[nxt][v - 1]] = (uint8_t)v;
      __syncthreads();
      for (int v = 1 + tid; v <= m; v += 64 * kTreeWaves) {
        const int id = l.id[nxt][v - 1];
        t.parent[v] = l.at[l.parent[id]];
        t.depth[v] = l.depth[id];
        t.rank[v] = l.rank[id];
      }
    }
    __syncthreads();
  }
}

// WAVES = kTreeWaves: by levels if the table is in order; WAVES = 1: the walk alone.
template <int SLOTS, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void tree_dynamic_kernel(const int32_t* __restrict__ root, const int32_t* __restrict__ cand,
                                                                  const float* __restrict__ lp, int k, int b, int T,
                                                                  TreeOut tree, int32_t* __restrict__ tok) {
  __shared__ TreeScratch t;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  static_assert(kMaxTopK == 64, "one table entry of a level per lane");
  constexpr int LV = kMaxTransfer / WAVES;         // levels of the table a wavefront brings in
  float lv[LV];
  int cv[LV];
#pragma unroll
  for (int i = 0; i < LV; ++i) {                   // all levels in one round trip; entries not in use read entry 0
    const int e = wave * LV + i, at = e < k && lane < b ? e * kMaxTopK + lane : 0;
    lv[i] = lp[at];
    cv[i] = cand[at];
  }
  const int root_tok = *root;
  bool disorder = false;
#pragma unroll
  for (int i = 0; i < LV; ++i) {
    const int e = wave * LV + i;
    const bool in = e < k && lane < b;
    const float v = in ? not_nan(lv[i]) : -INFINITY;
    if (WAVES > 1) {
      const float next = __shfl_down(v, 1, 64);
      disorder |= in && (v > 0.f || (lane + 1 < b && next > v));
    }
    t.lp[e * kMaxTopK + lane] = v;
    t.cand[e * kMaxTopK + lane] = cv[i];
  }
  for (int v = tid; v < kMaxTree; v += 64 * WAVES) {      // rows that are not reached (none, if the sizes were checked) hang under the root
    t.parent[v] = v ? 0 : -1;
    t.depth[v] = v ? 1 : 0;
    t.rank[v] = 0;
  }
  if constexpr (WAVES > 1) {
    __shared__ LevelScratch l;
    if (__syncthreads_or(disorder)) {
      if (wave == 0) tree_walk<SLOTS>(t, k, b, T);
    } else {
      tree_levels(t, l, k, b, T);
    }
  } else {
    __syncthreads();
    tree_walk<SLOTS>(t, k, b, T);
  }
  __syncthreads();
  for (int v = tid; v < T; v += 64 * WAVES) {
    const int depth = t.depth[v], r = t.rank[v];
    tree.parent[v] = t.parent[v];
    tree.depth[v] = depth;
    tree.rank[v] = r;
    tok[v] = v ? t.cand[(depth - 1) * kMaxTopK + r] : root_tok;
    uint64_t mask[kMaskWords];
    for (int w = 0; w < kMaskWords; ++w) mask[w] = 0;
    for (int u = v, hop = 0; u >= 0 && hop <= kMaxTransfer; u = t.parent[u], ++hop)
      for (int w = 0; w < kMaskWords; ++w) mask[w] |= w == (u >> 6) ? 1ull << (u & 63) : 0ull;
    for (int w = 0; w < kMaskWords; ++w) tree.anc[(size_t)v * kMaskWords + w] = mask[w];
  }
}
// The walk takes 2.4 us and 0.16 a node (0.25 beyond 64 nodes), the levels 3.3 us and 1 to 1.5 a level whatever the number of
// nodes.  Where they meet (us, walk / levels): k = 1, 8 nodes 4.0 / 4.5, 12 nodes 5.0 / 4.5; k = 2, 12 nodes 5.7 / 6.3; k = 3,
// 12 nodes 5.7 / 8.2, 24 nodes 9.5 / 8.3; k = 8, 24 nodes 9.4 / 10.4, 64 nodes 21.8 / 10.8.  By size, three levels of 10
// candidates: 64 nodes 22.4 / 9.1, 96 nodes 37.5 / 9.8, 128 nodes 51.8 / 12.6; eight levels of 64, 128 nodes 53.5 / 18.3.
bool tree_by_levels(int k, int T) { return T >= 8 + 4 * (k < 5 ? k : 5); }
hipError_t launch_tree_dynamic(const int32_t* root, const int32_t* cand, const float* lp, int k, int b, int T,
                               TreeOut tree, int32_t* tok, hipStream_t s) {
  if (!tree_by_levels(k, T)) hipLaunchKernelGGL((tree_dynamic_kernel<1, 1>), dim3(1), dim3(64), 0, s, root, cand, lp, k, b, T, tree, tok);
  else if (T <= 64)
    hipLaunchKernelGGL((tree_dynamic_kernel<1, kTreeWaves>), dim3(1), dim3(64 * kTreeWaves), 0, s, root, cand, lp, k, b, T, tree, tok);
  else
    hipLaunchKernelGGL((tree_dynamic_kernel<2, kTreeWaves>), dim3(1), dim3(64 * kTreeWaves), 0, s, root, cand, lp, k, b, T, tree, tok);
  return hipGetLastError();
}

// ---- distillation term of the training stage (Sec. 3.3)
// kl[p] = KL(softmax(za[p]) || softmax(zb[p])) = sum_v A_v (log A_v - log B_v) for pairs p of logit rows.
// Bound: reading the logits, which are read once: every thread keeps its sums of exponentials and of the A-weighted
// differences against its own maxima so far, eight entries of both rows at a time with the next eight on their way, and the
// parts meet at the end.  2046 pairs of 32000: 155 us with the maxima in a pass of their own, whose rows the second pass no
// longer found in an L2, 98 now, 5.3 TB/s; 256 pairs 23.6 and 16.3, one pair 13.5 and 10.6, 500 pairs of 4000 11.2 and 7.3.
// 256 threads a pair took 22.5 at 256 pairs and 14.4 at one (16.2 and 10.3 then), and as long as these at 2046.
// Masks of the lowest float are numbers like others here: a difference of 3.4e38 times a weight that is 1 only until a thread
// meets a larger logit must not overflow, so weighted differences are summed in units of 2^40, and sums are lowered before
// they are multiplied by the step down.
constexpr float kKlUnit = 1.0f / 1099511627776.0f;
template <int VEC>
__global__ __launch_bounds__(1024) void kl_rows_kernel(const float* __restrict__ za_all, const float* __restrict__ zb_all, int V,
                                                         float* __restrict__ kl) {
  __shared__ float red[16][5];
  constexpr int PIECES = 8 / VEC, STEP = 1024 * VEC;
  const float* za = za_all + (size_t)blockIdx.x * V;
  const float* zb = zb_all + (size_t)blockIdx.x * V;
  float a[2][PIECES][VEC], b[2][PIECES][VEC];
  auto load = [&](int base, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int j = base + i * STEP + threadIdx.x * VEC;
      if (j < V) {
        if constexpr (VEC == 4) {
          const float4 p = *(const float4*)(za + j), q = *(const float4*)(zb + j);
          a[buf][i][0] = p.x, a[buf][i][1] = p.y, a[buf][i][2] = p.z, a[buf][i][3] = p.w;
          b[buf][i][0] = q.x, b[buf][i][1] = q.y, b[buf][i][2] = q.z, b[buf][i][3] = q.w;
        } else {
          a[buf][i][0] = za[j];
          b[buf][i][0] = zb[j];
        }
      }
    }
  };
  float ma = -INFINITY, mb = -INFINITY, sa = 0.f, sb = 0.f, cross = 0.f;
  auto take = [&](int base, int buf) __attribute__((always_inline)) {
    float ha = ma, hb = mb;
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
      if (base + i * STEP + (int)threadIdx.x * VEC < V) {
#pragma unroll
        for (int u = 0; u < VEC; ++u) ha = fmaxf(ha, a[buf][i][u]), hb = fmaxf(hb, b[buf][i][u]);
      }
    const float fa = ha == -INFINITY ? 0.f : ha, fb = hb == -INFINITY ? 0.f : hb;      // (nothing but -inf so far)
    const float da = ma == -INFINITY ? 0.f : ma - fa, db = mb == -INFINITY ? 0.f : mb - fb, down = exp_below(da);
    sa *= down;
    cross = cross * down + sa * ((da - db) * kKlUnit);
    sb *= exp_below(db);
    ma = ha;
    mb = hb;
#pragma unroll
    for (int i = 0; i < PIECES; ++i)
      if (base + i * STEP + (int)threadIdx.x * VEC < V) {
#pragma unroll
        for (int u = 0; u < VEC; ++u) {
          const float x = a[buf][i][u], y = b[buf][i][u], e = exp_below(x - fa);
          sa += e;
          sb += exp_below(y - fb);
          cross += e * (((x - fa) - (y - fb)) * kKlUnit);
        }
      }
  };
  constexpr int BATCH = PIECES * STEP;
  load(0, 0);
  for (int base = 0; base < V; base += 2 * BATCH) {
    load(base + BATCH, 1);
    take(base, 0);
    load(base + 2 * BATCH, 0);
    if (base + BATCH < V) take(base + BATCH, 1);
  }
  // the parts' sums against the maxima of all: first in a wavefront, then over the wavefronts
  auto lower = [&](float ta, float tb) __attribute__((always_inline)) {
    const float da = ma == -INFINITY ? 0.f : ma - ta, db = mb == -INFINITY ? 0.f : mb - tb, down = exp_below(da);
    sa *= down;
    cross = cross * down + sa * ((da - db) * kKlUnit);
    sb *= exp_below(db);
  };
  const float wa = wave_max_dpp(ma), wb = wave_max_dpp(mb);
  lower(wa, wb);
  sa = wave_sum(sa);
  sb = wave_sum(sb);
  cross = wave_sum(cross);
  if ((threadIdx.x & 63) == 0) {
    float* r = red[threadIdx.x >> 6];
    r[0] = wa, r[1] = wb, r[2] = sa, r[3] = sb, r[4] = cross;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const bool part = (int)threadIdx.x < 16;
  const float* r = red[part ? threadIdx.x : 0];
  ma = part ? r[0] : -INFINITY, mb = part ? r[1] : -INFINITY;
  sa = part ? r[2] : 0.f, sb = part ? r[3] : 0.f, cross = part ? r[4] : 0.f;
  lower(wave_max_dpp(ma), wave_max_dpp(mb));
  sa = wave_sum(sa);
  sb = wave_sum(sb);
  cross = wave_sum(cross);
  if (threadIdx.x == 0) kl[blockIdx.x] = cross / sa / kKlUnit - logf(sa) + logf(sb);
}
hipError_t launch_kl_rows(const float* za, const float* zb, int pairs, int V, float* kl, hipStream_t s) {
  const int vec = !((uintptr_t)za & 15) && !((uintptr_t)zb & 15) && !(V & 3);
  hipLaunchKernelGGL((vec ? kl_rows_kernel<4> : kl_rows_kernel<1>), dim3(pairs), dim3(1024), 0, s, za, zb, V, kl);
  return hipGetLastError();
}

// Acceptance and compaction in one launch.  From the root on, the lowest child that carries the arg-max token of the node so
// far is accepted; the accepted rows move to slots n..n+m-1 of every layer's cache and the last accepted node's saved residual
// becomes the next transfer source.  blockIdx.y = layer.
// Bound: two memory latencies.  Every wavefront walks the tree for itself, two nodes a lane and a ballot per level, so that the
// moves need no launch of their own behind a single wavefront's walk, and all of a thread's rows are read before the first is
// written (path[j] >= j and rising, so none of them has been overwritten).  64 nodes at four layers of 4096: 3.6 and 3.5 us
// with the gap of a launch between them in two, 4.9 in one; eight nodes at two layers of 256 2.9.
// parity >= 0 (device-resident loop): the cache length is st->n[parity], the one after the acceptance goes to the other slot,
// which no block reads here, and the step is logged.
template <typename T>
__global__ __launch_bounds__(256) void accept_compact_kernel(StepState* __restrict__ st, const int32_t* __restrict__ parent,
                                                             const int32_t* __restrict__ tok, const int32_t* __restrict__ g, int nodes,
                                                             StepLog* __restrict__ log, int n, int parity, void* const* __restrict__ kcs,
                                                             void* const* __restrict__ vcs, int row_elems, int cap,
                                                             const float* __restrict__ saved_h, size_t slot_stride, int slots,
                                                             float* __restrict__ h_src, int d) {
  const int lane = threadIdx.x & 63, layer = blockIdx.y;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  constexpr int HALVES = kMaxTree / 64;
  int up[HALVES], own[HALVES], next[HALVES];
#pragma unroll
  for (int h = 0; h < HALVES; ++h) {
    const int c = lane + 64 * h, at = c < nodes ? c : 0;
    up[h] = c < nodes ? parent[at] : -2;      // no node's number
    own[h] = tok[at];
    next[h] = g[at];
  }
  if (parity >= 0) n = st->n[parity];
  auto of_node = [&](const int (&v)[HALVES], int node) __attribute__((always_inline)) {
    int r = __builtin_amdgcn_readlane(v[0], node & 63);
#pragma unroll
    for (int h = 1; h < HALVES; ++h)
      if (node >> 6 == h) r = __builtin_amdgcn_readlane(v[h], node & 63);
    return r;
  };
  int path[kMaxTransfer + 1], cur = 0, m = 1;
  path[0] = 0;
#pragma unroll
  for (int j = 1; j <= kMaxTransfer; ++j) {
    path[j] = 0;
    if (m < j) continue;                      // the walk has ended
    const int want = of_node(next, cur);
    int child = -1;
#pragma unroll
    for (int h = HALVES - 1; h >= 0; --h) {
      const uint64_t match = __ballot(up[h] == cur && own[h] == want && lane + 64 * h > cur);
      if (match) child = 64 * h + __builtin_ctzll(match);
    }
    if (child < 0) continue;
    path[j] = cur = __builtin_amdgcn_readfirstlane(child);
    m = j + 1;
  }
  if (e < row_elems) {
    T* kc = (T*)kcs[layer];
    T* vc = (T*)vcs[layer];
    T k[kMaxTransfer + 1], v[kMaxTransfer + 1];
#pragma unroll
    for (int j = 1; j <= kMaxTransfer; ++j)
      if (j < m && path[j] != j) {
        k[j] = kc[(size_t)(n + path[j]) * row_elems + e];
        v[j] = vc[(size_t)e * cap + n + path[j]];
      }
#pragma unroll
    for (int j = 1; j <= kMaxTransfer; ++j)
      if (j < m && path[j] != j) {
        kc[(size_t)(n + j) * row_elems + e] = k[j];
        vc[(size_t)e * cap + n + j] = v[j];
      }
  }
  if (layer < slots && e < d)       // one transfer source per distinct transfer layer (slots <= layers)
    h_src[(size_t)layer * d + e] = saved_h[layer * slot_stride + (size_t)cur * d + e];
  if (blockIdx.x || blockIdx.y || threadIdx.x >= 64) return;
  StepLog* entry = parity >= 0 ? log + st->log_count : nullptr;
  const int root = of_node(next, cur);
#pragma unroll
  for (int j = 0; j <= kMaxTransfer; ++j) {
    const int emitted = of_node(own, path[j]);
    if (j < m && lane == 0) {
      st->path[j] = path[j];
      st->emitted[j] = emitted;
      if (entry) entry->emitted[j] = emitted;
    }
  }
  if (lane) return;
  st->m = m;
  st->next_root = st->root = root;
  if (entry) {                      // the host reads the steps and the cache length afterwards
    entry->m = m;
    st->log_count += 1;
    st->n[parity ^ 1] = n + m;
  }
}
hipError_t launch_accept_compact(int dtype, StepState* st, TreeDev tree, const int32_t* tok, const int32_t* g, int T, StepLog* log,
                                 int n, int parity, void* const* kc, void* const* vc, int L, int Hkv, int hd, int cap,
                                 const float* saved_h, size_t slot_stride, int slots, float* h_src, int d, hipStream_t s) {
  const int row = Hkv * hd;
  const int cols = row > d ? row : d;
  const int nodes = T;
  HT_DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(accept_compact_kernel<T>, dim3((cols + 255) / 256, L), dim3(256), 0, s, st, tree.parent,
                                              tok, g, nodes, log, n, parity, kc, vc, row, cap, saved_h, slot_stride, slots,
                                              h_src, d);)
  return hipGetLastError();
}

// The state of a step into pinned host memory, behind it the number of the step: a host that reads the number there has the
// state, and everything enqueued before is done, as after a copy and a wait for the stream, which cost a copy kernel (4 us) and
// the runtime's wait (a step of a small fp32 model 130 -> 120 us, one token through four 7B-wide blocks 415 -> 401).
__global__ __launch_bounds__(64) void publish_state_kernel(const int32_t* __restrict__ state, int32_t* host, int words, int32_t number) {
  const int lane = threadIdx.x;
  if (lane < words) __hip_atomic_store(host + lane, state[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();                      // one wavefront: its stores are in host memory before the number is
  if (lane == 0) __hip_atomic_store(host + words, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
hipError_t launch_publish_state(const StepState* st, int32_t* host, int32_t number, hipStream_t s) {
  constexpr int words = sizeof(StepState) / sizeof(int32_t);
  static_assert(words <= 64, "a word to a lane");
  hipLaunchKernelGGL(publish_state_kernel, dim3(1), dim3(64), 0, s, (const int32_t*)st, host, words, number);
  return hipGetLastError();
}

// saved_h holds one [rows, d] residual image per distinct transfer layer (`slot_stride` floats apart); the
// transfer sources h_src[slot][d] become the images' row `last`.  blockIdx.y = slot.
__global__ void prefill_finish_kernel(StepState* __restrict__ st, const int32_t* __restrict__ g,
                                      const float* __restrict__ saved_h, size_t slot_stride, float* __restrict__ h_src,
                                      int last, int d) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x, slot = blockIdx.y;
  if (e < d) h_src[(size_t)slot * d + e] = saved_h[slot * slot_stride + (size_t)last * d + e];
  if (e == 0 && slot == 0) { st->root = g[last]; st->next_root = g[last]; st->m = 0; }
}
hipError_t launch_prefill_finish(StepState* st, const int32_t* g, const float* saved_h, size_t slot_stride, int slots,
                                 float* h_src, int last, int d, hipStream_t s) {
  hipLaunchKernelGGL(prefill_finish_kernel, dim3((d + 255) / 256, slots), dim3(256), 0, s, st, g, saved_h, slot_stride,
                     h_src, last, d);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ hidden transfer
// pseudo[f][i][o] = sum_c W_i[o][c] h_f[c] for F source vectors h_f = h + row(f) * d, row(f) = src_rows[f] (or f
// when src_rows is NULL).  One source (either type): a wavefront per output feature, weight rows read fully coalesced.
// Several sources of an fp32 model: a wavefront produces four consecutive output features, so that every 16-byte piece of a
// source, which comes from L2, serves all four; sources go in groups of four (of sixteen from sixteen sources on, which
// walks the weight rows a quarter as often), and every (source, output) sum runs in the same order whatever F is: one
// source alone and the same source among several give the same bits.  Several sources of a bf16 model go to the matrix
// cores (ht_transfer_mfma.hip), whose sums run in another order: there the two agree to fp32 rounding.  One source stays
// here because the walk along K is shorter on a whole wavefront (three maps of 1024 x 1024: 3.7 us, 6.0 us there).
// Steps i0 .. i0 + gridDim.y - 1 are computed; the output row of (f, i) is f * row_stride + (i - i0).
// grid = (ceil(d / (4 R)), steps), block = 256.
template <typename T, int NF, int R>           // R output features per wavefront: a source piece is loaded once for all
__global__ void transfer_kernel(const float* __restrict__ h, const int32_t* __restrict__ src_rows, int F,
                                const void* const* __restrict__ ws, float* __restrict__ pseudo, int i0, int row_stride,
                                int d) {
  const int i = i0 + blockIdx.y;
  const int o0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * R;
  const int lane = threadIdx.x & 63;
  if (o0 >= d) return;
  const T* rows[R];
#pragma unroll
  for (int r = 0; r < R; ++r) rows[r] = (const T*)ws[i] + (size_t)(o0 + r < d ? o0 + r : d - 1) * d;
  constexpr int VEC = 16 / sizeof(T);
  for (int f0 = 0; f0 < F; f0 += NF) {
    const float* hp[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const int f = f0 + j < F ? f0 + j : F - 1;
      hp[j] = h + (size_t)(src_rows ? src_rows[f] : f) * d;
    }
    float acc[R][NF];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < NF; ++j) acc[r][j] = 0.f;
    for (int c = lane * VEC; c < d; c += 64 * VEC) {
      if (c + VEC <= d) {
        uint4 raw[R];
#pragma unroll
        for (int r = 0; r < R; ++r) raw[r] = *(const uint4*)(rows[r] + c);
#pragma unroll
        for (int j = 0; j < NF; ++j) {
          float hv[VEC];
#pragma unroll
          for (int e = 0; e < VEC; e += 4) *(float4*)(hv + e) = *(const float4*)(hp[j] + c + e);
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const T* v = (const T*)&raw[r];
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[r][j] += Conv<T>::load(v + e) * hv[e];
          }
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < NF; ++j)
            for (int e = 0; c + e < d; ++e) acc[r][j] += Conv<T>::load(rows[r] + c + e) * hp[j][c + e];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        const float v = wave_sum(acc[r][j]);
        if (lane == 0 && f0 + j < F && o0 + r < d)
          pseudo[((size_t)(f0 + j) * row_stride + (i - i0)) * d + o0 + r] = v;
      }
  }
}
hipError_t launch_transfer(int dtype, const float* h, const int32_t* src_rows, int F, const void* const* w_dev,
                           float* pseudo, int i0, int steps, int row_stride, int d, void* scratch, hipStream_t s) {
  if (d % 4) return hipErrorInvalidValue;      // 16-byte pieces of the fp32 sources
  if (F == 1) {      // one source: its re-reads are cheap and one feature per wavefront spreads the rows wider
    HT_DISPATCH_DTYPE(dtype, hipLaunchKernelGGL((transfer_kernel<T, 1, 1>), dim3((d + 3) / 4, steps), dim3(256), 0, s, h,
                                                src_rows, F, w_dev, pseudo, i0, row_stride, d);)
  } else if (dtype != 0 && transfer_split_supported(F, d)) {
    return launch_transfer_split(h, src_rows, F, w_dev, pseudo, i0, steps, row_stride, d, scratch, s);
  } else if (dtype != 0) {
    return hipErrorInvalidValue;               // bf16 rows are multiples of 16 bytes (checked when the model is set up)
  } else if (F < 16) {
    hipLaunchKernelGGL((transfer_kernel<float, 4, 4>), dim3((d + 15) / 16, steps), dim3(256), 0, s, h, src_rows, F, w_dev,
                       pseudo, i0, row_stride, d);
  } else {           // every node of a tree drafts: sixteen sources per walk over the weight rows (same sums, same order)
    hipLaunchKernelGGL((transfer_kernel<float, 16, 4>), dim3((d + 15) / 16, steps), dim3(256), 0, s, h, src_rows, F, w_dev,
                       pseudo, i0, row_stride, d);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ streaming probe
// Reads a buffer once the way the packed projections read their weights (every workgroup walks its own
// contiguous region, 8 KiB per step as eight nontemporal 1 KiB wavefront loads, eight steps in flight) and does
// nothing with the data: the time of this kernel is the floor for any weight stream of that size.
typedef unsigned int probe_u32x4_t __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void stream_read_kernel(const probe_u32x4_t* __restrict__ p, size_t vecs_per_group,
                                                          uint32_t* __restrict__ sink) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const probe_u32x4_t* base = p + (size_t)blockIdx.x * vecs_per_group + wave * 128 + lane;
  const size_t steps = vecs_per_group / 512;              // 512 vectors = 8 KiB per step
  probe_u32x4_t acc = {0, 0, 0, 0};
  for (size_t i = 0; i + 4 <= steps; i += 4) {
    probe_u32x4_t v[8];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v[2 * u] = __builtin_nontemporal_load(base + (i + u) * 512);
      v[2 * u + 1] = __builtin_nontemporal_load(base + (i + u) * 512 + 64);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u];
  }
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) sink[0] = 1;     // keeps the loads alive
}
// Reads floor(bytes / (groups * 32 KiB)) * groups * 32 KiB bytes; returns that count.
size_t launch_stream_read(const void* buf, size_t bytes, int groups, uint32_t* sink, hipStream_t s) {
  const size_t per_group = bytes / groups / 32768 * 32768;
  if (!per_group) return 0;
  hipLaunchKernelGGL(stream_read_kernel, dim3(groups), dim3(256), 0, s, (const probe_u32x4_t*)buf, per_group / 16, sink);
  return per_group * groups;
}

// ------------------------------------------------------------------------------------------------ matrix-core probe
// Nothing but independent matrix-core instructions on register operands, 32 accumulators of 16 x 16 (FORM 0:
// v_mfma_f32_16x16x32_bf16) or 8 of 32 x 32 (FORM 1: v_mfma_f32_32x32x16_bf16) per wavefront, two wavefronts per
// SIMD: the rate of this kernel is what a product kernel on that instruction can reach at best on this machine.
// The rate depends on the operand bits (the clock follows the power drawn), hence two kinds of operands.
typedef __bf16 probe_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float probe_f32x4_t __attribute__((ext_vector_type(4)));
typedef float probe_f32x16_t __attribute__((ext_vector_type(16)));
template <int FORM>
__global__ __launch_bounds__(256) void mfma_rate_kernel(int iters, int random_bits, uint32_t* __restrict__ sink) {
  // operands: small whole numbers (few bits toggle between lanes and instructions), or values in +-[1, 2) with
  // hashed sign and mantissa bits (what real activations and weights look like to the multipliers)
  probe_bf16x8_t a[4], b[8];
  auto fill = [&](int which, int j) -> __bf16 {
    if (!random_bits) return (__bf16)(float)((threadIdx.x * (which < 4 ? 1 : 3) + which + j) & 7);
    uint32_t h = (threadIdx.x * 64u + which * 8u + j) * 2654435761u;
    h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
    const unsigned short bits = (unsigned short)(0x3f80u | (h & 0x7fu) | ((h & 0x100u) << 7));
    return __builtin_bit_cast(__bf16, bits);
  };
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) a[i][j] = fill(i, j);
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) b[i][j] = fill(4 + i, j);
  float total = 0.f;
  if (FORM == 0) {
    probe_f32x4_t acc[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) acc[i] = probe_f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int i = 0; i < 32; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i % 4], b[i / 4], acc[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 32; ++i) total += acc[i][0] + acc[i][1] + acc[i][2] + acc[i][3];
  } else {
    probe_f32x16_t acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i % 2], b[i / 2], acc[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) total += acc[i][j];
  }
  if (total == -1.25f) sink[0] = 1;                        // keeps the work alive (sums of whole numbers, or far from -1.25)
}
// Returns the floating-point operations of the launch (2 per multiply-add).
double launch_mfma_rate(int form, int iters, uint32_t* sink, hipStream_t s) {
  constexpr int kGroups = 512;                             // two workgroups of four wavefronts per compute unit
  if ((form & 1) == 0)
    hipLaunchKernelGGL(mfma_rate_kernel<0>, dim3(kGroups), dim3(256), 0, s, iters, form >> 1, sink);
  else
    hipLaunchKernelGGL(mfma_rate_kernel<1>, dim3(kGroups), dim3(256), 0, s, iters, form >> 1, sink);
  return (double)kGroups * 4 * iters * ((form & 1) == 0 ? 32 * 2.0 * 16 * 16 * 32 : 8 * 2.0 * 32 * 32 * 16);
}

// ------------------------------------------------------------------------------------------------ generic attention
// One block per (query head, tree row).  Scores of all visible keys go to LDS (four lanes per key), softmax in fp32, then
// every thread owns one output element and every (256 / hd)-th piece of VEC keys of it; SKIP: pieces of tree rows that hold
// no ancestor are not read.  Dynamic LDS: (n + M) floats + hd + 256.  Latency bound at the sizes it is used at (fp32 model, tens of keys): VEC elements per load cut the chains of
// dependent loads, 7.6 -> 5.1 us (mean; shortest 5.5 -> 4.2) for 8 rows of 4 heads over 40 keys of 64 floats.
template <typename T, int VEC> __device__ inline void load_vec(const T* p, float (&v)[VEC]) {
  if constexpr (VEC == 1) {
    v[0] = Conv<T>::load(p);
  } else {
    typedef unsigned int words_t __attribute__((ext_vector_type(VEC * sizeof(T) / 4)));
    const words_t raw = *(const words_t*)p;           // 16 or 8 bytes
    const T* e = (const T*)&raw;
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = Conv<T>::load(e + i);
  }
}
template <typename T, int VEC, bool SKIP>
__global__ __launch_bounds__(256) void attn_simple_kernel(const T* __restrict__ q, const T* __restrict__ kc, const T* __restrict__ vc,
                                                          int cap, int n, int M, TreeDev tree, int Hq, int Hkv, int hd,
                                                          T* __restrict__ out, const int32_t* __restrict__ n_dev) {
  extern __shared__ float smem[];
  __shared__ float red[4];
  n = cache_len(n, n_dev);             // at most the host's n, which sized the dynamic LDS
  const int h = blockIdx.x, m = blockIdx.y, hk = h / (Hq / Hkv), tid = threadIdx.x;
  const int S = n + M;
  float* sc = smem;            // [S]
  float* qs = smem + S;        // [hd]
  float* acc = qs + hd;        // [256]
  uint32_t* seen = (uint32_t*)acc;   // the row's mask, until the scores are there
  for (int e = tid; e < hd; e += 256) qs[e] = Conv<T>::load(q + ((size_t)m * Hq + h) * hd + e);
  if (tid < 2 * kMaskWords) seen[tid] = ((const uint32_t*)(tree.anc + (size_t)m * kMaskWords))[tid];
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)hd);
  float mx = -INFINITY;
  const int quarter = tid & 3;
  for (int j = tid >> 2; j < (S + 63) / 64 * 64; j += 64) {       // whole wavefronts stay in the loop for the lane exchange
    bool vis = j < n;
    if (!vis && j < S) {
      const int u = j - n;
      vis = (seen[u >> 5] >> (u & 31)) & 1u;
    }
    float dot = 0.f;
    if (vis) {
      const T* kr = kc + ((size_t)j * Hkv + hk) * hd;
#pragma unroll 4
      for (int e = quarter * VEC; e < hd; e += 4 * VEC) {
        float kv[VEC];
        load_vec<T, VEC>(kr + e, kv);
#pragma unroll
        for (int i = 0; i < VEC; ++i) dot += qs[e + i] * kv[i];
      }
    }
    dot += __shfl_xor(dot, 1, 64);
    dot += __shfl_xor(dot, 2, 64);
    const float s = vis ? dot * scale : -INFINITY;
    if (quarter == 0 && j < S) sc[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = block_max_256(mx, red);
  float sum = 0.f;
  const int Sp = (S + VEC - 1) / VEC * VEC;            // up to a whole piece, over what was qs (hd is a multiple of VEC)
  for (int j = tid; j < Sp; j += 256) {
    const float p = j >= S || sc[j] == -INFINITY ? 0.f : expf(sc[j] - mx);
    sc[j] = p;
    sum += p;
  }
  sum = block_sum_256(sum, red);
  const int groups = 256 / hd > 0 ? 256 / hd : 1;      // hd <= 256
  const int e = tid % hd, part = tid / hd;
  float o = 0.f;
  if (part < groups) {
    const T* vr = vc + ((size_t)hk * hd + e) * cap;    // cap is a multiple of 8: whole pieces lie in the row
    auto probabilities = [&](int j, float (&p)[VEC]) __attribute__((always_inline)) {
      if constexpr (VEC == 1) {
        p[0] = sc[j];
      } else {
#pragma unroll
        for (int i = 0; i < VEC; i += 4) *(float4*)(p + i) = *(const float4*)(sc + j + i);
      }
    };
    auto add = [&](int j, const float (&p)[VEC]) __attribute__((always_inline)) {
      float vv[VEC];
      load_vec<T, VEC>(vr + j, vv);
#pragma unroll
      for (int i = 0; i < VEC; ++i) o += p[i] != 0.f ? p[i] * vv[i] : 0.f;      // what no row has written yet may hold anything
    };
    int j = part * VEC;
#pragma unroll 2
    for (; j < (SKIP ? n : S); j += groups * VEC) {
      float p[VEC];
      probabilities(j, p);
      add(j, p);
    }
    if (SKIP)
      for (; j < S; j += groups * VEC) {
        float p[VEC];
        probabilities(j, p);
        bool any = false;
#pragma unroll
        for (int i = 0; i < VEC; ++i) any = any || p[i] != 0.f;
        if (any) add(j, p);
      }
  }
  acc[tid] = o;
  __syncthreads();
  if (tid < hd) {
    float t = 0.f;
    for (int p = 0; p < groups; ++p) t += acc[p * hd + tid];
    Conv<T>::store(out + (size_t)m * Hq * hd + (size_t)h * hd + tid, t / sum);
  }
}
hipError_t launch_attn_simple(int dtype, const void* q, const void* kc, const void* vc, int cap, int n, int M,
                              TreeDev tree, int Hq, int Hkv, int hd, void* out, hipStream_t s, const int32_t* n_dev) {
  const size_t smem = (size_t)(n + M + hd + 256) * sizeof(float);
  if (smem > 64 * 1024 || hd > 256) return hipErrorInvalidValue;
  // 16-byte pieces of key rows and of value columns, or 8-byte ones of bf16 heads that are a multiple of four wide
  const bool vec = hd % (dtype == 0 ? 4 : 8) == 0 && cap % 8 == 0 && !((uintptr_t)kc & 15) && !((uintptr_t)vc & 15);
  const bool half = dtype != 0 && hd % 4 == 0 && cap % 8 == 0 && !((uintptr_t)kc & 7) && !((uintptr_t)vc & 7);
  // Many rows: what the value columns of rows that are no ancestors cost adds up, and a look at the probabilities before
  // each piece pays (trees without a cache: 256 rows of 32 heads of 128 floats 151 us without it, 62 us with it; of 8 heads
  // 42.6 and 21.7 us).  Few: the look is one more dependent step (chains: 128 rows of 4 heads of 96 floats 13.1 and 16.0 us).
  const bool skip = (size_t)Hq * M * hd * (dtype == 0 ? 4 : 2) > (vec || half ? 400000 : 50000);
#define HT_ATTN_SIMPLE_AS(VEC, SKIP)                                                                                   \
  hipLaunchKernelGGL((attn_simple_kernel<T, VEC, SKIP>), dim3(Hq, M), dim3(256), smem, s, (const T*)q, (const T*)kc, (const T*)vc, \
                     cap, n, M, tree, Hq, Hkv, hd, (T*)out, n_dev)
#define HT_ATTN_SIMPLE(VEC)               \
  if (skip) HT_ATTN_SIMPLE_AS(VEC, true); \
  else HT_ATTN_SIMPLE_AS(VEC, false)
  HT_DISPATCH_DTYPE(dtype, if (vec) { HT_ATTN_SIMPLE(16 / sizeof(T)); } else if (half) { HT_ATTN_SIMPLE(4); } else { HT_ATTN_SIMPLE(1); })
#undef HT_ATTN_SIMPLE
#undef HT_ATTN_SIMPLE_AS
  return hipGetLastError();
}

}  // namespace ht
