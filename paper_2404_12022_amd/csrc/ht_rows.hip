// Products of the models that do not run on the matrix cores: fp32 (every launch of the pass) and bf16 shapes that do not
// pack (the plain product).  Few rows, row-major weights read once: one wavefront per output feature (or per pair of
// features that meet in the epilogue), eight token rows at a time, 16 bytes per lane and load, all loads of two steps
// issued before the first use; the eight rows' sums are reduced together (a row ends in eight lanes: ten lane exchanges
// for eight sums instead of forty-eight).
//
// What bounds these launches at the sizes they are used at (widths of a few hundred) is latency: a launch cannot end
// faster than one round trip to L2 plus the reduction, so on fp32 models everything that was a launch of its own rides
// along.  The RMSNorm of the input rows: every wavefront reads whole rows anyway and adds up their squares beside the
// products, the 1/rms factor multiplies the finished sums, the gain multiplies the weights.  Rotary and K/V append: a
// wavefront owns the features j and j + hd/2 of a head.  SiLU(gate) * up: a wavefront owns gate and up row j.  The
// residual add: every output element has one owner, which adds to the residual stream itself.  Five launches per decoder
// block instead of nine.  At 256 x 256, 8 rows: 16.3 us (scalar loads, four rows a time) -> 2.7 us (shortest 2.2).
#include "ht_common.h"

namespace ht {

namespace {

// Sums of MR values over the wavefront, MR a power of two up to 8: lane l ends with the sum of value l / (64 / MR).  Halves and
// rows of sixteen change places in a lane swap, the rest are DPP moves: lane exchanges through LDS, six in a row, were a fifth
// of a launch.
// lower half of 2 DIST lanes: a there plus a DIST lanes on; upper half: the same of b
template <int DIST> __device__ inline float fold_pair(float a, float b) {
  if constexpr (DIST == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else if constexpr (DIST == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else {
    static_assert(DIST == 8, "");
    const bool upper = threadIdx.x & 8;
    const float keep = upper ? b : a, give = upper ? a : b;
    return keep + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(give), 0x128, 0xf, 0xf, true));
  }
}
template <int CTRL> __device__ inline float add_dpp(float v) {
  return v + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
template <int N, int DIST> __device__ inline void fold_rows(float* v) {
  if constexpr (N >= 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = fold_pair<DIST>(v[i], v[i + N]);
    fold_rows<N / 2, DIST / 2>(v);
  }
}
template <int MR> __device__ inline float reduce_rows(float (&v)[MR]) {
  fold_rows<MR / 2, 32>(v);
  float s = v[0];
  s = add_dpp<0xb1>(s);                        // lane ^ 1
  s = add_dpp<0x4e>(s);                        // lane ^ 2
  s = add_dpp<0x141>(s);                       // the other four of eight
  if (MR <= 4) s = add_dpp<0x140>(s);          // the other eight of sixteen
  if (MR <= 2) s = fold_pair<16>(s, s);
  if (MR <= 1) s = fold_pair<32>(s, s);
  return s;
}

template <typename T, int VEC> __device__ inline void load_piece(const T* p, float (&v)[VEC]) {
  if constexpr (VEC == 1) {
    v[0] = Conv<T>::load(p);
  } else {
    const uint4 raw = *(const uint4*)p;                    // VEC * sizeof(T) = 16
    const T* e = (const T*)&raw;
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = Conv<T>::load(e + i);
  }
}

template <typename T, int VEC, int EPI, int MR>
__global__ __launch_bounds__(256) void rows_kernel(const T* __restrict__ a, const T* __restrict__ gain, float eps, WeightSegs w,
                                                   int M, int units, int K, RowsEpilogue ep) {
  constexpr int NF = EPI == ROWS_SILU || EPI == ROWS_QKV ? 2 : 1;    // weight rows of a wavefront
  constexpr bool NORM = EPI == ROWS_SILU || EPI == ROWS_QKV || EPI == ROWS_STORE_NORM;
  constexpr int U = MR == 2 ? 4 : 2;                                 // steps of 64 VEC columns whose loads go out together
  const int unit = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (unit >= units) return;
  // weight rows of this wavefront
  const T *row0, *row1 = nullptr;
  int seg = 0, local = unit, head = 0, j = 0;
  if (EPI == ROWS_QKV) {
    const int half = ep.hd / 2;
    head = unit / half;                                              // over the Hq q heads, then k heads, then v heads
    j = unit - head * half;
    seg = head < ep.Hq ? 0 : head < ep.Hq + ep.Hkv ? 1 : 2;
    const int h = seg == 0 ? head : seg == 1 ? head - ep.Hq : head - ep.Hq - ep.Hkv;
    head = h;
    row0 = (const T*)(seg == 0 ? w.w[0] : seg == 1 ? w.w[1] : w.w[2]) + ((size_t)h * ep.hd + j) * K;
    row1 = row0 + (size_t)half * K;
  } else if (EPI == ROWS_SILU) {
    row0 = (const T*)w.w[0] + (size_t)unit * K;
    row1 = (const T*)w.w[1] + (size_t)unit * K;
  } else {
    while (seg + 1 < w.nseg && local >= w.rows[seg]) { local -= w.rows[seg]; ++seg; }
    row0 = (const T*)w.w[seg] + (size_t)local * K;
  }
  for (int m0 = blockIdx.y * MR; m0 < M; m0 += gridDim.y * MR) {
    float acc[NF][MR], ss[MR];
#pragma unroll
    for (int r = 0; r < MR; ++r) {
      ss[r] = 0.f;
#pragma unroll
      for (int f = 0; f < NF; ++f) acc[f][r] = 0.f;
    }
    // what the epilogue reads is requested with the operands: a round trip less at the end (256-wide block, with the sums above: q|k|v
    // 4.20 -> 4.01 us, residual add 3.57 -> 3.29, SiLU 4.51 -> 4.32)
    const int m = m0 + lane / (64 / MR), mc = m < M ? m : M - 1;       // the row whose sum this lane ends with
    float2 turn = make_float2(0.f, 0.f);
    float before = 0.f;
    if (EPI == ROWS_QKV && seg != 2) turn = *(const float2*)(ep.cs + ((size_t)mc * (ep.hd / 2) + j) * 2);
    if (EPI == ROWS_ADD) before = ep.out[(size_t)mc * units + unit];
    for (int c0 = lane * VEC; c0 < K; c0 += U * 64 * VEC) {
      float wv[U][NF][VEC], av[U][MR][VEC], gv[U][VEC];
#pragma unroll
      for (int s = 0; s < U; ++s) {
        const int c = c0 + s * 64 * VEC;
        const bool in = c < K;                                       // K is a multiple of VEC
        const int cc = in ? c : c0;
#pragma unroll
        for (int f = 0; f < NF; ++f) load_piece<T, VEC>((f ? row1 : row0) + cc, wv[s][f]);
        if (NORM) load_piece<T, VEC>(gain + cc, gv[s]);
#pragma unroll
        for (int r = 0; r < MR; ++r) {
          const int m = m0 + r < M ? m0 + r : M - 1;
          load_piece<T, VEC>(a + (size_t)m * K + cc, av[s][r]);
        }
      }
#pragma unroll
      for (int s = 0; s < U; ++s) {
        if (c0 + s * 64 * VEC >= K) continue;
#pragma unroll
        for (int e = 0; e < VEC; ++e)
#pragma unroll
          for (int r = 0; r < MR; ++r) {
            const float x = av[s][r][e];
            if (NORM) ss[r] += x * x;
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[f][r] += (NORM ? wv[s][f][e] * gv[s][e] : wv[s][f][e]) * x;
          }
      }
    }
    float v[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) v[f] = reduce_rows<MR>(acc[f]);
    float scale = 1.f;
    if (NORM) scale = 1.0f / sqrtf(reduce_rows<MR>(ss) / (float)K + eps);
    if (lane % (64 / MR) || m >= M) continue;                        // one lane of a row's group stores
    if (EPI == ROWS_STORE) {
      ep.out[(size_t)m * units + unit] = v[0];
    } else if (EPI == ROWS_STORE_NORM) {
      ep.out[(size_t)m * units + unit] = v[0] * scale;
    } else if (EPI == ROWS_ADD) {
      const size_t i = (size_t)m * units + unit;
      const float x = before + v[0];
      ep.out[i] = x;
      if (ep.save) ep.save[i] = x;
    } else if (EPI == ROWS_SILU) {
      const float g = v[0] * scale, up = v[NF - 1] * scale;
      ep.out[(size_t)m * units + unit] = g / (1.0f + expf(-g)) * up;
    } else {
      const int half = ep.hd / 2, n = cache_len(ep.n, ep.n_dev);
      const float x = v[0] * scale, y = v[NF - 1] * scale;
      if (seg == 2) {
        float* col = ep.vc + ((size_t)head * ep.hd + j) * ep.cap + n + m;
        col[0] = x;
        col[(size_t)half * ep.cap] = y;
      } else {
        const float co = turn.x, si = turn.y;
        float* dst = seg == 0 ? ep.q + ((size_t)m * ep.Hq + head) * ep.hd + j
                              : ep.kc + ((size_t)(n + m) * ep.Hkv + head) * ep.hd + j;
        dst[0] = x * co - y * si;
        dst[half] = y * co + x * si;
      }
    }
  }
}

template <typename T, int VEC, int EPI>
void launch_rows_as(const void* a, const void* gain, float eps, const WeightSegs& w, int M, int units, int K,
                    const RowsEpilogue& ep, hipStream_t s) {
  // Rows per workgroup.  While the chip is short of work (1024 workgroups are four per compute unit) few rows on many
  // workgroups end soonest (256 x 256, 8 rows: 2.7 us at two rows each, 4.5 us at eight on a quarter of the workgroups);
  // beyond that eight, which read the weights a quarter as often, and the workgroup that has the weight rows at hand
  // takes the next eight.
  const int bx = (units + 3) / 4;
  auto fits = [&](int mr) { return (long)bx * ((M + mr - 1) / mr) <= 1024; };
#define HT_ROWS_AS(MR, GY)                                                                                                   \
  hipLaunchKernelGGL((rows_kernel<T, VEC, EPI, MR>), dim3(bx, GY), dim3(256), 0, s, (const T*)a, (const T*)gain, eps, w, M, units, \
                     K, ep)
  if (M <= 2 || fits(2)) HT_ROWS_AS(2, (M + 1) / 2);
  else if (M <= 4 || fits(4)) HT_ROWS_AS(4, (M + 3) / 4);
  else HT_ROWS_AS(8, (M + 7) / 8 < 1024 / bx ? (M + 7) / 8 : 1024 / bx > 1 ? 1024 / bx : 1);
#undef HT_ROWS_AS
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

// 16-byte loads need 16-byte rows: K a multiple of 16 / sizeof(T) and aligned bases.
hipError_t launch_gemm_simple(int dtype, const void* a, WeightSegs w, int M, int N, int K, float* out, hipStream_t s) {
  bool vec = aligned16(a) && K % (dtype == 0 ? 4 : 8) == 0;
  for (int i = 0; i < w.nseg; ++i) vec = vec && aligned16(w.w[i]);
  RowsEpilogue ep;
  ep.out = out;
  if (dtype == 0) {
    if (vec) launch_rows_as<float, 4, ROWS_STORE>(a, nullptr, 0.f, w, M, N, K, ep, s);
    else launch_rows_as<float, 1, ROWS_STORE>(a, nullptr, 0.f, w, M, N, K, ep, s);
  } else {
    if (vec) launch_rows_as<bf16_t, 8, ROWS_STORE>(a, nullptr, 0.f, w, M, N, K, ep, s);
    else launch_rows_as<bf16_t, 1, ROWS_STORE>(a, nullptr, 0.f, w, M, N, K, ep, s);
  }
  return hipGetLastError();
}

hipError_t launch_rows_f32(RowsEpi epi, const float* a, const void* gain, float eps, WeightSegs w, int M, int units, int K,
                           const RowsEpilogue& ep, hipStream_t s) {
  bool vec = aligned16(a) && K % 4 == 0 && (!gain || aligned16(gain));
  for (int i = 0; i < w.nseg; ++i) vec = vec && aligned16(w.w[i]);
#define HT_ROWS(E)                                                                  \
  case E:                                                                           \
    if (vec) launch_rows_as<float, 4, E>(a, gain, eps, w, M, units, K, ep, s);      \
    else launch_rows_as<float, 1, E>(a, gain, eps, w, M, units, K, ep, s);          \
    break;
  switch (epi) {
    HT_ROWS(ROWS_STORE_NORM) HT_ROWS(ROWS_ADD) HT_ROWS(ROWS_SILU) HT_ROWS(ROWS_QKV)
    default: return hipErrorInvalidValue;          // the plain product is launch_gemm_simple
  }
#undef HT_ROWS
  return hipGetLastError();
}

}  // namespace ht
