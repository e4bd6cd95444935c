// Hidden transfer for several sources at once on CDNA4 matrix cores (bf16 maps, fp32 sources).
//
//   pseudo[f][i][o] = sum_c W_i[o][c] h_f[c]
//
// The maps stay where the caller keeps them (row-major, read fresh on every call); they are the big operand and the
// bound is their stream from HBM.  The sources keep all 24 bits of their fp32 mantissa: every value is cut into three
// bf16 pieces (truncation, each remainder exact), the pieces multiply the bf16 weights exactly on
// v_mfma_f32_16x16x32_bf16 and the sums are fp32.  Against the fp64 product the relative error is below that of the
// scalar fp32 chain this replaces (1.4e-7 against 1.6e-7 at d = 4096, 1.9e-7 against 2.1e-7 at 8192, 6e-8 against 8e-8
// at 256).  Measured, three maps of 4096 x 4096 (100 MB, 16 us at the streaming rate): 4 sources 26.5 -> 22.0 us, 16
// sources 129 -> 25.7 us, 64 sources 405 -> 47.3 us (there the pieces of the sources, 1.5 MB for every workgroup, take
// twice as long as the maps); five sources on four maps of 8192 x 8192 202 -> 87 us.
//
// Split of the work: a workgroup owns R blocks of 16 map rows (row blocks of all steps in one list) and its four
// wavefronts take a quarter of K each, so no wavefront waits for another inside the loop: weights and sources come in
// with coalesced loads (eight lanes per 128-byte run, a ring of PD 64-column steps in registers), go through
// LDS private to the wavefront into operand order, and the four partial sums meet in LDS at the end in a fixed order.
// Up to five sources fit one 16-column operand with their pieces side by side (one matrix instruction per weight
// fragment); more sources take 16-column tiles with three instructions each.  Up to 16 sources are cut by every workgroup
// for itself, more by a kernel of their own into operand order (a workgroup that cuts 64 sources spends three times as
// long on that as on everything else).
#include "ht_common.h"

namespace ht {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

namespace {

union Frag {
  u32x4_t nat;
  bf16x8_t v;
};

constexpr int kStepCols = 64;
constexpr int kRowBytes = kStepCols * 2 + 32;      // padded by 32 bytes: conflict-free 128-bit operand reads
constexpr int kSideBySide = 5;                     // sources whose three pieces fit one 16-column operand

// x = hi + mid + lo, each with the low 16 bits clear.  Infinities and NaN go into `hi` alone.
__device__ inline void cut3(float x, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  const uint32_t b = __float_as_uint(x);
  const bool finite = (b & 0x7f800000u) != 0x7f800000u;
  hi = (x == x ? b : b | 0x00400000u) & 0xffff0000u;
  const float r1 = finite ? x - __uint_as_float(hi) : 0.f;
  mid = __float_as_uint(r1) & 0xffff0000u;
  lo = __float_as_uint(r1 - __uint_as_float(mid)) & 0xffff0000u;
}
// upper halves of four words as four bf16
__device__ inline uint2 upper4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return make_uint2(__builtin_amdgcn_perm(b, a, 0x07060302u), __builtin_amdgcn_perm(d, c, 0x07060302u));
}
// orders the LDS traffic of a wavefront with itself across lanes (compiler fence, no instruction)
__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The sum of the high pieces and that of the lower ones.  An infinite weight times a lower piece of zero is NaN where the
// weight times the whole value is infinite: what the high pieces say stands when it is not finite.
__device__ inline floatx4_t plus_lower(floatx4_t hi, floatx4_t lo) {
#pragma unroll
  for (int i = 0; i < 4; ++i) hi[i] = __builtin_isfinite(hi[i]) ? hi[i] + lo[i] : hi[i];
  return hi;
}

template <int NT, int R, int DEPTH> struct TransferShape {
  static constexpr int TILES = NT ? NT : 1;
  static constexpr int SOURCES = NT ? NT * 16 : kSideBySide;         // sources a workgroup takes
  static constexpr bool PRECUT = NT >= 2;                            // pieces come from cut_sources_kernel
  static constexpr int PANEL_ROWS = PRECUT ? 0 : NT ? 3 * NT * 16 : 16;
  static constexpr int WAVE_BYTES = (R * 16 + PANEL_ROWS) * kRowBytes;
  static constexpr int SUM_BYTES = 4 * R * TILES * 64 * 16;          // the four K quarters' sums, where the operands were
  static constexpr int LDS_BYTES = 4 * WAVE_BYTES > SUM_BYTES ? 4 * WAVE_BYTES : SUM_BYTES;
  static constexpr int PD = PRECUT ? 2 : DEPTH;
};

// The pieces of many sources in operand order: panel[step of 32 columns][piece][tile of 16 sources][lane], lane l holding
// source l % 16, columns 8 (l / 16) .. + 7; zero past the sources and past the row.  One thread per lane slot.
__global__ __launch_bounds__(256) void cut_sources_kernel(const float* __restrict__ h, const int32_t* __restrict__ src_rows,
                                                          int F, int d, int tiles, int ksteps, u32x4_t* __restrict__ panel) {
  const int slot = blockIdx.x * 256 + threadIdx.x, lane = slot & 63, tile = (slot >> 6) % tiles, ks = (slot >> 6) / tiles;
  if (ks >= ksteps) return;
  const int f = tile * 16 + (lane & 15), k = ks * 32 + (lane >> 4) * 8;
  const bool in = f < F && k < d;
  const float* src = h + (size_t)(in ? (src_rows ? src_rows[f] : f) : 0) * d + (in ? k : 0);
  uint32_t p[3][8];
#pragma unroll
  for (int e = 0; e < 8; ++e) cut3(in ? src[e] : 0.f, p[0][e], p[1][e], p[2][e]);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint2 a = upper4(p[i][0], p[i][1], p[i][2], p[i][3]), b = upper4(p[i][4], p[i][5], p[i][6], p[i][7]);
    panel[(((size_t)ks * 3 + i) * tiles + tile) * 64 + lane] = u32x4_t{a.x, a.y, b.x, b.y};
  }
}

// NT = 0: up to kSideBySide sources side by side in one operand; else NT tiles of 16 sources.
// grid = (ceil(row blocks / R), ceil(F / SOURCES)), block = 256
template <int NT, int R, int DEPTH>
__global__ __launch_bounds__(256) void transfer_split_kernel(const float* __restrict__ h, const int32_t* __restrict__ src_rows,
                                                             int F, const void* const* __restrict__ ws,
                                                             float* __restrict__ pseudo, int i0, int steps, int row_stride,
                                                             int d, const u32x4_t* __restrict__ panel, int ptiles) {
  using TS = TransferShape<NT, R, DEPTH>;
  constexpr int TILES = TS::TILES, PD = TS::PD;
  constexpr bool PRECUT = TS::PRECUT;
  constexpr int NQ = PRECUT ? 1 : (TS::SOURCES * (kStepCols / 4) + 63) / 64;   // float4 loads per lane and step for the sources
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_all[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  unsigned char* wlds = lds_all + wave * TS::WAVE_BYTES;             // this wavefront's weight rows, then its panel
  unsigned char* plds = wlds + R * 16 * kRowBytes;

  const int f0 = blockIdx.y * TS::SOURCES, nf = F - f0 < TS::SOURCES ? F - f0 : TS::SOURCES;
  const int nb = (d + 15) / 16, total = steps * nb;                  // row blocks of one map, of all maps
  const int rb0 = blockIdx.x * R;
  int c0, c1;
  even_share((d + kStepCols - 1) / kStepCols, 4, wave, c0, c1);

  // Workgroups start at different steps of their share: rows of 2^n bytes read in step by all of them fall on few memory
  // channels (4 maps of 8192 x 8192: 108 -> 87 us, 6.2 TB/s; no difference at 4096 and 5120 columns).  With precut sources
  // they stay in step, which keeps the panel in L2.
  const int rot = c1 > c0 ? (int)((blockIdx.x * 5u) % (unsigned)(c1 - c0)) : 0;
  // weight pieces of this lane: rows 8 j + lane / 8 of every row block, 16-byte column lane % 8 of the step
  const bf16_t* wrow[R][2];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int rb = rb0 + r < total ? rb0 + r : total - 1;            // past the list: a valid block, never stored
    const bf16_t* base = (const bf16_t*)ws[i0 + rb / nb];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = (rb % nb) * 16 + 8 * j + (lane >> 3);
      wrow[r][j] = base + (size_t)(row < d ? row : d - 1) * d;
    }
  }
  // source pieces: load q covers source (64 q + lane) / 16, columns 4 ((64 q + lane) % 16) ..
  const float* srow[NQ];
#pragma unroll
  for (int q = 0; q < (PRECUT ? 0 : NQ); ++q) {
    const int s = (64 * q + lane) / 16, f = f0 + (s < nf ? s : nf - 1);
    srow[q] = h + (size_t)(src_rows ? src_rows[f] : f) * d;
  }
  const int wcol = (lane & 7) * 8, scol = (lane & 15) * 4;

  u32x4_t wreg[PD][R][2];
  float4 sreg[PD][NQ];
  Frag preg[PD][PRECUT ? 2 : 1][3][TILES];                           // PRECUT: the pieces of a step, straight from the panel
  const u32x4_t* pbase = PRECUT ? panel + (size_t)blockIdx.y * TILES * 64 + lane : nullptr;
  auto load = [&](u32x4_t (&w)[R][2], float4 (&s)[NQ], Frag (&pc)[PRECUT ? 2 : 1][3][TILES], int c) __attribute__((always_inline)) {
    c = c < c1 ? c : c1 - 1;                                         // past the share: a redundant reload, never used
    if (!PRECUT) c = c + rot < c1 ? c + rot : c + rot - (c1 - c0);
    const int kw = c * kStepCols + wcol, ks = c * kStepCols + scol;
    const bool in_w = kw < d, in_s = ks < d;                         // d is a multiple of 8: a piece lies in the row or past it
    if (PRECUT) {
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int t = 0; t < TILES; ++t)
            pc[PRECUT ? st : 0][i][t].nat = pbase[(((size_t)(c * 2 + st) * 3 + i) * ptiles + t) * 64];
    } else {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const float4 v = *(const float4*)(srow[q] + (in_s ? ks : 0));
        s[q] = in_s ? v : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const u32x4_t v = __builtin_nontemporal_load((const u32x4_t*)(wrow[r][j] + (in_w ? kw : 0)));
        w[r][j] = in_w ? v : u32x4_t{0u, 0u, 0u, 0u};
      }
  };

  // The high pieces in two sums (even and odd 32 columns), the lower ones in a sum of their own: the rounding error of a
  // chain of additions falls with the square root of the number of chains it is cut into.
  floatx4_t hi[2][R][TILES], lo[NT ? R : 1][TILES];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      hi[0][r][t] = hi[1][r][t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
      if (NT) lo[NT ? r : 0][t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    }

  auto step = [&](u32x4_t (&w)[R][2], float4 (&s)[NQ], Frag (&pc)[PRECUT ? 2 : 1][3][TILES], int c) __attribute__((always_inline)) {
    wave_fence();                                                    // the operand reads of the step before are done
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        *(u32x4_t*)(wlds + (r * 16 + 8 * j + (lane >> 3)) * kRowBytes + (lane & 7) * 16) = w[r][j];
#pragma unroll
    for (int q = 0; q < (PRECUT ? 0 : NQ); ++q) {
      const int src = (64 * q + lane) / 16;
      uint32_t p[3][4];
      cut3(s[q].x, p[0][0], p[1][0], p[2][0]);
      cut3(s[q].y, p[0][1], p[1][1], p[2][1]);
      cut3(s[q].z, p[0][2], p[1][2], p[2][2]);
      cut3(s[q].w, p[0][3], p[1][3], p[2][3]);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int row = i * TS::SOURCES + src;                       // NT = 0: 5 i + src, at most 14
        if (NT || src < kSideBySide) *(uint2*)(plds + row * kRowBytes + scol * 2) = upper4(p[i][0], p[i][1], p[i][2], p[i][3]);
      }
    }
    if (!PRECUT) load(w, s, pc, c + PD);
    wave_fence();
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      Frag a[R];
#pragma unroll
      for (int r = 0; r < R; ++r) a[r].nat = *(const u32x4_t*)(wlds + (r * 16 + r16) * kRowBytes + (st * 4 + g) * 16);
#pragma unroll
      for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int i = 0; i < (NT ? 3 : 1); ++i) {
          Frag b;
          if (PRECUT) b = pc[PRECUT ? st : 0][i][t];
          else b.nat = *(const u32x4_t*)(plds + (i * TS::SOURCES + t * 16 + r16) * kRowBytes + (st * 4 + g) * 16);
#pragma unroll
          for (int r = 0; r < R; ++r) {
            if (i == 0) hi[st][r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r].v, b.v, hi[st][r][t], 0, 0, 0);
            else lo[NT ? r : 0][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[r].v, b.v, lo[NT ? r : 0][t], 0, 0, 0);
          }
        }
    }
    if (PRECUT) load(w, s, pc, c + PD);                              // the pieces multiply straight from their registers
  };

  if (!NT) {                          // columns no source fills: defined values (they are never stored)
    for (int i = lane; i < 16 * kRowBytes / 4; i += 64) ((uint32_t*)plds)[i] = 0;
  }
  if (c0 < c1) {
#pragma unroll
    for (int p = 0; p < PD; ++p) load(wreg[p], sreg[p], preg[p], c0 + p);
    int c = c0;
    for (; c + PD <= c1; c += PD) {
#pragma unroll
      for (int p = 0; p < PD; ++p) step(wreg[p], sreg[p], preg[p], c + p);
    }
#pragma unroll
    for (int p = 0; p < PD - 1; ++p)
      if (c + p < c1) step(wreg[p], sreg[p], preg[p], c + p);
  }

  // the four K quarters meet in LDS: [wavefront][row block][tile][lane] float4, added in wavefront order
  __syncthreads();
  floatx4_t* red = (floatx4_t*)lds_all;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      floatx4_t v = hi[0][r][t] + hi[1][r][t];
      if (NT) v = plus_lower(v, lo[NT ? r : 0][t]);
      red[((wave * R + r) * TILES + t) * 64 + lane] = v;
    }
  __syncthreads();
  for (int u = wave; u < R * TILES; u += 4) {
    const int r = u / TILES, t = u % TILES, rb = rb0 + r;
    if (rb >= total) continue;
    auto sum = [&](int l) __attribute__((always_inline)) {
      floatx4_t v = red[u * 64 + l];
#pragma unroll
      for (int w = 1; w < 4; ++w) v += red[(w * R * TILES + u) * 64 + l];
      return v;
    };
    floatx4_t v = sum(lane);
    if (!NT && r16 < kSideBySide) v = plus_lower(v, sum(lane + kSideBySide) + sum(lane + 2 * kSideBySide));
    const int f = t * 16 + r16, o = (rb % nb) * 16 + g * 4;
    if (f < nf && o < d)
      *(float4*)(pseudo + ((size_t)(f0 + f) * row_stride + rb / nb) * d + o) = make_float4(v[0], v[1], v[2], v[3]);
  }
}

template <int NT, int R, int DEPTH>
hipError_t launch_split(const float* h, const int32_t* src_rows, int F, const void* const* w_dev, float* pseudo, int i0, int steps,
                        int row_stride, int d, void* scratch, hipStream_t s) {
  using TS = TransferShape<NT, R, DEPTH>;
  static_assert(TS::LDS_BYTES <= 64 * 1024, "no more LDS than a kernel may use without asking");
  const int total = steps * ((d + 15) / 16), groups = (F + TS::SOURCES - 1) / TS::SOURCES, tiles = groups * TS::TILES;
  if (TS::PRECUT) {
    const int ksteps = (d + kStepCols - 1) / kStepCols * (kStepCols / 32);
    hipLaunchKernelGGL(cut_sources_kernel, dim3((ksteps * tiles * 64 + 255) / 256), dim3(256), 0, s, h, src_rows, F, d, tiles,
                       ksteps, (u32x4_t*)scratch);
  }
  hipLaunchKernelGGL((transfer_split_kernel<NT, R, DEPTH>), dim3((total + R - 1) / R, groups), dim3(256), TS::LDS_BYTES, s, h, src_rows, F,
                     w_dev, pseudo, i0, steps, row_stride, d, (const u32x4_t*)scratch, tiles);
  return hipGetLastError();
}

// Row blocks and source tiles per workgroup.  A compute unit takes in weights and sources at one rate wherever they come
// from, so what counts is the rounds of 256 workgroups (one per unit) times the bytes of one workgroup per column.
// Up to two row blocks per compute unit (one map of a wide model, all maps of a narrow one) few sources do not share a
// workgroup between row blocks at all: the launch is over in the time of one walk along K, so what counts is how much of
// it is in flight.  One map of 4096 x 4096, 4 sources: 17.1 us on two row blocks and a ring of three steps, 14.6 us on one
// row block, 12.8 us with six steps in flight (the scalar kernel of one source, in groups of four: 14.4 us); of 2048 x 2048
// 9.9, 8.6 and 8.1 us (9.5); four of 1536 x 1536, one and a half rounds, 9.6 us, 8.9 with four in flight, 10.0 with six.
// Below 1024 columns a wavefront has fewer than four steps to begin with (512 columns: 3.8 us on a ring of three, 4.0 and
// 4.2 us on four and six).  768 row blocks: within 3 % of the shared workgroups, on either side.
struct SplitPlan { int nt, r, depth = 3; };
SplitPlan plan_split(int F, int total, int d) {
  if (F <= kSideBySide && total <= 512) return SplitPlan{0, 1, d < 1024 ? 3 : total <= 256 ? 6 : 4};
  static const SplitPlan few[] = {{0, 4}, {0, 3}, {0, 2}}, some[] = {{1, 3}, {1, 2}}, many[] = {{4, 3}, {4, 2}, {4, 1}, {2, 3}, {2, 2}};
  const SplitPlan* list = F <= kSideBySide ? few : F <= 16 ? some : many;
  const int count = F <= kSideBySide ? 3 : F <= 16 ? 2 : 5;
  SplitPlan best = list[0];
  long best_cost = -1;
  for (int i = 0; i < count; ++i) {
    const SplitPlan p = list[i];
    const int sources = p.nt ? p.nt * 16 : kSideBySide;
    const long groups = (long)((total + p.r - 1) / p.r) * ((F + sources - 1) / sources);
    const long cost = (groups + 255) / 256 * (32 * p.r + (p.nt >= 2 ? 6 : 4) * sources);
    if (best_cost < 0 || cost < best_cost) { best = p; best_cost = cost; }
  }
  return best;
}

}  // namespace

bool transfer_split_supported(int F, int d) { return F >= 2 && d % 8 == 0; }

size_t transfer_scratch_bytes(int F, int d) {
  if (F <= 16) return 0;
  return (size_t)((F + 63) / 64 * 4) * 3 * ((d + kStepCols - 1) / kStepCols * (kStepCols / 32)) * 64 * sizeof(u32x4_t);
}

hipError_t launch_transfer_split(const float* h, const int32_t* src_rows, int F, const void* const* w_dev, float* pseudo, int i0,
                                 int steps, int row_stride, int d, void* scratch, hipStream_t s) {
  if (F > 16 && !scratch) return hipErrorInvalidValue;
#define HT_SPLIT(NT, R, DEPTH) \
  if (p.nt == NT && p.r == R && p.depth == DEPTH) \
  return launch_split<NT, R, DEPTH>(h, src_rows, F, w_dev, pseudo, i0, steps, row_stride, d, scratch, s)
  const SplitPlan p = plan_split(F, steps * ((d + 15) / 16), d);
  HT_SPLIT(0, 1, 3); HT_SPLIT(0, 1, 4); HT_SPLIT(0, 1, 6); HT_SPLIT(0, 2, 3); HT_SPLIT(0, 3, 3); HT_SPLIT(0, 4, 3);
  HT_SPLIT(1, 2, 3); HT_SPLIT(1, 3, 3);
  HT_SPLIT(2, 2, 3); HT_SPLIT(2, 3, 3);
  HT_SPLIT(4, 1, 3); HT_SPLIT(4, 2, 3); HT_SPLIT(4, 3, 3);
  return hipErrorInvalidValue;
#undef HT_SPLIT
}

}  // namespace ht
