// Skinny weight-streaming product for bf16 on CDNA4 matrix cores.
//
//   out[m][n] = sum_k a[m][k] * w[n][k]        m < M <= 128 tokens, fp32 accumulate (more rows: the
//                                                              token-tiled kernel further down)
//
// The weights are the big operand (N x K, read from HBM exactly once per pass); the activations are
// a small panel (M x K) that every workgroup re-reads from L2.  On v_mfma_f32_16x16x32_bf16 the weight
// rows are the MFMA "A" rows (16 output features per instruction) and the tokens are the "B" columns,
// so each lane ends with four consecutive output features of one token.
//
// Weight layout.  At model init every projection matrix is repacked once into MFMA-fragment order:
// fragment (rb, j) holds rows 16 rb .. 16 rb + 15 and columns 32 j .. 32 j + 31 as 64 lanes x 16 bytes
// (lane l: row l % 16, columns 8 (l / 16) .. + 7).  Eight row blocks form a tile; inside a tile the
// fragments are ordered K-step major (step j of row blocks 0..7, then step j+1, ..), so the workgroup that
// owns a tile reads one sequential stream of 8 KiB per K step while each wavefront load is still a fully
// coalesced 1 KiB that drops straight into MFMA operand registers: no LDS transpose, no partially used
// cache lines, sequential DRAM pages, and no two workgroups marching through memory at the same
// power-of-two stride (row-block-major order measured up to 15 % slower on a pure streaming test).  Row blocks can be ordered freely at pack time,
// and rows inside a block too: that is how gate and up rows meet in one wavefront for the fused SiLU epilogue and
// how a q or k feature meets its rotary partner inside one row block.
//
// The activation chunk (M x 64 columns) is staged once per workgroup in LDS (rows padded by 32 bytes:
// conflict-free 128-bit reads) and shared by the four wavefronts; a ring of PD weight chunks per
// wavefront stays in flight.  Split-K over blockIdx.y writes fp32 partial sums that the consumer adds
// in a fixed order (deterministic).
#include "ht_common.h"
#include <atomic>
#include <type_traits>

namespace ht {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

namespace {

constexpr int kChunkCols = 64;         // K elements per activation chunk (128 for the 16-row instance)
constexpr int kRingDepth = 3;          // weight chunks in flight per wavefront
constexpr int kPadCols = 128;          // packed weights are zero-padded along K to a multiple of this
constexpr int kTileBlocks = 8;         // row blocks interleaved per K step in the packed layout
constexpr int kRowPad = 32;            // bytes added to every activation row in LDS, see gemm_packed_kernel

union Frag {
  uint4 raw;
  u32x4_t nat;
  bf16x8_t v;
};

enum { EPI_F32 = 0, EPI_SILU = 1, EPI_QKV = 2, EPI_QKV_TAIL = 3 };     // ..TAIL: rows from qe.tail_row on have caches of their own

// --------------------------------------------------------------------------------------------- repack
// dst fragment order from row-major segments.  One thread per 16-byte piece.
__global__ void repack_kernel(WeightSegs w, int K, int KS, int n_rb, int mode, int head_blocks,
                              bf16_t* __restrict__ dst) {
  const size_t piece = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int n_tiles = (n_rb + kTileBlocks - 1) / kTileBlocks;
  const size_t total = (size_t)n_tiles * KS * kTileBlocks * 64;
  if (piece >= total) return;
  const int lane = (int)(piece & 63);
  const size_t frag = piece >> 6;
  const int rbt = (int)(frag % kTileBlocks);
  const int j = (int)((frag / kTileBlocks) % KS);
  const int tile = (int)(frag / ((size_t)kTileBlocks * KS));
  const int rb = tile * kTileBlocks + rbt;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (rb < n_rb) {
    int grow = rb * 16 + (lane & 15);       // source row in the concatenated segments
    if (mode == 1) {               // two equal segments interleaved block by block (gate, up)
      grow = (rb & 1) * w.rows[0] + (rb >> 1) * 16 + (lane & 15);
    } else if (mode == 2) {        // q | k | v: block b of a q or k head holds features 8b .. 8b+7 (rows 0..7) and
      const int hb = head_blocks;  // their rotary partners hd/2 + 8b .. (rows 8..15); v heads keep their order
      const int qk_rbs = (w.rows[0] + w.rows[1]) / 16;
      if (rb < qk_rbs) {
        const int in_head = rb % hb, r = lane & 15;
        grow = (rb - in_head) * 16 + (r < 8 ? 8 * in_head + r : 8 * hb + 8 * in_head + r - 8);
      }
    }
    int seg = 0;
    while (seg + 1 < w.nseg && grow >= w.rows[seg]) { grow -= w.rows[seg]; ++seg; }
    const int row = grow;
    const int k = j * 32 + (lane >> 4) * 8;
    if (k < K) v = *(const uint4*)((const bf16_t*)w.w[seg] + (size_t)row * K + k);
  }
  *(uint4*)(dst + piece * 8) = v;
}

// --------------------------------------------------------------------------------------------- epilogues
struct Epilogue : QkvEpilogue {
  float* first = nullptr;            // EPI_F32 without a K split: where the rows below first_rows go, in place of the output
  int32_t first_rows = 0;
  Epilogue() = default;
  Epilogue(const QkvEpilogue& q) : QkvEpilogue(q) {}
};
// Results of two row blocks, a and b, of the sixteen tokens of a tile, a token to a lane of sixteen: exchanged between the
// halves of the sixteen lanes so that `first` holds both blocks' results of the first eight tokens (a's in the lower lanes, b's
// in the upper) and `second` those of the others.  A store then touches half as many lines: what a compute unit needs for
// its results goes with the lines that each sixteen lanes of a store touch, not with the bytes.
__device__ __forceinline__ void pair_halves(uint32_t a, uint32_t b, bool lower, uint32_t& first, uint32_t& second) {
  const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(lower ? b : a), 0x128, 0xf, 0xf, true);   // 8 lanes on
  first = lower ? a : got;
  second = lower ? got : b;
}
// SiLU(gate) * up: 1 ulp reciprocal, bf16 result
__device__ __forceinline__ float silu_times(float gate, float up) { return gate * __builtin_amdgcn_rcpf(1.0f + __expf(-gate)) * up; }

// What a wavefront does with its finished sums acc[r][mt] (row block rb0 + r, token tile mt): the 1/rms factor of
// the token rows, then fp32 partial sums, SiLU(gate) * up, or rotary + q store / K,V append.  TILED (even R, rb0 even): the
// token-tiled kernel, which stores results of two row blocks together.
template <int MT, int R, int EPI, bool TILED = false>
__device__ __forceinline__ void finish_rows(floatx4_t (&acc)[R][MT], const float4 (&row_ss)[MT], int rb0, int wg1, int M,
                                            int N, void* __restrict__ outp, const Epilogue& qe, const RowScale& rs,
                                            int row0, int split) {
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int r16 = row0 + (lane & 15);                    // token row of tile mt: mt * 16 + r16, counted over the whole pass
  if (rs.ss) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const float4 q4 = row_ss[mt];
      const float sc = __builtin_amdgcn_rsqf((q4.x + q4.y + q4.z + q4.w) * rs.inv_d + rs.eps);   // 1 ulp
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r][mt] *= sc;
    }
  }
  if (EPI == EPI_F32 && TILED) {
    // (nontemporal: amounts that no L2 holds)
    float* dst = (float*)outp + (size_t)split * M * N;
    const bool lower = (lane & 8) == 0;
#pragma unroll
    for (int r = 0; r < R; r += 2) {
      const int rb = rb0 + r + (lower ? 0 : 1), n0 = rb * 16 + g * 4;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        u32x4_t first, second;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint32_t f, l;
          pair_halves(__float_as_uint(acc[r][mt][i]), __float_as_uint(acc[r + 1][mt][i]), lower, f, l);
          first[i] = f;
          second[i] = l;
        }
        const int m = row0 + mt * 16 + (lane & 7);
        if (rb < wg1) {
          if (m < M) __builtin_nontemporal_store(first, (u32x4_t*)((m < qe.first_rows ? qe.first : dst) + (size_t)m * N + n0));
          if (m + 8 < M)
            __builtin_nontemporal_store(second, (u32x4_t*)((m + 8 < qe.first_rows ? qe.first : dst) + (size_t)(m + 8) * N + n0));
        }
      }
    }
  } else if (EPI == EPI_F32) {
    float* dst = (float*)outp + (size_t)split * M * N;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (rb0 + r >= wg1) continue;
      const int n0 = (rb0 + r) * 16 + g * 4;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int m = mt * 16 + r16;
        if (m < M) *(floatx4_t*)((m < qe.first_rows ? qe.first : dst) + (size_t)m * N + n0) = acc[r][mt];
      }
    }
  } else if (EPI == EPI_SILU) {
    // row blocks come in pairs: block rb0 + 2 p holds gate rows, rb0 + 2 p + 1 the matching up rows: act = silu(gate) * up
    bf16_t* dst = (bf16_t*)outp;
    const int f = N / 2;
    auto act = [&](int pr, int mt) __attribute__((always_inline)) {      // (the launchers give this epilogue an even R)
      float o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = silu_times(acc[2 * pr][mt][i], acc[2 * pr + 1][mt][i]);
      return pack4_bf16(o[0], o[1], o[2], o[3]);
    };
    auto one_pair = [&](int pr) __attribute__((always_inline)) {
      if (rb0 + 2 * pr + 1 >= wg1) return;
      const int j0 = ((rb0 + 2 * pr) / 2) * 16 + g * 4;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int m = mt * 16 + r16;
        if (m < M) *(uint2*)(dst + (size_t)m * f + j0) = act(pr, mt);
      }
    };
#pragma unroll
    for (int pr = 0; pr < R / 2; pr += TILED ? 2 : 1) {
      if (!TILED || pr + 1 >= R / 2) {
        one_pair(pr);
      } else if (rb0 + 2 * pr + 3 < wg1) {
        const bool lower = (lane & 8) == 0;
        const int j = ((rb0 + 2 * pr) / 2 + (lower ? 0 : 1)) * 16 + g * 4;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const uint2 a = act(pr, mt), b = act(pr + 1 < R / 2 ? pr + 1 : pr, mt);
          uint2 first, second;
          pair_halves(a.x, b.x, lower, first.x, second.x);
          pair_halves(a.y, b.y, lower, first.y, second.y);
          const int m = row0 + mt * 16 + (lane & 7);
          if (m < M) *(uint2*)(dst + (size_t)m * f + j) = first;
          if (m + 8 < M) *(uint2*)(dst + (size_t)(m + 8) * f + j) = second;
        }
      } else {
        one_pair(pr);
        one_pair(pr + 1 < R / 2 ? pr + 1 : pr);
      }
    }
  } else {
    // q | k | v rows.  Block b of a q or k head holds features 8b .. 8b+7 of the head in MFMA rows 0..7 and their
    // rotary partners (feature + hd/2) in rows 8..15, so lanes 0..31 end with the low halves and the lane 32 further
    // on with the partner of the same feature: one exchange, rotate by the row's position, store q or append k to
    // the cache.  v rows are appended to the slot-contiguous value cache.
    const int hd = qe.hd, half = hd / 2, hb = hd / 16, n_now = cache_len(qe.n, qe.n_dev);
    const int q_blocks = qe.Hq * hb, qk_blocks = q_blocks + qe.Hkv * hb;
    const bool upper = g >= 2;
    // block r, a q or k block: rotated results of this lane's token
    auto rotated = [&](int r, int mt) __attribute__((always_inline)) {
      const int rb = rb0 + r, hrb = rb < q_blocks ? rb : rb - q_blocks, j = (hrb % hb) * 8 + (g & 1) * 4;
      const int own = mt * 16 + r16, m = own < M ? own : M - 1;
      const bool tail = EPI == EPI_QKV_TAIL && m >= qe.tail_row;
      const float* cs = EPI == EPI_QKV_TAIL && tail ? qe.tail_cs + (ptrdiff_t)(m - qe.tail_row) * hd : qe.cs + (size_t)m * hd;
      float o[4], other[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) other[i] = __shfl_xor(acc[r][mt][i], 32, 64);
      const float4 c01 = *(const float4*)(cs + j * 2), c23 = *(const float4*)(cs + j * 2 + 4);
      const float cs_[8] = {c01.x, c01.y, c01.z, c01.w, c23.x, c23.y, c23.z, c23.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 f = make_float2(cs_[2 * i], cs_[2 * i + 1]);
        o[i] = upper ? rope_high(other[i], acc[r][mt][i], f) : rope_low(acc[r][mt][i], other[i], f);
      }
      return pack4_bf16(o[0], o[1], o[2], o[3]);
    };
    auto put = [&](int rb, int m, uint2 v) __attribute__((always_inline)) {
      const bool is_q = rb < q_blocks, tail = EPI == EPI_QKV_TAIL && m >= qe.tail_row;
      const int hrb = is_q ? rb : rb - q_blocks, h = hrb / hb, j = (hrb % hb) * 8 + (g & 1) * 4 + (upper ? half : 0);
      bf16_t* dst = is_q   ? qe.q + ((size_t)m * qe.Hq + h) * hd + j
                    : tail ? qe.tail_kc + ((size_t)(qe.tail_n + m - qe.tail_row) * qe.Hkv + h) * hd + j
                           : qe.kc + ((size_t)(n_now + m) * qe.Hkv + h) * hd + j;
      *(uint2*)dst = v;
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int rb = rb0 + r;
      if (rb >= wg1) continue;                                  // uniform over the wavefront
      if (rb < qk_blocks) {
        if (TILED && (r & 1)) continue;                         // with the block before it: both of one head, whose blocks are even
        const bool lower = (lane & 8) == 0;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const uint2 a = rotated(r, mt);
          if (TILED) {
            const uint2 b = rotated(r + 1 < R ? r + 1 : r, mt);
            uint2 first, second;
            pair_halves(a.x, b.x, lower, first.x, second.x);
            pair_halves(a.y, b.y, lower, first.y, second.y);
            const int m = row0 + mt * 16 + (lane & 7);
            if (m < M) put(rb + (lower ? 0 : 1), m, first);
            if (m + 8 < M) put(rb + (lower ? 0 : 1), m + 8, second);
          } else {
            const int m = mt * 16 + r16;
            if (m < M) put(rb, m, a);
          }
        }
      } else {
        const int vb = rb - qk_blocks, h = vb / hb, e0 = (vb % hb) * 16 + g * 4;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const int m = mt * 16 + r16;
          if (m < M) {
            const uint2 v4 = pack4_bf16(acc[r][mt][0], acc[r][mt][1], acc[r][mt][2], acc[r][mt][3]);
            const bool tail = EPI == EPI_QKV_TAIL && m >= qe.tail_row;
            const size_t cap = tail ? qe.tail_cap : qe.cap;                        // feature e0 + i is i * cap further on
            bf16_t* col = (tail ? qe.tail_vc + qe.tail_n + m - qe.tail_row : qe.vc + n_now + m) + ((size_t)h * hd + e0) * cap;
            col[0] = (bf16_t)(v4.x & 0xffffu);
            col[cap] = (bf16_t)(v4.x >> 16);
            col[2 * cap] = (bf16_t)(v4.y & 0xffffu);
            col[3 * cap] = (bf16_t)(v4.y >> 16);
          }
        }
      }
    }
  }
}

// --------------------------------------------------------------------------------------------- product
// The hot loop is straight-line code (no predicated loads, no data-dependent branches) so that the
// compiler can keep exact outstanding-load counts and the weight ring really stays in flight: chunk
// indices past the end of this block's K range are clamped to its last chunk (a redundant, in-bounds
// reload that is never used), wavefront slots without a row block re-read one fragment (never stored), and
// activation columns past K are clamped into the row (they meet zero-padded weights).
template <int MT, int R, int WAVES, int EPI, int KC = kChunkCols, int PD = kRingDepth>
__global__ __launch_bounds__(64 * WAVES) void gemm_packed_kernel(const bf16_t* __restrict__ a,
                                                                 const bf16_t* __restrict__ wp, int M, int N, int K,
                                                                 int KS, void* __restrict__ outp, int nsplit,
                                                                 Epilogue qe, RowScale rs) {
  constexpr int STEPS = KC / 32;                         // MFMA steps per chunk
  // LDS row stride in bytes.  Measured with the bank-conflict counter, a 128-bit operand read of the sixteen rows of
  // a fragment takes 4 cycles with rows padded by 32 bytes, 8 with 16 bytes of padding and 16 with none.
  constexpr int ROWB = KC * 2 + kRowPad;
  constexpr int THREADS = 64 * WAVES;
  constexpr int ROWS = MT * 16;
  constexpr int PIECES = ROWS * (KC / 8);                // 16-byte pieces of the activation chunk
  static_assert(PIECES >= THREADS, "every thread stages at least one piece of the activation chunk");
  constexpr int APASS = (PIECES + THREADS - 1) / THREADS;   // surplus threads of the last pass repeat the last piece
  constexpr int STAGE = ROWS * ROWB;
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * STAGE];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int chunks = KS / STEPS;                         // KS is a multiple of STEPS (weights zero-padded)
  int c0, c1;
  even_share(chunks, nsplit, blockIdx.y, c0, c1);
  const int n_rb = N / 16;
  // The grid's workgroups share the row blocks evenly: workgroup b owns n_rb / G blocks, the first n_rb % G
  // workgroups one more (in whole pairs for the SiLU epilogue), at most R * WAVES of them (the launcher's
  // choice of G), R consecutive ones per wavefront.  A slot past the end of
  // the workgroup's range re-reads one fragment of its first block over and over (stride 0: cache hits, no HBM
  // traffic, same instruction stream) and stores nothing.
  constexpr int U = EPI == EPI_SILU ? 2 : 1;             // the SiLU epilogue needs both blocks of a (gate, up) pair
  const int units = (n_rb + U - 1) / U;
  int wg0, wg1;
  even_share(units, gridDim.x, blockIdx.x, wg0, wg1);
  wg0 *= U;
  wg1 *= U;
  const int rb0 = wg0 + wave * R;
  if (c0 >= c1) return;                                  // uniform over the block

  const u32x4_t* wbase[R];
  size_t wstep[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool own = rb0 + r < wg1;
    const int rb = own ? rb0 + r : wg0;
    wbase[r] = (const u32x4_t*)wp + ((size_t)(rb / kTileBlocks) * KS * kTileBlocks + rb % kTileBlocks) * 64 + lane;
    wstep[r] = own ? (size_t)kTileBlocks * 64 : 0;
  }
  const int last = c1 - 1;
  // All workgroups walk K in the same order on purpose: they then pull the same activation lines from
  // L2 at about the same time, which keeps the small panel resident while the weights stream through
  // (a staggered walk measured 12 % slower).
  auto load_w = [&](Frag (&dst)[R][STEPS], int c) __attribute__((always_inline)) {
    c = c < last ? c : last;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int s = 0; s < STEPS; ++s)
        dst[r][s].nat = __builtin_nontemporal_load(wbase[r] + (size_t)(c * STEPS + s) * wstep[r]);
  };
  // activation pieces of this thread: row p / 16, 16-byte column p % 16 of the chunk
  const bf16_t* arow[APASS];
  int acol[APASS], alds[APASS];
#pragma unroll
  for (int i = 0; i < APASS; ++i) {
    int p = tid + i * THREADS;
    p = p < PIECES ? p : PIECES - 1;
    // rows past the pass fetch its last row, whose lines are on their way already (9 rows of 11008 gated features over 4096
    // columns 29.6 -> 28.9 us, 33 of 5120 over 13824 27.9 -> 27.3)
    const int row = p / (KC / 8);
    arow[i] = a + (size_t)(row < M ? row : M - 1) * K;
    acol[i] = (p % (KC / 8)) * 8;
    alds[i] = (p / (KC / 8)) * ROWB + (p % (KC / 8)) * 16;
  }
  auto load_a = [&](u32x4_t (&dst)[APASS], int c) __attribute__((always_inline)) {
    c = c < last ? c : last;
#pragma unroll
    for (int i = 0; i < APASS; ++i) {
      int k = c * KC + acol[i];
      k = k < K - 8 ? k : K - 8;
      dst[i] = *(const u32x4_t*)(arow[i] + k);
    }
  };
  auto store_a = [&](const u32x4_t (&src)[APASS], int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < APASS; ++i) *(u32x4_t*)(&lds[stage * STAGE + alds[i]]) = src[i];
  };

  floatx4_t acc[R][MT];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[r][mt] = floatx4_t{0.f, 0.f, 0.f, 0.f};

  // Rows of a panel that was stored without its 1/rms factor: the factor multiplies the finished sums instead
  // (every K split scales its partial sums by the same factor).  The sums of squares are fetched here, ahead of
  // the weight stream (they are the oldest loads, so no wait ever stalls on them), and turned into factors in the
  // epilogue.
  float4 row_ss[MT];
  if (rs.ss) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = mt * 16 + r16;
      row_ss[mt] = *(const float4*)(rs.ss + (size_t)(m < M ? m : M - 1) * kNormParts);
    }
  }

  // Loads retire in issue order, so everything is issued oldest-needed-first: at chunk c the ring holds
  // weights of chunks c .. c+PD-1 and activations of chunks c+1 .. c+PD; each iteration consumes the
  // oldest of both and issues activation chunk c+PD+1, then weight chunk c+PD.
  Frag wreg[PD][R][STEPS];
  u32x4_t areg[PD][APASS];
  {
    u32x4_t first[APASS];
    load_a(first, c0);
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      load_a(areg[p], c0 + 1 + p);
      load_w(wreg[p], c0 + p);
    }
    store_a(first, 0);
  }
  __syncthreads();

  auto body = [&](Frag (&wslot)[R][STEPS], u32x4_t (&aslot)[APASS], int c) __attribute__((always_inline)) {
    const int stage = (c - c0) & 1;
    const unsigned char* ab = &lds[stage * STAGE + r16 * ROWB + g * 16];
    // activation fragments are read one MFMA step ahead of their use
    Frag b[2][MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) b[0][mt].nat = *(const u32x4_t*)(ab + mt * 16 * ROWB);
    store_a(aslot, stage ^ 1);                 // activation chunk c+1 becomes visible after the barrier below
    load_a(aslot, c + PD + 1);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + 1 < STEPS) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) b[(s + 1) & 1][mt].nat = *(const u32x4_t*)(ab + mt * 16 * ROWB + (s + 1) * 64);
      }
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[r][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wslot[r][s].v, b[s & 1][mt].v, acc[r][mt], 0, 0, 0);
    }
    load_w(wslot, c + PD);
    __syncthreads();
  };

  int c = c0;
  for (; c + PD <= c1; c += PD) {
#pragma unroll
    for (int p = 0; p < PD; ++p) body(wreg[p], areg[p], c + p);
  }
#pragma unroll
  for (int p = 0; p < PD - 1; ++p)
    if (c + p < c1) body(wreg[p], areg[p], c + p);                // uniform tail

  finish_rows<MT, R, EPI>(acc, row_ss, rb0, wg1, M, N, outp, qe, rs, 0, blockIdx.y);
}

// --------------------------------------------------------------------------------------------- product, many rows
// The same product tiled over the tokens as well, for passes of more rows than the weight stream can hide (prompts, the
// forward pass of the training stage, passes of more than 128 rows): a workgroup of WF x WT wavefronts owns 16 R WF weight
// rows and 16 MT WT token rows and walks its share of K in chunks of 64 columns.
//
// Bound: the matrix cores, if the operands reach them.  Both operands go through LDS (a chunk of weights and of tokens is
// fetched once per workgroup), straight from global memory with 16-byte LDS-direct loads, ST stages.  A wavefront
// multiplies 16 R weight rows by 16 MT tokens: at R = 4, MT = 8 it reads 12 KB from LDS for 32 matrix instructions.  Counted on
// gate/up at 4095 tokens: matrix cores busy 0.70 of the time, LDS 0.27 with these reads (no bank conflicts), wavefronts
// waiting 0.46 of their cycles; what is lost is lost between a read and the products that need it.  So the
// order of issue is what matters, and it is written out (sched_barrier fences): operands of the next 32 columns are
// read, a fragment or two at a time, between groups of four matrix instructions on the current ones, and the second half
// of a chunk also issues the loads of the chunk after next one by one (64 of them in a burst behind the barrier block
// the memory path for a thousand cycles, in which nothing multiplies: 1.25 -> 1.32 PFLOP/s at 4096^3).  One barrier per
// chunk, in its middle: there the next chunk has landed (its first operands are read before this chunk's last products)
// and every wavefront has read the last of this one, whose stage the loads then refill.
// Measured on random operands, 4096 tokens, against 128 x 256 tiles with weights loaded into registers (the kernel this
// replaces): 12288 x 4096 421 -> 312 us (1.32 PFLOP/s), 4096 x 4096 123 -> 107 us (1.28), 4096 x 11008 308 -> 259 us
// (1.43).  Tried and slower: weights straight into registers (1.25 - 1.39 PFLOP/s over the same three), four wavefronts of
// 128 x 128 (0.9 - 1.27), a ring of four or five stages of 32 columns (1.20 - 1.26).
//
// Smaller tiles, for launches that would not fill the chip with 256 x 256 ones, are bound by what a compute unit takes in: 50
// GB/s where the weights come from HBM, whatever is in flight beyond 32 KB, half that if the ring runs dry in between.  With
// two stages nothing is in flight at the barrier in the middle of a chunk (everything has landed by then), so these tiles
// have as many stages as LDS holds, and the barrier waits for the next chunk only: 256 rows of 12288 features over 4096
// columns in 128 x 128 tiles 57 us with two stages, 43 with three; 512 rows in 128 x 256 tiles 70 and 54.  Tried and slower: a
// tail without the loads past the end (3 % on 24 chunks and more; faster below 12).
//
// Workgroups are numbered so that those of one XCD (every eighth) work on blocks of 4 weight tiles x 8 token tiles at a
// time, and results that no L2 can hold leave it alone (nontemporal stores): 361 -> 312 us at 12288 x 4096.
//
// LDS layout of a stage: the weight fragments of the chunk, 1 KB each in operand order (step, row block), then the
// token rows of 128 bytes whose 16-byte pieces are XOR-swizzled by row (an LDS-direct load writes 64 consecutive pieces,
// so every lane picks the global piece that belongs at its place).
__device__ __forceinline__ void lds_load16(const void* from, void* to) {
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)from, (void __attribute__((address_space(3)))*)to, 16,
                                   0, 0);
}

// this wavefront's LDS-direct loads but the last N have landed and its LDS reads are done; then the others'
template <int N> __device__ __forceinline__ void tile_wait_then_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int WF, int R_, int WT, int MT, int ST> struct TileShape {
  static constexpr int R = R_, WAVES = WF * WT, BLOCKS = WF * R, FEATURES = BLOCKS * 16, TOKENS = WT * MT * 16;
  static constexpr int WBYTES = FEATURES * 128, STAGE = WBYTES + TOKENS * 128, LDS_BYTES = ST * STAGE;
  static constexpr int NW = 2 * BLOCKS / WAVES, NA = TOKENS / 8 / WAVES;   // LDS-direct loads per wavefront and chunk: weights, tokens
  static_assert(2 * BLOCKS % WAVES == 0 && TOKENS / 8 % WAVES == 0, "whole loads");
  static_assert((ST - 1) * (NW + NA) < 64, "the outstanding loads are counted in six bits");
};

template <int WF, int R, int WT, int MT, int ST, int EPI>
__global__ __launch_bounds__(64 * WF * WT) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_tile_kernel(
    const bf16_t* __restrict__ a, const bf16_t* __restrict__ wp, int M, int N, int K, int KS, void* __restrict__ outp,
    Epilogue qe, RowScale rs, int tile0, int n_tiles, int m_tiles, int nsplit) {
  using TS = TileShape<WF, R, WT, MT, ST>;
  constexpr int FB = TS::BLOCKS, NW = TS::NW, NA = TS::NA, STAGE = TS::STAGE, WBYTES = TS::WBYTES;
  extern __shared__ __attribute__((aligned(1024))) unsigned char tile_lds[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int wf = wave % WF, wt = wave / WF;
  // workgroup id -> (K split, weight tile, token tile): the tiles of a split, four weight tiles wide times eight token tiles
  // after the other, split by split, are dealt to the XCDs in eight runs of equal length.  (Whole weight tiles to an XCD left
  // some with a tile more than their 32 units take in a round: 1500 rows of 10752 features, 252 tiles, took two rounds.  So
  // did every split dealt by itself: 384 rows of 5120 features over 13824 columns in 3 x 81 tiles 90 us, 59 now.)
  const int tiles = n_tiles * m_tiles, per_xcd = (tiles * nsplit + 7) / 8, all = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (all >= tiles * nsplit) return;                     // uniform over the workgroup
  const int split = all / tiles, at = all - split * tiles;
  const int q = at / (4 * m_tiles), rem = at % (4 * m_tiles), nw = n_tiles - q * 4 < 4 ? n_tiles - q * 4 : 4;
  const int mg = rem / (8 * nw), in = rem % (8 * nw), mw = m_tiles - mg * 8 < 8 ? m_tiles - mg * 8 : 8;
  const int tl = q * 4 + in / mw, ty = mg * 8 + in % mw;
  const int tx = tile0 + tl;                             // the launch covers weight tiles tile0 .. tile0 + n_tiles - 1
  int c0, c1;
  even_share(KS / 2, nsplit, split, c0, c1);
  const int chunks = c1 - c0;
  if (chunks <= 0) return;                               // uniform over the workgroup
  const int row0 = ty * TS::TOKENS, n_rb = N / 16;

  // loads of this wavefront: NW of the chunk's weight fragments, counted row block by row block within a step (past the last
  // packed row block: that block, results never stored), and NA times eight token rows (past the pass: its last row, results
  // never stored)
  const int rb_last = (n_rb + kTileBlocks - 1) / kTileBlocks * kTileBlocks - 1;
  const u32x4_t* wsrc[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int f = wave * NW + i, own = tx * FB + f % FB, rb = own < rb_last ? own : rb_last;
    wsrc[i] = (const u32x4_t*)wp + (((size_t)(rb / kTileBlocks) * KS + 2 * c0 + f / FB) * kTileBlocks + rb % kTileBlocks) * 64;
  }
  const bf16_t* asrc[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int m = row0 + (wave * NA + i) * 8 + (lane >> 3);
    asrc[i] = a + (size_t)(m < M ? m : M - 1) * K;
  }
  const int pcol = c0 * 64 + ((lane & 7) ^ (lane >> 3)) * 8;
  auto fetch = [&](int i, int c, int stage) __attribute__((always_inline)) {
    unsigned char* base = tile_lds + stage * STAGE;
    if (i < NW) {
      lds_load16(wsrc[i] + (size_t)c * 16 * 64 + lane, base + (wave * NW + i) * 1024);
    } else {
      const int k = c * 64 + pcol;                         // columns past K meet zero-padded weights: any in-bounds piece
      lds_load16(asrc[i - NW] + (k < K - 8 ? k : K - 8), base + WBYTES + (wave * NA + i - NW) * 1024);
    }
  };
  const int wfrag = wf * R * 1024 + lane * 16, arow = WBYTES + (wt * MT * 16 + r16) * 128;
  auto read_w = [&](Frag& w, int stage, int s, int r) __attribute__((always_inline)) {
    w.nat = *(const u32x4_t*)(tile_lds + stage * STAGE + wfrag + (s * FB + r) * 1024);
  };
  auto read_a = [&](Frag& b, int stage, int s, int t) __attribute__((always_inline)) {
    b.nat = *(const u32x4_t*)(tile_lds + stage * STAGE + arow + t * 2048 + (((s * 4 + g) ^ (r16 & 7)) << 4));
  };

  floatx4_t acc[R][MT];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[r][t] = floatx4_t{0.f, 0.f, 0.f, 0.f};

  Frag w0[R], w1[R], b0[MT], b1[MT];                     // operands of the first and the second 32 columns of a chunk
  // Products of one half (w, b) between reads of the next half's operands (wn, bn: half `s` of `stage`) and, with FETCH,
  // the loads of chunk c into stage `into`.
  auto half = [&](Frag (&w)[R], Frag (&b)[MT], Frag (&wn)[R], Frag (&bn)[MT], int stage, int s, auto fetching, int c, int into)
      __attribute__((always_inline)) {
    constexpr bool FETCH = decltype(fetching)::value;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if (FETCH) {
#pragma unroll
        for (int i = t * (NW + NA) / MT; i < (t + 1) * (NW + NA) / MT; ++i) fetch(i, c, into);
      }
      read_a(bn[t], stage, s, t);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (MT >= R ? r == t : r * MT / R == t) read_w(wn[r], stage, s, r);
#pragma unroll
      for (int r = 0; r < R; ++r)
        acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[r].v, b[t].v, acc[r][t], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // chunk c in stage `st`; chunk c + ST goes into its stage (past the end: the last chunk again, never used; loops without
  // it in a tail of their own cost registers that are not there)
  auto body = [&](int c, int st) __attribute__((always_inline)) {
    half(w0, b0, w1, b1, st, 1, std::false_type{}, 0, 0);
    tile_wait_then_barrier<(ST - 2) * (NW + NA)>();
    __builtin_amdgcn_sched_barrier(0);
    half(w1, b1, w0, b0, st + 1 == ST ? 0 : st + 1, 0, std::true_type{}, c + ST < chunks ? c + ST : chunks - 1, st);
  };
#pragma unroll
  for (int p = 0; p < ST - 1; ++p)
#pragma unroll
    for (int i = 0; i < NW + NA; ++i) fetch(i, p < chunks ? p : chunks - 1, p);
  tile_wait_then_barrier<(ST - 2) * (NW + NA)>();
#pragma unroll
  for (int i = 0; i < NW + NA; ++i) fetch(i, ST - 1 < chunks ? ST - 1 : chunks - 1, ST - 1);
#pragma unroll
  for (int r = 0; r < R; ++r) read_w(w0[r], 0, 0, r);
#pragma unroll
  for (int t = 0; t < MT; ++t) read_a(b0[t], 0, 0, t);
  int c = 0;
  for (; c + ST <= chunks; c += ST) {
#pragma unroll
    for (int p = 0; p < ST; ++p) body(c + p, p);
  }
#pragma unroll
  for (int p = 0; p < ST - 1; ++p)
    if (c + p < chunks) body(c + p, p);
  tile_wait_then_barrier<0>();                           // nothing may still be writing LDS when the workgroup ends
  const int rb0 = tx * WF * R + wf * R;
  float4 row_ss[MT];
  if (rs.ss) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int m = row0 + (wt * MT + mt) * 16 + r16;
      row_ss[mt] = *(const float4*)(rs.ss + (size_t)(m < M ? m : M - 1) * kNormParts);
    }
  }
  finish_rows<MT, R, EPI, true>(acc, row_ss, rb0, n_rb, M, N, outp, qe, rs, row0 + wt * MT * 16, split);
}

// Workgroup shape.  R = 2 row blocks per wavefront when that still leaves >= 80 workgroups, else R = 1.
// Every workgroup re-reads the whole activation panel, and a compute unit ingests only ~45 GB/s (measured,
// weights + panel), so the fastest grid is the one closest to one workgroup on each of the 256 compute
// units: 3 wavefronts (6 row blocks) per workgroup when that gives <= 260 workgroups, else 4 (8 row
// blocks); split-K (gemm_mfma_splits) tops small-N grids up to about 256.
int rows_per_wave(int N) { return N / 16 / 8 >= 80 ? 2 : 1; }
int waves_per_group(int n_rb) { return (n_rb + 5) / 6 <= 260 ? 3 : 4; }

// With a token panel of more than 16 rows the panel a workgroup re-reads is no longer small beside its weight
// rows (64 weight rows against a 64-row panel: half of what it ingests).  When K is long enough to give every
// split 2048 columns, 128-row workgroups (R = 2, four wavefronts) on a deeper split-K halve that share at the
// same grid size: measured at M = 64, N x K = 5120 x 13824: 28.1 -> 25.5 us, 8192 x 28672: 83.7 -> 74.8 us,
// 10240 x 8192: 30.1 -> 28.1 us; at 4096 x 4096 and 4096 x 11008 (512 / 1376 columns per split) it loses or ties.
int wide_split(int M, int N, int K) {
  if (M <= 16) return 0;
  const int tiles = (N / 16 + 7) / 8;
  const int s = (256 + tiles / 2) / tiles;
  return s >= 2 && s <= kMaxSplitK && K / s >= 2048 ? s : 0;
}

template <int MT>
hipError_t launch_mt(const bf16_t* a, const PackedW& w, int M, void* out, int nsplit, int epi, const Epilogue& qe,
                     const RowScale& rs, hipStream_t s) {
  const int n_rb = w.N / 16;
  const int KS = w.Kp / 32;
  constexpr int KC = MT == 1 ? 128 : kChunkCols;     // the chunk must give every thread at least one 16-byte piece
  if (epi == EPI_F32 && wide_split(M, w.N, w.K)) {
    hipLaunchKernelGGL((gemm_packed_kernel<MT, 2, 4, EPI_F32, KC>), dim3((n_rb + 7) / 8, nsplit), dim3(256), 0, s, a,
                       w.p, M, w.N, w.K, KS, out, nsplit, qe, rs);
  } else if (epi == EPI_SILU || (epi == EPI_F32 && rows_per_wave(w.N) == 2)) {
    const bool three = waves_per_group(n_rb) == 3;
    // a grid just short of the 256 compute units is topped up to 256 (the kernel shares the row blocks evenly):
    // measured 32.3 -> 31.6 us at 22016 x 4096, M = 64, and 30.6 -> 29.2 us at M = 1
    int gx = three ? (n_rb + 5) / 6 : (n_rb + 7) / 8;
    if (gx >= 200 && gx < 256 && (epi == EPI_SILU || nsplit == 1)) gx = 256;
    const dim3 grid(gx, epi == EPI_SILU ? 1 : nsplit);
    if (epi == EPI_SILU) {
      if (three)
        hipLaunchKernelGGL((gemm_packed_kernel<MT, 2, 3, EPI_SILU, 128>), grid, dim3(192), 0, s, a, w.p, M, w.N, w.K, KS,
                           out, 1, qe, rs);
      else
        hipLaunchKernelGGL((gemm_packed_kernel<MT, 2, 4, EPI_SILU, KC>), grid, dim3(256), 0, s, a, w.p, M, w.N, w.K, KS,
                           out, 1, qe, rs);
    } else {
      if (three)
        hipLaunchKernelGGL((gemm_packed_kernel<MT, 2, 3, EPI_F32, 128>), grid, dim3(192), 0, s, a, w.p, M, w.N, w.K, KS,
                           out, nsplit, qe, rs);
      else
        hipLaunchKernelGGL((gemm_packed_kernel<MT, 2, 4, EPI_F32, KC>), grid, dim3(256), 0, s, a, w.p, M, w.N, w.K, KS,
                           out, nsplit, qe, rs);
    }
  } else if (epi == EPI_QKV) {
    // no split-K here, so one row block per wavefront and three or four wavefronts: 768 row blocks (a 4096-wide
    // model with full-size K/V heads) fill 256 workgroups exactly; measured 23.4 -> 21.6 us against two blocks
    // per wavefront in 192 workgroups of two
    const bool four = n_rb > 3 * 256;
    int gx = four ? (n_rb + 3) / 4 : (n_rb + 2) / 3;
    if (gx < 256 && n_rb >= 256) gx = 256;
    if (four)
      hipLaunchKernelGGL((gemm_packed_kernel<MT, 1, 4, EPI_QKV, KC>), dim3(gx, 1), dim3(256), 0, s, a, w.p, M, w.N, w.K,
                         KS, out, 1, qe, rs);
    else
      hipLaunchKernelGGL((gemm_packed_kernel<MT, 1, 3, EPI_QKV, KC>), dim3(gx, 1), dim3(192), 0, s, a, w.p, M, w.N, w.K,
                         KS, out, 1, qe, rs);
  } else {
    hipLaunchKernelGGL((gemm_packed_kernel<MT, 1, 4, EPI_F32, KC>), dim3((n_rb + 3) / 4, nsplit), dim3(256), 0, s, a,
                       w.p, M, w.N, w.K, KS, out, nsplit, qe, rs);
  }
  return hipGetLastError();
}

// A pass of up to 128 rows: the instance with the fewest token tiles that hold them.
hipError_t launch_rows(const bf16_t* ap, const PackedW& w, int rows, void* out, int nsplit, int epi,
                       const Epilogue& qe, const RowScale& rs, hipStream_t s) {
  if (rows <= 16) return launch_mt<1>(ap, w, rows, out, nsplit, epi, qe, rs, s);
  if (rows <= 32) return launch_mt<2>(ap, w, rows, out, nsplit, epi, qe, rs, s);
  if (rows <= 48) return launch_mt<3>(ap, w, rows, out, nsplit, epi, qe, rs, s);
  if (rows <= 64) return launch_mt<4>(ap, w, rows, out, nsplit, epi, qe, rs, s);
  if (rows <= 80) return launch_mt<5>(ap, w, rows, out, nsplit, epi, qe, rs, s);   // a 64-node tree plus a few pseudo rows
  if (rows <= 96) return launch_mt<6>(ap, w, rows, out, nsplit, epi, qe, rs, s);
  return launch_mt<8>(ap, w, rows, out, nsplit, epi, qe, rs, s);
}

template <int EPI>
hipError_t launch_wide(const void* a, const PackedW& w, int M, void* out, int nsplit, const Epilogue& qe, const RowScale& rs,
                       hipStream_t s);

// A workgroup of the streaming kernel holds at most 128 token rows (accumulators and the activation ring are registers):
// a pass of more rows goes to the token-tiled kernel.  The K split is the caller's.  At 256 rows of 4096 columns, against
// two launches of 128 rows: 12288 features 72 -> 39 us, 22016 81 -> 58, 4096 24 -> 18, 32000 105 -> 67; 4096 x 11008
// 51 -> 34.
hipError_t launch_any(const void* a, const PackedW& w, int M, void* out, int nsplit, int epi, const Epilogue& qe,
                      const RowScale& rs, hipStream_t s) {
  if (M <= 128) return launch_rows((const bf16_t*)a, w, M, out, nsplit, epi, qe, rs, s);
  if (epi == EPI_SILU) return launch_wide<EPI_SILU>(a, w, M, out, 1, qe, rs, s);
  if (epi == EPI_QKV) return launch_wide<EPI_QKV>(a, w, M, out, 1, qe, rs, s);
  return launch_wide<EPI_F32>(a, w, M, out, nsplit, qe, rs, s);
}

}  // namespace

bool gemm_mfma_supported(int M, int N, int K) { return M >= 1 && M <= kMaxRows && N % 16 == 0 && K % 8 == 0 && N >= 16; }

int packed_cols(int K) { return (K + kPadCols - 1) / kPadCols * kPadCols; }

size_t packed_weight_bytes(int N, int K) {
  const size_t rbs = (size_t)(N / 16 + kTileBlocks - 1) / kTileBlocks * kTileBlocks;
  return rbs * 16 * packed_cols(K) * sizeof(bf16_t);
}

// Decode passes and the public products of 129 - 256 rows keep this split, made for the streaming kernel, although they run on
// the token-tiled one: the product without a scratch argument promises the bits of the one with it, within 16 MiB of sums.
int gemm_mfma_splits(int M, int N, int K) {
  if (const int wide = wide_split(M, N, K)) return wide;
  const int n_rb = N / 16;
  const int per_wg = rows_per_wave(N) == 2 ? 2 * waves_per_group(n_rb) : 4;      // row blocks per workgroup
  const int tiles = (n_rb + per_wg - 1) / per_wg;
  int s = (256 + tiles / 2) / tiles;         // nearest grid to 256 workgroups
  const int chunks = (K + 127) / 128;
  if (s > chunks / 4) s = chunks / 4;        // at least 512 columns per split
  if (s > kMaxSplitK) s = kMaxSplitK;
  if (s < 1) s = 1;
  return s;
}

hipError_t launch_repack(WeightSegs w, int K, int mode, int head_dim, void* dst, hipStream_t s) {
  int rows = 0;
  for (int i = 0; i < w.nseg; ++i) rows += w.rows[i];
  const int n_rb = rows / 16, KS = packed_cols(K) / 32;
  const size_t pieces = (size_t)((n_rb + kTileBlocks - 1) / kTileBlocks) * kTileBlocks * KS * 64;
  hipLaunchKernelGGL(repack_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, s, w, K, KS, n_rb, mode,
                     head_dim / 16, (bf16_t*)dst);
  return hipGetLastError();
}

hipError_t launch_gemm_packed(const void* a, PackedW w, int M, float* out, int nsplit, hipStream_t s, RowScale rs, float* first,
                              int first_rows) {
  if (first && nsplit != 1) return hipErrorInvalidValue;
  Epilogue ep;
  ep.first = first;
  ep.first_rows = first ? first_rows : 0;
  return launch_any(a, w, M, out, nsplit, EPI_F32, ep, rs, s);
}

hipError_t launch_gemm_packed_silu(const void* a, PackedW w, int M, void* act, hipStream_t s, RowScale rs) {
  return launch_any(a, w, M, act, 1, EPI_SILU, QkvEpilogue{}, rs, s);
}

namespace {
// Above 64 KB of LDS a kernel has to ask: once per device (gemm_tile_prepare does it when a model is set up, so that no
// launch inside a stream capture has to).
template <int WF, int R, int WT, int MT, int ST, int EPI>
hipError_t allow_tile_lds() {
  using TS = TileShape<WF, R, WT, MT, ST>;
  if (TS::LDS_BYTES <= 64 * 1024) return hipSuccess;
  static std::atomic<bool> allowed[64];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!allowed[dev].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute((const void*)gemm_tile_kernel<WF, R, WT, MT, ST, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, TS::LDS_BYTES);
    if (e != hipSuccess) return e;
    allowed[dev].store(true, std::memory_order_release);
  }
  return hipSuccess;
}

// Features [from, to) of the product, `from` a multiple of the tile.
template <int WF, int R, int WT, int MT, int ST, int EPI>
hipError_t launch_tile(const bf16_t* a, const PackedW& w, int M, void* out, int nsplit, const Epilogue& qe, const RowScale& rs,
                       int from, int to, hipStream_t s) {
  using TS = TileShape<WF, R, WT, MT, ST>;
  const int n_tiles = (to - from + TS::FEATURES - 1) / TS::FEATURES, m_tiles = (M + TS::TOKENS - 1) / TS::TOKENS;
  const hipError_t e = allow_tile_lds<WF, R, WT, MT, ST, EPI>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_tile_kernel<WF, R, WT, MT, ST, EPI>), dim3(8 * ((n_tiles * m_tiles * nsplit + 7) / 8)), dim3(64 * TS::WAVES),
                     TS::LDS_BYTES, s, a, w.p, M, w.N, w.K, w.Kp / 32, out, qe, rs, from / TS::FEATURES, n_tiles, m_tiles, nsplit);
  return hipGetLastError();
}

// Tile of a product of M rows with a given K split: rounds of workgroups over the 256 compute units, times what a
// workgroup takes: `round` once (half of it goes with how full the round is: results written), and per chunk of 64 columns
// `chunk` plus `rows` for token rows that are there (a tile's rows past the pass fetch its last row over and over), `idle`
// less of both on an empty chip.  Microseconds, fitted to 560 launches of 129 - 4096 rows on 1024 - 57344 features over 1024 -
// 28672 columns, weights not in any cache: off by 7 % in the mean, and the tile it picks takes 0.6 % longer in the mean than
// the fastest of them all.  What it picks, and what the three tiles of two stages took that there were before (us):
//   64 x 64     1024 x 1024: 384 rows 7.1 (12.8)
//   64 x 128    4096 x 4096, two splits: 256 rows 18.4 (33)
//   96 x 128    12288 x 4096: 160 rows 31 (58), 256 rows 39 (59)
//   128 x 128   4096 x 11008, four splits: 256 rows 34 (43)
//   192 x 128   22016 x 4096: 256 rows 58 (76); 12288 x 4096: 512 rows 55 (128 x 256: 57), 300 rows 48 (52)
//   128 x 256   32000 x 4096: 256 rows 67 (89)
//   192 x 256   22016 x 4096: 512 rows 88 (104); 12288 x 4096: 1024 rows 88 (101)
//   256 x 256   27648 x 5120: 512 rows 126 (127); 12288 x 4096: 4096 rows 310 (319); everything large
struct TileCost { int features, tokens; float round, chunk, rows, idle; };
constexpr TileCost kTileCosts[] = {{256, 256, 14.1f, 1.411f, 0.f, 0.15f},   {128, 256, 9.0f, 0.646f, 0.132f, 0.17f},
                                   {192, 256, 10.4f, 1.154f, 0.f, 0.12f},   {192, 128, 7.4f, 0.541f, 0.090f, 0.08f},
                                   {128, 128, 5.1f, 0.437f, 0.070f, 0.07f}, {96, 128, 4.4f, 0.320f, 0.106f, 0.f},
                                   {64, 128, 3.5f, 0.278f, 0.071f, 0.f},    {64, 64, 1.4f, 0.219f, 0.f, 0.f}};
constexpr int kTiles = sizeof(kTileCosts) / sizeof(kTileCosts[0]);

// 256 x 256 tiles whose last round would leave half the chip or more without one: the weight tiles of the whole rounds;
// the other features go in 128 x 256 tiles, twice as many, and a second launch (2048 rows of 27648 features over 5120
// columns, 3.4 rounds: 460 us in one launch and 421 in two on one machine, 454 in two on another; 1024 of 22016 over 4096: 179
// and 146 - 166).  0: one launch.
int whole_round_tiles(int M, int N, int nsplit) {
  const int m_tiles = (M + 255) / 256, n_tiles = (N + 255) / 256, whole = (int)((long)n_tiles * m_tiles / 256 * 256 / m_tiles);
  return nsplit == 1 && whole > 0 && whole < n_tiles && 2L * (n_tiles - whole) * m_tiles <= 256 ? whole : 0;
}

float tile_us(const TileCost& t, int M, int N, int K, int nsplit) {
  const int m_tiles = (M + t.tokens - 1) / t.tokens;
  const long groups = (long)((N + t.features - 1) / t.features) * m_tiles * nsplit, whole = groups / 256;
  const float chunks = (float)((packed_cols(K) / 64 + nsplit - 1) / nsplit), rest = (float)(groups % 256) / 256.f;
  const float chunk = t.chunk + t.rows * (float)M / (float)(m_tiles * t.tokens);
  const float last = rest > 0.f ? t.round * 0.5f * (1.f + rest) + chunk * chunks * (1.f - t.idle * (1.f - rest)) : 0.f;
  return (float)whole * (t.round + chunk * chunks) + last;
}
struct TileChoice { int tile, whole; float us; };            // whole > 0: as whole_round_tiles
TileChoice best_tile(int M, int N, int K, int nsplit) {
  TileChoice best{0, 0, tile_us(kTileCosts[0], M, N, K, nsplit)};
  for (int i = 1; i < kTiles; ++i)
    if (const float us = tile_us(kTileCosts[i], M, N, K, nsplit); us < best.us) best = TileChoice{i, 0, us};
  if (const int whole = whole_round_tiles(M, N, nsplit)) {
    const float us = tile_us(kTileCosts[0], M, whole * 256, K, 1) + tile_us(kTileCosts[1], M, N - whole * 256, K, 1);
    if (us < best.us) best = TileChoice{0, whole, us};
  }
  return best;
}

// `tile`: index into kTileCosts
template <int EPI>
hipError_t launch_tile_of(int tile, const bf16_t* a, const PackedW& w, int M, void* out, int nsplit, const Epilogue& qe,
                          const RowScale& rs, int from, int to, hipStream_t s) {
  switch (tile) {
    case 0: return launch_tile<4, 4, 2, 8, 2, EPI>(a, w, M, out, nsplit, qe, rs, from, to, s);
    case 1: return launch_tile<2, 4, 4, 4, 3, EPI>(a, w, M, out, nsplit, qe, rs, from, to, s);
    case 2: return launch_tile<2, 6, 4, 4, 2, EPI>(a, w, M, out, nsplit, qe, rs, from, to, s);
    case 3: return launch_tile<2, 6, 4, 2, 3, EPI>(a, w, M, out, nsplit, qe, rs, from, to, s);
    case 4: return launch_tile<2, 4, 2, 4, 3, EPI>(a, w, M, out, nsplit, qe, rs, from, to, s);
    case 5: return launch_tile<1, 6, 4, 2, 4, EPI>(a, w, M, out, nsplit, qe, rs, from, to, s);
    case 6: return launch_tile<1, 4, 4, 2, 5, EPI>(a, w, M, out, nsplit, qe, rs, from, to, s);
    case 7: return launch_tile<1, 4, 4, 1, 5, EPI>(a, w, M, out, nsplit, qe, rs, from, to, s);
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t launch_wide(const void* a, const PackedW& w, int M, void* out, int nsplit, const Epilogue& qe, const RowScale& rs,
                       hipStream_t s) {
  const bf16_t* ap = (const bf16_t*)a;
  const TileChoice c = best_tile(M, w.N, w.K, nsplit);
  if (!c.whole) return launch_tile_of<EPI>(c.tile, ap, w, M, out, nsplit, qe, rs, 0, w.N, s);
  const hipError_t e = launch_tile_of<EPI>(0, ap, w, M, out, 1, qe, rs, 0, c.whole * 256, s);
  return e != hipSuccess ? e : launch_tile_of<EPI>(1, ap, w, M, out, 1, qe, rs, c.whole * 256, w.N, s);
}

template <int EPI>
hipError_t allow_tiles() {
  hipError_t e = allow_tile_lds<4, 4, 2, 8, 2, EPI>();
  if (e == hipSuccess) e = allow_tile_lds<2, 4, 4, 4, 3, EPI>();
  if (e == hipSuccess) e = allow_tile_lds<2, 6, 4, 4, 2, EPI>();
  if (e == hipSuccess) e = allow_tile_lds<2, 6, 4, 2, 3, EPI>();
  if (e == hipSuccess) e = allow_tile_lds<2, 4, 2, 4, 3, EPI>();
  if (e == hipSuccess) e = allow_tile_lds<1, 6, 4, 2, 4, EPI>();
  if (e == hipSuccess) e = allow_tile_lds<1, 4, 4, 2, 5, EPI>();
  if (e == hipSuccess) e = allow_tile_lds<1, 4, 4, 1, 5, EPI>();
  return e;
}
}  // namespace

hipError_t gemm_tile_prepare() {
  hipError_t e = allow_tiles<EPI_F32>();
  if (e == hipSuccess) e = allow_tiles<EPI_SILU>();
  if (e == hipSuccess) e = allow_tiles<EPI_QKV>();
  if (e == hipSuccess) e = allow_tiles<EPI_QKV_TAIL>();
  return e;
}

// A split pays for its partial sums where they are read: 0.6 us a million more of them in the kernel that adds them up (512
// rows of 4096: 7.1, 8.4 and 10.7 us for one, two and four; what writing them takes is in the tile's cost).  512 rows of 4096
// features over 11008 columns: 70 us without, 55 and 44 in two and four.  Beyond 64 MB of them no split saves anything (1987
// rows of 5120 features over 13824 columns: 271 us without, 299 and 319 in two and three).
size_t gemm_wide_part_bytes() { return (size_t)64 << 20; }
int gemm_wide_splits(int M, int N, int K) {
  int best = 1;
  float best_us = best_tile(M, N, K, 1).us;
  for (int sp = 2; sp <= kMaxSplitK && packed_cols(K) / 64 / sp >= 8; ++sp) {      // at least 512 columns per split
    if ((size_t)sp * M * N * sizeof(float) > gemm_wide_part_bytes()) break;
    const float us = best_tile(M, N, K, sp).us + (float)(sp - 1) * (float)M * (float)N * 0.6e-6f;
    if (us < best_us) { best = sp; best_us = us; }
  }
  return best;
}

int gemm_tile_of(int M, int N, int K, int nsplit) {
  const TileChoice c = best_tile(M, N, K, nsplit);
  return c.whole ? kTiles : c.tile;
}
hipError_t launch_gemm_tile(int tile, int epi, const void* a, PackedW w, int M, void* out, int nsplit, QkvEpilogue qe, hipStream_t s) {
  const bf16_t* ap = (const bf16_t*)a;
  if (tile < 0 || tile >= kTiles || (epi != EPI_F32 && nsplit != 1)) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_F32: return launch_tile_of<EPI_F32>(tile, ap, w, M, out, nsplit, qe, RowScale{}, 0, w.N, s);
    case EPI_SILU: return launch_tile_of<EPI_SILU>(tile, ap, w, M, out, 1, qe, RowScale{}, 0, w.N, s);
    case EPI_QKV: return launch_tile_of<EPI_QKV>(tile, ap, w, M, out, 1, qe, RowScale{}, 0, w.N, s);
    case EPI_QKV_TAIL: return launch_tile_of<EPI_QKV_TAIL>(tile, ap, w, M, out, 1, qe, RowScale{}, 0, w.N, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_wide(const void* a, PackedW w, int M, float* out, int nsplit, hipStream_t s, RowScale rs) {
  return launch_wide<EPI_F32>(a, w, M, out, nsplit, QkvEpilogue{}, rs, s);
}
hipError_t launch_gemm_wide_silu(const void* a, PackedW w, int M, void* act, hipStream_t s, RowScale rs) {
  return launch_wide<EPI_SILU>(a, w, M, act, 1, QkvEpilogue{}, rs, s);
}
hipError_t launch_gemm_wide_qkv(const void* a, PackedW w, int M, QkvEpilogue qe, hipStream_t s, RowScale rs) {
  if (qe.tail_kc) return launch_wide<EPI_QKV_TAIL>(a, w, M, nullptr, 1, qe, rs, s);
  return launch_wide<EPI_QKV>(a, w, M, nullptr, 1, qe, rs, s);
}

bool qkv_fusable(int head_dim) { return head_dim % 32 == 0; }

// The fused q|k|v product cannot split K, so its workgroups stay small (three or four row blocks); with few row
// blocks (70B-shaped grouped-query projections: 640) the 128-row split-K workgroups plus a separate rotary/append
// kernel are faster once the token panel is large (measured 41 us against 28 + 7 us at M = 64).
bool qkv_prefer_split(int M, int N) { return M > 16 && N / 16 / 4 < 176; }

hipError_t launch_gemm_packed_qkv(const void* a, PackedW w, int M, QkvEpilogue qe, hipStream_t s, RowScale rs) {
  return launch_any(a, w, M, nullptr, 1, EPI_QKV, qe, rs, s);
}

}  // namespace ht
