// Internal declarations shared by the HIP sources of libht (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stddef.h>

namespace ht {

typedef uint16_t bf16_t;   // raw bfloat16 bits

__host__ __device__ inline float bf16_to_float(bf16_t v) {
  union { uint32_t u; float f; } c;
  c.u = (uint32_t)v << 16;
  return c.f;
}
// round-to-nearest-even; NaN stays NaN
__host__ __device__ inline bf16_t float_to_bf16(float f) {
  union { uint32_t u; float f; } c;
  c.f = f;
  if ((c.u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((c.u >> 16) | 0x40u);
  c.u += 0x7fffu + ((c.u >> 16) & 1u);
  return (bf16_t)(c.u >> 16);
}

// Four floats to four bf16 (8 bytes) with the gfx950 pair conversion (round-to-nearest-even, NaN stays NaN: the same
// values as float_to_bf16).
__device__ inline uint2 pack4_bf16(float a, float b, float c, float d) {
  typedef float f2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
  const b2_t lo = __builtin_convertvector(f2_t{a, b}, b2_t), hi = __builtin_convertvector(f2_t{c, d}, b2_t);
  uint2 r;
  r.x = *(const uint32_t*)&lo;
  r.y = *(const uint32_t*)&hi;
  return r;
}

// Share `total` items over `parts` owners as evenly as possible: owner i gets [lo, hi), the first total % parts
// owners one item more.  One 32-bit division (a 64-bit one is a few hundred instructions in front of a kernel's
// first load).
__device__ inline void even_share(unsigned total, unsigned parts, unsigned i, int& lo, int& hi) {
  const unsigned q = total / parts, rem = total - q * parts;
  lo = (int)(i * q + (i < rem ? i : rem));
  hi = lo + (int)q + (i < rem ? 1 : 0);
}

// (cos, sin) of pos * base^(-2j/hd), evaluated in fp64 and rounded once.  The general functions of the library (a logarithm, an
// exponential, a sine and cosine of any argument: some 500 instructions) were most of what a launch of this took; here the
// angle is counted in turns, which leaves nothing to reduce but the whole turns and the quarters, and the rest are Taylor
// sums: the first term left out is 4e-18 of the result for |exponent| <= 1/2 and 5e-17 for |angle| <= pi / 4.  What an angle of
// thousands of turns multiplies, the frequency, is carried in two doubles.  Floats that are not the rounded exact value (positions
// below 8192, bases 100 to 10^6, heads of 64 to 128, 4.0 million): 1, with the general functions 16.
// rope_step: log2(base) / half, from the host, in two doubles of which the first has 24 bits (times j: exact).
inline double2 rope_step(float base, int half) {
  const long double step = log2l((long double)base) / half;
  const double hi = (double)(float)step;
  return make_double2(hi, (double)(step - (long double)hi));
}
__device__ inline double2 rope_turns(int j, double2 step) {      // base^(-2j/hd) / (2 pi)
  constexpr double ln2 = 0.69314718055994531, ln2_rest = 2.3190468138462996e-17;
  constexpr double per_turn = 0.15915494309189535, per_turn_rest = -9.8393383375912429e-18;
  const double x = -(double)j * step.x, k = rint(x), f = x - k, y = fma(f, ln2, fma(f, ln2_rest, -(double)j * step.y * ln2));
  double p = 1.0 / 6227020800.0;
  constexpr double c[12] = {1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320, 1.0 / 362880,
                            1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600};
#pragma unroll
  for (int i = 11; i >= 0; --i) p = fma(p, y, c[i]);
  p *= y;
  const double e = 1.0 + p, e_rest = p - (e - 1.0), t = e * per_turn;
  const double t_rest = fma(e, per_turn, -t) + fma(e, per_turn_rest, e_rest * per_turn);
  return make_double2(ldexp(t, (int)k), ldexp(t_rest, (int)k));
}
__device__ inline float2 rope_factor(int pos, double2 turns) {
#pragma clang fp contract(off)
  // (u rounded: its rest is added below, and a product fused into the subtraction would count it twice)
  const double n = (double)pos, u = n * turns.x, u_rest = fma(n, turns.x, -u) + n * turns.y;
  const double part = u - rint(u), quarter = rint(4.0 * part);
  const double a = (fma(quarter, -0.25, part) + u_rest) * 6.2831853071795865, z = a * a;
  double sn = -1.0 / 1307674368000.0, cn = 1.0 / 20922789888000.0;
  constexpr double cs[7] = {1.0, -1.0 / 6, 1.0 / 120, -1.0 / 5040, 1.0 / 362880, -1.0 / 39916800, 1.0 / 6227020800.0};
  constexpr double cc[8] = {1.0, -1.0 / 2, 1.0 / 24, -1.0 / 720, 1.0 / 40320, -1.0 / 3628800, 1.0 / 479001600, -1.0 / 87178291200.0};
#pragma unroll
  for (int i = 6; i >= 0; --i) sn = fma(sn, z, cs[i]);
#pragma unroll
  for (int i = 7; i >= 0; --i) cn = fma(cn, z, cc[i]);
  const float s = (float)(sn * a), c = (float)cn;
  const int k = (int)quarter;                                  // -2 .. 2
  const float2 odd = make_float2(k > 0 ? -s : s, k > 0 ? c : -c), even = make_float2(k ? -c : c, k ? -s : s);
  return k & 1 ? odd : even;
}

// The rotated pair of (a, b), a of the lower half of a head, b its partner: a cos - b sin, b cos + a sin.  Which of the two
// products is rounded before the sum is written out: left to the compiler it was one in one kernel and the other in the next
// (and for some elements of one kernel), and the keys of a prompt then depended on the tile that its rows were multiplied in.
__device__ inline float rope_low(float a, float b, float2 cs) { return fmaf(a, cs.x, -(b * cs.y)); }
__device__ inline float rope_high(float a, float b, float2 cs) { return fmaf(b, cs.x, a * cs.y); }

template <typename T> struct Conv;
template <> struct Conv<float> {
  __device__ static inline float load(const float* p) { return *p; }
  __device__ static inline void store(float* p, float v) { *p = v; }
};
template <> struct Conv<bf16_t> {
  __device__ static inline float load(const bf16_t* p) { return bf16_to_float(*p); }
  __device__ static inline void store(bf16_t* p, float v) { *p = float_to_bf16(v); }
};

constexpr int kMaxTree = 128;            // nodes of a tree (root included)
constexpr int kMaxRows = 256;            // rows of a pass: tree nodes plus the pseudo rows that ride along, or a prefill chunk
constexpr int kMaskWords = kMaxRows / 64;
constexpr int kMaxTopK = 64;
constexpr int kMaxTransfer = 8;
constexpr int kMaxSplitK = 8;
constexpr int kMaxLoopSteps = 64;        // steps per call of the device-resident loop

// Tree tables as the kernels see them (device pointers).
struct TreeDev {
  const int32_t* parent;     // [T]
  const int32_t* depth;      // [T]
  const int32_t* rank;       // [T]
  const uint64_t* anc;       // [rows][kMaskWords] bit u set iff row u is the row itself or an ancestor of it
};

// Device-resident decoder state written by the accept kernel and read back by the host.
struct StepState {
  int32_t root;                              // pending root token
  int32_t m;                                 // accepted count of the last step
  int32_t next_root;
  int32_t path[kMaxTransfer + 1];
  int32_t emitted[kMaxTransfer + 1];
  // device-resident loop (ht_decode_steps): cache length of step i in n[i & 1], steps logged so far
  int32_t n[2], log_count;
  int32_t pad[1];
};
// what one step of the device-resident loop leaves for the host
struct StepLog {
  int32_t m;
  int32_t emitted[kMaxTransfer + 1];
};

// Cache length of a pass: kernels take the host's value `n` and, for the device-resident loop, a pointer that
// overrides it (NULL otherwise).  The host value then only has to be an upper bound (it sizes grids and LDS).
__device__ inline int cache_len(int n, const int32_t* n_dev) { return n_dev ? *n_dev : n; }

// One weight operand made of up to three row segments sharing K (Wq|Wk|Wv, Wgate|Wup).
struct WeightSegs {
  const void* w[3];
  int32_t rows[3];
  int32_t nseg;
};

// ------------------------------------------------------------------------------------------------
// launchers (definitions in the .hip files); all enqueue on `s` and return the launch status
// ------------------------------------------------------------------------------------------------
// Where the tokens of a pass come from: tok[m], or, with `cand`, the tree's rule: the pending root and, for a node of depth e
// and rank r, cand[e - 1][r].  They are kept in `keep`, if given (`tok` itself is fine).
struct TokenSource {
  const int32_t* tok = nullptr;
  const StepState* st = nullptr;
  const int32_t *cand = nullptr, *depth = nullptr, *rank = nullptr;
  int32_t* keep = nullptr;
};
// The first norm of a pass, as launch_add_norm_parts works it out (bf16, d a multiple of 4 kNormParts)
struct FirstNorm {
  const bf16_t* gain = nullptr;
  bf16_t* u = nullptr;
  float* ss = nullptr;
};
// x[m] = emb[token m], or rows_in[m] when that is given, m < rows (0: none); cs[m] = rotary factors of position n + depth[m]
// (n + m without depths), m < cs_rows; with norm.gain (emb and gain on 8 bytes) also the norm of the rows
hipError_t launch_start_pass(int dtype, const void* emb, TokenSource tokens, const float* rows_in, float* x, int rows, int d,
                             float* cs, const int32_t* depth, int n, int cs_rows, int hd, float base, hipStream_t s,
                             const int32_t* n_dev = nullptr, FirstNorm norm = FirstNorm{});
hipError_t launch_load_rows(const float* src, float* x, int M, int d, hipStream_t s);
// bf16 models that do not pack: x[m] += part[m] (nsplit 0 or 1); optional save; u[m] = rmsnorm(x[m]) * gain
hipError_t launch_add_norm(float* x, const float* part, int nsplit, size_t part_stride, const void* gain,
                           void* u, float* save_h, int M, int d, float eps, hipStream_t s);
// The same with kNormParts workgroups per row (d a multiple of 4 kNormParts): each adds and stores its part of the
// row, leaves the sum of squares of that part in ss[m][part] and writes u[m] = x[m] * gain WITHOUT the 1/rms factor;
// the product that consumes u multiplies its output rows by RowScale::of(m) instead (bf16 only).
constexpr int kNormParts = 4;
hipError_t launch_add_norm_parts(float* x, const float* part, int nsplit, size_t part_stride, const void* gain, void* u,
                                 float* save_h, float* ss, int M, int d, hipStream_t s);
// 1 / rms of the rows of an activation panel written by launch_add_norm_parts; ss == NULL: rows are used as they are
struct RowScale {
  const float* ss = nullptr;
  float inv_d = 0.f, eps = 0.f;
};
// depth == NULL: row m sits at position n + m
hipError_t launch_rope_table(float* cs, const int32_t* depth, int n, int M, int hd, float base, hipStream_t s,
                             const int32_t* n_dev = nullptr);
// qkv may be `nsplit` split-K partial sums of [M][(Hq + 2 Hkv) hd] each
hipError_t launch_rope_append(const float* qkv, int nsplit, const float* cs, void* q, void* kc, void* vc,
                              int n, int M, int Hq, int Hkv, int hd, int cap, bool paired, hipStream_t s,
                              const int32_t* n_dev = nullptr);
// rows as they come from the caller, at positions n + depth[m]; `cs`: room for the factors of M rows
hipError_t launch_rope_append_split(int dtype, const void* q_in, const void* k_in, const void* v_in, const int32_t* depth,
                                    float base, float* cs, void* q, void* kc, void* vc, int n, int M, int Hq, int Hkv, int hd,
                                    int cap, hipStream_t s);
hipError_t launch_silu_mul(const float* gu, void* act, int M, int f, hipStream_t s);
hipError_t launch_argmax(const float* z, int32_t* g, int M, int V, hipStream_t s);
// cand[i] = top width[i % period + 1] entries of logit row src_row[i] (row i when src_row is NULL), i < rows;
// scratch: topk_scratch_bytes(rows) bytes for the per-slice survivors.  With `g`: also g[m] = arg-max of row m of z, m < T (rows of
// V); `widest`: the largest width then, which says whether the two share a launch
size_t topk_scratch_bytes(int rows);
hipError_t launch_topk(const float* d, int32_t* cand, const int32_t* width, void* scratch, int rows, int period,
                       const int32_t* src_row, int V, hipStream_t s, const float* z = nullptr, int32_t* g = nullptr, int T = 0, int widest = 0);
// kl[p] = KL(softmax(za[p]) || softmax(zb[p])), p < pairs, rows of V floats (Sec. 3.3 loss term)
hipError_t launch_kl_rows(const float* za, const float* zb, int pairs, int V, float* kl, hipStream_t s);
// Tree chosen from the draft distributions: lp[k][kMaxTopK] = log-probabilities of the b best candidates of every
// draft row (whole-row log-softmax); then the T - 1 best nodes by (summed lp desc, depth asc, rank path asc) fill
// the tree tables and the token row.  T <= kMaxTree, 1 <= b <= kMaxTopK, 1 <= k <= kMaxTransfer and
// T - 1 <= b + b^2 + .. + b^k are the caller's to check.
struct TreeOut {
  int32_t *parent, *depth, *rank;
  uint64_t* anc;
};
hipError_t launch_cand_logprob(const float* d, const int32_t* cand, int rows, int b, int V, float* lp, hipStream_t s);
hipError_t launch_tree_dynamic(const int32_t* root /*device*/, const int32_t* cand, const float* lp, int k, int b, int T,
                               TreeOut tree, int32_t* tok, hipStream_t s);
// parity >= 0 (device-resident loop): the cache length is st->n[parity], st->n[parity ^ 1] the one after the acceptance, and
// the step is appended to log[st->log_count++]; parity < 0: the cache length is n
hipError_t launch_accept_compact(int dtype, StepState* st, TreeDev tree, const int32_t* tok, const int32_t* g, int T, StepLog* log,
                                 int n, int parity, void* const* kc, void* const* vc, int L, int Hkv, int hd, int cap,
                                 const float* saved_h, size_t slot_stride, int slots, float* h_src, int d, hipStream_t s);
// *st to `host` (device-visible host memory, one word more than a StepState holds), then `number` to the word behind it
hipError_t launch_publish_state(const StepState* st, int32_t* host, int32_t number, hipStream_t s);
hipError_t launch_prefill_finish(StepState* st, const int32_t* g, const float* saved_h, size_t slot_stride, int slots,
                                 float* h_src, int last, int d, hipStream_t s);
// measurement aid: one pass over `buf` with the weight stream's access pattern; returns the bytes actually read
size_t launch_stream_read(const void* buf, size_t bytes, int groups, uint32_t* sink, hipStream_t s);
double launch_mfma_rate(int form, int iters, uint32_t* sink, hipStream_t s);
// pseudo[f * row_stride + (i - i0)] = W_i h_f for steps i0 <= i < i0 + steps and F sources
// h_f = h + (src_rows ? src_rows[f] : f) * d
hipError_t launch_transfer(int dtype, const float* h, const int32_t* src_rows, int F, const void* const* w_dev,
                           float* pseudo, int i0, int steps, int row_stride, int d, void* scratch, hipStream_t s);
// the same for several sources of a bf16 model, on the matrix cores (see ht_transfer_mfma.hip)
bool transfer_split_supported(int F, int d);
size_t transfer_scratch_bytes(int F, int d);   // device bytes launch_transfer needs for F sources of a bf16 model
hipError_t launch_transfer_split(const float* h, const int32_t* src_rows, int F, const void* const* w_dev, float* pseudo, int i0,
                                 int steps, int row_stride, int d, void* scratch, hipStream_t s);
hipError_t launch_convert_to_f32(int dtype, const void* src, float* dst, int n, hipStream_t s);
hipError_t launch_convert_to_bf16(const float* src, void* dst, size_t count, hipStream_t s);
// out[i] = sum_s part[s][i] in the fixed order s = 0, 1, ..
hipError_t launch_reduce_splits(const float* part, int nsplit, size_t stride, float* out, hipStream_t s);

// generic (any dtype, any shape) product: out[s=0][m][n] = sum_k a[m][k] w[n][k]
hipError_t launch_gemm_simple(int dtype, const void* a, WeightSegs w, int M, int N, int K, float* out, hipStream_t s);
// fp32 model: the products of a decoder block with what surrounds them (ht_rows.hip).  STORE: out[m][u]; STORE_NORM: the
// same on RMS-normalised rows of `a`; ADD: out[m][u] += , kept in `save` too when set; SILU: out[m][u] = silu(gate) * up
// on normalised rows, w = (gate, up); QKV: normalised rows, w = (q, k, v), one unit per (head, j < hd / 2), rotary, q
// stored, k and v appended at slot n + m.
enum RowsEpi { ROWS_STORE, ROWS_STORE_NORM, ROWS_ADD, ROWS_SILU, ROWS_QKV };
struct RowsEpilogue {
  float* out = nullptr;
  float* save = nullptr;
  const float* cs = nullptr;                 // (cos, sin) table [M][hd / 2]
  float *q = nullptr, *kc = nullptr, *vc = nullptr;
  int32_t n = 0, Hq = 0, Hkv = 0, hd = 0, cap = 0;
  const int32_t* n_dev = nullptr;            // overrides n when set (device-resident loop)
};
hipError_t launch_rows_f32(RowsEpi epi, const float* a, const void* gain, float eps, WeightSegs w, int M, int units, int K,
                           const RowsEpilogue& ep, hipStream_t s);
// bf16 MFMA product over weights repacked into MFMA-fragment order (see ht_gemm_mfma.hip)
struct PackedW {
  const bf16_t* p;   // fragment-ordered copy
  int32_t N, K, Kp;  // rows (multiple of 16), columns, columns rounded up to packed_cols(K)
};
bool gemm_mfma_supported(int M, int N, int K);
int packed_cols(int K);
size_t packed_weight_bytes(int N, int K);
int gemm_mfma_splits(int M, int N, int K);
// mode 0: row blocks in natural order over the concatenated segments; mode 1: two equal segments
// interleaved block by block (gate block i, up block i, gate block i+1, ..); mode 2: segments (q, k, v), in
// every q and k head the 16-row block p is followed by its rotary partner block p + head_dim/32
hipError_t launch_repack(WeightSegs w, int K, int mode, int head_dim, void* dst, hipStream_t s);
// out[s][m][n], s < nsplit (split-K partial sums, fp32); with nsplit 1, rows below first_rows go to `first` if that is given.  Up
// to 128 rows stream the weights, more run on the token-tiled kernel.
hipError_t launch_gemm_packed(const void* a, PackedW w, int M, float* out, int nsplit, hipStream_t s, RowScale rs = RowScale{},
                              float* first = nullptr, int first_rows = 0);
// w packed with mode 1 from (gate, up): act[m][j] = silu(a.gate_j) * (a.up_j), bf16 [M][N/2]
hipError_t launch_gemm_packed_silu(const void* a, PackedW w, int M, void* act, hipStream_t s, RowScale rs = RowScale{});
// w packed with mode 2 from (q, k, v): rotary at the row's position, q rows to `q`, k/v rows appended to the
// caches at slot n + m (all bf16); cs is the (cos, sin) table [M][hd/2]
struct QkvEpilogue {
  const float* cs;
  bf16_t *q, *kc, *vc;
  int32_t n, Hq, Hkv, hd, cap;
  const int32_t* n_dev = nullptr;            // overrides n when set (device-resident loop)
  // launch_gemm_wide_qkv with tail_kc set: rows from tail_row on take their rotary factors from tail_cs (row 0 on) and go
  // to slots tail_n .. of caches of their own; their q rows follow the others'
  int32_t tail_row = 0, tail_n = 0, tail_cap = 0;
  const float* tail_cs = nullptr;
  bf16_t *tail_kc = nullptr, *tail_vc = nullptr;
};
// The same products tiled over the tokens too, for passes of any number of rows: out fp32 [nsplit][M][N] (nsplit 1 or
// gemm_wide_splits); act bf16 [M][N/2] (w packed from (gate, up)); q | k | v as in launch_gemm_packed_qkv.
int gemm_wide_splits(int M, int N, int K);
size_t gemm_wide_part_bytes();                // the most partial sums gemm_wide_splits asks for, in bytes
hipError_t gemm_tile_prepare();              // once per device before the first launch that may sit inside a stream capture
hipError_t launch_gemm_wide(const void* a, PackedW w, int M, float* out, int nsplit, hipStream_t s, RowScale rs = RowScale{});
hipError_t launch_gemm_wide_silu(const void* a, PackedW w, int M, void* act, hipStream_t s, RowScale rs = RowScale{});
hipError_t launch_gemm_wide_qkv(const void* a, PackedW w, int M, QkvEpilogue qe, hipStream_t s, RowScale rs = RowScale{});
// for tests: the tile that these take (0 .. 7, the order of their table; 8: whole rounds of the first, the rest in the second),
// and a launch with a given one, `epi` 0 fp32 sums, 1 SiLU(gate) * up, 2 q | k | v, 3 the same with tail rows
int gemm_tile_of(int M, int N, int K, int nsplit);
hipError_t launch_gemm_tile(int tile, int epi, const void* a, PackedW w, int M, void* out, int nsplit, QkvEpilogue qe, hipStream_t s);
bool qkv_fusable(int head_dim);
bool qkv_prefer_split(int M, int N);
hipError_t launch_gemm_packed_qkv(const void* a, PackedW w, int M, QkvEpilogue qe, hipStream_t s,
                                  RowScale rs = RowScale{});

// attention over cache + tree rows; out[m][h*hd+e] in dtype
hipError_t launch_attn_simple(int dtype, const void* q, const void* kc, const void* vc, int cap, int n, int M,
                              TreeDev tree, int Hq, int Hkv, int hd, void* out, hipStream_t s,
                              const int32_t* n_dev = nullptr);
bool attn_mfma_supported(int M, int Hq, int Hkv, int hd);
size_t attn_mfma_scratch_bytes(int M, int Hq, int hd);
// once per device before the first launch that may sit inside a stream capture (kernel attributes)
hipError_t attn_mfma_prepare(int hd);
hipError_t launch_attn_mfma(const void* q, const void* kc, const void* vc, int cap, int n, int M, TreeDev tree, int Hq,
                            int Hkv, int hd, void* out, void* scratch, hipStream_t s, const int32_t* n_dev = nullptr);
// up to 128 rows as the caller has them: rotary at positions n + depth[m], append at slots n + m, attention, in one launch (and
// the merge of key slices); depth[m] <= m, as in every tree whose parents come before their children
bool attn_fresh_supported(int M, int Hq, int Hkv, int hd);
hipError_t launch_attn_fresh(const void* q, const void* k_new, const void* v_new, const int32_t* depth, float base, void* kc, void* vc,
                             int cap, int n, int M, TreeDev tree, int Hq, int Hkv, int hd, void* out, void* scratch, hipStream_t s);
hipError_t launch_attn_causal(const void* q, const void* kc, const void* vc, int cap, int n, int rows, TreeDev tree, int Hq, int Hkv,
                              int hd, void* out, hipStream_t s, const void* self_k = nullptr, const void* self_v = nullptr,
                              int self_cap = 0, void* scratch = nullptr);
size_t attn_causal_scratch_bytes(int rows, int Hq, int hd);

}  // namespace ht
