// Shared device helpers and the internal launch interface of the kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/autochunk_rt.h"

namespace ac {

typedef __bf16 bf16_t;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;

__device__ __forceinline__ float bf2f(bf16_t v) { return static_cast<float>(v); }
__device__ __forceinline__ bf16_t f2bf(float v) { return static_cast<bf16_t>(v); }  // nearest-even

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kVec = 4;  // elements per 16-byte access
  __device__ static __forceinline__ float ld(const float* p) { return *p; }
  __device__ static __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  static constexpr int kVec = 8;
  __device__ static __forceinline__ float ld(const bf16_t* p) { return bf2f(*p); }
  __device__ static __forceinline__ void st(bf16_t* p, float v) { *p = f2bf(v); }
};

// 16-byte vector load / store of kVec elements, widened to fp32.
__device__ __forceinline__ void load_vec(const float* p, float (&v)[4]) {
  f32x4 t = *reinterpret_cast<const f32x4*>(p);
  v[0] = t[0]; v[1] = t[1]; v[2] = t[2]; v[3] = t[3];
}
__device__ __forceinline__ void load_vec(const bf16_t* p, float (&v)[8]) {
  bf16x8 t = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = bf2f(t[i]);
}
__device__ __forceinline__ void store_vec(float* p, const float (&v)[4]) {
  f32x4 t = {v[0], v[1], v[2], v[3]};
  *reinterpret_cast<f32x4*>(p) = t;
}
__device__ __forceinline__ void store_vec(bf16_t* p, const float (&v)[8]) {
  bf16x8 t;
#pragma unroll
  for (int i = 0; i < 8; ++i) t[i] = f2bf(v[i]);
  *reinterpret_cast<bf16x8*>(p) = t;
}

// erf by the rational-exponential form of Abramowitz & Stegun 7.1.26 (|error| <= 1.5e-7):
// two quarter-rate ops (reciprocal, exp2) and a degree-5 Horner chain, about half the
// instructions of the library erff, which matters in a GEMM epilogue run on every element.
__device__ __forceinline__ float erf_as(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  float p = fmaf(1.061405429f, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  p *= t;
  const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * ax * ax);
  return copysignf(fmaf(-p, e, 1.0f), x);
}
__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erf_as(x * 0.70710678118654752f)); }
__device__ __forceinline__ float sigmoidf(float x) { return 1.0f / (1.0f + __expf(-x)); }

// The same by the hardware reciprocal and one Newton step, for the GEMM epilogues: 8 instructions where the division takes 13
// (q, k, v, gate and bias of 65536 rows of 128: 26.7 us; 27.7 with the division, 26.1 with the bare reciprocal).
// A quarter of the denominator is inverted, so that all of its range up to 2^128 has a normal reciprocal; the residual's clamp is
// for an infinite denominator (0 * inf) and lets NaN through.  Equal to sigmoidf for every fp32 input but for 33945 between
// -87.3 and -88.8, whose subnormal result is rounded twice (all 2^32 inputs compared; the bare reciprocal differs for 33
// million of them).
__device__ __forceinline__ float sigmoid_newton(float x) {
  const float d = fmaf(0.25f, __expf(-x), 0.25f), r = __builtin_amdgcn_rcpf(d);
  return 0.25f * fmaf(__builtin_amdgcn_fmed3f(fmaf(-d, r, 1.0f), -1.0f, 1.0f), r, r);
}

// GELU, tanh form: x (1 + tanh u) / 2 = max(x, 0) - |x| / (1 + e^(2|u|)) with u = sqrt(2/pi) (x + 0.044715 x^3), the denominator inverted
// as above.  14 instructions, where tanhf is a division, an exponential and two branches: what bounds the epilogue of a product is vector work
// (4000 x 4096 x 1024 57 -> 48 us).  Against 64 bits over N(0, 1): 2.8e-8 in 2-norm and 2.4e-7 at most, with tanhf 3.8e-8
// and 4.1e-7.  (From |x| = 16 on the second term is 0, and the clamp keeps inf * 0 out; x / 2 + |x| / 2 is NaN for -inf, as the product form is.)
__device__ __forceinline__ float gelu_tanh(float x) {
  const float a = fabsf(x);
  const float t = a * fmaf(x * x, 0.102943240f, 2.302208198f);        // 2 |u| log2 e
  const float d = fmaf(0.25f, __builtin_amdgcn_exp2f(t), 0.25f), r = __builtin_amdgcn_rcpf(d);
  const float s = 0.25f * fmaf(__builtin_amdgcn_fmed3f(fmaf(-d, r, 1.0f), -1.0f, 1.0f), r, r);
  return fmaf(-fminf(a, 16.0f), s, fmaf(0.5f, a, 0.5f * x));
}

template <int ACT> __device__ __forceinline__ float apply_act_bf16(float x) {
  if (ACT == AC_ACT_GELU_ERF) return gelu_erf(x);
  if (ACT == AC_ACT_GELU_TANH) return gelu_tanh(x);
  if (ACT == AC_ACT_RELU) return fmaxf(x, 0.0f);
  if (ACT == AC_ACT_SIGMOID) return sigmoid_newton(x);
  if (ACT == AC_ACT_SILU) return x * sigmoid_newton(x);
  return x;
}
__device__ __forceinline__ float apply_act_rt(float x, int act) {
  switch (act) {
    case AC_ACT_GELU_ERF: return gelu_erf(x);
    case AC_ACT_GELU_TANH: return gelu_tanh(x);
    case AC_ACT_RELU: return fmaxf(x, 0.0f);
    case AC_ACT_SIGMOID: return sigmoidf(x);
    case AC_ACT_SILU: return x * sigmoidf(x);
    default: return x;
  }
}

// GELU (erf form) from a table in LDS.  gelu(x) = x/2 + |x| h(|x|) with h(a) = erf(a / sqrt 2) / 2,
// and h is read from 385 entries (value, step to the next) at a spacing of 1/64, interpolated
// linearly: |error of h| <= (1/64)^2 / 8 * max|h''| = 7.4e-6, and from |x| = 6 on h is 1/2 to
// fp32.  Nine instructions and one LDS read per element instead of a reciprocal, an exponential
// and a dozen more, which matters because the epilogue of an 8-wave tile overlaps with nothing.
constexpr int kGeluEntries = 385;
constexpr size_t kGeluTableBytes = (size_t)kGeluEntries * 2 * sizeof(float);
__device__ __forceinline__ void gelu_table_fill(float* tab, int tid, int nt) {
  for (int i = tid; i < kGeluEntries; i += nt) {
    const float h0 = 0.5f * erf_as((float)i * (0.70710678118654752f / 64.0f));
    const float h1 = i + 1 < kGeluEntries ? 0.5f * erf_as((float)(i + 1) * (0.70710678118654752f / 64.0f)) : h0;
    tab[2 * i] = h0;
    tab[2 * i + 1] = h1 - h0;
  }
}
__device__ __forceinline__ float gelu_table(float x, const float* tab) {
  const float a = fabsf(x);
  const float u = a * 64.0f;
  unsigned idx = (unsigned)u;                       // saturating conversion
  idx = idx < (unsigned)(kGeluEntries - 1) ? idx : (unsigned)(kGeluEntries - 1);
  const f32x2 e = *reinterpret_cast<const f32x2*>(tab + 2 * idx);
  const float h = fmaf(e[1], __builtin_amdgcn_fractf(u), e[0]);
  return fmaf(a, h, 0.5f * x);
}

// m = q * period + r for a row index m < 2^31 (the launchers refuse more rows): a 32-bit division,
// a fraction of the instructions and registers of the 64-bit one.  A period of 2^31 or more (the
// "no period" value) gives q = 0, r = m.
__device__ __forceinline__ void split_row(int64_t m, int64_t period, int64_t& q, int64_t& r) {
  if (period > 0x7fffffffLL) { q = 0; r = m; return; }
  const uint32_t qq = (uint32_t)m / (uint32_t)period;
  q = qq;
  r = (int64_t)((uint32_t)m - qq * (uint32_t)period);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
// Sum over groups of G consecutive lanes (G a power of two <= 64).  Within sixteen lanes by rotations of the row: once lanes 8 apart hold the same sum
// a rotation by 4 is an exchange of lanes 4 apart, and so on, the sums (and bits) of the exchanges at no trip through LDS.
template <int N> __device__ __forceinline__ float rotate_row(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + N, 0xf, 0xf, true));
}
template <int G> __device__ __forceinline__ float group_sum(float v) {
  if constexpr (G >= 64) v += __shfl_xor(v, 32, 64);
  if constexpr (G >= 32) v += __shfl_xor(v, 16, 64);
  if constexpr (G >= 16) {
    v += rotate_row<8>(v);
    v += rotate_row<4>(v);
    v += rotate_row<2>(v);
    v += rotate_row<1>(v);
  } else {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  }
  return v;
}

// ---------------------------------------------------------------------------------------
// Launch interface used by the executor and by the ac_op_* entry points.
// ---------------------------------------------------------------------------------------

enum { kCausalColumns = 1, kCausalDepth = 2 };
struct LinearArgs {
  const void* a; int64_t lda;        // [m, k]
  const void* w; int64_t ldw;        // [n, k]
  const void* bias;                  // [n] or null
  const void* mul; int64_t ldmul;    // [m, n] or null
  const void* resid; int64_t ldr;    // [m, n] or null
  void* out; int64_t ldo;            // columns [0, n_split): out[m * ldo + n], or, with o_period > 0,
                                     // out[(m / o_period) * o_s1 + (m % o_period) * o_s2 + n]: rows regrouped
                                     // on the way out (e.g. positions (k, j) of a pair tensor stored as (j, k))
  int64_t o_period, o_s1, o_s2;
  // columns [n_split, n): out_t[(m / t_period) * t_s1 + (m % t_period) * t_s2 + (n - n_split) * t_s3]
  void* out_t; int64_t n_split; int64_t t_period, t_s1, t_s2, t_s3;
  int64_t m, n, k;
  int act;
  int dtype;
  // batch > 1: `batch` independent products; a, w and out advance by these strides (elements).
  // bias / mul / resid / out_t must be null then.
  int64_t batch, sa_b, sw_b, so_b;
  // batch > 1: nonzero = blocks take the products last to first.  Results are the same; a caller that runs
  // the same operands launch after launch alternates the direction so that each launch starts with the
  // products whose operands the one before touched last (they are the ones still in the memory-side cache).
  int batch_descending;
  // conv_c > 0: a is a stack of channels-last images [m / (conv_h * conv_w)][conv_h][conv_w][conv_c] and the
  // product is their 3x3 convolution (stride 1, zero padding 1): row m is a pixel, k = 9 * conv_c runs over
  // (window row, window column, input channel), w is [n][3][3][conv_c].  lda is ignored (= conv_c).
  int conv_h, conv_w, conv_c;
  // causal (bf16 matrix-core kernels only: linear_takes_causal): row m stands at position q_offset + m.  kCausalColumns: columns past a row's
  // position may be left unwritten; kCausalDepth: a's terms past a row's position are zeros and may be left out.
  int causal;
  int64_t q_offset;
  // gate > 0 (where linear_takes_gate: erf GELU): w and bias hold n = `gate` value rows and then as many gate rows, and out = value * act(gate).
  int64_t gate;
  // bias_period > 0: row m takes bias row m / bias_period (bias is [m / bias_period][n]): one bias vector per image
  int64_t bias_period;
};

struct AttnArgs {
  const void* q; int64_t ldq, sq_b;
  const void* k; int64_t ldk, sk_b;
  // v_transposed: v is vt[(h * head_dim + d) * ldv + key]; else row-major v[key * ldv + h * head_dim + d].
  const void* v; int64_t ldv, sv_b; int v_transposed;
  const void* bias; int64_t ld_bias, s_bias_h;   // bias[h * s_bias_h + (row) * ld_bias + key]
  const void* gate; int64_t ldg, sg_b;
  void* ctx; int64_t ldc, sc_b;
  int64_t batch, sq, sk;
  int heads, head_dim, causal;
  int64_t q_offset;
  int dtype;
  // n_splits > 1: the keys each query block sees are cut into n_splits runs handled by
  // separate blocks; partial results go to part_o [split][b][row][head][d] (fp32) and
  // part_ml [split][b][row][head][2] (running max, sum) and are merged by a second kernel.
  int n_splits;
  void* part_o;
  void* part_ml;
  int head_major;   // block order (head, problem, query block) instead of (problem, head, query block); set by launch_attention
};

// LayerNorm of short rows followed by several projections of the normalised rows, in one
// kernel: t = LN(x) stays on chip and every part computes act(t w^T + bias) or, for a gated
// pair, sigmoid(t w_gate^T + bias_gate) * (t w^T + bias), each with its own output layout.
constexpr int kMaxProjParts = 5;
constexpr int kMaxProjTiles = 48;
struct ProjPart {
  const void* w; const void* bias;             // [n, K], [n] or null
  const void* w_gate; const void* bias_gate;   // of a gated pair
  int gated;                                   // 1: out = sigmoid(t w_gate^T + bias_gate) * (t w^T + bias)
  int act;                                     // of a plain part
  int64_t n;
  void* out; int64_t ldo, o_period, o_s1, o_s2;            // row-major store (rows regrouped if o_period > 0), or
  void* out_t; int64_t t_period, t_s1, t_s2, t_s3;          // strided store of the whole part (see LinearArgs)
};
struct LnProjArgs {
  const void* x; int64_t ldx;      // [rows, K]; with x_period > 0 row r lies at x[(r / x_period) * x_s1 + (r % x_period) * x_s2]
  int64_t x_period, x_s1, x_s2;
  const void* gain; const void* shift; float eps;
  int64_t rows; int64_t k;
  int n_parts;
  ProjPart part[kMaxProjParts];
};
// Shapes the kernel covers (bf16, K = 64 or 128, every n a multiple of 4); a pure function of the
// shapes so that planning and execution take the same path.
bool ln_proj_shapes_ok(int dtype, int64_t k, const int64_t* n, int n_parts);
hipError_t launch_ln_proj(const LnProjArgs& p, hipStream_t s);

hipError_t launch_layernorm(const void* x, int64_t ldx, const void* gain, const void* shift, void* y,
                            int64_t ldy, int64_t rows, int64_t cols, float eps, int dtype,
                            hipStream_t s);
hipError_t launch_bias_act(const void* x, int64_t ldx, const void* bias, void* y, int64_t ldy,
                           int64_t rows, int64_t cols, int act, int dtype, hipStream_t s);
// y = a + b (op 0), a * b (op 1) or a * act(b) (op kOpGate + act)
constexpr int kOpGate = 16;
hipError_t launch_binary(const void* a, int64_t lda, const void* b, int64_t ldb, void* y, int64_t ldy,
                         int64_t rows, int64_t cols, int op, int dtype, hipStream_t s);
hipError_t launch_linear(const LinearArgs& g, hipStream_t s);
bool linear_takes_causal(const LinearArgs& g);
bool linear_takes_gate(const LinearArgs& g);
const char* linear_kernel_name(int64_t m, int64_t n, int64_t k, int64_t lda, int64_t ldw, int64_t batch, bool conv, int dtype);
// The end of a triangle update of rows of z (contiguous, bf16): out = z + sigmoid(LN(z) w_g^T + b_g) * (LN(o) w_o^T + b_o) with o channel-major,
// o[c * stride_c + row].  Row r of the result goes to (r / o_period) * o_s1 + (r % o_period) * o_s2 (o_period <= 0: r * c_z).
struct TriMulOutArgs {
  const void *z, *ln_in_g, *ln_in_b, *w_g, *b_g;
  const void* o; int64_t stride_c; const void *ln_out_g, *ln_out_b, *w_o, *b_o;
  void* out; int64_t o_period, o_s1, o_s2;
  int64_t rows, c_z, c_hidden;
  float eps;
};
bool trimul_out_shapes_ok(int dtype, int64_t c_z, int64_t c_hidden, int64_t row_unit);   // segments of whole multiples of `row_unit` rows
hipError_t launch_trimul_out(const TriMulOutArgs& p, hipStream_t s);
// out = z + act(LN(z) w_1^T + b_1) w_2^T + b_2 on rows of z, the hidden rows on chip; rows of the result as above.
struct TransitionArgs {
  const void *z, *ln_g, *ln_b, *w_1, *b_1, *w_2, *b_2;
  void* out; int64_t o_period, o_s1, o_s2;
  int64_t rows, c_z, hidden;
  int act;
  float eps;
};
bool transition_shapes_ok(int dtype, int64_t c_z, int64_t hidden, int act);
int64_t transition_least_rows(int64_t c_z, int64_t hidden, int act);
hipError_t launch_transition(const TransitionArgs& p, hipStream_t s);
// fp32 layers of few channels; rows contiguous.  out[rows, n] = LN(x) w^T + bias (64 or 128 channels, n in multiples of 64), and (32, 64 or 128)
// h = resid + ctx w_o^T + b_o; out = h + act(LN(h) w_1^T + b_1) w_2^T + b_2 with a feed-forward of 4 d columns.
struct LnLinearF32Args { const void *x, *gain, *shift, *w, *bias; void* out; int64_t rows, d, n; float eps; };
struct LayerTailF32Args { const void *ctx, *resid, *w_o, *b_o, *ln_g, *ln_b, *w_1, *b_1, *w_2, *b_2; void* out; int64_t rows, d; int act; float eps; };
bool ln_linear_f32_shapes_ok(int dtype, int64_t d, int64_t n);
hipError_t launch_ln_linear_f32(const LnLinearF32Args& p, hipStream_t s);
bool layer_tail_f32_shapes_ok(int dtype, int64_t d, int64_t hidden);
bool layer_tail_f32_ahead(int64_t d, int64_t launch_rows, int64_t rows);
hipError_t launch_layer_tail_f32(const LayerTailF32Args& p, hipStream_t s);
// GroupNorm (+ SiLU) of channels-last images [images, positions, channels]; partials: group_norm_workspace_bytes()
uint64_t group_norm_workspace_bytes(int64_t images, int groups);
hipError_t launch_group_norm(const void* x, const void* gain, const void* shift, void* y, void* partials, int64_t images,
                             int64_t positions, int channels, int groups, float eps, int act, int dtype, hipStream_t s);
// p = softmax(scale * s [causal]) over stored rows; row r is query r mod period at position
// q_offset + (r mod period).  A causal row's zeros are written up to the end of the row, or (row_tile > 0) as far as a
// kCausalDepth product of tiles of at most row_tile rows reads them.
hipError_t launch_softmax_rows(const void* src, int64_t lds, void* dst, int64_t ldd, int64_t rows, int64_t cols,
                               float scale, int causal, int64_t q_offset, int64_t period, int row_tile, int dtype, hipStream_t s);
hipError_t launch_attention(const AttnArgs& a, hipStream_t s);
int attention_key_splits(int64_t sq, int64_t sk, int heads, int64_t batch, int head_dim, int dtype, int v_transposed);
uint64_t attention_split_workspace_bytes(int64_t sq, int heads, int64_t batch, int head_dim, int n_splits);
// Row-major value matrix [keys, cols] -> transposed copy [cols, keys] (bf16), for callers
// of the attention entry point that hold v row-major.
hipError_t launch_transpose(const void* src, int64_t lds, void* dst, int64_t ldd, int64_t rows,
                            int64_t cols, int dtype, hipStream_t s);
// In-place transpose of `batch` square [n, n] matrices (row stride ld, `stride_b` apart).
hipError_t launch_transpose_square_inplace(void* data, int64_t ld, int64_t stride_b, int64_t n,
                                           int64_t batch, int dtype, hipStream_t s);
// dst[jj][i][:] = z[i][j0 + jj][:] for a pair tensor z[n][n][c] (the copy behind a column chunk).
hipError_t launch_gather_columns(const void* src, void* dst, int64_t n, int64_t c, int64_t j0, int64_t nj, int dtype,
                                 hipStream_t s);
// LayerNorm over channels of a channel-major tensor: src[c * stride_c + p] -> dst[p * ldd + c].
hipError_t launch_layernorm_channel_major(const void* src, int64_t stride_c, const void* gain,
                                          const void* shift, void* dst, int64_t ldd, int64_t positions,
                                          int64_t channels, float eps, int dtype, hipStream_t s);

// hipErrorInvalidValue-style refusal with a message for ac_last_error().
void set_error(const char* fmt, ...);

}  // namespace ac
