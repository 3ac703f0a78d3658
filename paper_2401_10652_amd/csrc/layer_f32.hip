// fp32 transformer layers of few channels: LayerNorm + packed projection in one kernel (64 or 128), and all that follows the attention core (output
// projection, residual, LayerNorm, feed-forward, residual) in another (32, 64 or, for some row counts, 128, the feed-forward four times as wide).  With the
// attention core 64 channels take three launches, 32, whose 96 packed columns are no multiple of 64, four.
//
// What bounds such a layer is the number of its launches, 3 to 5 us each whatever they do, and inside a launch the latency of loads and of the chain
// over k.  Both kernels therefore keep 16 rows of a block on chip from one step to the next, read weights (L2) straight into registers several matrix
// instructions ahead and across barriers, and run the four parts of a sum over k (linear_mfma_f32 gives each to a wave) as four independent
// chains of one wave, added in the same order: the bits are those of the separate kernels.
// 256 rows of 64 channels, one layer: 29.8 us in seven launches, 17.4 in three (3.5 + 5.4 + 9.5 on the device).
#include "common.h"

namespace ac {

constexpr int kRows = 16;     // rows per block

// 16 x 16 tiles of a product of 16 rows with TILES * 16 weight rows of K terms; wave w takes tiles w, w + 4, ...  A group is one step of 16 terms in each
// of the RUNS parts of k; a wave's groups go tile by tile, PD of them in flight.
template <int K, int TILES, int PD> struct RowProduct {
  static constexpr int RUNS = K / 16 < 4 ? K / 16 : 4, STEPS = K / 16 / RUNS, NT = (TILES + 3) / 4, GROUPS = NT * STEPS;
  const float* base;          // this lane's 4 terms of the first step of its weight row of tile `wave`
  int wave, l16, grp;
  f32x4 w[PD][RUNS], bias[NT];
  // term offset of step s of part r
  static __device__ __forceinline__ int term(int r, int s) { return (r * STEPS + s) * 16; }
  __device__ __forceinline__ bool active() const { return wave < TILES; }
  __device__ __forceinline__ void fetch(int g) {
#pragma unroll
    for (int r = 0; r < RUNS; ++r) w[g % PD][r] = *reinterpret_cast<const f32x4*>(base + (int64_t)(g / STEPS) * 64 * K + term(r, g % STEPS));
  }
  __device__ __forceinline__ void start(const float* weight, const float* biases, int wave_, int l16_, int grp_) {
    wave = wave_; l16 = l16_; grp = grp_;
    base = weight + (int64_t)((wave < TILES ? wave : 0) * 16 + l16) * K + 4 * grp;
#pragma unroll
    for (int g = 0; g < PD && g < GROUPS; ++g) fetch(g);
#pragma unroll
    for (int t = 0; t < NT; ++t) bias[t] = *reinterpret_cast<const f32x4*>(biases + (wave < TILES ? t * 4 + wave : 0) * 16 + 4 * grp);
  }
  // rows: this lane's 4 terms of row l16 at term 0 (LDS or memory); sink(tile of the wave, first column, sums + bias)
  template <typename S> __device__ __forceinline__ void run(const float* rows, S&& sink) {
    f32x4 acc[RUNS];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
      if (g % STEPS == 0) {
#pragma unroll
        for (int r = 0; r < RUNS; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      f32x4 a[RUNS];
#pragma unroll
      for (int r = 0; r < RUNS; ++r) a[r] = *reinterpret_cast<const f32x4*>(rows + term(r, g % STEPS));
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int r = 0; r < RUNS; ++r) acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[g % PD][r][e], a[r][e], acc[r], 0, 0, 0);
      if (g + PD < GROUPS) fetch(g + PD);
      __builtin_amdgcn_sched_barrier(0);
      if (g % STEPS == STEPS - 1) {
        f32x4 v = acc[0];
#pragma unroll
        for (int r = 1; r < RUNS; ++r)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += acc[r][e];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += bias[g / STEPS][e];
        if (active()) sink(g / STEPS, (g / STEPS * 4 + wave) * 16 + 4 * grp, v);
      }
    }
  }
};

__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// LayerNorm of the block's rows into LDS (rows D + 4 apart), D / 4 lanes per row, each with the gain and shift of its columns; row(r) is where row r lies.
template <int D, typename R> __device__ __forceinline__ void normalise_rows(R&& row, f32x4 g, f32x4 b, float eps, float* dst, int tid) {
  constexpr int G = D / 4, RPP = 256 / G;
  const int lg = tid % G;
#pragma unroll
  for (int r0 = 0; r0 < kRows; r0 += RPP) {
    const int r = r0 + tid / G;
    if (r >= kRows) break;
    const f32x4 v = ld4(row(r) + lg * 4);
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) sum += v[j];
    const float mean = group_sum<G>(sum) * (1.0f / D);
#pragma unroll
    for (int j = 0; j < 4; ++j) { const float d = v[j] - mean; sq += d * d; }
    const float rstd = rsqrtf(group_sum<G>(sq) * (1.0f / D) + eps);
    f32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (v[j] - mean) * rstd * g[j] + b[j];
    *reinterpret_cast<f32x4*>(dst + r * (D + 4) + lg * 4) = o;
  }
}

// out[rows, n] = LN(x) w^T + bias; blocks of the same rows share out the runs of 64 columns.
template <int D>
__global__ void __launch_bounds__(256) ln_linear_f32(LnLinearF32Args p) {
  __shared__ __attribute__((aligned(16))) float s_u[kRows * (D + 4)];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, l16 = lane % 16, grp = lane / 16;
  const int64_t m0 = (int64_t)blockIdx.x * kRows;
  const float *x = (const float*)p.x, *w = (const float*)p.w, *bias = (const float*)p.bias;
  const int runs = (int)(p.n / 64), lo = runs * (int)blockIdx.y / (int)gridDim.y, hi = runs * ((int)blockIdx.y + 1) / (int)gridDim.y;
  RowProduct<D, 4, 1> q;
  q.start(w + (int64_t)lo * 64 * D, bias + lo * 64, wave, l16, grp);
  const int lg = tid % (D / 4) * 4;
  normalise_rows<D>([&](int r) { return x + (m0 + r < p.rows ? m0 + r : p.rows - 1) * D; }, ld4((const float*)p.gain + lg), ld4((const float*)p.shift + lg), p.eps, s_u, tid);
  __syncthreads();
  for (int t = lo; t < hi; ++t) {
    q.run(s_u + l16 * (D + 4) + 4 * grp, [&](int, int c, f32x4 v) {
      if (m0 + l16 < p.rows) *reinterpret_cast<f32x4*>((float*)p.out + (m0 + l16) * p.n + t * 64 + c) = v;
    });
    if (t + 1 < hi) q.start(w + (int64_t)(t + 1) * 64 * D, bias + (t + 1) * 64, wave, l16, grp);
  }
}

// h = resid + ctx w_o^T + b_o;  out = h + act(LN(h) w_1^T + b_1) w_2^T + b_2.  (A block has read its rows of ctx and resid before it writes them: out may
// be either.)
template <int D>
__global__ void __launch_bounds__(256) layer_tail_f32(LayerTailF32Args p) {
  constexpr int F = 4 * D, HROW = D + 4, FROW = F + 4;
  __shared__ __attribute__((aligned(16))) float s_h[kRows * HROW], s_u[kRows * HROW], s_f[kRows * FROW];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, l16 = lane % 16, grp = lane / 16;
  const int64_t m0 = (int64_t)blockIdx.x * kRows, row = m0 + l16 < p.rows ? m0 + l16 : p.rows - 1;   // rows past the end shadow the last one; never stored
  RowProduct<D, D / 16, 2> o;
  RowProduct<D, F / 16, 4> up;
  RowProduct<F, D / 16, 4> down;
  o.start((const float*)p.w_o, (const float*)p.b_o, wave, l16, grp);
  f32x4 resid[o.NT];
#pragma unroll
  for (int t = 0; t < o.NT; ++t) resid[t] = ld4((const float*)p.resid + row * D + (o.active() ? t * 4 + wave : 0) * 16 + 4 * grp);
  const int lg = tid % (D / 4) * 4;
  const f32x4 gain = ld4((const float*)p.ln_g + lg), shift = ld4((const float*)p.ln_b + lg);
  up.start((const float*)p.w_1, (const float*)p.b_1, wave, l16, grp);
  o.run((const float*)p.ctx + row * D + 4 * grp, [&](int t, int c, f32x4 v) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] += resid[t][j];
    *reinterpret_cast<f32x4*>(s_h + l16 * HROW + c) = v;
  });
  __syncthreads();
  down.start((const float*)p.w_2, (const float*)p.b_2, wave, l16, grp);
  normalise_rows<D>([&](int r) { return s_h + r * HROW; }, gain, shift, p.eps, s_u, tid);
  __syncthreads();
  up.run(s_u + l16 * HROW + 4 * grp, [&](int, int c, f32x4 v) {
    if (p.act == AC_ACT_GELU_ERF) {      // (one branch per four values)
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = gelu_erf(v[j]);
    } else if (p.act == AC_ACT_GELU_TANH) {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = gelu_tanh(v[j]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = fmaxf(v[j], 0.0f);
    }
    *reinterpret_cast<f32x4*>(s_f + l16 * FROW + c) = v;
  });
  __syncthreads();
  down.run(s_f + l16 * FROW + 4 * grp, [&](int, int c, f32x4 v) {
    const f32x4 h = ld4(s_h + l16 * HROW + c);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] += h[j];
    if (m0 + l16 < p.rows) *reinterpret_cast<f32x4*>((float*)p.out + row * D + c) = v;
  });
}

bool ln_linear_f32_shapes_ok(int dtype, int64_t d, int64_t n) { return dtype == AC_F32 && (d == 64 || d == 128) && n >= 64 && n % 64 == 0 && n <= 65536; }
bool layer_tail_f32_shapes_ok(int dtype, int64_t d, int64_t hidden) { return dtype == AC_F32 && (d == 32 || d == 64 || d == 128) && hidden == 4 * d; }

// Whether the tail is ahead of its four launches, whose bits are the same, for launches of `launch_rows` rows in a layer of `rows`.  At 32 and 64
// channels it always is (one layer of 16 to 65536 rows, 64 channels: 14.6 to 171 us against 19.2 to 248; 32: 13.1 to 105 against 20.3 to 140).  At 128 every
// 16 rows read 576 KB of weights, one chain of loads that nothing hides while a CU has a block or two, and more than L2 gives once it has many: one layer of
// 256 rows 51.0 us against 32.1, 1024 rows 52.5 / 37.0, 2048 55.8 / 46.3, 4096 62.3 / 62.1, 6144 69.6 / 78.4, 16384 135 / 141, 32768 251 / 236, 65536 482 / 435.
bool layer_tail_f32_ahead(int64_t d, int64_t launch_rows, int64_t rows) { return d <= 64 || (launch_rows > 4096 && rows <= 20480); }

static bool at16(const void* p) { return p && (uintptr_t)p % 16 == 0; }

hipError_t launch_ln_linear_f32(const LnLinearF32Args& p, hipStream_t s) {
  if (p.rows <= 0) return hipSuccess;
  if (!ln_linear_f32_shapes_ok(AC_F32, p.d, p.n) || p.rows > 0x7fffffffLL) return hipErrorInvalidValue;
  for (const void* q : {p.x, p.gain, p.shift, p.w, p.bias, (const void*)p.out})
    if (!at16(q)) return hipErrorInvalidValue;
  // as many shares of the columns as a launch of few rows leaves places for
  const int64_t blocks = (p.rows + kRows - 1) / kRows, runs = p.n / 64, room = 1024 / blocks;
  const dim3 grid((unsigned)blocks, (unsigned)(room < 1 ? 1 : room < runs ? room : runs));
  if (p.d == 64) hipLaunchKernelGGL((ln_linear_f32<64>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((ln_linear_f32<128>), grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_layer_tail_f32(const LayerTailF32Args& p, hipStream_t s) {
  if (p.rows <= 0) return hipSuccess;
  if (!layer_tail_f32_shapes_ok(AC_F32, p.d, 4 * p.d) || p.rows > 0x7fffffffLL) return hipErrorInvalidValue;
  if (p.act != AC_ACT_GELU_ERF && p.act != AC_ACT_GELU_TANH && p.act != AC_ACT_RELU) return hipErrorInvalidValue;
  for (const void* q : {p.ctx, p.resid, p.w_o, p.b_o, p.ln_g, p.ln_b, p.w_1, p.b_1, p.w_2, p.b_2, (const void*)p.out})
    if (!at16(q)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((p.rows + kRows - 1) / kRows));
  if (p.d == 32) hipLaunchKernelGGL((layer_tail_f32<32>), grid, dim3(256), 0, s, p);
  else if (p.d == 64) hipLaunchKernelGGL((layer_tail_f32<64>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((layer_tail_f32<128>), grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

}  // namespace ac
