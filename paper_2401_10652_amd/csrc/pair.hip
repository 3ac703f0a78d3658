// Modules of the pair stack whose intermediates of a row fit on chip: the end of a triangle update (output gate, LayerNorm over the
// channels of the contraction, output projection, residual) and the transition (LayerNorm, both layers, residual).  bf16, 64 or 128
// channels.  A row's arithmetic does not depend on the launch it falls in.
#include "common.h"

namespace ac {

__device__ __forceinline__ bf16x8 ld8(const bf16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }
__device__ __forceinline__ void widen(const bf16x8& t, float (&v)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = bf2f(t[j]);
}
// One row of G * 8 values, eight of them in each of G lanes: (v - mean) / sqrt(var + eps) * gain + shift, the variance in a second pass.
template <int G> __device__ __forceinline__ bf16x8 normalise(const bf16x8& x, const bf16x8& gain, const bf16x8& shift, float eps) {
  float v[8];
  widen(x, v);
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) sum += v[j];
  const float mean = group_sum<G>(sum) * (1.0f / (8 * G));
  float sq = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) { const float d = v[j] - mean; sq += d * d; }
  const float rstd = rsqrtf(group_sum<G>(sq) * (1.0f / (8 * G)) + eps);
  bf16x8 o;
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = f2bf((v[j] - mean) * rstd * bf2f(gain[j]) + bf2f(shift[j]));
  return o;
}
// A value of this iteration: what is computed from it is not kept in registers over a loop.
template <typename V> __device__ __forceinline__ V here(V v) {
  typedef int words __attribute__((ext_vector_type(sizeof(V) / 4)));
  words w = __builtin_bit_cast(words, v);
  asm volatile("" : "+v"(w));
  return __builtin_bit_cast(V, w);
}
// Offset of row m of the result.
__device__ __forceinline__ int64_t result_row(int64_t m, int64_t period, int64_t s1, int64_t s2, int cz) {
  if (period == INT64_MAX) return m * cz;
  int64_t q, r;
  split_row(m, period, q, r);
  return q * s1 + r * s2;
}

// ------------------------------------------------------------------------------------
// The end of a triangle update.
// As three launches (LayerNorm + gate, LayerNorm over channels, projection with gate and residual) this moves eight times the pair tensor; here it
// is read once with the contraction's result and written once.  Both weights stay in registers, a wave's 32 output columns of each, for all the
// row tiles that a block walks, so LDS holds rows only and the loads of the next tile are in flight during this one.  The contraction's result is
// channel-major: two channels of a position go to LDS as one word, the 16-byte slots of a row permuted so that the writes of a wave meet every bank.
// 524288 rows of 128 and 128 channels: 90 + 83 + 136 us as three launches, 135 as one (3.0 TB/s; what bounds it is vector work, 1270 instructions a
// wave and tile, most of them the two LayerNorms and the widening of bf16); 40000 rows 28 and 19.
// ------------------------------------------------------------------------------------
template <int K, int C>
__global__ void __launch_bounds__(256, 2) trimul_out_bf16(TriMulOutArgs p) {
  constexpr int BM = 64, NT = 256, ZROW = K + 8, OROW = C + 8;
  constexpr int G = K / 8, RPP = NT / G, PZ = BM / RPP;        // lanes per row of z, rows per pass, passes
  constexpr int GO = C / 8, RPO = NT / GO, PO = BM / RPO;      // the same of the contraction's rows
  constexpr int WN = K / 32, WM = 4 / WN, SUB = 2 / WM;        // waves along columns and rows, 32-row tiles of a wave
  constexpr int ITEMS = C / 2 * (BM / 8) / NT;                 // (channel pair, run of eight positions) per thread
  __shared__ __attribute__((aligned(16))) bf16_t sZ[BM * ZROW];   // the rows of z; then of the result
  __shared__ __attribute__((aligned(16))) bf16_t sA[BM * ZROW];   // normalised
  __shared__ __attribute__((aligned(16))) bf16_t sO[BM * OROW];   // the contraction's rows, then normalised
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, wave_m = wave / WN, wave_n = wave % WN, l32 = lane % 32, half = lane / 32;
  const bf16_t *z = (const bf16_t*)p.z, *o = (const bf16_t*)p.o;
  bf16x8 wg[K / 16], wo[C / 16];
#pragma unroll
  for (int ks = 0; ks < K / 16; ++ks) wg[ks] = ld8((const bf16_t*)p.w_g + (wave_n * 32 + l32) * K + half * 8 + ks * 16);
#pragma unroll
  for (int ks = 0; ks < C / 16; ++ks) wo[ks] = ld8((const bf16_t*)p.w_o + (wave_n * 32 + l32) * C + half * 8 + ks * 16);
  const int col = wave_n * 32 + 4 * half;                      // this lane's columns: col + 8 q + 0..3
  bf16x4 bg[4], bo[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    bg[q] = *reinterpret_cast<const bf16x4*>((const bf16_t*)p.b_g + col + 8 * q);
    bo[q] = *reinterpret_cast<const bf16x4*>((const bf16_t*)p.b_o + col + 8 * q);
  }
  const int lz = tid % G, rz = tid / G, lo = tid % GO, ro = tid / GO;
  const bf16x8 g_in = ld8((const bf16_t*)p.ln_in_g + lz * 8), b_in = ld8((const bf16_t*)p.ln_in_b + lz * 8);
  const bf16x8 g_out = ld8((const bf16_t*)p.ln_out_g + lo * 8), b_out = ld8((const bf16_t*)p.ln_out_b + lo * 8);
  const int run = tid % (BM / 8), pair = tid / (BM / 8);       // (of item i: pair + 32 i)

  bf16x8 zr[PZ], orr[ITEMS][2];
  auto load = [&](int64_t m0) {
#pragma unroll
    for (int ps = 0; ps < PZ; ++ps) {
      int64_t r = m0 + ps * RPP + rz;
      if (r > p.rows - 1) r = p.rows - 1;                      // rows past the end shadow the last one; never stored
      zr[ps] = ld8(z + r * K + lz * 8);
    }
    const int64_t pos = m0 + run * 8 < p.rows ? m0 + run * 8 : 0;   // (whole runs: rows is a multiple of eight)
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
#pragma unroll
      for (int c = 0; c < 2; ++c) orr[i][c] = ld8(o + (2 * (pair + 32 * i) + c) * p.stride_c + pos);
  };
  const int64_t tiles = (p.rows + BM - 1) / BM;
  load((int64_t)blockIdx.x * BM);
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t m0 = t * BM;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int c = 2 * (pair + 32 * i), at = ((c / 8) ^ (run / 2 * 2)) * 8 + c % 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) *reinterpret_cast<bf16x2*>(sO + (run * 8 + e) * OROW + at) = bf16x2{orr[i][0][e], orr[i][1][e]};
    }
#pragma unroll
    for (int ps = 0; ps < PZ; ++ps) {
      const int at = (ps * RPP + rz) * ZROW + lz * 8;
      *reinterpret_cast<bf16x8*>(sZ + at) = zr[ps];            // (this thread read the last tile's result from there)
      *reinterpret_cast<bf16x8*>(sA + at) = normalise<G>(zr[ps], here(g_in), here(b_in), p.eps);
    }
    __syncthreads();
    if (t + gridDim.x < tiles) load((t + gridDim.x) * BM);
#pragma unroll
    for (int ps = 0; ps < PO; ++ps) {
      const int r = ps * RPO + ro;
      bf16_t* at = sO + r * OROW + (lo ^ (r / 16 * 2)) * 8;
      *reinterpret_cast<bf16x8*>(at) = normalise<GO>(ld8(at), here(g_out), here(b_out), p.eps);
    }
    __syncthreads();
#pragma unroll 1
    for (int s = 0; s < SUB; ++s) {
      const int row = (wave_m * SUB + s) * 32 + l32;
      f32x16 ag = {}, ao = {};
#pragma unroll
      for (int ks = 0; ks < K / 16; ++ks) ag = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wg[ks], ld8(sA + row * ZROW + half * 8 + ks * 16), ag, 0, 0, 0);
#pragma unroll
      for (int ks = 0; ks < C / 16; ++ks)
        ao = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wo[ks], ld8(sO + row * OROW + ((2 * ks + half) ^ (row / 16 * 2)) * 8), ao, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        bf16x4* at = reinterpret_cast<bf16x4*>(sZ + row * ZROW + col + 8 * q);
        const bf16x4 zv = *at, bgv = here(bg[q]), bov = here(bo[q]);
        bf16x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[j] = f2bf((ao[4 * q + j] + bf2f(bov[j])) * sigmoid_newton(ag[4 * q + j] + bf2f(bgv[j])) + bf2f(zv[j]));
        *at = v;
      }
    }
    __syncthreads();
#pragma unroll
    for (int ps = 0; ps < PZ; ++ps) {
      const int r = ps * RPP + rz;
      if (m0 + r < p.rows)
        *reinterpret_cast<bf16x8*>((bf16_t*)p.out + result_row(m0 + r, p.o_period, p.o_s1, p.o_s2, K) + lz * 8) = ld8(sZ + r * ZROW + lz * 8);
    }
  }
}

bool trimul_out_shapes_ok(int dtype, int64_t c_z, int64_t c_hidden, int64_t row_unit) {
  return dtype == AC_BF16 && (c_z == 64 || c_z == 128) && (c_hidden == 64 || c_hidden == 128) && row_unit % 8 == 0;
}

static bool at16(const void* p) { return p && (uintptr_t)p % 16 == 0; }

template <int K, int C> static void trimul_out_launch(const TriMulOutArgs& p, hipStream_t s) {
  // (two blocks per CU; 625 tiles take 18.9 us on 512 blocks and 20.2 on 313 of two tiles each)
  const int64_t tiles = (p.rows + 63) / 64;
  hipLaunchKernelGGL((trimul_out_bf16<K, C>), dim3((unsigned)(tiles < 512 ? tiles : 512)), dim3(256), 0, s, p);
}

hipError_t launch_trimul_out(const TriMulOutArgs& p_in, hipStream_t s) {
  TriMulOutArgs p = p_in;
  if (p.rows <= 0) return hipSuccess;
  if (!trimul_out_shapes_ok(AC_BF16, p.c_z, p.c_hidden, p.rows) || p.rows > 0x7fffffffLL || p.stride_c % 8 != 0) return hipErrorInvalidValue;
  for (const void* q : {p.z, p.ln_in_g, p.ln_in_b, p.w_g, p.b_g, p.o, p.ln_out_g, p.ln_out_b, p.w_o, p.b_o, (const void*)p.out})
    if (!at16(q)) return hipErrorInvalidValue;
  if (p.o_period <= 0) p.o_period = INT64_MAX;
  else if (p.o_s1 % 8 != 0 || p.o_s2 % 8 != 0) return hipErrorInvalidValue;
  if (p.c_z == 128) p.c_hidden == 128 ? trimul_out_launch<128, 128>(p, s) : trimul_out_launch<128, 64>(p, s);
  else p.c_hidden == 128 ? trimul_out_launch<64, 128>(p, s) : trimul_out_launch<64, 64>(p, s);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Transition.  A wave owns 32 rows, normalised in registers, and walks the hidden columns 32 at a time: the product is taken transposed (weight rows
// in the first operand), so that a lane holds hidden values of its own row, activated and rounded they are the second operand of the second product as
// they stand, and no hidden value leaves the registers.  For that the first product takes weight row pi(m) as its row m (pi swaps bits 2 and 3),
// which leaves a lane runs of eight consecutive hidden columns.  The weights of 64 hidden columns pass through LDS, twice buffered, one barrier each.
// 524288 rows of 128 channels and 512 hidden: 224 + 198 us as two launches, 167 as one (820 TFLOP/s; 175 in the compiler's own order, which reads each
// fragment right before its use); 40000 rows 31 and 23.  A CU's two blocks keep eight waves at two per SIMD.
// ------------------------------------------------------------------------------------
constexpr int kHiddenStep = 64;
constexpr int transition_buffer_elems(int k) { return kHiddenStep * (k + 8) + k * (kHiddenStep + 8); }
static size_t transition_lds(int k, int64_t hidden, int act) {
  return (2 * (size_t)transition_buffer_elems(k) + hidden) * sizeof(bf16_t) + (act == AC_ACT_GELU_ERF ? kGeluTableBytes : 0);
}

template <int K, int ACT>
__global__ void __launch_bounds__(256, 2) pair_transition_bf16(TransitionArgs p) {
  constexpr int BM = 128, NT = 256, HS = kHiddenStep, AROW = K + 8, HROW = HS + 8, BUF = transition_buffer_elems(K);
  constexpr int G = K / 8, RPP = NT / G, PASSES = BM / RPP;
  constexpr int CHUNKS = HS * K / 8 / NT;                      // 16-byte chunks of either weight tile per thread
  constexpr int NK = K / 16, NC = K / 32, AHEAD = 5;           // matrix instructions of 32 hidden columns in either product; 32-column tiles of the result
  static_assert(BM * AROW <= BUF, "the normalised rows pass through the second buffer");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16_t* buf = reinterpret_cast<bf16_t*>(smem_raw);           // [2]: w_1 rows [HS][K + 8], w_2 rows [K][HS + 8]
  bf16_t* b1 = buf + 2 * BUF;                                  // [hidden]
  float* gelu_tab = reinterpret_cast<float*>(b1 + p.hidden);
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, l32 = lane % 32, half = lane / 32;
  const int64_t m0 = (int64_t)blockIdx.x * BM;
  const bf16_t *z = (const bf16_t*)p.z, *w1 = (const bf16_t*)p.w_1, *w2 = (const bf16_t*)p.w_2;
  const int hidden = (int)p.hidden, steps = hidden / HS;
  if (ACT == AC_ACT_GELU_ERF) gelu_table_fill(gelu_tab, tid, NT);
  for (int c = tid; c < hidden / 8; c += NT) *reinterpret_cast<bf16x8*>(b1 + c * 8) = ld8((const bf16_t*)p.b_1 + c * 8);

  bf16x8 r1[CHUNKS], r2[CHUNKS];
  auto load = [&](int s) {
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int c = tid + NT * i;
      r1[i] = ld8(w1 + (int64_t)s * HS * K + c * 8);                             // (64 rows of w_1 are one run of memory)
      r2[i] = ld8(w2 + (int64_t)(c / (HS / 8)) * hidden + s * HS + c % (HS / 8) * 8);
    }
  };
  auto store = [&](bf16_t* b) {
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int c = tid + NT * i;
      *reinterpret_cast<bf16x8*>(b + c / G * AROW + c % G * 8) = r1[i];
      *reinterpret_cast<bf16x8*>(b + HS * AROW + c / (HS / 8) * HROW + c % (HS / 8) * 8) = r2[i];
    }
  };
  load(0);
  {
    const int lg = tid % G, rg = tid / G;
    const bf16x8 gain = ld8((const bf16_t*)p.ln_g + lg * 8), shift = ld8((const bf16_t*)p.ln_b + lg * 8);
    bf16x8 x[PASSES];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      int64_t r = m0 + ps * RPP + rg;
      if (r > p.rows - 1) r = p.rows - 1;                      // rows past the end shadow the last one; never stored
      x[ps] = ld8(z + r * K + lg * 8);
    }
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) *reinterpret_cast<bf16x8*>(buf + BUF + (ps * RPP + rg) * AROW + lg * 8) = normalise<G>(x[ps], gain, shift, p.eps);
  }
  store(buf);
  __syncthreads();
  bf16x8 fa[K / 16];
#pragma unroll
  for (int ks = 0; ks < K / 16; ++ks) fa[ks] = ld8(buf + BUF + (wave * 32 + l32) * AROW + half * 8 + ks * 16);
  __syncthreads();                                             // every wave has its rows: the second buffer is free
  f32x16 acc[K / 32] = {};
  const int pi = (l32 & ~12) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
  for (int s = 0; s < steps; ++s) {
    if (s + 1 < steps) load(s + 1);
    // The stage's matrix instructions in order: both 32-column halves of the first product, then of the second.  A fragment is read AHEAD
    // instructions before it is used, and a half is activated between the instructions that do not need it; the barriers pin that order.
    const bf16_t *b_1 = buf + (s & 1) * BUF + pi * AROW + half * 8, *b_2 = buf + (s & 1) * BUF + HS * AROW + l32 * HROW + half * 8;
    auto fragment = [&](int i) {
      const int u = i / NK % 2, j = i % NK;
      return i < 2 * NK ? ld8(b_1 + u * 32 * AROW + j * 16) : ld8(b_2 + j % NC * 32 * HROW + u * 32 + j / NC * 16);
    };
    f32x16 h[2] = {};
    bf16x8 bias[2][2], hv[2][2], f[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) f[i] = fragment(i);
#pragma unroll
    for (int i = 0; i < 4; ++i) bias[i / 2][i % 2] = ld8(b1 + s * HS + i * 16 + half * 8);   // (hidden columns 16 i + 8 half + 0..7 of row l32)
#pragma unroll
    for (int i = 0; i < 4 * NK; ++i) {
      const int part = i / NK, j = i % NK;
      if (part < 2) h[part] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % AHEAD], fa[j], h[part], 0, 0, 0);
      else acc[j % NC] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % AHEAD], hv[part - 2][j / NC], acc[j % NC], 0, 0, 0);
      if (i + AHEAD < 4 * NK) f[i % AHEAD] = fragment(i + AHEAD);
      if (part == 1 || part == 2) {
#pragma unroll
        for (int e = j * 16 / NK; e < (j + 1) * 16 / NK; ++e) {
          const float x = h[part - 1][e] + bf2f(bias[part - 1][e / 8][e % 8]);
          hv[part - 1][e / 8][e % 8] = f2bf(ACT == AC_ACT_GELU_ERF ? gelu_table(x, gelu_tab) : apply_act_bf16<ACT>(x));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (s + 1 < steps) store(buf + ((s + 1) & 1) * BUF);
    __syncthreads();
  }
  // bias and residual: the rows of z (again, from L2) lie in LDS while a lane adds to its own elements of them
  const int lg = tid % G, rg = tid / G;
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    int64_t r = m0 + ps * RPP + rg;
    if (r > p.rows - 1) r = p.rows - 1;
    *reinterpret_cast<bf16x8*>(buf + (ps * RPP + rg) * AROW + lg * 8) = ld8(z + r * K + lg * 8);
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < K / 32; ++c)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = c * 32 + 8 * q + 4 * half;
      const bf16x4 bias = *reinterpret_cast<const bf16x4*>((const bf16_t*)p.b_2 + col);
      bf16x4* at = reinterpret_cast<bf16x4*>(buf + (wave * 32 + l32) * AROW + col);
      const bf16x4 zv = *at;
      bf16x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = f2bf(acc[c][4 * q + j] + bf2f(bias[j]) + bf2f(zv[j]));
      *at = v;
    }
  __syncthreads();
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    const int r = ps * RPP + rg;
    if (m0 + r < p.rows)
      *reinterpret_cast<bf16x8*>((bf16_t*)p.out + result_row(m0 + r, p.o_period, p.o_s1, p.o_s2, K) + lg * 8) = ld8(buf + r * AROW + lg * 8);
  }
}

// (a hidden row of 1024 columns and the two buffers leave room for two blocks per CU)
bool transition_shapes_ok(int dtype, int64_t c_z, int64_t hidden, int act) {
  return dtype == AC_BF16 && (c_z == 64 || c_z == 128) && hidden > 0 && hidden % kHiddenStep == 0 && hidden <= 1024 &&
         (act == AC_ACT_RELU || act == AC_ACT_GELU_ERF || act == AC_ACT_GELU_TANH);
}

// Rows from which the one kernel is ahead of the two launches (LayerNorm and first layer, second layer), whose bits are the same.  A block walks the
// hidden columns by itself, 0.6 us per 64 of them with ReLU and 1.3 with GELU at 64 channels, 1.0 and 1.7 at 128, however few its rows are, where the
// two launches share them out.  us, one / two, GELU (erf), 128 channels: 512 hidden 19.2 / 11.0 at 576 rows, 19.3 / 16.1 at 6400, 19.4 / 23.1 at 10816;
// 1024 hidden 32.6 / 12.4 at 256, 33.0 / 26.5 at 9216, 33.3 / 35.6 at 14400; 128 hidden 8.5 / 9.9 at 64.  ReLU: 512 hidden 13.1 / 11.6 at 4096, 13.1 / 15.0 at
// 5184; 64 channels, 768 hidden 11.2 / 10.3 at 256, 11.4 / 14.9 at 5184.  (477 sizes, widths and activations: 7 are more than 4 % off the better one, 12 % at
// worst.)
int64_t transition_least_rows(int64_t c_z, int64_t hidden, int act) {
  const int64_t steps = hidden / kHiddenStep;
  if (act == AC_ACT_RELU) return steps <= (c_z == 64 ? 10 : 4) ? 0 : 4608;
  return steps <= (c_z == 64 ? 4 : 2) ? 0 : 4800 + 450 * steps;
}

template <int K, int ACT> static hipError_t transition_launch(const TransitionArgs& p, hipStream_t s) {
  auto kern = pair_transition_bf16<K, ACT>;
  static const hipError_t attr_status =
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)transition_lds(K, 1024, ACT));
  if (attr_status != hipSuccess) return attr_status;
  hipLaunchKernelGGL(kern, dim3((unsigned)((p.rows + 127) / 128)), dim3(256), transition_lds(K, p.hidden, ACT), s, p);
  return hipGetLastError();
}

hipError_t launch_transition(const TransitionArgs& p_in, hipStream_t s) {
  TransitionArgs p = p_in;
  if (p.rows <= 0) return hipSuccess;
  if (!transition_shapes_ok(AC_BF16, p.c_z, p.hidden, p.act) || p.rows > 0x7fffffffLL) return hipErrorInvalidValue;
  for (const void* q : {p.z, p.ln_g, p.ln_b, p.w_1, p.b_1, p.w_2, p.b_2, (const void*)p.out})
    if (!at16(q)) return hipErrorInvalidValue;
  if (p.o_period <= 0) p.o_period = INT64_MAX;
  else if (p.o_s1 % 8 != 0 || p.o_s2 % 8 != 0) return hipErrorInvalidValue;
  if (p.c_z == 128)
    return p.act == AC_ACT_RELU ? transition_launch<128, AC_ACT_RELU>(p, s)
           : p.act == AC_ACT_GELU_ERF ? transition_launch<128, AC_ACT_GELU_ERF>(p, s) : transition_launch<128, AC_ACT_GELU_TANH>(p, s);
  return p.act == AC_ACT_RELU ? transition_launch<64, AC_ACT_RELU>(p, s)
         : p.act == AC_ACT_GELU_ERF ? transition_launch<64, AC_ACT_GELU_ERF>(p, s) : transition_launch<64, AC_ACT_GELU_TANH>(p, s);
}

}  // namespace ac
