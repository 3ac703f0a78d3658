// Projection GEMMs of a chunked region: out = epilogue(a[m,k] . w[n,k]^T).
// (AutoChunk section 2.2: the QKV / output / feed-forward projections applied to one
// segment of rows; these are dense contractions and run on the bf16 matrix cores.)
//
// bf16 path: v_mfma_f32_32x32x16_bf16, block tiles of 32x64 to 256x256 by 64 k.  The weight rows
// feed the MFMA "A" operand and the activation rows the "B" operand, so that every lane ends up
// with one output row m and groups of 4 consecutive output columns n: the bias, multiplier
// and residual are then 8-byte vector accesses and the result is stored 8 bytes at a time.
// The K loop order does not depend on the tile's position in m, so a row's result is
// bitwise the same for every chunk length.
//
// fp32 path: v_mfma_f32_16x16x4_f32 on rows that can be read 16 bytes at a time.
// Odd shapes and strides of either type, and short fp32 sums of many columns: an LDS-tiled FMA kernel with full bounds checks.
#include "common.h"

#include <type_traits>

namespace ac {

// ------------------------------------------------------------------------------------
// Epilogue for one element (generic kernel) — bias, activation, multiplier, residual,
// then the row-major or the strided ("transposed") store.
// ------------------------------------------------------------------------------------
// Offset of row m in the row-major part of the output.
__device__ __forceinline__ int64_t out_row(const LinearArgs& g, int64_t m) {
  if (g.o_period == INT64_MAX) return m * g.ldo;
  int64_t q, r;
  split_row(m, g.o_period, q, r);
  return q * g.o_s1 + r * g.o_s2;
}
// Offset of row m in the strided ("transposed") part of the output.
__device__ __forceinline__ int64_t out_t_row(const LinearArgs& g, int64_t m) {
  int64_t q, r;
  split_row(m, g.t_period, q, r);
  return q * g.t_s1 + r * g.t_s2;
}

template <typename T>
__device__ __forceinline__ void epilogue_store_one(const LinearArgs& g, int64_t m, int64_t n, float v) {
  if (g.bias) v += Elem<T>::ld((const T*)g.bias + n);
  v = apply_act_rt(v, g.act);
  if (g.mul) v *= Elem<T>::ld((const T*)g.mul + m * g.ldmul + n);
  if (g.resid) v += Elem<T>::ld((const T*)g.resid + m * g.ldr + n);
  if (n < g.n_split) {
    Elem<T>::st((T*)g.out + out_row(g, m) + n, v);
  } else {
    const int64_t off = out_t_row(g, m) + (n - g.n_split) * g.t_s3;
    Elem<T>::st((T*)g.out_t + off, v);
  }
}

template <typename T>
__global__ void __launch_bounds__(256) linear_fma(LinearArgs g) {
  __shared__ float sa[16][65];
  __shared__ float sw[16][65];
  const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
  const int64_t m0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
  const T* a = (const T*)g.a + (int64_t)blockIdx.z * g.sa_b;
  const T* w = (const T*)g.w + (int64_t)blockIdx.z * g.sw_b;
  float acc[4][4] = {};
  for (int64_t k0 = 0; k0 < g.k; k0 += 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = threadIdx.x + 256 * i;
      const int row = idx / 16, kk = idx % 16;
      const bool kin = k0 + kk < g.k;
      sa[kk][row] = (kin && m0 + row < g.m) ? Elem<T>::ld(a + (m0 + row) * g.lda + k0 + kk) : 0.f;
      sw[kk][row] = (kin && n0 + row < g.n) ? Elem<T>::ld(w + (n0 + row) * g.ldw + k0 + kk) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float av[4], wv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { av[i] = sa[kk][ty * 4 + i]; wv[i] = sw[kk][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], wv[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
      if (m < g.m && n < g.n) {
        if (g.batch > 1) Elem<T>::st((T*)g.out + (int64_t)blockIdx.z * g.so_b + m * g.ldo + n, acc[i][j]);
        else epilogue_store_one<T>(g, m, n, acc[i][j]);
      }
    }
}

// ------------------------------------------------------------------------------------
// bf16 MFMA kernel, tiles staged through registers (128x128 on four waves, two blocks per CU, whose prologues and epilogues
// overlap; 64x64 and 32x64 for launches of at most one block per CU).
// ------------------------------------------------------------------------------------
constexpr int kBK = 64;            // k extent of one LDS stage
constexpr int kLdsRow = kBK + 8;   // padded row, in elements (144 bytes)
constexpr int kXcds = 8;

// Block id -> tile.  Consecutive block ids go round-robin to the 8 XCDs, each with its own
// L2; give every XCD a contiguous run of tiles, ordered in groups of 4 tile-rows so that
// tiles resident together share activation and weight panels.
// (`turn` rotates the runs among the XCDs: products whose tiles differ in work do not all give the same XCD the most.)
__device__ __forceinline__ void tile_of_block(int64_t tiles_m, int64_t tiles_n, int64_t& tm, int64_t& tn, int64_t turn = 0) {
  const int64_t nb = gridDim.x, pid = blockIdx.x;
  const int64_t q = nb / kXcds, r = nb % kXcds;
  const int64_t x = r == 0 ? (pid + turn) % kXcds : pid % kXcds, idx = pid / kXcds;
  const int64_t t = x * q + (x < r ? x : r) + idx;
  constexpr int64_t GM = 4;
  const int64_t width = GM * tiles_n;
  const int64_t group = t / width;
  const int64_t first = group * GM;
  const int64_t gsz = tiles_m - first < GM ? tiles_m - first : GM;
  tm = first + (t % width) % gsz;
  tn = (t % width) / gsz;
}

// ------------------------------------------------------------------------------------
// fp32 MFMA kernel: v_mfma_f32_16x16x4_f32, full fp32 operands and sums.
//
// What bounds it: fp32 launches here are small (a few hundred rows), so the time is the serial chain
// over k and the share of the chip's 1024 SIMDs that has a wave at all, not the 157 TFLOP/s.  Hence
// no LDS staging and no barrier in the k loop: a lane loads 16 bytes of its operand row straight
// into registers (4 consecutive k; the four lane groups of the instruction cover 16), element e of
// which is its operand of matrix instruction e, and loads run D steps ahead.  The four waves of a block
// share its output tile and take a quarter of k each (a quarter of the chain, four times the waves);
// the partial sums meet in LDS and are added in order.  Where k is cut depends on k alone, so a row's bits
// do not depend on the launch it falls in nor on the tile.
// Measured against the FMA kernel above: 64 x 64 x 256 40 -> 5.8 us, 256 x 512 x 2048 284 -> 15 us,
// 256 x 2048 x 512 78 -> 11.5 us, 1024 x 1536 x 512 86 -> 31 us.
// ------------------------------------------------------------------------------------
constexpr int kF32Runs = 4;
// Length of a run of k.
__device__ __forceinline__ int f32_run_len(int64_t k) { return (int)((k + 16 * kF32Runs - 1) / (16 * kF32Runs)) * 16; }

// bias, activation, multiplier, residual and the store for 4 consecutive columns of one row
__device__ __forceinline__ void epilogue_store_f32x4(const LinearArgs& g, bool vec, int64_t product, int64_t m, int64_t n, f32x4 v) {
  if (m >= g.m) return;
  if (vec && n + 4 <= g.n && n + 4 <= g.n_split) {
    if (g.bias) {
      const f32x4 t = *reinterpret_cast<const f32x4*>((const float*)g.bias + n);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] += t[j];
    }
    if (g.act != AC_ACT_NONE) {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = apply_act_rt(v[j], g.act);
    }
    if (g.mul) {
      const f32x4 t = *reinterpret_cast<const f32x4*>((const float*)g.mul + m * g.ldmul + n);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] *= t[j];
    }
    if (g.resid) {
      const f32x4 t = *reinterpret_cast<const f32x4*>((const float*)g.resid + m * g.ldr + n);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] += t[j];
    }
    *reinterpret_cast<f32x4*>((float*)g.out + product * g.so_b + out_row(g, m) + n) = v;
    return;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (n + j >= g.n) continue;
    if (g.batch > 1) ((float*)g.out)[product * g.so_b + m * g.ldo + n + j] = v[j];
    else epilogue_store_one<float>(g, m, n + j, v[j]);
  }
}

template <int TM, int TN>
__global__ void __launch_bounds__(256) linear_mfma_f32(LinearArgs g, int vec) {
  constexpr int BM = 16 * TM, BN = 16 * TN;   // block tile
  constexpr int D = 4;                        // k steps of 16 in flight
  __shared__ float part[kF32Runs * BM * (BN + 4)];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, l16 = lane % 16, grp = lane / 16;
  int64_t tm_, tn_;
  tile_of_block((g.m + BM - 1) / BM, (g.n + BN - 1) / BN, tm_, tn_);
  const int64_t m0 = tm_ * BM, n0 = tn_ * BN;
  const int64_t product = g.batch_descending ? (int64_t)gridDim.y - 1 - blockIdx.y : (int64_t)blockIdx.y;
  const float* a = (const float*)g.a + product * g.sa_b;
  const float* w = (const float*)g.w + product * g.sw_b;
  const float* ap[TM];
  const float* wp[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {   // rows past the end shadow the last one; never stored
    int64_t r = m0 + 16 * i + l16; if (r > g.m - 1) r = g.m - 1;
    ap[i] = a + r * g.lda;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    int64_t r = n0 + 16 * j + l16; if (r > g.n - 1) r = g.n - 1;
    wp[j] = w + r * g.ldw;
  }
  const int k = (int)g.k, run = f32_run_len(g.k);
  f32x4 acc[TM][TN];
  // operands of the 16 k from k0 on; past the end of k any valid address (nothing uses what comes)
  auto load = [&](f32x4 (&fa)[TM], f32x4 (&fw)[TN], int k0) {
    const int kk = k0 + 4 * grp, kc = kk < k ? kk : 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const f32x4*>(ap[i] + kc);
#pragma unroll
    for (int j = 0; j < TN; ++j) fw[j] = *reinterpret_cast<const f32x4*>(wp[j] + kc);
  };
  auto multiply = [&](const f32x4 (&fa)[TM], const f32x4 (&fw)[TN]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[j][e], fa[i][e], acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int lo = wave * run, hi = lo + run < k ? lo + run : k;
  if (lo < hi) {
    const int steps = (hi - lo) / 16;
    f32x4 fa[D][TM], fw[D][TN];
#pragma unroll
    for (int d = 0; d < D; ++d) load(fa[d], fw[d], lo + 16 * d);
    int s = 0;
    for (; s + D <= steps; s += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        multiply(fa[d], fw[d]);
        load(fa[d], fw[d], lo + 16 * (s + d + D));
      }
    }
#pragma unroll
    for (int d = 0; d + 1 < D; ++d)
      if (s + d < steps) multiply(fa[d], fw[d]);
    if (lo + 16 * steps < hi) {        // k ends inside a step: lane groups past the end multiply zeros
      load(fa[0], fw[0], lo + 16 * steps);
      const bool in = lo + 16 * steps + 4 * grp < hi;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) fa[0][i][e] = in ? fa[0][i][e] : 0.f;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) fw[0][j][e] = in ? fw[0][j][e] : 0.f;
      multiply(fa[0], fw[0]);
    }
  }
  // acc[i][j][r]: row m = m0 + 16 i + l16, column n = n0 + 16 j + 4 grp + r
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      *reinterpret_cast<f32x4*>(part + (wave * BM + 16 * i + l16) * (BN + 4) + 16 * j + 4 * grp) = acc[i][j];
  __syncthreads();
  for (int c = tid; c < BM * BN / 4; c += 256) {
    const int rl = c / (BN / 4), cl = (c % (BN / 4)) * 4;
    f32x4 v = *reinterpret_cast<const f32x4*>(part + rl * (BN + 4) + cl);
#pragma unroll
    for (int r = 1; r < kF32Runs; ++r) {
      const f32x4 t = *reinterpret_cast<const f32x4*>(part + (r * BM + rl) * (BN + 4) + cl);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += t[e];
    }
    epilogue_store_f32x4(g, vec, product, m0 + rl, n0 + cl, v);
  }
}

// Products over stored causal scores and probabilities: a tile whose columns lie past the positions of all its rows has nothing to do,
// and one whose rows stop seeing terms stops there (in whole steps).  16 heads of 1024 queries against 4096 keys, segment by segment: scores
// 55 -> 35 us on average, context 35 -> 20, the softmax between them 37 -> 32.
__device__ __forceinline__ bool tile_unseen(const LinearArgs& g, int64_t m0, int64_t n0, int bm) {
  return g.causal == kCausalColumns && n0 >= g.q_offset + m0 + bm;
}
__device__ __forceinline__ int64_t tile_depth(const LinearArgs& g, int64_t m0, int bm) {
  if (g.causal != kCausalDepth) return g.k;
  const int64_t seen = (g.q_offset + m0 + bm + kBK - 1) / kBK * kBK;
  return seen < g.k ? seen : g.k;
}

// Block id -> position in a 1-D list of work items such that each XCD gets a contiguous run.
__device__ __forceinline__ int64_t xcd_run(int64_t pid, int64_t nb) {
  const int64_t q = nb / kXcds, r = nb % kXcds;
  const int64_t x = pid % kXcds, idx = pid / kXcds;
  return x * q + (x < r ? x : r) + idx;
}

// The epilogue of one block.  A tile that lies wholly in the row-major part of the output
// is rounded to bf16 into LDS (free after the k loop) and written out with 16-byte stores
// whose lanes walk along rows; other tiles (strided store, narrow or misaligned outputs)
// store 8 bytes per lane straight from the registers.  GELU_TABLE: erf GELU from the table at gelu_tab, up to
// 9e-6 off at |x| = 1.4, and not by its formula (1.5e-7), which products of ragged depth keep from the FMA kernel.
constexpr int64_t kNearRow = 1 << 22;   // row strides from 0 to below: 256 rows span less than 2^31 bytes
// LDS_FREE: nobody reads `lds` any more.  Returns whether the block met at a barrier.
template <int ACT, int BM, int BN, int WAVES_M, int WAVES_N, bool GELU_TABLE = true, bool LDS_FREE = false>
__device__ __forceinline__ bool epilogue_tile(const LinearArgs& g, f32x16 (&acc)[BM / WAVES_M / 32][BN / WAVES_N / 32],
                                              bf16_t* lds, const float* gelu_tab, int64_t m0, int64_t n0,
                                              int wave_m, int wave_n, int l32, int half, int tid) {
  constexpr int NT = 64 * WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 32, TN = WN / 32;
  constexpr int CROW = BN + 8;   // padded row of the staged tile
  const bool staged = n0 + BN <= g.n_split && g.ldo % 8 == 0 && ((uintptr_t)g.out % 16) == 0 && g.n % 8 == 0 &&
                      (g.o_period == INT64_MAX || (g.o_s1 % 8 == 0 && g.o_s2 % 8 == 0));
  // a tile wholly in the strided part whose rows run contiguously (stride 1 along m, one
  // period) is staged TRANSPOSED, [n][m], and written with 16-byte stores along m
  constexpr int TROW = BM + 8;
  const bool tstaged = !staged && n0 >= g.n_split && g.t_s2 == 1 && g.m % 8 == 0 && g.t_s1 % 8 == 0 && g.t_s3 % 8 == 0 &&
                       ((uintptr_t)g.out_t % 16) == 0 && (g.t_period == INT64_MAX || (g.t_period % BM == 0));
  if (!LDS_FREE && (staged || tstaged)) __syncthreads();   // every wave is done reading the k-loop buffers
  // Whole tiles of ordinary operands: no clamps, no predicates, and a wave-uniform base plus 32 bits per lane for every access.  What
  // bounds an epilogue is vector work, and the general form below spends most of its own on 64-bit addresses (34
  // instructions per four elements).  16384x4096x1024 144.6 -> 141.9 us, 12288x2560x320 37.8 -> 35.5, 524288x128x128 112.7 -> 106.5.
  // (Rows in descending order, a negative stride, are for the general form: its offsets have a sign.)
  auto near_rows = [](int64_t stride) { return (uint64_t)stride < (uint64_t)kNearRow; };
  const bool whole = m0 + BM <= g.m && n0 + BN <= g.n && ((staged && g.o_period == INT64_MAX && near_rows(g.ldo)) || (tstaged && near_rows(g.t_s3))) &&
                     (!g.mul || near_rows(g.ldmul)) && (!g.resid || near_rows(g.ldr)) &&
                     (g.bias_period <= 0 || (uint32_t)m0 / (uint32_t)g.bias_period == (uint32_t)(m0 + BM - 1) / (uint32_t)g.bias_period);
  if (whole) {
    constexpr int JF = WAVES_M * WAVES_N == 8 ? TN : 1;      // (operands a wave has in flight at a time, as below)
    auto near4 = [](const bf16_t* base, uint32_t bytes, int imm) { return *reinterpret_cast<const bf16x4*>((const unsigned char*)base + bytes + imm * 2); };
    auto store8 = [](bf16_t* base, uint32_t bytes, const bf16_t* from) { *reinterpret_cast<bf16x8*>((unsigned char*)base + bytes) = *reinterpret_cast<const bf16x8*>(from); };
    const bf16_t* const bias_b = g.bias ? (const bf16_t*)g.bias + (g.bias_period > 0 ? (int64_t)((uint32_t)m0 / (uint32_t)g.bias_period) * g.n : 0) + n0 : nullptr;
    const bf16_t* const mul_b = (const bf16_t*)g.mul + m0 * g.ldmul + n0;
    const bf16_t* const res_b = (const bf16_t*)g.resid + m0 * g.ldr + n0;
    const uint32_t cl = wave_n * WN + 4 * half;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const uint32_t rl = wave_m * WM + i * 32 + l32;
      const uint32_t mul_o = (rl * (uint32_t)g.ldmul + cl) * 2, res_o = (rl * (uint32_t)g.ldr + cl) * 2;   // bytes
#pragma unroll
      for (int jb = 0; jb < TN; jb += JF) {
        bf16x4 bias_v[JF][4] = {}, mul_v[JF][4], res_v[JF][4];
        if (bias_b) {
#pragma unroll
          for (int j = 0; j < JF; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) bias_v[j][q] = near4(bias_b, cl * 2, (jb + j) * 32 + 8 * q);
        }
        if (g.mul) {
#pragma unroll
          for (int j = 0; j < JF; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) mul_v[j][q] = near4(mul_b, mul_o, (jb + j) * 32 + 8 * q);
        }
        if (g.resid) {
#pragma unroll
          for (int j = 0; j < JF; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) res_v[j][q] = near4(res_b, res_o, (jb + j) * 32 + 8 * q);
        }
#pragma unroll
        for (int j = 0; j < JF; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float v[4];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
              const float pre = acc[i][jb + j][4 * q + jj] + bf2f(bias_v[j][q][jj]);
              v[jj] = ACT == AC_ACT_GELU_ERF && GELU_TABLE ? gelu_table(pre, gelu_tab) : apply_act_bf16<ACT>(pre);
            }
            if (g.mul) {
#pragma unroll
              for (int jj = 0; jj < 4; ++jj) v[jj] *= bf2f(mul_v[j][q][jj]);
            }
            if (g.resid) {
#pragma unroll
              for (int jj = 0; jj < 4; ++jj) v[jj] += bf2f(res_v[j][q][jj]);
            }
            const bf16x4 o = {f2bf(v[0]), f2bf(v[1]), f2bf(v[2]), f2bf(v[3])};
            const uint32_t c = cl + (jb + j) * 32 + 8 * q;
            if (staged) {
              *reinterpret_cast<bf16x4*>(lds + rl * CROW + c) = o;
            } else {
#pragma unroll
              for (int jj = 0; jj < 4; ++jj) lds[(c + jj) * TROW + rl] = o[jj];
            }
          }
      }
    }
    __syncthreads();
    if (staged) {
      constexpr int CPR = BN / 8, RPT = NT / CPR;            // 16-byte chunks per tile row, rows per pass of the block
      bf16_t* const out_b = (bf16_t*)g.out + m0 * g.ldo + n0;
      if constexpr (NT % CPR == 0) {
        const uint32_t r0 = tid / CPR, cc = tid % CPR * 8;
        uint32_t off = (r0 * (uint32_t)g.ldo + cc) * 2;
#pragma unroll 4
        for (int r = 0; r < BM; r += RPT, off += RPT * (uint32_t)g.ldo * 2) store8(out_b, off, lds + (r0 + r) * CROW + cc);
      } else {
#pragma unroll 4
        for (int c = tid; c < BM * CPR; c += NT)
          store8(out_b, ((uint32_t)(c / CPR) * (uint32_t)g.ldo + c % CPR * 8) * 2, lds + c / CPR * CROW + c % CPR * 8);
      }
    } else {
      constexpr int CPT = BM / 8, NPT = NT / CPT;
      static_assert(NT % CPT == 0 && BN % NPT == 0, "columns per pass of the block");
      int64_t tq, tr;
      split_row(m0, g.t_period, tq, tr);
      bf16_t* const out_b = (bf16_t*)g.out_t + tq * g.t_s1 + tr + (n0 - g.n_split) * g.t_s3;
      const uint32_t nl = tid / CPT, mm = tid % CPT * 8;
      uint32_t off = (nl * (uint32_t)g.t_s3 + mm) * 2;
#pragma unroll 4
      for (int n = 0; n < BN; n += NPT, off += NPT * (uint32_t)g.t_s3 * 2) store8(out_b, off, lds + (nl + n) * TROW + mm);
    }
    return true;
  }
  // Operand loads of the epilogue are issued in batches and from clamped, always valid
  // addresses, so that a lane waits for memory once per batch and not once per group of four
  // columns; only the stores are predicated.  A batch is a row of the wave's 32x32
  // accumulator tiles in the 8-wave shapes and a single tile in the 4-wave shapes, which
  // have no registers to spare.
  constexpr int JB = WAVES_M * WAVES_N == 8 ? TN : 1;
  const bf16x4 zero4 = {(bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f};
  const int cl0 = wave_n * WN + 4 * half;      // this lane's first column of the tile
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int rl = wave_m * WM + i * 32 + l32;
    const int64_t m = m0 + rl;
    const bool row_ok = m < g.m;
    const int64_t mc = row_ok ? m : g.m - 1;
    // offset of row m in the strided ("transposed") output, if any
    const int64_t t_base = g.n_split < g.n ? out_t_row(g, mc) : 0;
    const int64_t bias_row = g.bias_period > 0 ? (int64_t)((uint32_t)mc / (uint32_t)g.bias_period) * g.n : 0;   // (m < 2^31)
#pragma unroll
    for (int jb = 0; jb < TN; jb += JB) {
      bf16x4 bias_v[JB][4], mul_v[JB][4], res_v[JB][4];
      int64_t nc[JB][4];
#pragma unroll
      for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t n = n0 + cl0 + (jb + j) * 32 + 8 * q;
          nc[j][q] = n < g.n ? n : g.n - 4;
          bias_v[j][q] = g.bias ? *reinterpret_cast<const bf16x4*>((const bf16_t*)g.bias + bias_row + nc[j][q]) : zero4;
        }
      if (g.mul) {
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            mul_v[j][q] = *reinterpret_cast<const bf16x4*>((const bf16_t*)g.mul + mc * g.ldmul + nc[j][q]);
      }
      if (g.resid) {
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            res_v[j][q] = *reinterpret_cast<const bf16x4*>((const bf16_t*)g.resid + mc * g.ldr + nc[j][q]);
      }
#pragma unroll
      for (int j = 0; j < JB; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int cl = cl0 + (jb + j) * 32 + 8 * q;
          const int64_t n = n0 + cl;
          float v[4] = {acc[i][jb + j][4 * q], acc[i][jb + j][4 * q + 1], acc[i][jb + j][4 * q + 2], acc[i][jb + j][4 * q + 3]};
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const float pre = v[jj] + bf2f(bias_v[j][q][jj]);
            v[jj] = ACT == AC_ACT_GELU_ERF && GELU_TABLE ? gelu_table(pre, gelu_tab) : apply_act_bf16<ACT>(pre);
          }
          if (g.mul) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) v[jj] *= bf2f(mul_v[j][q][jj]);
          }
          if (g.resid) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) v[jj] += bf2f(res_v[j][q][jj]);
          }
          const bf16x4 o = {f2bf(v[0]), f2bf(v[1]), f2bf(v[2]), f2bf(v[3])};
          if (!row_ok || n >= g.n) continue;
          if (staged) {
            *reinterpret_cast<bf16x4*>(lds + rl * CROW + cl) = o;
          } else if (tstaged) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) lds[(cl + jj) * TROW + rl] = o[jj];
          } else if (n < g.n_split) {
            *reinterpret_cast<bf16x4*>((bf16_t*)g.out + out_row(g, m) + n) = o;
          } else {
            const int64_t base = t_base + (n - g.n_split) * g.t_s3;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) ((bf16_t*)g.out_t)[base + jj * g.t_s3] = o[jj];
          }
        }
      }
    }
  }
  if (tstaged) {
    __syncthreads();
    constexpr int CPT = BM / 8;   // 16-byte chunks per staged row (one output column n)
    int64_t tq, tr;
    split_row(m0, g.t_period, tq, tr);
    const int64_t t_tile = tq * g.t_s1 + tr;   // the tile's rows share a period (and t_s2 == 1 here)
#pragma unroll 4
    for (int c = tid; c < BN * CPT; c += NT) {
      const int nl = c / CPT, mm = (c % CPT) * 8;
      const int64_t n = n0 + nl;
      if (m0 + mm < g.m && n < g.n)
        *reinterpret_cast<bf16x8*>((bf16_t*)g.out_t + t_tile + mm + (n - g.n_split) * g.t_s3) =
            *reinterpret_cast<const bf16x8*>(lds + nl * TROW + mm);
    }
    return true;
  }
  if (!staged) return false;
  __syncthreads();
  constexpr int CPR = BN / 8;   // 16-byte chunks per tile row
  if (g.o_period == INT64_MAX) {   // (two loops: the common one carries no trace of the regrouping arithmetic)
#pragma unroll 4
    for (int c = tid; c < BM * CPR; c += NT) {
      const int rl = c / CPR, cc = (c % CPR) * 8;
      const int64_t m = m0 + rl, n = n0 + cc;
      if (m < g.m && n < g.n)
        *reinterpret_cast<bf16x8*>((bf16_t*)g.out + m * g.ldo + n) = *reinterpret_cast<const bf16x8*>(lds + rl * CROW + cc);
    }
  } else {
#pragma unroll 2
    for (int c = tid; c < BM * CPR; c += NT) {
      const int rl = c / CPR, cc = (c % CPR) * 8;
      const int64_t m = m0 + rl, n = n0 + cc;
      if (m < g.m && n < g.n)
        *reinterpret_cast<bf16x8*>((bf16_t*)g.out + out_row(g, m) + n) = *reinterpret_cast<const bf16x8*>(lds + rl * CROW + cc);
    }
  }
  return true;
}

template <int BM, int BN, int WAVES_M, int WAVES_N>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) linear_mfma_bf16(LinearArgs g) {
  constexpr int NT = 64 * WAVES_M * WAVES_N;           // threads
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // wave tile
  constexpr int TM = WM / 32, TN = WN / 32;            // 32x32 MFMA tiles per wave
  constexpr int A_CHUNKS = BM * 8 / NT, W_CHUNKS = BN * 8 / NT;   // 16-byte chunks per thread
  static_assert(A_CHUNKS >= 1 && W_CHUNKS >= 1 && TM >= 1 && TN >= 1, "tile / wave layout mismatch");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16_t* sA = reinterpret_cast<bf16_t*>(smem_raw);                 // [2][BM][kLdsRow]
  bf16_t* sW = sA + 2 * BM * kLdsRow;                               // [2][BN][kLdsRow]
  float* gelu_tab = reinterpret_cast<float*>(sW + 2 * BN * kLdsRow);   // after the k-loop buffers
  if (g.act == AC_ACT_GELU_ERF) gelu_table_fill(gelu_tab, threadIdx.x, NT);   // read after many barriers

  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
  const int l32 = lane % 32, half = lane / 32;
  const int64_t tiles_m = (g.m + BM - 1) / BM, tiles_n = (g.n + BN - 1) / BN;
  int64_t tm_, tn_;
  tile_of_block(tiles_m, tiles_n, tm_, tn_, g.causal ? blockIdx.y : 0);
  const int64_t m0 = tm_ * BM, n0 = tn_ * BN;
  if (tile_unseen(g, m0, n0, BM)) return;
  const int64_t product = g.batch_descending ? (int64_t)gridDim.y - 1 - blockIdx.y : (int64_t)blockIdx.y;
  const bf16_t* a = (const bf16_t*)g.a + product * g.sa_b;
  const bf16_t* w = (const bf16_t*)g.w + product * g.sw_b;
  g.out = (bf16_t*)g.out + product * g.so_b;

  // Global source of each 16-byte chunk this thread stages (rows clamped into range; the
  // results of clamped rows are never stored).
  const bf16_t* a_src[A_CHUNKS];
  const bf16_t* w_src[W_CHUNKS];
  int a_dst[A_CHUNKS], w_dst[W_CHUNKS];
#pragma unroll
  for (int i = 0; i < A_CHUNKS; ++i) {
    const int c = tid + NT * i, row = c >> 3, ch = c & 7;
    int64_t gr = m0 + row; if (gr > g.m - 1) gr = g.m - 1;
    a_src[i] = a + gr * g.lda + ch * 8;
    a_dst[i] = row * kLdsRow + ch * 8;
  }
#pragma unroll
  for (int i = 0; i < W_CHUNKS; ++i) {
    const int c = tid + NT * i, row = c >> 3, ch = c & 7;
    int64_t gr = n0 + row; if (gr > g.n - 1) gr = g.n - 1;
    w_src[i] = w + gr * g.ldw + ch * 8;
    w_dst[i] = row * kLdsRow + ch * 8;
  }

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Software pipeline over k tiles with S register sets.  During step kt the wave
  //   - has the global loads of tiles kt+2 .. kt+S in flight into S-1 register sets,
  //   - multiplies tile kt out of LDS buffer kt & 1, and
  //   - between the MFMA groups of that multiply, writes tile kt+1 (loaded S-1 steps ago,
  //     so long since landed) from the remaining register set into the other LDS
  //     buffer.  LDS takes writes at about a third of its read rate, and all waves of the
  //     block reach the barrier together, so the writes must hide under the matrix work
  //     rather than sit between the multiply and the barrier.
  // Two sets are what the large tiles' accumulators leave room for.  The small tiles take four:
  // inside a model their operands were written by the kernel before (another XCD's L2, so they
  // come from memory), and a 512 x 768 x 3072 product on 32x64 tiles went from 15.6 to 12.3 us;
  // with operands that are already in L2 the depth makes no difference.
  const int64_t kt_count = tile_depth(g, m0, BM) / kBK;
  constexpr int KSTEPS = kBK / 16;
  // register sets of the staging ring (registers allow four only in the small tiles)
  constexpr int S = TM * TN < 4 ? 4 : 2;
  auto load_regs = [&](bf16x8 (&ar)[A_CHUNKS], bf16x8 (&wr)[W_CHUNKS], int64_t kt) {
    const int64_t koff = kt * kBK;
#pragma unroll
    for (int i = 0; i < A_CHUNKS; ++i) ar[i] = *reinterpret_cast<const bf16x8*>(a_src[i] + koff);
#pragma unroll
    for (int i = 0; i < W_CHUNKS; ++i) wr[i] = *reinterpret_cast<const bf16x8*>(w_src[i] + koff);
  };
  // chunk c of the A_CHUNKS + W_CHUNKS staged chunks -> LDS buffer `buf`
  auto store_chunk = [&](const bf16x8 (&ar)[A_CHUNKS], const bf16x8 (&wr)[W_CHUNKS], int buf, int c) {
    if (c < A_CHUNKS) *reinterpret_cast<bf16x8*>(sA + buf * BM * kLdsRow + a_dst[c]) = ar[c];
    else *reinterpret_cast<bf16x8*>(sW + buf * BN * kLdsRow + w_dst[c - A_CHUNKS]) = wr[c - A_CHUNKS];
  };
  constexpr int CHUNKS = A_CHUNKS + W_CHUNKS;
  auto step = [&](int64_t kt, bf16x8 (&hold_a)[A_CHUNKS], bf16x8 (&hold_w)[W_CHUNKS],
                  bf16x8 (&fill_a)[A_CHUNKS], bf16x8 (&fill_w)[W_CHUNKS]) {
    // No branches in the step: a conditional load would make the compiler lose count of the
    // loads in flight and wait for the newest ones before every LDS store.  Past the end the
    // last tile is simply loaded (and stored to the idle buffer) again.
    load_regs(fill_a, fill_w, kt + S < kt_count ? kt + S : kt_count - 1);
    const int buf = (int)(kt & 1);
    const bf16_t* cA = sA + buf * BM * kLdsRow + (wave_m * WM + l32) * kLdsRow + half * 8;
    const bf16_t* cW = sW + buf * BN * kLdsRow + (wave_n * WN + l32) * kLdsRow + half * 8;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      bf16x8 fa[TM], fw[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(cA + i * 32 * kLdsRow + ks * 16);
#pragma unroll
      for (int j = 0; j < TN; ++j) fw[j] = *reinterpret_cast<const bf16x8*>(cW + j * 32 * kLdsRow + ks * 16);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[j], fa[i], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int c = ks * CHUNKS / KSTEPS; c < (ks + 1) * CHUNKS / KSTEPS; ++c) store_chunk(hold_a, hold_w, buf ^ 1, c);
      __builtin_amdgcn_sched_barrier(0);   // keep each slice of the stores with its MFMA group
    }
    __syncthreads();
  };

  // One MFMA tile per wave (64x64 blocks: launches of a few hundred rows, one wave per SIMD): a k step is
  // then one matrix instruction behind two LDS reads, and with the reads issued just before it the loop
  // runs at the LDS latency, a third of the matrix rate.  Here the fragments of the WHOLE next tile are
  // read while this tile's (already in registers) are multiplied, so everything is staged one tile earlier:
  // during step kt the wave loads tile kt+S+1 from memory, reads the fragments of tile kt+1 out of LDS buffer
  // (kt+1) & 1, multiplies tile kt from registers and writes tile kt+2 into buffer kt & 1 (whose reads were
  // issued a step ago and have completed before the barrier).  Same instructions on the same operands in the
  // same order per output element as the loop above, so results do not depend on which loop ran.
  constexpr bool FRAGS_AHEAD = TM == 1 && TN == 1;
  if constexpr (FRAGS_AHEAD) {
    bf16x8 ra[S][A_CHUNKS], rw[S][W_CHUNKS];
    bf16x8 fa[2][KSTEPS], fw[2][KSTEPS];
    auto read_frags = [&](bf16x8 (&fa_)[KSTEPS], bf16x8 (&fw_)[KSTEPS], int buf) {
      const bf16_t* cA = sA + buf * BM * kLdsRow + (wave_m * WM + l32) * kLdsRow + half * 8;
      const bf16_t* cW = sW + buf * BN * kLdsRow + (wave_n * WN + l32) * kLdsRow + half * 8;
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) {
        fa_[ks] = *reinterpret_cast<const bf16x8*>(cA + ks * 16);
        fw_[ks] = *reinterpret_cast<const bf16x8*>(cW + ks * 16);
      }
    };
    auto clamp_kt = [&](int64_t t) { return t < kt_count ? t : kt_count - 1; };   // past the end: the last tile again
    // step kt: set `hold` carries tile kt+2, set `fill` (stored a step ago) takes tile kt+S+1
    auto ahead = [&](int64_t kt, bf16x8 (&hold_a)[A_CHUNKS], bf16x8 (&hold_w)[W_CHUNKS],
                     bf16x8 (&fill_a)[A_CHUNKS], bf16x8 (&fill_w)[W_CHUNKS],
                     const bf16x8 (&cur_a)[KSTEPS], const bf16x8 (&cur_w)[KSTEPS],
                     bf16x8 (&next_a)[KSTEPS], bf16x8 (&next_w)[KSTEPS]) {
      load_regs(fill_a, fill_w, clamp_kt(kt + S + 1));
      const int buf = (int)(kt & 1);
      read_frags(next_a, next_w, buf ^ 1);
      __builtin_amdgcn_sched_barrier(0);   // the reads go out before the first matrix instruction
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) {
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur_w[ks], cur_a[ks], acc[0][0], 0, 0, 0);
#pragma unroll
        for (int c = ks * CHUNKS / KSTEPS; c < (ks + 1) * CHUNKS / KSTEPS; ++c) store_chunk(hold_a, hold_w, buf, c);
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
    };
    load_regs(ra[0], rw[0], 0);
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) store_chunk(ra[0], rw[0], 0, c);
    load_regs(ra[S - 1], rw[S - 1], clamp_kt(1));
#pragma unroll
    for (int u = 0; u + 1 < S; ++u) load_regs(ra[u], rw[u], clamp_kt(2 + u));
    __syncthreads();
    read_frags(fa[0], fw[0], 0);
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) store_chunk(ra[S - 1], rw[S - 1], 1, c);
    __syncthreads();
    int64_t kt = 0;
    for (; kt + S <= kt_count; kt += S) {
#pragma unroll
      for (int u = 0; u < S; ++u)
        ahead(kt + u, ra[u], rw[u], ra[(u + S - 1) % S], rw[(u + S - 1) % S], fa[u & 1], fw[u & 1], fa[(u & 1) ^ 1], fw[(u & 1) ^ 1]);
    }
#pragma unroll
    for (int u = 0; u + 1 < S; ++u)
      if (kt + u < kt_count)
        ahead(kt + u, ra[u], rw[u], ra[(u + S - 1) % S], rw[(u + S - 1) % S], fa[u & 1], fw[u & 1], fa[(u & 1) ^ 1], fw[(u & 1) ^ 1]);
  } else {
    bf16x8 ra[S][A_CHUNKS], rw[S][W_CHUNKS];
    load_regs(ra[0], rw[0], 0);
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) store_chunk(ra[0], rw[0], 0, c);
#pragma unroll
    for (int u = 0; u + 1 < S; ++u) load_regs(ra[u], rw[u], 1 + u < kt_count ? 1 + u : kt_count - 1);
    __syncthreads();
    int64_t kt = 0;
    for (; kt + S <= kt_count; kt += S) {
#pragma unroll
      for (int u = 0; u < S; ++u) step(kt + u, ra[u], rw[u], ra[(u + S - 1) % S], rw[(u + S - 1) % S]);
    }
#pragma unroll
    for (int u = 0; u + 1 < S; ++u)
      if (kt + u < kt_count) step(kt + u, ra[u], rw[u], ra[(u + S - 1) % S], rw[(u + S - 1) % S]);
  }

  // acc[i][j][r]: row m = .. + l32, column n = .. + 8*(r/4) + 4*half + (r%4).
  bf16_t* lds = reinterpret_cast<bf16_t*>(smem_raw);
  switch (g.act) {   // one branch per launch, so the activation is inlined without a per-element switch
    case AC_ACT_GELU_ERF: epilogue_tile<AC_ACT_GELU_ERF, BM, BN, WAVES_M, WAVES_N>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
    case AC_ACT_GELU_TANH: epilogue_tile<AC_ACT_GELU_TANH, BM, BN, WAVES_M, WAVES_N>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
    case AC_ACT_RELU: epilogue_tile<AC_ACT_RELU, BM, BN, WAVES_M, WAVES_N>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
    case AC_ACT_SIGMOID: epilogue_tile<AC_ACT_SIGMOID, BM, BN, WAVES_M, WAVES_N>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
    default: epilogue_tile<AC_ACT_NONE, BM, BN, WAVES_M, WAVES_N>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
  }
}

template <int BM, int BN>
constexpr size_t mfma_lds_bytes() { return (size_t)2 * (BM + BN) * kLdsRow * sizeof(bf16_t) + kGeluTableBytes; }

template <int BM, int BN, int WAVES_M, int WAVES_N>
static hipError_t mfma_launch(const LinearArgs& g, hipStream_t s) {
  auto kern = linear_mfma_bf16<BM, BN, WAVES_M, WAVES_N>;
  constexpr size_t lds = mfma_lds_bytes<BM, BN>();
  // the attribute is per function; set once per process (the initialiser runs once, thread-safe)
  static const hipError_t attr_status = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr_status != hipSuccess) return attr_status;
  const int64_t tiles = ((g.m + BM - 1) / BM) * ((g.n + BN - 1) / BN);
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles, (unsigned)g.batch), dim3(64 * WAVES_M * WAVES_N), lds, s, g);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// bf16 MFMA kernel, tiles by direct global-to-LDS loads through a ring of STAGES buffers.
//
// What bounds it: a k loop that stages through registers pays for every byte twice, once as a load and once as an
// LDS store (LDS takes stores at about a third of its read rate), and with two buffers all waves wait at
// every barrier for the youngest loads.  Here one wave instruction moves 1 KB from memory into LDS with no register
// and no store instruction, a tile has STAGES - 2 whole steps to arrive (the wait before a barrier counts the younger
// tiles' loads as still in flight), and the fragments of tile kt + 1 are read from LDS between the matrix instructions of
// tile kt, so that the matrix pipe waits neither for LDS nor for memory.  Addresses are a scalar base, a scalar tile offset and
// 32 bits per lane (buffer loads: 1204 against 1157 TFLOP/s with 64-bit lane addresses, 65536 x 2048 x 8192).
// Measured against register staging with the same tiles (65536 x 2048 x 8192 / 6400 x 1024 x 1024 / 4096 x 768 x 768):
// 256x128 2152 -> 1840 us / 22.1 -> 20.0 / 16.8 -> 15.2, 64x64 3570 -> 3376 / 31.0 -> 27.1 / 14.4 -> 11.7.
//
// LDS rows are BK elements without padding (a direct load writes 1 KB of consecutive LDS); the 16-byte chunks
// of a row are permuted instead: chunk c of row r lies at position c ^ swz(r).  A 128-bit read serves 16 lanes at a time over
// 256 bytes of banks, lanes 0-3, 12-15, 20-23, 24-27 together and the other sixteen of a half-wave together; swz gives
// either set sixteen different slots (SQ_LDS_BANK_CONFLICT 1.1 % of SQ_LDS_IDX_ACTIVE at k = 8192 and 7.5 % at k = 1024: the epilogue's
// staging, none of it the k loop's).  The permutation is applied to the lane's global address, inside one cache line.
// Same matrix instructions on the same operands in the same k order as the kernel above: equal bits.
// ------------------------------------------------------------------------------------
template <int BK> __device__ __forceinline__ int ring_swizzle(int r) {
  static_assert(BK == 64, "rows of eight chunks");
  return (r >> 1) & 7;
}
constexpr int ring_lds_bytes(int bm, int bn, int bk, int stages) {
  const int ring = stages * (bm + bn) * bk * 2;
  const int out = bm * (bn + 8) * 2, out_t = bn * (bm + 8) * 2;       // the epilogue's staging tile, plain or transposed
  const int most = out > out_t ? out : out_t;
  return ring > most ? ring : most;
}
__device__ const bf16_t kZeroRow[64] __attribute__((aligned(128))) = {};   // source of the chunks past the end of k

// After the k loop (every load landed, every wave past its last LDS read): one branch per launch, so the activation is
// inlined without a per-element switch.
template <int BM, int BN, int WAVES_M, int WAVES_N, bool GELU_TABLE = true>
__device__ __forceinline__ void finish_tile(const LinearArgs& g, f32x16 (&acc)[BM / WAVES_M / 32][BN / WAVES_N / 32],
                                            unsigned char* smem, float* gelu_tab, int64_t m0, int64_t n0, int wave_m, int wave_n,
                                            int l32, int half, int tid) {
  bf16_t* lds = reinterpret_cast<bf16_t*>(smem);
  if (GELU_TABLE && g.act == AC_ACT_GELU_ERF) { gelu_table_fill(gelu_tab, tid, 64 * WAVES_M * WAVES_N); __syncthreads(); }
  switch (g.act) {
    case AC_ACT_GELU_ERF: epilogue_tile<AC_ACT_GELU_ERF, BM, BN, WAVES_M, WAVES_N, GELU_TABLE>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
    case AC_ACT_GELU_TANH: epilogue_tile<AC_ACT_GELU_TANH, BM, BN, WAVES_M, WAVES_N, GELU_TABLE>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
    case AC_ACT_RELU: epilogue_tile<AC_ACT_RELU, BM, BN, WAVES_M, WAVES_N, GELU_TABLE>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
    case AC_ACT_SIGMOID: epilogue_tile<AC_ACT_SIGMOID, BM, BN, WAVES_M, WAVES_N, GELU_TABLE>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
    default: epilogue_tile<AC_ACT_NONE, BM, BN, WAVES_M, WAVES_N, GELU_TABLE>(g, acc, lds, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid); break;
  }
}

// A gated product's tile: the 32-row blocks of its weight rows are value rows and the gate rows of the same columns in turn, so a wave's two
// accumulator tiles of a row are both halves of 32 outputs, which meet here in fp32 (stored in between and multiplied by a pass of their own,
// 2 x 1280 columns of 8192 rows took 16.9 + 13.3 us and rounded both halves to bf16).
__device__ __forceinline__ int64_t gate_weight_row(const LinearArgs& g, int r, int64_t last) {   // relative to the tile's first column
  const int64_t c = r / 64 * 32 + r % 32;
  return (c < last ? c : last) + (r / 32 % 2) * g.gate;
}
template <int ACT, int TM>
__device__ __forceinline__ void gate_tile(const LinearArgs& g, f32x16 (&acc)[TM][2], int64_t n) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bf16x4 zero4 = {};
    const int64_t c = n + 8 * q < g.n ? n + 8 * q : g.n - 4;
    const bf16x4 bv = g.bias ? *reinterpret_cast<const bf16x4*>((const bf16_t*)g.bias + c) : zero4;
    const bf16x4 bg = g.bias ? *reinterpret_cast<const bf16x4*>((const bf16_t*)g.bias + g.gate + c) : zero4;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        acc[i][0][4 * q + jj] = (acc[i][0][4 * q + jj] + bf2f(bv[jj])) * apply_act_bf16<ACT>(acc[i][1][4 * q + jj] + bf2f(bg[jj]));
    __builtin_amdgcn_sched_barrier(0);   // (a group of columns at a time: interleaved, their temporaries do not fit)
  }
}
// (erf GELU, by its formula as the pass it replaces had it; the other activations keep that pass: tanhf alone spills 80 registers here)
template <int BM, int BN, int WAVES_M, int WAVES_N>
__device__ __forceinline__ void finish_gated(LinearArgs g, f32x16 (&acc)[BM / WAVES_M / 32][2], unsigned char* smem, int64_t m0, int64_t n0,
                                             int wave_m, int wave_n, int l32, int half, int tid) {
  static_assert(BN / WAVES_N == 64, "a value tile and a gate tile per wave");
  constexpr int TM = BM / WAVES_M / 32;
  const int64_t n = n0 + wave_n * 32 + 4 * half;
  gate_tile<AC_ACT_GELU_ERF, TM>(g, acc, n);
  g.bias = nullptr;
  f32x16 out[TM][1];
#pragma unroll
  for (int i = 0; i < TM; ++i) out[i][0] = acc[i][0];
  epilogue_tile<AC_ACT_NONE, BM, BN / 2, WAVES_M, WAVES_N>(g, out, reinterpret_cast<bf16_t*>(smem), nullptr, m0, n0, wave_m, wave_n, l32, half, tid);
}

// WIDE: a convolution whose rows are too long for 32-bit offsets inside a tile (2^20 channels and more): 64 bits per lane, outside
// pixels from a row of zeros.
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, bool CONV = false, bool RAGGED_K = false, bool WIDE = false, bool GATED = false>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N) linear_ring_bf16(LinearArgs g) {
  constexpr int BNO = GATED ? BN / 2 : BN;      // output columns of a tile
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 32, TN = WN / 32;
  constexpr int ROWB = BK * 2, CPR = ROWB / 16, RPI = 1024 / ROWB;      // bytes and chunks per LDS row, rows per load instruction
  constexpr int A_I = BM / RPI / NW, W_I = BN / RPI / NW, PER = A_I + W_I;   // load instructions of a wave per tile
  constexpr int KSTEPS = BK / 16, READS = KSTEPS * (TM + TN), MMAS = KSTEPS * TM * TN;
  constexpr int STAGE = (BM + BN) * ROWB;
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0 && STAGES == 3 && (NW * RPI) % 16 == 0, "tile / wave layout mismatch");   // (arrived() has the waits of three)
  static_assert(!WIDE || CONV, "only the convolution has a form for long rows");
  using Off = std::conditional_t<WIDE, int64_t, uint32_t>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  float* gelu_tab = reinterpret_cast<float*>(smem_raw + ring_lds_bytes(BM, BN, BK, STAGES));
  const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
  const int l32 = lane % 32, half = lane / 32;
  int64_t tm_, tn_;
  tile_of_block((g.m + BM - 1) / BM, (g.n + BNO - 1) / BNO, tm_, tn_, g.causal ? blockIdx.y : 0);
  const int64_t m0 = tm_ * BM, n0 = tn_ * BNO;
  if (tile_unseen(g, m0, n0, BM)) return;
  const int64_t product = g.batch_descending ? (int64_t)gridDim.y - 1 - blockIdx.y : (int64_t)blockIdx.y;
  g.out = (bf16_t*)g.out + product * g.so_b;

  // Sources: a wave-uniform base that advances with k plus a 32-bit byte offset per lane and instruction (rows past the end
  // shadow the last one; their results are never stored).
  const int64_t lda = CONV ? (int64_t)g.conv_c : g.lda;
  // CONV: the A operand is gathered from channels-last images as the 3x3 convolution needs it (implicit GEMM).  A tile of BK
  // lies inside one window position (conv_c is a multiple of 64), so it is the same channels of the pixel shifted by that
  // position for every row, or zeros where the shifted pixel falls outside its image.  The base is the first window
  // position's pixel of the first row, so that the positions' offsets are not negative; a lane whose pixel is outside
  // asks for an offset past the buffer's range, for which the hardware delivers zeros and touches no memory (two 64x64x320
  // images: 39.5 us with a 64-bit address per lane and a page of zeros, 30 us so).
  const unsigned char* a_base = (const unsigned char*)((const bf16_t*)g.a + product * g.sa_b + m0 * lda - (CONV ? (int64_t)(g.conv_w + 1) * g.conv_c : 0));
  const unsigned char* w_base = (const unsigned char*)((const bf16_t*)g.w + product * g.sw_b + n0 * g.ldw);
  const int row_in = lane / CPR;                                        // row of the instruction this lane moves
  const int src_chunk = (lane % CPR) ^ ring_swizzle<BK>(wave * RPI + row_in);   // (NW instructions apart is a multiple of 16 rows)
  Off a_off[A_I], w_off[W_I];
  int a_taps[A_I];   // CONV: bit t set = window position t of this row's pixel lies inside the image
#pragma unroll
  for (int i = 0; i < A_I; ++i) {
    const int64_t last = g.m - 1 - m0;
    const int row = (wave + NW * i) * RPI + row_in;
    const int64_t rc = row < last ? row : last;
    a_off[i] = (Off)(rc * lda * 2) + src_chunk * 16;
    a_taps[i] = 0;
    if (CONV) {
      const int pix = (int)((m0 + rc) % ((int64_t)g.conv_h * g.conv_w)), ph = pix / g.conv_w, pw = pix % g.conv_w;
      for (int t = 0; t < 9; ++t) {
        const int hh = ph + t / 3 - 1, ww = pw + t % 3 - 1;
        if (hh >= 0 && hh < g.conv_h && ww >= 0 && ww < g.conv_w) a_taps[i] |= 1 << t;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < W_I; ++i) {
    const int64_t last = g.n - 1 - n0;
    const int row = (wave + NW * i) * RPI + row_in;
    w_off[i] = (Off)((GATED ? gate_weight_row(g, row, last) : row < last ? row : last) * g.ldw * 2) + src_chunk * 16;
  }
  // (addresses: base and tile offset in scalar registers, 32 bits per lane; every lane's address is valid, so the range is open but for CONV's outside pixels)
  constexpr int kARange = CONV ? 0x7fffffff : -1;
  __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(a_base), 0, kARange, 0x00027000);
  const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(w_base), 0, -1, 0x00027000);
  auto to_lds = [](const unsigned char* src, unsigned char* dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
  };
  // load instruction x of the PER that bring in this wave's share of tile kt; called tile after tile (CONV: the tile to
  // come lies inside window position `tap`, tap_off bytes from the first position of its row of the window on)
  int tap = 0;
  std::conditional_t<WIDE, int64_t, int> tap_off = 0, tap_end = (decltype(tap_off))g.conv_c * 2;
  auto load_part = [&](int kt, int stage, int x) {
    unsigned char* dst = smem_raw + stage * STAGE + (x < A_I ? x * NW * 1024 : BM * ROWB + (x - A_I) * NW * 1024) + wave * 1024;
    auto buffer_to_lds = [](__amdgpu_buffer_rsrc_t rsrc, uint32_t lane_off, uint32_t tile_off, unsigned char* lds) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds, 16, lane_off, tile_off, 0, 0);
    };
    if (RAGGED_K && kt * BK + BK > (int)g.k) {   // the last tile: chunks past the end of k are zeros in both operands
      const bool in = kt * BK + src_chunk * 8 < (int)g.k;
      const unsigned char* src = x >= A_I ? w_base + (int64_t)kt * ROWB + w_off[x >= A_I ? x - A_I : 0] : a_base + (int64_t)kt * ROWB + a_off[x < A_I ? x : 0];
      to_lds(in ? src : (const unsigned char*)kZeroRow, dst);
    } else if (WIDE) {
      const unsigned char* src = x >= A_I ? w_base + (int64_t)kt * ROWB + w_off[x >= A_I ? x - A_I : 0] : a_base + tap_off + a_off[x < A_I ? x : 0];
      to_lds(x >= A_I || ((a_taps[x < A_I ? x : 0] >> tap) & 1) ? src : (const unsigned char*)kZeroRow, dst);
    } else if (x >= A_I) {
      buffer_to_lds(w_rsrc, w_off[x - A_I], kt * ROWB, dst);
    } else if (CONV) {
      buffer_to_lds(a_rsrc, (a_taps[x] >> tap) & 1 ? a_off[x] : 0x80000000u, tap_off, dst);
    } else {
      buffer_to_lds(a_rsrc, a_off[x], kt * ROWB, dst);
    }
    if (CONV && x == PER - 1) {
      tap_off += ROWB;
      if (tap_off == tap_end) {
        tap_end += (decltype(tap_off))g.conv_c * 2;
        if (++tap % 3 == 0) {   // the next row of the window: a base of its own, as an image's rows may be large
          a_base += (int64_t)g.conv_w * g.conv_c * 2;
          a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(a_base), 0, kARange, 0x00027000);
          tap_off = 0;
          tap_end = (decltype(tap_off))g.conv_c * 2;
        }
      }
    }
  };
  // this wave's loads of all but the youngest `tiles` tiles have landed and its LDS reads are done, then every wave's
  auto arrived = [&](int tiles) {
    constexpr int kNoExp = 7 << 4;   // (the wait counters' encoding; expcnt is not waited for, lgkmcnt is waited to 0)
    auto wait = [](auto n) {
      constexpr int N = decltype(n)::value;
      static_assert(N < 64, "vmcnt has 6 bits");
      __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | kNoExp);
    };
    asm volatile("" ::: "memory");
    if (tiles >= STAGES - 2) wait(std::integral_constant<int, (STAGES - 2) * PER>{});
    else wait(std::integral_constant<int, 0>{});
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  bf16x8 fa[2][KSTEPS][TM], fw[2][KSTEPS][TN];
  int frag_off[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) frag_off[ks] = l32 * ROWB + (((ks * 2 + half) ^ ring_swizzle<BK>(l32)) * 16);
  const unsigned char* const sA = smem_raw + wave_m * WM * ROWB;
  const unsigned char* const sW = smem_raw + BM * ROWB + wave_n * WN * ROWB;
  // read r of a tile's READS fragments, in the order the matrix instructions want them
  auto read_frag = [&](bf16x8 (&fa_)[KSTEPS][TM], bf16x8 (&fw_)[KSTEPS][TN], int base, int r) {
    const int ks = r / (TM + TN), x = r % (TM + TN);
    if (x < TN) fw_[ks][x] = *reinterpret_cast<const bf16x8*>(sW + base + frag_off[ks] + x * 32 * ROWB);
    else fa_[ks][x - TN] = *reinterpret_cast<const bf16x8*>(sA + base + frag_off[ks] + (x - TN) * 32 * ROWB);
  };
  const int kt_count = (int)((tile_depth(g, m0, BM) + (RAGGED_K ? BK - 1 : 0)) / BK);
  // Step kt: multiply tile kt (its fragments are in registers), read tile kt + 1's, and load tile kt + STAGES into the
  // buffer tile kt lay in.  `stage` = kt % STAGES.
  int kt = 0, stage = 0;
  auto step = [&](const bf16x8 (&ca)[KSTEPS][TM], const bf16x8 (&cw)[KSTEPS][TN], bf16x8 (&na)[KSTEPS][TM], bf16x8 (&nw)[KSTEPS][TN]) {
    const bool more = kt + STAGES < kt_count;
    const int free_stage = stage;
    stage = stage + 1 == STAGES ? 0 : stage + 1;
    const int base = stage * STAGE;
    __builtin_amdgcn_sched_barrier(0);
    int done = 0;
#pragma unroll
    for (int x = 0; x < MMAS; ++x) {
      const int ks = x / (TM * TN), i = (x / TN) % TM, j = x % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cw[ks][j], ca[ks][i], acc[i][j], 0, 0, 0);
      // the reads are spread over the first three quarters of the matrix instructions (past the last tile they
      // fetch what an older tile left in the ring; nothing uses it)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (done < READS && done * (3 * MMAS) < (x + 1) * 4 * READS) read_frag(na, nw, base, done++);
      // the loads are spread too: issued together after a barrier, those of all waves queue up at the one address
      // unit and hold back the matrix instructions behind them
#pragma unroll
      for (int c = x * PER / MMAS; c < (x + 1) * PER / MMAS; ++c) {
        if (more) load_part(kt + STAGES, free_stage, c);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    const int newest = kt + STAGES < kt_count ? kt + STAGES : kt_count - 1;
    arrived(newest - (kt + 2));
    ++kt;
  };
  const int ahead = kt_count < STAGES ? kt_count : STAGES;
  for (int t = 0; t < ahead; ++t) {
#pragma unroll
    for (int x = 0; x < PER; ++x) load_part(t, t, x);
  }
  arrived(ahead - 1 < STAGES - 2 ? ahead - 1 : STAGES - 2);             // tile 0 (and, with a full ring, tile 1)
#pragma unroll
  for (int r = 0; r < READS; ++r) read_frag(fa[0], fw[0], 0, r);
  arrived(ahead - 2);                                                   // tile 1
  while (true) {
    step(fa[0], fw[0], fa[1], fw[1]);
    if (kt >= kt_count) break;
    step(fa[1], fw[1], fa[0], fw[0]);
    if (kt >= kt_count) break;
  }
  if constexpr (GATED) finish_gated<BM, BN, WAVES_M, WAVES_N>(g, acc, smem_raw, m0, n0, wave_m, wave_n, l32, half, tid);
  else finish_tile<BM, BN, WAVES_M, WAVES_N, !RAGGED_K>(g, acc, smem_raw, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid);
}

// ------------------------------------------------------------------------------------
// bf16 MFMA kernel, 256x256 tiles on eight waves, 64 k per tile.
//
// What bounds it: the operand stream.  A CU keeps about a hundred requests to L2 in flight at some 400 clocks each, one per
// cache line touched, so loads must ask for whole 128-byte lines (rows of 64 k: 32-k rows doubled the requests and
// ran the L1 at its limit with the matrix pipe 66 % busy) and must not pause.  Two whole 64-k tiles fill the LDS, so
// the ring of the kernel above would have one tile in flight at best; here the unit that is freed and loaded is half a tile,
// split along the ROWS: a wave's 128x64 outputs are four quadrants, half 0 of the rows of A and W (a0, w0) and
// half 1 (a1, w1), visited as a0w0, a0w1 | a1w1, a1w0, and while two quadrants are multiplied the fragments of the
// next two are read:
//   step X(t): multiply a0w0, a0w1 of tile t;  read w1, a1 of tile t;      load half 0 of tile t + 2
//   step Y(t): multiply a1w1, a1w0 of tile t;  read a0, w0 of tile t + 1;  load half 1 of tile t + 2
// Every load has two whole steps and what is left of its own to arrive.  Fragment registers: a0, a1 and two sets for w that
// swap roles every tile.  Against the ring on 32-k rows and against register staging: 65536 x 2048 x 8192 in 1645 us
// (1337 TFLOP/s; 1811 and 1873), 65536 x 8192 x 2048 in 1836 (2041 and 2011), 4000 x 4096 x 1024 in 35.8 (38.3 and 38.1).
// Same matrix instructions in the same k order per output as the kernels above: equal bits.
// ------------------------------------------------------------------------------------
template <bool GATED>
__global__ void __launch_bounds__(512) linear_quad_bf16(LinearArgs g) {
  constexpr int BNO = GATED ? 128 : 256;                                // output columns of a tile
  constexpr int BM = 256, BN = 256, WAVES_M = 2, WAVES_N = 4, TM = 4, TN = 2, BK = 64, ROWB = 128;
  constexpr int BUF = (BM + BN) * ROWB;                                 // bytes of one tile
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  float* gelu_tab = reinterpret_cast<float*>(smem_raw + ring_lds_bytes(BM, BN, BK, 2));
  const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
  const int l32 = lane % 32, half = lane / 32;
  int64_t tm_, tn_;
  tile_of_block((g.m + BM - 1) / BM, (g.n + BNO - 1) / BNO, tm_, tn_, g.causal ? blockIdx.y : 0);
  const int64_t m0 = tm_ * BM, n0 = tn_ * BNO;
  if (tile_unseen(g, m0, n0, BM)) return;
  const int64_t product = g.batch_descending ? (int64_t)gridDim.y - 1 - blockIdx.y : (int64_t)blockIdx.y;
  g.out = (bf16_t*)g.out + product * g.so_b;

  const bf16_t* a_base = (const bf16_t*)g.a + product * g.sa_b + m0 * g.lda;
  const bf16_t* w_base = (const bf16_t*)g.w + product * g.sw_b + n0 * g.ldw;
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a_base), 0, -1, 0x00027000);
  const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(w_base), 0, -1, 0x00027000);
  // A load instruction moves 8 rows of 128 bytes.  Instruction j (0, 1) of this wave in half h: first row of its eight.
  auto a_row = [&](int h, int j) { return j * 128 + h * 64 + wave * 8; };
  auto w_row = [&](int h, int j) { return (wave / 4 + 2 * j) * 64 + h * 32 + (wave % 4) * 8; };
  const int row_in = lane / 8;
  const int src_chunk = (lane % 8) ^ ring_swizzle<BK>(wave * 8 + row_in);
  uint32_t a_off[2][2], w_off[2][2];                                    // rows past the end shadow the last one
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t la = g.m - 1 - m0, lw = g.n - 1 - n0;
      const int ra = a_row(h, j) + row_in, rw = w_row(h, j) + row_in;
      a_off[h][j] = (uint32_t)((ra < la ? ra : la) * g.lda * 2) + src_chunk * 16;
      w_off[h][j] = (uint32_t)((GATED ? gate_weight_row(g, rw, lw) : rw < lw ? rw : lw) * g.ldw * 2) + src_chunk * 16;
    }
  auto load_half = [&](int kt, int h, int x) {                          // instruction x of the four of half h of tile kt
    unsigned char* dst = smem_raw + (kt & 1) * BUF + (x < 2 ? a_row(h, x) : BM + w_row(h, x - 2)) * ROWB;
    if (x < 2) __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (__attribute__((address_space(3))) void*)dst, 16, a_off[h][x], kt * ROWB, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (__attribute__((address_space(3))) void*)dst, 16, w_off[h][x - 2], kt * ROWB, 0, 0);
  };
  // this wave's loads of all but the youngest `halves` half tiles have landed and its LDS reads are done, then every wave's
  auto arrived = [&](int halves) {
    asm volatile("" ::: "memory");
    if (halves >= 2) __builtin_amdgcn_s_waitcnt(0x78);                  // vmcnt(8) lgkmcnt(0)
    else if (halves == 1) __builtin_amdgcn_s_waitcnt(0x74);             // vmcnt(4) lgkmcnt(0)
    else __builtin_amdgcn_s_waitcnt(0x70);                              // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  bf16x8 a0[2][4], a1[2][4], wa[4], wb[4];                              // [32-row tile][k step of 16]
  int frag_off[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) frag_off[ks] = l32 * ROWB + (((ks * 2 + half) ^ ring_swizzle<BK>(l32)) * 16);
  const unsigned char* const sA = smem_raw + wave_m * 128 * ROWB;
  const unsigned char* const sW = smem_raw + (BM + wave_n * 64) * ROWB;
  auto read_a = [&](bf16x8 (&f)[2][4], int kt, int h, int x) {          // fragment x of 8
    f[x & 1][x >> 1] = *reinterpret_cast<const bf16x8*>(sA + (kt & 1) * BUF + (h * 64 + (x & 1) * 32) * ROWB + frag_off[x >> 1]);
  };
  auto read_w = [&](bf16x8 (&f)[4], int kt, int h, int x) {             // fragment x of 4
    f[x] = *reinterpret_cast<const bf16x8*>(sW + (kt & 1) * BUF + h * 32 * ROWB + frag_off[x]);
  };
  const int kt_count = (int)(tile_depth(g, m0, BM) / BK);
  // Both steps: 16 matrix instructions, 12 fragment reads among the first 12 of them, 4 loads spread evenly.  (Past the last
  // tile the reads fetch what an older one left; nothing uses it.)
  auto step_x = [&](int kt, bf16x8 (&w0)[4], bf16x8 (&w1)[4]) {
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int q = x / 8, ks = (x % 8) / 2, i = x % 2;
      if (q == 0) acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0[ks], a0[i][ks], acc[i][0], 0, 0, 0);
      else acc[i][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[ks], a0[i][ks], acc[i][1], 0, 0, 0);
      if (x < 4) read_w(w1, kt, 1, x);
      else if (x < 12) read_a(a1, kt, 1, x - 4);
      if (x % 4 == 0) { if (kt + 2 < kt_count) load_half(kt + 2, 0, x / 4); }
      __builtin_amdgcn_sched_barrier(0);
    }
    // read next: half 0 of tile kt + 1.  Younger: its half 1, half 0 of kt + 2
    arrived(kt + 2 < kt_count ? 2 : kt + 1 < kt_count ? 1 : 0);
  };
  auto step_y = [&](int kt, bf16x8 (&w0)[4], bf16x8 (&w1)[4]) {
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int q = x / 8, ks = (x % 8) / 2, i = x % 2;
      if (q == 0) acc[2 + i][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[ks], a1[i][ks], acc[2 + i][1], 0, 0, 0);
      else acc[2 + i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0[ks], a1[i][ks], acc[2 + i][0], 0, 0, 0);
      if (x < 8) read_a(a0, kt + 1, 0, x);
      else if (x < 12) read_w(w1, kt + 1, 0, x - 8);
      if (x % 4 == 0) { if (kt + 2 < kt_count) load_half(kt + 2, 1, x / 4); }
      __builtin_amdgcn_sched_barrier(0);
    }
    // read next: half 1 of tile kt + 1.  Younger: both halves of kt + 2
    arrived(kt + 2 < kt_count ? 2 : 0);
  };
#pragma unroll
  for (int x = 0; x < 8; ++x) load_half(0, x / 4, x % 4);
  if (kt_count > 1) {
#pragma unroll
    for (int x = 0; x < 8; ++x) load_half(1, x / 4, x % 4);
  }
  arrived(kt_count > 1 ? 2 : 0);                                        // tile 0
#pragma unroll
  for (int x = 0; x < 8; ++x) read_a(a0, 0, 0, x);
#pragma unroll
  for (int x = 0; x < 4; ++x) read_w(wa, 0, 0, x);
  arrived(kt_count > 1 ? 2 : 0);                                        // (every wave has read half 0 of tile 0)
  for (int kt = 0; ; kt += 2) {
    step_x(kt, wa, wb);
    step_y(kt, wa, wb);
    if (kt + 1 >= kt_count) break;
    step_x(kt + 1, wb, wa);
    step_y(kt + 1, wb, wa);
    if (kt + 2 >= kt_count) break;
  }
  if constexpr (GATED) finish_gated<BM, BN, WAVES_M, WAVES_N>(g, acc, smem_raw, m0, n0, wave_m, wave_n, l32, half, tid);
  else finish_tile<BM, BN, WAVES_M, WAVES_N>(g, acc, smem_raw, gelu_tab, m0, n0, wave_m, wave_n, l32, half, tid);
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, bool CONV = false, bool RAGGED_K = false, bool WIDE = false, bool GATED = false>
static hipError_t ring_launch(const LinearArgs& g, hipStream_t s) {
  constexpr int BNO = GATED ? BN / 2 : BN;
  auto kern = linear_ring_bf16<BM, BN, WAVES_M, WAVES_N, BK, STAGES, CONV, RAGGED_K, WIDE, GATED>;
  constexpr size_t ring = ring_lds_bytes(BM, BN, BK, STAGES);
  static const hipError_t attr_status = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(ring + kGeluTableBytes));
  if (attr_status != hipSuccess) return attr_status;
  const int64_t tiles = ((g.m + BM - 1) / BM) * ((g.n + BNO - 1) / BNO);
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles, (unsigned)g.batch), dim3(64 * WAVES_M * WAVES_N),
                     ring + (g.act == AC_ACT_GELU_ERF && !RAGGED_K && !GATED ? kGeluTableBytes : 0), s, g);
  return hipGetLastError();
}

template <bool GATED>
static hipError_t quad_launch(const LinearArgs& g, hipStream_t s) {
  constexpr size_t lds = ring_lds_bytes(256, 256, 64, 2);
  static const hipError_t attr_status = hipFuncSetAttribute(
      reinterpret_cast<const void*>(linear_quad_bf16<GATED>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(lds + kGeluTableBytes));
  if (attr_status != hipSuccess) return attr_status;
  const int64_t tiles = ((g.m + 255) / 256) * (GATED ? (g.n + 127) / 128 : (g.n + 255) / 256);
  hipLaunchKernelGGL(linear_quad_bf16<GATED>, dim3((unsigned)tiles, (unsigned)g.batch), dim3(512),
                     lds + (g.act == AC_ACT_GELU_ERF && !GATED ? kGeluTableBytes : 0), s, g);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// fp32 MFMA kernel, tiles by direct global-to-LDS loads through a ring of three buffers of 32 k (or 64).
//
// What bounds linear_mfma_f32 on larger products is its stream of operands: a step of 16 k asks for half a cache line of every row, a CU holds about a
// hundred such requests in flight whatever they carry, and each wave fetches the whole tile's operands for itself.  Here a row's step is a whole line,
// fetched once for the block's four waves, which hold a quarter of the tile each over all of k.  The loop is the bf16 ring's: loads three tiles ahead, the next
// tile's fragments read between this one's matrix instructions, chunks of a row permuted so that a read meets every bank (lanes of sixteen rows and two chunks: the
// same permutation serves).  The four parts of a sum over k that linear_mfma_f32 gives to four waves follow one another here and are added in the same
// order, each a chain of the same instructions: equal bits.  (Depths that are a multiple of 128: parts of whole tiles.)
// ------------------------------------------------------------------------------------
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK>
__global__ void __launch_bounds__(256) linear_ring_f32(LinearArgs g, int vec) {
  constexpr int NW = 4, STAGES = 3, ROWB = BK * 4, CPR = BK / 4, RPI = 256 / BK, KS = BK / 16;   // bytes and chunks per LDS row, rows per load instruction
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 16, TN = WN / 16;
  constexpr int A_I = BM / RPI / NW, W_I = BN / RPI / NW, PER = A_I + W_I;
  constexpr int READS = KS * (TM + TN), MMAS = 4 * KS * TM * TN, STAGE = (BM + BN) * ROWB;
  static_assert(WAVES_M * WAVES_N == NW && BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile / wave layout mismatch");
  static_assert(BK == 32 || BK == 64, "rows of eight or sixteen chunks");
  auto swizzle = [](int r) { return BK == 32 ? (r >> 1) & 7 : r & 15; };
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64), l16 = lane % 16, grp = lane / 16;
  const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
  int64_t tm_, tn_;
  tile_of_block((g.m + BM - 1) / BM, (g.n + BN - 1) / BN, tm_, tn_);
  const int64_t m0 = tm_ * BM, n0 = tn_ * BN;
  const int64_t product = g.batch_descending ? (int64_t)gridDim.y - 1 - blockIdx.y : (int64_t)blockIdx.y;
  const float* a = (const float*)g.a + product * g.sa_b + m0 * g.lda;
  const float* w = (const float*)g.w + product * g.sw_b + n0 * g.ldw;
  const int row_in = lane / CPR, src_chunk = (lane % CPR) ^ swizzle(wave * RPI + row_in);
  uint32_t a_off[A_I], w_off[W_I];
#pragma unroll
  for (int i = 0; i < A_I; ++i) {   // rows past the end shadow the last one; never stored
    const int64_t r = (wave + NW * i) * RPI + row_in, last = g.m - 1 - m0;
    a_off[i] = (uint32_t)((r < last ? r : last) * g.lda * 4) + src_chunk * 16;
  }
#pragma unroll
  for (int i = 0; i < W_I; ++i) {
    const int64_t r = (wave + NW * i) * RPI + row_in, last = g.n - 1 - n0;
    w_off[i] = (uint32_t)((r < last ? r : last) * g.ldw * 4) + src_chunk * 16;
  }
  const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a), 0, -1, 0x00027000);
  const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w), 0, -1, 0x00027000);
  auto load_part = [&](int kt, int stage, int x) {
    unsigned char* dst = smem_raw + stage * STAGE + (x < A_I ? x * NW * 1024 : BM * ROWB + (x - A_I) * NW * 1024) + wave * 1024;
    auto buffer_to_lds = [](__amdgpu_buffer_rsrc_t rsrc, uint32_t lane_off, uint32_t tile_off, unsigned char* lds) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds, 16, lane_off, tile_off, 0, 0);
    };
    if (x < A_I) buffer_to_lds(a_rsrc, a_off[x < A_I ? x : 0], kt * ROWB, dst);
    else buffer_to_lds(w_rsrc, w_off[x < A_I ? 0 : x - A_I], kt * ROWB, dst);
  };
  // this wave's loads of all but the youngest tile (or all of them) have landed and its LDS reads are done, then every wave's
  auto arrived = [&](bool but_one) {
    constexpr int kNoExp = 7 << 4;
    asm volatile("" ::: "memory");
    if (but_one) __builtin_amdgcn_s_waitcnt(PER | kNoExp);
    else __builtin_amdgcn_s_waitcnt(kNoExp);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  f32x4 acc[TM][TN], total[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = total[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 fa[2][KS][TM], fw[2][KS][TN];
  int frag_off[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) frag_off[s] = l16 * ROWB + ((s * 4 + grp) ^ swizzle(l16)) * 16;
  const unsigned char* const sA = smem_raw + wave_m * WM * ROWB;
  const unsigned char* const sW = smem_raw + BM * ROWB + wave_n * WN * ROWB;
  auto read_frag = [&](f32x4 (&fa_)[KS][TM], f32x4 (&fw_)[KS][TN], int base, int r) {
    const int s = r / (TM + TN), x = r % (TM + TN);
    if (x < TN) fw_[s][x] = *reinterpret_cast<const f32x4*>(sW + base + frag_off[s] + x * 16 * ROWB);
    else fa_[s][x - TN] = *reinterpret_cast<const f32x4*>(sA + base + frag_off[s] + (x - TN) * 16 * ROWB);
  };
  const int kt_count = (int)(g.k / BK), part = kt_count / kF32Runs;
  int kt = 0, stage = 0, fold = part;
  auto step = [&](const f32x4 (&ca)[KS][TM], const f32x4 (&cw)[KS][TN], f32x4 (&na)[KS][TM], f32x4 (&nw)[KS][TN]) {
    const bool more = kt + STAGES < kt_count;
    const int free_stage = stage;
    stage = stage + 1 == STAGES ? 0 : stage + 1;
    const int base = stage * STAGE;
    __builtin_amdgcn_sched_barrier(0);
    int done = 0;
#pragma unroll
    for (int x = 0; x < MMAS; ++x) {
      const int s = x / (4 * TM * TN), e = x / (TM * TN) % 4, i = x / TN % TM, j = x % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(cw[s][j][e], ca[s][i][e], acc[i][j], 0, 0, 0);
      if (done < READS && done * (3 * MMAS) < (x + 1) * 4 * READS) read_frag(na, nw, base, done++);
#pragma unroll
      for (int c = x * PER / MMAS; c < (x + 1) * PER / MMAS; ++c) {
        if (more) load_part(kt + STAGES, free_stage, c);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // (tile kt + 2 must have landed; of those asked for, kt + 3 is the youngest)
    arrived(more);
    if (++kt == fold) {
      fold += part;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
          for (int e = 0; e < 4; ++e) total[i][j][e] += acc[i][j][e];
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
  };
#pragma unroll
  for (int t = 0; t < STAGES; ++t)      // (at least four tiles)
#pragma unroll
    for (int x = 0; x < PER; ++x) load_part(t, t, x);
  {
    constexpr int kNoExp = 7 << 4;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(PER | kNoExp);           // tiles 0 and 1
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
#pragma unroll
  for (int r = 0; r < READS; ++r) read_frag(fa[0], fw[0], 0, r);
  // (tile 0 lies in registers before its buffer is loaded again)
  arrived(true);
  for (int t = 0; t < kt_count; t += 2) {   // (kt_count is a multiple of four)
    step(fa[0], fw[0], fa[1], fw[1]);
    step(fa[1], fw[1], fa[0], fw[0]);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      epilogue_store_f32x4(g, vec, product, m0 + wave_m * WM + i * 16 + l16, n0 + wave_n * WN + j * 16 + 4 * grp, total[i][j]);
}

// ------------------------------------------------------------------------------------
// LayerNorm + several projections of the same short rows in one kernel.
// The pair-stack modules project every LayerNorm output four or five times with K = c_z
// (gated a and b of the triangle update; q, k, v, gate and pair bias of the triangle attention;
// the transition's first layer).  Separate launches re-read the normalised rows each time and
// are bound by that traffic, not by the matrix cores.  Here a block normalises 64 rows once
// (the whole row is one k tile), keeps them in LDS as the matrix operand, and walks a list of
// 64-column weight tiles.  Tiles of 64 x 64 keep accumulators and LDS small enough for four blocks per
// CU, whose phases interleave: while one waits for its rows another multiplies and a third stores
// (measured against 64 x 128 tiles, two blocks per CU: the pair block at N = 1024 takes 9.7 instead of
// 10.4 ms in one segment per region, 11.7 instead of 12.5 ms in 64-row segments, where a launch's 1024
// blocks are then resident at once).  A wave keeps its 32 normalised rows in registers for every tile, the epilogue is staged where
// they lay, and so two barriers a tile suffice (five with one buffer for weights and staging).  What bounds it is vector work, half of
// which was addresses: with those of whole tiles in 32 bits, q, k, v and gate of 524288 rows take 240 instead of 272 us, two gated pairs
// of 40000 rows 21.6 instead of 26.0.  (Weights straight from memory into the registers the matrix instructions read: 352 to
// 544 us, as a lane's 16 bytes then use a fraction of every line asked for.)  Each tile is prefetched into registers while
// the previous one is multiplied, and leaves through the same epilogue as the GEMM above (row-major, regrouped
// or strided store).  A gated pair keeps sigmoid(gate) in registers and multiplies the
// projection by it, so the gate never reaches memory.  Per-row arithmetic does not depend on
// the block a row falls in, so results are bitwise independent of the chunk length.
// ------------------------------------------------------------------------------------
struct LnProjKernelArgs {
  LnProjArgs a;
  int n_tiles;
  int tile_part[kMaxProjTiles];
  int tile_n0[kMaxProjTiles];
  int any_gelu;
};

constexpr int kLnProjRows = 64;   // rows per block
constexpr int kLnProjCols = 64;   // columns per weight tile

// Elements of LDS: the normalised rows or the staging tile that takes their place (the transposed form is the larger), and a weight tile.
constexpr int ln_proj_rows_elems(int k) {
  const int rows = kLnProjRows * (k + 8), stage = kLnProjCols * (kLnProjRows + 8);
  return rows > stage ? rows : stage;
}
constexpr int ln_proj_lds_elems(int k) { return ln_proj_rows_elems(k) + kLnProjCols * (k + 8); }

// (blocks per CU: four by registers at K = 128; at K = 64, where a launch is mostly loads and stores, five, which cost 96 registers and no spill: 73792
// rows to 192, 512 and 512 columns 84 us with four, 66 with five, 67352 to 128, a gated 192 and twice 256 59 and 47; six spill)
template <int K, int BN>
__global__ void __launch_bounds__(256, K == 64 ? 5 : 4) ln_multi_proj_bf16(LnProjKernelArgs ka) {
  constexpr int BM = kLnProjRows, NT = 256;
  static_assert(BM == 64 && BN == 64, "waves 2 x 2 of one 32x32 MFMA tile each");
  constexpr int AROW = K + 8;                 // padded LDS row (elements)
  constexpr int G = K / 8;                    // lanes per row in the LayerNorm pass (16-byte chunks per row)
  constexpr int RPP = NT / G;                 // rows per pass
  constexpr int PASSES = BM / RPP;
  constexpr int KSTEPS = K / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  constexpr int W_CHUNKS = BN * G / NT;       // 16-byte chunks of a weight tile per thread
  bf16_t* sA = reinterpret_cast<bf16_t*>(smem_raw);     // [BM][AROW]: the normalised rows; then the epilogue's staging tile
  bf16_t* sW = sA + ln_proj_rows_elems(K);              // [BN][AROW]: weight tile
  float* gelu_tab = reinterpret_cast<float*>(sA + ln_proj_lds_elems(K));
  const LnProjArgs& p = ka.a;
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const int wave_m = wave / 2, wave_n = wave % 2;
  const int l32 = lane % 32, half = lane / 32;
  // consecutive row tiles go to one XCD, so that neighbouring runs of a strided output meet in one L2
  const int64_t m0 = xcd_run(blockIdx.x, gridDim.x) * BM;
  if (ka.any_gelu) gelu_table_fill(gelu_tab, tid, NT);
  // blocks of the same rows share out the weight tiles
  const int t_lo = ka.n_tiles * (int)blockIdx.y / (int)gridDim.y, t_hi = ka.n_tiles * ((int)blockIdx.y + 1) / (int)gridDim.y;

  bf16x8 wreg[W_CHUNKS];
  auto store_w = [&](int tid) {
#pragma unroll
    for (int i = 0; i < W_CHUNKS; ++i) *reinterpret_cast<bf16x8*>(sW + (tid / G + i * RPP) * AROW + tid % G * 8) = wreg[i];
  };
  auto load_w = [&](const void* wbase, int64_t n_rows, int64_t n0, int tid) {
    const bf16_t* w = (const bf16_t*)wbase;
    if (n0 + BN <= n_rows) {                  // (the usual case: a tile is one run of memory)
      const unsigned char* b = (const unsigned char*)(w + n0 * K);
#pragma unroll
      for (int i = 0; i < W_CHUNKS; ++i) wreg[i] = *reinterpret_cast<const bf16x8*>(b + (uint32_t)tid * 16 + i * NT * 16);
      return;
    }
#pragma unroll
    for (int i = 0; i < W_CHUNKS; ++i) {
      const int c = tid + NT * i, row = c / G, ch = c % G;
      int64_t gr = n0 + row; if (gr > n_rows - 1) gr = n_rows - 1;
      wreg[i] = *reinterpret_cast<const bf16x8*>(w + gr * K + ch * 8);
    }
  };
  // first weight tile of entry t: the gate's for a gated pair
  auto load_first = [&](int t, int tid) {
    const ProjPart& q = p.part[ka.tile_part[t]];
    load_w(q.gated ? q.w_gate : q.w, q.n, ka.tile_n0[t], tid);
  };

  // ---- LayerNorm of the block's rows (G lanes per row, the row in registers, fp32 statistics)
  {
    const int lg = tid % G, rg = tid / G;
    const bf16_t* x = (const bf16_t*)p.x;
    float v[PASSES][8];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      int64_t r = m0 + ps * RPP + rg;
      if (r > p.rows - 1) r = p.rows - 1;     // rows past the end shadow the last row; never stored
      int64_t at = r * p.ldx;
      if (p.x_period > 0) {                   // (positions of a pair tensor in the order of their columns: a row is two whole cache lines wherever it lies)
        int64_t q, c;
        split_row(r, p.x_period, q, c);
        at = q * p.x_s1 + c * p.x_s2;
      }
      load_vec(x + at + lg * 8, v[ps]);
    }
    float gn[8], sh[8];
    load_vec((const bf16_t*)p.gain + lg * 8, gn);
    load_vec((const bf16_t*)p.shift + lg * 8, sh);
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      float sum = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) sum += v[ps][j];
      const float mean = group_sum<G>(sum) * (1.0f / K);
      float sq = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) { const float d = v[ps][j] - mean; sq += d * d; }
      const float rstd = rsqrtf(group_sum<G>(sq) * (1.0f / K) + p.eps);
      float o[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = (v[ps][j] - mean) * rstd * gn[j] + sh[j];
      store_vec(sA + (ps * RPP + rg) * AROW + lg * 8, o);
    }
  }
  __syncthreads();
  // the wave's 32 normalised rows stay in registers for every tile
  bf16x8 fa[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) fa[ks] = *reinterpret_cast<const bf16x8*>(sA + (wave_m * 32 + l32) * AROW + half * 8 + ks * 16);

  load_first(t_lo, tid);
  f32x16 acc[1][1];
  const bf16_t* cW = sW + (wave_n * 32 + l32) * AROW + half * 8;
  auto multiply = [&]() {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks)
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(cW + ks * 16), fa[ks], acc[0][0], 0, 0, 0);
  };
  // this lane's 4 consecutive columns of group q: acc[4q .. 4q+3]
  auto lane_bias = [&](const void* bias, int64_t n_total, int64_t n0, int q) {
    bf16x4 bv = {(bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f};
    if (!bias) return bv;
    const uint32_t c = wave_n * 32 + 8 * q + 4 * half, last = (uint32_t)(n_total - 4 - n0);      // (n < 2^31: at most 48 tiles)
    return *reinterpret_cast<const bf16x4*>((const unsigned char*)((const bf16_t*)bias + n0) + (c < last ? c : last) * 2);
  };

  for (int t = t_lo; t < t_hi; ++t) {
    const ProjPart& pp = p.part[ka.tile_part[t]];
    const int64_t n0 = ka.tile_n0[t];
    const bool gated = pp.gated != 0;
    // (opaque copy of the thread index: see the note at the epilogue below)
    int w_tid = tid;
    asm volatile("" : "+v"(w_tid));
    store_w(w_tid);
    __syncthreads();                         // the tile is in LDS (and, the first time, every wave has its rows: sA is free)
    // the next weight tile is in flight while this one is multiplied and stored
    if (gated) load_w(pp.w, pp.n, n0, w_tid);
    else if (t + 1 < t_hi) load_first(t + 1, w_tid);
    multiply();
    if (gated) {
      __syncthreads();                       // every wave is done reading the gate's weights
      // sigmoid(gate) stays in registers; the projection tile of the pair follows at once
      f32x16 sg;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bf16x4 bv = lane_bias(pp.bias_gate, pp.n, n0, q);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) sg[4 * q + jj] = sigmoid_newton(acc[0][0][4 * q + jj] + bf2f(bv[jj]));
      }
      store_w(w_tid);
      __syncthreads();
      if (t + 1 < t_hi) load_first(t + 1, w_tid);
      multiply();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bf16x4 bv = lane_bias(pp.bias, pp.n, n0, q);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) acc[0][0][4 * q + jj] = (acc[0][0][4 * q + jj] + bf2f(bv[jj])) * sg[4 * q + jj];
      }
    } else {
      // bias and activation here, one uniform branch per tile, so that the epilogue below exists once
      const int act = pp.act;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bf16x4 bv = lane_bias(pp.bias, pp.n, n0, q);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) acc[0][0][4 * q + jj] += bf2f(bv[jj]);
      }
      if (act == AC_ACT_GELU_ERF) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] = gelu_table(acc[0][0][r], gelu_tab);
      } else if (act == AC_ACT_SIGMOID) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] = sigmoid_newton(acc[0][0][r]);
      } else if (act == AC_ACT_RELU) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] = fmaxf(acc[0][0][r], 0.f);
      } else if (act == AC_ACT_GELU_TANH) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] = gelu_tanh(acc[0][0][r]);
      }
    }
    LinearArgs g{};
    g.out = pp.out; g.ldo = pp.ldo; g.o_period = pp.o_period; g.o_s1 = pp.o_s1; g.o_s2 = pp.o_s2;
    g.out_t = pp.out_t; g.n_split = pp.out_t ? 0 : pp.n;
    g.t_period = pp.t_period; g.t_s1 = pp.t_s1; g.t_s2 = pp.t_s2; g.t_s3 = pp.t_s3;
    g.m = p.rows; g.n = pp.n;
    // The epilogue's many per-lane addresses do not depend on the tile; hoisted out of this loop
    // they would occupy registers for the whole kernel (and spill).  Opaque copies of the lane
    // coordinates make them values of this iteration, recomputed per tile with a few ALU ops.
    int e_tid = tid, e_l32 = l32, e_half = half, e_wm = wave_m, e_wn = wave_n;
    asm volatile("" : "+v"(e_tid), "+v"(e_l32), "+v"(e_half), "+v"(e_wm), "+v"(e_wn));
    // The barrier between the staging tile's writes and reads is also where every wave is done with the weights; the tile is written
    // again behind the next tile's first barrier.
    if (!epilogue_tile<AC_ACT_NONE, BM, BN, 2, 2, true, true>(g, acc, sA, gelu_tab, m0, n0, e_wm, e_wn, e_l32, e_half, e_tid)) __syncthreads();
  }
}

// The same for many rows, where the parts make up 256 or 512 weight columns: weights in registers, 32 columns of each of SLOTS parts per wave (a
// gated pair: both weights of the same 32 columns), for all the row tiles that a block of eight waves walks.  The next tile's rows are normalised into a second
// buffer while this one's are multiplied, one barrier a tile, and a wave stores its own results through LDS of its own.  A part that is stored strided takes the
// product with its operands exchanged, which leaves a lane runs of rows instead of runs of columns.  The matrix instructions and their order are the kernel's
// above: equal bits.  What bounded that one is vector work and its two barriers per 64 columns: per 64 rows and 512 columns it also moves 128 KB of weights from L2
// through registers into LDS.  Two gated pairs of 1048576 rows of 128 367 -> 242 us (3.3 TB/s; 409 -> 255 by columns), q, k, v and gate of 524288 rows 232 -> 154,
// q and gate 147 -> 98; of 40000 rows 22.8 -> 17.8, 20000 rows 16.8 -> 15.6.  Beside 256 columns a few of one more part (the pair bias) are the work of one wave, in
// turn, with their weights in LDS: bias, k and v of 1048576 rows 312 -> 192.
struct LnProjSlice { int part, n0; };
struct LnProjSliceArgs { LnProjArgs a; LnProjSlice slice[16]; int narrow; };   // narrow: part of fewer than 32 columns, or -1

template <int K, int SLOTS, bool GATED, int BM, bool NARROW>
__global__ void __launch_bounds__(512) ln_proj_slices_bf16(LnProjSliceArgs ka) {
  constexpr int NT = 512, AROW = K + 8, G = K / 8, RPP = NT / G, PASSES = BM / RPP > 0 ? BM / RPP : 1, KSTEPS = K / 16, SUB = BM / 32;
  constexpr int W = GATED ? 2 : SLOTS, SROW = 40, TROW = BM + 8, STAGE = 32 * (TROW > SROW ? TROW : SROW);   // (a gated pair: gate, value)
  static_assert(!GATED || SLOTS == 1, "a pair per wave");
  __shared__ __attribute__((aligned(16))) bf16_t sA[2][BM * AROW];
  __shared__ __attribute__((aligned(16))) bf16_t sStage[8][STAGE];
  __shared__ __attribute__((aligned(16))) bf16_t sN[NARROW ? 32 * AROW : 8];     // the narrow part's weights (rows past its last shadow it)
  const LnProjArgs& p = ka.a;
  const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64), l32 = lane % 32, half = lane / 32;
  bf16_t* const stage = sStage[wave];
  bf16x8 w[W][KSTEPS];
  bf16x4 bias[W][4];                       // of the lane's columns 8 q + 4 half + 0..3
  float bias_t[W];                         // of its column, where the part is stored strided
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const LnProjSlice sl = ka.slice[GATED ? wave : wave + 8 * i];
    const ProjPart& q = p.part[sl.part];
    const bf16_t* wp = (const bf16_t*)(GATED && i == 0 ? q.w_gate : q.w) + (int64_t)(sl.n0 + l32) * K + half * 8;
    const bf16_t* bp = (const bf16_t*)(GATED && i == 0 ? q.bias_gate : q.bias);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) w[i][ks] = *reinterpret_cast<const bf16x8*>(wp + ks * 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) bias[i][j] = bp ? *reinterpret_cast<const bf16x4*>(bp + sl.n0 + 8 * j + 4 * half) : bf16x4{};
    bias_t[i] = bp ? bf2f(bp[sl.n0 + l32]) : 0.f;
  }
  const int lg = tid % G, rg = tid / G;
  const bf16_t* x = (const bf16_t*)p.x;
  const bf16x8 gain = *reinterpret_cast<const bf16x8*>((const bf16_t*)p.gain + lg * 8), shift = *reinterpret_cast<const bf16x8*>((const bf16_t*)p.shift + lg * 8);
  bf16x8 xr[PASSES];
  auto load = [&](int64_t t) {
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      int64_t r = t * BM + ps * RPP + rg;
      if (r > p.rows - 1) r = p.rows - 1;     // rows past the end shadow the last row; never stored
      int64_t at = r * p.ldx;
      if (p.x_period > 0) {
        int64_t q, c;
        split_row(r, p.x_period, q, c);
        at = q * p.x_s1 + c * p.x_s2;
      }
      xr[ps] = *reinterpret_cast<const bf16x8*>(x + at + lg * 8);
    }
  };
  auto normalise = [&](bf16_t* dst) {
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      float v[8], sum = 0.f, sq = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) { v[j] = bf2f(xr[ps][j]); sum += v[j]; }
      const float mean = group_sum<G>(sum) * (1.0f / K);
#pragma unroll
      for (int j = 0; j < 8; ++j) { const float d = v[j] - mean; sq += d * d; }
      const float rstd = rsqrtf(group_sum<G>(sq) * (1.0f / K) + p.eps);
      float o[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] = (v[j] - mean) * rstd * bf2f(gain[j]) + bf2f(shift[j]);
      if (RPP <= BM || rg < BM) store_vec(dst + (ps * RPP + rg) * AROW + lg * 8, o);
    }
  };
  if (NARROW) {
    const ProjPart& q = p.part[ka.narrow];
    for (int c = tid; c < 32 * G; c += NT)
      *reinterpret_cast<bf16x8*>(sN + c / G * AROW + c % G * 8) =
          *reinterpret_cast<const bf16x8*>((const bf16_t*)q.w + (c / G < (int)q.n ? c / G : (int)q.n - 1) * K + c % G * 8);
  }
  const int64_t tiles = (p.rows + BM - 1) / BM;
  load(blockIdx.x);
  normalise(sA[0]);
  if (blockIdx.x + (int64_t)gridDim.x < tiles) load(blockIdx.x + (int64_t)gridDim.x);
  __syncthreads();
  auto stage_strided = [&](const f32x16& v, int s) {      // this lane's column, its rows of 32-row tile s
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<bf16x4*>(stage + l32 * TROW + s * 32 + 8 * j + 4 * half) = bf16x4{f2bf(v[4 * j]), f2bf(v[4 * j + 1]), f2bf(v[4 * j + 2]), f2bf(v[4 * j + 3])};
  };
  auto store_strided = [&](const ProjPart& q, int n0, int columns, int64_t m0) {
    __builtin_amdgcn_wave_barrier();         // (a wave's LDS operations are in order)
#pragma unroll
    for (int c = 0; c < BM / 16; ++c) {      // 32 columns of BM / 8 runs of eight rows
      const int e = lane + 64 * c, n = e / (BM / 8), mm = e % (BM / 8) * 8;
      int64_t qq, rr;
      split_row(m0 + mm, q.t_period, qq, rr);
      if (n < columns && m0 + mm < p.rows)
        *reinterpret_cast<bf16x8*>((bf16_t*)q.out_t + qq * q.t_s1 + rr + (n0 + n) * q.t_s3) = *reinterpret_cast<const bf16x8*>(stage + n * TROW + mm);
    }
    __builtin_amdgcn_wave_barrier();
  };
  int buf = 0, turn = 0;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x, buf ^= 1, turn = (turn + 1) % 8) {
    if (t + gridDim.x < tiles) {
      normalise(sA[buf ^ 1]);
      if (t + 2 * (int64_t)gridDim.x < tiles) load(t + 2 * (int64_t)gridDim.x);
    }
    const int64_t m0 = t * BM;
    bf16x8 fa[SUB][KSTEPS];
#pragma unroll
    for (int s = 0; s < SUB; ++s)
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) fa[s][ks] = *reinterpret_cast<const bf16x8*>(sA[buf] + (s * 32 + l32) * AROW + half * 8 + ks * 16);
#pragma unroll
    for (int i = 0; i < SLOTS; ++i) {
      const LnProjSlice sl = ka.slice[wave + 8 * i];
      const ProjPart& q = p.part[sl.part];
      const int act = q.act;
      if (GATED || q.out_t) {
#pragma unroll
        for (int s = 0; s < SUB; ++s) {
          f32x16 g = {}, v = {};
#pragma unroll
          for (int ks = 0; ks < KSTEPS; ++ks) {
            if (GATED) g = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][ks], w[0][ks], g, 0, 0, 0);
            v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][ks], w[GATED ? 1 : i][ks], v, 0, 0, 0);
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) v[r] += bias_t[GATED ? 1 : i];
          if (GATED) {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] *= sigmoid_newton(g[r] + bias_t[0]);
          } else if (act == AC_ACT_SIGMOID) {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = sigmoid_newton(v[r]);
          }
          stage_strided(v, s);
        }
        store_strided(q, sl.n0, 32, m0);
      } else {
#pragma unroll
        for (int s = 0; s < SUB; ++s) {
          f32x16 v = {};
#pragma unroll
          for (int ks = 0; ks < KSTEPS; ++ks) v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[i][ks], fa[s][ks], v, 0, 0, 0);
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * j + e] += bf2f(bias[i][j][e]);
          if (act == AC_ACT_SIGMOID) {
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = sigmoid_newton(v[r]);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
            *reinterpret_cast<bf16x4*>(stage + l32 * SROW + 8 * j + 4 * half) = bf16x4{f2bf(v[4 * j]), f2bf(v[4 * j + 1]), f2bf(v[4 * j + 2]), f2bf(v[4 * j + 3])};
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int c = 0; c < 2; ++c) {      // 32 rows of four runs of eight columns
            const int e = lane + 64 * c, r = e / 4, cc = e % 4 * 8;
            if (m0 + s * 32 + r < p.rows)
              *reinterpret_cast<bf16x8*>((bf16_t*)q.out + (m0 + s * 32 + r) * q.ldo + sl.n0 + cc) = *reinterpret_cast<const bf16x8*>(stage + r * SROW + cc);
          }
          __builtin_amdgcn_wave_barrier();
        }
      }
    }
    if (NARROW && wave == turn) {            // (a tile's narrow columns are one wave's, each in its turn)
      const ProjPart& q = p.part[ka.narrow];
      const float b = q.bias ? bf2f(((const bf16_t*)q.bias)[l32 < (int)q.n ? l32 : (int)q.n - 1]) : 0.f;
#pragma unroll
      for (int s = 0; s < SUB; ++s) {
        f32x16 v = {};
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
          v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][ks], *reinterpret_cast<const bf16x8*>(sN + l32 * AROW + half * 8 + ks * 16), v, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] += b;
        stage_strided(v, s);
      }
      store_strided(q, 0, (int)q.n, m0);
    }
    __syncthreads();
  }
}

bool ln_proj_shapes_ok(int dtype, int64_t k, const int64_t* n, int n_parts) {
  if (dtype != AC_BF16 || (k != 64 && k != 128)) return false;
  if (n_parts < 1 || n_parts > kMaxProjParts) return false;
  int64_t tiles = 0;
  for (int i = 0; i < n_parts; ++i) {
    if (n[i] < 4 || n[i] % 4 != 0) return false;
    tiles += (n[i] + kLnProjCols - 1) / kLnProjCols;
  }
  return tiles <= kMaxProjTiles;
}

// Whether some part's results may lie on top of the input rows (by the ranges of addresses that they span).
static bool ln_proj_overlaps(const LnProjArgs& p) {
  auto span = [&](int64_t period, int64_t s1, int64_t s2, int64_t n, int64_t sn, int64_t& lo, int64_t& hi) {
    const int64_t q = (p.rows - 1) / period * s1, r = ((p.rows < period ? p.rows : period) - 1) * s2, c = (n - 1) * sn;
    lo = (q < 0 ? q : 0) + (r < 0 ? r : 0) + (c < 0 ? c : 0);
    hi = (q > 0 ? q : 0) + (r > 0 ? r : 0) + (c > 0 ? c : 0);
  };
  int64_t x0, x1;
  if (p.x_period > 0) span(p.x_period, p.x_s1, p.x_s2, p.k, 1, x0, x1);
  else span(INT64_MAX, 0, p.ldx, p.k, 1, x0, x1);
  const bf16_t *x_lo = (const bf16_t*)p.x + x0, *x_hi = (const bf16_t*)p.x + x1 + 1;
  for (int i = 0; i < p.n_parts; ++i) {
    const ProjPart& pp = p.part[i];
    const bf16_t* out = (const bf16_t*)(pp.out_t ? pp.out_t : pp.out);
    int64_t lo, hi;
    if (pp.out_t) span(pp.t_period, pp.t_s1, pp.t_s2, pp.n, pp.t_s3, lo, hi);
    else if (pp.o_period == INT64_MAX) span(INT64_MAX, 0, pp.ldo, pp.n, 1, lo, hi);
    else span(pp.o_period, pp.o_s1, pp.o_s2, pp.n, 1, lo, hi);
    if (out + lo < x_hi && x_lo < out + hi + 1) return true;
  }
  return false;
}

template <int K, int BN>
static hipError_t ln_proj_launch(const LnProjKernelArgs& ka, hipStream_t s) {
  auto kern = ln_multi_proj_bf16<K, BN>;
  constexpr size_t lds_max = (size_t)ln_proj_lds_elems(K) * sizeof(bf16_t) + kGeluTableBytes;
  static const hipError_t attr_status = hipFuncSetAttribute(
      reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
  if (attr_status != hipSuccess) return attr_status;
  // the GELU table is only there when a part needs it
  const size_t lds = lds_max - (ka.any_gelu ? 0 : kGeluTableBytes);
  const int64_t blocks = (ka.a.rows + kLnProjRows - 1) / kLnProjRows;
  // Four blocks fit a CU (five at K = 64).  A launch of few rows would leave places empty and walk all its weight tiles one after
  // another: the tiles are then shared out over as many blocks per 64 rows as there is room for, each of which
  // normalises the rows again (8000 rows of 128, q, k, v, gate of the triangle attention: 19 -> 8.4 us).  Where results may
  // lie on the rows (a projection in place) one block has to have read them all before it writes, as without shares.
  const int64_t room = ln_proj_overlaps(ka.a) ? 1 : 1024 / blocks;
  const unsigned shares = (unsigned)(room < 1 ? 1 : room < ka.n_tiles ? room : ka.n_tiles);
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks, shares), dim3(256), lds, s, ka);
  return hipGetLastError();
}

// The slices of the parts for the kernel of whole slices, if it covers them: 8 or 16 of 32 columns (8 gated pairs), whole 16-byte chunks of rows or
// columns in every store, no result on the rows; beside eight a plain part of fewer columns that is stored strided (the pair bias).  Returns their number, or 0.
static int ln_proj_slices(const LnProjArgs& p, LnProjSliceArgs& sa) {
  int n = 0;
  sa.narrow = -1;
  for (int i = 0; i < p.n_parts; ++i) {
    const ProjPart& q = p.part[i];
    const bool narrow = q.n < 32 && q.out_t && !q.gated && q.act == AC_ACT_NONE && sa.narrow < 0;
    if ((q.n % 32 != 0 && !narrow) || q.gated != p.part[0].gated || (q.gated ? q.act != AC_ACT_NONE : q.act != AC_ACT_NONE && q.act != AC_ACT_SIGMOID)) return 0;
    if (q.out_t) {
      if (q.t_s2 != 1 || q.t_s1 % 8 != 0 || q.t_s3 % 8 != 0 || p.rows % 8 != 0 || (q.t_period != INT64_MAX && q.t_period % 8 != 0) || (uintptr_t)q.out_t % 16 != 0) return 0;
    } else if (q.gated || q.o_period != INT64_MAX || q.ldo % 8 != 0 || (uintptr_t)q.out % 16 != 0) {
      return 0;
    }
    if (narrow) { sa.narrow = i; continue; }
    for (int n0 = 0; n0 < q.n; n0 += 32, ++n) {
      if (n == 16) return 0;
      sa.slice[n] = LnProjSlice{i, n0};
    }
  }
  return (n == 8 || (n == 16 && !p.part[0].gated && sa.narrow < 0)) && !ln_proj_overlaps(p) ? n : 0;
}
// Where the kernel of whole slices is ahead.  It has a block per CU, which first loads all its weights and, up to 8192 rows, uses them for one tile; the
// kernel of 64-column tiles shares a short launch's columns out over more blocks.  The bits are the same.  us, slices / tiles, 128 wide: q, k, v and gate 7.7 /
// 5.2 at 256 rows, 8.9 / 8.2 at 8192, 10.1 / 10.3 at 9000, 12.8 / 14.4 at 18000; two gated pairs 7.3 / 6.2 at 256, 9.6 / 8.4 at 10400, 12.5 / 13.2 at 18000;
// bias, k and v 5.7 / 5.2 at 1024, 5.9 / 5.9 at 4096, 6.2 / 6.9 at 8192; k and v alone 4.9 / 5.1 at 256.  64 wide: the pairs 8.3 / 7.6 at 16384, 12.9 / 12.5 at 32768,
// 14.7 / 17.6 at 36000; bias, k and v 6.9 / 6.3 at 13000, 6.9 / 8.1 at 14400; k and v alone (one strided) 4.6 / 4.7 at 968, 7.2 / 6.1 at 10440, 6.3 / 6.4 at 13992.
static bool ln_proj_slices_ahead(const LnProjArgs& p, const LnProjSliceArgs& sa, int slices) {
  if (p.part[0].gated) return p.rows > (p.k == 128 ? 16384 : 32768);
  if (sa.narrow >= 0) return p.rows > (p.k == 128 ? 4096 : 13312);
  return slices == 16 ? p.rows > 8192 : p.k == 128 || p.rows <= 8192 || p.rows > 13312;
}
template <int K, int SLOTS, bool GATED, bool NARROW = false> static hipError_t ln_proj_slices_launch(const LnProjSliceArgs& sa, hipStream_t s) {
  const int64_t rows = sa.a.rows;
  // one block per CU; tiles of 32 rows while a block has less than eight of 64 (20000 rows: 625 of 32 are three a block, 313 of 64 two, with twice the work)
  if (rows < 64 * 256 * 8) hipLaunchKernelGGL((ln_proj_slices_bf16<K, SLOTS, GATED, 32, NARROW>), dim3((unsigned)((rows + 31) / 32 < 256 ? (rows + 31) / 32 : 256)), dim3(512), 0, s, sa);
  else hipLaunchKernelGGL((ln_proj_slices_bf16<K, SLOTS, GATED, 64, NARROW>), dim3(256), dim3(512), 0, s, sa);
  return hipGetLastError();
}

hipError_t launch_ln_proj(const LnProjArgs& p_in, hipStream_t s) {
  if (p_in.rows <= 0) return hipSuccess;
  LnProjKernelArgs ka{};
  ka.a = p_in;
  LnProjArgs& p = ka.a;
  int64_t ns[kMaxProjParts];
  if (p.n_parts < 1 || p.n_parts > kMaxProjParts) return hipErrorInvalidValue;
  for (int i = 0; i < p.n_parts; ++i) ns[i] = p.part[i].n;
  if (!ln_proj_shapes_ok(AC_BF16, p.k, ns, p.n_parts)) return hipErrorNotSupported;
  if ((p.x_period > 0 ? p.x_s1 % 8 != 0 || p.x_s2 % 8 != 0 : p.ldx % 8 != 0) || ((uintptr_t)p.x % 16) != 0 || ((uintptr_t)p.gain % 16) != 0 || ((uintptr_t)p.shift % 16) != 0)
    return hipErrorNotSupported;
  if (p.rows > 0x7fffffffLL) return hipErrorInvalidValue;
  for (int i = 0; i < p.n_parts; ++i) {
    ProjPart& pp = p.part[i];
    if (!pp.w || ((uintptr_t)pp.w % 16) != 0 || ((uintptr_t)pp.w_gate % 16) != 0) return hipErrorNotSupported;
    if (pp.gated && !pp.w_gate) return hipErrorInvalidValue;
    if (((uintptr_t)pp.bias % 8) != 0 || ((uintptr_t)pp.bias_gate % 8) != 0) return hipErrorNotSupported;
    if (pp.out_t == nullptr && (pp.out == nullptr || pp.ldo % 4 != 0 || ((uintptr_t)pp.out % 8) != 0)) return hipErrorNotSupported;
    if (pp.t_period <= 0) pp.t_period = INT64_MAX;
    if (pp.o_period <= 0) pp.o_period = INT64_MAX;
    if (pp.o_period != INT64_MAX && (pp.o_s1 % 4 != 0 || pp.o_s2 % 4 != 0)) return hipErrorNotSupported;
    if (pp.act == AC_ACT_GELU_ERF && !pp.gated) ka.any_gelu = 1;
  }
  LnProjSliceArgs sa{};
  if (const int slices = ln_proj_slices(p, sa); slices > 0 && ln_proj_slices_ahead(p, sa, slices)) {
    sa.a = p;
    const bool gated = p.part[0].gated != 0;
    if (sa.narrow >= 0) return p.k == 128 ? ln_proj_slices_launch<128, 1, false, true>(sa, s) : ln_proj_slices_launch<64, 1, false, true>(sa, s);
    if (p.k == 128) return gated ? ln_proj_slices_launch<128, 1, true>(sa, s) : slices == 16 ? ln_proj_slices_launch<128, 2, false>(sa, s) : ln_proj_slices_launch<128, 1, false>(sa, s);
    return gated ? ln_proj_slices_launch<64, 1, true>(sa, s) : slices == 16 ? ln_proj_slices_launch<64, 2, false>(sa, s) : ln_proj_slices_launch<64, 1, false>(sa, s);
  }
  for (int i = 0; i < p.n_parts; ++i)
    for (int64_t n0 = 0; n0 < p.part[i].n; n0 += kLnProjCols) {   // a gated pair is one entry: two weight tiles, one output tile
      ka.tile_part[ka.n_tiles] = i;
      ka.tile_n0[ka.n_tiles++] = (int)n0;
    }
  return p.k == 128 ? ln_proj_launch<128, kLnProjCols>(ka, s) : ln_proj_launch<64, kLnProjCols>(ka, s);
}

static bool aligned_to(const void* p, uintptr_t a) { return p == nullptr || ((uintptr_t)p % a) == 0; }

static bool mfma_eligible(const LinearArgs& g) {
  if (g.dtype != AC_BF16) return false;
  if (g.k % 8 != 0) return false;
  if (g.n % 4 != 0 || g.n_split % 4 != 0) return false;
  if (g.lda % 8 != 0 || g.ldw % 8 != 0) return false;
  if (!aligned_to(g.a, 16) || !aligned_to(g.w, 16)) return false;
  if (g.n_split > 0 && (g.ldo % 4 != 0 || !aligned_to(g.out, 8))) return false;
  if (g.o_period != INT64_MAX && (g.o_s1 % 4 != 0 || g.o_s2 % 4 != 0)) return false;
  if (g.batch > 1 && (g.sa_b % 8 != 0 || g.sw_b % 8 != 0 || g.so_b % 4 != 0)) return false;
  if (g.bias && !aligned_to(g.bias, 8)) return false;
  if (g.mul && (g.ldmul % 4 != 0 || !aligned_to(g.mul, 8))) return false;
  if (g.resid && (g.ldr % 4 != 0 || !aligned_to(g.resid, 8))) return false;
  return true;
}

// Tile shapes of the bf16 GEMM, and the one with the least estimated time.  A launch is tiles / 256 rounds of the CUs of k / 64
// steps plus a prologue and an epilogue per tile, plus what is paid once.  A last round that is partly empty counts whole
// for the shapes that have a CU to themselves (1.25 rounds of 256x256 tiles of 8192 x 2560 x 320 take 39.7 us, two take 37) and half
// for those that share it.  The three times of a shape, in us, are fitted to 68 launches of 512 to 65536 rows x 64 to
// 4096 columns x 64 to 4096 deep, batched ones among them, on which the choice is within 5 % of the best shape; on 140 others of 1 to 70000 rows
// and ragged sizes it is 2 % off on average and 23 % at worst.  Shapes whose blocks share a CU pay little per tile and more per step.  Examples (us; 256x256 / 256x128 / 128x128 ring / 128x128 / 128x64 /
// 64x64 / 32x64):  65536x1024x1024  144 / 181 / 230 / 182 / 236 / 251 / 359;  6400x1024x1024  27 / 20 / 23 / 23 / 26 / 27 / 35;
// 4000x1024x4096  78 / 56 / 42 / 46 / 52 / 64 / 83;  512x1024x4096  72 / 43 / 27 / 40 / 29 / 21 / 14.5.
// What 32x64 pays once is set by launches of one round inside models, whose operands another kernel has just written: 128x2048x512 takes
// 7.0 us on it and 8.1 on 64x64 (which 5.4 us instead of 5.0 had preferred), 128x1536x384 6.7 and 7.7, 152x4096x1024 (320 tiles)
// 10.0 and 9.0.
// 128x192 fills rounds that the others leave half empty or padded (6400x768x3072 47.2 us on 256x128, 43.8 on it; 2048x3072x768 19.1 and 17.0;
// 1600x3072x768 17.0 and 14.7).  Its prices are fitted to 475 launches of 256 to 65536 rows whose operands another kernel has just written: the choice
// among all seven is 1.8 % off the best on those on average, 1.6 % on 465 others and 34 % at worst (14105x576x512).  Inside stacks of twelve
// layers, one after another without a pause, it is mostly ahead of 256x128 too: 3200 rows, d 768, in two launches a layer 2210 -> 2160 us, 6144 rows
// 4235 -> 4115, 2048 rows in one 1219 -> 1212; 4096 rows in two, whose 256 tiles load every CU at once, 2447 -> 2500.
// The k order is the same for all of them, and so are the bits.
enum TileShape { kQuad, k256x128, k128x128Ring, k128x192, k128x128, k128x64, k64x64, k32x64, kTileShapes };
// A grid dimension counts its threads in 32 bits: a shape whose blocks of a launch are more than that is not a choice.
static bool grid_fits(int64_t tiles, int threads) { return tiles <= 0xffffffffLL / threads; }
static int64_t tiles_of(const LinearArgs& g, int bm, int bn) { return ((g.m + bm - 1) / bm) * ((g.n + bn - 1) / bn); }
// The loops that exist for a shape: kPlain any k of whole tiles, kRagged k that ends inside one, kConv the convolution, kWide row strides of 2^22 elements and more (8 MB:
// the ring and quad loops address a tile's rows with 32-bit byte offsets; the register-staged ones with 64-bit pointers).
enum Form { kPlain = 1, kConv = 2, kWide = 4, kRagged = 8 };
// (blocks that have a CU to themselves pay whole rounds, those that share it half of the last one's empty part)
static double estimate_us(int64_t tiles, double steps, double step, double tile, double once, bool alone) {
  const double exact = (double)tiles / 256, whole = (double)((tiles + 255) / 256);
  const double rounds = whole <= 1 ? 1 : alone ? whole : 0.5 * (exact + whole);
  return rounds * (steps * step + tile) + once;
}
static TileShape best_tile(const LinearArgs& g, Form form) {
  struct Cost { int bm, bn, threads; double step, tile, once; bool alone; int forms; };
  static const Cost costs[kTileShapes] = {{256, 256, 512, 1.06, 11.9, 0.0, true, kPlain},         {256, 128, 512, 0.65, 8.1, 0.0, true, kPlain | kRagged},
                                          {128, 128, 512, 0.46, 4.4, 1.0, true, kPlain | kConv},  {128, 192, 512, 0.58, 6.5, 1.85, true, kPlain},
                                          {128, 128, 256, 0.52, 2.7, 4.4, false, kPlain | kWide},
                                          {128, 64, 256, 0.36, 1.4, 4.3, false, kPlain | kConv},  {64, 64, 256, 0.17, 0.8, 4.8, false, kPlain | kConv | kWide | kRagged},
                                          {32, 64, 128, 0.13, 0.65, 5.0, false, kPlain | kWide}};
  int best = -1;
  double best_t = 0;
  for (int c = 0; c < kTileShapes; ++c) {
    if (!(costs[c].forms & form)) continue;
    if (!grid_fits(tiles_of(g, costs[c].bm, costs[c].bn), costs[c].threads)) continue;
    const int64_t tiles = tiles_of(g, costs[c].bm, costs[c].bn) * g.batch;
    const double t = estimate_us(tiles, (double)((g.k + kBK - 1) / kBK), costs[c].step, costs[c].tile, costs[c].once, costs[c].alone);
    if (best < 0 || t < best_t) { best = c; best_t = t; }
  }
  return best < 0 ? (form == kConv ? k128x128Ring : form == kWide ? k128x128 : form == kRagged ? k256x128 : kQuad) : (TileShape)best;
}

// The convolution's tile: its sums are long (9 C_in) and its columns few, so the time per step decides, and that depends on how many CUs load
// at once.  A launch takes the larger of what one block needs by itself (`step1`, `once1`) and what the rounds need with every CU busy
// (a lone block's rounds count whole); between an empty and a full first round the two are mixed.  Fitted to 422
// launches (up to 100000 pixels, 128 to 640 channels in, 64 to 640 out): the choice is 0.2 % off the best of four on those, 0.4 % on 434 others and 14 % at worst
// (nine 55x89 images, 128 to 192).  Four 64x64 images of 320 channels: 51.9 on 128x128 and 128x64 (whose last
// columns are half padding), 47.8 on 64x64, 39.2 on 128x192; eight of 192: 37.8 / 35.9 / 36.8 / 26.8; four of 512: 84.5 / 94.8 / 110.9 / 97.5.
// (64 input channels: nine steps, as short as a product, and priced as one.)
static TileShape best_conv_tile(const LinearArgs& g) {
  if (g.conv_c == 64) return best_tile(g, kConv);
  struct Cost { TileShape shape; int bm, bn, threads; double step, tile, once, step1, once1; bool alone; };
  static const Cost costs[] = {{k128x192, 128, 192, 512, 0.67, 5.5, 1.5, 0.44, 9.6, true}, {k128x128Ring, 128, 128, 512, 0.506, 4.8, 1.1, 0.38, 7.2, true},
                               {k128x64, 128, 64, 256, 0.32, 1.6, 4.3, 0.36, 7.3, false},  {k64x64, 64, 64, 256, 0.18, 0.47, 4.9, 0.278, 5.6, false}};
  TileShape best = k128x128Ring;
  double best_t = 0;
  for (const Cost& c : costs) {
    const int64_t tiles = tiles_of(g, c.bm, c.bn);
    if (!grid_fits(tiles, c.threads)) continue;
    const double steps = (double)(g.k / kBK), exact = (double)tiles / 256, whole = (double)((tiles + 255) / 256);
    const double rounds = whole <= 1 ? 1 : c.alone ? whole : 0.5 * (exact + whole);
    const double one = steps * c.step1 + c.once1, busy = rounds * (steps * c.step + c.tile) + c.once;
    const double t = busy <= one ? one : one + (busy - one) * (exact < 1 ? exact : 1);
    if (best_t == 0 || t < best_t) { best = c.shape; best_t = t; }
  }
  return best;
}

// A gated product's tile, of the three whose waves hold a value and a gate tile of the same columns.  Its epilogue evaluates erf by formula for half of its
// accumulators, so it has prices of its own, fitted to 64 to 8192 rows x 2 * 256 to 2 * 5120 weight rows x 64 to 1280 deep; the choice is within 4 % of the
// best of the three on all of those, and ahead of product and gating pass apart.  In us, 64x128 / 256x128 / 256x256 / apart: 64 x 2*5120 x 1280 12.7 / 20.4 /
// 31.5 / 13.4; 512 of the same 30.7 / 25.3 / 36.0 / 32.6; 1024 50.1 / 49.4 / 39.1 / 47.0; 256 x 2*1280 x 320 6.8 / 11.1 / 16.5 / 10.0; 8192 of the same
// 35.2 / 36.4 / 36.5 / 46.9.  (128x128 on four or eight waves is never the best of them.)
static TileShape best_gated_tile(const LinearArgs& g) {
  struct Cost { TileShape shape; int bm, bn, threads; double step, tile, once; bool alone; };
  static const Cost costs[] = {{kQuad, 256, 128, 512, 1.5, 11.0, 0.0, true}, {k256x128, 256, 64, 512, 0.85, 8.0, 0.0, true}, {k64x64, 64, 64, 256, 0.32, 1.8, 4.0, false}};
  TileShape best = kQuad;
  double best_t = 0;
  for (const Cost& c : costs) {                    // (bn: columns of the result)
    const int64_t tiles = tiles_of(g, c.bm, c.bn);
    if (!grid_fits(tiles, c.threads)) continue;
    const double t = estimate_us(tiles, (double)(g.k / kBK), c.step, c.tile, c.once, c.alone);
    if (best_t == 0 || t < best_t) { best = c.shape; best_t = t; }
  }
  return best;
}

// fp32 products whose rows can be read 16 bytes at a time
static bool mfma_f32_eligible(const LinearArgs& g) {
  if (g.k % 4 != 0 || g.k > (1 << 30) || g.lda % 4 != 0 || g.ldw % 4 != 0 || g.bias_period > 0) return false;
  if (g.batch > 1 && (g.sa_b % 4 != 0 || g.sw_b % 4 != 0)) return false;
  return aligned_to(g.a, 16) && aligned_to(g.w, 16);
}
// ... and whose epilogue operands and output can be moved 16 bytes at a time
static bool f32_rows_vectorisable(const LinearArgs& g) {
  if (g.n_split % 4 != 0 || g.ldo % 4 != 0 || !aligned_to(g.out, 16)) return false;
  if (g.batch > 1 && g.so_b % 4 != 0) return false;
  if (g.o_period != INT64_MAX && (g.o_s1 % 4 != 0 || g.o_s2 % 4 != 0)) return false;
  if (g.mul && (g.ldmul % 4 != 0 || !aligned_to(g.mul, 16))) return false;
  if (g.resid && (g.ldr % 4 != 0 || !aligned_to(g.resid, 16))) return false;
  return aligned_to(g.bias, 16);
}

template <int TM, int TN>
static hipError_t mfma_f32_launch(const LinearArgs& g, hipStream_t s) {
  const int64_t tiles = ((g.m + 16 * TM - 1) / (16 * TM)) * ((g.n + 16 * TN - 1) / (16 * TN));
  hipLaunchKernelGGL((linear_mfma_f32<TM, TN>), dim3((unsigned)tiles, (unsigned)g.batch), dim3(256), 0, s, g, f32_rows_vectorisable(g) ? 1 : 0);
  return hipGetLastError();
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int BK>
static hipError_t ring_f32_launch(const LinearArgs& g, hipStream_t s) {
  auto kern = linear_ring_f32<BM, BN, WAVES_M, WAVES_N, BK>;
  constexpr int lds = 3 * (BM + BN) * BK * 4;
  static const hipError_t attr_status = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr_status != hipSuccess) return attr_status;
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles_of(g, BM, BN), (unsigned)g.batch), dim3(256), lds, s, g, f32_rows_vectorisable(g) ? 1 : 0);
  return hipGetLastError();
}

// The kernel a product runs on: a function of sizes, types, strides and alignment, decided on the host.
enum Route { kFma, kF32_32x64, kF32_32x32, kF32_32x16, kF32_16x16, kF32Ring32x64, kF32Ring32x32, kF32Ring32x32Deep, kRouteQuad, kRing256x128, kRing128x128, kRing128x192, kStaged128x128, kRing128x64, kRing64x64,
             kStaged64x64, kStaged32x64, kRagged256x128, kRagged64x64, kConv128x128, kConv128x192, kConv128x64, kConv64x64, kConvWide64x64, kRoutes };
static const char* const kRouteName[kRoutes] = {
    "fma 64x64", "f32 32x64", "f32 32x32", "f32 32x16", "f32 16x16", "f32-ring 32x64", "f32-ring 32x32", "f32-ring-deep 32x32", "quad 256x256", "ring 256x128", "ring 128x128", "ring 128x192", "staged 128x128", "ring 128x64", "ring 64x64",
    "staged 64x64", "staged 32x64", "ragged 256x128", "ragged 64x64", "conv 128x128", "conv 128x192", "conv 128x64", "conv 64x64", "conv-wide 64x64"};

static bool wide_rows(const LinearArgs& g) { return g.lda >= (1 << 22) || g.ldw >= (1 << 22); }

static Route bf16_route(const LinearArgs& g) {
  if (wide_rows(g)) {
    if (g.k % kBK != 0) return kFma;
    const TileShape staged = best_tile(g, kWide);
    return staged == k128x128 ? kStaged128x128 : staged == k64x64 ? kStaged64x64 : kStaged32x64;
  }
  if (g.k % kBK != 0) {
    // a depth that is no multiple of a tile's 64 (whole rows of 16-byte chunks all the same): the products over the positions of
    // a pair tensor, whose size is a sequence's length.  128 products of 40 x 200 x 200: 42 us in the FMA kernel, 8.9 us here.
    // Chosen among the two shapes that are built for it (4 products of 2000 x 2100 x 1000: 72 us on 256x128, 87 on 64x64).
    return best_tile(g, kRagged) == k64x64 ? kRagged64x64 : kRagged256x128;
  }
  switch (best_tile(g, kPlain)) {
    case kQuad: return kRouteQuad;
    case k256x128: return kRing256x128;
    case k128x128Ring: return kRing128x128;
    case k128x192: return kRing128x192;
    case k128x128: return kStaged128x128;
    case k128x64: return kRing128x64;
    // (alone on its CU and with a long k such a block gains nothing from direct loads and the register-staged loop, which also keeps a whole tile's
    // fragments in registers, is ahead: 512 x 1024 x 4096 18.1 against 20.7 us, 1000 x 1024 x 4096 inside a model 22 against 26;
    // with two or three blocks per CU it is behind: 512 x 3072 x 768 11.3 against 10.4)
    case k64x64: return g.k >= 512 && tiles_of(g, 64, 64) * g.batch <= 256 ? kStaged64x64 : kRing64x64;
    default: return kStaged32x64;
  }
}

static Route f32_route(const LinearArgs& g) {
  // Many columns of at most 64 terms: what is left is the store of the output, at which the FMA kernel's 64x64 tiles are ahead once there are
  // rows for it (16000 x 1024 x 64 61 against 77 us, 16000 x 8192 x 32 278 against 360) and behind before (256 x 1024 x 64 12.5 against 4.9).
  // By k and n alone, as the two kernels sum in different orders and a row's bits must not depend on the launch's rows.
  if (g.k <= 64 && g.n >= 1024) return kFma;
  // Depths of whole tiles in each of a sum's four parts: the ring where a launch has the rows and columns for it, the kernel whose waves share out k where it
  // is short of blocks and a quarter of the chain counts.  Estimated time: steps x the larger of what one block needs by itself (ring) and what its rounds
  // need together, plus per tile, plus once, in us; fitted to 80 products of 68 to 16000 rows x 72 to 2848 columns x 128 to 3968 deep, on which the choice is
  // 1 % off the best of the five on average and 6 % at worst and 1.23 times ahead of the best without the ring.  us, 32x64 / 32x32 ring, 32x64 / 32x32 / 32x16 /
  // 16x16 shared: 1024 x 1536 x 512 19.2 / 21.7, 33.1 / 34.9 / 49.8 / 65.1; 1024 x 512 x 2048 29.9 / 31.8, 30.1 / 34.9 / 49.8 / 65.0; 256 x 512 x 2048 28.6 / 25.1,
  // 29.0 / 18.6 / 15.0 / 18.8; 16000 x 512 x 512 79 / 92, 149 / 172 / 250 / 330; 96 x 512 x 2048 29 / 25, 29 / 19 / 15 / 11.  (Rings of 64x64 and 128x64 are never
  // more than 1 % ahead.)  Over 404 more products, half of them of 40 rows or columns at most and many in batches, the choice is 1.11 times ahead of the four shared tiles
  // by their prices below; 9 are more than 4 % behind, all but one of 22 rows or columns at most (64 products of 1 x 704 x 2048 69 -> 81 us, 8 of 1 x 2244 x 4352 65 -> 82; a
  // line at 16 rows and columns would cost more than it gives: 64 of 2460 x 12 x 768 103 us, 140 on shared tiles).
  if (g.k % 128 == 0 && g.k <= (1 << 26) && !wide_rows(g)) {
    // Where the parts are whole tiles of 64 terms too, the 32x32 ring takes those: half the barriers, which a launch of one or two blocks per CU waits at
    // (1024 x 512 x 2048 31.0 -> 28.1, 256 x 512 x 2048 24.5 -> 20.1, 1024 x 512 x 512 10.8 -> 10.2); 32x64 gains up to 7 % by it there and loses 18 % in
    // larger launches, two of whose blocks fit a CU instead of four (16000 x 512 x 512 82 -> 97).
    struct Cost { Route route; int bm, bn; double once, step1, tile, step; };
    static const Cost costs[6] = {{kF32Ring32x64, 32, 64, 5.48, 0.706, 0.38, 0.548}, {kF32Ring32x32, 32, 32, 5.42, 0.608, 0.03, 0.356}, {kF32Ring32x32Deep, 32, 32, 5.27, 0.447, 0.27, 0.343},
                                  {kF32_32x32, 32, 32, 3.77, 0, 1.17, 0.445}, {kF32_32x16, 32, 16, 3.35, 0, 0.83, 0.337}, {kF32_16x16, 16, 16, 3.34, 0, 0.53, 0.226}};
    int best = -1;
    double best_t = 0;
    for (int c = 0; c < 6; ++c) {
      if (costs[c].route == (g.k % 256 == 0 ? kF32Ring32x32 : kF32Ring32x32Deep)) continue;
      const int64_t tiles = tiles_of(g, costs[c].bm, costs[c].bn);
      if (!grid_fits(tiles, 256)) continue;
      const double steps = (double)(g.k / 64), exact = (double)(tiles * g.batch) / 256, whole = (double)((tiles * g.batch + 255) / 256);
      const double rounds = costs[c].step1 > 0 && whole > 1 ? 0.5 * (exact + whole) : whole;       // (the ring's blocks share a CU)
      const double busy = rounds * steps * costs[c].step, one = steps * costs[c].step1, t = (busy > one ? busy : one) + rounds * costs[c].tile + costs[c].once;
      if (best < 0 || t < best_t) { best = c; best_t = t; }
    }
    return best < 0 ? kFma : costs[best].route;
  }
  // Other depths: the tile of least estimated time: rounds of 256 tiles x (k / 64 steps + prologue and epilogue), plus what is paid once, in us.  Within 4 % the
  // larger tile, which reads less per output (4000 x 2048 x 96: 40.5 us on 32x64, 50.0 on 32x32).  On 170 products of 1 to 20000 rows x 4 to 8192 columns x 36 to
  // 8192 deep, no depth a multiple of 128, the choice is 0.9 % off the best of the four on average and 27 % at worst (644 x 3808 x 5032, 403 us on
  // 32x64 and 318 on 32x32); by area alone a row past a multiple of the large tiles would send 777 x 512 x 500 to 16x16, 12.9 us, where 32x64 takes 10.3.
  struct Cost { int bm, bn; double step, tile, once; };
  static const Cost costs[4] = {{32, 64, 0.77, 1.9, 2.5}, {32, 32, 0.38, 0.9, 3.0}, {32, 16, 0.27, 0.5, 3.1}, {16, 16, 0.18, 0.25, 3.2}};
  int best = -1;
  double best_t = 0;
  for (int c = 0; c < 4; ++c) {
    const int64_t tiles = tiles_of(g, costs[c].bm, costs[c].bn);
    if (!grid_fits(tiles, 256)) continue;
    const double rounds = (double)((tiles * g.batch + 255) / 256);
    const double t = rounds * ((double)((g.k + 63) / 64) * costs[c].step + costs[c].tile) + costs[c].once;
    if (best < 0 || t < 0.96 * best_t) { best = c; best_t = t; }
  }
  return best < 0 ? kFma : (Route)(kF32_32x64 + best);
}

static Route linear_route(const LinearArgs& g) {
  if (g.conv_c > 0) {
    if (g.conv_c >= (1 << 20)) return kConvWide64x64;   // (192 weight rows of 9 * 2^20 channels are 3.6e9 bytes, the most that 32-bit offsets hold)
    switch (best_conv_tile(g)) {
      case k128x128Ring: return kConv128x128;
      case k128x192: return kConv128x192;
      case k128x64: return kConv128x64;
      default: return kConv64x64;
    }
  }
  if (mfma_eligible(g)) return bf16_route(g);
  if (g.dtype == AC_F32 && mfma_f32_eligible(g)) return f32_route(g);
  return kFma;
}

bool linear_takes_causal(const LinearArgs& g_in) {
  LinearArgs g = g_in;
  g.o_period = g.t_period = INT64_MAX;
  return g.dtype == AC_BF16 && linear_route(g) != kFma;
}

// A gated product: erf GELU, whole k tiles, no other epilogue operand, and its weight rows within 32-bit byte offsets of a tile.
bool linear_takes_gate(const LinearArgs& g_in) {
  LinearArgs g = g_in;
  g.o_period = g.t_period = INT64_MAX;
  return g.dtype == AC_BF16 && g.act == AC_ACT_GELU_ERF && g.k % kBK == 0 && g.n == g.gate && g.n_split == g.n && g.batch <= 1 && !g.mul && !g.resid && g.conv_c == 0 && g.bias_period == 0 &&
         !wide_rows(g) && (g.gate + 256) * g.ldw < (1ll << 30) && g.m <= 0x7fffffffLL && aligned_to(g.bias, 8) && mfma_eligible(g);
}

const char* linear_kernel_name(int64_t m, int64_t n, int64_t k, int64_t lda, int64_t ldw, int64_t batch, bool conv, int dtype) {
  LinearArgs g{};
  g.m = m; g.n = g.n_split = g.ldo = n; g.k = k; g.lda = lda; g.ldw = ldw; g.batch = batch; g.dtype = dtype; g.o_period = g.t_period = INT64_MAX;
  g.sa_b = m * lda; g.sw_b = n * ldw; g.so_b = m * n;
  if (conv) g.conv_c = (int)(k / 9);
  return kRouteName[linear_route(g)];
}

hipError_t launch_linear(const LinearArgs& g_in, hipStream_t s) {
  LinearArgs g = g_in;
  if (g.m <= 0 || g.n <= 0) return hipSuccess;
  if (g.k <= 0) return hipErrorInvalidValue;
  if (g.out_t == nullptr) g.n_split = g.n;
  if (g.n_split > g.n) g.n_split = g.n;
  if (g.t_period <= 0) g.t_period = INT64_MAX;
  if (g.o_period <= 0) g.o_period = INT64_MAX;
  if (g.batch < 1) g.batch = 1;
  if (g.batch > 1 && g.o_period != INT64_MAX) return hipErrorInvalidValue;
  if (g.batch > 1 && (g.bias || g.mul || g.resid || g.out_t || g.act != AC_ACT_NONE)) return hipErrorInvalidValue;
  if (g.batch > 65535 || g.m > 0x7fffffffLL) return hipErrorInvalidValue;
  if (g.conv_c > 0) {
    // 3x3 convolution as an implicit GEMM; bf16 images with channels in multiples of 64 only
    if (g.dtype != AC_BF16 || g.conv_c % kBK != 0 || g.conv_h < 1 || g.conv_w < 1 || g.k != 9 * (int64_t)g.conv_c ||
        g.m % ((int64_t)g.conv_h * g.conv_w) != 0 || g.batch != 1)
      return hipErrorInvalidValue;
    g.lda = g.conv_c;
    if (!mfma_eligible(g)) return hipErrorInvalidValue;
  }
  if (g.gate > 0) {
    if (!linear_takes_gate(g_in)) return hipErrorInvalidValue;
    switch (best_gated_tile(g)) {
      case kQuad: return quad_launch<true>(g, s);
      case k256x128: return ring_launch<256, 128, 4, 2, 64, 3, false, false, false, true>(g, s);
      default: return ring_launch<64, 128, 2, 2, 64, 3, false, false, false, true>(g, s);
    }
  }
  switch (linear_route(g)) {
    case kF32_32x64: return mfma_f32_launch<2, 4>(g, s);
    case kF32_32x32: return mfma_f32_launch<2, 2>(g, s);
    case kF32_32x16: return mfma_f32_launch<2, 1>(g, s);
    case kF32_16x16: return mfma_f32_launch<1, 1>(g, s);
    case kF32Ring32x64: return ring_f32_launch<32, 64, 1, 4, 32>(g, s);
    case kF32Ring32x32: return ring_f32_launch<32, 32, 2, 2, 32>(g, s);
    case kF32Ring32x32Deep: return ring_f32_launch<32, 32, 2, 2, 64>(g, s);
    case kRouteQuad: return quad_launch<false>(g, s);
    case kRing256x128: return ring_launch<256, 128, 4, 2, 64, 3>(g, s);
    case kRing128x128: return ring_launch<128, 128, 2, 4, 64, 3>(g, s);
    case kRing128x192: return ring_launch<128, 192, 4, 2, 64, 3>(g, s);
    case kStaged128x128: return mfma_launch<128, 128, 2, 2>(g, s);
    case kRing128x64: return ring_launch<128, 64, 2, 2, 64, 3>(g, s);
    case kRing64x64: return ring_launch<64, 64, 2, 2, 64, 3>(g, s);
    case kStaged64x64: return mfma_launch<64, 64, 2, 2>(g, s);
    case kStaged32x64: return mfma_launch<32, 64, 1, 2>(g, s);
    case kRagged256x128: return ring_launch<256, 128, 4, 2, 64, 3, false, true>(g, s);
    case kRagged64x64: return ring_launch<64, 64, 2, 2, 64, 3, false, true>(g, s);
    case kConv128x128: return ring_launch<128, 128, 2, 4, 64, 3, true>(g, s);
    case kConv128x192: return ring_launch<128, 192, 4, 2, 64, 3, true>(g, s);
    case kConv128x64: return ring_launch<128, 64, 2, 2, 64, 3, true>(g, s);
    case kConv64x64: return ring_launch<64, 64, 2, 2, 64, 3, true>(g, s);
    case kConvWide64x64: return ring_launch<64, 64, 2, 2, 64, 3, true, false, true>(g, s);
    default: break;
  }
  dim3 grid((unsigned)((g.n + 63) / 64), (unsigned)((g.m + 63) / 64), (unsigned)g.batch);
  if (g.dtype == AC_BF16) hipLaunchKernelGGL((linear_fma<bf16_t>), grid, dim3(256), 0, s, g);
  else hipLaunchKernelGGL((linear_fma<float>), grid, dim3(256), 0, s, g);
  return hipGetLastError();
}

}  // namespace ac
