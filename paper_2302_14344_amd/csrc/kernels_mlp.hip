// HIP kernels (gfx950) of the warm-start network: a perceptron with ReLU hidden layers
// and a linear output, BF16 operands on the matrix cores with FP32 accumulation, FP32
// master weights and Adam.
//
// Networks of at most kFusedLayers layers of at most kFusedWidth run in whole-network kernels:
// the forward pass (and inference) carries 32 rows of the batch through every layer in one
// launch, the backward pass carries the gradients back the same way in a second, forms every
// layer's weight gradient in a third and adds the partial sums in a fourth.  Wider networks
// go through one tiled GEMM per product, C[M x N] = opA[M x K] opB[K x N], whose operands are
// addressed through strides (so X W^T, dZ W and dZ^T X are the same kernel) and converted to
// BF16 while they are staged into LDS.  A 256-thread workgroup owns a 64 x 64 tile of C; each
// of its four waves owns 32 x 32 = 2 x 2 tiles of gfx950's 16x16x32 BF16 MFMA (one instruction
// per tile per 32-deep block of K), fed from LDS by one 16-byte read per operand and lane
// (tile rows padded to 80 bytes, which keeps those reads 16-byte aligned and spreads the rows
// over the banks).  Epilogues fuse the bias, the ReLU and the BF16 store of the next layer's
// input, or the ReLU mask of the backward pass.
#include <type_traits>

#include "mlp_internal.hpp"
#include "row_walk.hpp"

namespace subadmm {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even on the bit pattern (NaN kept quiet).
__device__ inline uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ inline float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

template <typename X>
__device__ inline uint16_t as_bf16(X v);
template <>
__device__ inline uint16_t as_bf16<float>(float v) { return to_bf16(v); }
template <>
__device__ inline uint16_t as_bf16<uint16_t>(uint16_t v) { return v; }

constexpr int kBM = 64, kBN = 64, kBK = 32, kPad = 8;

template <typename TA, typename TB>
__global__ void __launch_bounds__(256) gemm_bf16_kernel(GemmArgs<TA, TB> g) {
  __shared__ __align__(16) uint16_t As[kBM][kBK + kPad];
  __shared__ __align__(16) uint16_t Bt[kBN][kBK + kPad];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  const int wm = wv >> 1, wn = wv & 1;
  const long m0 = (long)blockIdx.y * kBM, n0 = (long)blockIdx.x * kBN;
  const long kb = (long)blockIdx.z * g.k_chunk;
  const long ke = kb + g.k_chunk < g.K ? kb + g.k_chunk : g.K;

  f32x4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

  for (long k0 = kb; k0 < ke; k0 += kBK) {
    // stage opA(m0.., k0..) and opB(k0.., n0..) as BF16; the faster-varying index of each
    // thread is the operand's unit-stride one, so global reads coalesce
#pragma unroll
    for (int q = 0; q < (kBM * kBK) / 256; ++q) {
      const int e = tid + 256 * q;
      int m, k;
      if (g.a_m_fast) { m = e % kBM; k = e / kBM; } else { k = e % kBK; m = e / kBK; }
      const long gm = m0 + m, gk = k0 + k;
      uint16_t v = 0;
      if (gm < g.M && gk < ke) v = as_bf16<TA>(g.A[gm * g.sam + gk * g.sak]);
      As[m][k] = v;
    }
#pragma unroll
    for (int q = 0; q < (kBN * kBK) / 256; ++q) {
      const int e = tid + 256 * q;
      int n, k;
      if (g.b_n_fast) { n = e % kBN; k = e / kBN; } else { k = e % kBK; n = e / kBK; }
      const long gn = n0 + n, gk = k0 + k;
      uint16_t v = 0;
      if (gn < g.N && gk < ke) v = as_bf16<TB>(g.B[gk * g.sbk + gn * g.sbn]);
      Bt[n][k] = v;
    }
    __syncthreads();
    // lane l supplies row l % 16 of A's tile and column l % 16 of B's with the eight k of
    // group l / 16; A and B take the same k assignment, so each product is a 32-deep sum
    static_assert(kBK % 32 == 0 && ((kBK + kPad) * 2) % 16 == 0, "16-byte fragment reads");
#pragma unroll
    for (int kk = 0; kk < kBK; kk += 32) {
      bf16x8_t af[2], bfr[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint16_t* pa = &As[32 * wm + 16 * i + (lane & 15)][kk + 8 * (lane >> 4)];
        af[i] = *reinterpret_cast<const bf16x8_t*>(pa);
        const uint16_t* pb = &Bt[32 * wn + 16 * i + (lane & 15)][kk + 8 * (lane >> 4)];
        bfr[i] = *reinterpret_cast<const bf16x8_t*>(pb);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }

  // epilogue: lane holds rows 4*(lane/16) + r, column lane % 16 of each 16 x 16 tile
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const long m = m0 + 32 * wm + 16 * i + 4 * (lane >> 4) + r;
        const long n = n0 + 32 * wn + 16 * j + (lane & 15);
        if (m >= g.M || n >= g.N) continue;
        float v = acc[i][j][r];
        switch (g.epi) {
          case EPI_STORE:
            g.C[(long)blockIdx.z * g.c_split + m * g.ldc + n] = v;
            break;
          case EPI_BIAS_F32:
            g.C[m * g.ldc + n] = v + g.bias[n];
            break;
          case EPI_BIAS_RELU_BF16: {
            v += g.bias[n];
            g.out_bf16[m * g.ldo + n] = to_bf16(v > 0.f ? v : 0.f);
            break;
          }
          case EPI_RELU_MASK: {
            const uint16_t a = g.mask[m * g.ldm + n];  // the ReLU output of the forward pass
            g.C[m * g.ldc + n] = (a != 0 && (a & 0x8000u) == 0) ? v : 0.f;
            break;
          }
        }
      }
}

template <typename TA, typename TB>
hipError_t launch_gemm(const GemmArgs<TA, TB>& g, int splits, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  dim3 grid((unsigned)((g.N + kBN - 1) / kBN), (unsigned)((g.M + kBM - 1) / kBM), (unsigned)splits);
  hipLaunchKernelGGL((gemm_bf16_kernel<TA, TB>), grid, dim3(256), 0, s, g);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Whole-network forward pass: 32 rows of the batch per workgroup of eight waves, the hidden
// activations in LDS (two 32 x 264 BF16 buffers), wave w owning columns 32 w .. 32 w + 31 of
// every layer.  Per 32-deep k block a wave issues four 16x16x32 BF16 MFMAs from two LDS reads
// (activations) and two fragments of weights, which come straight from L2 into registers: a
// layer's whole share (8 k blocks x 2 column tiles) sits in 64 registers, and as a k block is
// consumed its registers are refilled with the next layer's, so the loads are in flight over
// the epilogue and the barrier.  The k blocks, the instruction, the bias, the ReLU and the
// BF16 rounding are those of gemm_bf16_kernel in the same order (same bits per row).
//
// Bound by L2 reads of the weights (270 KB per workgroup for 27-256-256-256-15, ~64 bytes per
// clock and CU) and the latency of the dependent layers.  Measured for that network: inference
// of 15,393 rows 47 us (64 rows per workgroup of four waves, weights loaded where used) -> 18 us
// a pass; 30 us with the weights in plain rows and one workgroup per CU.  The forward pass of
// 8,192 rows takes one launch of 19 us where four GEMMs, a cast and a copy took ~100 us.
// ------------------------------------------------------------------------------------
constexpr int kFusedLd = kFusedWidth + 8;  // 528-byte rows: 16-byte aligned fragment reads
constexpr int kFusedThreads = 512;
constexpr unsigned kFusedResident = 512;  // workgroups of that size the device holds at once (two a CU)
constexpr int kKBlocks = kFusedWidth / 32;

__device__ inline bf16x8_t load8(const uint16_t* p) { return *reinterpret_cast<const bf16x8_t*>(p); }

// This lane's fragment of operand tile (nt, s) of a matrix of K columns; zero beyond the matrix
// (nt, s and the sizes are the same for the whole wave).
__device__ inline bf16x8_t frag(const uint16_t* W, int nt, int N, int s, int K, int lane) {
  if (16 * nt < N && 32 * s < K) return load8(W + ((long)nt * ((K + 31) >> 5) + s) * 512 + 8 * lane);
  const uint4 z = make_uint4(0u, 0u, 0u, 0u);
  return __builtin_bit_cast(bf16x8_t, z);
}

// rows 0..31 of buf (width entries, zero padded) to rows r0.. of dst (ld entries per row)
template <int kThreads>
__device__ inline void store_rows(const uint16_t (*buf)[kFusedLd], uint16_t* dst, long r0, long rows, int width) {
  const int ld = mlp_ld(width), nv = ld >> 3;
  for (int q = threadIdx.x; q < kFusedRows * nv; q += kThreads) {
    const int r = q / nv, c = (q - r * nv) << 3;
    if (r0 + r < rows) *reinterpret_cast<uint4*>(dst + (r0 + r) * ld + c) = *reinterpret_cast<const uint4*>(&buf[r][c]);
  }
}

template <bool kKeep, int kThreads>
__global__ void __launch_bounds__(kThreads, 4) mlp_forward_kernel(MlpFusedArgs a) {
  __shared__ __align__(16) uint16_t buf[2][kFusedRows][kFusedLd];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid) >> 6;
  const int g = lane >> 4, cl = lane & 15;
  const long r0 = (long)blockIdx.x * kFusedRows;
  bf16x8_t wr[kKBlocks][2];
  float bn[2];
  auto fetch = [&](int l, int s) {
    const int K = a.net.w[l], N = a.net.w[l + 1];
#pragma unroll
    for (int j = 0; j < 2; ++j)
      wr[s][j] = frag(a.Wbf + a.net.off_Wbf[l], 2 * wv + j, N, s, K, lane);
  };
  auto fetch_bias = [&](int l) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = 32 * wv + 16 * j + cl;
      bn[j] = n < a.net.w[l + 1] ? a.P[a.net.off_b[l] + n] : 0.f;
    }
  };
#pragma unroll
  for (int s = 0; s < kKBlocks; ++s) fetch(0, s);
  fetch_bias(0);
  {
    // input rows, zero beyond the width up to the next multiple of 32 and beyond the batch
    const int w0 = a.net.w[0], kp = (w0 + 31) / 32 * 32;
    for (int q = tid; q < kFusedRows * kp; q += kThreads) {
      const int r = q / kp, c = q - r * kp;
      uint16_t v = 0;
      if (r0 + r < a.batch && c < w0) {
        const float xv = a.x[(r0 + r) * w0 + c];
        v = a.scale ? to_bf16(xv * a.scale[c] + a.shift[c]) : to_bf16(xv);
      }
      buf[0][r][c] = v;
    }
  }
  __syncthreads();
  if (kKeep) store_rows<kThreads>(buf[0], a.act + a.net.off_act[0], r0, a.batch, a.net.w[0]);
  int cur = 0;
  for (int l = 0; l < a.net.L; ++l) {
    const int K = a.net.w[l], N = a.net.w[l + 1];
    const bool last = l + 1 == a.net.L;
    f32x4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kKBlocks; ++s) {
      if (32 * s < K && 32 * wv < N) {
        bf16x8_t af[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) af[i] = load8(&buf[cur][16 * i + cl][32 * s + 8 * g]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], wr[s][j], acc[i][j], 0, 0, 0);
      }
      if (!last) fetch(l + 1, s);
    }
    const int nxt = cur ^ 1;
    const int np = (N + 31) / 32 * 32;
    // lane holds rows 4 g + r, column cl of each 16 x 16 tile
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = 32 * wv + 16 * j + cl;
      if (n >= np) continue;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * i + 4 * g + r;
          const float v = acc[i][j][r] + bn[j];
          if (last) {
            if (n < N && r0 + row < a.batch) {
              a.y[(r0 + row) * N + n] = v;
              if (a.y2) a.y2[(r0 + row) * N + n] = v;
            }
          } else {
            buf[nxt][row][n] = n < N ? to_bf16(v > 0.f ? v : 0.f) : (uint16_t)0;
          }
        }
    }
    if (last) break;
    fetch_bias(l + 1);
    __syncthreads();
    cur = nxt;
    if (kKeep) store_rows<kThreads>(buf[cur], a.act + a.net.off_act[l + 1], r0, a.batch, N);
  }
}

hipError_t launch_fused_forward(const MlpFusedArgs& a, hipStream_t s) {
  if (a.batch <= 0) return hipSuccess;
  const dim3 grid((unsigned)((a.batch + kFusedRows - 1) / kFusedRows));
  const auto go = [&](auto threads) -> hipError_t {
    constexpr int T = decltype(threads)::value;
    if (a.act)
      hipLaunchKernelGGL((mlp_forward_kernel<true, T>), grid, dim3(T), 0, s, a);
    else
      hipLaunchKernelGGL((mlp_forward_kernel<false, T>), grid, dim3(T), 0, s, a);
    return hipGetLastError();
  };
  // A wave owns 32 columns, so narrow layers leave most of eight waves without products; with no more
  // waves than the widest layer needs twice as many workgroups are resident (four, by LDS).  While the
  // grid fits the device at once, and in a single layer, the idle waves help with the rows instead.
  // Inference of 65,536 rows: 12-64-64-6 36.8 us with eight waves and 28.7 with two, 12-100-100-6
  // 37.8 and 24.0 with four; 40-9 17.8 with eight and 20.3 with two.
  int w = 0;
  for (int k = 1; k <= a.net.L; ++k) w = a.net.w[k] > w ? a.net.w[k] : w;
  const bool fewer = grid.x > kFusedResident && a.net.L > 1;
  if (fewer && w <= 64) return go(std::integral_constant<int, 128>{});
  if (fewer && w <= 128) return go(std::integral_constant<int, 256>{});
  return go(std::integral_constant<int, kFusedThreads>{});
}

// ------------------------------------------------------------------------------------
// Backward pass, first launch: the loss, the output gradient dz_L = wt (y - target) and the
// chain dz_k = (dz_{k+1} W_k) masked by the ReLU, 32 rows per workgroup as in the forward
// pass with the transposed weights as operand.  dz_k is stored in FP32 (the bias gradients sum
// it); each product rounds it to BF16 as it takes it as an operand.  30 us for 8,192 rows of
// 27-256-256-256-15 (three GEMMs of 56 us, a loss gradient and a serial loss sum of 23 us before).
// ------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kFusedThreads) mlp_chain_kernel(MlpBackArgs a) {
  __shared__ __align__(16) uint16_t buf[2][kFusedRows][kFusedLd];
  __shared__ double lred[kFusedThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid) >> 6;
  const int g = lane >> 4, cl = lane & 15;
  const int L = a.net.L, NL = a.net.w[L];
  double lsum = 0.0;
  bf16x8_t wr[kKBlocks][2];
  // operand rows of layer k (k = L - 1 .. 1): column n of the result is row n of W_k^T
  auto fetch = [&](int k, int s) {
    const int K = a.net.w[k + 1], N = a.net.w[k];
#pragma unroll
    for (int j = 0; j < 2; ++j)
      wr[s][j] = frag(a.WT + a.net.off_WT[k], 2 * wv + j, N, s, K, lane);
  };
  // threads per column of the output gradient: groups of rows
  int pc = 1;
  while (pc < NL) pc <<= 1;
  const int c = tid & (pc - 1), rg = tid / pc, ng = kFusedThreads / pc;
  const int npl = (NL + 31) / 32 * 32;
  for (long r0 = (long)blockIdx.x * kFusedRows; r0 < a.batch; r0 += (long)gridDim.x * kFusedRows) {
    if (L > 1) {
#pragma unroll
      for (int s = 0; s < kKBlocks; ++s) fetch(L - 1, s);
    }
    __syncthreads();
    for (int q = tid; q < kFusedRows * (npl - NL); q += kFusedThreads) buf[0][q / (npl - NL)][NL + q % (npl - NL)] = 0;
    for (int r = rg; c < NL && r < kFusedRows; r += ng) {
      float d = 0.f;
      if (r0 + r < a.batch) {
        const long e = (r0 + r) * NL + c;
        const float res = a.y[e] - a.target[e];
        const float w = a.wt ? a.wt[e] : 1.f;
        d = w * res;
        lsum += 0.5 * (double)w * (double)res * (double)res;
        a.dz[a.net.off_dz[L] + (r0 + r) * mlp_ld(NL) + c] = d;
      }
      buf[0][r][c] = to_bf16(d);
    }
    __syncthreads();
    int cur = 0;
    for (int k = L - 1; k >= 1; --k) {
      const int K = a.net.w[k + 1], N = a.net.w[k], np = (N + 31) / 32 * 32, ld = mlp_ld(N);
      // the ReLU outputs of the forward pass at this lane's results (used after the products)
      uint16_t mk[2][2][4];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int n = 32 * wv + 16 * j + cl;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const long row = r0 + 16 * i + 4 * g + r;
            mk[i][j][r] = n < N && row < a.batch ? a.act[a.net.off_act[k] + row * ld + n] : (uint16_t)0;
          }
      }
      f32x4_t acc[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < kKBlocks; ++s) {
        if (32 * s < K && 32 * wv < N) {
          bf16x8_t af[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) af[i] = load8(&buf[cur][16 * i + cl][32 * s + 8 * g]);
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], wr[s][j], acc[i][j], 0, 0, 0);
        }
        if (k > 1) fetch(k - 1, s);
      }
      const int nxt = cur ^ 1;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int n = 32 * wv + 16 * j + cl;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint16_t m = mk[i][j][r];
            const float v = (m != 0 && (m & 0x8000u) == 0) ? acc[i][j][r] : 0.f;
            const long row = r0 + 16 * i + 4 * g + r;
            if (n < N && row < a.batch) a.dz[a.net.off_dz[k] + row * ld + n] = v;
            if (n < np) buf[nxt][16 * i + 4 * g + r][n] = to_bf16(v);
          }
      }
      __syncthreads();
      cur = nxt;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, 64);
  if (lane == 0) lred[wv] = lsum;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int q = 0; q < kFusedThreads / 64; ++q) t += lred[q];
    a.lpart[blockIdx.x] = t;
  }
}

// Second launch: the weight gradients dW_k = dz_{k+1}^T act_k of every layer, one 64 x 64 tile
// of one layer over one chunk of the batch per workgroup (four waves, 2 x 2 MFMA tiles each),
// and the partial column sums of every dz (the bias gradients).  Both operands of a weight
// gradient have the batch as the product's k index, so a thread reads 8 rows x 4 columns of
// each, transposes them in registers and stores 16-byte fragments to LDS.  Chunks, k blocks and
// sums are those of the per-product path (gemm_bf16_kernel, colsum_partial_kernel), so the
// gradients are the same bits.  24 us at 8,192 rows (29 without loading a stage ahead) where
// four GEMMs of ~56 us with two-byte strided staging and eight sums took ~350 us.  A training
// step (forward, backward, Adam) 640 -> 79 us.
constexpr int kWtDepth = 128;              // batch rows per stage
constexpr int kWtLd = kWtDepth + 8;        // 272-byte rows

// Four entries of a row as they lie in memory, and as BF16 packed in pairs.
__device__ inline uint2 raw4(const uint16_t* p) { return *reinterpret_cast<const uint2*>(p); }
__device__ inline float4 raw4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ inline uint2 pack4(uint2 v) { return v; }
__device__ inline uint2 pack4(float4 f) {
  return make_uint2((uint32_t)to_bf16(f.x) | ((uint32_t)to_bf16(f.y) << 16),
                    (uint32_t)to_bf16(f.z) | ((uint32_t)to_bf16(f.w) << 16));
}

// One operand's stage: a thread's 8 rows x 4 columns of src (rows of mlp_ld(width) entries),
// loaded ahead of the stage and stored transposed, dst[c][m] = src[row0 + m][c0 + c], zero
// beyond `rows` and beyond the width (what pads the rows is not read as a value).
template <typename X>
struct Stage {
  decltype(raw4((const X*)nullptr)) v[8];
  __device__ void load(const X* src, long row0, long rows, int width, int c0) {
    const int c = c0 + 4 * (threadIdx.x & 15), mg = threadIdx.x >> 4, ld = mlp_ld(width);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const long row = row0 + 8 * mg + r;
      v[r] = {};
      if (row < rows && c < ld) v[r] = raw4(src + row * ld + c);
    }
  }
  __device__ void store(uint16_t (*dst)[kWtLd], int width, int c0) const {
    const int cq = threadIdx.x & 15, mg = threadIdx.x >> 4;
    uint2 w[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) w[r] = pack4(v[r]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t o[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const uint32_t e0 = q < 2 ? w[2 * h].x : w[2 * h].y, e1 = q < 2 ? w[2 * h + 1].x : w[2 * h + 1].y;
        o[h] = (q & 1) ? (e0 >> 16) | (e1 & 0xffff0000u) : (e0 & 0xffffu) | (e1 << 16);
      }
      if (c0 + 4 * cq + q >= width) o[0] = o[1] = o[2] = o[3] = 0;
      *reinterpret_cast<uint4*>(&dst[4 * cq + q][8 * mg]) = make_uint4(o[0], o[1], o[2], o[3]);
    }
  }
};

__global__ void __launch_bounds__(256) mlp_weight_grad_kernel(MlpBackArgs a) {
  __shared__ __align__(16) uint16_t As[64][kWtLd];
  __shared__ __align__(16) uint16_t Bs[64][kWtLd];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if ((int)blockIdx.x >= a.tiles * a.splits) {
    // column sums: 64 columns of one layer's dz over one chunk of rows, four row groups
    int t = (int)blockIdx.x - a.tiles * a.splits, k = 0, boff = 0;
    for (;; ++k) {
      const int nb = (a.net.w[k + 1] + 63) / 64 * kBiasSplits;
      if (t < nb) break;
      t -= nb;
      boff += a.net.w[k + 1];
    }
    const int N = a.net.w[k + 1], ld = mlp_ld(N), c = (t / kBiasSplits) * 64 + lane, q = t % kBiasSplits;
    const long per = (a.batch + kBiasSplits - 1) / kBiasSplits;
    const long r0 = (long)q * per, r1 = r0 + per < a.batch ? r0 + per : a.batch;
    const float* dz = a.dz + a.net.off_dz[k + 1];
    float (*red)[64] = reinterpret_cast<float(*)[64]>(&As[0][0]);
    float s = 0.f;
    if (c < N) {
#pragma unroll 8
      for (long r = r0 + wv; r < r1; r += 4) s += dz[r * ld + c];
    }
    red[wv][lane] = s;
    __syncthreads();
    if (wv == 0 && c < N)
      a.cpart[(long)q * a.n_bias + boff + c] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    return;
  }
  // the tile: layers one after another
  int t = (int)blockIdx.x % a.tiles, k = 0, tn = 0, tk = 0;
  const int split = (int)blockIdx.x / a.tiles;
  for (;; ++k) {
    tn = (a.net.w[k + 1] + 63) / 64;
    tk = (a.net.w[k] + 63) / 64;
    if (t < tn * tk) break;
    t -= tn * tk;
  }
  const int N = a.net.w[k + 1], K = a.net.w[k];
  const int n0 = (t / tk) * 64, k0 = (t % tk) * 64;
  const long m0 = (long)split * a.chunk, m1 = m0 + a.chunk < a.batch ? m0 + a.chunk : a.batch;
  const float* dz = a.dz + a.net.off_dz[k + 1];
  const uint16_t* act = a.act + a.net.off_act[k];
  const int wm = wv >> 1, wn = wv & 1, g = lane >> 4, cl = lane & 15;
  f32x4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  Stage<float> sa;
  Stage<uint16_t> sb;
  sa.load(dz, m0, m1, N, n0);
  sb.load(act, m0, m1, K, k0);
  for (long m = m0; m < m1; m += kWtDepth) {
    sa.store(As, N, n0);
    sb.store(Bs, K, k0);
    __syncthreads();
    if (m + kWtDepth < m1) {
      sa.load(dz, m + kWtDepth, m1, N, n0);
      sb.load(act, m + kWtDepth, m1, K, k0);
    }
#pragma unroll
    for (int kk = 0; kk < kWtDepth; kk += 32) {
      bf16x8_t af[2], bf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = load8(&As[32 * wm + 16 * i + cl][kk + 8 * g]);
        bf[i] = load8(&Bs[32 * wn + 16 * i + cl][kk + 8 * g]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  float* out = a.part + (long)split * a.n_params + a.net.off_W[k];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int n = n0 + 32 * wm + 16 * i + 4 * g + r, kc = k0 + 32 * wn + 16 * j + cl;
        if (n < N && kc < K) out[(long)n * K + kc] = acc[i][j][r];
      }
}

// Third launch: the gradient from the partial sums, one thread per parameter and in order, and
// the loss.
__global__ void __launch_bounds__(256) mlp_reduce_kernel(MlpBackArgs a, int param_blocks) {
  __shared__ double lred[256];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < param_blocks) {
    const long i = (long)blockIdx.x * 256 + tid;
    if (i >= a.n_params) return;
    const float* p = a.part + i;
    long stride = a.n_params;
    int n = a.splits;
    for (int k = 0, boff = 0; k < a.net.L; boff += a.net.w[++k]) {
      if (i >= a.net.off_b[k] && i < a.net.off_b[k] + a.net.w[k + 1]) {
        p = a.cpart + boff + (i - a.net.off_b[k]);
        stride = a.n_bias;
        n = kBiasSplits;
      }
    }
    float s = 0.f;
#pragma unroll 16
    for (int q = 0; q < n; ++q) s += p[(long)q * stride];
    a.grad[i] = s;
    if (a.grad2) a.grad2[i] = s;
    return;
  }
  double s = 0.0;
  for (int q = tid; q < a.chain_blocks; q += 256) s += a.lpart[q];
  lred[tid] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) lred[tid] += lred[tid + h];
    __syncthreads();
  }
  if (tid == 0 && a.loss) *a.loss = (float)lred[0];
}

hipError_t launch_fused_backward(MlpBackArgs a, hipStream_t s) {
  if (a.batch <= 0) return hipSuccess;
  const long rows = (a.batch + kFusedRows - 1) / kFusedRows;
  a.chain_blocks = (int)(rows < kChainBlocks ? rows : kChainBlocks);
  const long per = (a.batch + kWeightSplits - 1) / kWeightSplits;
  a.chunk = (int)((per + 31) / 32 * 32);
  a.splits = (int)((a.batch + a.chunk - 1) / a.chunk);
  a.tiles = 0;
  int sums = 0;
  for (int k = 0; k < a.net.L; ++k) {
    a.tiles += ((a.net.w[k + 1] + 63) / 64) * ((a.net.w[k] + 63) / 64);
    sums += (a.net.w[k + 1] + 63) / 64 * kBiasSplits;
  }
  hipLaunchKernelGGL(mlp_chain_kernel, dim3(a.chain_blocks), dim3(kFusedThreads), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mlp_weight_grad_kernel, dim3(a.tiles * a.splits + sums), dim3(256), 0, s, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int pb = (int)((a.n_params + 255) / 256);
  hipLaunchKernelGGL(mlp_reduce_kernel, dim3(pb + 1), dim3(256), 0, s, a, pb);
  return hipGetLastError();
}

// Minibatch gather: dst row r = src row idx[r] (FP32 rows of `width` entries); a row whose
// index lies outside [0, n_rows) is filled with NaN.
__global__ void gather_rows_kernel(const float* src, long n_rows, int width, const int32_t* idx, int count,
                                   float* dst) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= (long)count * width) return;
  const long r = k / width;
  const int c = (int)(k - r * width);
  const int32_t i = idx[r];
  dst[k] = (i >= 0 && i < n_rows) ? src[(long)i * width + c] : __builtin_nanf("");
}

hipError_t launch_gather_rows(const float* src, long n_rows, int width, const int32_t* idx, int count, float* dst,
                              hipStream_t s) {
  const long n = (long)count * width;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, n_rows, width, idx,
                     count, dst);
  return hipGetLastError();
}

template hipError_t launch_gemm<float, uint16_t>(const GemmArgs<float, uint16_t>&, int, hipStream_t);
template hipError_t launch_gemm<uint16_t, uint16_t>(const GemmArgs<uint16_t, uint16_t>&, int, hipStream_t);
template hipError_t launch_gemm<float, float>(const GemmArgs<float, float>&, int, hipStream_t);

// ------------------------------------------------------------------------------------
// Element-wise kernels
// ------------------------------------------------------------------------------------
// Network input in BF16: y = bf16(x * scale + shift) per column, formed in FP32 (bf16(x) without
// an affine map); y rows of ldy entries.
__global__ void cast_rows_kernel(const float* x, const float* scale, const float* shift, long rows, int width,
                                 uint16_t* y, int ldy) {
  // row and column by carry: a 64-bit division per entry cost 2% of a 300-256-7 network's pass
  const long n = rows * width, step = (long)gridDim.x * blockDim.x;
  RowWalk at((int)(blockIdx.x * blockDim.x + threadIdx.x), (int)step, width);
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step, at.next()) {
    const int c = at.col;
    y[(long)at.row * ldy + c] = scale ? to_bf16(x[i] * scale[c] + shift[c]) : to_bf16(x[i]);
  }
}

// dY = wt * (y - target); per-block partial sums of 0.5 wt (y - target)^2 in FP64.
__global__ void __launch_bounds__(256) loss_grad_kernel(const float* y, const float* t, const float* wt, float* dy,
                                                         long n, double* partial) {
  __shared__ double red[256];
  double acc = 0.0;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const float r = y[i] - t[i];
    const float w = wt ? wt[i] : 1.f;
    dy[i] = w * r;
    acc += 0.5 * (double)w * (double)r * (double)r;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void loss_sum_kernel(const double* partial, int n, float* loss) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += partial[i];
    *loss = (float)s;
  }
}

// Column sums of a rows x cols FP32 matrix in two fixed-order stages (bias gradients).
__global__ void __launch_bounds__(256) colsum_partial_kernel(const float* a, long rows, int cols, long rows_per,
                                                              float* partial) {
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int g = threadIdx.x >> 6;  // 4 row groups
  __shared__ float red[4][64];
  const long r0 = (long)blockIdx.y * rows_per;
  const long r1 = r0 + rows_per < rows ? r0 + rows_per : rows;
  float s = 0.f;
  if (c < cols)
    for (long r = r0 + g; r < r1; r += 4) s += a[r * cols + c];
  red[g][threadIdx.x & 63] = s;
  __syncthreads();
  if (g == 0 && c < cols) {
    const float t = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
    partial[(long)blockIdx.y * cols + c] = t;
  }
}

// out[i] = sum over s of partial[s * n + i] (fixed order)
__global__ void sum_partials_kernel(const float* partial, int splits, long n, float* out) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    float s = 0.f;
    for (int q = 0; q < splits; ++q) s += partial[(long)q * n + i];
    out[i] = s;
  }
}

// Adam on the FP32 master parameters (g set), and the weights' BF16 copies in both orientations
// (the backward pass reads them transposed), one thread per parameter.
__global__ void update_kernel(MlpNet net, AdamArgs a) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += (long)gridDim.x * blockDim.x) {
    float p = a.p[i];
    if (a.g) {
      const float g = a.g[i];
      const float mi = a.b1 * a.m[i] + (1.f - a.b1) * g;
      const float vi = a.b2 * a.v[i] + (1.f - a.b2) * g * g;
      a.m[i] = mi;
      a.v[i] = vi;
      p -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
      a.p[i] = p;
    }
    int k = 0;
    while (k + 1 < net.L && i >= net.off_W[k + 1]) ++k;
    const long o = i - net.off_W[k];
    const int K = net.w[k], N = net.w[k + 1];
    if (o >= (long)N * K) continue;  // a bias
    const int n = (int)(o / K), c = (int)(o - (long)n * K);
    const uint16_t h = to_bf16(p);
    if (net.tiled) {
      a.Wbf[net.off_Wbf[k] + mlp_tile_at(n, c, K)] = h;
      a.WT[net.off_WT[k] + mlp_tile_at(c, n, N)] = h;
    } else {
      a.Wbf[net.off_Wbf[k] + (long)n * mlp_ld(K) + c] = h;
    }
  }
}

hipError_t launch_cast_rows(const float* x, const float* scale, const float* shift, long rows, int width, uint16_t* y,
                            int ldy, hipStream_t s) {
  const long n = rows * width;
  if (n <= 0) return hipSuccess;
  const long blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
  hipLaunchKernelGGL(cast_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, x, scale, shift, rows, width, y, ldy);
  return hipGetLastError();
}

hipError_t launch_loss_grad(const float* y, const float* t, const float* wt, float* dy, long n, double* partial,
                            int max_blocks, float* loss, hipStream_t s) {
  long blocks = (n + 255) / 256;
  if (blocks > max_blocks) blocks = max_blocks;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(loss_grad_kernel, dim3((unsigned)blocks), dim3(256), 0, s, y, t, wt, dy, n, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !loss) return e;
  hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(64), 0, s, partial, (int)blocks, loss);
  return hipGetLastError();
}

hipError_t launch_colsum(const float* a, long rows, int cols, float* partial, int splits, float* out, hipStream_t s) {
  const long rows_per = (rows + splits - 1) / splits;
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((unsigned)((cols + 63) / 64), (unsigned)splits), dim3(256), 0, s, a,
                     rows, cols, rows_per, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((cols + 255) / 256)), dim3(256), 0, s, partial, splits,
                     (long)cols, out);
  return hipGetLastError();
}

hipError_t launch_sum_partials(const float* partial, int splits, long n, float* out, hipStream_t s) {
  const long blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
  hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)blocks), dim3(256), 0, s, partial, splits, n, out);
  return hipGetLastError();
}

hipError_t launch_update(const MlpNet& net, const AdamArgs& a, hipStream_t s) {
  const long blocks = (a.n + 255) / 256 < 4096 ? (a.n + 255) / 256 : 4096;
  hipLaunchKernelGGL(update_kernel, dim3((unsigned)blocks), dim3(256), 0, s, net, a);
  return hipGetLastError();
}

}  // namespace subadmm
