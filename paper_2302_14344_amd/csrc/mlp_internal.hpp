// Internal declarations of the warm-start network kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace subadmm {

enum : int { EPI_STORE = 0, EPI_BIAS_F32 = 1, EPI_BIAS_RELU_BF16 = 2, EPI_RELU_MASK = 3 };

// C[M x N] = opA[M x K] opB[K x N]; opA(m, k) = A[m * sam + k * sak],
// opB(k, n) = B[k * sbk + n * sbn].  BF16 storage is passed as uint16_t bit patterns.
template <typename TA, typename TB>
struct GemmArgs {
  const TA* A;
  long sam, sak;
  const TB* B;
  long sbk, sbn;
  long M, N, K;
  long k_chunk;        // K range of one split (multiple of the K tile)
  int a_m_fast;        // 1 if sam == 1 (stage A with m as the fast index)
  int b_n_fast;        // 1 if sbn == 1
  int epi;             // EPI_*
  float* C;
  long ldc;
  long c_split;        // offset between the partial results of successive splits
  const float* bias;
  uint16_t* out_bf16;
  long ldo;
  const uint16_t* mask;
  long ldm;
};

template <typename TA, typename TB>
hipError_t launch_gemm(const GemmArgs<TA, TB>& g, int splits, hipStream_t s);
// y[r][c] = bf16(x[r][c] * scale[c] + shift[c]) (or bf16(x) without scale), x dense rows of
// `width`, y rows of ldy entries
hipError_t launch_cast_rows(const float* x, const float* scale, const float* shift, long rows, int width, uint16_t* y,
                            int ldy, hipStream_t s);
hipError_t launch_gather_rows(const float* src, long n_rows, int width, const int32_t* idx, int count, float* dst,
                              hipStream_t s);
hipError_t launch_loss_grad(const float* y, const float* t, const float* wt, float* dy, long n, double* partial,
                            int max_blocks, float* loss, hipStream_t s);
hipError_t launch_colsum(const float* a, long rows, int cols, float* partial, int splits, float* out, hipStream_t s);
hipError_t launch_sum_partials(const float* partial, int splits, long n, float* out, hipStream_t s);
// Rows of BF16 matrices (activations, their gradients) are padded with zeros to a multiple of
// eight entries, so every 16-byte load of eight is aligned.
inline __host__ __device__ int mlp_ld(int w) { return (w + 7) & ~7; }
// BF16 copies of the weights.  Wide networks: rows of mlp_ld entries.  Networks in the
// whole-network kernels: 16 x 32 tiles in the order a wave's lanes read them as an MFMA
// operand, so that a fragment is one contiguous kilobyte: entry (n, k) of a matrix of K columns
// sits in tile (n / 16, k / 32) at lane 16 ((k / 8) % 4) + n % 16, entry k % 8, zero padded.
inline __host__ __device__ long mlp_tiles(int N, int K) { return (long)((N + 15) / 16) * ((K + 31) / 32); }
inline __host__ __device__ long mlp_tile_at(int n, int k, int K) {
  const long tile = (long)(n >> 4) * ((K + 31) / 32) + (k >> 5);
  return tile * 512 + 8 * (16 * ((k >> 3) & 3) + (n & 15)) + (k & 7);
}

// Layer table of a network (all kernels below).
constexpr int kMaxLayers = 16;
struct MlpNet {
  int L;
  int w[kMaxLayers + 1];
  long off_W[kMaxLayers], off_b[kMaxLayers];    // FP32 parameter layout
  long off_Wbf[kMaxLayers], off_WT[kMaxLayers]; // BF16 copies (w[k+1] x w[k]), and transposed
  int tiled;                                    // layout of the BF16 copies (WT: tiled only)
  long off_act[kMaxLayers + 1];                 // rows of ld(w[k]): the input of layer k
  long off_dz[kMaxLayers + 1];                  // k >= 1: gradient at the output of layer k - 1
};

// BF16 copies of the FP32 parameters P (both orientations); with g: one Adam step on P first.
struct AdamArgs {
  float *p, *m, *v;
  const float* g;  // nullptr: only the copies
  uint16_t *Wbf, *WT;
  long n;
  float lr, b1, b2, eps, c1, c2;
};
hipError_t launch_update(const MlpNet& net, const AdamArgs& a, hipStream_t s);

// Whole-network kernels, for networks of at most kFusedLayers layers of at most kFusedWidth.
constexpr int kFusedLayers = 8, kFusedWidth = 256;
constexpr int kFusedRows = 32;          // batch rows of a workgroup at a time
constexpr int kChainBlocks = 1024;      // most workgroups of the gradient chain
constexpr int kWeightSplits = 16;       // batch splits of the weight gradients at most
constexpr int kBiasSplits = 64;         // row chunks of the bias gradients
struct MlpFusedArgs {
  MlpNet net;
  const float* x;        // batch x w[0]
  const float* scale;    // input affine (nullptr: none)
  const float* shift;
  const float* P;
  const uint16_t* Wbf;
  float *y, *y2;         // batch x w[L]; y2: second copy (nullptr: none)
  uint16_t* act;         // nullptr: activations are not kept
  long batch;
};
hipError_t launch_fused_forward(const MlpFusedArgs& a, hipStream_t s);

struct MlpBackArgs {
  MlpNet net;
  const float *y, *target, *wt;  // wt may be nullptr
  const uint16_t *act, *WT;
  float* dz;
  float* part;           // kWeightSplits x n_params: partial weight gradients
  float* cpart;          // kBiasSplits x n_bias: partial bias gradients
  double* lpart;         // chain workgroups: partial losses
  float *grad, *grad2, *loss;  // grad2, loss: optional
  long batch, n_params;
  int n_bias;            // sum of w[1..L]
  int chain_blocks, splits, chunk, tiles;  // set by launch_fused_backward
};
hipError_t launch_fused_backward(MlpBackArgs a, hipStream_t s);

}  // namespace subadmm

struct subadmm_mlp;
int32_t mlp_input_width(const subadmm_mlp* m);
int32_t mlp_output_width(const subadmm_mlp* m);
int32_t mlp_max_batch(const subadmm_mlp* m);
hipStream_t mlp_stream(const subadmm_mlp* m);
// advances on every bind and input-affine change (what a captured forward pass depends on)
uint64_t mlp_generation(const subadmm_mlp* m);
// subadmm_mlp_forward with its launches on stream s (a capture stream or the bound one)
int mlp_forward_on(subadmm_mlp* m, hipStream_t s, int32_t batch, const float* x, float* y);
// subadmm_mlp_infer on stream s: the fused inference when the widths allow it, else the forward
int mlp_infer_on(subadmm_mlp* m, hipStream_t s, int32_t batch, const float* x, float* y);
