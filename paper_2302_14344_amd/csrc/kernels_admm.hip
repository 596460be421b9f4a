// HIP kernels (gfx950) for the per-step factorisation and the ADMM iteration of the
// subsystem-based ADMM method (arXiv 2302.14344, Algorithm 1).
//
// factor_kernel: one workgroup per subsystem.  Forms K_i = A_i + beta_i J_c,i^T J_c,i
//   (Eq. (15), beta_i of Eq. (23)), Jacobi-scales it, factorises it in LDS (Cholesky)
//   and precomputes the slot-space operators of the x-update:
//     H_i = J K^-1 J^T (nc x nc),  d_i = J K^-1 b,  G_i = K^-1 J^T,  c_i = K^-1 b,
//   so that, with w_i = beta_i z_i - u_i,
//     x_i = J v_hat_i = d_i + H_i w_i   and   v_hat_i = c_i + G_i w_i,
//   which is Eq. (15) followed by x = J v_hat, reassociated.  The per-iteration work is
//   then one small dense matrix-vector product per subsystem with no sequential chain.
// loop_kernel: one workgroup per scene runs the whole iteration in one launch, with the
//   slot state in LDS:
//     x-update (Eq. 15) -> y = beta x + u (Eq. 18) -> residual (Eq. 22, deterministic
//     block reduction) -> stopping test -> z-update (Eq. 16-21) -> dual update (Eq. 14).
//   After a z-update u_i,j = -lambda_j and w = beta z - u = y + 2 lambda, so the kernel
//   keeps (y, w, u) per slot row.
#include <type_traits>

#include "exchange.hpp"
#include "internal.hpp"
#include "mfma.hpp"
#include "rigid_device.hpp"
#include "row_walk.hpp"

namespace subadmm {

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Orders the LDS accesses of one wave's lanes (a wave's LDS instructions complete in
// issue order; the fences keep the compiler from moving accesses across this point).
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The threads that factorise one subsystem: the whole workgroup (workgroup barriers), or
// one wave (its 64 lanes, wave-level fences), so that the waves of a workgroup factorise
// different small subsystems at the same time.
struct GroupWg {
  static constexpr bool kWave = false;
  __device__ static int rank() { return threadIdx.x; }
  __device__ static int size() { return blockDim.x; }
  __device__ static int wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x) >> 6; }
  __device__ static int waves() { return blockDim.x >> 6; }
  __device__ static void sync() { __syncthreads(); }
};
struct GroupWave {
  static constexpr bool kWave = true;
  __device__ static int rank() { return threadIdx.x & 63; }
  __device__ static int size() { return 64; }
  __device__ static int wave() { return 0; }
  __device__ static int waves() { return 1; }
  __device__ static void sync() { wave_lds_fence(); }
};

// Subsystems a single wave factorises: small ones (n <= 64, at most 64 right-hand sides) whose
// working arrays fit the wave's share of LDS.
__host__ __device__ inline bool wave_factor_fits(int n, int nc, size_t cs, size_t slice) {
  return n <= 64 && nc + 1 <= 64 && factor_bytes(n, nc, cs) <= slice;
}

template <typename T>
__device__ inline T dev_sqrt(T x);
template <>
__device__ inline float dev_sqrt<float>(float x) { return __builtin_sqrtf(x); }
template <>
__device__ inline double dev_sqrt<double>(double x) { return __builtin_sqrt(x); }

// ------------------------------------------------------------------------------------
// Per-step factorisation and slot-space operators (Alg. 1 factorisation step)
// ------------------------------------------------------------------------------------
// Entry i of p where `in`, else zero, without a branch around the load (p[0] is readable), so
// that the loads of a tile product are in flight together.
template <typename C, typename P>
__device__ inline C tile_at(P p, int i, bool in) {
  const C v = p[in ? i : 0];
  return in ? v : (C)0;
}

// Factorisation of subsystem i by the thread group Grp (the workgroup or one wave), with its
// working arrays at sm (LDS, or a global scratch area of the same layout); red (workgroup
// form only) and bad are scratch shared by the group.
//
// Every O(n^2) and O(n^3) part is 16 x 16 tile products on the matrix cores: K's penalty term,
// a left-looking blocked Cholesky whose diagonal tiles one wave factorises and inverts in
// registers (the inverse replaces the tile), the block forward substitution of the right-hand
// sides, H = T^T T, and the block back substitution.  A wave owns 16 right-hand sides from
// start to end, so the substitutions have no barrier; the group synchronises three times per
// 16 columns of the factor.  A tile's arithmetic does not depend on which wave forms it, so
// the workgroup and the wave form agree except in the trace sums' grouping of Eq. 23.  Products are
// subtracted from the entry itself, the accumulator starting from it (added up first, their sum
// stays at the entry's size while the remainder shrinks, and multipliers of 300-DOF subsystems
// were 1.9 times as far from the exact ones).
//
// Bound by latency: the diagonal tiles (~2.7 us each, one wave) and chains of tile products; few
// subsystems leave the matrix cores mostly idle.  Measured against the column-by-column form
// (a barrier per column of the factor and per four pivot rows of the substitutions): 48 DOF with
// 75 slot rows 78 -> 33 us, 127 DOF 260 -> 86 us, 285 DOF in device memory 4790 -> 462 us; the
// legged batch's classes, side by side, 80 -> 57 us and 85 -> 66 us (one subsystem per wave).
template <typename T, typename C, typename Grp = GroupWg, typename P = C*, int kUnroll = 1>
__device__ __attribute__((always_inline)) inline void factor_body(const FactorArgs<T>& a, const int i, P sm,
                                                                 double (*red)[16], int& bad) {
  const int tid = Grp::rank();
  const int bd = Grp::size();
  const int n = a.t.sub_n[i];
  const int nc = a.t.sub_nc[i];
  // LDS leading dimensions are odd so that strided accesses fall in distinct banks
  const int ld = n | 1;
  P K = sm;                   // n x n, row-major with leading dimension ld, lower used
  P X = K + n * ld;           // (nc + 1) columns of length n, column stride ld: J rows, then b,
                              // solved in place
  P Jl = X;                   // the first nc columns: J (nc x n, row-major, leading dimension ld)
  P sc = X + (nc + 1) * ld;   // Jacobi scaling 1/sqrt(K_rr); n more entries are not used

  const T* A = a.A + a.t.sub_A[i];
  const T* J = a.J + a.t.sub_J[i];
  const T* b = a.b + a.t.sub_dof[i];
  if (tid == 0) bad = 0;
  const RowWalk first(tid, bd, n);
  RowWalk e = first;
#pragma unroll 4
  for (int t = tid; t < n * n; t += bd, e.next()) K[e.row * ld + e.col] = (C)A[t];
  e = first;
#pragma unroll 4
  for (int t = tid; t < nc * n; t += bd, e.next()) Jl[e.row * ld + e.col] = (C)J[t];
  for (int t = tid; t < n; t += bd) X[nc * ld + t] = (C)b[t];
  Grp::sync();

  // Eq. (23): beta_i = Tr(A_i) / Tr(J^T J); Tr(J^T J) = |J|_F^2.
  double trA = 0.0, trJ = 0.0;
  for (int t = tid; t < n; t += bd) trA += (double)K[t * ld + t];
  e = first;
  for (int t = tid; t < nc * n; t += bd, e.next()) {
    const C v = Jl[e.row * ld + e.col];
    trJ = tfma((double)v, (double)v, trJ);
  }
  if constexpr (Grp::kWave) {
    trA = wave_sum(trA);
    trJ = wave_sum(trJ);
  } else {
    const int lane = tid & 63, wv = tid >> 6;
    double s0 = wave_sum(trA), s1 = wave_sum(trJ);
    if (lane == 0) { red[0][wv] = s0; red[1][wv] = s1; }
    Grp::sync();
    trA = 0.0; trJ = 0.0;
    for (int w = 0; w < bd / 64; ++w) { trA += red[0][w]; trJ += red[1][w]; }
  }
  C beta;
  if (a.rho > 0.0) beta = (C)a.rho;
  else beta = trJ > 0.0 ? (C)(trA / trJ) : (C)1;

  typedef Mfma<C> M;
  typedef typename M::V MV;
  const int lane = threadIdx.x & 63, g = lane >> 4, cn = lane & 15;
  const int wv = Grp::wave(), nwv = Grp::waves();
  const int nt = (n + 15) >> 4;  // tile rows of K
  // K += beta J^T J, a wave per lower tile (k runs over the rows of J)
  for (int tt = wv; tt < nt * (nt + 1) / 2; tt += nwv) {
    int I = 0;
    while ((I + 1) * (I + 2) / 2 <= tt) ++I;
    const int ra = 16 * I + cn, rb = 16 * (tt - I * (I + 1) / 2) + cn;
    MV acc = {0, 0, 0, 0};
#pragma unroll kUnroll
    for (int k0 = 0; k0 < nc; k0 += 16) {
      C av[4], bv[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = k0 + M::k(s, g);
        av[s] = tile_at<C>(Jl, k * ld + ra, k < nc && ra < n);
        bv[s] = tile_at<C>(Jl, k * ld + rb, k < nc && rb < n);
      }
      acc = M::mul(av, bv, acc);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 16 * I + M::k(q, g);
      if (r < n && rb <= r) K[r * ld + rb] = tfma(beta, (C)acc[q], (C)K[r * ld + rb]);
    }
  }
  Grp::sync();
  for (int r = tid; r < n; r += bd) {
    C dgl = K[r * ld + r];
    if (!(dgl > (C)0)) { bad = 1; dgl = (C)1; }
    sc[r] = (C)1 / dev_sqrt<C>(dgl);
  }
  Grp::sync();
  // K_hat = S K S, J_hat = J S (S = diag(sc)).
  e = first;
  for (int t = tid; t < n * n; t += bd, e.next())
    if (e.col <= e.row) K[e.row * ld + e.col] *= sc[e.row] * sc[e.col];
  e = first;
  for (int t = tid; t < (nc + 1) * n; t += bd, e.next()) X[e.row * ld + e.col] *= sc[e.col];  // J_hat rows, then S b
  Grp::sync();

  // Cholesky factor L of K_hat, 16 columns at a time; diagonal tiles hold their inverses.
  for (int p = 0; p < nt; ++p) {
    const int p0 = 16 * p, jb = n - p0 < 16 ? n - p0 : 16;
    if (p > 0) {
      // -U_Ip = -K_Ip + sum_{k < p} L_Ik L_pk^T: the lane holds U[cn][row(q, g)]
      for (int I = p + wv; I < nt; I += nwv) {
        const int ri = 16 * I + cn;
        MV acc;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = p0 + M::k(q, g);
          acc[q] = -tile_at<C>(K, ri * ld + c, ri < n && c < n && c <= ri);
        }
#pragma unroll kUnroll
        for (int k0 = 0; k0 < p0; k0 += 16) {
          C av[4], bv[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int k = k0 + M::k(s, g);
            av[s] = tile_at<C>(K, (p0 + cn) * ld + k, cn < jb);
            bv[s] = tile_at<C>(K, ri * ld + k, ri < n);
          }
          acc = M::mul(av, bv, acc);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = p0 + M::k(q, g);
          if (ri < n && c < n && c <= ri) K[ri * ld + c] = -acc[q];
        }
      }
      Grp::sync();
    }
    if (wv == 0) {
      if (!diag_tile<C>(K + (p0 * ld + p0), ld, jb) && lane == 0) bad = 1;
    }
    Grp::sync();
    if (p + 1 < nt) {
      // L_Ip = U_Ip L_pp^-T (jb = 16: tiles below the diagonal follow a full one)
      for (int I = p + 1 + wv; I < nt; I += nwv) {
        const int ri = 16 * I + cn;
        C av[4], bv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int k = M::k(s, g);
          av[s] = tile_at<C>(K, ri * ld + p0 + k, ri < n);
          bv[s] = tile_at<C>(K, (p0 + cn) * ld + p0 + k, k <= cn);
        }
        MV out = {0, 0, 0, 0};
        out = M::mul(av, bv, out);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = 16 * I + M::k(q, g);
          if (r < n) K[r * ld + p0 + cn] = out[q];
        }
      }
      Grp::sync();
    }
  }

  // T = L^-1 [J_hat^T | S b] by block forward substitution in place, then H = T_J^T T_J and
  // d = T_J^T T_b (= J_hat K_hat^-1 J_hat^T and J_hat K_hat^-1 S b), then block back
  // substitution in place gives K_hat^-1 [J_hat^T | S b] for G and c.  A lane reads back only
  // the entries of X that it wrote itself.
  T* H = a.H + a.t.sub_H[i];
  T* dd = a.d + a.t.sub_slot[i];
  T* G = a.G + a.t.sub_J[i];
  T* cv = a.cvec + a.t.sub_dof[i];
  const int m = nc + 1, nct = (m + 15) >> 4;
  for (int ct = wv; ct < nct; ct += nwv) {
    const int c = 16 * ct + cn;
    P x = X + (c < m ? c : 0) * ld;
    for (int I = 0; I < nt; ++I) {
      const int i0 = 16 * I, ri = i0 + cn;
      MV acc;
      C lv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = M::k(q, g);
        acc[q] = -tile_at<C>(x, i0 + k, c < m && i0 + k < n);
        lv[q] = tile_at<C>(K, ri * ld + i0 + k, k <= cn && ri < n);
      }
#pragma unroll kUnroll
      for (int k0 = 0; k0 < i0; k0 += 16) {
        C av[4], bv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int k = k0 + M::k(s, g);
          av[s] = tile_at<C>(K, ri * ld + k, ri < n);
          bv[s] = tile_at<C>(x, k, c < m);
        }
        acc = M::mul(av, bv, acc);
      }
      C bv[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) bv[s] = -acc[s];
      MV out = {0, 0, 0, 0};
      out = M::mul(lv, bv, out);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = i0 + M::k(q, g);
        if (c < m && r < n) x[r] = out[q];
      }
    }
  }
  Grp::sync();
  for (int tt = wv; tt < nct * (nct + 1) / 2; tt += nwv) {
    int I = 0;
    while ((I + 1) * (I + 2) / 2 <= tt) ++I;
    const int J = tt - I * (I + 1) / 2;
    const int ca = 16 * I + cn, cb = 16 * J + cn;
    P xa = X + (ca < m ? ca : 0) * ld;
    P xb = X + (cb < m ? cb : 0) * ld;
    MV acc = {0, 0, 0, 0};
#pragma unroll kUnroll
    for (int k0 = 0; k0 < n; k0 += 16) {
      C av[4], bv[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = k0 + M::k(s, g);
        av[s] = tile_at<C>(xa, k, ca < m && k < n);
        bv[s] = tile_at<C>(xb, k, cb < m && k < n);
      }
      acc = M::mul(av, bv, acc);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 16 * I + M::k(q, g);
      const T v = (T)acc[q];
      if (r < nc && cb < nc) {
        H[cb * nc + r] = v;
        H[r * nc + cb] = v;
      } else if (r == nc && cb < nc) {
        dd[cb] = v;
      }
    }
  }
  Grp::sync();
  for (int ct = wv; ct < nct; ct += nwv) {
    const int c = 16 * ct + cn;
    P x = X + (c < m ? c : 0) * ld;
    for (int I = nt - 1; I >= 0; --I) {
      const int i0 = 16 * I;
      MV acc;
      C lv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = M::k(q, g);
        acc[q] = -tile_at<C>(x, i0 + k, c < m && i0 + k < n);
        lv[q] = tile_at<C>(K, (i0 + k) * ld + i0 + cn, cn <= k && i0 + k < n);
      }
#pragma unroll kUnroll
      for (int k0 = i0 + 16; k0 < n; k0 += 16) {
        C av[4], bv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int k = k0 + M::k(s, g);
          av[s] = tile_at<C>(K, k * ld + i0 + cn, k < n);
          bv[s] = tile_at<C>(x, k, c < m && k < n);
        }
        acc = M::mul(av, bv, acc);
      }
      C bv[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) bv[s] = -acc[s];
      MV out = {0, 0, 0, 0};
      out = M::mul(lv, bv, out);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = i0 + M::k(q, g);
        if (c < m && r < n) {
          x[r] = out[q];
          // G = S X_J, c = S X_b
          const T v = (T)(sc[r] * out[q]);
          if (c < nc) G[c * n + r] = v;
          else cv[r] = v;
        }
      }
    }
  }
  if (tid == 0) {
    a.beta[i] = (T)beta;
    if (bad) atomicOr(a.flags, FLAG_NOT_SPD);
  }
}

template <typename T, typename C>
__global__ void __launch_bounds__(512) factor_kernel(FactorArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[2][16];
  __shared__ int bad;
  factor_body<T, C>(a, a.order[a.first + blockIdx.x], reinterpret_cast<C*>(smem_raw), red, bad);
}

constexpr int kBigThreads = 1024;
// Subsystems whose working arrays exceed the LDS: the same factorisation with its working
// arrays in device memory (scr + off[i] bytes), one 1024-thread workgroup each (a workgroup's
// barriers order its device-memory accesses as they do its LDS accesses).
template <typename T, typename C>
__global__ void __launch_bounds__(kBigThreads) factor_global_kernel(FactorArgs<T> a, char* scr, const int64_t* off) {
  __shared__ double red[2][16];
  __shared__ int bad;
  const int i = a.order[a.first + blockIdx.x];
  factor_body<T, C, GroupWg, C*, 4>(a, i, reinterpret_cast<C*>(scr + off[i]), red, bad);
}

// Small subsystems: each wave of a 256-thread workgroup factorises one subsystem in its
// quarter of the LDS (slice bytes), with no workgroup barrier.
template <typename T, typename C>
__global__ void __launch_bounds__(256) factor_wave_kernel(FactorArgs<T> a, int count, int slice) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ int bad[4];
  const int wv = threadIdx.x >> 6;
  const int k = blockIdx.x * 4 + wv;
  if (k >= count) return;
  factor_body<T, C, GroupWave>(a, a.order[a.first + k], reinterpret_cast<C*>(smem_raw + (size_t)wv * slice), nullptr,
                               bad[wv]);
}

// ------------------------------------------------------------------------------------
// Contact projection of Eq. (21) in the scalar metric of Eq. (18): exact Signorini-
// Coulomb solution lambda_n = max(0, p_n), lambda_t = p_t clipped to the disc of radius
// mu lambda_n along p_t.
// ------------------------------------------------------------------------------------
template <typename T>
__device__ inline T disc_scale(T cap, T tn2);
template <>
__device__ inline float disc_scale<float>(float cap, float tn2) {
  // The hardware reciprocal square root reads a denormal input as zero: a tangential part
  // below ~1e-19 (tn2 under the smallest normal float, met on separating contacts at rest)
  // would give cap * inf, NaN for cap = 0.  Such inputs take the FP64 square root, where
  // every FP32 value is normal.
  if (!(cap > 0.0f)) return 0.0f;
  if (tn2 >= __FLT_MIN__) return cap * __builtin_amdgcn_rsqf(tn2);
  return (float)((double)cap / __builtin_sqrt((double)tn2));
}
template <>
__device__ inline double disc_scale<double>(double cap, double tn2) { return cap / __builtin_sqrt(tn2); }

// Tested on squares (|p_t|^2 > (mu lambda_n)^2); the disc scale mu lambda_n / |p_t| uses the
// hardware reciprocal square root in FP32 (1 ulp; FP64 for inputs below the normal range)
// and the correctly rounded forms in FP64.
template <typename T>
__device__ inline void contact_project(const T* p, T mu, T* lam, int model) {
  if (model == 1) {
    cone_project<T>(p, mu, lam);
    return;
  }
  const T ln = p[0] > (T)0 ? p[0] : (T)0;
  const T tn2 = p[1] * p[1] + p[2] * p[2];
  const T cap = mu * ln;
  lam[0] = ln;
  if (tn2 > cap * cap) {
    const T f = disc_scale<T>(cap, tn2);
    lam[1] = f * p[1];
    lam[2] = f * p[2];
  } else {
    lam[1] = p[1];
    lam[2] = p[2];
  }
}

// e + ya ib0 + yb ib1 (the bracket of Eq. 17-21) and the soft z-update of Eq. 20,
// lambda = -k (e + alpha sum y/beta) / (1 + w alpha k), with explicit fused multiply-adds,
// so that every form of the z-update rounds the same way.
__device__ inline float zfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double zfma(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <typename T>
__device__ inline T zsum(T e, T ya, T ib0, T yb, T ib1) {
  return zfma(yb, ib1, zfma(ya, ib0, e));
}
template <typename T>
__device__ inline T zsoft(T e, T ya, T ib0, T yb, T ib1, T k, T alpha) {
  return -k * zfma(alpha, zfma(yb, ib1, ya * ib0), e) / zfma(alpha * k, ib0 + ib1, (T)1);
}

// z-update (Eq. 16-21) and dual update (Eq. 14) of one interface of a fixed class, with
// the loops over its rows at their real length.

// z-update (Eq. 16-21) and dual update (Eq. 14) of an interface with more than two members
// (|S_j| up to 4): the bracket of Eq. 17-21 sums e_j and y_i / beta_i over every member and
// the weight w = sum 1/beta_i; lambda then acts on every member alike.  Member slots are
// read from the topology tables: y, u at slot - s0 (scene-local), w at the member's w
// offset (padded per-subsystem blocks when kPadW).  Used for the rare interfaces of this
// kind only, so the per-thread state of the common ones stays as it is.
template <typename T, bool kPadW>
__device__ inline void z_update_multi(const LoopArgs<T>& a, const int j, const int s0, const T* ev, const T* y,
                                      T* u, T* w) {
  const int nm = a.t.if_nsub[j], dim = a.t.if_dim[j], kind = a.t.if_kind[j];
  int ps[kMaxMembers], qs[kMaxMembers];
  T ib[kMaxMembers];
  T wsum = (T)0;
  for (int m = 0; m < kMaxMembers; ++m) {
    ps[m] = qs[m] = 0;
    ib[m] = (T)0;
    if (m >= nm) continue;
    const int i = m == 0 ? a.t.if_sub0[j] : m == 1 ? a.t.if_sub1[j] : a.t.if_subx[2 * j + m - 2];
    const int g = m == 0 ? a.t.if_slot0[j] : m == 1 ? a.t.if_slot1[j] : a.t.if_slotx[2 * j + m - 2];
    ps[m] = g - s0;
    qs[m] = (kPadW ? a.t.sub_wq[i] : a.t.sub_slot[i] - s0) + (g - a.t.sub_slot[i]);
    ib[m] = (T)1 / a.beta[i];
    wsum += ib[m];
  }
  T p[kMaxIfDim], lam[kMaxIfDim];
  for (int k = 0; k < kMaxIfDim; ++k) {
    p[k] = (T)0;
    if (k >= dim) continue;
    T sy = (T)0;
    for (int m = 0; m < nm; ++m) sy += y[ps[m] + k] * ib[m];
    p[k] = kind == KIND_SOFT ? -a.ksoft[j] * (ev[k] + a.asoft[j] * sy) / ((T)1 + wsum * a.asoft[j] * a.ksoft[j])
                             : -(ev[k] + sy) / wsum;
  }
  T cl[3];
  contact_project<T>(p, a.mu[j], cl, a.contact_model);
  for (int k = 0; k < kMaxIfDim; ++k) {
    T v = p[k];
    if (kind == KIND_HARD_INEQ) v = v > (T)0 ? v : (T)0;
    if (kind == KIND_CONTACT && k < 3) v = cl[k];
    lam[k] = v;
  }
  for (int m = 0; m < nm; ++m)
    for (int k = 0; k < dim; ++k) {
      const T yk = y[ps[m] + k];
      u[ps[m] + k] = -lam[k];
      w[qs[m] + k] = yk + (T)2 * lam[k];
    }
}

// The same update from a descriptor staged in LDS at the start of the solve (the members'
// rows and inverse penalties and the interface's constants), so that an iteration reads no
// topology from device memory.  Same arithmetic in the same order.  A dependent chain of
// device-memory reads (member, slot, penalty, division) set the iteration's time before: one
// solve of 200 ragged scenes with couplings of up to four members, FP32, 1248 us
// without the descriptors and 735 us with them (686 since rows go three at a time).
template <typename T>
struct MultiDesc {
  T ib[kMaxMembers];
  T wsum, mu, k, alpha;
  int32_t ps[kMaxMembers];  // first slot row in y, u; -1: no such member
  int32_t qs[kMaxMembers];  // first entry in w
};
static_assert(sizeof(MultiDesc<float>) == kMultiDescF32 && sizeof(MultiDesc<double>) == kMultiDescF64, "LDS plan");

template <typename T, bool kPadW>
__device__ inline void multi_desc(const LoopArgs<T>& a, const int j, const int s0, MultiDesc<T>& d) {
  const int nm = a.t.if_nsub[j];
  T wsum = (T)0;
  for (int m = 0; m < kMaxMembers; ++m) {
    d.ps[m] = -1;
    d.qs[m] = 0;
    d.ib[m] = (T)0;
    if (m >= nm) continue;
    const int i = m == 0 ? a.t.if_sub0[j] : m == 1 ? a.t.if_sub1[j] : a.t.if_subx[2 * j + m - 2];
    const int g = m == 0 ? a.t.if_slot0[j] : m == 1 ? a.t.if_slot1[j] : a.t.if_slotx[2 * j + m - 2];
    d.ps[m] = g - s0;
    d.qs[m] = (kPadW ? a.t.sub_wq[i] : a.t.sub_slot[i] - s0) + (g - a.t.sub_slot[i]);
    d.ib[m] = (T)1 / a.beta[i];
    wsum += d.ib[m];
  }
  d.wsum = wsum;
  d.mu = a.mu[j];
  d.k = a.ksoft[j];
  d.alpha = a.asoft[j];
}

// Three rows at a time (couplings of four to six rows take two turns; a contact has three): six at once
// hold the members' y in so many registers that fewer scenes are resident (2,000 scenes of
// couplings of three, FP64, 100 iterations: 2.17 ms without descriptors, 2.48 with six rows at once,
// 1.46 with three; the 200 ragged scenes above 751 and 686 us a solve with six and three).
template <typename T>
__device__ inline void z_update_desc(const MultiDesc<T>& d, const int kind, const int dim, const int model, const T* ev,
                                     const T* y, T* u, T* w) {
#pragma unroll 1
  for (int k0 = 0; k0 < dim; k0 += 3) {
    T ym[kMaxMembers][3], p[3];
#pragma unroll
    for (int m = 0; m < kMaxMembers; ++m)
#pragma unroll
      for (int k = 0; k < 3; ++k) ym[m][k] = y[(d.ps[m] >= 0 ? d.ps[m] : 0) + (k0 + k < dim ? k0 + k : 0)];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      T sy = (T)0;
#pragma unroll
      for (int m = 0; m < kMaxMembers; ++m) {
        const T t = zfma(ym[m][k], d.ib[m], sy);
        sy = d.ps[m] >= 0 ? t : sy;
      }
      const T e = ev[k0 + k < dim ? k0 + k : 0];
      p[k] = kind == KIND_SOFT ? -d.k * zfma(d.alpha, sy, e) / zfma(d.wsum * d.alpha, d.k, (T)1) : -(e + sy) / d.wsum;
    }
    if (kind == KIND_CONTACT) {
      const T q[3] = {p[0], p[1], p[2]};
      contact_project<T>(q, d.mu, p, model);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const T lam = kind == KIND_HARD_INEQ ? (p[k] > (T)0 ? p[k] : (T)0) : p[k];
      if (k0 + k < dim) {
#pragma unroll
        for (int m = 0; m < kMaxMembers; ++m) {
          if (d.ps[m] >= 0) {
            u[d.ps[m] + k0 + k] = -lam;
            w[d.qs[m] + k0 + k] = ym[m][k] + (T)2 * lam;
          }
        }
      }
    }
  }
}

template <typename T, int D, int KIND>
__device__ inline void z_update_fixed(const T* ev, T ib0, T ib1, T iws, T mu, int p0, int p1, int q0, int q1,
                                      const T* y, T* u, T* w, int model) {
  T ya[D], yb[D], lam[D];
#pragma unroll
  for (int k = 0; k < D; ++k) {
    ya[k] = y[p0 + k];
    yb[k] = y[p1 + k];
  }
#pragma unroll
  for (int k = 0; k < D; ++k) lam[k] = -zsum(ev[k], ya[k], ib0, yb[k], ib1) * iws;
  if (KIND == KIND_CONTACT) {
    const T p3[3] = {lam[0], lam[1], lam[2]};
    contact_project<T>(p3, mu, lam, model);
  } else if (KIND == KIND_HARD_INEQ) {
#pragma unroll
    for (int k = 0; k < D; ++k) lam[k] = lam[k] > (T)0 ? lam[k] : (T)0;
  }
#pragma unroll
  for (int k = 0; k < D; ++k) {
    u[p0 + k] = -lam[k];
    w[q0 + k] = ya[k] + (T)2 * lam[k];
  }
  if (p1 != p0) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      u[p1 + k] = -lam[k];
      w[q1 + k] = yb[k] + (T)2 * lam[k];
    }
  }
}

// ------------------------------------------------------------------------------------
// Wave-level sum with DPP cross-lane moves (fixed order, so deterministic).  After the
// four in-row steps every lane of a 16-lane row holds the row sum; the two broadcast
// steps fold rows 0+1 into row 1 and rows 0..3 into row 3; lane 63 holds the total.
// ------------------------------------------------------------------------------------
__device__ inline float dpp_f(float v, int ctrl_sel) {
  int x = __float_as_int(v);
  int y;
  switch (ctrl_sel) {
    case 0: y = __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false); break;   // quad_perm [1,0,3,2]
    case 1: y = __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false); break;   // quad_perm [2,3,0,1]
    case 2: y = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false); break;  // row_half_mirror
    case 3: y = __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, false); break;  // row_mirror
    case 4: y = __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false); break;  // row_bcast:15
    default: y = __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false); break; // row_bcast:31
  }
  return __int_as_float(y);
}

__device__ inline double dpp_d(double v, int ctrl_sel) {
  const long long b = __double_as_longlong(v);
  int lo = (int)(b & 0xffffffffLL), hi = (int)(b >> 32);
  int l2, h2;
  switch (ctrl_sel) {
    case 0: l2 = __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xF, 0xF, false); h2 = __builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xF, 0xF, false); break;
    case 1: l2 = __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xF, 0xF, false); h2 = __builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xF, 0xF, false); break;
    case 2: l2 = __builtin_amdgcn_update_dpp(0, lo, 0x141, 0xF, 0xF, false); h2 = __builtin_amdgcn_update_dpp(0, hi, 0x141, 0xF, 0xF, false); break;
    case 3: l2 = __builtin_amdgcn_update_dpp(0, lo, 0x140, 0xF, 0xF, false); h2 = __builtin_amdgcn_update_dpp(0, hi, 0x140, 0xF, 0xF, false); break;
    case 4: l2 = __builtin_amdgcn_update_dpp(0, lo, 0x142, 0xA, 0xF, false); h2 = __builtin_amdgcn_update_dpp(0, hi, 0x142, 0xA, 0xF, false); break;
    default: l2 = __builtin_amdgcn_update_dpp(0, lo, 0x143, 0xC, 0xF, false); h2 = __builtin_amdgcn_update_dpp(0, hi, 0x143, 0xC, 0xF, false); break;
  }
  const long long r = ((long long)(unsigned)h2 << 32) | (long long)(unsigned)l2;
  return __longlong_as_double(r);
}

__device__ inline float dpp_sel(float v, int k) { return dpp_f(v, k); }
__device__ inline double dpp_sel(double v, int k) { return dpp_d(v, k); }

// Sum over the 64 lanes of a wave; the result is valid in lane 63.
template <typename A>
__device__ inline A wave_total_lane63(A v) {
  v += dpp_sel(v, 0);
  v += dpp_sel(v, 1);
  v += dpp_sel(v, 2);
  v += dpp_sel(v, 3);
  v += dpp_sel(v, 4);
  v += dpp_sel(v, 5);
  return v;
}

// ------------------------------------------------------------------------------------
// Whole ADMM iteration of one scene per workgroup.
//
// Slot row r is owned by lane kLanes*r (kLanes = 1 or 2 lanes share its dot product,
// combined with a DPP swap); kLanes = 0: a host map gives each lane its row and part, a
// row taking 1, 2 or 4 aligned lanes (combined with quad DPP).  Interface i0 + t is owned
// by thread t.  Their constant data stay in registers for the whole iteration.
//
// Every form adds a lane's share of a row's 16-byte vector products in one order: in groups
// of four, the t-th vector of a group to partial sum t mod 4, the vectors after the last full
// group to partial 0, and the lane's sum is (p0 + p1) + (p2 + p3); the lanes of a split row
// then add their sums pairwise, then by quads.
//
// LDS (kHInLds): the scene's H_i in a blocked layout of 16-byte vectors, vector
// (cb, r) = H_i[r][V*cb .. V*cb + V-1] at sub_hq[i] + cb * nc_i + r (zero padded), so
// that consecutive lanes of one subsystem read consecutive vectors; w in per-subsystem
// blocks padded to a multiple of V (read as broadcast vectors); y and u per slot row.
// Without kHInLds H is read from global memory in its plain column-major layout.
// Every phase issues its loads before their first use.
// ------------------------------------------------------------------------------------
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  using type = float4;
  static constexpr int N = 4;
  __device__ static float dot(const float4& a, const float4& b) {
    return (a.x * b.x + a.y * b.y) + (a.z * b.z + a.w * b.w);
  }
  __device__ static float get(const float4& a, int q) { return q == 0 ? a.x : q == 1 ? a.y : q == 2 ? a.z : a.w; }
  __device__ static float4 make(const float* v) { return make_float4(v[0], v[1], v[2], v[3]); }
};
template <>
struct Vec16<double> {
  using type = double2;
  static constexpr int N = 2;
  __device__ static double dot(const double2& a, const double2& b) { return a.x * b.x + a.y * b.y; }
  __device__ static double get(const double2& a, int q) { return q == 0 ? a.x : a.y; }
  __device__ static double2 make(const double* v) { return make_double2(v[0], v[1]); }
};

// Where the iteration kernel reads H_i: global memory or LDS (blocked layout).
constexpr int kHGlobal = 0, kHLds = 1;

template <typename T>
__device__ inline T pair_sum(T v) {
  return v + dpp_sel(v, 0);  // quad_perm [1,0,3,2]: adds the neighbouring lane
}

// Partial sums of one lane's share of x_r = H_i[r] . w_i from the blocked LDS layout: the
// row's vectors part, part + kp, ... (count cnt), H vector stride hs, w vector stride kp.
template <typename T, typename VT>
__device__ inline T row_dot_share(const VT* Hv, const VT* Wv, int cnt, int hs, int kp) {
  T acc[4] = {(T)0, (T)0, (T)0, (T)0};
  int t = 0;
  for (; t + 3 < cnt; t += 4) {
    VT hv[4], wq[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      hv[k] = Hv[(t + k) * hs];
      wq[k] = Wv[(t + k) * kp];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] += Vec16<T>::dot(hv[k], wq[k]);
  }
  for (; t < cnt; ++t) acc[0] += Vec16<T>::dot(Hv[t * hs], Wv[t * kp]);
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The whole iteration of scene sc by the workgroup; smem_raw is the dynamic LDS area, red a
// workgroup-shared scratch for the residual sums.  kMulti: the problem has interfaces of more
// than two members (a form of its own, so that the others do not carry its registers).  kOutlined:
// called from the multi-step kernel.
template <typename T, int kHMode, int kLanes, bool kMulti = false, bool kOutlined = false>
__device__ __attribute__((always_inline)) inline void loop_body(const LoopArgs<T>& a, const int sc,
                                                               unsigned char* smem_raw, T (*red)[8]) {
  static_assert(kLanes > 0 || kHMode == 1, "split rows need the LDS layout");
  using VT = typename Vec16<T>::type;
  constexpr int V = Vec16<T>::N;
  constexpr bool kHInLds = kHMode == kHLds;
  constexpr bool kPadW = kHInLds;  // w in padded per-subsystem blocks
  const int tid = threadIdx.x;
  const int bd = blockDim.x;
  const int nwave = bd >> 6;
  const int lane = tid & 63, wv = tid >> 6;
  if (a.skip_converged && a.skip_converged[sc]) return;
  const int s0 = a.t.sc_slot[sc], s1 = a.t.sc_slot[sc + 1];
  const int ns = s1 - s0;
  const int i0 = a.t.sc_if[sc], i1 = a.t.sc_if[sc + 1];
  const int sb = a.t.sc_sub[sc], se = a.t.sc_sub[sc + 1];
  const long long h0 = a.t.sub_H[sb];
  const int nhq = kHInLds ? a.t.sc_hq[sc] : 0;
  const int nwq = kPadW ? a.t.sc_wq[sc] : ns;
  VT* Hq = reinterpret_cast<VT*>(smem_raw);
  T* w = reinterpret_cast<T*>(Hq + nhq);  // padded blocks (kPadW) or per slot row
  T* y = w + nwq;
  T* u = y + ns;

  if (kHInLds) {
    // stage H_i into the blocked layout and clear the padded w area
    for (int i = sb; i < se; ++i) {
      const int nci = a.t.sub_nc[i];
      const int nq = (nci + V - 1) / V;
      const T* Hg = a.H + a.t.sub_H[i];
      VT* dst = Hq + a.t.sub_hq[i];
      for (int q = tid; q < nq * nci; q += bd) {
        const int cb = q / nci, rr = q - cb * nci;
        T v[V];
#pragma unroll
        for (int k = 0; k < V; ++k) {
          const int c = cb * V + k;
          v[k] = c < nci ? Hg[c * nci + rr] : (T)0;
        }
        dst[q] = Vec16<T>::make(v);
      }
    }
    for (int q = tid; q < nwq; q += bd) w[q] = (T)0;
    __syncthreads();
  }

  // slot row handled by this lane (and the lane's share of its dot product)
  int r, part, kp;
  if constexpr (kLanes == 0) {
    const int code = a.t.rmap[(size_t)sc * bd + tid];
    r = code >= 0 ? code >> 5 : ns;
    kp = code >= 0 ? (code >> 2) & 7 : 1;
    part = code >= 0 ? code & 3 : 0;
  } else {
    r = tid / kLanes;
    part = tid - r * kLanes;
    kp = kLanes;
  }
  const bool in_slot = r < ns;
  const bool owner = in_slot && part == 0;
  int nc = 0, hoff = 0, wo = 0, loc = 0;
  T be = (T)0, dr = (T)0;
  if (in_slot) {
    const int g = s0 + r;
    const int i = a.t.slot_sub[g];
    nc = a.t.sub_nc[i];
    loc = a.t.slot_loc[g];
    if (kHInLds) {
      hoff = a.t.sub_hq[i] + loc;
      wo = a.t.sub_wq[i];
    } else {
      hoff = (int)(a.t.sub_H[i] - h0) + loc;
      wo = a.t.sub_slot[i] - s0;
    }
    be = a.beta[i];
    dr = a.d[g];
    if (owner) {
      // warm start: w^0 = beta z^0 - u^0, y^0 = beta z^0 + u^0
      const T z0 = a.z_in ? a.z_in[g] : (T)0;
      const T u0 = a.u_in ? a.u_in[g] : (T)0;
      w[wo + loc] = be * z0 - u0;
      y[r] = be * z0 + u0;
      u[r] = u0;
    }
  }
  // interface owned by this thread (waves hold one interface class when the map is given)
  const bool use_map = a.t.zmap && a.t.zmap_block == bd;
  const int code = use_map ? a.t.zmap[(long)sc * bd + tid] : i0 + tid;
  // a map entry is an interface, or one row of an interface whose rows are independent
  // (equality, hard and soft rows of one or two members): j | (row + 1) << kZRowShift
  const int j = code >= 0 ? (code & kZIfMask) : code;
  const int zrow = code >= 0 ? (code >> kZRowShift) - 1 : -1;
  const bool has_if = use_map ? j >= 0 : j < i1;
  int kind = 0, dim = 0, p0 = 0, p1 = 0, q0 = 0, q1 = 0, erow = 0;
  bool multi = false;
  T ib0 = (T)0, ib1 = (T)0, iws = (T)0, mu = (T)0, ksj = (T)0, asj = (T)0;
  // the scene's e rows are staged in LDS after u (read by the z-update with its y loads
  // rather than held in registers for the whole iteration)
  T* el = u + ns;
  const int row0 = a.t.if_row[i0];
  for (int q = tid; q < a.t.if_row[i1] - row0; q += bd) el[q] = a.e[row0 + q];
  const T* ev = el;
  // descriptors of the scene's interfaces of more than two members, after the e rows
  MultiDesc<T>* md = nullptr;
  __shared__ int n_multi;
  if constexpr (kMulti) {
    md = reinterpret_cast<MultiDesc<T>*>((reinterpret_cast<uintptr_t>(el + (a.t.if_row[i1] - row0)) + 15) & ~(uintptr_t)15);
    if (tid == 0) n_multi = 0;
    __syncthreads();
  }
  if (has_if) {
    kind = a.t.if_kind[j];
    dim = a.t.if_dim[j];
    multi = kMulti && a.t.if_nsub[j] > 2;
    const bool two = a.t.if_nsub[j] == 2;
    const int sa = a.t.if_sub0[j];
    const int sbb = two ? a.t.if_sub1[j] : sa;
    const int k0 = zrow >= 0 ? zrow : 0;  // first row of this lane's share
    if (zrow >= 0) dim = 1;
    p0 = a.t.if_slot0[j] - s0 + k0;
    p1 = two ? a.t.if_slot1[j] - s0 + k0 : p0;
    const int wa = kPadW ? a.t.sub_wq[sa] : a.t.sub_slot[sa] - s0;
    const int wb = kPadW ? a.t.sub_wq[sbb] : a.t.sub_slot[sbb] - s0;
    q0 = wa + (a.t.if_slot0[j] - a.t.sub_slot[sa]) + k0;
    q1 = two ? wb + (a.t.if_slot1[j] - a.t.sub_slot[sbb]) + k0 : q0;
    ib0 = (T)1 / a.beta[sa];
    ib1 = two ? (T)1 / a.beta[sbb] : (T)0;
    iws = (T)1 / (ib0 + ib1);
    mu = a.mu[j];
    ksj = a.ksoft[j];
    asj = a.asoft[j];
    erow = a.t.if_row[j] + k0;
    ev = el + (erow - row0);
    if constexpr (kMulti) {
      if (multi && a.multi_lds) {
        q1 = atomicAdd(&n_multi, 1);  // not used as a member's row here
        multi_desc<T, kPadW>(a, j, s0, md[q1]);
      }
    }
  }
  const T tol2 = (T)(a.tol * a.tol);
  // partials of absent waves stay zero, so that all eight are read as vectors
  if (tid < 16) red[tid >> 3][tid & 7] = (T)0;
  __syncthreads();

  int it = 0, conv = 0;
  T th = (T)0, yy = (T)0;
  for (int l = 0; l < a.max_iters; ++l) {
    it = l + 1;
    // x-update (Eq. 15 reassociated): x = d + H w; y = beta x + u (Eq. 18).
    T x = (T)0;
    if (in_slot) {
      if (kHInLds) {
        const int nq = (nc + V - 1) / V;
        const int cnt = (nq - part + kp - 1) / kp;
        x = row_dot_share<T, VT>(Hq + hoff + part * nc, reinterpret_cast<const VT*>(w + wo) + part, cnt, kp * nc,
                                 kp);
      } else {
        const T* Hr = a.H + h0 + hoff;
        const T* wr = w + wo;
        T acc[4] = {(T)0, (T)0, (T)0, (T)0};
        int c = part;
        for (; c + 3 * kLanes < nc; c += 4 * kLanes) {
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[k] += Hr[(c + k * kLanes) * nc] * wr[c + k * kLanes];
        }
        for (; c < nc; c += kLanes) acc[0] += Hr[c * nc] * wr[c];
        x = (acc[0] + acc[1]) + (acc[2] + acc[3]);
      }
    }
    if (kLanes == 2) x = pair_sum(x);
    if (kLanes == 0) {
      const T s2 = x + dpp_sel(x, 0);   // quad_perm [1,0,3,2]: the pair's sum
      const T s4 = s2 + dpp_sel(s2, 1);  // quad_perm [2,3,0,1]: the quad's sum
      x = kp == 1 ? x : kp == 2 ? s2 : s4;
    }
    T pth = (T)0, pyy = (T)0;
    if (owner) {
      // u[r] addressed from y's row (u = y + ns, ns scene-uniform), so that no second
      // per-lane address is held across the iteration
      const T yn = be * (dr + x) + y[r + ns];
      const T df = yn - y[r];
      pth = df * df;
      pyy = yn * yn;
      y[r] = yn;
    }
    // Residual of Eq. (22) and |y|^2, reduced in a fixed order.
    pth = wave_total_lane63(pth);
    pyy = wave_total_lane63(pyy);
    if (lane == 63) {
      // the wave index as a wave-uniform (scalar) value: the slot's address is formed anew
      // instead of being held in a vector register across the iteration
      const int sw = __builtin_amdgcn_readfirstlane(tid) >> 6;
      red[0][sw] = pth;
      red[1][sw] = pyy;
    }
    __syncthreads();
    {
      // the partials as 16-byte vectors (a few LDS reads per wave instead of sixteen)
      T tp[8], yp[8];
#pragma unroll
      for (int q = 0; q < 8; q += V) {
        const VT t4 = *reinterpret_cast<const VT*>(&red[0][q]);
        const VT y4 = *reinterpret_cast<const VT*>(&red[1][q]);
#pragma unroll
        for (int k = 0; k < V; ++k) {
          tp[q + k] = Vec16<T>::get(t4, k);
          yp[q + k] = Vec16<T>::get(y4, k);
        }
      }
      th = (T)0;
      yy = (T)0;
#pragma unroll
      for (int q = 0; q < 8; ++q) { th += tp[q]; yy += yp[q]; }
    }
    // r_theta = sqrt(theta)/max(|y|, 1e-12) <= tol, tested on squares
    if (!__builtin_isfinite((double)th) || !__builtin_isfinite((double)yy)) {
      if (tid == 0) atomicOr(a.flags, FLAG_NONFINITE);
      break;
    }
    if ((double)th <= (double)tol2 * ((double)yy > 1e-24 ? (double)yy : 1e-24)) { conv = 1; break; }
    if (l + 1 == a.max_iters) break;

    // z-update (Eq. 16-21) and dual update (Eq. 14): u = -lambda, w = y + 2 lambda.
    if (kMulti && has_if && multi) {
      if (!a.multi_lds)
        z_update_multi<T, kPadW>(a, j, s0, ev, y, u, w);
      else
        z_update_desc<T>(md[q1], kind, dim, a.contact_model, ev, y, u, w);
    } else if (has_if && kind == KIND_CONTACT) {
      z_update_fixed<T, 3, KIND_CONTACT>(ev, ib0, ib1, iws, mu, p0, p1, q0, q1, y, u, w, a.contact_model);
    } else if (has_if && kind == KIND_EQUALITY && dim == 5) {
      z_update_fixed<T, 5, KIND_EQUALITY>(ev, ib0, ib1, iws, mu, p0, p1, q0, q1, y, u, w, 0);
    } else if (has_if && kind == KIND_EQUALITY && dim == 1) {
      z_update_fixed<T, 1, KIND_EQUALITY>(ev, ib0, ib1, iws, mu, p0, p1, q0, q1, y, u, w, 0);
    } else if (has_if && kind == KIND_HARD_INEQ && dim == 1) {
      z_update_fixed<T, 1, KIND_HARD_INEQ>(ev, ib0, ib1, iws, mu, p0, p1, q0, q1, y, u, w, 0);
    } else if (has_if) {
      T ya[kMaxIfDim], yb[kMaxIfDim], p[kMaxIfDim], lam[kMaxIfDim];
#pragma unroll
      for (int k = 0; k < kMaxIfDim; ++k) {
        const int kk = k < dim ? k : 0;  // in-bounds address for unused rows
        ya[k] = y[p0 + kk];
        yb[k] = y[p1 + kk];
      }
      // soft (Eq. 20) or the p of Eq. 17-21 (ev holds the interface's rows in LDS)
#pragma unroll
      for (int k = 0; k < kMaxIfDim; ++k) {
        const T ek = k < dim ? ev[k] : (T)0;
        p[k] = kind == KIND_SOFT ? zsoft(ek, ya[k], ib0, yb[k], ib1, ksj, asj)
                                 : -zsum(ek, ya[k], ib0, yb[k], ib1) * iws;
      }
      // equality and soft: lambda = p; hard inequality: max(0, p); contact: Eq. (21)
      T cl[3];
      // written here, so that it is not carried from one iteration to the next in three registers
      if constexpr (kOutlined) cl[0] = cl[1] = cl[2] = (T)0;
      contact_project<T>(p, mu, cl, a.contact_model);
#pragma unroll
      for (int k = 0; k < kMaxIfDim; ++k) {
        T v = p[k];
        if (kind == KIND_HARD_INEQ) v = v > (T)0 ? v : (T)0;
        if (kind == KIND_CONTACT && k < 3) v = cl[k];
        lam[k] = v;
      }
#pragma unroll
      for (int k = 0; k < kMaxIfDim; ++k) {
        if (k < dim) {
          u[p0 + k] = -lam[k];
          w[q0 + k] = ya[k] + (T)2 * lam[k];
          if (p1 != p0) {
            u[p1 + k] = -lam[k];
            w[q1 + k] = yb[k] + (T)2 * lam[k];
          }
        }
      }
    }
    __syncthreads();
  }
  __syncthreads();

  // v_hat = c + G w (from the last x-update's w).
  const int d0 = a.t.sc_dof[sc], d1 = a.t.sc_dof[sc + 1];
  for (int dg = d0 + tid; dg < d1; dg += bd) {
    int i = sb;
    while (i + 1 < se && a.t.sub_dof[i + 1] <= dg) ++i;
    const int n = a.t.sub_n[i];
    const int rr = dg - a.t.sub_dof[i];
    const int nci = a.t.sub_nc[i];
    const int woi = kPadW ? a.t.sub_wq[i] : a.t.sub_slot[i] - s0;
    const T* G = a.G + a.t.sub_J[i] + rr;
    T v = a.cvec[dg];
    for (int c = 0; c < nci; ++c) v += G[c * n] * w[woi + c];
    if (a.v_hat) a.v_hat[dg] = v;
  }
  // final z^l, u^l and lambda = -u.
  if (owner) {
    a.z_out[s0 + r] = (w[wo + loc] + u[r]) / be;
    a.u_out[s0 + r] = u[r];
  }
  if (a.lambda && has_if) {
    for (int k = 0; k < dim; ++k) a.lambda[erow + k] = -u[p0 + k];
  }
  if (tid == 0) {
    const double yn = __builtin_sqrt((double)yy);
    a.st_iters[sc] = it;
    a.st_total[sc] += it;
    if (!conv) a.st_unconv[sc] += 1;
    if (a.st_fallback) a.st_fallback[sc] += 1;
    a.st_conv[sc] = conv;
    a.st_theta[sc] = (double)th;
    a.st_rtheta[sc] = __builtin_sqrt((double)th) / (yn > 1e-12 ? yn : 1e-12);
  }
}

template <typename T, int kHMode, int kLanes, bool kMulti>
__global__ void __launch_bounds__(512) loop_kernel(LoopArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ __align__(16) T red[2][8];
  loop_body<T, kHMode, kLanes, kMulti>(a, blockIdx.x, smem_raw, red);
}

// ------------------------------------------------------------------------------------
// Team form of the iteration (used when a scene's blocked H fits in LDS).  Every
// interface j owns a team of |S_j| d_j consecutive lanes inside one wave, one lane per
// member slot row (member 0's rows, then member 1's).  A lane computes its row's x and
// y (Eq. 15, 18); the team exchanges y with cross-lane shuffles and every lane of the
// team evaluates the interface's z-update (Eq. 16-21) and keeps its own row's dual
// u = -lambda (Eq. 14) in a register.  Only w = beta z - u is shared through LDS; it is
// double buffered by iteration parity, so the z-update of iteration l proceeds while
// the residual of iteration l is still being reduced, and one barrier per iteration
// serves both.  When the residual test stops the iteration at l, the z-update of l is
// discarded: v_hat uses the w buffer of iteration l and the kept u.
// ------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(512) team_loop_kernel(LoopArgs<T> a) {
  using VT = typename Vec16<T>::type;
  constexpr int V = Vec16<T>::N;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ T red[2][2][8];
  const int sc = blockIdx.x;
  const int tid = threadIdx.x;
  const int bd = blockDim.x;
  const int nwave = bd >> 6;
  const int lane = tid & 63, wv = tid >> 6;
  if (a.skip_converged && a.skip_converged[sc]) return;
  const int s0 = a.t.sc_slot[sc];
  const int sb = a.t.sc_sub[sc], se = a.t.sc_sub[sc + 1];
  const int nhq = a.t.sc_hq[sc];
  const int nwq = a.t.sc_wq[sc];
  VT* Hq = reinterpret_cast<VT*>(smem_raw);
  T* wbuf0 = reinterpret_cast<T*>(Hq + nhq);
  T* wbuf1 = wbuf0 + nwq;

  for (int i = sb; i < se; ++i) {
    const int nci = a.t.sub_nc[i];
    const int nq = (nci + V - 1) / V;
    const T* Hg = a.H + a.t.sub_H[i];
    VT* dst = Hq + a.t.sub_hq[i];
    for (int q = tid; q < nq * nci; q += bd) {
      const int cb = q / nci, rr = q - cb * nci;
      T v[V];
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const int c = cb * V + k;
        v[k] = c < nci ? Hg[c * nci + rr] : (T)0;
      }
      dst[q] = Vec16<T>::make(v);
    }
  }
  for (int q = tid; q < 2 * nwq; q += bd) wbuf0[q] = (T)0;
  __syncthreads();

  // lane role
  const int code = a.t.lane_code[(size_t)sc * bd + tid];
  const bool act = code >= 0;
  const int j = act ? (code >> 4) : a.t.sc_if[sc];
  const int pos = act ? (code & 15) : 0;
  int kind = 0, dim = 1, two = 0, mem = 0, k_me = 0, nc = 0, hoff = 0, wo = 0, loc = 0, g = 0;
  T ib0 = (T)0, ib1 = (T)0, iws = (T)0, mu = (T)0, be = (T)1, dr = (T)0, ksj = (T)0, asj = (T)0;
  T ev[kMaxIfDim];
#pragma unroll
  for (int k = 0; k < kMaxIfDim; ++k) ev[k] = (T)0;
  T u_cur = (T)0, y_cur = (T)0;
  if (act) {
    kind = a.t.if_kind[j];
    dim = a.t.if_dim[j];
    two = a.t.if_nsub[j] == 2;
    mem = pos / dim;
    k_me = pos - mem * dim;
    const int sa = a.t.if_sub0[j];
    const int sbb = two ? a.t.if_sub1[j] : sa;
    const int i = mem ? sbb : sa;
    g = (mem ? a.t.if_slot1[j] : a.t.if_slot0[j]) + k_me;
    nc = a.t.sub_nc[i];
    loc = g - a.t.sub_slot[i];
    hoff = a.t.sub_hq[i] + loc;
    wo = a.t.sub_wq[i];
    be = a.beta[i];
    dr = a.d[g];
    ib0 = (T)1 / a.beta[sa];
    ib1 = two ? (T)1 / a.beta[sbb] : (T)0;
    iws = (T)1 / (ib0 + ib1);
    mu = a.mu[j];
    ksj = a.ksoft[j];
    asj = a.asoft[j];
#pragma unroll
    for (int k = 0; k < kMaxIfDim; ++k)
      if (k < dim) ev[k] = a.e[a.t.if_row[j] + k];
    // warm start: w^0 = beta z^0 - u^0, y^0 = beta z^0 + u^0
    const T z0 = a.z_in ? a.z_in[g] : (T)0;
    const T u0 = a.u_in ? a.u_in[g] : (T)0;
    u_cur = u0;
    y_cur = be * z0 + u0;
    wbuf0[wo + loc] = be * z0 - u0;
  }
  const int base = lane - pos;               // first lane of the team in this wave
  const int off_b = two ? dim : 0;           // member 1's rows follow member 0's
  const int nq = (nc + V - 1) / V;
  const T tol2 = (T)(a.tol * a.tol);
  __syncthreads();

  int it = 0, conv = 0;
  T th = (T)0, yy = (T)0;
  for (int l = 0; l < a.max_iters; ++l) {
    it = l + 1;
    const T* wc = (l & 1) ? wbuf1 : wbuf0;
    T* wn = (l & 1) ? wbuf0 : wbuf1;
    // x-update (Eq. 15 reassociated): x = d + H w, then y = beta x + u (Eq. 18)
    const T xr = row_dot_share<T, VT>(Hq + hoff, reinterpret_cast<const VT*>(wc + wo), nq, nc, 1);
    const T yn = be * (dr + xr) + u_cur;
    const T df = yn - y_cur;
    T pth = act ? df * df : (T)0;
    T pyy = act ? yn * yn : (T)0;

    // z-update of the lane's interface from the team's y (Eq. 16-21); ib1 = 0 for a
    // one-member interface, whose second shuffle then reads the first member again
    T p[kMaxIfDim];
#pragma unroll
    for (int k = 0; k < kMaxIfDim; ++k) {
      const int kk = k < dim ? k : 0;
      const T ya = __shfl(yn, base + kk, 64);
      const T yb = __shfl(yn, base + off_b + kk, 64);
      p[k] = kind == KIND_SOFT ? zsoft(ev[k], ya, ib0, yb, ib1, ksj, asj) : -zsum(ev[k], ya, ib0, yb, ib1) * iws;
    }
    T cl[3];
    contact_project<T>(p, mu, cl, a.contact_model);
    T lam_me = (T)0;
#pragma unroll
    for (int k = 0; k < kMaxIfDim; ++k) {
      T v = p[k];
      if (kind == KIND_HARD_INEQ) v = v > (T)0 ? v : (T)0;
      if (kind == KIND_CONTACT && k < 3) v = cl[k];
      if (k == k_me) lam_me = v;
    }
    if (act) wn[wo + loc] = yn + (T)2 * lam_me;  // w = beta z - u with u = -lambda

    // residual of Eq. (22) and |y|^2 of this x-update, reduced in a fixed order
    pth = wave_total_lane63(pth);
    pyy = wave_total_lane63(pyy);
    if (lane == 63) { red[l & 1][0][wv] = pth; red[l & 1][1][wv] = pyy; }
    __syncthreads();
    {
      T tp[8], yp[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        tp[q] = q < nwave ? red[l & 1][0][q] : (T)0;
        yp[q] = q < nwave ? red[l & 1][1][q] : (T)0;
      }
      th = (T)0;
      yy = (T)0;
#pragma unroll
      for (int q = 0; q < 8; ++q) { th += tp[q]; yy += yp[q]; }
    }
    y_cur = yn;
    if (!__builtin_isfinite((double)th) || !__builtin_isfinite((double)yy)) {
      if (tid == 0) atomicOr(a.flags, FLAG_NONFINITE);
      break;
    }
    // r_theta = sqrt(theta)/max(|y|, 1e-12) <= tol, tested on squares
    if ((double)th <= (double)tol2 * ((double)yy > 1e-24 ? (double)yy : 1e-24)) { conv = 1; break; }
    if (l + 1 == a.max_iters) break;
    u_cur = -lam_me;
  }
  __syncthreads();

  // v_hat = c + G w with the w of the last x-update
  const T* wf = ((it - 1) & 1) ? wbuf1 : wbuf0;
  const int d0 = a.t.sc_dof[sc], d1 = a.t.sc_dof[sc + 1];
  for (int dg = d0 + tid; dg < d1; dg += bd) {
    int i = sb;
    while (i + 1 < se && a.t.sub_dof[i + 1] <= dg) ++i;
    const int n = a.t.sub_n[i];
    const int rr = dg - a.t.sub_dof[i];
    const int nci = a.t.sub_nc[i];
    const T* G = a.G + a.t.sub_J[i] + rr;
    const T* wi = wf + a.t.sub_wq[i];
    T v = a.cvec[dg];
    for (int c = 0; c < nci; ++c) v += G[c * n] * wi[c];
    if (a.v_hat) a.v_hat[dg] = v;
  }
  if (act) {
    a.z_out[g] = (wf[wo + loc] + u_cur) / be;
    a.u_out[g] = u_cur;
    if (a.lambda && mem == 0) a.lambda[a.t.if_row[j] + k_me] = -u_cur;
  }
  if (tid == 0) {
    const double yn2 = __builtin_sqrt((double)yy);
    a.st_iters[sc] = it;
    a.st_total[sc] += it;
    if (!conv) a.st_unconv[sc] += 1;
    if (a.st_fallback) a.st_fallback[sc] += 1;
    a.st_conv[sc] = conv;
    a.st_theta[sc] = (double)th;
    a.st_rtheta[sc] = __builtin_sqrt((double)th) / (yn2 > 1e-12 ? yn2 : 1e-12);
  }
  (void)s0;
}

// ------------------------------------------------------------------------------------
// Wave form of the iteration: one wave per scene and no workgroup barrier.  Lane l owns
// the slot rows l, l + 64, ... (at most kWaveRows of them) and the scene's interface l.
// The LDS layout is the blocked one of loop_kernel; a wave's LDS operations complete in
// the order it issues them, so fences that keep the compiler from moving LDS accesses
// across them order the x-update's y stores before the z-update's loads and the
// z-update's u, w stores before the next x-update.  The residual is one DPP wave sum,
// read by every lane from lane 63.  Per row and per interface the arithmetic is the one
// of loop_kernel with one lane per row.
// ------------------------------------------------------------------------------------
constexpr int kWaveRows = 4;

__device__ inline float bcast_lane63(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ inline double bcast_lane63(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), 63);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned int)hi << 32) | (unsigned int)lo));
}

template <typename T>
__global__ void __launch_bounds__(64) wave_loop_kernel(LoopArgs<T> a) {
  using VT = typename Vec16<T>::type;
  constexpr int V = Vec16<T>::N;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int sc = blockIdx.x;
  const int lane = threadIdx.x;
  if (a.skip_converged && a.skip_converged[sc]) return;
  const int s0 = a.t.sc_slot[sc], s1 = a.t.sc_slot[sc + 1];
  const int ns = s1 - s0;
  const int i0 = a.t.sc_if[sc], i1 = a.t.sc_if[sc + 1];
  const int sb = a.t.sc_sub[sc], se = a.t.sc_sub[sc + 1];
  const int nhq = a.t.sc_hq[sc];
  const int nwq = a.t.sc_wq[sc];
  VT* Hq = reinterpret_cast<VT*>(smem_raw);
  T* w = reinterpret_cast<T*>(Hq + nhq);  // padded per-subsystem blocks
  T* y = w + nwq;
  T* u = y + ns;

  // stage H_i into the blocked layout and clear the padded w area
  for (int i = sb; i < se; ++i) {
    const int nci = a.t.sub_nc[i];
    const int nq = (nci + V - 1) / V;
    const T* Hg = a.H + a.t.sub_H[i];
    VT* dst = Hq + a.t.sub_hq[i];
    for (int q = lane; q < nq * nci; q += 64) {
      const int cb = q / nci, rr = q - cb * nci;
      T v[V];
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const int c = cb * V + k;
        v[k] = c < nci ? Hg[c * nci + rr] : (T)0;
      }
      dst[q] = Vec16<T>::make(v);
    }
  }
  for (int q = lane; q < nwq; q += 64) w[q] = (T)0;
  wave_lds_fence();

  // the lane's slot rows
  int nc[kWaveRows], hoff[kWaveRows], wo[kWaveRows], loc[kWaveRows];
  T be[kWaveRows], dr[kWaveRows];
#pragma unroll
  for (int q = 0; q < kWaveRows; ++q) {
    const int r = lane + 64 * q;
    nc[q] = 0;
    hoff[q] = 0;
    wo[q] = 0;
    loc[q] = 0;
    be[q] = (T)1;
    dr[q] = (T)0;
    if (r < ns) {
      const int g = s0 + r;
      const int i = a.t.slot_sub[g];
      nc[q] = a.t.sub_nc[i];
      loc[q] = a.t.slot_loc[g];
      hoff[q] = a.t.sub_hq[i] + loc[q];
      wo[q] = a.t.sub_wq[i];
      be[q] = a.beta[i];
      dr[q] = a.d[g];
      // warm start: w^0 = beta z^0 - u^0, y^0 = beta z^0 + u^0
      const T z0 = a.z_in ? a.z_in[g] : (T)0;
      const T u0 = a.u_in ? a.u_in[g] : (T)0;
      w[wo[q] + loc[q]] = be[q] * z0 - u0;
      y[r] = be[q] * z0 + u0;
      u[r] = u0;
    }
  }
  // the lane's interface
  const int j = i0 + lane;
  const bool has_if = j < i1;
  int kind = 0, dim = 0, p0 = 0, p1 = 0, q0 = 0, q1 = 0;
  T ib0 = (T)0, ib1 = (T)0, iws = (T)0, mu = (T)0, ksj = (T)0, asj = (T)0;
  T ev[kMaxIfDim];
#pragma unroll
  for (int k = 0; k < kMaxIfDim; ++k) ev[k] = (T)0;
  if (has_if) {
    kind = a.t.if_kind[j];
    dim = a.t.if_dim[j];
    const bool two = a.t.if_nsub[j] == 2;
    const int sa = a.t.if_sub0[j];
    const int sbb = two ? a.t.if_sub1[j] : sa;
    p0 = a.t.if_slot0[j] - s0;
    p1 = two ? a.t.if_slot1[j] - s0 : p0;
    q0 = a.t.sub_wq[sa] + (a.t.if_slot0[j] - a.t.sub_slot[sa]);
    q1 = two ? a.t.sub_wq[sbb] + (a.t.if_slot1[j] - a.t.sub_slot[sbb]) : q0;
    ib0 = (T)1 / a.beta[sa];
    ib1 = two ? (T)1 / a.beta[sbb] : (T)0;
    iws = (T)1 / (ib0 + ib1);
    mu = a.mu[j];
    ksj = a.ksoft[j];
    asj = a.asoft[j];
#pragma unroll
    for (int k = 0; k < kMaxIfDim; ++k)
      if (k < dim) ev[k] = a.e[a.t.if_row[j] + k];
  }
  const T tol2 = (T)(a.tol * a.tol);
  wave_lds_fence();

  int it = 0, conv = 0;
  T th = (T)0, yy = (T)0;
  for (int l = 0; l < a.max_iters; ++l) {
    it = l + 1;
    // x-update (Eq. 15 reassociated) and y = beta x + u (Eq. 18) for the lane's rows
    T pth = (T)0, pyy = (T)0;
#pragma unroll
    for (int q = 0; q < kWaveRows; ++q) {
      const int r = lane + 64 * q;
      if (r < ns) {
        const int nq = (nc[q] + V - 1) / V;
        const T x = row_dot_share<T, VT>(Hq + hoff[q], reinterpret_cast<const VT*>(w + wo[q]), nq, nc[q], 1);
        const T yn = be[q] * (dr[q] + x) + u[r];
        const T df = yn - y[r];
        pth += df * df;
        pyy += yn * yn;
        y[r] = yn;
      }
    }
    // residual of Eq. (22) and |y|^2: one wave sum, the same value in every lane
    th = bcast_lane63(wave_total_lane63(pth));
    yy = bcast_lane63(wave_total_lane63(pyy));
    if (!__builtin_isfinite((double)th) || !__builtin_isfinite((double)yy)) {
      if (lane == 0) atomicOr(a.flags, FLAG_NONFINITE);
      break;
    }
    if ((double)th <= (double)tol2 * ((double)yy > 1e-24 ? (double)yy : 1e-24)) { conv = 1; break; }
    if (l + 1 == a.max_iters) break;
    wave_lds_fence();

    // z-update (Eq. 16-21) and dual update (Eq. 14): u = -lambda, w = y + 2 lambda
    if (has_if) {
      T ya[kMaxIfDim], yb[kMaxIfDim], p[kMaxIfDim], lam[kMaxIfDim];
#pragma unroll
      for (int k = 0; k < kMaxIfDim; ++k) {
        const int kk = k < dim ? k : 0;  // in-bounds address for unused rows
        ya[k] = y[p0 + kk];
        yb[k] = y[p1 + kk];
      }
#pragma unroll
      for (int k = 0; k < kMaxIfDim; ++k)
        p[k] = kind == KIND_SOFT ? zsoft(ev[k], ya[k], ib0, yb[k], ib1, ksj, asj)
                                 : -zsum(ev[k], ya[k], ib0, yb[k], ib1) * iws;
      T cl[3];
      contact_project<T>(p, mu, cl, a.contact_model);
#pragma unroll
      for (int k = 0; k < kMaxIfDim; ++k) {
        T v = p[k];
        if (kind == KIND_HARD_INEQ) v = v > (T)0 ? v : (T)0;
        if (kind == KIND_CONTACT && k < 3) v = cl[k];
        lam[k] = v;
      }
#pragma unroll
      for (int k = 0; k < kMaxIfDim; ++k) {
        if (k < dim) {
          u[p0 + k] = -lam[k];
          w[q0 + k] = ya[k] + (T)2 * lam[k];
          if (p1 != p0) {
            u[p1 + k] = -lam[k];
            w[q1 + k] = yb[k] + (T)2 * lam[k];
          }
        }
      }
    }
    wave_lds_fence();
  }
  wave_lds_fence();

  // v_hat = c + G w (from the last x-update's w).
  const int d0 = a.t.sc_dof[sc], d1 = a.t.sc_dof[sc + 1];
  for (int dg = d0 + lane; dg < d1; dg += 64) {
    int i = sb;
    while (i + 1 < se && a.t.sub_dof[i + 1] <= dg) ++i;
    const int n = a.t.sub_n[i];
    const int rr = dg - a.t.sub_dof[i];
    const int nci = a.t.sub_nc[i];
    const int woi = a.t.sub_wq[i];
    const T* G = a.G + a.t.sub_J[i] + rr;
    T v = a.cvec[dg];
    for (int c = 0; c < nci; ++c) v += G[c * n] * w[woi + c];
    if (a.v_hat) a.v_hat[dg] = v;
  }
  // final z^l, u^l and lambda = -u.
#pragma unroll
  for (int q = 0; q < kWaveRows; ++q) {
    const int r = lane + 64 * q;
    if (r < ns) {
      a.z_out[s0 + r] = (w[wo[q] + loc[q]] + u[r]) / be[q];
      a.u_out[s0 + r] = u[r];
    }
  }
  if (a.lambda && has_if) {
    for (int k = 0; k < dim; ++k) a.lambda[a.t.if_row[j] + k] = -u[p0 + k];
  }
  if (lane == 0) {
    const double yn = __builtin_sqrt((double)yy);
    a.st_iters[sc] = it;
    a.st_total[sc] += it;
    if (!conv) a.st_unconv[sc] += 1;
    if (a.st_fallback) a.st_fallback[sc] += 1;
    a.st_conv[sc] = conv;
    a.st_theta[sc] = (double)th;
    a.st_rtheta[sc] = __builtin_sqrt((double)th) / (yn > 1e-12 ? yn : 1e-12);
  }
}

template <typename T>
hipError_t launch_wave_loop(const LoopArgs<T>& a, int max_slot_scene, int max_if_scene, int max_hq_scene,
                            int max_wq_scene, hipStream_t s) {
  if (a.t.n_scene == 0) return hipSuccess;
  if (max_slot_scene > 64 * kWaveRows || max_if_scene > 64) return hipErrorInvalidValue;
  const int ns = max_slot_scene > 0 ? max_slot_scene : 1;
  const size_t lds = 16 * (size_t)max_hq_scene + sizeof(T) * ((size_t)max_wq_scene + 2 * (size_t)ns) + 64;
  if (lds > 150 * 1024) return hipErrorInvalidValue;
  hipLaunchKernelGGL(wave_loop_kernel<T>, dim3(a.t.n_scene), dim3(64), lds, s, a);
  return hipGetLastError();
}
template hipError_t launch_wave_loop<float>(const LoopArgs<float>&, int, int, int, int, hipStream_t);
template hipError_t launch_wave_loop<double>(const LoopArgs<double>&, int, int, int, int, hipStream_t);

template <typename T>
hipError_t launch_team_loop(const LoopArgs<T>& a, int max_hq_scene, int max_wq_scene, hipStream_t s) {
  if (a.t.n_scene == 0) return hipSuccess;
  const int threads = a.t.team_block;
  if (threads < 64 || threads > 512 || threads % 64) return hipErrorInvalidValue;
  const size_t lds = 16 * (size_t)max_hq_scene + sizeof(T) * 2 * (size_t)max_wq_scene + 64;
  if (lds > 150 * 1024) return hipErrorInvalidValue;
  hipLaunchKernelGGL(team_loop_kernel<T>, dim3(a.t.n_scene), dim3(threads), lds, s, a);
  return hipGetLastError();
}

template hipError_t launch_team_loop<float>(const LoopArgs<float>&, int, int, hipStream_t);
template hipError_t launch_team_loop<double>(const LoopArgs<double>&, int, int, hipStream_t);

template <typename T>
hipError_t launch_factor(const FactorArgs<T>& a, int count, int max_n, int max_nc, bool fp64, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const size_t cs = fp64 ? sizeof(double) : sizeof(T);
  const size_t lds = factor_bytes(max_n, max_nc, cs);
  if (lds > 160 * 1024 - 1024) return hipErrorInvalidValue;
  // a class of small subsystems: one wave each, four per workgroup
  const size_t slice = (lds + 15) / 16 * 16;
  if (wave_factor_fits(max_n, max_nc, cs, kWaveFactorSlice) && slice <= kWaveFactorSlice) {
    const int blocks = (count + 3) / 4;
    if (fp64)
      hipLaunchKernelGGL((factor_wave_kernel<T, double>), dim3(blocks), dim3(256), 4 * slice, s, a, count, (int)slice);
    else
      hipLaunchKernelGGL((factor_wave_kernel<T, T>), dim3(blocks), dim3(256), 4 * slice, s, a, count, (int)slice);
    return hipGetLastError();
  }
  // a class of few subsystems (the largest ones) is latency-bound: give each more threads; so
  // are subsystems of more DOFs than that, whose LDS leaves room for one workgroup per CU
  int threads = count < 256 ? 512 : count < 2048 ? 256 : 128;
  if (max_n > kMaxFactorDof) return hipErrorInvalidValue;
  while (threads < max_n - 1) threads *= 2;
  if (fp64)
    hipLaunchKernelGGL((factor_kernel<T, double>), dim3(count), dim3(threads), lds, s, a);
  else
    hipLaunchKernelGGL((factor_kernel<T, T>), dim3(count), dim3(threads), lds, s, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_factor_global(const FactorArgs<T>& a, int count, int max_n, bool fp64, char* scr, const int64_t* off,
                                hipStream_t s) {
  if (count == 0) return hipSuccess;
  if (max_n > kMaxFactorDof) return hipErrorInvalidValue;
  if (fp64)
    hipLaunchKernelGGL((factor_global_kernel<T, double>), dim3(count), dim3(kBigThreads), 0, s, a, scr, off);
  else
    hipLaunchKernelGGL((factor_global_kernel<T, T>), dim3(count), dim3(kBigThreads), 0, s, a, scr, off);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_loop(const LoopArgs<T>& a, int max_slot_scene, int max_if_scene, long long max_h_scene,
                       int max_hq_scene, int max_wq_scene, int max_nc, hipStream_t s) {
  (void)max_h_scene;
  if (a.t.n_scene == 0) return hipSuccess;
  const int ns = max_slot_scene > 0 ? max_slot_scene : 1;
  // two lanes per slot row while the block stays within 4 waves (so that four or more
  // scenes stay resident per CU), else one
  const bool two = 2 * ns <= kTwoLaneMax && max_if_scene <= kTwoLaneMax;
  const int need = two ? (2 * ns > max_if_scene ? 2 * ns : max_if_scene) : (ns > max_if_scene ? ns : max_if_scene);
  const int threads = (need + 63) / 64 * 64;
  if (threads > 512) return hipErrorInvalidValue;
  const size_t rows = (size_t)a.t.max_row_scene;  // the scene's e rows, staged after u
  const size_t slots = sizeof(T) * (3 * (size_t)ns + rows);
  const size_t with_h = 16 * (size_t)max_hq_scene + sizeof(T) * ((size_t)max_wq_scene + 2 * (size_t)ns + rows) + 64;
  const bool hl = with_h <= 150 * 1024;
  (void)max_nc;
  if (!hl && slots > 150 * 1024) return hipErrorInvalidValue;
  const auto go = [&](auto multi) -> hipError_t {
    constexpr bool kMulti = decltype(multi)::value;
    LoopArgs<T> b = a;
    size_t lds = hl ? with_h : slots;
    if constexpr (kMulti) {
      // descriptors in LDS where they still fit beside the rest; in the last 64-96 bytes per
      // interface below the limit the operators keep LDS and the topology is read each iteration
      const size_t more = sizeof(MultiDesc<T>) * (size_t)a.t.max_multi_scene + 16;
      b.multi_lds = lds + more <= 150 * 1024 ? 1 : 0;
      if (b.multi_lds) lds += more;
    }
    const dim3 grid(a.t.n_scene);
    if (hl && a.t.rmap && a.t.rmap_block <= 512) {
      hipLaunchKernelGGL((loop_kernel<T, kHLds, 0, kMulti>), grid, dim3(a.t.rmap_block), lds, s, b);
    } else if (hl && two) {
      hipLaunchKernelGGL((loop_kernel<T, kHLds, 2, kMulti>), grid, dim3(threads), lds, s, b);
    } else if (hl) {
      hipLaunchKernelGGL((loop_kernel<T, kHLds, 1, kMulti>), grid, dim3(threads), lds, s, b);
    } else if (two) {
      hipLaunchKernelGGL((loop_kernel<T, kHGlobal, 2, kMulti>), grid, dim3(threads), lds, s, b);
    } else {
      hipLaunchKernelGGL((loop_kernel<T, kHGlobal, 1, kMulti>), grid, dim3(threads), lds, s, b);
    }
    return hipGetLastError();
  };
  return a.t.max_multi_scene > 0 ? go(std::true_type{}) : go(std::false_type{});
}

// ------------------------------------------------------------------------------------
// Several whole time steps per launch (Alg. 1 repeated), one workgroup per scene: the
// construction of the scene's subsystems, their factorisations one after another, the
// iteration, and the state update of its bodies, then the next step.  A scene does not
// wait for the others between steps, so the launch lasts as long as the largest sum of
// iterations over the steps of one scene rather than the sum over steps of the largest
// per-step count.  Every phase is the per-step kernels' code; the barriers between phases
// order the global-memory writes and reads of the workgroup.
// ------------------------------------------------------------------------------------
// The phases read their arguments through the argument block in device memory, and the
// block's address passes through an empty asm statement at the start of each phase: the
// compiler cannot move a phase's argument loads into another phase, so no phase keeps the
// others' arguments live in registers.
template <typename T>
__device__ __attribute__((always_inline)) inline const StepsArgs<T>* phase_args(const StepsArgs<T>* p) {
  uint64_t v = reinterpret_cast<uint64_t>(p);
  asm volatile("" : "+s"(v));
  return reinterpret_cast<const StepsArgs<T>*>(v);
}

// The factorisations and the iteration called out of line, so that each has its own registers:
// with the factorisations inlined their diagonal tiles' rows cost the iteration spills (512 legged
// scenes, two steps: 3.55 ms before the matrix-core form, 3.71 with it inlined), and with the
// iteration inlined beside the calls it read 5 to 9 spilled registers per iteration in FP64 and
// any change of a factorisation moved its spills (FP64 chain of 8 links, 100 steps: 345 us a step
// before the matrix-core factorisation, 356 with the iteration inlined, 290 now; FP32 240 either
// way, two steps of 512 legged scenes 3.32 ms either way).  The LDS area is passed as its LDS offset, so that it is addressed directly.
template <typename T, typename C>
__device__ __attribute__((noinline)) void factor_wave_outlined(const FactorArgs<T>& a, const int i, const uint32_t lds) {
  __shared__ int bad[4];
  factor_body<T, C, GroupWave>(a, i, (__attribute__((address_space(3))) C*)lds, nullptr, bad[threadIdx.x >> 6]);
}
template <typename T, typename C>
__device__ __attribute__((noinline)) void factor_lds_outlined(const FactorArgs<T>& a, const int i, const uint32_t lds) {
  __shared__ double red[2][16];
  __shared__ int bad;
  factor_body<T, C, GroupWg>(a, i, (__attribute__((address_space(3))) C*)lds, red, bad);
}
template <typename T, typename C>
__device__ __attribute__((noinline)) void factor_global_outlined(const FactorArgs<T>& a, const int i, C* scr) {
  __shared__ double red[2][16];
  __shared__ int bad;
  factor_body<T, C, GroupWg>(a, i, scr, red, bad);
}

template <typename T, int kLanes>
__device__ __attribute__((noinline)) void loop_outlined(const LoopArgs<T>& a, const int sc, const uint32_t lds) {
  __shared__ __align__(16) T red[2][8];
  loop_body<T, kHLds, kLanes, false, true>(a, sc, (unsigned char*)(__attribute__((address_space(3))) unsigned char*)lds, red);
}

template <typename T, typename C, int kLanes>
__global__ void __launch_bounds__(256, 4) steps_kernel(const StepsArgs<T>* __restrict__ ap) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
  // workgroups are dispatched round-robin over the XCDs and their CUs in block order, so the
  // order decides which scenes share a CU
  const int sc = ap->sc_order[blockIdx.x];
  const int n_steps = ap->n_steps;
  const int tid = threadIdx.x, bd = blockDim.x;
  for (int step = 0; step < n_steps; ++step) {
    {
      // construction (Eq. 2-5) of the scene's subsystems at once: disjoint blocks of A, b, J
      // and rows of e
      const StepsArgs<T>& a = *phase_args(ap);
      const int sb = a.l.t.sc_sub[sc], se = a.l.t.sc_sub[sc + 1];
      rigid_assemble_scene<T, true>(a.l.t, a.m, sb, se, a.st.pos, a.st.rot, a.st.vel, a.st.omega, a.dt, a.A, a.b,
                                    a.J, a.e);
    }
    __syncthreads();
    {
      // penalty (Eq. 23) and factorisation per subsystem: the small subsystems one per wave,
      // the waves taking them in turn, each in its share of the LDS; then the others with the
      // whole workgroup, in LDS when they fit
      const StepsArgs<T>& a = *phase_args(ap);
      const int sb = a.l.t.sc_sub[sc], se = a.l.t.sc_sub[sc + 1];
      const int nwave = bd >> 6, wv = tid >> 6;
      const size_t slice = (size_t)a.lds_factor / (size_t)nwave / 16 * 16;
      int k = 0;
      for (int i = sb; i < se; ++i) {
        if (!wave_factor_fits(a.l.t.sub_n[i], a.l.t.sub_nc[i], sizeof(C), slice)) continue;
        if (k++ % nwave == wv)
          factor_wave_outlined<T, C>(a.f, i, lds0 + (uint32_t)(wv * slice));
      }
      __syncthreads();
      for (int i = sb; i < se; ++i) {
        if (wave_factor_fits(a.l.t.sub_n[i], a.l.t.sub_nc[i], sizeof(C), slice)) continue;
        if (factor_bytes(a.l.t.sub_n[i], a.l.t.sub_nc[i], sizeof(C)) <= (size_t)a.lds_factor)
          factor_lds_outlined<T, C>(a.f, i, lds0);
        else
          factor_global_outlined<T, C>(a.f, i, reinterpret_cast<C*>(a.fscr + a.sc_fscr[sc]));
        __syncthreads();
      }
    }
    // the iteration (Eq. 15-22, 14) from the previous step's values or cold
    loop_outlined<T, kLanes>(phase_args(ap)->l, sc, lds0);
    __syncthreads();
    {
      // state update (Eq. 2)
      const StepsArgs<T>& a = *phase_args(ap);
      const int sb = a.l.t.sc_sub[sc], se = a.l.t.sc_sub[sc + 1];
      for (int q = a.m.sub_body_off[sb] + tid; q < a.m.sub_body_off[se]; q += bd)
        rigid_advance_body<T>(a.l.t, a.m, a.st, a.l.v_hat, a.dt, a.m.sub_body[q]);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------
// Scenes too large for one workgroup (Alg. 1 over the whole problem): one launch per phase
// of each iteration.  x-update (Eq. 15, 18) one thread per slot row with the operators in
// device memory; residual (Eq. 22) and stopping test one workgroup per scene, summing the
// slot rows of the scene in a fixed order; z-update (Eq. 16-21) and dual update (Eq. 14) one
// thread per interface.  A scene that stops keeps its values: the later launches skip it.
// Same iteration as the per-scene kernel (u = -lambda, w = y + 2 lambda kept per slot row).
// ------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) large_init_kernel(LargeArgs<T> a) {
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const LoopArgs<T>& l = a.l;
  if (g < l.t.n_scene) a.done[g] = 0;
  if (g >= a.n_slot) return;
  const T be = l.beta[l.t.slot_sub[g]];
  const T z0 = l.z_in ? l.z_in[g] : (T)0;
  const T u0 = l.u_in ? l.u_in[g] : (T)0;
  a.w[g] = be * z0 - u0;
  a.y[g] = be * z0 + u0;
  a.u[g] = u0;
}

// x-update of slot row g (Eq. 15 reassociated, y = beta x + u) with its residual terms (kSquare
// false: the terms before they are squared)
template <typename T, bool kSquare = true>
__device__ inline void large_xupdate_row(const LargeArgs<T>& a, const long g) {
  const LoopArgs<T>& l = a.l;
  const int i = l.t.slot_sub[g];
  const int nc = l.t.sub_nc[i], loc = l.t.slot_loc[g];
  const T* H = l.H + l.t.sub_H[i] + loc;  // column-major: H_i[loc][c] at c * nc + loc
  const T* w = a.w + l.t.sub_slot[i];
  T acc[4] = {(T)0, (T)0, (T)0, (T)0};
  int c = 0;
  for (; c + 3 < nc; c += 4) {
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] += H[(long)(c + k) * nc] * w[c + k];
  }
  for (; c < nc; ++c) acc[0] += H[(long)c * nc] * w[c];
  const T x = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  const T yn = l.beta[i] * (l.d[g] + x) + a.u[g];
  const double df = (double)yn - (double)a.y[g];
  a.dy2[g] = kSquare ? df * df : df;
  a.yy2[g] = kSquare ? (double)yn * (double)yn : (double)yn;
  a.y[g] = yn;
}

template <typename T>
__global__ void __launch_bounds__(256) large_xupdate_kernel(LargeArgs<T> a) {
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= a.n_slot) return;
  if (a.done[a.sub_scene[a.l.t.slot_sub[g]]]) return;
  large_xupdate_row<T>(a, g);
}

// The stopping test of scene sc from its sums of Eq. 22; writes the statistics and the scene's
// stop flag; returns whether the scene stopped.
template <typename T>
__device__ inline int large_decide(const LargeArgs<T>& a, const int sc, const int l_iter, const double th,
                                   const double yy) {
  const LoopArgs<T>& l = a.l;
  const int it = l_iter + 1;
  const bool bad = !__builtin_isfinite(th) || !__builtin_isfinite(yy);
  const bool cv = !bad && th <= l.tol * l.tol * (yy > 1e-24 ? yy : 1e-24);
  if (bad) atomicOr(l.flags, FLAG_NONFINITE);
  const bool stop = cv || bad || it == l.max_iters;
  if (stop) {
    a.done[sc] = 1;
    const double yn = __builtin_sqrt(yy);
    l.st_iters[sc] = it;
    l.st_total[sc] += it;
    if (!cv) l.st_unconv[sc] += 1;
    l.st_conv[sc] = cv ? 1 : 0;
    l.st_theta[sc] = th;
    l.st_rtheta[sc] = __builtin_sqrt(th) / (yn > 1e-12 ? yn : 1e-12);
  }
  return stop ? 1 : 0;
}

// Residual of Eq. 22 of scene sc by the first 256 threads of its workgroup (threads take
// rows tid, tid + 256, ...; waves summed in a fixed order, whatever the workgroup's size)
// and the stopping test; returns on every thread whether the scene stopped (statistics
// written by thread 0).
template <typename T>
__device__ inline bool large_residual_scene(const LargeArgs<T>& a, const int sc, const int l_iter,
                                            double (*red)[4], int* stop) {
  const LoopArgs<T>& l = a.l;
  const int s0 = l.t.sc_slot[sc], s1 = l.t.sc_slot[sc + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid < 256) {
    double th = 0.0, yy = 0.0;
    for (int g = s0 + tid; g < s1; g += 256) {
      th += a.dy2[g];
      yy += a.yy2[g];
    }
    th = wave_total_lane63(th);
    yy = wave_total_lane63(yy);
    if (lane == 63) {
      red[0][wv] = th;
      red[1][wv] = yy;
    }
  }
  __syncthreads();
  if (tid == 0)
    *stop = large_decide<T>(a, sc, l_iter, (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]),
                            (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]));
  __syncthreads();
  return *stop != 0;
}

template <typename T>
__global__ void __launch_bounds__(256) large_residual_kernel(LargeArgs<T> a, int l_iter) {
  __shared__ double red[2][4];
  __shared__ int stop;
  const int sc = blockIdx.x;
  if (a.done[sc]) return;
  large_residual_scene<T>(a, sc, l_iter, red, &stop);
}

// z-update (Eq. 16-21) and dual update of interface j on the global slot arrays
template <typename T>
__device__ inline void large_zupdate_if(const LargeArgs<T>& a, const int j) {
  const LoopArgs<T>& l = a.l;
  const int sa = l.t.if_sub0[j];
  if (l.t.if_nsub[j] > 2) {
    // the multi-member form on the global slot arrays (scene offset 0, unpadded w)
    T ev[kMaxIfDim];
    for (int k = 0; k < kMaxIfDim; ++k) ev[k] = k < l.t.if_dim[j] ? l.e[l.t.if_row[j] + k] : (T)0;
    z_update_multi<T, false>(l, j, 0, ev, a.y, a.u, a.w);
    return;
  }
  const bool two = l.t.if_nsub[j] == 2;
  const int sb = two ? l.t.if_sub1[j] : sa;
  const int kind = l.t.if_kind[j], dim = l.t.if_dim[j];
  const int p0 = l.t.if_slot0[j], p1 = two ? l.t.if_slot1[j] : p0;
  const T ib0 = (T)1 / l.beta[sa], ib1 = two ? (T)1 / l.beta[sb] : (T)0;
  const T iws = (T)1 / (ib0 + ib1);
  T ya[kMaxIfDim], yb[kMaxIfDim], p[kMaxIfDim];
#pragma unroll
  for (int k = 0; k < kMaxIfDim; ++k) {
    const int kk = k < dim ? k : 0;
    const T ev = k < dim ? l.e[l.t.if_row[j] + k] : (T)0;
    ya[k] = a.y[p0 + kk];
    yb[k] = two ? a.y[p1 + kk] : (T)0;
    p[k] = kind == KIND_SOFT ? zsoft(ev, ya[k], ib0, yb[k], ib1, l.ksoft[j], l.asoft[j])
                             : -zsum(ev, ya[k], ib0, yb[k], ib1) * iws;
  }
  T cl[3];
  contact_project<T>(p, l.mu[j], cl, l.contact_model);
#pragma unroll
  for (int k = 0; k < kMaxIfDim; ++k) {
    if (k >= dim) continue;
    T v = p[k];
    if (kind == KIND_HARD_INEQ) v = v > (T)0 ? v : (T)0;
    if (kind == KIND_CONTACT && k < 3) v = cl[k];
    a.u[p0 + k] = -v;
    a.w[p0 + k] = ya[k] + (T)2 * v;
    if (two) {
      a.u[p1 + k] = -v;
      a.w[p1 + k] = yb[k] + (T)2 * v;
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) large_zupdate_kernel(LargeArgs<T> a) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.l.t.n_if) return;
  if (a.done[a.sub_scene[a.l.t.if_sub0[j]]]) return;
  large_zupdate_if<T>(a, j);
}

// Outputs after the iteration: v_hat of DOF g (c + G w of the last x-update's w), z and u
// of slot row g, lambda of interface g (= -u at its first member)
template <typename T>
__device__ inline void large_final_item(const LargeArgs<T>& a, const long g, const bool dof, const bool slot,
                                        const bool iface) {
  const LoopArgs<T>& l = a.l;
  if (dof && g < a.n_dof && l.v_hat) {
    // subsystem of DOF g: the last i with sub_dof[i] <= g
    int lo = 0, hi = l.t.n_sub - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (l.t.sub_dof[mid] <= g) lo = mid;
      else hi = mid - 1;
    }
    const int i = lo, n = l.t.sub_n[i], nc = l.t.sub_nc[i], rr = (int)(g - l.t.sub_dof[i]);
    const T* G = l.G + l.t.sub_J[i] + rr;
    const T* w = a.w + l.t.sub_slot[i];
    T v = l.cvec[g];
    for (int c = 0; c < nc; ++c) v += G[(long)c * n] * w[c];
    l.v_hat[g] = v;
  }
  if (slot && g < a.n_slot) {
    const T be = l.beta[l.t.slot_sub[g]];
    l.z_out[g] = (a.w[g] + a.u[g]) / be;
    l.u_out[g] = a.u[g];
  }
  if (iface && g < l.t.n_if && l.lambda) {
    const int dim = l.t.if_dim[g];
    for (int k = 0; k < dim; ++k) l.lambda[l.t.if_row[g] + k] = -a.u[l.t.if_slot0[g] + k];
  }
}

template <typename T>
__global__ void __launch_bounds__(256) large_final_kernel(LargeArgs<T> a) {
  large_final_item<T>(a, (long)blockIdx.x * blockDim.x + threadIdx.x, true, true, true);
}

// The whole iteration of one scene by one workgroup of 256 to 1024 threads (for scenes
// beyond the per-scene kernel's LDS layout but whose iteration one workgroup carries well):
// the same per-row x-update, per-scene residual (same summation order) and per-interface
// z-update as the phase kernels, with workgroup barriers in place of kernel boundaries, on
// the same global slot arrays.  Bitwise equal to the phase kernels.  residual(it): the stopping
// test of iteration it, from terms that are squared as kSquare says.
template <typename T, bool kSquare, typename R>
__device__ inline void large_scene_iterate(const LargeArgs<T>& a, const int sc, R&& residual) {
  const LoopArgs<T>& l = a.l;
  const int tid = threadIdx.x, bd = blockDim.x;
  const int s0 = l.t.sc_slot[sc], s1 = l.t.sc_slot[sc + 1];
  const int i0 = l.t.sc_if[sc], i1 = l.t.sc_if[sc + 1];
  const int d0 = l.t.sc_dof[sc], d1 = l.t.sc_dof[sc + 1];
  for (int it = 0; it < l.max_iters; ++it) {
    for (int g = s0 + tid; g < s1; g += bd) large_xupdate_row<T, kSquare>(a, g);
    __syncthreads();
    if (residual(it)) break;
    for (int j = i0 + tid; j < i1; j += bd) large_zupdate_if<T>(a, j);
    __syncthreads();
  }
  for (int g = d0 + tid; g < d1; g += bd) large_final_item<T>(a, g, true, false, false);
  for (int g = s0 + tid; g < s1; g += bd) large_final_item<T>(a, g, false, true, false);
  for (int j = i0 + tid; j < i1; j += bd) large_final_item<T>(a, j, false, false, true);
}

template <typename T>
__global__ void __launch_bounds__(1024) large_scene_kernel(LargeArgs<T> a) {
  __shared__ double red[2][4];
  __shared__ int stop;
  const int sc = blockIdx.x;
  const LoopArgs<T>& l = a.l;
  const int s0 = l.t.sc_slot[sc], s1 = l.t.sc_slot[sc + 1];
  if (threadIdx.x == 0) a.done[sc] = 0;
  for (int g = s0 + threadIdx.x; g < s1; g += blockDim.x) {
    const T be = l.beta[l.t.slot_sub[g]];
    const T z0 = l.z_in ? l.z_in[g] : (T)0;
    const T u0 = l.u_in ? l.u_in[g] : (T)0;
    a.w[g] = be * z0 - u0;
    a.y[g] = be * z0 + u0;
    a.u[g] = u0;
  }
  __syncthreads();
  large_scene_iterate<T, true>(a, sc, [&](int it) { return large_residual_scene<T>(a, sc, it, red, &stop); });
}

// ------------------------------------------------------------------------------------
// Large scenes, several workgroups per scene in one launch.  The host cuts every scene into
// runs of consecutive subsystems; a workgroup keeps its run's operators H_i in LDS (the
// blocked layout of loop_kernel), its slot vectors too, one interface per thread in
// registers, and iterates without kernel boundaries.  Per iteration the workgroups of a
// scene exchange the y of the interfaces that join two of them (both compute that
// interface's z-update from the same y) and the residual partials.
//
// Exchange: every value travels as 64-bit words of 32 data bits and a 32-bit tag, stored and
// loaded with agent-scope relaxed atomics (coherent across the XCDs' L2s); the tag names the
// launch and the iteration, so a word validates itself and a reader polls the word it needs.
// Two buffers in turn: a workgroup stores iteration l + 2 only after it has seen every
// partial of l + 1, and a partial of l + 1 is stored after its workgroup has read all it
// needs of l.  Tags start at a counter in device memory that the tail kernel advances after
// each launch (so replays of a captured launch use fresh tags).
//
// The grid fits the device (checked at bind), but another stream's kernels may hold CUs, so
// every wait is bounded: when it expires the workgroup marks the scene lost and leaves, and
// the tail kernel runs that scene again from its start values (kept in y, u, w) with one
// workgroup.  Per-row and per-interface arithmetic and its order are those of the phase
// kernels, so v_hat, lambda, z and u of an iteration are the same bits.  The residual is summed by
// lanes, waves and workgroups, in the tail kernel too: what a wait that expires changes is the time.
//
// Bound by latency: one exchange through the coherent point and the three workgroup barriers
// around it per iteration, ~2.7 us, against the phase kernels' three launches (~20 us) or one
// workgroup reading the operators from device memory (10.2 us).  Measured per launch of the
// iteration, FP32: the 640-segment cable at 60 iterations 1180 -> 183 us, the stirring of 216
// spheres at 60 iterations 1030 -> 181 us, 64 mixed scenes at 100 iterations 1020 -> 276 us.
// All loads of a poll are in flight together and the z-update runs three rows wide unless the
// wave holds a larger interface (with a wait per value and all waves six wide: 4.2 us).
// ------------------------------------------------------------------------------------
// x_r of one slot row from the blocked layout in the order of large_xupdate_row: column c
// goes to partial sum c mod 4 while a full group of four remains, the rest to partial 0 (the
// zero padding beyond the last column adds zeros).
__device__ inline float cluster_row_dot(const float4* Hv, const float4* Wv, int nc, int hs) {
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  const int nq = nc >> 2;
  int q = 0;
  for (; q + 3 < nq; q += 4) {
    float4 h[4], w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      h[k] = Hv[(q + k) * hs];
      w[k] = Wv[q + k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      acc[0] = zfma(h[k].x, w[k].x, acc[0]);
      acc[1] = zfma(h[k].y, w[k].y, acc[1]);
      acc[2] = zfma(h[k].z, w[k].z, acc[2]);
      acc[3] = zfma(h[k].w, w[k].w, acc[3]);
    }
  }
  for (; q < nq; ++q) {
    const float4 h = Hv[q * hs], w = Wv[q];
    acc[0] = zfma(h.x, w.x, acc[0]);
    acc[1] = zfma(h.y, w.y, acc[1]);
    acc[2] = zfma(h.z, w.z, acc[2]);
    acc[3] = zfma(h.w, w.w, acc[3]);
  }
  if (nc & 3) {
    const float4 h = Hv[nq * hs], w = Wv[nq];
    acc[0] = zfma(h.z, w.z, zfma(h.y, w.y, zfma(h.x, w.x, acc[0])));
  }
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}
__device__ inline double cluster_row_dot(const double2* Hv, const double2* Wv, int nc, int hs) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int nq = (nc >> 2) * 2;
  for (int q = 0; q < nq; q += 2) {
    const double2 h0 = Hv[q * hs], w0 = Wv[q], h1 = Hv[(q + 1) * hs], w1 = Wv[q + 1];
    acc[0] = zfma(h0.x, w0.x, acc[0]);
    acc[1] = zfma(h0.y, w0.y, acc[1]);
    acc[2] = zfma(h1.x, w1.x, acc[2]);
    acc[3] = zfma(h1.y, w1.y, acc[3]);
  }
  for (int q = nq; 2 * q < nc; ++q) {
    const double2 h = Hv[q * hs], w = Wv[q];
    acc[0] = zfma(h.y, w.y, zfma(h.x, w.x, acc[0]));
  }
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// One slot row's operator entries held in registers: NV full 16-byte vectors (zero beyond the
// row's own) and the tail vector.  Same order of the products as cluster_row_dot.
template <int NV>
struct RowRegs {
  float4 h[NV], tail;
  __device__ void load(const float* Hg, int nc) {
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const bool on = 4 * q + 3 < nc;
      h[q].x = on ? Hg[(long)(4 * q) * nc] : 0.f;
      h[q].y = on ? Hg[(long)(4 * q + 1) * nc] : 0.f;
      h[q].z = on ? Hg[(long)(4 * q + 2) * nc] : 0.f;
      h[q].w = on ? Hg[(long)(4 * q + 3) * nc] : 0.f;
    }
    const int c = nc & ~3;
    tail.x = c < nc ? Hg[(long)c * nc] : 0.f;
    tail.y = c + 1 < nc ? Hg[(long)(c + 1) * nc] : 0.f;
    tail.z = c + 2 < nc ? Hg[(long)(c + 2) * nc] : 0.f;
    tail.w = 0.f;
  }
  // w: the subsystem's padded vectors; nw: how many there are (at least one).  Vectors beyond
  // them are read again from the first (their H is zero).
  __device__ float dot(const float4* w, int nq, int ntail) const {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    float4 wv[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) wv[q] = w[q < nq ? q : 0];
    const float4 wt = w[ntail];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      acc[0] = zfma(h[q].x, wv[q].x, acc[0]);
      acc[1] = zfma(h[q].y, wv[q].y, acc[1]);
      acc[2] = zfma(h[q].z, wv[q].z, acc[2]);
      acc[3] = zfma(h[q].w, wv[q].w, acc[3]);
    }
    acc[0] = zfma(tail.z, wt.z, zfma(tail.y, wt.y, zfma(tail.x, wt.x, acc[0])));
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
  }
};

// The kernel's arguments, read again from the kernel-argument segment: what is only needed
// after (or rarely in) the iteration is not held in scalar registers across it.
template <typename A>
__device__ __attribute__((always_inline)) inline const A& args_again() {
  uint64_t v = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(v));
  return *reinterpret_cast<const A*>(v);
}

// z-update of one interface of D rows at most from its members' y (Eq. 16-21).
template <typename T, int D>
__device__ inline void cluster_z(const T* ev, const T* ya, const T* yb, T ib0, T ib1, T iws, T mu, T ksj, T asj, int kind,
                                 int model, T* lam) {
  if (kind == KIND_SOFT) {
#pragma unroll
    for (int k = 0; k < D; ++k) lam[k] = zsoft(ev[k], ya[k], ib0, yb[k], ib1, ksj, asj);
    return;
  }
#pragma unroll
  for (int k = 0; k < D; ++k) lam[k] = -zsum(ev[k], ya[k], ib0, yb[k], ib1) * iws;
  if (kind == KIND_CONTACT) {
    const T p3[3] = {lam[0], lam[1], lam[2]};
    contact_project<T>(p3, mu, lam, model);
  } else if (kind == KIND_HARD_INEQ) {
#pragma unroll
    for (int k = 0; k < D; ++k) lam[k] = lam[k] > (T)0 ? lam[k] : (T)0;
  }
}

// NV > 0 (FP32, one slot row per thread, rows of at most 4 NV + 3 columns): the operator rows
// in registers; NV = 0: in LDS.
template <typename T, int NV>
__global__ void __launch_bounds__(kClusterThreads) cluster_scene_kernel(ClusterArgs<T> a) {
  using VT = typename Vec16<T>::type;
  using X = Tagged<T>;
  constexpr int V = Vec16<T>::N;
  constexpr int kRows = NV > 0 ? 1 : kClusterRows / kClusterThreads;  // slot rows per thread
  constexpr int kWaves = kClusterThreads / 64;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ __align__(16) double red[2][kWaves];
  __shared__ __align__(16) double pred[2][kWaves];
  __shared__ int s_lost;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid) >> 6;
  const int wg = a.order[blockIdx.x];
  const int32_t* dsc = a.wg + 8 * (long)wg;
  const int sc = dsc[0], sb = dsc[1], se = dsc[2], first = dsc[5], count = dsc[6], own = dsc[7];
  const int s0 = a.g.l.t.sub_slot[sb], ns = a.g.l.t.sub_slot[se] - s0;
  const int hq0 = a.g.l.t.sub_hq[sb], wq0 = a.g.l.t.sub_wq[sb];
  const int lastq = (a.g.l.t.sub_nc[se - 1] + V - 1) / V;
  const int nhq = NV > 0 ? 0 : a.g.l.t.sub_hq[se - 1] - hq0 + lastq * a.g.l.t.sub_nc[se - 1];
  // one vector more than the padded blocks: an absent tail vector's address
  const int nwq = a.g.l.t.sub_wq[se - 1] - wq0 + (lastq + 1) * V;
  VT* Hq = reinterpret_cast<VT*>(smem_raw);
  T* w = reinterpret_cast<T*>(Hq + nhq);
  T* y = w + nwq;
  T* u = y + ns;
  const uint32_t tag0 = *a.epoch;

  for (int q = tid; q < nwq; q += kClusterThreads) w[q] = (T)0;
  if (tid == 0) s_lost = 0;
  if (tid < 2 * kWaves) red[tid / kWaves][tid % kWaves] = 0.0;
  __syncthreads();
  int nc[kRows], hoff[kRows], wo[kRows];
  long bx[kRows];
  T be[kRows], dr[kRows];
  RowRegs<(NV > 0 ? NV : 1)> hr;
#pragma unroll
  for (int p = 0; p < kRows; ++p) {
    const LoopArgs<T>& l = a.g.l;
    const int r = tid + p * kClusterThreads;
    nc[p] = hoff[p] = wo[p] = 0;
    bx[p] = -1;
    be[p] = (T)1;
    dr[p] = (T)0;
    if (r < ns) {
      const int g = s0 + r;
      const int i = l.t.slot_sub[g], loc = l.t.slot_loc[g];
      nc[p] = l.t.sub_nc[i];
      hoff[p] = l.t.sub_hq[i] - hq0 + loc;
      wo[p] = l.t.sub_wq[i] - wq0;
      be[p] = l.beta[i];
      dr[p] = l.d[g];
      if (a.bidx[g] >= 0) bx[p] = (long)a.bidx[g] * X::N;
      const T* Hg = l.H + l.t.sub_H[i] + loc;
      if constexpr (NV > 0) {
        hr.load(Hg, nc[p]);
      } else {
        for (int cb = 0; cb * V < nc[p]; ++cb) {
          T v[V];
#pragma unroll
          for (int k = 0; k < V; ++k) v[k] = cb * V + k < nc[p] ? Hg[(long)(cb * V + k) * nc[p]] : (T)0;
          Hq[hoff[p] + cb * nc[p]] = Vec16<T>::make(v);
        }
      }
      const T z0 = l.z_in ? l.z_in[g] : (T)0;
      const T u0 = l.u_in ? l.u_in[g] : (T)0;
      const T wi = be[p] * z0 - u0, yi = be[p] * z0 + u0;
      w[wo[p] + loc] = wi;
      y[r] = yi;
      u[r] = u0;
      a.g.w[g] = wi;  // start values, for the tail kernel
      a.g.y[g] = yi;
      a.g.u[g] = u0;
    }
  }
  // this thread's interface: local slots pa, pb (-1: the other workgroup's, read from the
  // exchange buffer at xo)
  const int f = dsc[3] + tid;
  const bool has_if = f < dsc[4];
  int kind = -1, dim = 0, pa = -1, pb = -1, qa = 0, qb = 0;
  long xo = -1;
  bool xa = false, two = false;
  T ib0 = (T)0, ib1 = (T)0, iws = (T)0, mu = (T)0, ksj = (T)0, asj = (T)0;
  T ev[kMaxIfDim];
#pragma unroll
  for (int k = 0; k < kMaxIfDim; ++k) ev[k] = (T)0;
  if (has_if) {
    const LoopArgs<T>& l = a.g.l;
    const int j = a.if_list[f];
    kind = l.t.if_kind[j];
    dim = l.t.if_dim[j];
    two = l.t.if_nsub[j] == 2;
    const int sa = l.t.if_sub0[j], sbb = two ? l.t.if_sub1[j] : sa;
    ib0 = (T)1 / l.beta[sa];
    ib1 = two ? (T)1 / l.beta[sbb] : (T)0;
    iws = (T)1 / (ib0 + ib1);
    mu = l.mu[j];
    ksj = l.ksoft[j];
    asj = l.asoft[j];
    const int erow = l.t.if_row[j];
#pragma unroll
    for (int k = 0; k < kMaxIfDim; ++k)
      if (k < dim) ev[k] = l.e[erow + k];
    const int g0 = l.t.if_slot0[j];
    if (sa >= sb && sa < se) {
      pa = g0 - s0;
      qa = l.t.sub_wq[sa] - wq0 + (g0 - l.t.sub_slot[sa]);
    } else {
      xo = (long)a.bidx[g0] * X::N;
      xa = true;
    }
    if (two) {
      const int g1 = l.t.if_slot1[j];
      if (sbb >= sb && sbb < se) {
        pb = g1 - s0;
        qb = l.t.sub_wq[sbb] - wq0 + (g1 - l.t.sub_slot[sbb]);
      } else {
        xo = (long)a.bidx[g1] * X::N;
      }
    }
  }
  // addresses for the loads of absent rows and members (their values are not used)
  const int la = pa >= 0 ? pa : 0, lb = pb >= 0 ? pb : 0;
  const int big = __any(dim > 3) ? 1 : 0;  // this wave holds interfaces of more than three rows
  const int npw = (count + 63) / 64;       // waves that read the scene's partials
  const int max_iters = a.g.l.max_iters, model = a.g.l.contact_model;
  const double tol2 = a.g.l.tol * a.g.l.tol;
  const long y_par = a.n_ex * X::N, p_par = (long)a.n_wg * 4;
  unsigned long long* const ybuf = a.ybuf;
  unsigned long long* const part = a.part + 4 * (long)first;
  __syncthreads();

  int it = 0, conv = 0;
  double th = 0.0, yy = 0.0;
  bool lost = false;
  for (int li = 0; li < max_iters; ++li) {
    it = li + 1;
    const uint32_t tag = tag0 + (uint32_t)it;
    unsigned long long* yb = ybuf + (li & 1 ? y_par : 0);
    unsigned long long* pt = part + (li & 1 ? p_par : 0);
    // x-update (Eq. 15 reassociated), y = beta x + u (Eq. 18), published where another
    // workgroup's interface reads it
    double pth = 0.0, pyy = 0.0;
#pragma unroll
    for (int p = 0; p < kRows; ++p) {
      const int r = tid + p * kClusterThreads;
      if (r < ns) {
        const T yo = y[r], uo = u[r];
        T x;
        if constexpr (NV > 0)
          x = hr.dot(reinterpret_cast<const VT*>(w + wo[p]), nc[p] >> 2, nc[p] >> 2);
        else
          x = cluster_row_dot(Hq + hoff[p], reinterpret_cast<const VT*>(w + wo[p]), nc[p], nc[p]);
        const T yn = be[p] * (dr[p] + x) + uo;
        if (bx[p] >= 0) X::put(yb + bx[p], yn, tag);
        const double df = (double)yn - (double)yo;
        pth = __builtin_fma(df, df, pth);
        pyy = __builtin_fma((double)yn, (double)yn, pyy);
        y[r] = yn;
      }
    }
    if (wv * 64 < ns) {
      pth = wave_total_lane63(pth);
      pyy = wave_total_lane63(pyy);
      if (lane == 63) {
        red[0][wv] = pth;
        red[1][wv] = pyy;
      }
    }
    __syncthreads();
    // the workgroup's partials (waves in a fixed order), published by the first two threads
    double sth = 0.0, syy = 0.0;
    if (tid < 2) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < kWaves; ++q) s += red[tid][q];
      Tagged<double>::put(pt + 4 * own + 2 * tid, s, tag);
    }
    // the local members' y, then the waits: the scene's partials (one thread per workgroup of
    // the scene) and the other workgroup's y of this thread's interface, all loads of a poll
    // in flight together
    T ya[kMaxIfDim], yc[kMaxIfDim], yr[kMaxIfDim];
    auto stage = [&](auto dc) {
      constexpr int D = decltype(dc)::value;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        const int kk = k < dim ? k : 0;
        ya[k] = y[la + kk];
        yc[k] = y[lb + kk];
        yr[k] = (T)0;
      }
      bool pw = tid < count, yw = xo >= 0;
      const unsigned long long* py = yb + (yw ? xo : 0);
      const unsigned long long* pp = pt + 4 * (pw ? tid : 0);
      long long t0 = 0;
      for (unsigned n = 0; pw || yw;) {
        double p0, p1;
        bool okp = Tagged<double>::get(pp, &p0, tag);
        okp = Tagged<double>::get(pp + 2, &p1, tag) & okp;
        T v[D];
        bool oky = true;
        if (yw) {
#pragma unroll
          for (int k = 0; k < D; ++k) oky = X::get(py + (k < dim ? k : 0) * X::N, &v[k], tag) & oky;
          if (oky) {
#pragma unroll
            for (int k = 0; k < D; ++k) yr[k] = v[k];
            yw = false;
          }
        }
        if (pw && okp) {
          sth = p0;
          syy = p1;
          pw = false;
        }
        if (pw || yw) {
          const ClusterArgs<T>& b = args_again<ClusterArgs<T>>();
          if ((++n & 63) == 0 || b.wait_ticks == 0) {
            const long long now = wall_clock64();
            if (t0 == 0) t0 = now;
            if (now - t0 >= b.wait_ticks ||
                __hip_atomic_load(b.lost + sc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
              s_lost = 1;
              break;
            }
          }
        }
      }
#pragma unroll
      for (int k = 0; k < D; ++k) {
        ya[k] = xa ? yr[k] : ya[k];
        yc[k] = !two ? (T)0 : pb >= 0 ? yc[k] : yr[k];
      }
    };
    if (big)
      stage(std::integral_constant<int, kMaxIfDim>{});
    else
      stage(std::integral_constant<int, 3>{});
    if (wv < npw) {
      sth = wave_total_lane63(sth);
      syy = wave_total_lane63(syy);
      if (lane == 63) {
        pred[0][wv] = sth;
        pred[1][wv] = syy;
      }
    }
    __syncthreads();
    // the test of Eq. 22, from the same sums in every workgroup of the scene
    th = pred[0][0];
    yy = pred[1][0];
    for (int q = 1; q < npw; ++q) {
      th += pred[0][q];
      yy += pred[1][q];
    }
    if (s_lost) {
      lost = true;
      break;
    }
    if (!__builtin_isfinite(th) || !__builtin_isfinite(yy)) {
      if (tid == 0) atomicOr(args_again<ClusterArgs<T>>().g.l.flags, FLAG_NONFINITE);
      break;
    }
    if (th <= tol2 * (yy > 1e-24 ? yy : 1e-24)) {
      conv = 1;
      break;
    }
    if (it == max_iters) break;
    // z-update (Eq. 16-21) and dual update (Eq. 14)
    auto update = [&](auto dc) {
      constexpr int D = decltype(dc)::value;
      T lam[D];
      cluster_z<T, D>(ev, ya, yc, ib0, ib1, iws, mu, ksj, asj, kind, model, lam);
#pragma unroll
      for (int k = 0; k < D; ++k) {
        if (k < dim) {
          if (pa >= 0) {
            u[pa + k] = -lam[k];
            w[qa + k] = ya[k] + (T)2 * lam[k];
          }
          if (pb >= 0) {
            u[pb + k] = -lam[k];
            w[qb + k] = yc[k] + (T)2 * lam[k];
          }
        }
      }
    };
    if (has_if) {
      if (big)
        update(std::integral_constant<int, kMaxIfDim>{});
      else
        update(std::integral_constant<int, 3>{});
    }
    __syncthreads();
  }
  const ClusterArgs<T>& b = args_again<ClusterArgs<T>>();
  const LoopArgs<T>& l = b.g.l;
  if (lost) {
    if (tid == 0) __hip_atomic_store(b.lost + sc, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  // v_hat = c + G w, z, u, lambda = -u of this workgroup's subsystems
  if (l.v_hat) {
    const int d0 = l.t.sub_dof[sb], d1 = l.t.sub_dof[se];
    for (int dg = d0 + tid; dg < d1; dg += kClusterThreads) {
      int i = sb;
      while (i + 1 < se && l.t.sub_dof[i + 1] <= dg) ++i;
      const int n = l.t.sub_n[i], nci = l.t.sub_nc[i];
      const T* G = l.G + l.t.sub_J[i] + (dg - l.t.sub_dof[i]);
      const T* wi = w + (l.t.sub_wq[i] - wq0);
      T v = l.cvec[dg];
      for (int c = 0; c < nci; ++c) v += G[(long)c * n] * wi[c];
      l.v_hat[dg] = v;
    }
  }
#pragma unroll
  for (int p = 0; p < kRows; ++p) {
    const int r = tid + p * kClusterThreads;
    if (r < ns) {
      l.z_out[s0 + r] = (w[wo[p] + l.t.slot_loc[s0 + r]] + u[r]) / be[p];
      l.u_out[s0 + r] = u[r];
    }
  }
  if (has_if && pa >= 0 && l.lambda) {
    const int erow = l.t.if_row[b.if_list[f]];
    for (int k = 0; k < dim; ++k) l.lambda[erow + k] = -u[pa + k];
  }
  if (tid == 0 && wg == first) {
    const double yn = __builtin_sqrt(yy);
    l.st_iters[sc] = it;
    l.st_conv[sc] = conv;
    l.st_theta[sc] = th;
    l.st_rtheta[sc] = __builtin_sqrt(th) / (yn > 1e-12 ? yn : 1e-12);
  }
}

// Residual of Eq. 22 of scene sc by one workgroup in the order of the scene's workgroups `first` to
// first + count - 1 in cluster_scene_kernel (its rows per lane, lanes, waves, workgroups), so that a
// scene that is run again stops at the iteration where it would have, and the stopping test.
template <typename T>
__device__ inline bool cluster_residual_scene(const ClusterArgs<T>& a, const int sc, const int first, const int count,
                                              const int l_iter, double (*part)[kClusterThreads], double (*pred)[8],
                                              int* stop) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nwv = blockDim.x >> 6;
  const int32_t* sub_slot = a.g.l.t.sub_slot;
  for (int m = wv; m < count; m += nwv) {
    const int32_t* dsc = a.wg + 8 * (long)(first + m);
    const int s0 = sub_slot[dsc[1]], ns = sub_slot[dsc[2]] - s0;
    double sth = 0.0, syy = 0.0;
    for (int q = 0; q < kClusterThreads / 64 && 64 * q < ns; ++q) {
      double pth = 0.0, pyy = 0.0;
      for (int r = 64 * q + lane; r < ns; r += kClusterThreads) {
        const double df = a.g.dy2[s0 + r], yn = a.g.yy2[s0 + r];
        pth = __builtin_fma(df, df, pth);
        pyy = __builtin_fma(yn, yn, pyy);
      }
      sth += wave_total_lane63(pth);
      syy += wave_total_lane63(pyy);
    }
    if (lane == 63) {
      part[0][m] = sth;
      part[1][m] = syy;
    }
  }
  __syncthreads();
  const int npw = (count + 63) / 64;
  for (int q = wv; q < npw; q += nwv) {
    const int m = 64 * q + lane;
    const double sth = wave_total_lane63(m < count ? part[0][m] : 0.0);
    const double syy = wave_total_lane63(m < count ? part[1][m] : 0.0);
    if (lane == 63) {
      pred[0][q] = sth;
      pred[1][q] = syy;
    }
  }
  __syncthreads();
  if (tid == 0) {
    double th = pred[0][0], yy = pred[1][0];
    for (int q = 1; q < npw; ++q) {
      th += pred[0][q];
      yy += pred[1][q];
    }
    *stop = large_decide<T>(a.g, sc, l_iter, th, yy);
  }
  __syncthreads();
  return *stop != 0;
}

// After the cluster kernel, one workgroup per scene: the totals of a scene that ran through,
// or the whole iteration of one whose waits expired; then the tags of the next launch.
template <typename T>
__global__ void __launch_bounds__(1024) cluster_tail_kernel(ClusterArgs<T> a) {
  __shared__ double part[2][kClusterThreads];
  __shared__ double pred[2][8];
  __shared__ int stop, s_first;
  const int sc = blockIdx.x;
  if (sc == 0 && threadIdx.x == 0) *a.epoch += (uint32_t)a.g.l.max_iters + 1u;
  if (a.lost[sc]) {
    for (int m = threadIdx.x; m < a.n_wg; m += blockDim.x)
      if (a.wg[8 * (long)m] == sc) s_first = a.wg[8 * (long)m + 5];
    __syncthreads();
    if (threadIdx.x == 0) {
      a.lost[sc] = 0;
      atomicAdd(a.again, 1);
    }
    const int first = s_first, count = a.wg[8 * (long)first + 6];
    large_scene_iterate<T, false>(a.g, sc, [&](int it) {
      return cluster_residual_scene<T>(a, sc, first, count, it, part, pred, &stop);
    });
  } else if (threadIdx.x == 0) {
    a.g.l.st_total[sc] += a.g.l.st_iters[sc];
    if (!a.g.l.st_conv[sc]) a.g.l.st_unconv[sc] += 1;
  }
}

// The form for rows of at most max_nc columns and `rows` slot rows per workgroup.
template <typename T, typename F>
hipError_t cluster_form(int max_nc, int rows, F&& f) {
  if constexpr (sizeof(T) == sizeof(float)) {
    if (rows <= kClusterThreads) {
      if (max_nc <= 24 + 3) return f(std::integral_constant<int, 6>{});
      if (max_nc <= 48 + 3) return f(std::integral_constant<int, 12>{});
      if (max_nc <= 72 + 3) return f(std::integral_constant<int, 18>{});
    }
  }
  return f(std::integral_constant<int, 0>{});
}

// Workgroups the device holds at once with `lds` bytes of dynamic LDS each.
template <typename T>
hipError_t cluster_capacity(const ClusterShape& c, int* wgs) {
  *wgs = 0;
  return cluster_form<T>(c.max_nc, c.rows, [&](auto nv) -> hipError_t {
    constexpr int NV = decltype(nv)::value;
    const size_t lds = NV > 0 ? c.lds_w : c.lds;
    const void* fn = reinterpret_cast<const void*>(&cluster_scene_kernel<T, NV>);
    int dev = 0, cus = 0, per = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kClusterThreads, lds);
    if (e == hipSuccess) *wgs = per * cus;
    return e;
  });
}
template hipError_t cluster_capacity<float>(const ClusterShape&, int*);
template hipError_t cluster_capacity<double>(const ClusterShape&, int*);

template <typename T>
hipError_t launch_cluster(const ClusterArgs<T>& a, const ClusterShape& c, int tail_threads, hipStream_t s) {
  if (a.g.l.t.n_scene == 0 || a.n_wg == 0) return hipSuccess;
  const hipError_t e = cluster_form<T>(c.max_nc, c.rows, [&](auto nv) -> hipError_t {
    constexpr int NV = decltype(nv)::value;
    hipLaunchKernelGGL((cluster_scene_kernel<T, NV>), dim3(a.n_wg), dim3(kClusterThreads), NV > 0 ? c.lds_w : c.lds, s, a);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(cluster_tail_kernel<T>, dim3(a.g.l.t.n_scene), dim3(tail_threads), 0, s, a);
  return hipGetLastError();
}
template hipError_t launch_cluster<float>(const ClusterArgs<float>&, const ClusterShape&, int, hipStream_t);
template hipError_t launch_cluster<double>(const ClusterArgs<double>&, const ClusterShape&, int, hipStream_t);

__global__ void __launch_bounds__(256) large_alldone_kernel(const int32_t* done, int n_scene, int32_t* all_done) {
  __shared__ int open;
  if (threadIdx.x == 0) open = 0;
  __syncthreads();
  for (int s = threadIdx.x; s < n_scene; s += blockDim.x)
    if (!done[s]) open = 1;
  __syncthreads();
  if (threadIdx.x == 0) *all_done = open ? 0 : 1;
}

template <typename T>
hipError_t launch_large_scene(const LargeArgs<T>& a, int threads, hipStream_t s) {
  if (a.l.t.n_scene == 0) return hipSuccess;
  if (threads < 256 || threads > 1024 || threads % 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(large_scene_kernel<T>, dim3(a.l.t.n_scene), dim3(threads), 0, s, a);
  return hipGetLastError();
}

template hipError_t launch_large_scene<float>(const LargeArgs<float>&, int, hipStream_t);
template hipError_t launch_large_scene<double>(const LargeArgs<double>&, int, hipStream_t);

// ADMM's standard primal and dual residuals (Boyd et al. 2011, Sec. 3.3) of the iterate a
// solve returns, one 256-thread workgroup per scene: from the returned (z, u) (z_in, u_in)
// one more x-update (Eq. 15) and the z- and dual update (Eq. 16-21, 14) that would follow
// it, on the large-scene slot arrays as scratch (nothing returned is changed).  The
// x-update gives the x of the iteration's last x-update, from which v_hat was formed.
//   r_prim = |x - z'| / max(|x|, |z'|),  r_dual = |beta (z' - z)| / |u'|,  floors 1e-12,
// sums in FP64 over the scene's slot rows (threads take rows tid, tid + 256, ...; waves
// added in a fixed order).
template <typename T>
__global__ void __launch_bounds__(256) boyd_residual_kernel(LargeArgs<T> a, double* r_prim, double* r_dual) {
  __shared__ double red[5][4];
  const int sc = blockIdx.x;
  const LoopArgs<T>& l = a.l;
  const int tid = threadIdx.x, bd = blockDim.x, lane = tid & 63, wv = tid >> 6;
  const int s0 = l.t.sc_slot[sc], s1 = l.t.sc_slot[sc + 1];
  const int i0 = l.t.sc_if[sc], i1 = l.t.sc_if[sc + 1];
  for (int g = s0 + tid; g < s1; g += bd) {
    const T be = l.beta[l.t.slot_sub[g]];
    a.w[g] = be * l.z_in[g] - l.u_in[g];
    a.u[g] = l.u_in[g];
    a.y[g] = (T)0;
  }
  __syncthreads();
  for (int g = s0 + tid; g < s1; g += bd) large_xupdate_row<T>(a, g);
  __syncthreads();
  for (int j = i0 + tid; j < i1; j += bd) large_zupdate_if<T>(a, j);
  __syncthreads();
  // after the z-update: u' = -lambda and w' = y + 2 lambda, so z' = (w' + u') / beta
  double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int g = s0 + tid; g < s1; g += bd) {
    const double be = (double)l.beta[l.t.slot_sub[g]];
    const double x = ((double)a.y[g] - (double)l.u_in[g]) / be;
    const double zn = ((double)a.w[g] + (double)a.u[g]) / be;
    const double dz = be * (zn - (double)l.z_in[g]);
    const double un = (double)a.u[g];
    v[0] += (x - zn) * (x - zn);
    v[1] += x * x;
    v[2] += zn * zn;
    v[3] += dz * dz;
    v[4] += un * un;
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const double t = wave_total_lane63(v[k]);
    if (lane == 63) red[k][wv] = t;
  }
  __syncthreads();
  if (tid == 0) {
    double q[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) q[k] = (red[k][0] + red[k][1]) + (red[k][2] + red[k][3]);
    const double nx = __builtin_sqrt(q[1] > q[2] ? q[1] : q[2]), nu = __builtin_sqrt(q[4]);
    r_prim[sc] = __builtin_sqrt(q[0]) / (nx > 1e-12 ? nx : 1e-12);
    r_dual[sc] = __builtin_sqrt(q[3]) / (nu > 1e-12 ? nu : 1e-12);
  }
}

template <typename T>
hipError_t launch_boyd_residuals(const LargeArgs<T>& a, double* r_prim, double* r_dual, hipStream_t s) {
  if (a.l.t.n_scene == 0) return hipSuccess;
  hipLaunchKernelGGL(boyd_residual_kernel<T>, dim3(a.l.t.n_scene), dim3(256), 0, s, a, r_prim, r_dual);
  return hipGetLastError();
}
template hipError_t launch_boyd_residuals<float>(const LargeArgs<float>&, double*, double*, hipStream_t);
template hipError_t launch_boyd_residuals<double>(const LargeArgs<double>&, double*, double*, hipStream_t);

template <typename T>
hipError_t launch_large_loop(const LargeArgs<T>& a, hipStream_t s, int poll_every, int32_t* host_flag) {
  const unsigned bs = 256;
  const long most = a.n_slot > a.n_dof ? a.n_slot : a.n_dof;
  const long fin = most > a.l.t.n_if ? most : a.l.t.n_if;
  const long first = a.n_slot > a.l.t.n_scene ? a.n_slot : a.l.t.n_scene;
  hipLaunchKernelGGL(large_init_kernel<T>, dim3((unsigned)((first + bs - 1) / bs)), dim3(bs), 0, s, a);
  hipError_t e = hipGetLastError();
  for (int it = 0; it < a.l.max_iters && e == hipSuccess; ++it) {
    if (a.n_slot > 0)
      hipLaunchKernelGGL(large_xupdate_kernel<T>, dim3((unsigned)((a.n_slot + bs - 1) / bs)), dim3(bs), 0, s, a);
    hipLaunchKernelGGL(large_residual_kernel<T>, dim3(a.l.t.n_scene), dim3(bs), 0, s, a, it);
    if (it + 1 < a.l.max_iters && a.l.t.n_if > 0)
      hipLaunchKernelGGL(large_zupdate_kernel<T>, dim3((unsigned)((a.l.t.n_if + bs - 1) / bs)), dim3(bs), 0, s, a);
    e = hipGetLastError();
    if (e == hipSuccess && poll_every > 0 && host_flag && (it + 1) % poll_every == 0 && it + 1 < a.l.max_iters) {
      // every scene stopped: the launches left would return at once, so none are issued
      hipLaunchKernelGGL(large_alldone_kernel, dim3(1), dim3(bs), 0, s, a.done, a.l.t.n_scene, a.all_done);
      e = hipGetLastError();
      if (e == hipSuccess) e = hipMemcpyAsync(host_flag, a.all_done, sizeof(int32_t), hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      if (e == hipSuccess && *host_flag) break;
    }
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(large_final_kernel<T>, dim3((unsigned)((fin + bs - 1) / bs)), dim3(bs), 0, s, a);
  return hipGetLastError();
}

template hipError_t launch_large_loop<float>(const LargeArgs<float>&, hipStream_t, int, int32_t*);
template hipError_t launch_large_loop<double>(const LargeArgs<double>&, hipStream_t, int, int32_t*);

template <typename T>
hipError_t launch_steps(const StepsArgs<T>& a, const StepsArgs<T>* dev_args, int max_slot_scene, int max_if_scene,
                        int max_hq_scene, int max_wq_scene, bool fp64, size_t lds, hipStream_t s) {
  if (a.l.t.n_scene == 0 || a.n_steps == 0) return hipSuccess;
  const int ns = max_slot_scene > 0 ? max_slot_scene : 1;
  const bool two = 2 * ns <= kTwoLaneMax && max_if_scene <= kTwoLaneMax;
  const int need = two ? (2 * ns > max_if_scene ? 2 * ns : max_if_scene) : (ns > max_if_scene ? ns : max_if_scene);
  const int threads = (need + 63) / 64 * 64;
  (void)max_hq_scene;
  (void)max_wq_scene;
  // at most 256 threads, and at most 128 VGPRs (the launch bound of four waves per SIMD), so
  // that four scenes of the multi-step kernel share a CU
  if (threads > 256 || lds > 150 * 1024) return hipErrorInvalidValue;
  // split rows within the default block: its lane map is built for exactly this block
  const bool split = a.l.t.rmap && a.l.t.rmap_block == threads;
  if (fp64 && split)
    hipLaunchKernelGGL((steps_kernel<T, double, 0>), dim3(a.l.t.n_scene), dim3(threads), lds, s, dev_args);
  else if (split)
    hipLaunchKernelGGL((steps_kernel<T, T, 0>), dim3(a.l.t.n_scene), dim3(threads), lds, s, dev_args);
  else if (fp64 && two)
    hipLaunchKernelGGL((steps_kernel<T, double, 2>), dim3(a.l.t.n_scene), dim3(threads), lds, s, dev_args);
  else if (fp64)
    hipLaunchKernelGGL((steps_kernel<T, double, 1>), dim3(a.l.t.n_scene), dim3(threads), lds, s, dev_args);
  else if (two)
    hipLaunchKernelGGL((steps_kernel<T, T, 2>), dim3(a.l.t.n_scene), dim3(threads), lds, s, dev_args);
  else
    hipLaunchKernelGGL((steps_kernel<T, T, 1>), dim3(a.l.t.n_scene), dim3(threads), lds, s, dev_args);
  return hipGetLastError();
}

template hipError_t launch_steps<float>(const StepsArgs<float>&, const StepsArgs<float>*, int, int, int, int, bool,
                                        size_t, hipStream_t);
template hipError_t launch_steps<double>(const StepsArgs<double>&, const StepsArgs<double>*, int, int, int, int, bool,
                                         size_t, hipStream_t);
template hipError_t launch_factor<float>(const FactorArgs<float>&, int, int, int, bool, hipStream_t);
template hipError_t launch_factor<double>(const FactorArgs<double>&, int, int, int, bool, hipStream_t);
template hipError_t launch_factor_global<float>(const FactorArgs<float>&, int, int, bool, char*, const int64_t*,
                                                hipStream_t);
template hipError_t launch_factor_global<double>(const FactorArgs<double>&, int, int, bool, char*, const int64_t*,
                                                 hipStream_t);
template hipError_t launch_loop<float>(const LoopArgs<float>&, int, int, long long, int, int, int, hipStream_t);
template hipError_t launch_loop<double>(const LoopArgs<double>&, int, int, long long, int, int, int, hipStream_t);

}  // namespace subadmm
