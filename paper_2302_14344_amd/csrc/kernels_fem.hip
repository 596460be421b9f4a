// HIP kernels (gfx950) of the deformable-body path: co-rotated linear-tetrahedron blocks,
// one subsystem per block (arXiv 2302.14344, Sec. II soft constraints folded into A_i, b_i;
// Algorithm 1 with multi-block subsystems).
//
// fem_assemble_kernel: one workgroup per block.  Eq. (2) with the elastic potential psi
//   linearised about the start-of-step positions x:
//     A = (2/t) M + (t/2) K(x),   b = (2/t) M v - d psi(x)^T + M g,
//   with per-tetrahedron rotation R (orthogonal polar factor of F = sum_a x_a g_a^T, by
//   Newton's iteration R <- (R + R^-T)/2), rest stiffness blocks
//     K0_ab = V (lambda g_a g_b^T + mu g_b g_a^T + mu (g_a . g_b) I),
//   co-rotated K_ab = R K0_ab R^T and elastic forces f_a = -R (V sigma) g_a with
//   sigma = lambda tr(G) I + mu (G + G^T), G = sum_b (R^T x_b - X_b) g_b^T.  A is written
//   by node pair (gather over the tetrahedra sharing the pair, so each entry is formed
//   once, in a fixed order).
// fem_factor_kernel: one workgroup per block, FP64 (or an FP32 trial on every block, FP64 again
//   for blocks whose condition estimate exceeds a threshold).  beta (Eq. 23), K = A + beta J^T J
//   in a permuted order with the constrained DOFs last, Cholesky factor L (with y = L^-1 b),
//   the inverse of the trailing factor block T = L_DD^-1, and S = T^T T, which is K^-1
//   restricted to the constrained DOFs (the Schur-complement inverse).  Since every slot row
//   of a block selects one DOF with sign +-1, the x-update of Eq. (15) followed by
//   x = J v_hat is  x = J_D (c_D + S J_D^T w)  with c = K^-1 b: one dense m x m product per
//   block.  The O(n^3) parts are 16 x 16 tile products on the FP64 (FP32) matrix cores.
// fem_loop_kernel: one launch with every block resident, one workgroup per block.  Each
//   workgroup does the z-update (Eq. 16-21) of the interfaces that touch its block
//   (two-member interfaces are computed by both members from the same y, so both obtain
//   the same lambda), the dual update (Eq. 14), the x-update and its share of the residual
//   (Eq. 22), and tests the residual of its scene.  The values exchanged between workgroups (y,
//   the residual's partials and totals) carry their iteration's number and are written and
//   polled with agent-scope atomics, which reach the point of coherence across the chip's
//   L2 caches: no grid barrier and no device-wide cache write-back per iteration.
// fem_vhat_kernel: v_hat = K^-1 (b + J^T w) after the iteration, from the factorisation's
//   y = L^-1 P b and T = L_DD^-1 (each block's factors in the precision it was factorised in): v_D = T^T (y_D + T e_D), v_O = L_OO^-T (y_O - L_DO^T v_D).
#include <algorithm>
#include <type_traits>

#include "exchange.hpp"
#include "internal.hpp"
#include "mfma.hpp"

namespace subadmm {

namespace {

constexpr int kFemThreads = 256;
constexpr int kNb = 16;  // factorisation block size

__device__ inline void mat3_inv(const double* m, double* o, double& det) {
  det = m[0] * (m[4] * m[8] - m[5] * m[7]) - m[1] * (m[3] * m[8] - m[5] * m[6]) + m[2] * (m[3] * m[7] - m[4] * m[6]);
  const double id = 1.0 / det;
  o[0] = (m[4] * m[8] - m[5] * m[7]) * id;
  o[1] = (m[2] * m[7] - m[1] * m[8]) * id;
  o[2] = (m[1] * m[5] - m[2] * m[4]) * id;
  o[3] = (m[5] * m[6] - m[3] * m[8]) * id;
  o[4] = (m[0] * m[8] - m[2] * m[6]) * id;
  o[5] = (m[2] * m[3] - m[0] * m[5]) * id;
  o[6] = (m[3] * m[7] - m[4] * m[6]) * id;
  o[7] = (m[1] * m[6] - m[0] * m[7]) * id;
  o[8] = (m[0] * m[4] - m[1] * m[3]) * id;
}

// Orthogonal polar factor: Newton's iteration X <- (X + X^-T) / 2 from X = F (quadratic
// convergence for non-singular F); at most 60 steps.
__device__ inline bool polar_rotation(const double* F, double* R) {
  double X[9], Xi[9];
  for (int k = 0; k < 9; ++k) X[k] = F[k];
  for (int it = 0; it < 60; ++it) {
    double det;
    mat3_inv(X, Xi, det);
    if (!(det != 0.0) || !__builtin_isfinite(det)) return false;
    double diff = 0.0, nrm = 0.0;
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) {
        const double nv = 0.5 * (X[r * 3 + c] + Xi[c * 3 + r]);
        const double d = nv - X[r * 3 + c];
        diff += d * d;
        nrm += nv * nv;
        X[r * 3 + c] = nv;
      }
    if (diff <= 1e-30 * nrm) break;
  }
  for (int k = 0; k < 9; ++k) R[k] = X[k];
  return true;
}

}  // namespace

// ------------------------------------------------------------------------------------
// Assembly
// ------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(kFemThreads)
    fem_assemble_kernel(Topo t, FemModel f, const T* pos, const T* vel, double dt, double* A, double* b, double* scr,
                        int32_t* flags) {
  const int i = blockIdx.x;
  const int tid = threadIdx.x;
  const int n = t.sub_n[i];
  const int node0 = f.node_off[i];
  const int t0 = f.tet_off[i], t1 = f.tet_off[i + 1];
  const double lam = f.lame_l[i], mu = f.lame_m[i];
  // per tetrahedron: R and R P with P = V sigma (9 + 9 doubles in scratch)
  for (int e = t0 + tid; e < t1; e += blockDim.x) {
    const int32_t* vn = f.tet_node + 4 * (long)e;
    const double* g = f.tet_g + 12 * (long)e;
    double x[4][3];
    for (int a = 0; a < 4; ++a)
      for (int c = 0; c < 3; ++c) x[a][c] = (double)pos[3 * (long)vn[a] + c];
    double F[9];
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) {
        double s = 0.0;
        for (int a = 0; a < 4; ++a) s += x[a][r] * g[3 * a + c];
        F[r * 3 + c] = s;
      }
    double R[9];
    if (!polar_rotation(F, R)) {
      atomicOr(flags, FLAG_NONFINITE);
      for (int k = 0; k < 9; ++k) R[k] = (k % 4 == 0) ? 1.0 : 0.0;
    }
    double G[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int bb = 0; bb < 4; ++bb) {
      double du[3];
      for (int c = 0; c < 3; ++c)
        du[c] = R[0 * 3 + c] * x[bb][0] + R[1 * 3 + c] * x[bb][1] + R[2 * 3 + c] * x[bb][2] -
                f.rest[3 * (long)vn[bb] + c];
      for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) G[r * 3 + c] += du[r] * g[3 * bb + c];
    }
    const double V = f.tet_vol[e];
    const double tr = G[0] + G[4] + G[8];
    double P[9], RP[9];
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) P[r * 3 + c] = V * ((r == c ? lam * tr : 0.0) + mu * (G[r * 3 + c] + G[c * 3 + r]));
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) RP[r * 3 + c] = R[r * 3 + 0] * P[0 * 3 + c] + R[r * 3 + 1] * P[1 * 3 + c] + R[r * 3 + 2] * P[2 * 3 + c];
    double* o = scr + 18 * (long)e;
    for (int k = 0; k < 9; ++k) {
      o[k] = R[k];
      o[9 + k] = RP[k];
    }
  }
  double* Ai = A + t.sub_A[i];
  const long nn = (long)n * n;
  for (long k = tid; k < nn; k += blockDim.x) Ai[k] = 0.0;
  __syncthreads();
  const double h = 0.5 * dt, m2 = 2.0 / dt;
  const int p0 = f.pair_off[i], p1 = f.pair_off[i + 1];
  for (int q = p0 + tid; q < p1; q += blockDim.x) {
    const int ab = f.pair_ab[q];
    const int na = ab & 0xffff, nb = ab >> 16;
    double K[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int en = f.pent_off[q]; en < f.pent_off[q + 1]; ++en) {
      const int code = f.pent[en];
      const int e = t0 + (code >> 4);
      const int va = (code >> 2) & 3, vb = code & 3;
      const double* R = scr + 18 * (long)e;
      const double* ga = f.tet_g + 12 * (long)e + 3 * va;
      const double* gb = f.tet_g + 12 * (long)e + 3 * vb;
      const double V = f.tet_vol[e];
      double ra[3], rb[3];
      for (int r = 0; r < 3; ++r) {
        ra[r] = R[r * 3 + 0] * ga[0] + R[r * 3 + 1] * ga[1] + R[r * 3 + 2] * ga[2];
        rb[r] = R[r * 3 + 0] * gb[0] + R[r * 3 + 1] * gb[1] + R[r * 3 + 2] * gb[2];
      }
      const double dot = ga[0] * gb[0] + ga[1] * gb[1] + ga[2] * gb[2];
      for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) K[r * 3 + c] += V * (lam * ra[r] * rb[c] + mu * rb[r] * ra[c] + (r == c ? mu * dot : 0.0));
    }
    const double md = na == nb ? m2 * f.mass[node0 + na] : 0.0;
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) Ai[(long)(3 * na + r) * n + 3 * nb + c] = h * K[r * 3 + c] + (r == c ? md : 0.0);
  }
  // b = (2/t) M v + elastic forces + M g
  const int nnode = n / 3;
  for (int a = tid; a < nnode; a += blockDim.x) {
    const int gnode = node0 + a;
    const int q = f.node_diag[gnode];
    double fa[3] = {0.0, 0.0, 0.0};
    for (int en = f.pent_off[q]; en < f.pent_off[q + 1]; ++en) {
      const int code = f.pent[en];
      const int e = t0 + (code >> 4);
      const int va = (code >> 2) & 3;
      const double* RP = scr + 18 * (long)e + 9;
      const double* ga = f.tet_g + 12 * (long)e + 3 * va;
      for (int r = 0; r < 3; ++r) fa[r] -= RP[r * 3 + 0] * ga[0] + RP[r * 3 + 1] * ga[1] + RP[r * 3 + 2] * ga[2];
    }
    const double ma = f.mass[gnode];
    double* bo = b + t.sub_dof[i] + 3 * a;
    for (int c = 0; c < 3; ++c) bo[c] = m2 * ma * (double)vel[3 * (long)gnode + c] + fa[c] - (c == 2 ? ma * f.gravity : 0.0);
  }
}

// Interface errors: nodal equality e = gamma (x_p - x_q) / t, ground contact
// e = (z_p / t, 0, 0); position differences formed in FP64.
template <typename T>
__global__ void fem_rows_kernel(Topo t, FemModel f, const T* pos, double dt, T* e) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= t.n_if) return;
  T* ej = e + t.if_row[j];
  const long p = f.if_node0[j];
  if (t.if_kind[j] == KIND_CONTACT) {
    ej[0] = (T)((double)pos[3 * p + 2] / dt);
    ej[1] = (T)0;
    ej[2] = (T)0;
  } else {
    const long q = f.if_node1[j];
    for (int c = 0; c < 3; ++c) ej[c] = (T)(f.baumgarte * ((double)pos[3 * p + c] - (double)pos[3 * q + c]) / dt);
  }
}

// ------------------------------------------------------------------------------------
// Factorisation
// ------------------------------------------------------------------------------------
namespace {

// Inverse of the ib x ib (ib <= 16) lower-triangular tile at L (leading dimension ldl) into X
// (leading dimension ldx, strict upper triangle zero), one wave: lane r (mod 16) holds row r of
// the tile and column r of the inverse; forward substitution of the identity, column by column.
template <typename F>
__device__ __attribute__((noinline)) void tri_inverse(const F* L, int ldl, int ib, F* X, int ldx) {
  const int lane = threadIdx.x & 63, r = lane & 15;
  F row[16], x[16];
  static_for<16>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
    const bool in = r < ib && c <= r;
    const F v = L[in ? (long)r * ldl + c : 0];
    row[c] = in ? v : (F)0;
    x[c] = c == r ? (F)1 : (F)0;
  });
  static_for<16>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    if (j < ib) {
      x[j] /= row_bcast<j>(row[j]);
      static_for<15 - j>([&](auto qc) {
        constexpr int c = j + 1 + decltype(qc)::value;
        x[c] = tfma(-row_bcast<c>(row[j]), x[j], x[c]);
      });
    }
  });
  static_for<16>([&](auto qc) {
    constexpr int q = decltype(qc)::value;
    if (lane < ib && q < ib) X[(long)q * ldx + r] = q >= r ? x[q] : (F)0;
  });
}

}  // namespace

// Factor precision F.  F = float is a trial on every block: after its Cholesky factor it
// takes kappa_est = (max_r L_rr / min_r L_rr)^2, a lower bound on the condition number of K
// (every pivot L_rr^2 lies between K's extreme eigenvalues); when kappa_est > kmax or a pivot
// is not positive it records the block for FP64 (prec = 1) and stops before writing what the
// FP64 run reads again (b, and A, which later holds T), else it completes in FP32 (prec = 0),
// its L and T kept as FP32 in the same buffers.  F = double with gate = 1 runs only the
// blocks the trial recorded; with gate = 0 it runs every block and records prec = 1 and its
// own kappa_est.
//
// One block's factorisation is bound by the latency of its chain (load a tile row, multiply,
// diagonal tile, next panel), two blocks a CU for 512 of them: eight waves, four tiles of loads
// in flight per wave, the diagonal tile in registers (~6,400 cycles) beside the other tile rows of
// its panel, and column blocks of T that a wave carries through without a barrier.  Measured,
// FP64: 20 blocks of 225 DOFs 859 -> 231 us, 512 blocks of 375 DOFs 2868 -> 1685 us (before: four
// waves, a load per product waited for, the diagonal tile in LDS column by column).
constexpr int kFemFactorThreads = 512;
template <typename T, typename F>
__global__ void __launch_bounds__(kFemFactorThreads, 4)
    fem_factor_kernel(Topo t, FemModel f, const double* A, double* b, double rho, T* beta, double* L, double* Tw,
                      T* S, T* cd, int32_t* flags, int32_t* prec, double* kest, double kmax, int gate) {
  typedef Mfma<F> M;
  typedef typename M::V V;
  constexpr bool kTrial = sizeof(F) == sizeof(float);
  constexpr int kPad = 16 / (int)sizeof(F);  // panel rows 16 bytes apart in the banks
  __shared__ int s_bad;
  extern __shared__ __align__(16) double fsm_raw[];
  F* fsm = reinterpret_cast<F*>(fsm_raw);
  const int i = blockIdx.x;
  if (!kTrial && gate && prec[i] == 0) return;
  const int tid = threadIdx.x;
  const int bd = blockDim.x;
  const int n = t.sub_n[i];
  const int m = f.m[i];
  const int o = n - m;
  const int nc = t.sub_nc[i];
  const int dof0 = t.sub_dof[i];
  const double* Ai = A + t.sub_A[i];
  F* Li = reinterpret_cast<F*>(L + t.sub_A[i]);
  const int32_t* perm = f.perm + dof0;
  const int pn = n > 32 ? n : 32;   // panel columns (at least 32)
  F* dinv = fsm;                    // 16 x 16: the diagonal tile, then its factor's inverse
  F* panel = dinv + kNb * kNb;      // kNb x (pn + kPad): one row panel of L
  F* vec = panel + (long)(pn + kPad) * kNb;  // n
  if (tid == 0) s_bad = 0;

  // Eq. (23): beta = Tr(A) / Tr(J^T J), Tr(J^T J) = slot rows (each selects one DOF); in
  // FP64 for either F (the first 256 doubles of LDS, before anything else uses them)
  double* redd = fsm_raw;
  if (tid < kFemThreads) {
    double tr = 0.0;
    for (int r = tid; r < n; r += kFemThreads) tr += Ai[(long)r * n + r];
    redd[tid] = tr;
  }
  __syncthreads();
  for (int s = kFemThreads / 2; s > 0; s >>= 1) {
    if (tid < s) redd[tid] += redd[tid + s];
    __syncthreads();
  }
  const double be = rho > 0.0 ? rho : (nc > 0 ? redd[0] / (double)nc : 1.0);
  __syncthreads();
  if (tid == 0) beta[i] = (T)be;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), nwv = bd >> 6;

  // K = P (A + beta J^T J) P^T, lower triangle: a wave per four rows, lanes along them (the rows
  // of A are gathered through the permutation, kept in LDS), eight loads in flight
  {
    int* pl = reinterpret_cast<int*>(vec);
    for (int r = tid; r < n; r += bd) pl[r] = perm[r];
    __syncthreads();
    for (int r0 = 4 * wv; r0 < n; r0 += 4 * nwv)
      for (int c0 = 0; c0 < r0 + 4 && c0 < n; c0 += 128) {
        double v[4][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c = c0 + 64 * h + lane;
          const int pc = pl[c < n ? c : 0];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int r = r0 + q;
            v[q][h] = Ai[r < n && c <= r ? (long)pl[r] * n + pc : 0];
          }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int r = r0 + q, c = c0 + 64 * h + lane;
            if (r < n && c <= r) {
              double k = v[q][h];
              if (c == r) k += be * (double)f.jtj[dof0 + pl[r]];
              Li[(long)r * n + c] = (F)k;
            }
          }
      }
    __syncthreads();
  }

  // Left-looking blocked Cholesky on the matrix cores, 16-column panels J: every tile row
  // I >= J first forms U_IJ = K_IJ - sum_{K<J} L_IK L_JK^T (the row panel L_J,<J staged in
  // LDS, shared by the waves), then the diagonal tile is factorised (the wave that formed it, while
  // the others form theirs) and L_IJ = U_IJ L_JJ^-T for I > J.  b (permuted) is carried as one
  // more row, below the matrix, so its factor row is y = L^-1 b (forward substitution for
  // free).  K is read once and every L tile written once (the right-looking update read and
  // wrote the whole trailing matrix per panel); a wave keeps its first kKeep tiles U_IJ in
  // registers in between (4 cover blocks of up to 464 DOFs), further ones in their place.
  constexpr int kKeep = 4;
  F* yrow = vec;  // LDS, n (the permutation list kept there is no longer needed)
  for (int c = tid; c < n; c += bd) yrow[c] = (F)b[dof0 + perm[c]];
  double* yout = b + dof0;
  const int nbn = (n + kNb - 1) / kNb;  // tile rows of K; tile row nbn holds b's row alone
  const int g = lane >> 4, cn = lane & 15;
  __syncthreads();
  for (int J = 0; J < nbn; ++J) {
    const int j0 = J * kNb, jb = min(kNb, n - j0), ps = j0 + kPad;
    // stage L_J,<J (jb x j0) in LDS
    for (int rr = wv; rr < jb; rr += nwv) {
      const F* src = Li + (long)(j0 + rr) * n;
#pragma unroll 4
      for (int c = lane; c < j0; c += 64) panel[rr * ps + c] = src[c];
    }
    __syncthreads();
    // U_IJ of one tile row: the lane holds U_IJ[cn][k(r, g)], r = 0..3, of the row at Ri (a lane
    // beyond the tile's rows or columns computes with valid entries that are not used)
    auto u_tile = [&](auto Ri) -> V {
      F kij[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = M::k(r, g);
        kij[r] = Ri[j0 + (c < jb ? c : 0)];
      }
      V acc = {0, 0, 0, 0};
      const F* pr = panel + cn * ps + 4 * g;
      auto Rk = Ri + 4 * g;
      auto step = [&](auto uc, int K) {
        constexpr int U = decltype(uc)::value;
        F av[U][4], bv[U][4];
#pragma unroll
        for (int q = 0; q < U; ++q)
#pragma unroll
          for (int s2 = 0; s2 < 4; ++s2) bv[q][s2] = Rk[(K + q) * kNb + s2];  // L_IK[cn][k]
#pragma unroll
        for (int q = 0; q < U; ++q)
#pragma unroll
          for (int s2 = 0; s2 < 4; ++s2) av[q][s2] = pr[(K + q) * kNb + s2];  // L_JK[cn][k]
#pragma unroll
        for (int q = 0; q < U; ++q) acc = M::mul(av[q], bv[q], acc);  // (L_IK L_JK^T)[cn][k(r, g)]
      };
      int K = 0;
      for (; K + 4 <= J; K += 4) step(std::integral_constant<int, 4>{}, K);
      for (; K < J; ++K) step(std::integral_constant<int, 1>{}, K);
      V u;
#pragma unroll
      for (int r = 0; r < 4; ++r) u[r] = kij[r] - acc[r];
      return u;
    };
    // L_IJ of one tile row from U_IJ, ib rows at Ri (leading dimension n)
    auto l_tile = [&](const V& u, auto Ri, int ib) {
      F av[4], bv[4];
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        const int c = M::k(s2, g);
        av[s2] = c < jb ? u[s2] : (F)0;  // U_IJ[cn][c]
        bv[s2] = dinv[cn * kNb + c];     // (L_JJ^-T)[c][cn]
      }
      V out = {0, 0, 0, 0};
      out = M::mul(av, bv, out);  // lane register r: L_IJ[k(r, g)][cn]
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rr = M::k(r, g);
        if (rr < ib && cn < jb) Ri[(long)rr * n + j0 + cn] = out[r];
      }
    };
    V keep[kKeep];
    if (wv == 0) {
      const V u = u_tile(Li + (long)(j0 + (cn < jb ? cn : 0)) * n);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = M::k(r, g);
        dinv[cn * kNb + c] = cn < jb && c <= cn ? u[r] : (F)0;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (!diag_tile<F, F*, F*>(dinv, kNb, jb, Li + (long)j0 * n + j0, n) && lane == 0) {
        if (kTrial)
          s_bad = 1;
        else
          atomicOr(flags, FLAG_NOT_SPD);
      }
    } else {
      static_for<kKeep>([&](auto tc) {
        constexpr int q = decltype(tc)::value;
        const int I = J + wv + (nwv - 1) * q, i0 = I * kNb;
        if (I < nbn)
          keep[q] = u_tile(Li + (long)min(i0 + cn, n - 1) * n);
        else if (I == nbn)
          keep[q] = u_tile(yrow);
      });
      for (int I = J + wv + (nwv - 1) * kKeep; I <= nbn; I += nwv - 1) {
        const int i0 = I * kNb;
        auto out_of_place = [&](auto Ri, bool in) {
          const V u = u_tile(Ri);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (in && M::k(r, g) < jb) Ri[j0 + M::k(r, g)] = u[r];
        };
        if (I < nbn)
          out_of_place(Li + (long)min(i0 + cn, n - 1) * n, i0 + cn < n);
        else
          out_of_place(yrow, cn == 0);
      }
    }
    __syncthreads();
    if (wv > 0) {
      static_for<kKeep>([&](auto tc) {
        constexpr int q = decltype(tc)::value;
        const int I = J + wv + (nwv - 1) * q, i0 = I * kNb;
        if (I < nbn)
          l_tile(keep[q], Li + (long)i0 * n, min(kNb, n - i0));
        else if (I == nbn)
          l_tile(keep[q], yrow, 1);
      });
      for (int I = J + wv + (nwv - 1) * kKeep; I <= nbn; I += nwv - 1) {
        const int i0 = I * kNb;
        auto in_place = [&](auto Ri, auto R0, int ib) {
          V u;
#pragma unroll
          for (int r = 0; r < 4; ++r) u[r] = Ri[j0 + (M::k(r, g) < jb ? M::k(r, g) : 0)];
          l_tile(u, R0, ib);
        };
        if (I < nbn)
          in_place(Li + (long)min(i0 + cn, n - 1) * n, Li + (long)i0 * n, min(kNb, n - i0));
        else
          in_place(yrow, yrow, 1);
      }
    }
    __syncthreads();
  }

  // kappa_est from the factor's diagonal (each wave reduces its share, then every thread
  // combines the waves' values in the same order)
  {
    F dmx = 0, dmn = 0;
    bool any = false;
    for (int r = tid; r < n; r += bd) {
      const F d = Li[(long)r * n + r];
      dmx = any ? (d > dmx ? d : dmx) : d;
      dmn = any ? (d < dmn ? d : dmn) : d;
      any = true;
    }
    double mx = any ? (double)dmx : 0.0, mn = any ? (double)dmn : __builtin_inf();
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      mx = fmax(mx, __shfl_xor(mx, off));
      mn = fmin(mn, __shfl_xor(mn, off));
    }
    double* kr = reinterpret_cast<double*>(dinv);  // dinv is not needed after the factor
    if (lane == 0) {
      kr[2 * wv] = mx;
      kr[2 * wv + 1] = mn;
    }
    __syncthreads();
    mx = kr[0];
    mn = kr[1];
    for (int w = 1; w < nwv; ++w) {
      mx = fmax(mx, kr[2 * w]);
      mn = fmin(mn, kr[2 * w + 1]);
    }
    const double ratio = mx / mn;
    const double kap = ratio * ratio;
    const bool to64 = kTrial && (s_bad != 0 || !(kap <= kmax));
    if (tid == 0 && (kTrial || !gate)) {
      prec[i] = kTrial ? (to64 ? 1 : 0) : 1;
      kest[i] = s_bad != 0 ? __builtin_inf() : kap;
    }
    if (to64) return;  // uniform over the workgroup
  }

  // T = L_DD^-1 (m x m lower, in this block's A storage: m^2 <= n^2), by 16-row blocks:
  // T_II = L_II^-1, then for I > J  T_IJ = -T_II sum_{K=J}^{I-1} L_IK T_KJ, column block by
  // column block: one wave forms a column block from its diagonal down (no barrier), every
  // 16 x 16 product on the matrix cores.  The long column blocks are dealt first.
  F* Ti = reinterpret_cast<F*>(Tw + t.sub_A[i]);
  const int nbk = (m + kNb - 1) / kNb;
  const F* Ld = Li + (long)o * n + o;  // L_DD[r][c] = Ld[r * n + c]
  for (int I = wv; I < nbk; I += nwv) {
    const int i0 = I * kNb;
    tri_inverse<F>(Ld + (long)i0 * n + i0, n, min(kNb, m - i0), Ti + (long)i0 * m + i0, m);
  }
  __syncthreads();
  for (int q = 0; q * nwv < nbk; ++q) {
    const int J = q * nwv + ((q & 1) ? nwv - 1 - wv : wv);
    const int j0 = J * kNb;  // a full block where J < nbk - 1
    for (int I = J + 1; I < nbk; ++I) {
      const int i0 = I * kNb, ib = min(kNb, m - i0);
      const F* Lr = Ld + (long)(i0 + (cn < ib ? cn : 0)) * n;
      F tv[4];
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        const int kk = M::k(s2, g);
        const F v = Ti[(long)(i0 + (cn < ib ? cn : 0)) * m + i0 + (kk < ib ? kk : 0)];
        tv[s2] = kk < ib ? v : (F)0;
      }
      V acc = {0, 0, 0, 0};
      auto step = [&](auto uc, int K) {
        constexpr int U = decltype(uc)::value;
        F av[U][4], bv[U][4];
#pragma unroll
        for (int q2 = 0; q2 < U; ++q2)
#pragma unroll
          for (int s2 = 0; s2 < 4; ++s2) {
            const int kk = (K + q2) * kNb + M::k(s2, g);  // K < I: a full block
            av[q2][s2] = Lr[kk];
            bv[q2][s2] = Ti[(long)kk * m + j0 + cn];
          }
#pragma unroll
        for (int q2 = 0; q2 < U; ++q2) acc = M::mul(av[q2], bv[q2], acc);
      };
      int K = J;
      for (; K + 4 <= I; K += 4) step(std::integral_constant<int, 4>{}, K);
      for (; K < I; ++K) step(std::integral_constant<int, 1>{}, K);
      // T_IJ = -T_II acc: acc (lane: rows k(r, g) of column cn) is the B operand as it stands
      F bv[4];
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) bv[s2] = acc[s2];
      V out = {0, 0, 0, 0};
      out = M::mul(tv, bv, out);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = M::k(r, g);
        if (row < ib) Ti[(long)(i0 + row) * m + j0 + cn] = -out[r];
      }
      // the next row blocks read this one back in other lanes
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
  }
  __syncthreads();

  // S = T^T T, lower 16 x 16 tiles: S_IJ = sum_{K >= I} T_KI^T T_KJ, a wave per tile.  Tile
  // layout of the iteration: entry (R, C) at ((R >> 2) * 16 + C) * 4 + (R & 3), so lane l
  // holds rows 16 I + 4 (l / 16) + k of column 16 J + l % 16 as four consecutive entries.
  T* Si = S + f.sq_off[i];
  const int ntile = nbk * (nbk + 1) / 2;
  for (int tt = wv; tt < ntile; tt += nwv) {
    int I = 0;
    while ((I + 1) * (I + 2) / 2 <= tt) ++I;
    const int J = tt - I * (I + 1) / 2;
    const int a0 = I * kNb, b0 = J * kNb;
    const F* Ta = Ti + (a0 + cn < m ? a0 + cn : a0);
    const F* Tb = Ti + (b0 + cn < m ? b0 + cn : b0);
    V acc = {0, 0, 0, 0};
    auto step = [&](auto uc, int K) {  // full row blocks
      constexpr int U = decltype(uc)::value;
      F av[U][4], bv[U][4];
#pragma unroll
      for (int q2 = 0; q2 < U; ++q2)
#pragma unroll
        for (int s2 = 0; s2 < 4; ++s2) {
          const int kk = (K + q2) * kNb + M::k(s2, g);
          av[q2][s2] = Ta[(long)kk * m];
          bv[q2][s2] = Tb[(long)kk * m];
        }
#pragma unroll
      for (int q2 = 0; q2 < U; ++q2) acc = M::mul(av[q2], bv[q2], acc);
    };
    int K = I;
    for (; K + 4 <= nbk - 1; K += 4) step(std::integral_constant<int, 4>{}, K);
    for (; K < nbk - 1; ++K) step(std::integral_constant<int, 1>{}, K);
    {  // the last row block
      F av[4], bv[4];
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        const int kk = K * kNb + M::k(s2, g);
        const F va = Ta[(long)(kk < m ? kk : 0) * m], vb = Tb[(long)(kk < m ? kk : 0) * m];
        av[s2] = kk < m ? va : (F)0;
        bv[s2] = kk < m ? vb : (F)0;
      }
      acc = M::mul(av, bv, acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = M::k(r, g);  // entry (row, cn) of the tile
      Si[(long)tt * 256 + (((row >> 2) * 16 + cn) << 2) + (row & 3)] =
          (a0 + row < m && b0 + cn < m) ? (T)acc[r] : (T)0;
    }
  }

  // y = L^-1 P b (permuted order) replaces b in its storage (b is not read again this step)
  for (int c = tid; c < n; c += bd) yout[c] = (double)yrow[c];
  // c = K^-1 b on the constrained DOFs (the last m of the permuted order): with y = L^-1 b,
  // c_D = L_DD^-T y_D = T^T y_D
  for (int j = tid; j < m; j += bd) {
    double v = 0.0;
    int k = j;
    for (; k + 8 <= m; k += 8) {
      F tk[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) tk[q] = Ti[(long)(k + q) * m + j];
#pragma unroll
      for (int q = 0; q < 8; ++q) v += (double)tk[q] * (double)yrow[o + k + q];
    }
    for (; k < m; ++k) v += (double)Ti[(long)k * m + j] * (double)yrow[o + k];
    cd[f.dkey_off[i] + j] = (T)v;
  }
}

// v_hat = K^-1 (b + J^T w), original DOF order, from what the factorisation kept: y = L^-1 P b
// (permuted order, in b's storage) and T = L_DD^-1 (in A's storage).  With e = P J^T w, which
// is non-zero on the constrained DOFs only, L^-1 (P b + e) = y + [0; T e_D], hence
//   v_D = L_DD^-T (y_D + T e_D) = T^T (y_D + T e_D),   v_O = L_OO^-T (y_O - L_DO^T v_D).
namespace {

// One DPP step on a double (both 32-bit halves moved by the same control).
template <int kCtrl, int kRowMask>
__device__ inline double dpp_double(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), kCtrl, kRowMask, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, kRowMask, 0xF, false);
  return __longlong_as_double(((long long)(unsigned)hi << 32) | (long long)(unsigned)lo);
}

// Sum over the 64 lanes of a wave in a fixed order (DPP only): pairs, quads, half rows and
// rows of 16, then rows 0+1 into row 1 and rows 0..3 into row 3; lane 63 holds the total.
__device__ inline double wave_sum_lane63(double v) {
  v += dpp_double<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
  v += dpp_double<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
  v += dpp_double<0x141, 0xF>(v);  // row_half_mirror
  v += dpp_double<0x140, 0xF>(v);  // row_mirror
  v += dpp_double<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_double<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Value of one lane (uniform index) in all lanes.
__device__ inline double wave_lane(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

constexpr int kVhatParts = 4;

// kVhatParts partial sums of out[j] = sum_{k in [lo(j), m)} M[k ld + j] x[k], j < cols, by waves: a wave
// per 64 columns and part of the rows, eight loads in flight; part p's sum goes to part[p cols + j].
template <bool kLower, typename F>
__device__ inline void vhat_columns(const F* M, long ld, int cols, int rows, const double* x, double* part) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nwv = blockDim.x >> 6;
  const int chunks = (cols + 63) / 64, per = (rows + kVhatParts - 1) / kVhatParts;
  for (int c = wv; c < chunks * kVhatParts; c += nwv) {
    const int p = c / chunks, j = (c - p * chunks) * 64 + lane;
    if (j >= cols) continue;
    int k = p * per;
    const int end = min(k + per, rows);
    if (kLower && j > k) k = j;
    double s = 0.0;
    for (; k + 8 <= end; k += 8) {
      F v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = M[(k + q) * ld + j];
#pragma unroll
      for (int q = 0; q < 8; ++q) s = __builtin_fma((double)v[q], x[k + q], s);
    }
    for (; k < end; ++k) s = __builtin_fma((double)M[k * ld + j], x[k], s);
    part[p * cols + j] = s;
  }
}

// The v_hat solve of one block with its factors L, T stored in precision F (sums in FP64).
// Bound by the latency of its chain of products and of the back substitution: rows of T across
// the lanes of a wave and its columns in four parts of the sum (both read whole lines, many loads
// in flight), and the back substitution by 64 columns, in registers within them.  Measured, FP64
// factors: 20 blocks of 225 DOFs 63 -> 26 us, 512 blocks of 375 DOFs 325 -> 105 us (before: a thread
// per row or column, one load at a time, and a step of the back substitution per column).
template <typename T, typename F>
__device__ inline void fem_vhat_block(const Topo& t, const FemModel& f, int i, const F* Li, const F* Ti,
                                      const double* yb, const T* w, T* v_hat, double* vsm) {
  const int tid = threadIdx.x;
  const int bd = blockDim.x;
  const int n = t.sub_n[i];
  const int m = f.m[i];
  const int o = n - m;
  const int dof0 = t.sub_dof[i];
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), nwv = bd >> 6;
  const int32_t* perm = f.perm + dof0;
  const double* yi = yb + dof0;
  double* v = vsm;                    // n, permuted order
  double* ed = v + n;                 // m: e_D
  double* zd = ed + m;                // m: y_D + T e_D
  double* part = zd + m;              // kVhatParts x max(m, o)
  for (int k = tid; k < m; k += bd) {
    const int g = f.dkey_off[i] + k;
    double s = 0.0;
    for (int q = f.dk_off[g]; q < f.dk_off[g + 1]; ++q) {
      const int sl = f.dk_slot[q];
      s += (double)f.slot_sgn[sl] * (double)w[sl];
    }
    ed[k] = s;
  }
  __syncthreads();
  // z_D = y_D + T e_D: a wave per four rows
  for (int k0 = 4 * wv; k0 < m; k0 += 4 * nwv) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int p = lane; p < k0 + 4; p += 64) {
      F tv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool in = k0 + q < m && p <= k0 + q;
        tv[q] = Ti[in ? (long)(k0 + q) * m + p : 0];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (k0 + q < m && p <= k0 + q) s[q] = __builtin_fma((double)tv[q], ed[p], s[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double r = wave_sum_lane63(s[q]);
      if (lane == 63 && k0 + q < m) zd[k0 + q] = yi[o + k0 + q] + r;
    }
  }
  __syncthreads();
  vhat_columns<true, F>(Ti, m, m, m, zd, part);
  __syncthreads();
  for (int j = tid; j < m; j += bd) {
    double s = 0.0;
    for (int p = 0; p < kVhatParts; ++p) s += part[p * m + j];
    v[o + j] = s;
  }
  __syncthreads();
  vhat_columns<false, F>(Li + (long)o * n, n, o, m, v + o, part);
  __syncthreads();
  for (int c = tid; c < o; c += bd) {
    double s = 0.0;
    for (int p = 0; p < kVhatParts; ++p) s += part[p * o + c];
    v[c] = yi[c] - s;
  }
  __syncthreads();
  // L_OO^T v_O = (y_O - L_DO^T v_D): back substitution, 64 columns at a time from the last.  Within
  // them one wave, lane r holding column c0 + r; the rest of the columns by the workgroup.
  for (int c0 = (o - 1) & ~63; c0 >= 0; c0 -= 64) {
    const int cw = min(64, o - c0);
    const F* Lc = Li + (long)c0 * n + c0;
    if (wv == 0) {
      double x = lane < cw ? v[c0 + lane] : 0.0;
      const double dg = lane < cw ? (double)Lc[(long)lane * n + lane] : 1.0;
      const double inv = 1.0 / dg;
      for (int cb = (cw - 1) & ~7; cb >= 0; cb -= 8) {
        F row[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) row[q] = Lc[cb + q < cw && lane < cb + q ? (long)(cb + q) * n + lane : 0];
#pragma unroll
        for (int q = 7; q >= 0; --q) {
          if (cb + q < cw) {
            // the quotient, corrected by its remainder
            const double y0 = x * inv;
            const double y1 = __builtin_fma(__builtin_fma(-dg, y0, x), inv, y0);
            const double vc = wave_lane(y1, cb + q);
            x = lane == cb + q ? y1 : lane < cb + q ? __builtin_fma(-(double)row[q], vc, x) : x;
          }
        }
      }
      if (lane < cw) v[c0 + lane] = x;
    }
    __syncthreads();
    for (int r = tid; r < c0; r += bd) {
      double s = v[r];
      const F* Lr = Li + (long)c0 * n + r;
      int c = cw - 1;
      for (; c >= 7; c -= 8) {
        F lv[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) lv[q] = Lr[(long)(c - q) * n];
#pragma unroll
        for (int q = 0; q < 8; ++q) s = __builtin_fma(-(double)lv[q], v[c0 + c - q], s);
      }
      for (; c >= 0; --c) s = __builtin_fma(-(double)Lr[(long)c * n], v[c0 + c], s);
      v[r] = s;
    }
    __syncthreads();
  }
  for (int r = tid; r < n; r += bd) v_hat[dof0 + perm[r]] = (T)v[r];
}

}  // namespace

// prec[i] (written by the factorisation): 1 = the block's L and T are FP64, 0 = FP32.
template <typename T>
__global__ void __launch_bounds__(kFemFactorThreads)
    fem_vhat_kernel(Topo t, FemModel f, const double* L, const double* Tw, const double* yb, const int32_t* prec,
                    const T* w, T* v_hat) {
  extern __shared__ __align__(16) double vsm[];
  const int i = blockIdx.x;
  if (prec[i])
    fem_vhat_block<T, double>(t, f, i, L + t.sub_A[i], Tw + t.sub_A[i], yb, w, v_hat, vsm);
  else
    fem_vhat_block<T, float>(t, f, i, reinterpret_cast<const float*>(L + t.sub_A[i]),
                             reinterpret_cast<const float*>(Tw + t.sub_A[i]), yb, w, v_hat, vsm);
}

// ------------------------------------------------------------------------------------
// Iteration
// ------------------------------------------------------------------------------------
namespace {

// Values exchanged between the workgroups of the iteration are tagged words (Tagged): the
// number of the iteration travels with the value, so a reader polls the value itself: no
// barrier, no counters, nothing to reset.
//   y (per slot row): two buffers by iteration parity.  A block writes y of iteration l + 2
//     after its z-update of l + 1, for which it needed the neighbour's y of l + 1, written
//     after the neighbour's z-update of l: the entry of iteration l has been read.
//   residual partials (per block) and totals (per scene): rings of kRing.  The partial of l + 4
//     is written after the block's test of l + 1, whose total the scene's first block
//     wrote after it had read every partial of l; the total of l + 4 after every block wrote
//     its partial of l + 4, which it did after its test of l.
constexpr int kRing = 4;
// polls per wait before a workgroup gives up (FLAG_BARRIER)
constexpr long kMaxPolls = 1l << 24;

template <typename T>
__device__ inline T fsqrt(T x);
template <>
__device__ inline float fsqrt<float>(float x) { return __builtin_sqrtf(x); }
template <>
__device__ inline double fsqrt<double>(double x) { return __builtin_sqrt(x); }

// Wave totals of two values to sums[0], sums[1].
__device__ inline void wave_sums(double v0, double v1, double* sums) {
  v0 = wave_sum_lane63(v0);
  v1 = wave_sum_lane63(v1);
  if ((threadIdx.x & 63) == 63) {
    sums[0] = v0;
    sums[1] = v1;
  }
}
// True in the wave that arrives last of a power of two of waves, which then sees what each wrote to
// LDS before it arrived (no barrier).
__device__ inline bool arrive_last(int* arrived, int waves) {
  int n = 0;
  if ((threadIdx.x & 63) == 63) n = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
  n = __builtin_amdgcn_readlane(n, 63);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return (n & (waves - 1)) == waves - 1;
}

constexpr int kMaxFemSlots = 512;  // slot rows per block (two per thread)

// Sum over the 16 lanes of each row of the wave (every lane receives its row's sum).  The
// pairing (lanes 8 apart, then 4, 2, 1 apart within the row) is the same for both forms.
__device__ inline float row_sum16(float x) {
  // DPP row rotations by 8, 4, 2, 1 lanes (row_ror:n = 0x120 + n)
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x124, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x122, 0xf, 0xf, false));
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x121, 0xf, 0xf, false));
  return x;
}
__device__ inline double row_sum16(double x) {
  x += __shfl_xor(x, 8, 64);
  x += __shfl_xor(x, 4, 64);
  x += __shfl_xor(x, 2, 64);
  x += __shfl_xor(x, 1, 64);
  return x;
}

// Four consecutive entries of a 16-byte-aligned row.
template <typename T>
struct Quad;
template <>
struct Quad<float> {
  float4 v;
  __device__ void load(const float* p) { v = *reinterpret_cast<const float4*>(p); }
  __device__ void fma(float r, float* acc) const {
    acc[0] += v.x * r;
    acc[1] += v.y * r;
    acc[2] += v.z * r;
    acc[3] += v.w * r;
  }
  __device__ void store(float* p) const { *reinterpret_cast<float4*>(p) = v; }
  __device__ void zero() { v = make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ void to(float* o) const {
    o[0] = v.x;
    o[1] = v.y;
    o[2] = v.z;
    o[3] = v.w;
  }
};
template <>
struct Quad<double> {
  double2 a, b;
  __device__ void load(const double* p) {
    a = *reinterpret_cast<const double2*>(p);
    b = *reinterpret_cast<const double2*>(p + 2);
  }
  __device__ void fma(double r, double* acc) const {
    acc[0] += a.x * r;
    acc[1] += a.y * r;
    acc[2] += b.x * r;
    acc[3] += b.y * r;
  }
  __device__ void zero() {
    a = make_double2(0.0, 0.0);
    b = a;
  }
  __device__ void store(double* p) const {
    *reinterpret_cast<double2*>(p) = a;
    *reinterpret_cast<double2*>(p + 2) = b;
  }
  __device__ void to(double* o) const {
    o[0] = a.x;
    o[1] = a.y;
    o[2] = b.x;
    o[3] = b.y;
  }
};

}  // namespace

// Operator-product schedules.  A block's S is stored as its lower 16 x 16 tiles in row
// order; the four waves of the workgroup split the tiles of a block with MT tile rows
// evenly in that order.  In the fixed-size forms (template MT > 0, blocks of at most MT tile
// rows, rows beyond the block's own skipped) every tile's row and column are compile-time
// constants, so a tile costs its eight FMAs and nothing else: the lane's rd entries of
// every tile column, its column sums and the tile operands sit in registers under fixed
// names.  Resident form (R > 0): each wave keeps its first R tiles in registers and the
// rest in LDS for the whole step; R = 0 reads them from device memory every iteration.
constexpr int kResTiles = 35;
constexpr int kMtClasses[] = {8, 12, 16, 19};

__host__ __device__ constexpr int tri_row(int t) {
  int I = 0;
  while ((I + 1) * (I + 2) / 2 <= t) ++I;
  return I;
}
__host__ __device__ constexpr int wave_tile_beg(int mt, int w) { return (mt * (mt + 1) / 2) * w / 4; }
__host__ __device__ constexpr int wave_tile_count(int mt, int w) {
  return wave_tile_beg(mt, w + 1) - wave_tile_beg(mt, w);
}
// LDS tiles of the resident form kept by the waves before wave w
__host__ __device__ constexpr int lds_tiles_before(int mt, int R, int w) {
  int n = 0;
  for (int v = 0; v < w; ++v) n += wave_tile_count(mt, v) > R ? wave_tile_count(mt, v) - R : 0;
  return n;
}

// Tile arithmetic as chains of explicit fused multiply-adds (no separate multiplies or
// adds the compiler could fuse differently in different instantiations), so every form of
// the product rounds identically.
__device__ inline float fmat(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fmat(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <typename T>
__device__ inline T dot4_acc(const T* e, const T* r, T acc) {
  return fmat(e[3], r[3], fmat(e[2], r[2], fmat(e[1], r[1], fmat(e[0], r[0], acc))));
}

template <typename T>
struct MatvecArgs {
  const T* rd;   // LDS, 16 MT entries (zero beyond m)
  T* ow;         // LDS, this wave's 16 MT partial products
  const T* sg;   // block's tiles in device memory, + 4 lane
  const T* sl;   // this wave's LDS tiles
  int mt;
};

// Loads wave W's tiles before the iteration (resident form).
template <typename T, int MT, int R, int W>
__device__ __forceinline__ void load_tiles(Quad<T>* sreg, const MatvecArgs<T>& c) {
  constexpr int beg = wave_tile_beg(MT, W), cnt = wave_tile_count(MT, W), RR = R < cnt ? R : cnt;
  static_for<cnt>([&](auto rc) {
    constexpr int r = decltype(rc)::value, t = beg + r, I = tri_row(t);
    if constexpr (r < RR) {
      if (I < c.mt) sreg[r].load(c.sg + (long)t * 256); else sreg[r].zero();
    } else {
      // rows beyond the block's own are stored as zero tiles
      Quad<T> v;
      if (I < c.mt) v.load(c.sg + (long)t * 256); else v.zero();
      v.store(const_cast<T*>(c.sl) + 4 * (threadIdx.x & 63) + (r - RR) * 256);
    }
  });
}

// lanes' values a, b: rows of 16 lanes 1, 3 of a exchanged with rows 0, 2 of b
__device__ inline void swap_rows16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
// the upper half of a exchanged with the lower half of b
__device__ inline void swap_rows32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// One wave's share of S rd (fixed-size form): tile (I, J) adds T rd_J to rows I and, below the
// diagonal, T^T rd_I to rows J.  Row sums are reduced over the 16 lanes of a row when the tile
// row (or the wave's range) ends; column sums stay per lane and are added at the end, one
// row group after another, four columns at a time by lane-row exchanges (no LDS), which
// leaves lane row g with column 4 q + g.  Which entries of ow a wave writes is fixed: the
// others hold zero from the start of the step.
// A tile costs its eight FMAs (32 cycles) and nothing else (rd is zero-padded to MT rows), the
// four row sums of a tile row are reduced side by side.  Measured for blocks of 267 constrained DOFs, two workgroups per
// CU: 10,250 cycles with a branch per tile and LDS exchanges per column, 3,300 to 4,100 now.
template <int MT, int R, int W>
__device__ __forceinline__ void matvec_fixed(const Quad<float>* sreg, const MatvecArgs<float>& c) {
  constexpr int beg = wave_tile_beg(MT, W), cnt = wave_tile_count(MT, W), RR = R < cnt ? R : cnt;
  constexpr int end = beg + cnt, Ib = tri_row(beg), Ie = tri_row(end - 1);
  int lane = (int)threadIdx.x & 63;
  asm volatile("" : "+v"(lane));  // the lane's addresses are formed here, not held over the iteration
  const int g4 = lane >> 4, cc = lane & 15;
  const float* sl = c.sl + 4 * lane;
  float rdl[Ie + 1], cacc[4 * ((Ie + 3) / 4) + 1];
  static_for<Ie + 1>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    rdl[j] = c.rd[16 * j + cc];
  });
  static_for<4 * ((Ie + 3) / 4)>([&](auto jc) { cacc[decltype(jc)::value] = 0.f; });
  const float4* rq = reinterpret_cast<const float4*>(c.rd) + g4;
  float4 rin = rq[4 * Ib];
  // tiles not in registers (LDS, or device memory when R = 0) are read PD tiles ahead into
  // a ring of registers; scheduling barriers at the tile boundaries keep the compiler from
  // hoisting further loads (which would cost registers the resident tiles need)
  constexpr int PD = R > 0 ? 2 : 8;
  Quad<float> pf[PD];
  // the device-memory tile addresses and the row tests are formed here, in the iteration, from
  // opaque copies (otherwise they are hoisted out of the iteration loop and held in registers)
  const float* sgp = nullptr;
  int mt = c.mt;
  if constexpr (R == 0) {
    sgp = c.sg;
    asm volatile("" : "+v"(sgp));
    asm volatile("" : "+s"(mt));
  }
  auto fetch = [&](auto qc) {
    constexpr int q = decltype(qc)::value, tq = beg + q;
    if constexpr (q >= RR && q < cnt) {
      if constexpr (R > 0)
        pf[q % PD].load(sl + (q - RR) * 256);  // zero tiles beyond the block's rows
      else
        pf[q % PD].load(sgp + (tri_row(tq) < mt ? (long)tq * 256 : 0l));  // not used beyond them
    }
  };
  // tile q is fetched at position q - PD; the first PD positions are fetched here
  static_for<PD>([&](auto qc) { fetch(qc); });
  static_for<Ie - Ib + 1>([&](auto ic) {
    constexpr int I = Ib + decltype(ic)::value, first = I * (I + 1) / 2;
    constexpr int t0 = first > beg ? first : beg, t1 = first + I + 1 < end ? first + I + 1 : end;
    // the resident form's tiles beyond the block's rows are zero: no branch, so that the reduction
    // of one row overlaps the products of the next
    if (R > 0 || I < mt) {
      const float ri[4] = {rin.x, rin.y, rin.z, rin.w};
      if constexpr (I < Ie) rin = rq[4 * (I + 1)];
      float racc[4] = {0.f, 0.f, 0.f, 0.f};
      static_for<t1 - t0>([&](auto rc) {
        constexpr int t = t0 + decltype(rc)::value, r = t - beg, J = t - first;
        if constexpr (r >= RR - PD) __builtin_amdgcn_sched_barrier(0);
        Quad<float> v;
        if constexpr (r < RR)
          v = sreg[r];
        else
          v = pf[r % PD];
        fetch(std::integral_constant<int, r + PD>{});
        float e4[4];
        v.to(e4);
#pragma unroll
        for (int k = 0; k < 4; ++k) racc[k] = fmat(e4[k], rdl[J], racc[k]);
        if constexpr (J < I) cacc[J] = dot4_acc(e4, ri, cacc[J]);
      });
      // a wave's tiles of one row are consecutive: each of its rows is stored once
      float4 q;
      q.x = row_sum16(racc[0]);
      q.y = row_sum16(racc[1]);
      q.z = row_sum16(racc[2]);
      q.w = row_sum16(racc[3]);
      if (cc == 0) *reinterpret_cast<float4*>(c.ow + 16 * I + 4 * g4) = q;
    }
  });
  __builtin_amdgcn_sched_barrier(0);
  // columns J < Ie; those from Ib on add to the row sums stored above
  static_for<(Ie + 3) / 4>([&](auto qc) {
    constexpr int q = decltype(qc)::value, c0 = 4 * q;
    swap_rows16(cacc[c0], cacc[c0 + 1]);
    swap_rows16(cacc[c0 + 2], cacc[c0 + 3]);
    float s0 = cacc[c0] + cacc[c0 + 1], s1 = cacc[c0 + 2] + cacc[c0 + 3];
    swap_rows32(s0, s1);
    cacc[c0] = s0 + s1;
  });
  float old[(Ie + 3) / 4 + 1];
  static_for<(Ie + 3) / 4>([&](auto qc) {
    constexpr int q = decltype(qc)::value;
    old[q] = 0.f;
    if constexpr (4 * q + 3 >= Ib) {
      const float v = c.ow[64 * q + 16 * g4 + cc];
      old[q] = 4 * q + g4 >= Ib ? v : 0.f;
    }
  });
  static_for<(Ie + 3) / 4>([&](auto qc) {
    constexpr int q = decltype(qc)::value;
    if (4 * q + 3 < Ie || 4 * q + g4 < Ie) c.ow[64 * q + 16 * g4 + cc] = old[q] + cacc[4 * q];
  });
}

// MT > 0: fixed-size operator product (blocks of at most MT tile rows); R > 0 resident
// (two workgroups per CU, so at most 256 VGPRs per lane), R = 0 read every iteration.
// MT = 0 (R = 0): any block size; tile coordinates at run time, column sums reduced over
// the lane groups and added to LDS per tile.
//
// Bound by latency: an iteration waits for its neighbours' y only (one exchange through the
// point of coherence) and has four workgroup barriers.  The residual of iteration l is summed
// while iteration l + 1 runs (each block's partial by the scene's first block, in a fixed order)
// and tested at the end of l + 2; a step that turns out to have stopped at l returns the values
// of l from a ring of the last four, so results and counts are those of a test in every
// iteration.  Measured per iteration: 512 blocks of 231 to 294 constrained DOFs 12.1 -> 5.1 us,
// 20 blocks of at most 165 6.9 -> 2.9 us (before: the test of every partial by every block inside
// the iteration, ten barriers, a wait per exchanged value).
constexpr int kFemRed = 20;  // doubles: own partial (4 waves x 2), scene's sum (4 x 2), total (2 + 2)
//
// Workgroups per CU, which bound the number of blocks of a launch: two of the resident form, three
// or four of the others (the registers are held to that).  kFar: the ring in device memory, for
// the launches whose blocks would not all be resident with it in LDS (blocks of more than ~415 slot
// rows beside LDS tiles, large FP64 blocks in numbers).
template <typename T, int R, int MT, bool kFar = false>
__global__ void __launch_bounds__(kFemThreads, R > 0 ? 2 : MT == 0 ? (sizeof(T) == 8 ? 2 : 3) : MT <= 12 ? 4 : 3)
    fem_loop_kernel(FemLoopArgs<T> a) {
  typedef Tagged<T> X;
  typedef Tagged<double> XD;
  extern __shared__ __align__(16) double lsm[];
  const int i = blockIdx.x;
  const int tid = threadIdx.x;
  const int bd = blockDim.x;
  const Topo& t = a.t;
  const int n_slot = t.sc_slot[t.n_scene];
  const int s0 = t.sub_slot[i];
  const int nc = t.sub_nc[i];
  const int m = a.f.m[i];
  const int mt = (m + 15) >> 4;  // 16 x 16 tiles of S per side
  const int scene = [&] {
    int lo = 0, hi = t.n_scene - 1;  // sc_sub[scene] <= i < sc_sub[scene + 1]
    while (lo < hi) {
      const int mid = (lo + hi + 1) / 2;
      if (t.sc_sub[mid] <= i) lo = mid; else hi = mid - 1;
    }
    return lo;
  }();
  // LDS: reductions, the constrained-DOF vectors (16-byte aligned), the static data of this
  // block's interface groups, rings of y and lambda, w in the order of the DOFs it acts on
  const int mtw = MT > 0 ? 16 * MT : a.max_mt16;
  double* red = lsm;
  T* rd = reinterpret_cast<T*>(lsm + kFemRed);              // mtw (zero beyond m)
  T* outw = rd + mtw;                                       // per wave mtw partial products
  T* gT = outw + 4 * mtw;                                   // 8 per group: ib0, ib1, iws, mu, e0..e2
  int* gI = reinterpret_cast<int*>(gT + 8 * a.max_ng);      // 4 per group: q0, other slot, kind | dim << 4 | first << 8
  const int rs = kFar ? nc : a.max_nc;                      // ring stride
  T* const near = reinterpret_cast<T*>(gI + 4 * a.max_ng);
  T* yr;                                                    // kRing x nc
  if constexpr (kFar) yr = a.ring + 2 * kRing * (long)s0; else yr = near;
  T* lr = yr + kRing * rs;                                  // kRing x nc
  T* ws = near + (kFar ? 0 : 2 * kRing * a.max_nc);         // nc + 4: sign times w
  int* kb = reinterpret_cast<int*>(ws + a.max_nc + 4);      // mtw: range of each DOF in ws, begin | end << 16
  uint16_t* pos = reinterpret_cast<uint16_t*>(kb + mtw);    // nc: entry of ws << 1 | (sign < 0)
  uint16_t* dof = pos + a.max_nc;                           // nc: constrained DOF << 1 | (sign < 0)
  const T be = a.beta[i];
  const T* Si = a.S + a.f.sq_off[i];
  const int dk0 = a.f.dkey_off[i];
  __shared__ int ngroup, s_lost, arrived[2];

  // per-step static data
  const int kbase = a.f.dk_off[dk0];
  for (int q = tid; q < nc; q += bd) {
    const int ql = a.f.dk_slot[kbase + q] - s0;
    pos[ql] = (uint16_t)((q << 1) | (a.f.slot_sgn[s0 + ql] < 0 ? 1 : 0));
    dof[q] = (uint16_t)((a.f.slot_dk[s0 + q] << 1) | (a.f.slot_sgn[s0 + q] < 0 ? 1 : 0));
  }
  for (int k = tid; k < m; k += bd) kb[k] = (a.f.dk_off[dk0 + k] - kbase) | ((a.f.dk_off[dk0 + k + 1] - kbase) << 16);
  // c = K^-1 b at the thread's slots
  T cds[2] = {(T)0, (T)0};
  for (int r = 0; r < 2; ++r)
    if (tid + r * bd < nc) cds[r] = a.cd[dk0 + a.f.slot_dk[s0 + tid + r * bd]];
  if (tid == 0) {
    ngroup = 0;
    s_lost = 0;
    arrived[0] = arrived[1] = 0;
  }
  for (int k = tid; k < 5 * mtw; k += bd) rd[k] = (T)0;  // and outw
  __syncthreads();
  // interface groups that touch this block: the first slot row of each
  for (int q = tid; q < nc; q += bd) {
    const int sl = s0 + q;
    if ((t.slot_mk[sl] & 7) != 0) continue;
    const int g = atomicAdd(&ngroup, 1);
    const int j = t.slot_if[sl];
    const bool two = t.if_nsub[j] == 2;
    const bool first = t.if_slot0[j] == sl;
    const T ib0 = (T)1 / a.beta[t.if_sub0[j]];
    const T ib1 = two ? (T)1 / a.beta[t.if_sub1[j]] : (T)0;
    gI[4 * g + 0] = q;
    gI[4 * g + 1] = !two ? -1 : first ? t.if_slot1[j] : t.if_slot0[j];
    gI[4 * g + 2] = t.if_kind[j] | (t.if_dim[j] << 4) | (first ? 256 : 0);
    gI[4 * g + 3] = 0;
    gT[8 * g + 0] = ib0;
    gT[8 * g + 1] = ib1;
    gT[8 * g + 2] = (T)1 / (ib0 + ib1);
    gT[8 * g + 3] = a.mu[j];
    for (int k = 0; k < 3; ++k) gT[8 * g + 4 + k] = k < t.if_dim[j] ? a.e[t.if_row[j] + k] : (T)0;
    gT[8 * g + 7] = (T)0;
  }
  // initial values (ring entry of iteration -1): y^0 := beta z^0 + u^0 (relation after every
  // z/u-update), w = beta z - u
  const auto z0_of = [&](int q) -> T { return a.z_in ? a.z_in[s0 + q] : (T)0; };
  const auto u0_of = [&](int q) -> T { return a.u_in ? a.u_in[s0 + q] : (T)0; };
  for (int q = tid; q < nc; q += bd) {
    const T z0 = z0_of(q), u0 = u0_of(q);
    const int pq = pos[q];
    const T w0 = fmat(be, z0, -u0);
    ws[pq >> 1] = (pq & 1) ? -w0 : w0;
    yr[(kRing - 1) * rs + q] = fmat(be, z0, u0);
    lr[(kRing - 1) * rs + q] = -u0;
  }
  __syncthreads();
  const int ng = ngroup;
  // operator product: the lower tiles in row order, split evenly over the four waves
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g4 = lane >> 4, cc = lane & 15;
  T* ow = outw + wv * mtw;
  // resident operator: registers, then LDS (16-byte aligned after the other arrays)
  Quad<T> sreg[(MT > 0 && R > 0) ? R : 1];
  MatvecArgs<T> mv;
  mv.rd = rd;
  mv.ow = ow;
  mv.sg = Si + 4 * lane;
  mv.mt = mt;
  {
    // by offset from the LDS base (an aligned pointer made from an integer would lose its
    // address space and turn the tile reads into flat loads)
    const int used = (int)(reinterpret_cast<unsigned char*>(dof + a.max_nc) - reinterpret_cast<unsigned char*>(lsm));
    T* slds = reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(lsm) + ((used + 15) & ~15));
    mv.sl = slds + lds_tiles_before(MT, R, wv) * 256;
  }
  if constexpr (MT > 0 && R > 0) {
    switch (wv) {
      case 0: load_tiles<T, MT, R, 0>(sreg, mv); break;
      case 1: load_tiles<T, MT, R, 1>(sreg, mv); break;
      case 2: load_tiles<T, MT, R, 2>(sreg, mv); break;
      default: load_tiles<T, MT, R, 3>(sreg, mv); break;
    }
  }
  // run-time schedule (MT = 0): this wave's first tile
  const int n_tile = mt * (mt + 1) / 2;
  const int t_beg = (n_tile * wv) / 4, t_end = (n_tile * (wv + 1)) / 4;
  int I0 = 0;
  while ((I0 + 1) * (I0 + 2) / 2 <= t_beg) ++I0;
  const int J0 = t_beg - I0 * (I0 + 1) / 2;

  const int sub0 = t.sc_sub[scene], sub1 = t.sc_sub[scene + 1];
  int it = 0, conv = 0;
  int kept = -1;  // iteration whose z-update is the result; -1: the initial values
  double th_s = 0.0, rt_s = 0.0;
  // iteration l, and beyond the last iteration what is left of the residual's way
  for (int l = 0; a.max_iters > 0; ++l) {
    const bool run = l < a.max_iters;
    unsigned long long* ybuf = a.ybuf + (long)(l & 1) * n_slot * X::N;
    const uint32_t tag = (uint32_t)l + 1;
    const auto part_of = [&](int k, int q) { return a.part + ((long)(k & 3) * t.n_sub + q) * 4; };
    const auto total_of = [&](int k) {
      return a.part + 16 * (long)t.n_sub + ((long)(k & 3) * t.n_scene + scene) * 4 * kPartCopies;
    };
    // indices of the phases below are formed from an opaque copy (otherwise the addresses of
    // every phase are held in registers over the operator product)
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    double pth = 0.0, pyy = 0.0;
    if (run) {
      // x-update (Eq. 15): rd = J_D^T w; vd = cd + S rd; x = J_D vd; y = beta x + u (Eq. 18)
      for (int k = tid; k < m; k += bd) {
        const int range = kb[k], end = range >> 16;
        T s = (T)0;
        for (int beg = range & 0xffff; beg < end; beg += 4) {
          T v[4];
#pragma unroll
          for (int h = 0; h < 4; ++h) v[h] = ws[beg + h];
#pragma unroll
          for (int h = 0; h < 4; ++h) s += beg + h < end ? v[h] : (T)0;
        }
        rd[k] = s;
      }
      if constexpr (MT == 0)
        for (int k = tid; k < 4 * mtw; k += bd) outw[k] = (T)0;
      __syncthreads();
      // S rd with S symmetric and only its lower tiles stored: a tile (I, J) adds T rd_J to
      // rows I and, below the diagonal, T^T rd_I to rows J
      if constexpr (MT > 0) {
        switch (wv) {
          case 0: matvec_fixed<MT, R, 0>(sreg, mv); break;
          case 1: matvec_fixed<MT, R, 1>(sreg, mv); break;
          case 2: matvec_fixed<MT, R, 2>(sreg, mv); break;
          default: matvec_fixed<MT, R, 3>(sreg, mv); break;
        }
      } else {
        int I = I0, J = J0;
        T racc[4] = {(T)0, (T)0, (T)0, (T)0};
        bool pending = false;
        auto row_flush = [&]() {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const T q = row_sum16(racc[k]);
            if (cc == 0) ow[16 * I + 4 * g4 + k] += q;
            racc[k] = (T)0;
          }
        };
        const T* base = Si + 4 * lane;
        for (int t = t_beg; t < t_end; t += 8) {
          Quad<T> v[8];
#pragma unroll
          for (int r = 0; r < 8; ++r)
            if (t + r < t_end) v[r].load(base + (long)(t + r) * 256);
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            if (t + r >= t_end) break;
            T e4[4];
            v[r].to(e4);
            const T rj = rd[16 * J + cc];
#pragma unroll
            for (int k = 0; k < 4; ++k) racc[k] = fmat(e4[k], rj, racc[k]);
            pending = true;
            if (J < I) {
              T cp = dot4_acc(e4, rd + 16 * I + 4 * g4, (T)0);
              cp += __shfl_xor(cp, 16, 64);
              cp += __shfl_xor(cp, 32, 64);
              if (g4 == 0) ow[16 * J + cc] += cp;
              ++J;
            } else {
              row_flush();
              pending = false;
              ++I;
              J = 0;
            }
          }
        }
        if (pending) row_flush();
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int q = tid + r * bd;
        if (q < nc) {
          const int dq = dof[q];
          T s = (T)0;
#pragma unroll
          for (int k = 0; k < 4; ++k) s += outw[k * mtw + (dq >> 1)];
          const T yo = yr[((l - 1) & 3) * rs + q], lo = lr[((l - 1) & 3) * rs + q];
          const T v = cds[r] + s, x = (dq & 1) ? -v : v;
          const T yn = fmat(be, x, -lo);
          const T df = yn - yo;
          X::put(ybuf + (long)(s0 + q) * X::N, yn, tag);
          pth += (double)df * (double)df;
          pyy += (double)yn * (double)yn;
          yr[(l & 3) * rs + q] = yn;
        }
      }
    }
    __syncthreads();
    // residual of Eq. (22): this block's sums, published by the wave that finishes last
    if (run) {
      wave_sums(pth, pyy, red + 2 * wv);
      if (arrive_last(&arrived[0], 4) && lane < 2) {
        double v = 0.0;
        for (int q = 0; q < 4; ++q) v += red[2 * q + lane];
        XD::put(part_of(l, i) + 2 * lane, v, tag);
      }
    }
    bool lost = false;
    // the scene's sum of iteration l - 1, by the waves of its first block that have the least of the
    // z-update to do (the first block is the slowest otherwise): every partial, in the order of
    // 256 strided sums, of which wave 3 forms 0..127 and wave 2 the others, two partials a lane
    // in flight (four would spill the resident operator)
    if (i == sub0 && wv >= 2 && l >= 1 && l <= a.max_iters) {
      const int v0 = 2 * (3 - wv);
      const unsigned long long* base = part_of(l - 1, 0);
      double th[2] = {0.0, 0.0}, yy[2] = {0.0, 0.0};
      for (int q0 = sub0 + 64 * v0 + lane; q0 < sub1; q0 += kFemThreads) {
        double pt[2], py[2];
        for (long polls = 0; !lost; ++polls) {
          bool ok = true;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int q = q0 + 64 * h;
            const unsigned long long* pp = base + 4u * (unsigned)(q < sub1 ? q : q0);
            ok = XD::get(pp, &pt[h], tag - 1) & ok;
            ok = XD::get(pp + 2, &py[h], tag - 1) & ok;
          }
          if (ok) break;
          lost = polls > kMaxPolls;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const bool in = q0 + 64 * h < sub1;
          th[h] += in ? pt[h] : 0.0;
          yy[h] += in ? py[h] : 0.0;
        }
      }
      wave_sums(th[0], yy[0], red + 8 + 2 * v0);
      wave_sums(th[1], yy[1], red + 10 + 2 * v0);
      if (arrive_last(&arrived[1], 2) && lane < 2 * kPartCopies) {
        double v = 0.0;
        for (int q = 0; q < 4; ++q) v += red[8 + 2 * q + (lane & 1)];
        XD::put(total_of(l - 1) + 2 * lane, v, tag - 1);
      }
    }
    // z-update (Eq. 16-21) and dual update (Eq. 14) of the interfaces touching this block
    if (l + 1 < a.max_iters) {
      const T* yc = yr + (l & 3) * rs;
      T* lc = lr + (l & 3) * rs;
      for (int g = tid; g < ng; g += bd) {
        const int q0 = gI[4 * g + 0], other = gI[4 * g + 1], kdim = gI[4 * g + 2];
        const int kind = kdim & 15, dim = (kdim >> 4) & 15;
        const bool first = (kdim & 256) != 0;
        T gt[8], yw[3], yo[3] = {(T)0, (T)0, (T)0};
        int pq[3];
#pragma unroll
        for (int k = 0; k < 8; ++k) gt[k] = gT[8 * g + k];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          yw[k] = yc[q0 + (k < dim ? k : 0)];
          pq[k] = pos[q0 + (k < dim ? k : 0)];
        }
        // the other member's y, all values of a poll in flight together.  Once one wait of this
        // thread has expired the iteration is abandoned and nothing further is polled
        if (other >= 0) {
          const unsigned long long* py = ybuf + (long)other * X::N;
          for (long polls = 0; !lost; ++polls) {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < 3; ++k) ok = X::get(py + (k < dim ? k : 0) * X::N, &yo[k], tag) & ok;
            if (ok) break;
            lost = polls > kMaxPolls;
          }
        }
        const T ib0 = gt[0], ib1 = gt[1], iws = gt[2], mu = gt[3];
        T p[3], lv[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const T ya = k < dim ? (first ? yw[k] : yo[k]) : (T)0;
          const T yb = k < dim ? (first ? yo[k] : yw[k]) : (T)0;
          p[k] = -fmat(yb, ib1, fmat(ya, ib0, gt[4 + k])) * iws;
        }
        if (kind == KIND_CONTACT && a.contact_model == 1) {
          cone_project<T>(p, mu, lv);
        } else if (kind == KIND_CONTACT) {
          const T ln = p[0] > (T)0 ? p[0] : (T)0;
          const T tn = fsqrt<T>(p[1] * p[1] + p[2] * p[2]);
          const T cap = mu * ln;
          lv[0] = ln;
          if (tn <= cap) {
            lv[1] = p[1];
            lv[2] = p[2];
          } else {
            const T fct = cap / tn;
            lv[1] = fct * p[1];
            lv[2] = fct * p[2];
          }
        } else if (kind == KIND_HARD_INEQ) {
          for (int k = 0; k < 3; ++k) lv[k] = p[k] > (T)0 ? p[k] : (T)0;
        } else {
          for (int k = 0; k < 3; ++k) lv[k] = p[k];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          if (k < dim) {
            const T w = fmat((T)2, lv[k], yw[k]);
            lc[q0 + k] = lv[k];
            ws[pq[k] >> 1] = (pq[k] & 1) ? -w : w;
          }
        }
      }
    }
    // the total of l - 2
    if (l >= 2 && tid == 191) {  // wave 2
      double v0 = 0.0, v1 = 0.0;
      const unsigned long long* pt = total_of(l - 2) + 4 * (i % kPartCopies);
      for (long polls = 0; !lost; ++polls) {
        bool ok = XD::get(pt, &v0, tag - 2);
        ok = XD::get(pt + 2, &v1, tag - 2) & ok;
        if (ok) break;
        lost = polls > kMaxPolls;
      }
      red[16] = v0;
      red[17] = v1;
    }
    if (lost) s_lost = 1;
    __syncthreads();
    if (s_lost) {
      if (tid == 0) atomicOr(a.flags, FLAG_BARRIER);
      it = (run ? l : a.max_iters - 1) + 1;
      kept = it - 2;
      break;
    }
    if (l >= 2) {
      // every block of the scene reads the same total, so all take the same decision
      const double p0 = red[16], p1 = red[17];
      const double tol2 = a.tol * a.tol;
      const bool bad = !__builtin_isfinite(p0) || !__builtin_isfinite(p1);
      const bool cv = !bad && p0 <= tol2 * (p1 > 1e-24 ? p1 : 1e-24);
      if (cv || bad || l - 1 == a.max_iters) {
        if (bad && i == sub0 && tid == 0) atomicOr(a.flags, FLAG_NONFINITE);
        it = l - 1;
        kept = l - 3;
        conv = cv;
        th_s = p0;
        rt_s = __builtin_sqrt(p0) / __builtin_sqrt(p1 > 1e-24 ? p1 : 1e-24);
        break;
      }
    }
  }
  __syncthreads();
  // outputs of this block: final (z, u), the w of the last x-update, lambda rows of the
  // interfaces whose member 0 is this block
  for (int q = tid; q < nc; q += bd) {
    const int sl = s0 + q;
    T z, u, w, lam;
    if (kept < 0) {
      z = z0_of(q);
      u = u0_of(q);
      w = fmat(be, z, -u);
      lam = -u;
    } else {
      const T yk = yr[(kept & 3) * rs + q];
      lam = lr[(kept & 3) * rs + q];
      z = (yk + lam) / be;
      u = -lam;
      w = fmat((T)2, lam, yk);
    }
    if (a.z_out) a.z_out[sl] = z;
    if (a.u_out) a.u_out[sl] = u;
    a.w_out[sl] = w;
    const int j = t.slot_if[sl];
    const int mk = t.slot_mk[sl];
    if (a.lambda && (mk >> 3) == 0) a.lambda[t.if_row[j] + (mk & 7)] = lam;
  }
  if (tid == 0 && i == t.sc_sub[scene]) {
    a.st_iters[scene] = it;
    a.st_conv[scene] = conv;
    a.st_theta[scene] = th_s;
    a.st_rtheta[scene] = rt_s;
    a.st_total[scene] += it;
    if (!conv) a.st_unconv[scene] += 1;
  }
}

template <typename T>
__global__ void fem_advance_kernel(int64_t n_dof, const T* v_hat, T dt, T* pos, T* vel) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_dof) return;
  const T vh = v_hat[k];
  pos[k] += dt * vh;
  vel[k] = (T)2 * vh - vel[k];
}

template <typename T>
__global__ void fem_export_kernel(Topo t, FemModel f, const double* A, const double* b, T* Ao, T* bo, T* Jo) {
  const int i = blockIdx.x;
  const int n = t.sub_n[i];
  const long nn = (long)n * n;
  for (long k = threadIdx.x; k < nn; k += blockDim.x) Ao[t.sub_A[i] + k] = (T)A[t.sub_A[i] + k];
  for (int r = threadIdx.x; r < n; r += blockDim.x) bo[t.sub_dof[i] + r] = (T)b[t.sub_dof[i] + r];
  const int nc = t.sub_nc[i];
  T* Ji = Jo + t.sub_J[i];
  for (long k = threadIdx.x; k < (long)nc * n; k += blockDim.x) Ji[k] = (T)0;
  __syncthreads();
  for (int q = threadIdx.x; q < nc; q += blockDim.x) {
    const int sl = t.sub_slot[i] + q;
    Ji[(long)q * n + f.slot_dof[sl]] = (T)f.slot_sgn[sl];
  }
}

// ------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------
template <typename T>
hipError_t launch_fem_assemble(const Topo& t, const FemModel& f, const T* pos, const T* vel, double dt, double* A,
                               double* b, double* scr, int32_t* flags, hipStream_t s) {
  if (t.n_sub == 0) return hipSuccess;
  hipLaunchKernelGGL(fem_assemble_kernel<T>, dim3(t.n_sub), dim3(kFemThreads), 0, s, t, f, pos, vel, dt, A, b, scr,
                     flags);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fem_rows(const Topo& t, const FemModel& f, const T* pos, double dt, T* e, hipStream_t s) {
  if (t.n_if == 0) return hipSuccess;
  hipLaunchKernelGGL(fem_rows_kernel<T>, dim3((t.n_if + 255) / 256), dim3(256), 0, s, t, f, pos, dt, e);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fem_factor(const Topo& t, const FemModel& f, const double* A, double* b, double rho, T* beta,
                             double* L, double* tinv, T* S, T* cd, int32_t* flags, int32_t* prec, double* kest,
                             double kmax, int max_n, int max_m, hipStream_t s) {
  if (t.n_sub == 0) return hipSuccess;
  (void)max_m;
  const size_t pn = max_n > 32 ? (size_t)max_n : 32;
  // diagonal tile, row panel (rows padded by up to four entries), vector; at least the 256 doubles
  // of the trace's reduction
  const size_t words = std::max<size_t>(kNb * kNb + (pn + 4) * kNb + (size_t)max_n, 2 * kFemThreads);
  auto go = [&](auto kern, size_t lds, double km, int gate) -> hipError_t {
    if (lds > 64 * 1024) {
      const hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (ea != hipSuccess) return ea;
    }
    hipLaunchKernelGGL(kern, dim3(t.n_sub), dim3(kFemFactorThreads), lds, s, t, f, A, b, rho, beta, L, tinv, S, cd, flags,
                       prec, kest, km, gate);
    return hipGetLastError();
  };
  if constexpr (std::is_same<T, float>::value) {
    if (kmax > 0.0) {
      // FP32 trial on every block, then FP64 on the blocks it recorded
      const hipError_t e = go(&fem_factor_kernel<T, float>, sizeof(float) * words, kmax, 0);
      if (e != hipSuccess) return e;
      return go(&fem_factor_kernel<T, double>, sizeof(double) * words, 0.0, 1);
    }
  }
  return go(&fem_factor_kernel<T, double>, sizeof(double) * words, 0.0, 0);
}

// Clears the exchange buffers (no iteration has tag 0).
__global__ void fem_clear_kernel(unsigned long long* y, long n_y, unsigned long long* part, long n_part) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n_y) y[k] = 0;
  if (k < n_part) part[k] = 0;
}

template <typename T, int R, int MT, bool kFar = false>
static hipError_t resident_fem_loop(const FemLoopArgs<T>& a, size_t lds, int cus, bool& fits, hipStream_t s) {
  int per_cu = 0;
  const void* fn = reinterpret_cast<const void*>(&fem_loop_kernel<T, R, MT, kFar>);
  if (lds > 64 * 1024) {
    const hipError_t ea = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (ea != hipSuccess) {
      (void)hipGetLastError();
      fits = false;
      return hipSuccess;
    }
  }
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kFemThreads, lds);
  if (e != hipSuccess) return e;
  fits = (long)per_cu * cus >= a.t.n_sub;
  if (!fits) return hipSuccess;
  // An ordinary dispatch: the grid fits the device at this occupancy, so every workgroup is
  // resident once the work queued before it on the stream has drained.  The kernel needs
  // nothing else of a cooperative launch (no grid-wide sync object; workgroups exchange
  // through polled buffers whose waits are bounded and report FLAG_BARRIER on expiry), and
  // a cooperative launch would put the dispatch on the runtime's separate cooperative queue.
  hipLaunchKernelGGL((fem_loop_kernel<T, R, MT, kFar>), dim3(a.t.n_sub), dim3(kFemThreads), lds, s, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fem_loop(const FemLoopArgs<T>& a, int* form, hipStream_t s) {
  *form = 0;
  if (a.t.n_sub == 0) return hipSuccess;
  if (a.max_nc > kMaxFemSlots) return hipErrorInvalidValue;
  {
    const long n_y = 2 * (long)Tagged<T>::N * a.n_slot, n_part = (long)fem_part_words(a.t.n_sub, a.t.n_scene);
    const long n = n_y > n_part ? n_y : n_part;
    hipLaunchKernelGGL(fem_clear_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a.ybuf, n_y, a.part,
                       n_part);
    const hipError_t ze = hipGetLastError();
    if (ze != hipSuccess) return ze;
  }
  const auto lds_of = [&](int mtw, bool far = false) -> size_t {
    return sizeof(double) * kFemRed + sizeof(T) * (5 * (size_t)mtw + 8 * (size_t)a.max_ng) +
           sizeof(int) * 4 * (size_t)a.max_ng + sizeof(T) * (((far ? 0 : 2 * kRing) + 1) * (size_t)a.max_nc + 4) +
           sizeof(int) * (size_t)mtw + 2 * sizeof(uint16_t) * (size_t)a.max_nc + 16;
  };
  int dev = 0, cus = 0, lds_max = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  if (e != hipSuccess) return e;
  const int mt = a.max_mt16 / 16;
  bool fits = false;
  if constexpr (std::is_same<T, float>::value) {
    // smallest fixed-size class that holds every block
    int MT = 0;
    for (int c : kMtClasses)
      if (mt <= c) {
        MT = c;
        break;
      }
    if (MT > 0) {
      auto run = [&](auto mtc) -> hipError_t {
        constexpr int M = decltype(mtc)::value;
        if (a.resident) {
          constexpr size_t tiles = (size_t)lds_tiles_before(M, kResTiles, 4) * 256 * sizeof(T);
          if (lds_of(16 * M) + tiles <= (size_t)lds_max) {
            const hipError_t er = resident_fem_loop<T, kResTiles, M>(a, lds_of(16 * M) + tiles, cus, fits, s);
            if (fits) *form = kResTiles;
            if (er != hipSuccess || fits) return er;
          }
          // operators partly in LDS: beside them the ring leaves room for two blocks a CU up to ~415
          // slot rows (289 blocks of 300 DOFs, 462 rows: 5.5 us an iteration with the ring in
          // device memory, 11.1 streaming the operators instead)
          if constexpr (tiles > 0) {
            if (lds_of(16 * M, true) + tiles <= (size_t)lds_max) {
              const hipError_t er = resident_fem_loop<T, kResTiles, M, true>(a, lds_of(16 * M, true) + tiles, cus, fits, s);
              if (fits) *form = kResTiles;
              if (er != hipSuccess || fits) return er;
            }
          }
        }
        return resident_fem_loop<T, 0, M>(a, lds_of(16 * M), cus, fits, s);
      };
      switch (MT) {
        case 8: e = run(std::integral_constant<int, 8>{}); break;
        case 12: e = run(std::integral_constant<int, 12>{}); break;
        case 16: e = run(std::integral_constant<int, 16>{}); break;
        default: e = run(std::integral_constant<int, 19>{}); break;
      }
      if (e != hipSuccess || fits) return e;
    }
  }
  e = resident_fem_loop<T, 0, 0>(a, lds_of(a.max_mt16), cus, fits, s);
  if (e != hipSuccess || fits) return e;
  e = resident_fem_loop<T, 0, 0, true>(a, lds_of(a.max_mt16, true), cus, fits, s);
  if (e != hipSuccess) return e;
  return fits ? hipSuccess : hipErrorCooperativeLaunchTooLarge;
}

template <typename T>
hipError_t launch_fem_vhat(const Topo& t, const FemModel& f, const double* L, const double* Tw, const double* y,
                           const int32_t* prec, const T* w, T* v_hat, int max_n, hipStream_t s) {
  if (t.n_sub == 0) return hipSuccess;
  const size_t lds = sizeof(double) * (3 + kVhatParts) * (size_t)max_n;
  hipLaunchKernelGGL(fem_vhat_kernel<T>, dim3(t.n_sub), dim3(kFemFactorThreads), lds, s, t, f, L, Tw, y, prec, w, v_hat);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fem_advance(int64_t n_dof, const T* v_hat, T dt, T* pos, T* vel, hipStream_t s) {
  if (n_dof == 0) return hipSuccess;
  hipLaunchKernelGGL(fem_advance_kernel<T>, dim3((unsigned)((n_dof + 255) / 256)), dim3(256), 0, s, n_dof, v_hat, dt,
                     pos, vel);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fem_export(const Topo& t, const FemModel& f, const double* A, const double* b, T* Ao, T* bo, T* Jo,
                             hipStream_t s) {
  if (t.n_sub == 0) return hipSuccess;
  hipLaunchKernelGGL(fem_export_kernel<T>, dim3(t.n_sub), dim3(kFemThreads), 0, s, t, f, A, b, Ao, bo, Jo);
  return hipGetLastError();
}

#define SUBADMM_FEM_INST(T)                                                                                          \
  template hipError_t launch_fem_assemble<T>(const Topo&, const FemModel&, const T*, const T*, double, double*,    \
                                             double*, double*, int32_t*, hipStream_t);                              \
  template hipError_t launch_fem_rows<T>(const Topo&, const FemModel&, const T*, double, T*, hipStream_t);          \
  template hipError_t launch_fem_factor<T>(const Topo&, const FemModel&, const double*, double*, double, T*,       \
                                           double*, double*, T*, T*, int32_t*, int32_t*, double*, double, int, int, \
                                           hipStream_t);                                                            \
  template hipError_t launch_fem_loop<T>(const FemLoopArgs<T>&, int*, hipStream_t);                                  \
  template hipError_t launch_fem_vhat<T>(const Topo&, const FemModel&, const double*, const double*, const double*, \
                                         const int32_t*, const T*, T*, int, hipStream_t);                           \
  template hipError_t launch_fem_advance<T>(int64_t, const T*, T, T*, T*, hipStream_t);                             \
  template hipError_t launch_fem_export<T>(const Topo&, const FemModel&, const double*, const double*, T*, T*, T*,  \
                                           hipStream_t);
SUBADMM_FEM_INST(float)
SUBADMM_FEM_INST(double)
#undef SUBADMM_FEM_INST

}  // namespace subadmm
