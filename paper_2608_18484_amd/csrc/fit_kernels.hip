// Probe-fitted residual reconstruction of the SparsePR operator for gfx950
// (Sec. 4.2; App. A.3): the weighted probe statistics, the residual basis and
// ridge solve, and the correction + restore of every row to the original order
// (eq. final_reconstructed_output), with the probe rows taking their exact
// dense rows.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "device_utils.hpp"
#include "sparsepr_internal.hpp"
#include "jacobi_lds.hpp"
#include "tridiag_eig.hpp"

namespace sparsepr {

// ---------------------------------------------------------------------------
// Probe-fitted residual fit (Sec. 4.2; App. A.3), per head: the statistics
// (k_fit_prep), the three products over the probes (k_fit_gram), the basis
// beside the ridge solve (k_fit_solve, two blocks) and Y (k_fit_map):
//   alpha_p = w_p / sum w;  mu_x, mu_R weighted means;
//   s_x = sqrt(sum alpha (x - mu_x)^2 + eps);  xbar = (x - mu_x)/s_x;
//   Rbar = R - mu_R;  w~_p = M w_p / sum w;
//   Psi = leading r eigenvectors of Rbar^T W Rbar (right singular vectors of
//         W^1/2 Rbar), keeping sigma > 1e-6 sigma_1;
//   (xbar^T W xbar + lambda I) X = xbar^T W Rbar,  Y = X Psi,
// so Y = B_lambda Psi and the correction of row i is xbar_i Y Psi^T + mu_R.
// ---------------------------------------------------------------------------

// Per-head scratch of the fit: xbar [M][D], rbar [M][D], w~ [M] (all double).
struct FitScratch {
  double *xb, *rb, *wt;
};

__device__ __forceinline__ FitScratch fit_scratch(const Geom& g, const Work& w, int bh) {
  const size_t D = g.dv, M = g.M;
  double* base = w.fitscr + (size_t)bh * (2 * M * D + M);
  FitScratch f;
  f.xb = base;
  f.rb = f.xb + M * D;
  f.wt = f.rb + M * D;
  return f;
}

// Weighted statistics of the probes (eqs. app_normalized_weights ...
// app_regression_weights): mu_x, mu_R, s_x, xbar, Rbar and w~.  Thread
// (c, s) takes column c of every (1024 / D)-th probe, so that a head's three
// passes over its gathered probe rows are 16 short chains of loads at 128
// probes instead of 128 (36 us with one thread per column).
template <int D>
__global__ __launch_bounds__(1024) void k_fit_prep(Geom g, Work w) {
  constexpr int SP = 1024 / D;
  __shared__ double swsh;
  __shared__ double sred[3][SP][D];
  const int bq = blockIdx.x, bh = bq % g.BH, tid = threadIdx.x;
  const int np = w.nprobes[bh];
  const int r = g.r;
  float* fv = w.fitv + (size_t)bq * 3 * D;
  float* Y = w.fity + (size_t)bq * D * r;
  float* Psi = w.fitpsi + (size_t)bq * D * r;
  for (int i = tid; i < D * r; i += 1024) {
    Y[i] = 0.f;
    Psi[i] = 0.f;
  }
  if (np == 0) {
    for (int c = tid; c < D; c += 1024) {
      fv[c] = 0.f;
      fv[D + c] = 1.f;
      fv[2 * D + c] = 0.f;
    }
    if (tid == 0) w.stats[(size_t)bh * 16 + ST_FIT_RANK] = 0;
    return;
  }
  const FitScratch f = fit_scratch(g, w, bq);
  const int32_t* pr = w.probes + (size_t)bh * g.M;
  const float* pwt = w.pw + (size_t)bh * g.M;
  const float* osp = w.osp + (size_t)bq * g.N * D;
  const float* odp = w.odp + (size_t)bq * g.M * D;
  if (tid < 64) {
    // fixed order: lane-strided partial sums, then the wave sum
    double s = 0.0;
    for (int p = tid; p < np; p += 64) s += (double)pwt[p];
    s = wave_sum_d(s);
    if (tid == 0) swsh = s;
  }
  __syncthreads();
  const double sw = swsh;
  for (int p = tid; p < np; p += 1024) f.wt[p] = (double)np * (double)pwt[p] / sw;
  const int c = tid % D, st = tid / D;
  // column sums over the strips, in strip order
  auto total = [&](int which) {
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < SP; ++j) t += sred[which][j][c];
    return t;
  };
  double mx = 0.0, mr = 0.0;
#pragma unroll 8
  for (int p = st; p < np; p += SP) {
    const double al = (double)pwt[p] / sw;
    const double x = osp[(size_t)pr[p] * D + c];
    mx += al * x;
    mr += al * ((double)odp[(size_t)p * D + c] - x);
  }
  sred[0][st][c] = mx;
  sred[1][st][c] = mr;
  __syncthreads();
  mx = total(0);
  mr = total(1);
  double vx = 0.0;
#pragma unroll 8
  for (int p = st; p < np; p += SP) {
    const double al = (double)pwt[p] / sw;
    const double t = (double)osp[(size_t)pr[p] * D + c] - mx;
    vx += al * t * t;
  }
  sred[2][st][c] = vx;
  __syncthreads();
  const double sx = sqrt(total(2) + (double)g.eps_x);
#pragma unroll 8
  for (int p = st; p < np; p += SP) {
    const double x = osp[(size_t)pr[p] * D + c];
    f.xb[(size_t)p * D + c] = (x - mx) / sx;
    f.rb[(size_t)p * D + c] = ((double)odp[(size_t)p * D + c] - x) - mr;
  }
  if (st == 0) {
    fv[c] = (float)mx;
    fv[D + c] = (float)sx;
    fv[2 * D + c] = (float)mr;
  }
}

// The weighted Gram matrices of the fit, one 32 x 32 tile per block:
// which = 0: H = Rbar^T W Rbar (its eigenvectors are the right singular
// vectors of W^1/2 Rbar, eq. app_probe_residual_basis); which = 1:
// S = xbar^T W xbar + lambda I (eq. app_ridge_closed_form); which = 2:
// xbar^T W Rbar, the right-hand side of the ridge solve before the projection
// onto the residual subspace.
template <int D>
__global__ __launch_bounds__(256) void k_fit_gram(Geom g, Work w) {
  constexpr int PB = 64;
  __shared__ double sa[PB][33], sb[PB][33];
  __shared__ double swt[PB];
  const int bq = blockIdx.z, bh = bq % g.BH, which = blockIdx.y, tid = threadIdx.x;
  const int np = w.nprobes[bh];
  if (np == 0) return;
  const int ti = blockIdx.x / (D / 32), tj = blockIdx.x % (D / 32);
  const FitScratch f = fit_scratch(g, w, bq);
  const double* srca = which == 0 ? f.rb : f.xb;
  const double* srcb = which == 1 ? f.xb : f.rb;
  const int li = tid / 8, lj = (tid % 8) * 4;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int p0 = 0; p0 < np; p0 += PB) {
    const int pn = min(PB, np - p0);
    __syncthreads();
    for (int i = tid; i < pn * 32; i += 256) {
      const int p = i / 32, c = i % 32;
      sa[p][c] = srca[(size_t)(p0 + p) * D + ti * 32 + c];
      sb[p][c] = srcb[(size_t)(p0 + p) * D + tj * 32 + c];
    }
    for (int p = tid; p < pn; p += 256) swt[p] = f.wt[p0 + p];
    __syncthreads();
    for (int p = 0; p < pn; ++p) {
      const double a = swt[p] * sa[p][li];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += a * sb[p][lj + e];
    }
  }
  double* G = w.fitgram + ((size_t)bq * 3 + which) * D * D;
  const int i = ti * 32 + li;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int j = tj * 32 + lj + e;
    G[(size_t)i * D + j] = acc[e] + ((which == 1 && i == j) ? (double)g.ridge : 0.0);
  }
}

// X = S^-1 B for a symmetric positive definite S, S, B and X D x D in double
// (X over B), by one block of 1024 threads: S = L diag(d) L^T by right-looking
// elimination on the augmented matrix [S | B], which lives in registers
// (thread = one column x one strip of rows, row i in strip i % 4).  Step j
// publishes row j (double-buffered, so one barrier per step): by symmetry it
// is also the column every row subtracts, and scaled by 1 / d_j it is row j of
// L^T (kept in U, row stride D + 1) and of diag(d)^-1 L^-1 B (kept over B).
// Then L^T X is solved, one wave per column of B.  Returns false when a pivot
// is not positive.  (A Cholesky factorisation with S in LDS, two barriers per
// column and separate triangular solves took 256 us of a block at D = 128.)
template <int D>
__device__ __forceinline__ bool fit_spd_solve(const double* __restrict__ Sg, double* __restrict__ B, double* U) {
  constexpr int S = 4, NR = D / S, BK = 8, NB = NR / BK, LU = D + 1;
  static_assert(2 * S * D <= 1024, "one thread per column and strip");
  typedef double blk __attribute__((ext_vector_type(BK)));
  __shared__ __attribute__((aligned(16))) double rowb[2][2][D];
  const int tid = threadIdx.x, lane = tid & 63;
  const int c = tid % D, strip = __builtin_amdgcn_readfirstlane(tid / D);
  const bool rhs = strip >= S;
  const int s = strip % S;
  const bool act = strip < 2 * S;  // D = 64: the other waves only meet the barriers
  auto pos = [](int i) { return (i % S) * NR + i / S; };
  blk a[NB];
  if (act) {
#pragma unroll
    for (int bk = 0; bk < NB; ++bk)
#pragma unroll
      for (int e = 0; e < BK; ++e) {
        const int i = s + S * (bk * BK + e);
        a[bk][e] = (rhs ? B : Sg)[(size_t)i * D + c];
      }
    if (s == 0) rowb[0][rhs][rhs ? c : pos(c)] = a[0][0];
  }
  bool ok = true;
  for (int jj = 0; jj < D; ++jj) {
    const int j = __builtin_amdgcn_readfirstlane(jj);
    const int cur = j & 1;
    __syncthreads();
    const double* x = rowb[cur][0];
    const double dj = x[pos(j)];
    ok = ok && dj > 0.0;
    if (act) {
      const double f = rowb[cur][rhs][rhs ? c : pos(c)] / dj;
      if (s == j % S) {
        if (!rhs)
          U[j * LU + c] = f;
        else
          B[(size_t)j * D + c] = f;
      }
      const double* xs = x + s * NR;
#pragma unroll
      for (int bk = 0; bk < NB; ++bk)
        if (S * BK * (bk + 1) > j + 1) {
#pragma unroll
          for (int e = 0; e < BK; ++e) a[bk][e] = fma(-xs[bk * BK + e], f, a[bk][e]);
        }
      if (j + 1 < D && s == (j + 1) % S) {
        const int u = (j + 1) / S;
        double v = a[0][0];
#pragma unroll
        for (int bk = 0; bk < NB; ++bk)
          if (u / BK == bk) {
#pragma unroll
            for (int e = 0; e < BK; ++e) v = u % BK == e ? a[bk][e] : v;
          }
        rowb[cur ^ 1][rhs][rhs ? c : pos(c)] = v;
      }
    }
  }
  __syncthreads();
  if (!ok) return false;  // every thread saw the same pivots
  constexpr int NU = D / 64, CW = D / 16;  // rows per lane, columns per wave
  const int wv = tid >> 6;
  // a wave's columns four at a time, lane l holding unknowns l, l + 64 of
  // each; each solved one is subtracted from the rows above it
  for (int t0 = wv * CW; t0 < (wv + 1) * CW; t0 += 4) {
    double y[4][NU];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int u = 0; u < NU; ++u) y[q][u] = B[(size_t)(lane + 64 * u) * D + t0 + q];
    double nl[NU];  // the next column's entries, one step ahead of their use
#pragma unroll
    for (int u = 0; u < NU; ++u) nl[u] = U[(lane + 64 * u) * LU + D - 1];
#pragma unroll 1
    for (int j = D - 1; j > 0; --j) {
      double l[NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        l[u] = lane + 64 * u < j ? nl[u] : 0.0;
        nl[u] = U[(lane + 64 * u) * LU + j - 1];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double yj = tri_readlane(NU > 1 && j >= 64 ? y[q][NU - 1] : y[q][0], j & 63);
#pragma unroll
        for (int u = 0; u < NU; ++u) y[q][u] = fma(-l[u], yj, y[q][u]);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int u = 0; u < NU; ++u) B[(size_t)(lane + 64 * u) * D + t0 + q] = y[q][u];
  }
  return true;
}

// The fit's two serial solves, side by side (blockIdx.y):
//  * 1: X = (xbar^T W xbar + lambda I)^-1 xbar^T W Rbar, over the Gram kernel's
//    third matrix; one after the other with the basis, for the r projected
//    right-hand sides only, the block took 320 us at D = 128, now as long as
//    the basis alone;
//  * 0: Psi = leading r eigenvectors of H with sigma > 1e-6 sigma_1
//    (tridiagonal solver, or cyclic Jacobi in LDS when its check fails).
// k_fit_map then forms Y = X Psi = B_lambda Psi, so the correction of row i is
// xbar_i Y Psi^T + mu_R.
// T is the eigensolver's precision.  Double A and V of a 128 x 128 problem do not
// both fit in LDS; V (VG) then lives in the head's global scratch.
template <int D, typename T>
__global__ __launch_bounds__(1024) void k_fit_solve(Geom g, Work w) {
  constexpr int LD = D + 1, LV = jacobi_vt_ld<D>();
  constexpr bool VG = (size_t)D * (LD + LV) * sizeof(T) > 140 * 1024;
  constexpr size_t JAC = (size_t)D * (LD + (VG ? 0 : LV)) * sizeof(T),
                   CHOL = (size_t)D * LD * sizeof(double);
  __shared__ __attribute__((aligned(16))) unsigned char smem[JAC > CHOL ? JAC : CHOL];
  __shared__ JacobiRot<T> rot[D / 2];
  __shared__ TriWork<D, T, 1024> tw;
  __shared__ int order[D];
  __shared__ int flag, rank_s;
  const int bq = blockIdx.x, bh = bq % g.BH, tid = threadIdx.x;
  const int np = w.nprobes[bh];
  if (np == 0) return;
  const int r = g.r;
  float* Psi = w.fitpsi + (size_t)bq * D * r;
  double* H = w.fitgram + (size_t)bq * 3 * D * D;
  int64_t* st = w.stats + (size_t)bh * 16;
  if (blockIdx.y == 1) {
    double* X = H + 2 * D * D;
    if (!fit_spd_solve<D>(H + D * D, X, (double*)smem)) {
      // no map: the correction is the mean residual
      for (int e = tid; e < D * D; e += 1024) X[e] = 0.0;
      if (tid == 0) atomicOr((unsigned long long*)&st[ST_FLAGS], (unsigned long long)SPARSEPR_FLAG_FIT_NOT_PD);
    }
    return;
  }
  T* Am = (T*)smem;
  T* Vm = VG ? (T*)(w.fitvec + (size_t)bq * D * LV) : Am + D * LD;  // transposed (jacobi_eig_lds)
  if (g.ridge_only) {
    // ridge estimator alone (Table probe_estimator_ablation): Psi = I
    for (int e = tid; e < D * D; e += 1024) Vm[(e / D) * LV + (e % D)] = (e / D == e % D) ? T(1) : T(0);
    if (tid < D) order[tid] = tid;
    if (tid == 0) rank_s = D;
    __syncthreads();
  } else {
    const double scl = tri_scale<D>(H);  // only ratios of the eigenvalues are used
    tri_reduce_reg<D, T, 1024>([&](int e) { return (T)(scl * H[e]); }, Am, tw);
    tri_eigvals<D, T, 1024>(tw, r + 1);
    if (tid == 0) {
      // rank: the leading t < r with sigma_t > 1e-6 sigma_1.  In double the
      // float eigenvalues of the multisection cannot place an eigenvalue
      // near 1e-12 lambda_1, so a retained range reaching below 1e-5
      // lambda_1 is left to the Jacobi solve.
      const double l1 = tw.lamf[0];
      const double s1 = l1 > 0.0 ? sqrt(l1) : 0.0;
      int rk = 0;
      bool amb = false;
      // a zero matrix (one probe, or residuals that are all the same) has rank
      // 0; the search only finds the padding of its empty interval
      for (int t = 0; t < r && t < D && tw.fnorm > 0.f; ++t) {
        const double lt = tw.lamf[t];
        if (sizeof(T) == 8 && !(lt >= 1e-5 * l1)) amb = true;
        const double st = lt > 0.0 ? sqrt(lt) : 0.0;
        if (s1 > 0.0 && st > 1e-6 * s1)
          ++rk;
        else
          break;
      }
      rank_s = amb ? -1 : rk;
    }
    __syncthreads();
    if (rank_s >= 0) tri_vectors<D, false>(tw, Vm, LV, rank_s, w.eigscr + (size_t)bq * 2 * D * D, (double*)nullptr);
    if (rank_s >= 0 && tw.ok) {
      tri_back_rows<D, T, 1024>(Am, tw, Vm, LV, rank_s);
      if (tid < D) order[tid] = tid;
    } else {
      if (tid == 0)
        atomicOr((unsigned long long*)&w.stats[(size_t)bh * 16 + ST_FLAGS], (unsigned long long)SPARSEPR_FLAG_EIG_JACOBI);
      for (int e = tid; e < D * D; e += 1024) Am[(e / D) * LD + (e % D)] = (T)(scl * H[e]);
      __syncthreads();
      jacobi_eig_lds<D, T, 1024>(Am, Vm, rot, &flag, sizeof(T) == 8 ? T(1e-12) : T(1e-4));
      if (tid < D) {
        // a NaN diagonal (non-finite input) ranks as -inf, so the ranks stay
        // a permutation and every order[] entry is written
        const T li = eig_rank_key(Am[tid * LD + tid]);
        int rank = 0;
        for (int j = 0; j < D; ++j) {
          const T lj = eig_rank_key(Am[j * LD + j]);
          rank += (lj > li) || (lj == li && j < tid);
        }
        order[rank] = tid;
      }
      __syncthreads();
      if (tid == 0) {
        const double l1 = Am[order[0] * LD + order[0]];
        const double s1 = l1 > 0.0 ? sqrt(l1) : 0.0;
        int rk = 0;
        for (int t = 0; t < r && t < D; ++t) {
          const double lt = Am[order[t] * LD + order[t]];
          const double st = lt > 0.0 ? sqrt(lt) : 0.0;
          if (s1 > 0.0 && st > 1e-6 * s1)
            ++rk;
          else
            break;
        }
        rank_s = rk;
      }
    }
    __syncthreads();
  }
  const int rk = rank_s;
  // Psi for the correction in float; k_fit_map takes it as solved, in double,
  // over H, which is done with
  for (int i = tid; i < D * r; i += 1024) {
    const int row = i / r, t = i % r;
    const double p = t < rk ? (double)Vm[order[t] * LV + row] : 0.0;
    H[i] = p;
    if (t < rk) Psi[i] = (float)p;
  }
  if (tid == 0) st[ST_FIT_RANK] = rk;
}

// Y = X Psi (both from k_fit_solve) in double, 16 directions per block.
template <int D>
__global__ __launch_bounds__(1024) void k_fit_map(Geom g, Work w) {
  constexpr int RS = 16, GT = 1024 / D, TP = RS / GT;  // directions per thread
  __shared__ double ps[D][RS];
  const int bq = blockIdx.y, bh = bq % g.BH, tid = threadIdx.x;
  if (w.nprobes[bh] == 0) return;
  const int r = g.r, t0 = blockIdx.x * RS;
  float* Y = w.fity + (size_t)bq * D * r;
  const double* Psi = w.fitgram + (size_t)bq * 3 * D * D;
  const double* X = Psi + 2 * D * D;
  for (int i = tid; i < D * RS; i += 1024) ps[i / RS][i % RS] = t0 + i % RS < r ? Psi[(i / RS) * r + t0 + i % RS] : 0.0;
  __syncthreads();
  const int c = tid / GT, q = (tid % GT) * TP;
  double acc[TP];
#pragma unroll
  for (int u = 0; u < TP; ++u) acc[u] = 0.0;
#pragma unroll 16
  for (int e = 0; e < D; ++e) {
    const double x = X[(size_t)c * D + e];
#pragma unroll
    for (int u = 0; u < TP; ++u) acc[u] += x * ps[e][q + u];
  }
#pragma unroll
  for (int u = 0; u < TP; ++u)
    if (t0 + q + u < r) Y[(size_t)c * r + t0 + q + u] = (float)acc[u];
}

// Correction and restore (eq. probe_residual_estimate and
// final_reconstructed_output): out_i = x_i + mu_R + ((x_i - mu_x)/s_x) Y Psi^T
// for the video rows; dense-prefix rows keep their (exact) sparse output.
// Probe rows are overwritten afterwards by k_probe_scatter.
template <int D>
__global__ __launch_bounds__(256) void k_correct(Geom g, Work w, void* out, int chunks) {
  // `chunks` chunks of 64 rows per block.  Thread (row = tid / 4,
  // quarter = tid % 4) owns the columns [quarter * D/4, quarter * D/4 + D/4)
  // of its row, held in registers; its partial of t = xbar Y
  // (Y = B_lambda Psi) over those columns is summed with the other quarters'
  // by lane exchange within the quad, and it forms its columns of
  // x + mu_R + t Psi^T.  The rank is processed in slices of 16 directions,
  // staged in LDS once per block when the rank fits one slice.
  constexpr int CW = D / 4, RS = 16;
  __shared__ __attribute__((aligned(16))) float fy[D][RS];
  __shared__ __attribute__((aligned(16))) float fp[D][RS];
  __shared__ __attribute__((aligned(16))) float fvs[3][D];  // mu_x, 1 / s_x, mu_R
  const int bq = blockIdx.y, bh = bq % g.BH, tid = threadIdx.x;
  const int r = g.r;
  const int rw = tid >> 2, qtr = tid & 3;
  const float* fv = w.fitv + (size_t)bq * 3 * D;
  const float* Y = w.fity + (size_t)bq * D * r;
  const float* Psi = w.fitpsi + (size_t)bq * D * r;
  const bool one_slice = r <= RS;
  auto stage = [&](int t0) {
    const int tn = min(RS, r - t0);
    for (int i = tid; i < D * RS; i += 256) {
      const int c = i / RS, t = i % RS;
      // 16-byte slot t/4 is XOR-swizzled by the column's quarter, so the
      // four quarters of a quad read different banks
      const int sl = (((t >> 2) ^ (c / CW)) & 3) * 4 + (t & 3);
      fy[c][sl] = t < tn ? Y[c * r + t0 + t] : 0.f;
      fp[c][sl] = t < tn ? Psi[c * r + t0 + t] : 0.f;
    }
  };
  // mu_x, 1 / s_x (one division per column and block, not per row), mu_R
  for (int i = tid; i < 3 * D; i += 256) fvs[i / D][i % D] = i / D == 1 ? 1.f / fv[i] : fv[i];
  if (one_slice) stage(0);
  __syncthreads();
  for (int chunk = 0; chunk < chunks; ++chunk) {
    const int row = (blockIdx.x * chunks + chunk) * 64 + rw;
    if ((blockIdx.x * chunks + chunk) * 64 >= g.N) break;  // uniform over the block
    const bool valid = row < g.N;
    const bool text = row < g.ntext;
    const float* src = w.osp + ((size_t)bq * g.N + (valid ? row : 0)) * D + qtr * CW;
    float x[CW], acc[CW];
#pragma unroll
    for (int c4 = 0; c4 < CW / 4; ++c4) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (valid) v = *(const float4*)(src + 4 * c4);
      x[4 * c4] = v.x;
      x[4 * c4 + 1] = v.y;
      x[4 * c4 + 2] = v.z;
      x[4 * c4 + 3] = v.w;
    }
#pragma unroll
    for (int c = 0; c < CW; ++c) acc[c] = 0.f;
    for (int t0 = 0; t0 < r; t0 += RS) {
      if (!one_slice) {
        __syncthreads();
        stage(t0);
        __syncthreads();
      }
      float tp[RS];
#pragma unroll
      for (int t = 0; t < RS; ++t) tp[t] = 0.f;
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const int col = qtr * CW + c;
        const float xb = (x[c] - fvs[0][col]) * fvs[1][col];
#pragma unroll
        for (int t4 = 0; t4 < RS / 4; ++t4) {
          const float4 y4 = *(const float4*)&fy[col][(t4 ^ qtr) * 4];
          tp[4 * t4] = fmaf(xb, y4.x, tp[4 * t4]);
          tp[4 * t4 + 1] = fmaf(xb, y4.y, tp[4 * t4 + 1]);
          tp[4 * t4 + 2] = fmaf(xb, y4.z, tp[4 * t4 + 2]);
          tp[4 * t4 + 3] = fmaf(xb, y4.w, tp[4 * t4 + 3]);
        }
      }
#pragma unroll
      for (int t = 0; t < RS; ++t) {
        tp[t] += tri_dpp<kDppXor1>(tp[t]);
        tp[t] += tri_dpp<kDppXor2>(tp[t]);
      }
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const int col = qtr * CW + c;
        float a = acc[c];
#pragma unroll
        for (int t4 = 0; t4 < RS / 4; ++t4) {
          const float4 p4 = *(const float4*)&fp[col][(t4 ^ qtr) * 4];
          a = fmaf(tp[4 * t4], p4.x, a);
          a = fmaf(tp[4 * t4 + 1], p4.y, a);
          a = fmaf(tp[4 * t4 + 2], p4.z, a);
          a = fmaf(tp[4 * t4 + 3], p4.w, a);
        }
        acc[c] = a;
      }
    }
    if (!valid) continue;
    const int64_t dst = q_base(g, bh, bq / g.BH) + (int64_t)row * g.sn + qtr * CW;
    float o[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) o[c] = text ? x[c] : x[c] + fvs[2][qtr * CW + c] + acc[c];
    if (g.bf16) {
      uint16_t* op = (uint16_t*)out + dst;
#pragma unroll
      for (int c8 = 0; c8 < CW / 8; ++c8) {
        uint32_t wd[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint16_t lo = __builtin_bit_cast(uint16_t, (__bf16)o[c8 * 8 + 2 * e]);
          const uint16_t hi = __builtin_bit_cast(uint16_t, (__bf16)o[c8 * 8 + 2 * e + 1]);
          wd[e] = (uint32_t)lo | ((uint32_t)hi << 16);
        }
        *(uint4*)(op + c8 * 8) = make_uint4(wd[0], wd[1], wd[2], wd[3]);
      }
    } else {
      float* op = (float*)out + dst;
#pragma unroll
      for (int c4 = 0; c4 < CW / 4; ++c4)
        *(float4*)(op + 4 * c4) = make_float4(o[4 * c4], o[4 * c4 + 1], o[4 * c4 + 2], o[4 * c4 + 3]);
    }
  }
}

// Probe rows take their exact dense rows (eq. final_reconstructed_output).
__global__ __launch_bounds__(128) void k_probe_scatter(Geom g, Work w, void* out) {
  const int p = blockIdx.x, bq = blockIdx.y, bh = bq % g.BH, c = threadIdx.x;
  if (p >= w.nprobes[bh] || c >= g.dv) return;
  const int row = w.probes[(size_t)bh * g.M + p];
  const float v = w.odp[((size_t)bq * g.M + p) * g.dv + c];
  const int64_t idx = q_base(g, bh, bq / g.BH) + (int64_t)row * g.sn + c;
  if (g.bf16) {
    const __bf16 b = (__bf16)v;
    ((uint16_t*)out)[idx] = __builtin_bit_cast(uint16_t, b);
  } else {
    ((float*)out)[idx] = v;
  }
}

template <int D>
static void fit_d(const Geom& g, const Work& w, void* out, hipStream_t s, hipEvent_t* ev) {
  // all G * BH query heads in one launch
  const int BQ = g.BH * g.G;
  k_fit_prep<D><<<BQ, 1024, 0, s>>>(g, w);
  if (g.M > 0) {  // without probes the statistics are all of the fit
    k_fit_gram<D><<<dim3((D / 32) * (D / 32), 3, BQ), 256, 0, s>>>(g, w);
    // float inputs (whose outputs are held to float rounding) and d = 64 get
    // the double solve; bf16 inputs of d = 128 the float one
    auto solve = [&](auto t) { k_fit_solve<D, decltype(t)><<<dim3(BQ, 2), 1024, 0, s>>>(g, w); };
    if constexpr (D <= 64)
      solve(0.0);
    else if (g.bf16)
      solve(0.f);
    else
      solve(0.0);
    k_fit_map<D><<<dim3((g.r + 15) / 16, BQ), 1024, 0, s>>>(g, w);
  }
  if (ev) (void)hipEventRecord(ev[3], s);
  const int chunks = row_chunks(g.N, BQ);
  k_correct<D><<<dim3((g.N + 64 * chunks - 1) / (64 * chunks), BQ), 256, 0, s>>>(g, w, out, chunks);
  if (g.M > 0) k_probe_scatter<<<dim3(g.M, BQ), 128, 0, s>>>(g, w, out);
  if (ev) (void)hipEventRecord(ev[4], s);
}

void launch_fit_correct(const Geom& g, const Work& w, void* out, hipStream_t s, hipEvent_t* ev) {
  if (g.d == 64)
    fit_d<64>(g, w, out, s, ev);
  else
    fit_d<128>(g, w, out, s, ev);
}

}  // namespace sparsepr
