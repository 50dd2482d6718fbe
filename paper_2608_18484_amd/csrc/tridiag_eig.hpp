// Symmetric eigensolver for the response bases (App. B.1, B.2) and the
// probe-residual basis (App. A.3 eq. app_probe_residual_basis), one block of
// NT threads per D x D matrix, in four stages:
//
//  1. Householder reduction to tridiagonal form, A = Q T Q^T with
//     Q = H_0 H_1 ... H_{D-3}, beta[k] the scale of reflector k: tri_reduce
//     (A in LDS, reflectors below its subdiagonal) or tri_reduce_reg (A in
//     registers, reflectors in the rows of V).
//  2. tri_eigvals: the leading eigenvalues of T by multisection of its Sturm
//     counts in float (8 or 16 threads per eigenvalue, each counting at one
//     point of the current bracket), descending; ones closer than that
//     resolves are told apart in double before their vectors (tri_refine).
//  3. tri_vectors: for the leading nvec eigenvalues, the twisted
//     factorisation of T - lambda I in double (stationary and progressive
//     pivot chains, each vector's two chains in different waves; twist index
//     at the smallest |gamma|, found by a group of 8 lanes per vector) with
//     Rayleigh-quotient corrections lambda += gamma / |z|^2, then the twisted
//     vector.  The vectors' tridiagonal residuals and mutual orthogonality
//     are then checked; ok = 0 reports a numerically repeated eigenvalue
//     (whose twisted vectors coincide) so that the caller can use its Jacobi
//     solver instead.
//  4. tri_back, tri_back_rows: the vectors are multiplied by Q (reflectors
//     applied last to first), each by a group of lanes of one wave with no
//     barriers.
//
// Every stage is a serial chain of one block, so latency is what counts:
//  * tri_reduce takes four barriers per column and one wave forms each
//    reflector: 231 us at D = 128 (1.8 us per column); tri_reduce_reg two
//    barriers, 146 us in float and 206 in double (D = 64, double: 65 us);
//  * the vectors' products, one lane per side and three sweeps over pivots
//    in global memory, were two thirds of stage 3 (97 us for 64 vectors at
//    D = 128); formed by all 8 lanes and kept in registers, stage 3 takes
//    about 60;
//  * with a fixed two Rayleigh passes, vectors of eigenvalues closer than
//    about 1e-3 of the largest kept more than 1e-9 of their neighbours, so
//    that double solves fell back to Jacobi on most inputs (0.93-1.0 ms a
//    solve at D = 64, 3 ms at D = 128).  The passes now go on until the
//    correction is small against the gap to the neighbouring eigenvalues
//    (their quotient bounds the vector's share of them).
//
// The float response bases of D = 128 keep the sequential forms (tri_reduce,
// SEQ vectors, tri_back): thousands of k-means decisions per head turn on their
// last bits, and a basis with other roundings, however exact, regroups a few
// rows of the largest calls.  The response bases of D = 64 and every
// probe-residual basis (float for bf16 inputs of D = 128, else double) use the
// others.
#pragma once
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>

namespace sparsepr {

template <int D, typename T, int NT = 1024>
struct TriWork {
  // tri_reduce_reg: waves holding the matrix.  At D = 128 two per SIMD (one
  // wave alone issues an instruction only every other slot: 186 us with 4
  // waves, 138 with 8); at D = 64 each wave has little to do beside the
  // scalars that every wave forms (65 us with 4, 70 with 8).  S strips of NR
  // rows (row i belongs to strip i % S).
  static constexpr int RW = D == 128 ? 8 : 4;
  static constexpr int S = RW * 64 / D, NR = D / S;
  static_assert(RW * 64 <= NT && S >= 2, "thread mapping");
  double d[D], e[D];         // diagonal, subdiagonal e[i] = T[i+1][i]; e[D-1] = 0
  float2 de[D];              // float (d[i], e2[i-1]) for the Sturm counts
  float lamf[D];             // leading eigenvalues from multisection, descending
  double lamv[D];            // Rayleigh-corrected eigenvalues of the vectors
  T beta[D];                 // reflector scales
  union {
    struct {  // tri_reduce_reg: rows k and k + 1 of the current step (double-
              // buffered), partial sums of A x and each wave's w = p - K v,
              // all in strip order
      alignas(16) T xb[2][D];
      alignas(16) T yb[2][D];
      alignas(16) T part[S][D];
      alignas(16) T ww[RW][D];
    };
    struct {  // tri_reduce: reflector v, w = p - K v, partial sums of p = A v
      T hv[D], hw[D];
      T lpart[NT / D][D];
    };
  };
  float glo, ghi, fnorm;
  double pivd;
  int ok, again;
};

// Lane exchanges by DPP (no LDS round trip): quad_perm [1,0,3,2] and
// [2,3,0,1] swap neighbours and pairs within each group of four lanes,
// row_half_mirror reverses each group of eight, row_mirror each row of 16.
enum : int { kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140 };

template <int CTRL>
__device__ __forceinline__ float tri_dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ double tri_dpp(double v) {
  const long long u = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(u & 0xffffffff), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// Sum over each aligned group of W lanes (W = 8 or 16), in every lane.
template <int W, typename T>
__device__ __forceinline__ T tri_group_sum(T v) {
  static_assert(W == 8 || W == 16, "group width");
  v += tri_dpp<kDppXor1>(v);
  v += tri_dpp<kDppXor2>(v);
  v += tri_dpp<kDppHalfMirror>(v);
  if constexpr (W == 16) v += tri_dpp<kDppMirror>(v);
  return v;
}

template <typename T>
__device__ __forceinline__ T tri_readlane(T v, int l) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
  } else {
    const long long u = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(u & 0xffffffff), l);
    const int hi = __builtin_amdgcn_readlane((int)(u >> 32), l);
    return __builtin_bit_cast(T, ((long long)hi << 32) | (unsigned int)lo);
  }
}

// Sum over the whole wave, in every lane.
template <typename T>
__device__ __forceinline__ T tri_wave_sum(T v) {
  v = tri_group_sum<16>(v);
  return (tri_readlane(v, 0) + tri_readlane(v, 16)) + (tri_readlane(v, 32) + tri_readlane(v, 48));
}

// Stage 1.  A: D x D symmetric in LDS, row stride D + 1 (overwritten: the
// updated trailing blocks and, below the subdiagonal, the reflectors).
template <int D, typename T, int NT>
__device__ void tri_reduce(T* A, TriWork<D, T, NT>& tw) {
  constexpr int LD = D + 1, S = NT / D, U = (D + 63) / 64;
  static_assert(S >= 1 && NT % D == 0, "thread mapping");
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int c = tid % D, s = tid / D;
  for (int k = 0; k < D - 1; ++k) {
    if (wid == 0) {
      // reflector H = I - beta v v^T taking x = A[k+1.., k] to alpha e_1
      T x[U];
      T st = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = k + 1 + lane + 64 * u;
        x[u] = i < D ? A[i * LD + k] : T(0);
        if (i > k + 1) st += x[u] * x[u];
      }
      st = tri_wave_sum(st);
      const T x0 = A[(k + 1) * LD + k];
      T alpha = x0, b = 0, v0 = x0;
      if (st > T(0)) {
        const T nrm = sqrt(x0 * x0 + st);
        alpha = x0 >= T(0) ? -nrm : nrm;
        v0 = x0 - alpha;
        b = T(-1) / (alpha * v0);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = k + 1 + lane + 64 * u;
        if (i < D) {
          const T vi = i == k + 1 ? v0 : x[u];
          tw.hv[i] = vi;
          A[i * LD + k] = vi;
        }
      }
      if (lane == 0) {
        tw.beta[k] = b;
        tw.e[k] = (double)alpha;
        tw.d[k] = (double)A[k * LD + k];
      }
    }
    __syncthreads();
    const T b = tw.beta[k];
    if (b == T(0)) continue;  // uniform: the trailing block is already reduced
    // p = beta A22 v, column c summed over rows j = k+1+s, k+1+s+S, ...
    if (c > k) {
      T acc = 0;
      for (int j = k + 1 + s; j < D; j += S) acc += A[j * LD + c] * tw.hv[j];
      tw.lpart[s][c] = acc;
    }
    __syncthreads();
    if (wid == 0) {
      T p[U], pv = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = k + 1 + lane + 64 * u;
        p[u] = 0;
        if (i < D) {
          T acc = 0;
#pragma unroll
          for (int q = 0; q < S; ++q) acc += tw.lpart[q][i];
          p[u] = b * acc;
          pv += p[u] * tw.hv[i];
        }
      }
      const T K = T(0.5) * b * tri_wave_sum(pv);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = k + 1 + lane + 64 * u;
        if (i < D) tw.hw[i] = p[u] - K * tw.hv[i];
      }
    }
    __syncthreads();
    // A22 -= v w^T + w v^T
    if (c > k) {
      const T vc = tw.hv[c], wc = tw.hw[c];
      for (int i = k + 1 + s; i < D; i += S) A[i * LD + c] -= tw.hv[i] * wc + tw.hw[i] * vc;
    }
    __syncthreads();
  }
  if (tid == 0) {
    tw.d[D - 1] = (double)A[(D - 1) * LD + D - 1];
    tw.e[D - 1] = 0.0;
  }
  __syncthreads();
}

// Power of two that takes the largest diagonal entry of a positive semidefinite
// double matrix, and with it every entry, to [1, 2) (1 for a matrix without a
// positive finite diagonal): the float stages square entries and their
// rounding noise, which leaves the float range for entries beyond 1e19 and
// below 1e-12.  Each wave finds it for itself.
template <int D>
__device__ __forceinline__ double tri_scale(const double* A) {
  const int lane = threadIdx.x & 63;
  double m = 0.0;
#pragma unroll
  for (int u = 0; u < D / 64; ++u) m = fmax(m, A[(size_t)(lane + 64 * u) * (D + 1)]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  return m > 0.0 && m <= DBL_MAX ? ldexp(1.0, -ilogb(m)) : 1.0;
}

// Stage 1 with the matrix in registers.  load(e): element e of the D x D symmetric matrix (row-major).
// Step k takes x = row k right of the diagonal to alpha e_1 by H = I - beta
// v v^T, v = x + (v0 - x0) e_{k+1}, and applies A <- A - v w^T - w v^T,
// w = p - K v, p = beta A v, K = beta p.v / 2.  A x is summed while every
// wave forms the reflector's scalars, A v = A x + (v0 - x0) A e_{k+1} taking
// the difference from row k + 1 (y).  Each wave then forms w for itself, and
// the strips owning rows k + 1 and k + 2 publish them for the next step: two
// barriers per step.  Rows and columns up to k are left alone by zeros in
// x and w.  Waves beyond RW only meet the barriers.
// A float matrix has its largest entry near 1 (tri_scale).  A row whose
// squares sum to at most TINY, 1e-15 of that at most and far below its
// rounding, counts as reduced: beta = 2 / v.v would leave the range of T.
template <int D, typename T, int NT, class Load>
__device__ void tri_reduce_reg(Load load, T* V, TriWork<D, T, NT>& tw) {
  using W = TriWork<D, T, NT>;
  constexpr int RW = W::RW, S = W::S, NR = W::NR, U = D / 64;
  constexpr int BK = 8, NB = NR / BK;
  constexpr T TINY = sizeof(T) == 4 ? T(1e-30) : T(1e-200);
  static_assert(NR % BK == 0, "row blocks");
  typedef T blk __attribute__((ext_vector_type(BK)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool red = wid < RW;
  const int c = tid % D, s = __builtin_amdgcn_readfirstlane(tid / D) % S;
  auto pos = [](int i) { return (i % S) * NR + i / S; };
  auto row_at = [](int q) { return q / NR + S * (q % NR); };
  blk a[NB];
  // register of row s + S u (u is wave-uniform): selects inside its block
  // (a dynamic index would put the matrix in scratch memory)
  auto pick = [&](int u) {
    T r = a[0][0];
#pragma unroll
    for (int bk = 0; bk < NB; ++bk)
      if (u / BK == bk) {
#pragma unroll
        for (int e = 0; e < BK; ++e) r = u % BK == e ? a[bk][e] : r;
      }
    return r;
  };
  if (red) {
#pragma unroll
    for (int bk = 0; bk < NB; ++bk)
#pragma unroll
      for (int e = 0; e < BK; ++e) a[bk][e] = load((s + S * (bk * BK + e)) * D + c);
    if (s == 0) {
      tw.xb[0][pos(c)] = c > 0 ? a[0][0] : T(0);
      if (c == 0) tw.d[0] = (double)a[0][0];
    } else if (s == 1) {
      tw.yb[0][pos(c)] = a[0][0];
    }
  }
  __syncthreads();
  for (int kk = 0; kk < D - 1; ++kk) {
    const int k = __builtin_amdgcn_readfirstlane(kk);  // keeps every test on it scalar
    const int cur = k & 1;
    const T* x = tw.xb[cur];
    const T* xs = x + s * NR;
    T xl[U], alpha = 0, b = 0, v0 = 0, x0 = 0;
    if (red) {
      T st = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = lane + 64 * u;
        xl[u] = x[q];
        if (row_at(q) != k + 1) st += xl[u] * xl[u];
      }
      x0 = x[pos(k + 1)];
      T acc[2] = {0, 0};
#pragma unroll
      for (int bk = 0; bk < NB; ++bk)
        if (S * BK * (bk + 1) > k + 1) {
#pragma unroll
          for (int e = 0; e < BK; ++e) acc[e & 1] = fma(a[bk][e], xs[bk * BK + e], acc[e & 1]);
        }
      tw.part[s][pos(c)] = acc[0] + acc[1];
      st = tri_wave_sum(st);
      alpha = x0;
      v0 = x0;
      if (st > TINY) {
        const T nrm = sqrt(fma(x0, x0, st));
        alpha = x0 >= T(0) ? -nrm : nrm;
        v0 = x0 - alpha;
        // beta = 2 / v.v of the rounded v keeps H orthogonal to rounding
        b = T(1) / (T(0.5) * fma(v0, v0, st));
      }
    }
    __syncthreads();
    if (red) {
      const T dl = v0 - x0;
      T p[U], vl[U], pv = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = lane + 64 * u, i = row_at(q);
        T t = dl * tw.yb[cur][q];
#pragma unroll
        for (int j = 0; j < S; ++j) t += tw.part[j][q];
        p[u] = i > k ? b * t : T(0);
        vl[u] = i == k + 1 ? v0 : xl[u];
        pv += p[u] * vl[u];
      }
      const T K = T(0.5) * b * tri_wave_sum(pv);
      T* ww = tw.ww[wid];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = lane + 64 * u;
        ww[q] = p[u] - K * vl[u];
        if (wid == 0) V[k * D + row_at(q)] = vl[u];
      }
      if (tid == 0) {
        tw.beta[k] = b;
        tw.e[k] = (double)alpha;
      }
      // ww is this wave's own: its reads only have to follow its writes
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const T wc = ww[pos(c)], vc = c == k + 1 ? v0 : x[pos(c)];
      const T* ws = ww + s * NR;
#pragma unroll
      for (int bk = 0; bk < NB; ++bk)
        if (S * BK * (bk + 1) > k + 1) {
#pragma unroll
          for (int e = 0; e < BK; ++e)
            a[bk][e] = fma(-xs[bk * BK + e], wc, fma(-ws[bk * BK + e], vc, a[bk][e]));
        }
      if (s == (k + 1) % S) {
        // row k + 1 took x0 where its reflector entry is v0
        const T r = pick((k + 1) / S) - dl * wc;
        tw.xb[cur ^ 1][pos(c)] = c > k + 1 ? r : T(0);
        if (c == k + 1) tw.d[k + 1] = (double)r;
      } else if (s == (k + 2) % S && k + 2 < D) {
        tw.yb[cur ^ 1][pos(c)] = pick((k + 2) / S);
      }
    }
    __syncthreads();
  }
  if (tid == 0) tw.e[D - 1] = 0.0;
  __syncthreads();
}

// Number of eigenvalues of T below x (float Sturm sequence).  Every e^2 is
// at least FLT_MIN, so a zero pivot gives an infinite next pivot (never a
// NaN) and the sequence continues from the one after, as with a pivot of
// -0 or an infinitesimal one.
template <int D>
__device__ __forceinline__ int tri_sturm_f(const float2* de, float x) {
  float q = 1.f;
  int cnt = 0;
#pragma unroll 16
  for (int i = 0; i < D; ++i) {
    const float2 v = de[i];
    q = fmaf(-v.y, __builtin_amdgcn_rcpf(q), v.x - x);
    cnt += q < 0.f;
  }
  return cnt;
}

// Multisection by groups of G lanes: tw.lamf[t], t < need, = the t-th largest
// eigenvalue, from the interval [glo, ghi]; each round divides a bracket by
// G + 1, and the rounds take it below float resolution.
template <int G, int D, typename T, int NT>
__device__ void tri_multisect(TriWork<D, T, NT>& tw, int need) {
  constexpr int ROUNDS = G >= 16 ? 7 : 9;
  const int tid = threadIdx.x;
  const int t = tid / G, sl = tid % G;  // eigenvalue, lane of its group
  if (t >= need) return;  // whole groups
  const int j = D - 1 - t;              // its ascending index
  float a = tw.glo, b = tw.ghi;
  for (int rnd = 0; rnd < ROUNDS; ++rnd) {
    const float h = (b - a) / (float)(G + 1);
    const float x = fmaf((float)(sl + 1), h, a);
    const int below = tri_sturm_f<D>(tw.de, x) <= j;  // lambda_j >= x
    // the points whose count is <= j form a prefix of the group
    int u = 0;
#pragma unroll
    for (int o = 0; o < G; ++o) u += __shfl(below, (tid & ~(G - 1)) + o);
    const float na = u == 0 ? a : fmaf((float)u, h, a);
    const float nb = u == G ? b : fmaf((float)(u + 1), h, a);
    a = na;
    b = fmaxf(nb, na);
  }
  if (sl == 0) tw.lamf[t] = 0.5f * (a + b);
}

// Stage 2: tw.lamf[t], t < min(need, D) = the leading eigenvalues of T,
// descending.  The rounds are bound by instruction issue once every SIMD has
// more than two waves, so few eigenvalues take 16 lanes each (seven rounds)
// and many take 8 (nine rounds).
template <int D, typename T, int NT>
__device__ void tri_eigvals(TriWork<D, T, NT>& tw, int need) {
  static_assert(NT >= 8 * D, "8 lanes per eigenvalue");
  const int tid = threadIdx.x;
  need = min(need, D);
  if (tid < D) {
    tw.de[tid] = make_float2((float)tw.d[tid], tid > 0 ? fmaxf((float)(tw.e[tid - 1] * tw.e[tid - 1]), FLT_MIN) : 0.f);
    tw.lamf[tid] = 0.f;
  }
  __syncthreads();
  if (tid < 64) {
    // Gershgorin interval and the double pivot floor
    float lo = FLT_MAX, hi = -FLT_MAX;
    double md2 = 0.0;
    for (int i = tid; i < D; i += 64) {
      const float r = (float)(fabs(tw.e[i]) + (i > 0 ? fabs(tw.e[i - 1]) : 0.0));
      lo = fminf(lo, (float)tw.d[i] - r);
      hi = fmaxf(hi, (float)tw.d[i] + r);
      md2 = fmax(md2, tw.e[i] * tw.e[i]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo = fminf(lo, __shfl_xor(lo, o));
      hi = fmaxf(hi, __shfl_xor(hi, o));
      md2 = fmax(md2, __shfl_xor(md2, o));
    }
    if (tid == 0) {
      const float w = fmaxf(fabsf(lo), fabsf(hi));
      tw.glo = lo - 1e-6f * w - FLT_MIN;
      tw.ghi = hi + 1e-6f * w + FLT_MIN;
      tw.fnorm = w;
      tw.pivd = DBL_MIN * fmax(1.0, md2);
    }
  }
  __syncthreads();
  if (need * 16 <= NT / 2)
    tri_multisect<16, D, T, NT>(tw, need);
  else
    tri_multisect<8, D, T, NT>(tw, need);
  __syncthreads();
}

// Reciprocal to about 1 ulp: the hardware estimate and two Newton steps, a
// third of an IEEE division's dependent chain, for the Sturm counts of
// tri_refine, which take only the signs of the pivots.  These stay within
// [DBL_MIN, 1 / DBL_MIN] in magnitude (tri_guard and the floor's scale).
__device__ __forceinline__ double tri_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

template <int D>
__device__ __forceinline__ double tri_guard(double x, double piv) {
  return fabs(x) < piv ? -piv : x;
}

// Eigenvalues closer together than the float multisection resolves: the
// leading n, each searched again by Sturm counts in double in a bracket of
// 4e-6 of the norm around its float value (whose error is below 4e-7), by
// groups of 8 lanes, to lamv.  Nine rounds divide the bracket by 4e8.
template <int D, typename T, int NT>
__device__ void tri_refine(TriWork<D, T, NT>& tw, int n) {
  constexpr int G = 8;
  const int tid = threadIdx.x, t = tid / G, sl = tid % G;
  if (t >= n) return;  // whole groups
  const int j = D - 1 - t;
  const double piv = tw.pivd, w = 2e-6 * (double)tw.fnorm;
  double a = (double)tw.lamf[t] - w, b = (double)tw.lamf[t] + w;
  for (int rnd = 0; rnd < 9; ++rnd) {
    const double h = (b - a) / (G + 1);
    const double x = fma((double)(sl + 1), h, a);
    double q = tri_guard<D>(tw.d[0] - x, piv);
    int cnt = q < 0.0;
#pragma unroll 8
    for (int i = 0; i < D - 1; ++i) {
      q = tri_guard<D>((tw.d[i + 1] - x) - tw.e[i] * (tw.e[i] * tri_rcp(q)), piv);
      cnt += q < 0.0;
    }
    const int below = cnt <= j;  // lambda_j >= x
    int u = 0;
#pragma unroll
    for (int o = 0; o < G; ++o) u += __shfl(below, (tid & ~(G - 1)) + o);
    const double na = u == 0 ? a : fma((double)u, h, a);
    const double nb = u == G ? b : fma((double)(u + 1), h, a);
    a = na;
    b = fmax(nb, na);
  }
  if (sl == 0) tw.lamv[t] = 0.5 * (a + b);
}

// One chain of the twisted factorisation of T - lam I for vector t: the
// stationary pivots dp (top down, `fwd`) or the progressive pivots dm
// (bottom up).  scr holds [2][D][D] doubles (dp, dm), entry (i, t) at
// i * D + t, so that each wave's accesses are contiguous.  SEQ also
// keeps the ratios rho_i = e_i / dp_i and sig_i = e_i / dm_{i+1} in rat
// ([2][D][D], the same layout).
template <int D, bool SEQ, typename T, int NT>
__device__ void tri_chain(const TriWork<D, T, NT>& tw, double lam, double* __restrict__ scr,
                          double* __restrict__ rat, int t, bool fwd) {
  const double piv = tw.pivd;
  if (fwd) {
    double* __restrict__ sdp = scr;
    double dp = tri_guard<D>(tw.d[0] - lam, piv);
    sdp[t] = dp;
#pragma unroll 8
    for (int i = 0; i < D - 1; ++i) {
      const double rho = tw.e[i] / dp;
      if (SEQ) rat[i * D + t] = rho;
      dp = tri_guard<D>((tw.d[i + 1] - lam) - tw.e[i] * rho, piv);
      sdp[(i + 1) * D + t] = dp;
    }
  } else {
    double* __restrict__ sdm = scr + D * D;
    double dm = tri_guard<D>(tw.d[D - 1] - lam, piv);
    sdm[(D - 1) * D + t] = dm;
#pragma unroll 8
    for (int i = D - 2; i >= 0; --i) {
      const double sig = tw.e[i] / dm;
      if (SEQ) rat[D * D + i * D + t] = sig;
      dm = tri_guard<D>((tw.d[i] - lam) - tw.e[i] * sig, piv);
      sdm[i * D + t] = dm;
    }
  }
}

// Product sweep of one side of the twisted vector (z_r = 1): above r,
// z_i = -rho_i z_{i+1}; below it, z_{i+1} = -sig_i z_i.  Both sides take
// the same instruction stream (the side is per lane), so two lanes of one
// wave sweep them together.  Multiplies each entry by `scale` and stores it
// to row when `store`; returns the sum of the squares of the unscaled
// entries.  Ratios are loaded 16 at a time ahead of the dependent products.
template <int D, typename T>
__device__ double tri_sweep(const double* __restrict__ rat, int t, int r, bool up, double scale, bool store,
                            T* __restrict__ row) {
  // step j uses ratio index up ? r-1-j : r+j and stores entry r -/+ (1+j)
  const double* __restrict__ base = up ? rat : rat + D * D;
  const int len = up ? r : D - 1 - r;
  const int dir = up ? -1 : 1;
  const int i0 = up ? r - 1 : r;
  double nrm = 0.0, z = 1.0;
  for (int j0 = 0; j0 < len; j0 += 16) {
    double f[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) f[u] = j0 + u < len ? base[(i0 + dir * (j0 + u)) * D + t] : 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (j0 + u < len) {
        z = -f[u] * z;
        nrm += z * z;
        if (store) row[r + dir * (1 + j0 + u)] = (T)(z * scale);
      }
    }
  }
  return nrm;
}

// Entries of the twisted vector (z_r = 1), D / 8 consecutive ones per lane of
// the vector's group of 8 (lane s): above r, z_i = f_i z_{i+1} with
// f_i = -e_i / dp_i; below it, z_i = f_i z_{i-1} with f_i = -e_{i-1} / dm_i.
// Each lane forms its ratios and their running products from its end nearer
// r, then multiplies them by the products of the lanes between.  Returns the
// group's sum of squares.
template <int D, typename T, int NT>
__device__ double tri_twisted(const TriWork<D, T, NT>& tw, const double* __restrict__ scr, int t, int r,
                              int s, double* z) {
  constexpr int NE = D / 8;
  const int i0 = s * NE;
#pragma unroll
  for (int u = 0; u < NE; ++u) {
    const int i = i0 + u;
    z[u] = scr[(i < r ? 0 : D * D) + i * D + t];
  }
#pragma unroll
  for (int u = 0; u < NE; ++u) {
    const int i = i0 + u;
    const double e = tw.e[i < r ? i : (i > r ? i - 1 : 0)];
    z[u] = i == r ? 1.0 : -e / z[u];
  }
  // products within the lane: downwards for the entries after r, upwards for
  // those before it (entry r is 1 in both)
#pragma unroll
  for (int u = 1; u < NE; ++u)
    if (i0 + u > r) z[u] *= i0 + u - 1 >= r ? z[u - 1] : 1.0;
#pragma unroll
  for (int u = NE - 2; u >= 0; --u)
    if (i0 + u < r) z[u] *= i0 + u + 1 <= r ? z[u + 1] : 1.0;
  // the whole lane's product towards the far side: its last entry (below r)
  // or its first (above r); lanes are combined in order of distance from r
  const int sr = r / NE, lane0 = (threadIdx.x & 63) & ~7;
  const double far = s >= sr ? z[NE - 1] : z[0];
  double m = 1.0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    // lane sr itself is cut at r: its two sides' products are its end entries
    const double lo = __shfl(far, lane0 + j), first = __shfl(z[0], lane0 + j);
    if (s > sr && j >= sr && j < s) m *= lo;
    if (s < sr && j <= sr && j > s) m *= j == sr ? first : lo;
  }
  double nrm = 0.0;
#pragma unroll
  for (int u = 0; u < NE; ++u) {
    if (s != sr) z[u] *= m;
    nrm += z[u] * z[u];
  }
  return tri_group_sum<8>(nrm);
}

// Stage 3.  VT: row t (stride LV) receives the eigenvector of lamf[t] for
// t < nvec (tridiagonal coordinates); tw.lamv[t] its corrected eigenvalue
// (lamf[nvec], when nvec < D, is read for the gap below the last one).
// scr, rat: this block's [2][D][D] doubles of global scratch each (rat for
// SEQ only).  The two pivot
// chains of a factorisation run in different waves; the twist search, the
// vector's products and the checks use a group of 8 lanes per vector.
// SEQ: the products one after another in two lanes, and
// exactly one correction.
template <int D, bool SEQ, typename T, int NT>
__device__ void tri_vectors(TriWork<D, T, NT>& tw, T* VT, int LV, int nvec, double* scr, double* rat) {
  static_assert(NT >= 8 * D && D % 32 == 0, "8 lanes per vector");
  constexpr int MAXP = 6;
  const int tid = threadIdx.x;
  const int t8 = tid >> 3, s8 = tid & 7;  // vector and lane of its group
  if (tid < D) tw.lamv[tid] = (double)tw.lamf[tid];
  if (tid == 0) {
    tw.ok = 1;
    tw.again = 0;
  }
  __syncthreads();
  const double tn = fmax((double)tw.fnorm, DBL_MIN);
  // distance to the neighbouring eigenvalues
  auto gap_of = [&](auto* lam) {
    double gap = tn;
    if (t8 > 0) gap = fmin(gap, (double)lam[t8 - 1] - (double)lam[t8]);
    if (t8 + 1 < D) gap = fmin(gap, (double)lam[t8] - (double)lam[t8 + 1]);
    return gap;
  };
  double conv = 0.0;
  if constexpr (!SEQ) {
    // a correction that starts nearer to another eigenvalue converges to that
    // one: closer ones are told apart first
    double gap = t8 < nvec ? gap_of(tw.lamf) : tn;
    if (s8 == 0 && !(gap >= 4e-6 * tn)) tw.again = 1;
    __syncthreads();
    const bool close = tw.again;
    __syncthreads();
    if (close) {
      tri_refine<D, T, NT>(tw, min(nvec + 1, D));
      if (tid == 0) tw.again = 0;
      __syncthreads();
      if (t8 < nvec) gap = gap_of(tw.lamv);
    }
    // a correction of size c leaves the vector about c / gap of its neighbours
    conv = sizeof(T) == 4 ? fmax(1e-7 * gap, 1e-14 * tn) : fmax(1e-12 * gap, 4e-15 * tn);
    __syncthreads();
  }
  T* row = VT + (size_t)t8 * LV;
  constexpr int NE = D / 8;
  for (int pass = 0;; ++pass) {
    // pivot chains: threads [0, D) bottom up, [D, 2D) top down
    if (tid < 2 * D && (tid % D) < nvec) tri_chain<D, SEQ>(tw, tw.lamv[tid % D], scr, rat, tid % D, tid >= D);
    __syncthreads();
    double nrm = 1.0, corr = 0.0, z[SEQ ? 1 : NE];
    int r = 0;
    if (t8 < nvec) {
      const int t = t8;
      const double lam = tw.lamv[t];
      // twist index: smallest |gamma_k|, k = s8 + 8j; ties to the smaller k
      double bg = 0.0, ba = -1.0;
      int bk = D;
#pragma unroll 8
      for (int k = s8; k < D; k += 8) {
        const double gk = scr[k * D + t] + scr[D * D + k * D + t] - (tw.d[k] - lam);
        const double ak = fabs(gk);
        if (ba < 0.0 || ak < ba) {
          ba = ak;
          bg = gk;
          bk = k;
        }
      }
      auto take = [&](double oa, double og, int ok) {
        if (oa < ba || (oa == ba && ok < bk)) {
          ba = oa;
          bg = og;
          bk = ok;
        }
      };
      take(tri_dpp<kDppXor1>(ba), tri_dpp<kDppXor1>(bg), __builtin_amdgcn_mov_dpp(bk, kDppXor1, 0xF, 0xF, true));
      take(tri_dpp<kDppXor2>(ba), tri_dpp<kDppXor2>(bg), __builtin_amdgcn_mov_dpp(bk, kDppXor2, 0xF, 0xF, true));
      take(tri_dpp<kDppHalfMirror>(ba), tri_dpp<kDppHalfMirror>(bg),
           __builtin_amdgcn_mov_dpp(bk, kDppHalfMirror, 0xF, 0xF, true));
      // one lane's choice for the group (NaN pivots can leave them apart)
      r = __shfl(bk, (tid & 63) & ~7);
      if constexpr (SEQ) {
        // the first pass needs |z|^2 for the correction, the last one to
        // normalise
        double side = s8 < 2 ? tri_sweep<D, T>(rat, t, r, s8 == 0, 1.0, false, row) : 0.0;
        side += tri_dpp<kDppXor1>(side);
        nrm = 1.0 + side;
      } else {
        nrm = tri_twisted<D, T, NT>(tw, scr, t, r, s8, z);
      }
      corr = bg / nrm;
      const bool next = SEQ ? pass == 0 : pass + 1 < MAXP && !(fabs(corr) <= conv);
      if (s8 == 0 && next) tw.again = 1;
    }
    __syncthreads();
    const bool more = tw.again;
    if (t8 < nvec) {
      if (!more) {
        const double sc = 1.0 / sqrt(nrm);
        if constexpr (SEQ) {
          if (s8 == 0) row[r] = (T)sc;
          if (s8 < 2) tri_sweep<D, T>(rat, t8, r, s8 == 0, sc, true, row);
        } else {
#pragma unroll
          for (int u = 0; u < NE; ++u) row[s8 * NE + u] = (T)(z[u] * sc);
        }
      }
      if (s8 == 0 && (!SEQ || more)) tw.lamv[t8] += corr;
    }
    __syncthreads();
    if (!more) break;
    if (tid == 0) tw.again = 0;
  }
  // residual |T z - lam z| per vector (8 lanes), then pairwise orthogonality:
  // each group keeps its vector in registers and meets the later ones
  constexpr int NC = D / 32;  // 4-entry pieces per lane: piece j starts at (8 j + s8) * 4
  typedef T T4 __attribute__((ext_vector_type(4)));
  const double tol = sizeof(T) == 4 ? 1e-4 : 1e-9;
  bool bad = false;
  if (t8 < nvec) {
    const double lam = tw.lamv[t8];
    for (int i = s8; i < D; i += 8) {
      double y = (tw.d[i] - lam) * (double)row[i];
      if (i > 0) y += tw.e[i - 1] * (double)row[i - 1];
      if (i < D - 1) y += tw.e[i] * (double)row[i + 1];
      bad |= !(fabs(y) <= tol * tn);  // NaN too
    }
    T4 z[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) z[j] = *(const T4*)(row + (8 * j + s8) * 4);
    // from the first vector after the wave's first: uniform over the wave
    for (int b = __builtin_amdgcn_readfirstlane(t8) + 1; b < nvec; ++b) {
      const T* zb = VT + (size_t)b * LV;
      double dot = 0.0;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const T4 y = *(const T4*)(zb + (8 * j + s8) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) dot = fma((double)z[j][e], (double)y[e], dot);
      }
      dot = tri_group_sum<8>(dot);
      if (b > t8) bad |= !(fabs(dot) <= tol);
    }
  }
  if (bad) tw.ok = 0;
  __syncthreads();
}

// Stage 4.  VT rows t < nvec <- Q applied to them.  A holds the reflectors
// of tri_reduce below its subdiagonal.  Vector t belongs to the GV = NT / D
// lanes of one group, lane s holding its entries s, s + GV, ... in
// registers for all D - 2 reflectors; group sums go by DPP, so the stage
// needs no barrier and each reflector costs one read of its column.
template <int D, typename T, int NT>
__device__ void tri_back(const T* A, const TriWork<D, T, NT>& tw, T* VT, int LV, int nvec) {
  constexpr int LD = D + 1, GV = NT / D, NZ = D / GV;
  static_assert(GV == 8 || GV == 16, "lanes per vector");
  const int tid = threadIdx.x, t = tid / GV, s = tid % GV;
  if (t < nvec) {  // whole groups of lanes
    T* row = VT + (size_t)t * LV;
    T z[NZ];
#pragma unroll
    for (int u = 0; u < NZ; ++u) z[u] = row[s + GV * u];
    for (int k = D - 3; k >= 0; --k) {
      const T b = tw.beta[k];
      if (b == T(0)) continue;
      T v[NZ];
      T dot = 0;
#pragma unroll
      for (int u = 0; u < NZ; ++u) {
        const int i = s + GV * u;
        const T a = A[i * LD + k];
        v[u] = i > k ? a : T(0);
        dot += v[u] * z[u];
      }
      const T f = b * tri_group_sum<GV>(dot);
#pragma unroll
      for (int u = 0; u < NZ; ++u) z[u] -= f * v[u];
    }
#pragma unroll
    for (int u = 0; u < NZ; ++u) row[s + GV * u] = z[u];
  }
  __syncthreads();
}

// Stage 4 with the reflectors in the rows of V (tri_reduce_reg).  Vector t belongs to the 8 lanes of one group, each
// holding D / 8 of its entries in registers for all D - 2 reflectors, in
// pieces of four so that a reflector is read by 16-byte accesses; group sums
// go by DPP, so the stage needs no barrier.
template <int D, typename T, int NT>
__device__ void tri_back_rows(const T* V, const TriWork<D, T, NT>& tw, T* VT, int LV, int nvec) {
  constexpr int NC = D / 32;
  typedef T T4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, t = tid >> 3, s = tid & 7;
  if (t < nvec) {  // whole groups of lanes
    T* row = VT + (size_t)t * LV;
    T4 z[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) z[j] = *(const T4*)(row + (8 * j + s) * 4);
    for (int k = D - 3; k >= 0; --k) {
      const T b = tw.beta[k];
      T4 v[NC];
      T dot = 0;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        v[j] = *(const T4*)(V + k * D + (8 * j + s) * 4);
        dot += (v[j].x * z[j].x + v[j].y * z[j].y) + (v[j].z * z[j].z + v[j].w * z[j].w);
      }
      const T f = b * tri_group_sum<8>(dot);
#pragma unroll
      for (int j = 0; j < NC; ++j) z[j] -= f * v[j];
    }
#pragma unroll
    for (int j = 0; j < NC; ++j) *(T4*)(row + (8 * j + s) * 4) = z[j];
  }
  __syncthreads();
}

}  // namespace sparsepr
