// FP64 symmetric eigensolver for the Gram matrix G = Y^T Y (Khat x Khat):
// the leading K_n eigenpairs give the leading K_n left singular vectors of Y
// (Section 2.2: the SVD step of an HOOI invocation) as Y V_K S_K^-1.
//
// One workgroup of 512 threads, the matrix resident in LDS when it fits:
//   1. Householder tridiagonalisation G = Q T Q^T.  Reflector k is
//      I - tau_k v v^T on rows/columns k+1..n-1 with v_0 = 1; it is built from
//      row k (G stays symmetric), and row k is never touched again, so the
//      reflector is kept as that row plus the scale that turns it into v.
//      Per step: p = tau A22 v (four threads per row), then the symmetric
//      rank-2 update A22 -= v w^T + w v^T with w = p - (tau/2)(p.v) v; two
//      barriers per step.
//   2. The K largest eigenvalues of T by multisection: a group of 16-64 lanes
//      inside one wavefront per eigenvalue, two Sturm counts per lane (the
//      number of eigenvalues below x, from the signs of the LDL^T pivots), and
//      a ballot that picks the sub-interval holding the eigenvalue; no
//      barriers, as many rounds as FP64 resolution needs.
//   3. Eigenvectors of T by inverse iteration: one LU factorisation of
//      T - lambda I with partial pivoting per eigenvalue, then two solves from
//      a seeded start vector.
//   4. Back-transformation z <- H_0 ... H_{n-3} z, half a wavefront per vector,
//      then CholeskyQR2 of the K vectors (modified Gram-Schmidt when a pivot is
//      not safely positive).
#include <cmath>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "lanes.hpp"

namespace tk {

constexpr int EIG_THREADS = 512;
constexpr int EIG_WAVES = EIG_THREADS / 64;

// Offsets, in doubles, of the solver's arrays.  A (n x (n+1)) comes first; the
// rest follows it, in LDS or in the global workspace.
struct EigLayout {
  int64_t A, d, e, e2, tau, scl, p, red, Z, lu, lam, gm;
  int64_t a_size, total;
};

static EigLayout eig_layout(int n, int K) {
  EigLayout L{};
  int64_t o = 0;
  L.A = o; o += (int64_t)n * (n + 1);
  L.a_size = o;
  L.d = o; o += n;
  L.e = o; o += n;
  L.e2 = o; o += n;
  L.tau = o; o += n;
  L.scl = o; o += n;
  L.p = o; o += n;
  L.red = o; o += 64;
  L.Z = o; o += (int64_t)K * n;
  L.lu = o; o += (int64_t)K * 5 * n;   // per vector: 1/u0, u1, u2, multiplier, pivot flag
  L.lam = o; o += K;
  L.gm = o; o += 2 * (int64_t)K * K + 2;
  L.total = o;
  return L;
}

__device__ __forceinline__ double wave_sum(double x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

__device__ __forceinline__ double half_sum(double x) {   // over each 32-lane half
  for (int off = 16; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// Data-parallel-primitive move of a double (both 32-bit halves with the same control; every lane has a source).
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)(b & 0xffffffffLL), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sum over each row of 16 lanes, in every lane of the row: swap neighbours,
// swap pairs (quad permutes), then mirror within 8 and within 16 lanes.
__device__ __forceinline__ double row16_sum(double x) {
  x += dpp_mov<0xB1>(x);    // quad_perm [1,0,3,2]
  x += dpp_mov<0x4E>(x);    // quad_perm [2,3,0,1]
  x += dpp_mov<0x141>(x);   // row_half_mirror
  x += dpp_mov<0x140>(x);   // row_mirror
  return x;
}

// Sum of x over the wave, in every lane: rows of 16, then rows and halves
// exchanged (each swap leaves the two operands' sums over both places).
__device__ __forceinline__ double wave_sum_u(double x) {
  x = row16_sum(x);
  long long b = __double_as_longlong(x);
  int lo = (int)(unsigned)(b & 0xffffffffLL), hi = (int)(b >> 32);
  auto l2 = __builtin_amdgcn_permlane16_swap(lo, lo, false, true);
  auto h2 = __builtin_amdgcn_permlane16_swap(hi, hi, false, true);
  x = __longlong_as_double(((long long)h2[0] << 32) | (unsigned)l2[0]) +
      __longlong_as_double(((long long)h2[1] << 32) | (unsigned)l2[1]);
  b = __double_as_longlong(x);
  lo = (int)(unsigned)(b & 0xffffffffLL);
  hi = (int)(b >> 32);
  l2 = __builtin_amdgcn_permlane32_swap(lo, lo, false, true);
  h2 = __builtin_amdgcn_permlane32_swap(hi, hi, false, true);
  return __longlong_as_double(((long long)h2[0] << 32) | (unsigned)l2[0]) +
         __longlong_as_double(((long long)h2[1] << 32) | (unsigned)l2[1]);
}

// Sum over the workgroup: wave sums, then every thread adds the wave partials in order.
__device__ __forceinline__ double block_sum(double x, double* red) {
  x = wave_sum(x);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < EIG_WAVES; ++w) s += red[w];
  __syncthreads();
  return s;
}

// Eigenvalues of the symmetric tridiagonal (d, e) below x0 and below x1 (two
// independent recurrences interleaved).
__device__ __forceinline__ void sturm_count2(const double* d, const double* e2, int n, double x0, double x1,
                                             double pivmin, int& c0, int& c1) {
  double q0 = d[0] - x0, q1 = d[0] - x1;
  if (fabs(q0) < pivmin) q0 = -pivmin;
  if (fabs(q1) < pivmin) q1 = -pivmin;
  c0 = q0 < 0.0;
  c1 = q1 < 0.0;
  for (int i = 1; i < n; ++i) {
    const double di = d[i], ei = e2[i - 1];
    q0 = di - x0 - ei / q0;
    q1 = di - x1 - ei / q1;
    if (fabs(q0) < pivmin) q0 = -pivmin;
    if (fabs(q1) < pivmin) q1 = -pivmin;
    c0 += q0 < 0.0;
    c1 += q1 < 0.0;
  }
}

// Counter-based start vector entry (SplitMix64 mix of (j, i)) in [-1, 1).
__device__ __forceinline__ double start_entry(int j, int i) {
  unsigned long long z = 0x9E3779B97F4A7C15ULL * (unsigned long long)(j * 1315423911u + i + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  z ^= z >> 31;
  return (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// Modified Gram-Schmidt over the K rows of Z (each of length n), block-wide.
template <class P>
__device__ void mgs_rows(P Z, int K, int n, double* red) {
  for (int j = 0; j < K; ++j) {
    P zj = Z + (int64_t)j * n;
    for (int i = 0; i < j; ++i) {
      P zi = Z + (int64_t)i * n;
      double s = 0.0;
      for (int t = threadIdx.x; t < n; t += blockDim.x) s += zi[t] * zj[t];
      s = block_sum(s, red);
      for (int t = threadIdx.x; t < n; t += blockDim.x) zj[t] -= s * zi[t];
      __syncthreads();
    }
    double s = 0.0;
    for (int t = threadIdx.x; t < n; t += blockDim.x) s += zj[t] * zj[t];
    s = block_sum(s, red);
    const double inv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
    for (int t = threadIdx.x; t < n; t += blockDim.x) zj[t] *= inv;
    __syncthreads();
  }
}

// Orthonormalise the K rows of Z by CholeskyQR twice (Gram matrix of the rows,
// its Cholesky factor R, rows <- R^-T rows); falls back to modified
// Gram-Schmidt when a pivot is not safely positive.  gm: 2*K*K doubles + a flag,
// tmp: K*n.
template <class P>
__device__ void orth_rows(P Z, int K, int n, P gm, P tmp, double* red) {
  P R = gm + K * K;
  int* flag = reinterpret_cast<int*>(&gm[2 * K * K]);
  for (int pass = 0; pass < 2; ++pass) {
    for (int q = threadIdx.x; q < K * K; q += blockDim.x) {
      const int a = q / K, b = q - a * K;
      double s = 0.0;
      if (a <= b)
        for (int t = 0; t < n; ++t) s += Z[(int64_t)a * n + t] * Z[(int64_t)b * n + t];
      gm[q] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int ok = 1;
      double dmax = 0.0;
      for (int i = 0; i < K; ++i) dmax = fmax(dmax, gm[i * K + i]);
      for (int i = 0; i < K * K; ++i) R[i] = 0.0;
      for (int j = 0; j < K && ok; ++j) {
        double dj = gm[j * K + j];
        for (int k = 0; k < j; ++k) dj -= R[k * K + j] * R[k * K + j];
        if (!(dj > 1e-20 * dmax)) { ok = 0; break; }
        const double rjj = sqrt(dj);
        R[j * K + j] = rjj;
        for (int i = j + 1; i < K; ++i) {
          double v = gm[j * K + i];
          for (int k = 0; k < j; ++k) v -= R[k * K + j] * R[k * K + i];
          R[j * K + i] = v / rjj;
        }
      }
      *flag = ok;
    }
    __syncthreads();
    if (!*flag) {  // (rare) nearly dependent vectors
      mgs_rows(Z, K, n, red);
      return;
    }
    // rows: q_j = (z_j - sum_{i<j} R[i][j] q_i) / R[j][j], solved column by column in parallel over t
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
      for (int j = 0; j < K; ++j) {
        double v = Z[(int64_t)j * n + t];
        for (int i = 0; i < j; ++i) v -= R[i * K + j] * tmp[(int64_t)i * n + t];
        tmp[(int64_t)j * n + t] = v / R[j * K + j];
      }
      for (int j = 0; j < K; ++j) Z[(int64_t)j * n + t] = tmp[(int64_t)j * n + t];
    }
    __syncthreads();
  }
}

// MODE 2: everything in LDS.  MODE 1: A in the global workspace, the rest in
// LDS.  MODE 0: everything in the global workspace.
template <int MODE>
__global__ __launch_bounds__(EIG_THREADS) void k_syev_topk(const double* __restrict__ G, int n, int K, int Kout,
                                                           EigLayout L, double* __restrict__ gws,
                                                           double* __restrict__ lam_out, double* __restrict__ VK) {
  extern __shared__ double sh[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform
  const int stride = n + 1;
  double* A = MODE == 2 ? sh : gws;
  // the remaining arrays: in LDS (MODE 1 and 2, after A only in MODE 2) or after A in the workspace
  auto at = [&](int64_t off) -> double* { return MODE == 0 ? gws + off : sh + (off - (MODE == 1 ? L.a_size : 0)); };
  double* d = at(L.d);
  double* e = at(L.e);
  double* e2 = at(L.e2);
  double* tau = at(L.tau);
  double* scl = at(L.scl);
  double* p = at(L.p);
  double* red = at(L.red);
  double* Z = at(L.Z);
  double* lu = at(L.lu);
  double* lam = at(L.lam);
  double* gm = at(L.gm);

  for (int i = wave; i < n; i += EIG_WAVES)
    for (int j = lane; j < n; j += 64) A[(int64_t)i * stride + j] = G[(int64_t)i * n + j];
  __syncthreads();

  // 1. tridiagonalisation
  for (int k = 0; k + 2 < n; ++k) {
    const int m = n - k - 1;
    const double* rowk = A + (int64_t)k * stride + (k + 1);   // x_0..x_{m-1}, later the reflector
    double s = 0.0;
    for (int i = lane + 1; i < m; i += 64) s += rowk[i] * rowk[i];
    const double xn2 = wave_sum(s);     // every wave computes the same value
    const double alpha = rowk[0];
    if (xn2 == 0.0) {                   // the column is already reduced: identity reflector
      if (tid == 0) {
        d[k] = A[(int64_t)k * stride + k];
        e[k] = alpha;
        tau[k] = 0.0;
        scl[k] = 0.0;
      }
      continue;
    }
    const double beta = -copysign(sqrt(alpha * alpha + xn2), alpha);
    const double t = (beta - alpha) / beta;
    const double scale = 1.0 / (alpha - beta);
    // p = t * A22 v, four threads per row
    for (int i0 = 0; i0 < m; i0 += EIG_THREADS / 4) {
      const int i = i0 + (tid >> 2), sub = tid & 3;
      double acc = 0.0;
      if (i < m) {
        const double* row = A + (int64_t)(k + 1 + i) * stride + (k + 1);
        for (int j = sub; j < m; j += 4) acc += row[j] * (j == 0 ? 1.0 : rowk[j] * scale);
      }
      acc += __shfl_xor(acc, 1, 64);
      acc += __shfl_xor(acc, 2, 64);
      if (i < m && sub == 0) p[i] = t * acc;
    }
    __syncthreads();
    double pv = 0.0;
    for (int i = lane; i < m; i += 64) pv += p[i] * (i == 0 ? 1.0 : rowk[i] * scale);
    const double kc = 0.5 * t * wave_sum(pv);
    // A22 -= v w^T + w v^T, rows over waves, columns over lanes
    for (int i = wave; i < m; i += EIG_WAVES) {
      const double vi = i == 0 ? 1.0 : rowk[i] * scale;
      const double wi = p[i] - kc * vi;
      double* row = A + (int64_t)(k + 1 + i) * stride + (k + 1);
      for (int j = lane; j < m; j += 64) {
        const double vj = j == 0 ? 1.0 : rowk[j] * scale;
        const double wj = p[j] - kc * vj;
        row[j] -= vi * wj + wi * vj;
      }
    }
    if (tid == 0) {
      d[k] = A[(int64_t)k * stride + k];
      e[k] = beta;
      tau[k] = t;
      scl[k] = scale;
    }
    __syncthreads();
  }
  if (tid == 0) {
    if (n >= 2) {
      d[n - 2] = A[(int64_t)(n - 2) * stride + (n - 2)];
      e[n - 2] = A[(int64_t)(n - 2) * stride + (n - 1)];
      tau[n - 2] = 0.0;
    }
    d[n - 1] = A[(int64_t)(n - 1) * stride + (n - 1)];
    e[n - 1] = 0.0;
    tau[n - 1] = 0.0;
  }
  __syncthreads();
  for (int i = tid; i < n; i += EIG_THREADS) e2[i] = e[i] * e[i];
  __syncthreads();

  // Gershgorin interval and scales (every thread, same order)
  double glo = 1e300, ghi = -1e300, emax = 0.0, tnorm = 0.0;
  for (int i = 0; i < n; ++i) {
    const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0);
    glo = fmin(glo, d[i] - r);
    ghi = fmax(ghi, d[i] + r);
    emax = fmax(emax, i + 1 < n ? e2[i] : 0.0);
    tnorm = fmax(tnorm, fabs(d[i]) + r);
  }
  const double eps = 2.220446049250313e-16;
  const double pivmin = fmax(2.2250738585072014e-308, eps * eps * emax);
  const double widen = 2.0 * eps * fmax(fabs(glo), fabs(ghi)) + pivmin;
  glo -= widen;
  ghi += widen;

  // 2. multisection: MS lanes (inside one wave) per eigenvalue, two points per lane
  {
    const int MS = K <= 8 ? 64 : (K <= 16 ? 32 : 16);
    const int NP = 2 * MS;                       // points per round -> NP + 1 sub-intervals
    const int g = tid / MS, q = tid % MS;
    const int gbase = lane & ~(MS - 1);
    const unsigned long long gmask = MS == 64 ? ~0ULL : (((1ULL << MS) - 1) << gbase);
    const double tol = 2.0 * eps * fmax(fabs(glo), fabs(ghi)) + pivmin;
    int rounds = 1;
    for (double w = ghi - glo; w > tol && rounds < 24; w /= (double)(NP + 1)) ++rounds;
    const bool act = g < K;
    const int idx = n - 1 - g;                   // ascending index of the g-th largest
    double a = glo, b = ghi;
    for (int r = 0; r < rounds; ++r) {
      const double h = (b - a) / (double)(NP + 1);
      const double x0 = a + h * (double)(2 * q + 1), x1 = a + h * (double)(2 * q + 2);
      int c0 = 0, c1 = 0;
      if (act) sturm_count2(d, e2, n, x0, x1, pivmin, c0, c1);
      // points with at most idx eigenvalues below them lie below the eigenvalue
      const unsigned long long m0 = __ballot(c0 <= idx) & gmask, m1 = __ballot(c1 <= idx) & gmask;
      const int P = __popcll(m0) + __popcll(m1);
      const double na = P == 0 ? a : a + h * (double)P;
      const double nb = P == NP ? b : a + h * (double)(P + 1);
      a = na;
      b = nb;
    }
    if (act && q == 0) lam[g] = 0.5 * (a + b);
  }
  __syncthreads();

  // 3. eigenvectors of T by inverse iteration, thread j for eigenvector j
  const double tiny = eps * fmax(tnorm, pivmin);
  for (int j = tid; j < K; j += EIG_THREADS) {
    double lj = lam[j];
    // separate (numerically) equal eigenvalues so the factorisations differ
    for (int i = 0; i < j; ++i)
      if (fabs(lam[i] - lj) < 10.0 * eps * fmax(tnorm, 1e-300)) lj -= 10.0 * eps * fmax(tnorm, 1e-300);
    double* ui = lu + (int64_t)j * 5 * n;   // 1/u0
    double* u1 = ui + n;
    double* u2 = u1 + n;
    double* ml = u2 + n;
    double* pv = ml + n;
    double* z = Z + (int64_t)j * n;
    double a0 = d[0] - lj, a1 = n > 1 ? e[0] : 0.0, a2 = 0.0;
    for (int i = 0; i < n - 1; ++i) {
      const double c = e[i], nd = d[i + 1] - lj, ns = i + 1 < n - 1 ? e[i + 1] : 0.0;
      if (fabs(c) > fabs(a0)) {         // swap rows i and i+1
        const double mlt = a0 / c;
        ui[i] = 1.0 / c; u1[i] = nd; u2[i] = ns; ml[i] = mlt; pv[i] = 1.0;
        a0 = a1 - mlt * nd;
        a1 = a2 - mlt * ns;
      } else {
        if (a0 == 0.0) a0 = tiny;
        const double mlt = c / a0;
        ui[i] = 1.0 / a0; u1[i] = a1; u2[i] = a2; ml[i] = mlt; pv[i] = 0.0;
        a0 = nd - mlt * a1;
        a1 = ns - mlt * a2;
      }
      a2 = 0.0;
    }
    if (a0 == 0.0) a0 = tiny;
    ui[n - 1] = 1.0 / a0; u1[n - 1] = 0.0; u2[n - 1] = 0.0; ml[n - 1] = 0.0; pv[n - 1] = 0.0;
    for (int i = 0; i < n; ++i) z[i] = start_entry(j, i);
    for (int it = 0; it < 2; ++it) {
      for (int i = 0; i < n - 1; ++i) {
        if (pv[i] != 0.0) {
          const double t0 = z[i];
          z[i] = z[i + 1];
          z[i + 1] = t0 - ml[i] * z[i + 1];
        } else {
          z[i + 1] -= ml[i] * z[i];
        }
      }
      double z1 = 0.0, z2 = 0.0, nrm = 0.0;
      for (int i = n - 1; i >= 0; --i) {
        const double s = (z[i] - u1[i] * z1 - u2[i] * z2) * ui[i];
        z[i] = s;
        z2 = z1;
        z1 = s;
        nrm += s * s;
      }
      nrm = nrm > 0.0 ? 1.0 / sqrt(nrm) : 0.0;
      for (int i = 0; i < n; ++i) z[i] *= nrm;
    }
  }
  __syncthreads();

  // 4. back-transformation, half a wave per vector (both halves run every
  // iteration: the shuffles need the whole wave)
  {
    const int half = lane >> 5, hl = lane & 31;
    for (int j0 = 0; j0 < K; j0 += 2 * EIG_WAVES) {
      const int j = j0 + 2 * wave + half;
      const bool on = j < K;
      double* z = Z + (int64_t)(on ? j : 0) * n;
      for (int k = n - 3; k >= 0; --k) {
        const double t = tau[k];
        if (t == 0.0) continue;
        const int m = n - k - 1;
        const double* rowk = A + (int64_t)k * stride + (k + 1);
        const double sc = scl[k];
        double s = 0.0;
        if (on)
          for (int i = hl; i < m; i += 32) s += (i == 0 ? 1.0 : rowk[i] * sc) * z[k + 1 + i];
        s = half_sum(s);
        if (on)
          for (int i = hl; i < m; i += 32) z[k + 1 + i] -= t * s * (i == 0 ? 1.0 : rowk[i] * sc);
      }
    }
  }
  __syncthreads();
  orth_rows(Z, K, n, gm, lu, red);
  for (int t = tid; t < n * K; t += EIG_THREADS) {
    const int i = t / K, j = t - i * K;
    VK[(int64_t)i * Kout + j] = Z[(int64_t)j * n + i];
  }
  for (int j = tid; j < K; j += EIG_THREADS) lam_out[j] = lam[j];
}

// ---- K-hat <= 128: register-resident variant ----------------------------------------------------
//
// One workgroup of four waves, one per SIMD; what bounds it is the chain of
// dependent FP64 operations, so each phase is laid out for a short chain and
// few LDS reads.
//
//   1. Tridiagonalisation.  Wave w keeps rows I = 4u + w of the matrix in
//      registers, lane l its columns J = l and l + 64.  Step k needs p = tau A v
//      of the reflector built from x = row k.  With u = x - beta e_{k+1},
//      v = u / (alpha - beta), the waves multiply A with the raw x in the same
//      pass over the registers that applies reflector k - 1 (A x needs neither
//      beta nor tau, so the norm's reduction, root and reciprocals run beside
//      it), and A u = A x - beta A e_{k+1} follows from row k + 1, which its
//      owner publishes.  The waves' partial products and that row meet in LDS
//      (double-buffered by step parity): one barrier per step.  Every wave then
//      forms v, w and the next x on its own, once with J over the lanes and
//      once with the wave's own rows over the lanes of each 16-lane row, from
//      where a 64-bit row broadcast hands v_I, w_I and x_I to the pass.
//   2. Eigenvalues by multisection on the Sturm sequence of the leading
//      principal minors, p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}: two
//      multiply-adds per step and no division.  T is scaled by a power of two to
//      norm [1, 2) and e^2 floored at 1e-36 (a perturbation below 1e-18 of the
//      norm), so that eight steps cannot underflow (each shrinks the pair
//      (p_i, p_{i-1}) by at most e^2 / 6); the pair is rescaled every eighth step.
//      How far it goes: see small_is_fine.
//   3. Inverse iteration, lane j of one row of 16 for vector j.  What it needs is
//      all the LDS holds beside the packed reflectors, so n up to 128 runs here.
//   4. Back-transformation, a row of 16 lanes per vector, and, where
//      eigenvalues are close (fine: always), modified Gram-Schmidt over the
//      rows, twice.
//
// Measured at n = 100, K = 10 (one launch): 354 -> 161 us against a form with the
// matrix in LDS, eight waves, whose passes were bound by LDS reads (three
// broadcast reads per row) and whose Sturm steps divided.  Of the 161:
// tridiagonalisation 104, multisection 17, LU 17, solves 10, back-transformation
// 12.  n = 25, K = 5: 76 -> 35.
constexpr int SM_N = 128;
constexpr int SM_WAVES = 4;
constexpr int SM_THREADS = 64 * SM_WAVES;

struct SmallLayout {
  int64_t v, d, e, tau, lam, Z, lu, part, row, total;
};

// doubles of the packed reflectors: reflector k keeps columns from the 16-column
// block of its first entry, k + 1
__host__ __device__ constexpr int small_voff(int m, int NG) {
  const int b = m >> 4, i = m & 15;
  return 16 * (16 * (b * NG - b * (b - 1) / 2) + i * (NG - b));
}

static SmallLayout small_layout(int n) {
  SmallLayout L{};
  const int NG = (n + 15) / 16;
  int64_t o = 0;
  L.v = o; o += small_voff(n > 1 ? n - 1 : 1, NG);
  L.d = o; o += SM_N + 16;
  L.e = o; o += SM_N + 16;
  L.tau = o; o += SM_N;
  L.lam = o; o += 16;
  L.Z = o; o += 16 * (int64_t)n;
  // the LU factors share their place with the tridiagonalisation's buffers
  L.lu = o;
  L.part = o;
  L.row = o + 2 * SM_WAVES * SM_N;
  o += std::max<int64_t>(64 * (int64_t)n, 2 * SM_WAVES * SM_N + 3 * SM_N);
  L.total = o;
  return L;
}

// Up to n (n + 6 K) = 16640 (n = 102 at K = 10, 89 at K = 16) an eigenvalue stops
// at 1e-11 of the norm: inverse iteration needs no more, the SVD step's
// CholeskyQR2 restores what is left in U, and the eigenvalues only scale its
// columns.  Larger problems are taken to FP64
// resolution as in the general solver: the Rayleigh-Ritz steps of the block-Krylov solver
// for ranks from 12 on are among them, and an eigenvalue's error there is a
// floor of the residual that a caller's eig_tol is compared with (n = 121, K = 11:
// 196 us to 1e-11, 213 to FP64 resolution, 1517 in the general solver).
static bool small_is_fine(int n, int K) { return n * (n + 6 * K) > 16640; }

// Newton-refined hardware reciprocal
__device__ __forceinline__ double rcp2(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}

// value at column J (wave-uniform) of a row held as NC registers
template <int NC>
__device__ __forceinline__ double col_of(const double (&x)[NC], int J) {
  const double a = lane_value(x[0], J & 63), b = lane_value(x[NC - 1], J & 63);   // both read: a select of two registers
  return J < 64 ? a : b;                                          // by index would put them in memory
}

// NG: 16-row groups of the matrix (n <= 16 NG).
template <int NG>
__global__ __launch_bounds__(SM_THREADS) void k_syev_small(const double* __restrict__ G, int n, int K, int Kout,
                                                           bool fine, SmallLayout L, double* __restrict__ lam_out,
                                                           double* __restrict__ VK) {
  extern __shared__ __align__(16) double sh[];
  constexpr int NC = NG <= 4 ? 1 : 2;     // columns per lane, and row-layout registers
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform
  const int l16 = lane & 15;
  double* V = sh + L.v;
  double* d = sh + L.d;
  double* e = sh + L.e;
  double* tau = sh + L.tau;
  double* lam = sh + L.lam;
  double* Z = sh + L.Z;

  for (int i = tid; i < SM_N + 16; i += SM_THREADS) d[i] = e[i] = 0.0;
  __syncthreads();

  // 1. tridiagonalisation
  {
    double* part = sh + L.part;
    double* rowb = sh + L.row;
    double a[NG * 4][NC];
    int J[NC], Ir[NC];   // this lane's columns; its rows in the row layout
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      J[c] = lane + 64 * c;
      Ir[c] = 4 * (l16 + 16 * c) + wave;
    }
#pragma unroll
    for (int u = 0; u < NG * 4; ++u) {
      const int I = 4 * u + wave;
#pragma unroll
      for (int c = 0; c < NC; ++c) a[u][c] = (I < n && J[c] < n) ? G[(int64_t)I * n + J[c]] : 0.0;
    }
    double x[NC], xr[NC], v[NC], w[NC], nvr[NC], nwr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      x[c] = (J[c] >= 1 && J[c] < n) ? G[J[c]] : 0.0;
      xr[c] = (Ir[c] >= 1 && Ir[c] < n) ? G[Ir[c]] : 0.0;
      v[c] = w[c] = nvr[c] = nwr[c] = 0.0;
    }
    double beta, t, scale;
    // the reflector that maps the entries J >= j0 of x to beta e_{j0} (the
    // identity when those past j0 are zero)
    auto reflect = [&](int j0) __attribute__((always_inline)) {
      double s = 0.0;
#pragma unroll
      for (int c = 0; c < NC; ++c) s = fma(x[c], J[c] > j0 ? x[c] : 0.0, s);
      const double xn2 = wave_sum_u(s);
      const double alpha = col_of<NC>(x, j0);
      // root of h = alpha^2 + xn2 from the hardware's 1 / sqrt(h), refined twice
      const double h = fma(alpha, alpha, xn2);
      double y = __builtin_amdgcn_rsq(h);
      double g = h * y, hf = 0.5 * y;
      double r = fma(-hf, g, 0.5);
      g = fma(g, r, g);
      hf = fma(hf, r, hf);
      r = fma(-hf, g, 0.5);
      g = fma(g, r, g);
      hf = fma(hf, r, hf);
      g = fma(fma(-g, g, h), hf, g);
      const double bt = -copysign(g, alpha);
      // factors 0 and 1, not selects of the results: those become a branch
      const bool id = xn2 == 0.0;
      const double on = id ? 0.0 : 1.0, am = id ? 1.0 : alpha - bt;
      beta = id ? alpha : bt;
      t = on * (am * copysign(2.0 * (id ? 1.0 : hf), alpha));
      scale = on * rcp2(am);
    };
    // rows of the groups from G0 on: A -= v w^T + w v^T (UPD), acc = A x, both
    // over the columns from C0 on; row kp, which lies in group G0, goes to the
    // row buffer.  Waves that do not own it write to a spare one: no branches,
    // so that the next reflector's chain runs among these multiply-adds.
    auto pass = [&](auto upd, auto g0, int kp, int buf) __attribute__((always_inline)) {
      constexpr bool UPD = decltype(upd)::value;
      constexpr int G0 = decltype(g0)::value, C0 = G0 >= 5 ? NC - 1 : 0;
      double acc[NC][2] = {};
      static_for<4 * (NG - G0)>([&](auto ui) __attribute__((always_inline)) {
        constexpr int u = decltype(ui)::value + 4 * G0, r = u >> 4, ln = u & 15;
        const double xI = row_bcast<ln>(xr[r]);
        if constexpr (UPD) {
          const double vI = row_bcast<ln>(nvr[r]), wI = row_bcast<ln>(nwr[r]);
#pragma unroll
          for (int c = C0; c < NC; ++c) a[u][c] = fma(wI, v[c], fma(vI, w[c], a[u][c]));
        }
#pragma unroll
        for (int c = C0; c < NC; ++c) acc[c][u & 1] = fma(a[u][c], xI, acc[c][u & 1]);
      });
      if constexpr (UPD) {
        double* rb = rowb + ((kp & 3) == wave ? buf : 2) * SM_N;
        const int q = (kp >> 2) & 3;
#pragma unroll
        for (int c = C0; c < NC; ++c) {
          const double a0 = a[4 * G0][c], a1 = a[4 * G0 + 1][c], a2 = a[4 * G0 + 2][c], a3 = a[4 * G0 + 3][c];
          const double lo = q & 1 ? a1 : a0, hi = q & 1 ? a3 : a2;
          rb[lane + 64 * c] = q & 2 ? hi : lo;
        }
      }
      double* pb = part + (buf * SM_WAVES + wave) * SM_N;
#pragma unroll
      for (int c = C0; c < NC; ++c) pb[lane + 64 * c] = acc[c][0] + acc[c][1];
    };
    using std::true_type;
    using std::false_type;
    // row 1 for step 0 comes the same way as the later ones
    if (wave == 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) rowb[lane + 64 * c] = (n > 1 && J[c] < n) ? G[n + J[c]] : 0.0;
    }
    pass(false_type{}, std::integral_constant<int, 0>{}, 0, 0);
    if (n >= 2) {
      reflect(1);
    } else {
      beta = t = scale = 0.0;
    }
    if (tid == 0) {
      d[0] = G[0];
      e[0] = beta;
      if (n == 2) d[1] = G[3];
    }
    double* const spare = rowb + 2 * SM_N + lane;   // where masked stores go
    // step k, k + 2 in group G0
    auto step = [&](auto g0, int k) __attribute__((always_inline)) {
      constexpr int G0 = decltype(g0)::value, C0 = G0 >= 5 ? NC - 1 : 0;
      const int buf = k & 1;
      __syncthreads();
      // y = A x, and row k + 1 of A, in both layouts
      double y[NC], yr[NC], rp[NC], rpr[NC];
      const double* pb = part + buf * SM_WAVES * SM_N;
      const double* rb = rowb + buf * SM_N;
#pragma unroll
      for (int c = C0; c < NC; ++c) {
        double s[SM_WAVES];
#pragma unroll
        for (int ww = 0; ww < SM_WAVES; ++ww) s[ww] = pb[ww * SM_N + J[c]];
        rp[c] = rb[J[c]];
        y[c] = (s[0] + s[1]) + (s[2] + s[3]);
      }
#pragma unroll
      for (int c = C0; c < NC; ++c) {
        double s[SM_WAVES];
#pragma unroll
        for (int ww = 0; ww < SM_WAVES; ++ww) s[ww] = pb[ww * SM_N + Ir[c]];
        rpr[c] = rb[Ir[c]];
        yr[c] = (s[0] + s[1]) + (s[2] + s[3]);
      }
      const double ts = t * scale;
      double pv = 0.0;
#pragma unroll
      for (int c = C0; c < NC; ++c) {
        v[c] = J[c] == k + 1 ? 1.0 : x[c] * scale;   // x is zero up to column k
        w[c] = J[c] > k ? ts * fma(-beta, rp[c], y[c]) : 0.0;
        pv = fma(w[c], v[c], pv);
      }
      // the reflector, for the back-transformation (every wave the same values)
      const int vb = ((k + 1) >> 4) << 4;
      double* vk = V + small_voff(k + 1, NG) - vb;
#pragma unroll
      for (int c = C0; c < NC; ++c) *(J[c] >= vb && J[c] < 16 * NG ? vk + J[c] : spare) = v[c];
      *(lane == 0 ? tau + k : spare) = t;
      const double kc = 0.5 * t * wave_sum_u(pv);
#pragma unroll
      for (int c = C0; c < NC; ++c) w[c] = fma(-kc, v[c], w[c]);
      const double wk1 = col_of<NC>(w, k + 1);
#pragma unroll
      for (int c = C0; c < NC; ++c) {
        const double nx = rp[c] - fma(wk1, v[c], w[c]);   // row k + 1 after reflector k
        *(J[c] == k + 1 ? d + k + 1 : spare) = nx;
        x[c] = J[c] > k + 1 ? nx : 0.0;
      }
#pragma unroll
      for (int c = C0; c < NC; ++c) {
        const double vr = Ir[c] == k + 1 ? 1.0 : xr[c] * scale;
        const double wr = fma(-kc, vr, Ir[c] > k ? ts * fma(-beta, rpr[c], yr[c]) : 0.0);
        const double nx = rpr[c] - fma(wk1, vr, wr);
        xr[c] = Ir[c] > k + 1 ? nx : 0.0;
        nvr[c] = -vr;
        nwr[c] = -wr;
      }
      reflect(k + 2);
      *(lane == 0 ? e + k + 1 : spare) = beta;
      pass(true_type{}, g0, k + 2, buf ^ 1);
    };
    static_for<NG>([&](auto g0) __attribute__((always_inline)) {
      constexpr int G0 = decltype(g0)::value;
      const int k1 = min(16 * G0 + 14, n - 2);
      for (int k = max(16 * G0 - 2, 0); k < k1; ++k) step(g0, k);
    });
    __syncthreads();
    if (n >= 3 && tid == 0) d[n - 1] = rowb[(n & 1) * SM_N + n - 1];
  }
  __syncthreads();
  // norm and Gershgorin interval of T (every wave, same order), then T scaled
  // by a power of two to norm [1, 2)
  double glo = 1e300, ghi = -1e300, tnorm = 0.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int i = lane + 64 * c;
    if (i < n) {
      const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0);
      glo = fmin(glo, d[i] - r);
      ghi = fmax(ghi, d[i] + r);
      tnorm = fmax(tnorm, fabs(d[i]) + r);
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    glo = fmin(glo, __shfl_xor(glo, off, 64));
    ghi = fmax(ghi, __shfl_xor(ghi, off, 64));
    tnorm = fmax(tnorm, __shfl_xor(tnorm, off, 64));
  }
  const int ex = tnorm > 0.0 ? ilogb(tnorm) : 0;
  __syncthreads();   // the unscaled entries have been read
  for (int i = tid; i < n; i += SM_THREADS) {
    d[i] = ldexp(d[i], -ex);
    e[i] = i + 1 < n ? ldexp(e[i], -ex) : 0.0;
  }
  glo = ldexp(glo, -ex);
  ghi = ldexp(ghi, -ex);
  tnorm = ldexp(tnorm, -ex);
  const double eps = 2.220446049250313e-16;
  const double widen = 4.0 * eps * fmax(fmax(fabs(glo), fabs(ghi)), 1.0);
  glo -= widen;
  ghi += widen;
  // start vectors of the inverse iteration
  for (int i = tid; i < 16 * n; i += SM_THREADS) Z[i] = start_entry(i & 15, i >> 4);
  __syncthreads();

  // 2. multisection until the interval is below 1e-11 of the norm (fine: at
  // FP64's resolution)
  {
    // eigenvalues below x: sign changes of the sequence
    auto count = [&](double xp) __attribute__((always_inline)) {
      double pm = 0.0, pc = 1.0;
      uint32_t sg = 0;
      int cnt = 0;
      auto one = [&](double di, double e2) __attribute__((always_inline)) {
        const double pn = fma(di - xp, pc, -(e2 * pm));
        pm = pc;
        pc = pn;
        sg = __builtin_amdgcn_alignbit(sg, (uint32_t)(__double_as_longlong(pn) >> 32), 31);
      };
      auto rescale = [&]() __attribute__((always_inline)) {
        const int q = -__builtin_amdgcn_frexp_exp(fmax(fabs(pc), fabs(pm)));
        pc = __builtin_amdgcn_ldexp(pc, q);
        pm = __builtin_amdgcn_ldexp(pm, q);
      };
      for (int i0 = 0; i0 < n; i0 += 16) {
        const double dr = d[i0 + l16], er = i0 + l16 > 0 ? e[i0 + l16 - 1] : 0.0;
        const double e2r = fmax(er * er, 1e-36);
        if (i0 + 16 <= n) {
          static_for<16>([&](auto ii) __attribute__((always_inline)) {
            constexpr int i = decltype(ii)::value;
            one(row_bcast<i>(dr), row_bcast<i>(e2r));
            if constexpr ((i & 7) == 7) rescale();
          });
          cnt += __popc((sg ^ (sg >> 1)) & 0xffffu);
        } else {
          const int m = n - i0;
          static_for<16>([&](auto ii) __attribute__((always_inline)) {
            constexpr int i = decltype(ii)::value;
            if (i < m) {
              one(row_bcast<i>(dr), row_bcast<i>(e2r));
              if constexpr ((i & 7) == 7) rescale();
            }
          });
          cnt += __popc((sg ^ (sg >> 1)) & ((1u << m) - 1));
        }
      }
      return cnt;
    };
    const int MS = K <= 4 ? 64 : K <= 8 ? 32 : 16;   // lanes per eigenvalue, one point each
    const int g = tid / MS, q = tid & (MS - 1);
    const unsigned long long gmask = MS == 64 ? ~0ULL : ((1ULL << MS) - 1) << (lane & ~(MS - 1));
    const double tol = fine ? 2.0 * eps * fmax(fabs(glo), fabs(ghi)) : 1e-11 * fmax(tnorm, 1.0);
    const int idx = n - 1 - g;
    // joint first round: one point per thread over the whole interval
    int* cnt0 = reinterpret_cast<int*>(sh + L.part);
    const double h0 = (ghi - glo) / (double)(SM_THREADS + 1);
    cnt0[tid] = count(glo + h0 * (double)(tid + 1));
    __syncthreads();
    int t0 = -1, t1 = SM_THREADS - 1;   // largest t with cnt0[t] <= idx (counts rise with x)
    while (t0 < t1) {
      const int mid = (t0 + t1 + 1) >> 1;
      if (cnt0[mid] <= idx) t0 = mid; else t1 = mid - 1;
    }
    double lo = t0 < 0 ? glo : glo + h0 * (double)(t0 + 1);
    double hi = t0 >= SM_THREADS - 1 ? ghi : glo + h0 * (double)(t0 + 2);
    int rounds = 0;
    for (double wd = h0; wd > tol && rounds < 32; wd /= (double)(MS + 1)) ++rounds;
    // a wave with no eigenvalue of its own skips; within a wave all lanes count
    if (wave * (64 / MS) < K) {
      for (int r = 0; r < rounds; ++r) {
        const double h = (hi - lo) / (double)(MS + 1);
        const int cn = count(lo + h * (double)(q + 1));
        const int P = __popcll(__ballot(cn <= idx) & gmask);
        const double na = P == 0 ? lo : lo + h * (double)P;
        const double nb = P == MS ? hi : lo + h * (double)(P + 1);
        lo = na;
        hi = nb;
      }
      if (g < K && q == 0) lam[g] = 0.5 * (lo + hi);
    }
  }
  __syncthreads();

  // 3. eigenvectors of T by inverse iteration, lane j of the first row of 16
  // for vector j: one LU factorisation of T - lambda I with partial pivoting,
  // two solves from the seeded start vector (the first forward elimination runs
  // with the factorisation).  Step i of vector j keeps {multiplier, u2/u0} in P
  // and {1/u0, u1/u0} in U; the rows were swapped where u2/u0 is not +0 (a zero
  // of a swapped row is stored as -0).
  if (tid < 16) {
    const int j = min(tid, K - 1);
    double lj = lam[j];
    const double sep = 10.0 * eps * fmax(tnorm, 1.0);
    // separate (numerically) equal eigenvalues so the factorisations differ
    for (int i = 0; i < j; ++i)
      if (fabs(lam[i] - lj) < sep) lj -= sep;
    double2* P = reinterpret_cast<double2*>(sh + L.lu) + tid;
    double2* U = P + 16 * n;
    double* z = Z + tid;
    const double tiny = eps * fmax(tnorm, 1.0);
    double a0 = d[0] - lj, a1 = e[0];
    double cur = z[0];
    auto lu_step = [&](int i, double c, double dn, double ns, double nz) __attribute__((always_inline)) {
      const double nd = dn - lj;
      const bool sw = fabs(c) > fabs(a0);
      const double p0 = sw ? c : (a0 == 0.0 ? tiny : a0);
      const double r = rcp2(p0);
      const double m0 = (sw ? a0 : c) * r;
      const double y1 = sw ? nd : a1, x1 = sw ? a1 : nd;   // the pivot row's entry, the other row's
      const double y2 = ns * r;
      P[16 * i] = double2{m0, sw ? (y2 == 0.0 ? -0.0 : y2) : 0.0};
      U[16 * i] = double2{r, y1 * r};
      z[16 * i] = sw ? nz : cur;
      cur = sw ? fma(-m0, nz, cur) : fma(-m0, cur, nz);
      a0 = fma(-m0, y1, x1);
      a1 = sw ? -(m0 * ns) : ns;
    };
    const int nl = n - 1;
    int i0 = 0;
    for (; i0 < nl; i0 += 16) {
      // rows i0 .. i0+15 over the lanes (entries past the end are zero)
      const double ce = e[i0 + tid], cd = d[i0 + 1 + tid], cs = i0 + 1 + tid < nl ? e[i0 + 1 + tid] : 0.0;
      double nz[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) nz[i] = z[16 * min(i0 + i + 1, nl)];
      if (i0 + 16 <= nl) {
        static_for<16>([&](auto ii) __attribute__((always_inline)) {
          constexpr int i = decltype(ii)::value;
          lu_step(i0 + i, row_bcast<i>(ce), row_bcast<i>(cd), row_bcast<i>(cs), nz[i]);
        });
      } else {
        static_for<16>([&](auto ii) __attribute__((always_inline)) {
          constexpr int i = decltype(ii)::value;
          if (i0 + i < nl) lu_step(i0 + i, row_bcast<i>(ce), row_bcast<i>(cd), row_bcast<i>(cs), nz[i]);
        });
      }
    }
    if (a0 == 0.0) a0 = tiny;
    P[16 * nl] = double2{0.0, 0.0};
    U[16 * nl] = double2{rcp2(a0), 0.0};
    z[16 * nl] = cur;
    constexpr int CH = 8;   // steps whose operands are loaded together
    for (int it = 0; it < 2; ++it) {
      if (it == 1) {   // forward elimination with the row interchanges
        cur = z[0];
        auto fw = [&](int i, double nz, double2 p) __attribute__((always_inline)) {
          const bool sw = __double_as_longlong(p.y) != 0;
          z[16 * i] = sw ? nz : cur;
          cur = sw ? fma(-p.x, nz, cur) : fma(-p.x, cur, nz);
        };
        int i = 0;
        for (; i + CH <= nl; i += CH) {
          double nz[CH];
          double2 p[CH];
#pragma unroll
          for (int s = 0; s < CH; ++s) { nz[s] = z[16 * (i + s + 1)]; p[s] = P[16 * (i + s)]; }
#pragma unroll
          for (int s = 0; s < CH; ++s) fw(i + s, nz[s], p[s]);
        }
        for (; i < nl; ++i) fw(i, z[16 * (i + 1)], P[16 * i]);
        z[16 * nl] = cur;
      }
      // back substitution
      double z1 = 0.0, z2 = 0.0;
      auto bw = [&](int i, double zi, double2 u, double u2) __attribute__((always_inline)) {
        const double s = fma(-u.y, z1, fma(-u2, z2, zi * u.x));
        z[16 * i] = s;
        z2 = z1;
        z1 = s;
      };
      int i = nl;
      for (; i - CH + 1 >= 0; i -= CH) {
        double zi[CH], u2[CH];
        double2 u[CH];
#pragma unroll
        for (int s = 0; s < CH; ++s) { zi[s] = z[16 * (i - s)]; u2[s] = P[16 * (i - s)].y; u[s] = U[16 * (i - s)]; }
#pragma unroll
        for (int s = 0; s < CH; ++s) bw(i - s, zi[s], u[s], u2[s]);
      }
      for (; i >= 0; --i) bw(i, z[16 * i], U[16 * i], P[16 * i].y);
    }
  }
  __syncthreads();

  // 4. back-transformation: row of 16 lanes q of wave w holds vector 4w + q,
  // entry l16 + 16 t in z[t]
  const int vec = 4 * wave + (lane >> 4);
  double z[NG];
  {
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < NG; ++t) {
      const int i = l16 + 16 * t;
      z[t] = i < n && vec < K ? Z[16 * i + vec] : 0.0;
      s = fma(z[t], z[t], s);
    }
    s = row16_sum(s);
    s = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
#pragma unroll
    for (int t = 0; t < NG; ++t) z[t] *= s;
  }
  if (4 * wave < K) {
    // reflectors whose first entry m = k + 1 lies in 16-entry block b touch blocks b ..
    static_for<NG>([&](auto bi) __attribute__((always_inline)) {
      constexpr int b = NG - 1 - decltype(bi)::value, NB = NG - b;
      const int mhi = min(16 * b + 15, n - 2), mlo = max(16 * b, 1);
      if (mhi < mlo) return;
      double vn[NB], tn;
      auto fetch = [&](int m) __attribute__((always_inline)) {
        const double* vk = V + small_voff(m, NG) + l16;
#pragma unroll
        for (int t = 0; t < NB; ++t) vn[t] = vk[16 * t];
        tn = tau[m - 1];
      };
      fetch(mhi);
      for (int m = mhi; m >= mlo; --m) {
        double vv[NB];
        const double tk_ = tn;
#pragma unroll
        for (int t = 0; t < NB; ++t) vv[t] = vn[t];
        fetch(max(m - 1, mlo));   // one step ahead of its use
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int t = 0; t < NB; ++t) {
          if (t & 1) s1 = fma(vv[t], z[b + t], s1);
          else s0 = fma(vv[t], z[b + t], s0);
        }
        const double s = -tk_ * row16_sum(s0 + s1);
#pragma unroll
        for (int t = 0; t < NB; ++t) z[b + t] = fma(s, vv[t], z[b + t]);
      }
    });
  }
  // inverse iteration leaves vectors of eigenvalues more than 1e-3 ||T|| apart
  // orthogonal to working accuracy; closer ones are orthonormalised together
  bool cluster = fine;
  for (int j = 1; j < K; ++j) cluster |= fabs(lam[j - 1] - lam[j]) < 1e-3 * tnorm;
  if (cluster) {
    double* qb = sh + L.part;   // the current vector, double-buffered
    for (int pass = 0; pass < 2; ++pass) {
      for (int j = 0; j < K; ++j) {
        double* q = qb + (j & 1) * SM_N;
        if (vec == j) {
          double s = 0.0;
#pragma unroll
          for (int t = 0; t < NG; ++t) s = fma(z[t], z[t], s);
          s = row16_sum(s);
          s = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
#pragma unroll
          for (int t = 0; t < NG; ++t) {
            z[t] *= s;
            q[l16 + 16 * t] = z[t];
          }
        }
        __syncthreads();
        double qv[NG], s = 0.0;
#pragma unroll
        for (int t = 0; t < NG; ++t) {
          qv[t] = q[l16 + 16 * t];
          s = fma(qv[t], z[t], s);
        }
        s = vec > j ? row16_sum(s) : 0.0;
#pragma unroll
        for (int t = 0; t < NG; ++t) z[t] = fma(-s, qv[t], z[t]);
      }
      __syncthreads();
    }
  }
  if (vec < K) {
#pragma unroll
    for (int t = 0; t < NG; ++t) {
      const int i = l16 + 16 * t;
      if (i < n) VK[(int64_t)i * Kout + vec] = z[t];
    }
  }
  if (tid < K) lam_out[tid] = ldexp(lam[tid], ex);
}

void eig_topk_krylov(Ctx* c, const double* G, int n, int K, int Kout, double* lam_k, double* VK, int mode);

constexpr int KRYLOV_MIN_N = 192;   // above this, and for K <= 16, the block-Krylov solver

// Leading K eigenpairs of G (n0 x n0, FP64): lam_k[0..K) descending and VK (n0 x K).
// Eigenpairs beyond n0 (K > n0) are reported as zero eigenvalues.  mode >= 0
// lets the Krylov solver start from that mode's previous eigenvectors.
// The dense solvers (one workgroup): LDS-resident for K-hat up to about 128,
// otherwise with the matrix in LDS or global memory.
void eig_topk_dense(Ctx* c, const double* G, int n0, int K, double* lam_k, double* VK) {
  const int Ke = K < n0 ? K : n0;
  TK_REQUIRE(Ke <= 32, TK_ERR_UNSUPPORTED, "eigensolve: more than 32 eigenpairs");
  const size_t lim = c->lds_per_block;
  const SmallLayout SL = small_layout(n0);
  const bool small = n0 <= SM_N && Ke <= 16 && (size_t)SL.total * 8 <= lim;
  const EigLayout L = eig_layout(n0, Ke);
  ensure(c, c->work, sizeof(double) * (size_t)(L.total + 16));
  if (K > Ke) TK_HIP(hipMemsetAsync(lam_k, 0, sizeof(double) * K, c->stream));
  double* ws = c->work.as<double>();
  if (small) {
    switch ((n0 + 15) / 16) {
#define TK_SMALL_CASE(NG)                                                                                       \
      case NG:                                                                                                  \
        hipLaunchKernelGGL(k_syev_small<NG>, dim3(1), dim3(SM_THREADS), (size_t)SL.total * 8, c->stream, G, n0, \
                           Ke, K, small_is_fine(n0, Ke), SL, lam_k, VK);                                        \
        break;
      TK_SMALL_CASE(1) TK_SMALL_CASE(2) TK_SMALL_CASE(3) TK_SMALL_CASE(4)
      TK_SMALL_CASE(5) TK_SMALL_CASE(6) TK_SMALL_CASE(7) TK_SMALL_CASE(8)
#undef TK_SMALL_CASE
      default: fail(TK_ERR_UNSUPPORTED, "eigensolve: size out of range");
    }
  } else if ((size_t)L.total * 8 <= lim) {
    hipLaunchKernelGGL(k_syev_topk<2>, dim3(1), dim3(EIG_THREADS), (size_t)L.total * 8, c->stream, G, n0, Ke, K, L,
                       ws, lam_k, VK);
  } else if ((size_t)(L.total - L.a_size) * 8 <= lim) {
    hipLaunchKernelGGL(k_syev_topk<1>, dim3(1), dim3(EIG_THREADS), (size_t)(L.total - L.a_size) * 8, c->stream,
                       G, n0, Ke, K, L, ws, lam_k, VK);
  } else {
    hipLaunchKernelGGL(k_syev_topk<0>, dim3(1), dim3(EIG_THREADS), 0, c->stream, G, n0, Ke, K, L, ws, lam_k, VK);
  }
  TK_CHECK_LAUNCH();
}

void eig_topk(Ctx* c, const double* G, int n0, int K, double* lam_k, double* VK, int mode) {
  const int Ke = K < n0 ? K : n0;
  TK_REQUIRE(Ke <= 32, TK_ERR_UNSUPPORTED, "eigensolve: more than 32 eigenpairs");
  const SmallLayout SL = small_layout(n0);
  const bool small = n0 <= SM_N && Ke <= 16 && (size_t)SL.total * 8 <= c->lds_per_block;
  if (!small && n0 >= KRYLOV_MIN_N && Ke <= 16) {
    eig_topk_krylov(c, G, n0, Ke, K, lam_k, VK, mode);
    return;
  }
  eig_topk_dense(c, G, n0, K, lam_k, VK);
}

}  // namespace tk
