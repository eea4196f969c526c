// New factor from the leading eigenpairs of G = Y^T Y (Section 2.2: the new
// F_n holds the leading K_n left singular vectors of Y_(n)):
//   U  = Y W,  W = V_K diag(lam_k)^(-1/2)     (R_n x K_n; FP32 MFMA for K <= 16,
//                                              else FP64 accumulation)
//   CholeskyQR2 in FP64: A = U^T U, A = R^T R (Cholesky), U <- U R^-1, twice,
//   which restores orthonormality to working precision;
//   F_n = U on the nonempty slices' rows, zero elsewhere (FP64 master),
//   plus the padded FP32 working copy the TTM-chain gathers.
// Columns whose singular value is zero (rank deficiency) are completed on the
// host with unit vectors e_i (lowest i not yet spanned, Gram-Schmidt in FP64).
#include <cmath>

#include "common.hpp"
#include "lanes.hpp"

namespace tk {

void tall_times_small(Ctx* c, const float* Y, int64_t R, int khat, const double* W, int K, double* U);

constexpr int FT_ROWS = 64;  // rows of Y per workgroup

// U = Y W and per-workgroup partial of U^T U.  W (khat x K, FP64) is in LDS;
// Y rows are staged through LDS with a padded stride, FT_ROWS at a time, over
// `tiles` consecutive tiles per workgroup.
__global__ __launch_bounds__(256) void k_uw(const float* __restrict__ Y, int64_t R, int khat,
                                            const double* __restrict__ W, int K, int tiles, double* __restrict__ U,
                                            double* __restrict__ part) {
  extern __shared__ double shd[];
  double* w = shd;                                      // khat * K
  double* ut = w + (size_t)khat * K;                    // FT_ROWS * K
  float* yt = reinterpret_cast<float*>(ut + FT_ROWS * K);  // FT_ROWS * (khat + 1)
  const int ys = khat + 1;
  for (int i = threadIdx.x; i < khat * K; i += blockDim.x) w[i] = W[i];
  double acc[4] = {0.0, 0.0, 0.0, 0.0};  // entries tid, tid+256, ... of U^T U (K <= 32)
  for (int tt = 0; tt < tiles; ++tt) {
    const int64_t r0 = ((int64_t)blockIdx.x * tiles + tt) * FT_ROWS;
    if (r0 >= R) break;
    const int nr = (int)min<int64_t>(FT_ROWS, R - r0);
    __syncthreads();
    for (int i = threadIdx.x; i < nr * khat; i += blockDim.x) {
      const int r = i / khat, cc = i - r * khat;
      yt[r * ys + cc] = Y[(r0 + r) * khat + cc];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nr * K; i += blockDim.x) {
      const int r = i / K, k = i - r * K;
      double s = 0.0;
      for (int cc = 0; cc < khat; ++cc) s += (double)yt[r * ys + cc] * w[cc * K + k];
      ut[r * K + k] = s;
      U[(r0 + r) * K + k] = s;
    }
    __syncthreads();
    for (int q = 0; q < 4; ++q) {
      const int i = threadIdx.x + 256 * q;
      if (i < K * K) {
        const int a = i / K, b = i - a * K;
        double s = acc[q];
        for (int r = 0; r < nr; ++r) s += ut[r * K + a] * ut[r * K + b];
        acc[q] = s;
      }
    }
  }
  for (int q = 0; q < 4; ++q) {
    const int i = threadIdx.x + 256 * q;
    if (i < K * K) part[(int64_t)blockIdx.x * K * K + i] = acc[q];
  }
}

typedef float floatx4_f __attribute__((ext_vector_type(4)));
typedef double doublex4_f __attribute__((ext_vector_type(4)));

constexpr int UW_WAVES = 16;      // waves per workgroup of the K <= 16 kernels, at most
constexpr int UW_SH = 32;         // doubles of scratch scaled_w needs

// The waves' Grams, summed in wave order: this workgroup's K x K partial.
// Register r of lane (q, j) = (l/16, l%16) holds entry (q + 4r, j); tiles: 256
// doubles per wave, free in every wave.
__device__ __forceinline__ void write_gram_part(const doublex4_f& g, int K, double* tiles, double* __restrict__ part) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r) tiles[wave * 256 + ((lane >> 4) + 4 * r) * 16 + (lane & 15)] = g[r];
  __syncthreads();
  if (threadIdx.x < 256) {
    double s = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += tiles[w * 256 + threadIdx.x];
    const int a = threadIdx.x >> 4, b = threadIdx.x & 15;
    if (a < K && b < K) part[(int64_t)blockIdx.x * K * K + a * K + b] = s;
  }
}

// W = V_K diag(lam)^(-1/2).  A column whose eigenvalue is at or below the
// Gram's rounding floor is not a direction of Y: an exactly zero singular
// value of Y shows up in the FP32 Gram as an eigenvalue of the size of the
// Gram's rounding error, below u ||Y||_F^2 (u = 2^-24), so eigenvalues up to
// RANK_FLOOR * trace(G) are taken as zero.  Such a column sets flag bit 2
// (rank deficiency) and gets W = 0.  Above the floor a small eigenvalue is
// kept: its vector is only as accurate as the Gram allows, but it lies in the
// range of Y.
constexpr double RANK_FLOOR = 4.0 / 16777216.0;   // 4 u

// What the kernels below form W from: lam null: W = VK as given.  diag[i *
// dstride], i < khat: the Gram's diagonal (dstride = khat + 1 in the Gram
// itself, 1 for a separate vector).
struct FactorW {
  const double* VK;    // khat x K
  const double* lam;
  const double* diag;
  int64_t dstride;
  int* flag;           // set to the failure bits of W (0 or 2)
  int* kvalid;         // columns above the floor
};

// W as the B operand of the FP32 MFMA in LDS: wl[16 c + j], zero beyond khat
// and K.  Every workgroup forms its own (a launch and a trip through memory
// less); `first` also writes the flag and the count.
__device__ __forceinline__ void scaled_w(const FactorW& w, int khat, int K, bool first, double* sh, float* wl) {
  const int kpad = (khat + 15) & ~15;
  const int wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  if (w.lam) {
    double t = 0.0;
    for (int i = threadIdx.x; i < khat; i += blockDim.x) t += w.diag[(int64_t)i * w.dstride];
    for (int d = 32; d > 0; d >>= 1) t += __shfl_xor(t, d);
    if ((threadIdx.x & 63) == 0) sh[wave] = t;
    __syncthreads();
    double tr = 0.0;
    for (int i = 0; i < waves; ++i) tr += sh[i];
    const double floor_ = RANK_FLOOR * tr;
    if (threadIdx.x < 16) {
      const int k = threadIdx.x;
      const bool ok = k < K && k < khat && w.lam[k] > floor_ && w.lam[k] > 0.0;   // only khat eigenpairs exist
      sh[16 + k] = ok ? 1.0 / sqrt(w.lam[k]) : 0.0;
      const unsigned good = (unsigned)__ballot(ok) & 0xffffu;
      if (first && k == 0) {   // eigenvalues come in descending order
        w.kvalid[0] = __ffs(~good) - 1;
        w.flag[0] = good == (1u << K) - 1 ? 0 : 2;
      }
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < kpad * 16; i += blockDim.x) {
    const int c = i >> 4, j = i & 15;
    const double sc = w.lam ? sh[16 + j] : 1.0;
    wl[i] = (c < khat && j < K && sc != 0.0) ? (float)(w.VK[(int64_t)c * K + j] * sc) : 0.f;
  }
  __syncthreads();
}

// U's 16-row tile t = Y W by v_mfma_f32_16x16x4_f32: lane l reads four
// consecutive columns (s + 4*(l/16) .. +3) of row l%16 of the tile; MFMA u
// contracts column s + 4k + u of Y (k = l/16) with row s + 4k + u of W.
// Register r of lane (q, j) is U[4q + r][j].  VEC: khat % 4 == 0 (16-byte loads).
template <bool VEC>
__device__ __forceinline__ floatx4_f uw_tile(const float* __restrict__ Y, int64_t R, int khat, const float* wl,
                                             int64_t t) {
  const int lane = threadIdx.x & 63;
  const int i16 = lane & 15, q = lane >> 4;
  const int kpad = (khat + 15) & ~15;
  const int64_t row = t * 16 + i16;
  const bool rok = row < R;
  const float* yr = Y + row * khat;
  floatx4_f c = {0.f, 0.f, 0.f, 0.f};
  // four 16-column steps per iteration, their loads issued before the first
  // MFMA (the MFMAs keep their order: same U as one step at a time)
  for (int s = 0; s < kpad; s += 64) {
    float y[4][4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int col = s + 16 * d + 4 * q;
      if (VEC) {
        const float4 v = (rok && col < khat) ? *reinterpret_cast<const float4*>(yr + col) : float4{0.f, 0.f, 0.f, 0.f};
        y[d][0] = v.x; y[d][1] = v.y; y[d][2] = v.z; y[d][3] = v.w;
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) y[d][u] = (rok && col + u < khat) ? yr[col + u] : 0.f;
      }
    }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      if (s + 16 * d >= kpad) break;   // the same in every lane
      const int col = s + 16 * d + 4 * q;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(y[d][u], wl[(col + u) * 16 + i16], c, 0, 0, 0);
    }
  }
  return c;
}

// U = Y W on the matrix cores (K <= 16), one 16-row tile per wave at a time;
// bounded by the read of Y.  At most 256 workgroups of 4 to 16 waves, so that
// the step after sums at most 256 partials.  ROWS: U's rows go to dF at their
// slices in FP32 and nothing else is written; else U (FP64) and the
// workgroup's partial U^T U (FP64 MFMA of the same registers).
template <bool VEC, bool ROWS>
__global__ __launch_bounds__(64 * UW_WAVES) void k_uw_mfma(const float* __restrict__ Y, int64_t R, int khat,
                                                           FactorW w, int K, double* __restrict__ U,
                                                           double* __restrict__ part,
                                                           const int32_t* __restrict__ row_slice,
                                                           float* __restrict__ dF) {
  extern __shared__ __align__(16) double shd[];   // UW_SH, then W (or the waves' Grams)
  float* wl = reinterpret_cast<float*>(shd + UW_SH);
  scaled_w(w, khat, K, blockIdx.x == 0, shd, wl);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int waves = blockDim.x >> 6;
  const int i16 = lane & 15, q = lane >> 4;
  doublex4_f g = {0.0, 0.0, 0.0, 0.0};
  const int64_t ntile = (R + 15) >> 4;
  for (int64_t t = (int64_t)blockIdx.x * waves + wave; t < ntile; t += (int64_t)gridDim.x * waves) {
    const floatx4_f c = uw_tile<VEC>(Y, R, khat, wl, t);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t rr = t * 16 + 4 * q + r;
      if (rr < R && i16 < K) {
        if (ROWS)
          dF[(int64_t)row_slice[rr] * K + i16] = c[r];
        else
          U[rr * K + i16] = (double)c[r];
      }
    }
    if (!ROWS)
#pragma unroll
      for (int r = 0; r < 4; ++r) g = __builtin_amdgcn_mfma_f64_16x16x4f64((double)c[r], (double)c[r], g, 0, 0, 0);
  }
  if (!ROWS) {
    __syncthreads();   // every wave has read its last W
    write_gram_part(g, K, shd + UW_SH, part);
  }
}

// flag[0]: this mode's failure bits; flag[1]: 1 + the first failed mode of the invocation
__device__ __forceinline__ void record_flag(int* flag, int n, int bits) {
  flag[FLAG_BITS + n] = bits;
  if (bits && !flag[1]) flag[1] = n + 1;
}

// Where the last product writes the factor: its FP64 master (slice order) and
// its FP32 working copy (storage labels), unless an earlier mode of a deferred
// invocation failed.
struct FactorOut {
  const int32_t* row_slice;
  const int32_t* label;
  double* F64;
  float* F32;
  int kp32;
  int* flag;
  int n;
  int deferred;   // flag[1] skips the writes
  int record;     // this mode's bits are recorded (record_flag)
};

// flag[1] may already be this mode's own (recorded by a faster workgroup)
__device__ __forceinline__ bool skip_writes(const FactorOut& o) {
  if (!o.deferred) return false;
  const int a = o.flag[1];
  return a != 0 && a != o.n + 1;
}

__device__ __forceinline__ void write_factor(const FactorOut& o, int64_t rr, int K, int k, double v) {
  const int64_t l = o.row_slice[rr];
  o.F64[l * K + k] = v;
  o.F32[(int64_t)o.label[l] * o.kp32 + k] = (float)v;
}

// U <- U Rinv on the FP64 matrix cores (K <= 16), 16-row tiles: lane l supplies
// A[i = l%16][k = l/16] = U[row i][4s + k] and B[k][j = l%16] = Rinv[4s + k][j]
// for s = 0..3; v_mfma_f64_16x16x4_f64 returns D[l/16 + 4r][l%16] in register r.
// Not FINAL: write U back and the partial U^T U of the result.  FINAL: write
// the rows straight into the factor.
template <bool FINAL>
__global__ __launch_bounds__(64 * UW_WAVES) void k_rinv_mfma(double* __restrict__ U, int64_t R, int K,
                                                             const double* __restrict__ Rinv,
                                                             double* __restrict__ part, FactorOut o) {
  extern __shared__ __align__(16) double shd[];   // not FINAL: 256 per wave
  if (FINAL) {
    const bool skip = skip_writes(o);
    if (o.record && blockIdx.x == 0 && threadIdx.x == 0) record_flag(o.flag, o.n, o.flag[0]);
    if (skip) return;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int waves = blockDim.x >> 6;
  const int i16 = lane & 15, q = lane >> 4;
  double rb[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = 4 * s + q;
    rb[s] = (k < K && i16 < K) ? Rinv[k * K + i16] : 0.0;
  }
  doublex4_f g = {0.0, 0.0, 0.0, 0.0};
  const int64_t ntile = (R + 15) >> 4;
  for (int64_t t = (int64_t)blockIdx.x * waves + wave; t < ntile; t += (int64_t)gridDim.x * waves) {
    const double* ur = U + min(t * 16 + i16, R - 1) * K;
    doublex4_f c = {0.0, 0.0, 0.0, 0.0};
    double a[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) a[s] = ur[min(4 * s + q, K - 1)];   // all loads at once
#pragma unroll
    for (int s = 0; s < 4; ++s)
      c = __builtin_amdgcn_mfma_f64_16x16x4f64(t * 16 + i16 < R && 4 * s + q < K ? a[s] : 0.0, rb[s], c, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t rr = t * 16 + q + 4 * r;
      if (rr < R && i16 < K) {
        if (FINAL)
          write_factor(o, rr, K, i16, c[r]);
        else
          U[rr * K + i16] = c[r];
      }
    }
    if (!FINAL) {
      // every lane has read its U values above before any lane overwrote them:
      // a tile's rows are read and written by the same wave only
#pragma unroll
      for (int r = 0; r < 4; ++r) g = __builtin_amdgcn_mfma_f64_16x16x4f64(c[r], c[r], g, 0, 0, 0);
    }
  }
  if (!FINAL) write_gram_part(g, K, shd, part);
}

// U <- U Rinv (upper triangular, K x K) and partial U^T U of the result, over
// `tiles` consecutive 64-row tiles per workgroup.
__global__ __launch_bounds__(256) void k_apply_rinv(double* __restrict__ U, int64_t R, int K, int tiles,
                                                    const double* __restrict__ Rinv, double* __restrict__ part) {
  extern __shared__ double shd[];
  double* ri = shd;               // K * K
  double* ut = ri + K * K;        // FT_ROWS * K (old rows)
  double* un = ut + FT_ROWS * K;  // FT_ROWS * K (new rows)
  for (int i = threadIdx.x; i < K * K; i += blockDim.x) ri[i] = Rinv[i];
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int tt = 0; tt < tiles; ++tt) {
    const int64_t r0 = ((int64_t)blockIdx.x * tiles + tt) * FT_ROWS;
    if (r0 >= R) break;
    const int nr = (int)min<int64_t>(FT_ROWS, R - r0);
    __syncthreads();
    for (int i = threadIdx.x; i < nr * K; i += blockDim.x) ut[i] = U[r0 * K + i];
    __syncthreads();
    // new[r][k] = sum_{j <= k} old[r][j] * Rinv[j][k]
    for (int i = threadIdx.x; i < nr * K; i += blockDim.x) {
      const int r = i / K, k = i - r * K;
      double s = 0.0;
      for (int j = 0; j <= k; ++j) s += ut[r * K + j] * ri[j * K + k];
      un[i] = s;
      U[r0 * K + i] = s;
    }
    __syncthreads();
    for (int q = 0; q < 4; ++q) {
      const int i = threadIdx.x + 256 * q;
      if (i < K * K) {
        const int a = i / K, b = i - a * K;
        double s = acc[q];
        for (int r = 0; r < nr; ++r) s += un[r * K + a] * un[r * K + b];
        acc[q] = s;
      }
    }
  }
  for (int q = 0; q < 4; ++q) {
    const int i = threadIdx.x + 256 * q;
    if (i < K * K) part[(int64_t)blockIdx.x * K * K + i] = acc[q];
  }
}

// Fixed-order sum of nparts rows of K*K doubles: one block per entry group.
__global__ __launch_bounds__(256) void k_sum_parts(const double* __restrict__ part, int nparts, int KK,
                                                   double* __restrict__ out) {
  __shared__ double sh[256];
  for (int e = blockIdx.x; e < KK; e += gridDim.x) {
    double s = 0.0;
    for (int p = threadIdx.x; p < nparts; p += blockDim.x) s += part[(int64_t)p * KK + e];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) out[e] = sh[0];
    __syncthreads();
  }
}

// One wavefront: column j = lane of R^-T (z[i] = R^-1[j][i]) for A = R^T R, A
// symmetric K x K in LDS (row stride NP, at least 16), K <= NP.  Lane j keeps
// column j of A and of the identity, both under the factorisation's row
// operations; the other columns' entries come across lanes (rows of 16 lanes
// alike for NP <= 16), so nothing waits on LDS: 5.9 us of kernel at K = 5 and
// 11.8 us at K = 10 with the matrix in LDS, 5.7 us at K = 10 with the partials'
// sum (2.8 to 4.6 us before) in the same launch.
// False when a pivot is not positive relative to the largest diagonal.  A
// column of U zeroed below the rank floor (W = 0, so U's column is exactly 0.0)
// has an exactly zero row and column in A = U^T U, and every earlier step
// leaves them so: R[j][j] = 1 is taken for it, so that U R^-1 keeps it zero and
// the other columns come out orthonormal; it is not a failure (the completion
// adds that direction).
template <int NP>
__device__ __forceinline__ bool chol_rinv(const double* A, int K, double (&z)[NP]) {
  constexpr int LS = NP <= 16 ? 16 : NP;
  int j = threadIdx.x & (LS - 1);
  asm volatile("" : "+v"(j));   // compared here: masks kept over a caller's loop spill
  double x[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) x[i] = (i < K && j < K) ? A[i * LS + j] : 0.0;
  auto entry = [&](auto row, auto col) __attribute__((always_inline)) {
    constexpr int r = decltype(row)::value, c = decltype(col)::value;
    if constexpr (NP <= 16)
      return row_bcast<c>(x[r]);
    else
      return lane_value(x[r], c);
  };
  double dmax = 0.0;
  uint32_t zero = 0;
  static_for<NP>([&](auto ii) __attribute__((always_inline)) {
    constexpr int i = decltype(ii)::value;
    const double d = entry(ii, ii);
    dmax = fmax(dmax, d);   // the padding's zeros change nothing
    zero |= d == 0.0 ? 1u << i : 0u;
    z[i] = j == i ? 1.0 : 0.0;
  });
  bool ok = dmax > 0.0;
  static_for<NP>([&](auto cc) __attribute__((always_inline)) {
    constexpr int c = decltype(cc)::value;
    if (c >= K) return;   // the same in every lane
    const double d = entry(cc, cc);
    const bool none = __ballot(j > c && x[c] != 0.0) == 0;   // row c beyond the diagonal is exactly zero
    const bool zr = ((zero >> c) & 1) && d == 0.0 && none;
    const bool pos = d > 1e-16 * dmax;
    ok = ok && (pos || zr);
    const double dd = pos ? d : 1.0;
    double y = __builtin_amdgcn_rsq(dd);   // 1 / sqrt, refined twice
    double e = fma(-dd * y, y, 1.0);
    y = fma(0.5 * y, e, y);
    e = fma(-dd * y, y, 1.0);
    y = fma(0.5 * y, e, y);
    x[c] *= y;
    z[c] *= y;
    static_for<NP - 1 - c>([&](auto ii) __attribute__((always_inline)) {
      constexpr int i = decltype(ii)::value + c + 1;
      const double r = -entry(cc, std::integral_constant<int, i>{});
      x[i] = fma(r, x[c], x[i]);
      z[i] = fma(r, z[c], z[i]);
    });
  });
  return ok;
}

// Rinv = R^-1 of the Cholesky factor of the sum of nparts K x K blocks (in
// fixed order), in one workgroup; the identity and flag bit 1 when it fails.
// NP = 32: one block only.
template <int NP>
__global__ __launch_bounds__(NP <= 16 ? 1024 : 256) void k_sum_chol(const double* __restrict__ part, int nparts, int K,
                                                                    double* __restrict__ Rinv,
                                                                    int* __restrict__ flag) {
  constexpr int LS = NP <= 16 ? 16 : NP;
  __shared__ double A[LS * LS];
  __shared__ double acc[1024];
  const int E = K * K;
  if (NP <= 16) {
    // a group of threads per share of the blocks, a thread per entry
    const int gs = E <= 64 ? 64 : E <= 128 ? 128 : 256, G = 1024 / gs;
    const int e = threadIdx.x & (gs - 1), g = threadIdx.x / gs;
    double s = 0.0;
    if (e < E)
      for (int p = g; p < nparts; p += 8 * G) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)min(p + u * G, nparts - 1) * E + e];   // loads together
#pragma unroll
        for (int u = 0; u < 8; ++u) s += p + u * G < nparts ? v[u] : 0.0;
      }
    acc[threadIdx.x] = s;
    __syncthreads();
    if ((int)threadIdx.x < E) {
      double t = 0.0;
      for (int h = 0; h < G; ++h) t += acc[h * gs + threadIdx.x];
      A[(threadIdx.x / K) * LS + threadIdx.x % K] = t;
    }
  } else {
    for (int i = threadIdx.x; i < E; i += blockDim.x) A[(i / K) * LS + i % K] = part[i];
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  double z[NP];
  const bool ok = chol_rinv<NP>(A, K, z);
  const int j = threadIdx.x;
  if (!ok && j == 0) flag[0] |= 1;
  if (j < K)
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (i < K) Rinv[j * K + i] = ok ? z[i] : (i == j ? 1.0 : 0.0);
}

// The whole factor step of a mode with few rows (R <= 16 UW_WAVES, K <= 16) in
// one workgroup: U = Y W, both CholeskyQR passes and the factor's rows, with U
// in registers (a 16-row tile per wave) throughout.  Such a step is all
// latency: with ten launches it took 39 us at R = 200, Khat = 25, as one 11 us.
// A tile's product with R^-1 goes through LDS into
// row-major operand order; the row order inside a tile stays that of uw_tile.
template <bool VEC, int NP>
__global__ __launch_bounds__(64 * UW_WAVES) void k_factor_wg(const float* __restrict__ Y, int R, int khat, FactorW w,
                                                             int K, FactorOut o) {
  constexpr int TS = 17;   // row stride of a tile in LDS
  extern __shared__ __align__(16) double shd[];
  double* tiles = shd;                             // a tile per wave; the waves' Grams
  double* gm = tiles + UW_WAVES * 16 * TS;         // 16 x 16
  double* ri = gm + 256;                           // 16 x 16
  double* sh = ri + 256;                           // UW_SH
  float* wl = reinterpret_cast<float*>(sh + UW_SH);
  __shared__ int bad;
  const int lane = threadIdx.x & 63, j = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool skip = skip_writes(o);
  if (threadIdx.x == 0) bad = 0;
  scaled_w(w, khat, K, true, sh, wl);
  const int ntile = (R + 15) >> 4;
  doublex4_f u = {0.0, 0.0, 0.0, 0.0};
  if (wave < ntile) {
    const floatx4_f c = uw_tile<VEC>(Y, R, khat, wl, wave);
#pragma unroll
    for (int r = 0; r < 4; ++r) u[r] = (double)c[r];
  }
  double* mine = tiles + wave * 16 * TS;
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    doublex4_f g = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 4; ++r) g = __builtin_amdgcn_mfma_f64_16x16x4f64(u[r], u[r], g, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) mine[(q + 4 * r) * 16 + j] = g[r];
    __syncthreads();
    if (threadIdx.x < 256) {
      double t = 0.0;
#pragma unroll
      for (int v = 0; v < UW_WAVES; ++v) t += tiles[v * 16 * TS + threadIdx.x];
      gm[threadIdx.x] = t;
    }
    __syncthreads();
    if (wave == 0) {
      double z[NP];
      const bool ok = chol_rinv<NP>(gm, K, z);
      if (!ok && lane == 0) bad = 1;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const double v = i < NP ? z[i < NP ? i : 0] : 0.0;
        ri[j * 16 + i] = j < K && i < K ? (ok ? v : (i == j ? 1.0 : 0.0)) : 0.0;   // the rows of 16 lanes alike
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) mine[(q + 4 * r) * TS + j] = u[r];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    doublex4_f d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      d = __builtin_amdgcn_mfma_f64_16x16x4f64(mine[j * TS + 4 * s + q], ri[(4 * s + q) * 16 + j], d, 0, 0, 0);
    u = d;
    __syncthreads();   // the tiles' places become the Grams' again
  }
  if (threadIdx.x == 0) {
    const int bits = o.flag[0] | bad;   // written by this thread in scaled_w
    o.flag[0] = bits;
    if (o.record) record_flag(o.flag, o.n, bits);
  }
  if (skip) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int rr = 16 * wave + 4 * q + r;
    if (rr < R && j < K) write_factor(o, rr, K, j, u[r]);
  }
}

// W of scaled_w in memory (khat x K), for ranks above 16 and for W too large
// for LDS; the flag's bit is set, not cleared.
__global__ __launch_bounds__(256) void k_make_w(const double* __restrict__ VK, const double* __restrict__ lam,
                                                const double* __restrict__ diag, int64_t dstride, int khat, int K,
                                                double* __restrict__ W, int* __restrict__ flag,
                                                int* __restrict__ kvalid) {
  __shared__ double red[256];
  double t = 0.0;
  for (int i = threadIdx.x; i < khat; i += 256) t += diag[(int64_t)i * dstride];
  red[threadIdx.x] = t;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double floor_ = RANK_FLOOR * red[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {   // eigenvalues come in descending order
    int kv = 0;
    while (kv < K && kv < khat && lam[kv] > floor_ && lam[kv] > 0.0) ++kv;
    *kvalid = kv;
  }
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < khat * K; i += gridDim.x * blockDim.x) {
    const int k = i % K;
    const bool ok = k < khat && lam[k] > floor_ && lam[k] > 0.0;  // only khat eigenpairs exist
    W[i] = ok ? VK[i] / sqrt(lam[k]) : 0.0;
    if (!ok && i < K) atomicOr(flag, 2);
  }
}

// F64[row_slice[r]] = U[r] (index order); the FP32 working copy of the same
// rows at their storage labels.
__global__ void k_scatter_factor(const double* __restrict__ U, int64_t R, int K, const int32_t* __restrict__ row_slice,
                                 const int32_t* __restrict__ label, double* __restrict__ F64, float* __restrict__ F32,
                                 int kp32, const int* __restrict__ abort) {
  if (abort && *abort) return;   // an earlier mode of this invocation failed
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < R * K; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / K;
    const int k = (int)(i - r * K);
    const int64_t l = row_slice[r];
    const int64_t s = label[l];
    const double v = U[i];
    F64[l * K + k] = v;
    F32[s * kp32 + k] = (float)v;
  }
}

// The FP32 working copy of a whole FP64 factor at the storage labels (padding stays zero).
__global__ void k_factor_copies(const double* __restrict__ F64, int64_t L, int K, const int32_t* __restrict__ label,
                                float* __restrict__ F32, int kp32) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < L * K; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t l = i / K;
    const int k = (int)(i - l * K);
    const int64_t s = label[l];
    F32[s * kp32 + k] = (float)F64[i];
  }
}

void refresh_factor_copies(Ctx* c, int n) {
  const int64_t L = c->dims[n];
  const int K = c->K[n];
  TK_HIP(hipMemsetAsync(c->F32[n].get(), 0, c->F32[n].bytes(), c->stream));
  hipLaunchKernelGGL(k_factor_copies, dim3(grid_for(L * K, 256)), dim3(256), 0, c->stream, c->F64[n].as<double>(), L,
                     K, c->plan[n].label.as<int32_t>(), c->F32[n].as<float>(), c->kp32[n]);
  TK_CHECK_LAUNCH();
}

// ---- completion of a rank-deficient factor ----------------------------------------------------
//
// The factor's computed columns are orthonormalised, the ones that vanish are
// dropped, and the missing columns are unit vectors: at the lowest-index empty
// slices when the mode has enough of them (the computed columns are zero on
// those rows), else e_i (lowest i first) made orthogonal to everything before
// them.  The columns are not unique; only their span with the computed ones
// and their orthonormality are fixed.
//
// On the device: two passes of (Gram F^T F, FP64 over the L rows; Gram-Schmidt
// of the columns in coefficient space on the host, K x K; F <- F T in place).
// The unit-vector columns then need only the rows i of F that are tried: a new
// column is Q b + sum_r a_r e_{i_r}, with Q the orthonormal computed columns,
// so its coefficients follow from those rows, F <- F B adds the Q parts, and
// the few tried rows are written from the host.

constexpr int CG_ROWS = 64;   // rows per LDS tile

// part[b] = sum over block b's rows of F[i, :]^T F[i, :]  (K x K, row-major)
__global__ __launch_bounds__(256) void k_gram64_parts(const double* __restrict__ F, int64_t L, int K,
                                                      int64_t rows_per_block, double* __restrict__ part) {
  __shared__ double tile[CG_ROWS * 32];
  const int KK = K * K;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  const int64_t r1 = std::min<int64_t>(L, r0 + rows_per_block);
  for (int64_t t0 = r0; t0 < r1; t0 += CG_ROWS) {
    const int nr = (int)std::min<int64_t>(CG_ROWS, r1 - t0);
    for (int i = threadIdx.x; i < nr * K; i += 256) tile[i] = F[t0 * K + i];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = threadIdx.x + 256 * q;
      if (e < KK) {
        const int a = e / K, b = e - a * K;
        double s = 0.0;
        for (int r = 0; r < nr; ++r) s += tile[r * K + a] * tile[r * K + b];
        acc[q] += s;
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = threadIdx.x + 256 * q;
    if (e < KK) part[(int64_t)blockIdx.x * KK + e] = acc[q];
  }
}

// F[i, :] <- F[i, :] T  (T: K x K row-major), in place
__global__ __launch_bounds__(256) void k_rows_times(double* __restrict__ F, int64_t L, int K,
                                                    const double* __restrict__ T) {
  __shared__ double Ts[32 * 32];
  __shared__ double in[CG_ROWS * 32];
  __shared__ double out[CG_ROWS * 32];
  for (int i = threadIdx.x; i < K * K; i += 256) Ts[i] = T[i];
  for (int64_t t0 = (int64_t)blockIdx.x * CG_ROWS; t0 < L; t0 += (int64_t)gridDim.x * CG_ROWS) {
    const int nr = (int)std::min<int64_t>(CG_ROWS, L - t0);
    __syncthreads();
    for (int i = threadIdx.x; i < nr * K; i += 256) in[i] = F[t0 * K + i];
    __syncthreads();
    for (int o = threadIdx.x; o < nr * K; o += 256) {
      const int r = o / K, b = o - r * K;
      double s = 0.0;
      for (int a = 0; a < K; ++a) s += in[r * K + a] * Ts[a * K + b];
      out[o] = s;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nr * K; i += 256) F[t0 * K + i] = out[i];
  }
}

namespace {

// Gram of F64[n] (K x K, FP64) on the host.
std::vector<double> factor_gram(Ctx* c, int n, double* dev) {
  const int64_t L = c->dims[n];
  const int K = c->K[n];
  const int KK = K * K;
  const int nb = (int)std::max<int64_t>(1, std::min<int64_t>(1024, ceil_div(L, 4096)));
  const int64_t rpb = ceil_div(L, nb);
  double* part = dev + 2 * KK;
  hipLaunchKernelGGL(k_gram64_parts, dim3(nb), dim3(256), 0, c->stream, c->F64[n].as<double>(), L, K, rpb, part);
  TK_CHECK_LAUNCH();
  hipLaunchKernelGGL(k_sum_parts, dim3(std::min(KK, 1024)), dim3(256), 0, c->stream, part, nb, KK, dev);
  TK_CHECK_LAUNCH();
  std::vector<double> A((size_t)KK);
  d2h(c, A.data(), dev, A.size());
  c->sync();
  return A;
}

// Modified Gram-Schmidt, twice per column, of the columns of F in the inner
// product of their Gram A: T's columns 0..g-1 give F T orthonormal columns;
// a column whose remainder is at most 1e-6 of its norm is dropped.
int coeff_gram_schmidt(const std::vector<double>& A, int K, std::vector<double>& T) {
  auto dot = [&](const std::vector<double>& x, const std::vector<double>& y) {
    double s = 0.0;
    for (int a = 0; a < K; ++a) {
      if (x[a] == 0.0) continue;
      double t = 0.0;
      for (int b = 0; b < K; ++b) t += A[(size_t)a * K + b] * y[b];
      s += x[a] * t;
    }
    return s;
  };
  std::vector<std::vector<double>> acc;
  for (int k = 0; k < K; ++k) {
    const double n0 = std::sqrt(std::max(A[(size_t)k * K + k], 0.0));
    if (!(n0 > 0.0)) continue;
    std::vector<double> v((size_t)K, 0.0);
    v[k] = 1.0;
    for (int pass = 0; pass < 2; ++pass)
      for (const auto& u : acc) {
        const double d = dot(u, v);
        for (int a = 0; a < K; ++a) v[a] -= d * u[a];
      }
    const double nv = std::sqrt(std::max(dot(v, v), 0.0));
    if (nv > 1e-6 * n0) {
      for (double& x : v) x /= nv;
      acc.push_back(std::move(v));
    }
  }
  T.assign((size_t)K * K, 0.0);
  for (size_t j = 0; j < acc.size(); ++j)
    for (int a = 0; a < K; ++a) T[(size_t)a * K + j] = acc[j][a];
  return (int)acc.size();
}

void apply_rows_times(Ctx* c, int n, const std::vector<double>& T, double* dev) {
  const int64_t L = c->dims[n];
  const int K = c->K[n];
  h2d(c, dev + K * K, T.data(), T.size());
  hipLaunchKernelGGL(k_rows_times, dim3(grid_for(ceil_div(L, CG_ROWS), 1, 4096)), dim3(256), 0, c->stream,
                     c->F64[n].as<double>(), L, K, dev + K * K);
  TK_CHECK_LAUNCH();
  c->sync();   // T's host copy may go
}

}  // namespace

// ids[t], t < M: the t-th empty slice (ascending) of a mode with nonempty
// slices row_slice[0..R) (ascending).  Before row_slice[r] lie row_slice[r] - r
// empty ids, so the t-th is t + r for the first r with row_slice[r] - r > t
// (r = R when the empty ids past the last nonempty slice are reached).
__global__ void k_find_empty(const int32_t* __restrict__ row_slice, int64_t R, int M, int32_t* __restrict__ ids) {
  const int t = threadIdx.x;
  if (t >= M) return;
  int64_t lo = 0, hi = R;   // first r in [0, R] with row_slice[r] - r > t
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)row_slice[mid] - mid > t) hi = mid; else lo = mid + 1;
  }
  ids[t] = (int32_t)(t + lo);
}

// Column g + t of factor n becomes e_{ids[t]} (its FP64 row and its FP32 copy at
// the row's storage label): the rows were zero, as rows of empty slices are.
__global__ void k_set_units(const int32_t* __restrict__ ids, int M, int g, int K, const int32_t* __restrict__ label,
                            double* __restrict__ F64, float* __restrict__ F32, int kp32) {
  const int t = threadIdx.x;
  if (t >= M) return;
  const int64_t i = ids[t];
  F64[i * K + g + t] = 1.0;
  F32[(int64_t)label[i] * kp32 + g + t] = 1.0f;
}

// Zero the rows ids[0..M) of factor n (FP64 and FP32 copy), unless an earlier
// mode of this invocation failed.
__global__ void k_zero_rows(const int32_t* __restrict__ ids, int M, int K, const int32_t* __restrict__ label,
                            double* __restrict__ F64, float* __restrict__ F32, int kp32, const int* __restrict__ abort) {
  if (abort && *abort) return;
  for (int q = threadIdx.x; q < M * K; q += blockDim.x) {
    const int t = q / K, k = q - t * K;
    const int64_t i = ids[t];
    F64[i * K + k] = 0.0;
    F32[(int64_t)label[i] * kp32 + k] = 0.0f;
  }
}

// Returns true when the missing columns are unit vectors at rows of empty slices.
static bool complete_on_device(Ctx* c, int n, int g_known) {
  const int64_t L = c->dims[n];
  const int K = c->K[n];
  const int KK = K * K;
  TK_REQUIRE(K <= 32, TK_ERR_UNSUPPORTED, "completion: rank above 32");
  ensure(c, c->small64, sizeof(double) * (size_t)KK * (2 + 1024));
  double* dev = c->small64.as<double>();
  // orthonormal computed columns: two passes, unless the factor step already
  // orthonormalised them (its only failure was the rank floor)
  int g = K;
  if (g_known >= 0) {
    g = g_known;
  } else {
    for (int pass = 0; pass < 2; ++pass) {
      const std::vector<double> A = factor_gram(c, n, dev);
      std::vector<double> T;
      g = coeff_gram_schmidt(A, K, T);
      apply_rows_times(c, n, T, dev);
    }
  }
  if (g == K) {
    refresh_factor_copies(c, n);
    c->sync();
    return false;
  }
  // a mode with enough empty slices: the computed columns vanish on those rows,
  // so unit vectors there are already orthogonal to them and to each other
  const ModePlan& pl = c->plan[n];
  const int M = K - g;
  if (L - pl.L_nz >= M) {
    ensure(c, c->unit_rows[n], sizeof(int32_t) * 32);
    int32_t* ids = c->unit_rows[n].as<int32_t>();
    hipLaunchKernelGGL(k_find_empty, dim3(1), dim3(32), 0, c->stream, pl.row_slice.as<int32_t>(), pl.L_nz, M, ids);
    TK_CHECK_LAUNCH();
    if (g_known < 0) refresh_factor_copies(c, n);   // the passes above rewrote F64
    hipLaunchKernelGGL(k_set_units, dim3(1), dim3(32), 0, c->stream, ids, M, g, K, pl.label.as<int32_t>(),
                       c->F64[n].as<double>(), c->F32[n].as<float>(), c->kp32[n]);
    TK_CHECK_LAUNCH();
    c->n_unit_rows[n] = M;
    c->sync();
    return true;
  }
  // unit vectors e_i, lowest i first.  A column is (b, a): Q b + sum_r a[r] e_{cand[r]}.
  struct Col {
    std::vector<double> b, a;
  };
  std::vector<int64_t> cand;            // tried rows, in order
  std::vector<std::vector<double>> qrow; // Q[cand[r], 0..g-1]
  std::vector<Col> added;
  auto inner = [&](const Col& x, const Col& y) {
    double s = 0.0;
    for (int j = 0; j < g; ++j) s += x.b[j] * y.b[j];
    for (size_t r = 0; r < cand.size(); ++r) {
      double qx = 0.0, qy = 0.0;
      for (int j = 0; j < g; ++j) {
        qx += qrow[r][j] * x.b[j];
        qy += qrow[r][j] * y.b[j];
      }
      s += y.a[r] * qx + x.a[r] * qy + x.a[r] * y.a[r];
    }
    return s;
  };
  std::vector<double> rows_h;
  int64_t rows_at = 0, rows_n = 0;
  for (int64_t i = 0; g + (int)added.size() < K; ++i) {
    TK_REQUIRE(i < L, TK_ERR_NUMERIC, "completion: unit vectors exhausted");
    if (i >= rows_at + rows_n) {   // read the next rows of Q
      rows_at = i;
      rows_n = std::min<int64_t>(256, L - i);
      rows_h.resize((size_t)rows_n * K);
      d2h(c, rows_h.data(), c->F64[n].as<double>() + i * K, rows_h.size());
      c->sync();
    }
    cand.push_back(i);
    qrow.emplace_back(rows_h.begin() + (i - rows_at) * K, rows_h.begin() + (i - rows_at) * K + g);
    for (auto& col : added) col.a.push_back(0.0);
    Col v{std::vector<double>((size_t)g), std::vector<double>(cand.size(), 0.0)};
    v.a.back() = 1.0;
    for (int pass = 0; pass < 2; ++pass) {
      // against Q's columns: <Q e_j, v> = v.b[j] + sum_r v.a[r] Q[cand[r], j]
      std::vector<double> d((size_t)g, 0.0);
      for (int j = 0; j < g; ++j) {
        double t = v.b[j];
        for (size_t r = 0; r < cand.size(); ++r) t += v.a[r] * qrow[r][j];
        d[j] = t;
      }
      for (int j = 0; j < g; ++j) v.b[j] -= d[j];
      for (const auto& u : added) {
        const double t = inner(u, v);
        for (int j = 0; j < g; ++j) v.b[j] -= t * u.b[j];
        for (size_t r = 0; r < cand.size(); ++r) v.a[r] -= t * u.a[r];
      }
    }
    const double nv = std::sqrt(std::max(inner(v, v), 0.0));
    if (nv > 0.5) {
      for (double& x : v.b) x /= nv;
      for (double& x : v.a) x /= nv;
      added.push_back(std::move(v));
    }
  }
  // F <- F B: column j < g stays, column g + t = Q b_t (columns g.. of F are zero)
  std::vector<double> B((size_t)KK, 0.0);
  for (int j = 0; j < g; ++j) B[(size_t)j * K + j] = 1.0;
  for (size_t t = 0; t < added.size(); ++t)
    for (int j = 0; j < g; ++j) B[(size_t)j * K + g + t] = added[t].b[j];
  apply_rows_times(c, n, B, dev);
  // the tried rows: Q[i] B + the unit-vector parts
  std::vector<double> patch(cand.size() * (size_t)K);
  for (size_t r = 0; r < cand.size(); ++r) {
    double* row = patch.data() + r * K;
    for (int j = 0; j < g; ++j) row[j] = qrow[r][j];
    for (size_t t = 0; t < added.size(); ++t) {
      double s = added[t].a[r];
      for (int j = 0; j < g; ++j) s += qrow[r][j] * added[t].b[j];
      row[g + t] = s;
    }
  }
  // the tried rows are 0 .. cand.size()-1, contiguous
  h2d(c, c->F64[n].as<double>(), patch.data(), patch.size());
  refresh_factor_copies(c, n);
  c->sync();
  return false;
}

void complete_factor(Ctx* c, int n, int g);
int computed_columns(Ctx* c, const int* flag_dev, int n);

namespace {

// Waves per workgroup for ntile 16-row tiles: at most 256 workgroups (one per
// CU), their waves as even as can be.
int uw_waves(int64_t ntile) { return (int)std::min<int64_t>(UW_WAVES, std::max<int64_t>(4, ceil_div(ntile, 256))); }
int uw_groups(int64_t ntile) { return (int)std::min<int64_t>(256, ceil_div(ntile, uw_waves(ntile))); }
size_t uw_lds(int khat, int waves) {
  return sizeof(double) * UW_SH + std::max(sizeof(float) * 16 * (size_t)((khat + 15) & ~15),
                                           sizeof(double) * 256 * (size_t)waves);
}

}  // namespace

// dF[row_slice[r]] = Y[r] W (FP32) for K <= 16 on the matrix cores, W khat x K
// in FP64 (rounded to FP32 for the MFMA operands).
void uw_rows(Ctx* c, const float* Y, int64_t R, int khat, const double* W, int K, const int32_t* row_slice, float* dF) {
  TK_REQUIRE(K <= 16, TK_ERR_UNSUPPORTED, "Y W on the matrix cores: K above 16");
  const int64_t ntile = std::max<int64_t>(1, ceil_div(R, 16));
  const int waves = uw_waves(ntile);
  const size_t lds = uw_lds(khat, waves);
  // (2 KB of room asked for beside W, as for the Grams of four waves)
  TK_REQUIRE(sizeof(float) * 16 * (size_t)((khat + 15) & ~15) + 2048 <= c->lds_per_block && lds <= c->lds_per_block,
             TK_ERR_UNSUPPORTED, "Y W: Khat too large for LDS");
  const FactorW w{W, nullptr, nullptr, 0, nullptr, nullptr};
  const dim3 g(uw_groups(ntile)), t(64 * waves);
  if (khat % 4 == 0)
    hipLaunchKernelGGL((k_uw_mfma<true, true>), g, t, lds, c->stream, Y, R, khat, w, K, nullptr, nullptr, row_slice,
                       dF);
  else
    hipLaunchKernelGGL((k_uw_mfma<false, true>), g, t, lds, c->stream, Y, R, khat, w, K, nullptr, nullptr, row_slice,
                       dF);
  TK_CHECK_LAUNCH();
}

// zero a buffer (2-byte units) unless an earlier mode of this invocation failed
__global__ void k_clear_unless(uint16_t* __restrict__ p, int64_t n16, const int* __restrict__ abort) {
  if (*abort) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

__global__ void k_flag_record(int* flag, int n) { record_flag(flag, n, flag[0]); }

// New factor n from Y (R x khat) and the leading eigenpairs (lam_k, VK).
// Returns true when the completion path ran.
// deferred = false: the failure check reads flag_dev[0] on the host and
// completes the factor at once.
// deferred = true (a Gauss-Seidel invocation that checks once at its end):
// flag_dev[1] = 1 + the first failed mode of the invocation, or 0.  Once it is
// set, this call leaves factor n as it was (the caller runs the mode again
// after completing the failed factor); a failure of this mode sets it when
// R >= K, and is completed at once when R < K.
bool form_factor(Ctx* c, int n, const float* Y, int64_t R, int khat, const double* gdiag, int64_t dstride,
                 const double* lam_k, const double* VK, int* flag_dev, bool deferred) {
  const int* abort = deferred ? flag_dev + 1 : nullptr;
  const bool check_flag = !deferred || R < c->K[n];
  const int K = c->K[n];
  TK_REQUIRE(K <= 32, TK_ERR_UNSUPPORTED, "factor step: rank above 32");
  const bool mfma = K <= 16;
  const int64_t ntile = std::max<int64_t>(1, ceil_div(R, mfma ? 16 : FT_ROWS));
  const int tiles = (int)std::max<int64_t>(1, ceil_div(ntile, 1024));
  const int waves = uw_waves(ntile);
  const int nwg = mfma ? uw_groups(ntile) : (int)ceil_div(ntile, tiles);
  ensure(c, c->U64, sizeof(double) * (size_t)std::max<int64_t>(R, 1) * K);
  ensure(c, c->small64, sizeof(double) * ((size_t)khat * K + 3 * (size_t)K * K + (size_t)nwg * K * K));
  double* W = c->small64.as<double>();
  double* Rinv = W + (size_t)khat * K;
  double* Asum = Rinv + (size_t)K * K;
  double* part = Asum + (size_t)K * K;
  double* U = c->U64.as<double>();
  const ModePlan& pl = c->plan[n];
  const FactorW fw{VK, lam_k, gdiag, dstride, flag_dev, flag_dev + FLAG_KVALID + n};
  const FactorOut fo{pl.row_slice.as<int32_t>(), pl.label.as<int32_t>(), c->F64[n].as<double>(),
                     c->F32[n].as<float>(), c->kp32[n], flag_dev, n, deferred, !check_flag};
  // W in LDS: its kernels form it and set the flag themselves
  const bool w_lds = mfma && R > 0 && uw_lds(khat, waves) <= c->lds_per_block;
  if (!w_lds) {
    TK_HIP(hipMemsetAsync(flag_dev, 0, sizeof(int), c->stream));
    hipLaunchKernelGGL(k_make_w, dim3(grid_for((int64_t)khat * K, 256, 64)), dim3(256), 0, c->stream, VK, lam_k,
                       gdiag, dstride, khat, K, W, flag_dev, flag_dev + FLAG_KVALID + n);
    TK_CHECK_LAUNCH();
  }
  // rows of empty slices (never written below) must be zero: clear the copies
  // only when something else may have written them (tk_set_factor, completion)
  auto clear_factor = [&]() {
    if (!c->fac_dirty[n] && c->n_unit_rows[n] > 0) {
      const int M = c->n_unit_rows[n];
      hipLaunchKernelGGL(k_zero_rows, dim3(1), dim3(256), 0, c->stream, c->unit_rows[n].as<int32_t>(), M, K,
                         pl.label.as<int32_t>(), c->F64[n].as<double>(), c->F32[n].as<float>(), c->kp32[n], abort);
      TK_CHECK_LAUNCH();
      c->n_unit_rows[n] = 0;
      return;
    }
    if (!c->fac_dirty[n]) return;
    c->n_unit_rows[n] = 0;
    if (abort) {
      // deferred check: a later pass may have to keep this factor as it was;
      // the clear then does not happen, and the driver marks the factor dirty
      // again before that pass
      for (Buf* b : {&c->F64[n], &c->F32[n]}) {
        const int64_t n16 = (int64_t)(b->bytes() / 2);
        hipLaunchKernelGGL(k_clear_unless, dim3(grid_for(n16, 256, 4096)), dim3(256), 0, c->stream,
                           b->as<uint16_t>(), n16, abort);
        TK_CHECK_LAUNCH();
      }
    } else {
      TK_HIP(hipMemsetAsync(c->F64[n].get(), 0, c->F64[n].bytes(), c->stream));
      TK_HIP(hipMemsetAsync(c->F32[n].get(), 0, c->F32[n].bytes(), c->stream));
    }
    c->fac_dirty[n] = false;
  };
  auto reduce_chol = [&]() {
    if (K <= 8) {
      hipLaunchKernelGGL(k_sum_chol<8>, dim3(1), dim3(1024), 0, c->stream, part, nwg, K, Rinv, flag_dev);
    } else if (K <= 16) {
      hipLaunchKernelGGL(k_sum_chol<16>, dim3(1), dim3(1024), 0, c->stream, part, nwg, K, Rinv, flag_dev);
    } else {
      hipLaunchKernelGGL(k_sum_parts, dim3(std::min(K * K, 1024)), dim3(256), 0, c->stream, part, nwg, K * K, Asum);
      TK_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_sum_chol<32>, dim3(1), dim3(256), 0, c->stream, Asum, 1, K, Rinv, flag_dev);
    }
    TK_CHECK_LAUNCH();
  };
  const bool vec = khat % 4 == 0;
  const size_t wg_lds = sizeof(double) * (UW_WAVES * 16 * 17 + 512 + UW_SH) +
                        sizeof(float) * 16 * (size_t)((khat + 15) & ~15);
  // One workgroup for the whole step up to a tile per wave and 2^15 entries of
  // Y: 20 us at R = 256, Khat = 128, the five launches 28.  At R = 997,
  // Khat = 100 (four tiles per wave) one workgroup took 43 us, they 28.
  bool recorded = false;
  if (w_lds && R <= 16 * UW_WAVES && R * khat <= (1 << 15) && wg_lds <= c->lds_per_block) {
    clear_factor();
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(1), dim3(64 * UW_WAVES), wg_lds, c->stream, Y, (int)R, khat, fw, K, fo);
    };
    if (K <= 8)
      vec ? go(k_factor_wg<true, 8>) : go(k_factor_wg<false, 8>);
    else
      vec ? go(k_factor_wg<true, 16>) : go(k_factor_wg<false, 16>);
    TK_CHECK_LAUNCH();
    recorded = true;
  } else if (R > 0 && mfma) {
    const dim3 g(nwg), t(64 * waves);
    if (w_lds) {
      const size_t lds = uw_lds(khat, waves);
      if (vec)
        hipLaunchKernelGGL((k_uw_mfma<true, false>), g, t, lds, c->stream, Y, R, khat, fw, K, U, part, nullptr,
                           nullptr);
      else
        hipLaunchKernelGGL((k_uw_mfma<false, false>), g, t, lds, c->stream, Y, R, khat, fw, K, U, part, nullptr,
                           nullptr);
      TK_CHECK_LAUNCH();
    } else {
      // W too large for LDS: U = Y W as a tall-skinny FP64 product, then the
      // workgroups' row ranges of U^T U
      tall_times_small(c, Y, R, khat, W, K, U);
      hipLaunchKernelGGL(k_gram64_parts, dim3(nwg), dim3(256), 0, c->stream, U, R, K, ceil_div(R, nwg), part);
      TK_CHECK_LAUNCH();
    }
    reduce_chol();
    const size_t lds = sizeof(double) * 256 * (size_t)waves;
    hipLaunchKernelGGL(k_rinv_mfma<false>, g, t, lds, c->stream, U, R, K, Rinv, part, fo);
    TK_CHECK_LAUNCH();
    reduce_chol();
    clear_factor();
    hipLaunchKernelGGL(k_rinv_mfma<true>, g, t, 0, c->stream, U, R, K, Rinv, part, fo);
    TK_CHECK_LAUNCH();
    recorded = true;
  } else if (R > 0) {
    size_t lds = sizeof(double) * ((size_t)khat * K + FT_ROWS * K) + sizeof(float) * FT_ROWS * (size_t)(khat + 1);
    if (lds <= c->lds_per_block) {
      hipLaunchKernelGGL(k_uw, dim3(nwg), dim3(256), lds, c->stream, Y, R, khat, W, K, tiles, U, part);
      TK_CHECK_LAUNCH();
    } else {
      // W too large for LDS: U = Y W as a tall-skinny product, then the
      // workgroups' row ranges of U^T U
      tall_times_small(c, Y, R, khat, W, K, U);
      hipLaunchKernelGGL(k_gram64_parts, dim3(nwg), dim3(256), 0, c->stream, U, R, K, ceil_div(R, nwg), part);
      TK_CHECK_LAUNCH();
    }
    for (int pass = 0; pass < 2; ++pass) {
      reduce_chol();
      hipLaunchKernelGGL(k_apply_rinv, dim3(nwg), dim3(256), sizeof(double) * ((size_t)K * K + 2 * FT_ROWS * K),
                         c->stream, U, R, K, tiles, Rinv, part);
      TK_CHECK_LAUNCH();
    }
    clear_factor();
    hipLaunchKernelGGL(k_scatter_factor, dim3(grid_for(R * K, 256)), dim3(256), 0, c->stream, U, R, K,
                       pl.row_slice.as<int32_t>(), pl.label.as<int32_t>(), c->F64[n].as<double>(),
                       c->F32[n].as<float>(), c->kp32[n], abort);
    TK_CHECK_LAUNCH();
  } else {
    clear_factor();
  }
  if (!check_flag) {
    if (!recorded) {
      hipLaunchKernelGGL(k_flag_record, dim3(1), dim3(1), 0, c->stream, flag_dev, n);
      TK_CHECK_LAUNCH();
    }
    return false;
  }
  int hflag[2] = {0, 0};
  d2h(c, hflag, flag_dev, deferred ? 2 : 1);
  c->sync();
  if (hflag[1]) return false;   // an earlier mode failed: this mode runs again later
  if (hflag[0] || R < K) {
    if (!c->opt.complete_rank_deficient) fail(TK_ERR_NUMERIC, "rank-deficient penultimate matrix");
    complete_factor(c, n, hflag[0] == 2 && R >= K ? computed_columns(c, flag_dev, n) : -1);
    return true;
  }
  return false;
}

// Columns of factor n above the rank floor, as its factor step recorded them.
int computed_columns(Ctx* c, const int* flag_dev, int n) {
  int kv = 0;
  d2h(c, &kv, flag_dev + FLAG_KVALID + n, 1);
  c->sync();
  return kv;
}

// Complete factor n (rank-deficient penultimate matrix) on the host.
// g >= 0: the factor step failed only on the rank floor, so columns 0..g-1
// are already orthonormal and the rest exactly zero.
void complete_factor(Ctx* c, int n, int g) {
  ++c->counters.rank_completions;
  c->completed_once = true;
  // the unit-vector rows of empty slices are zeroed by the next factor step
  // (only those rows after a completion by k_set_units, all of them otherwise)
  if (!complete_on_device(c, n, g)) c->fac_dirty[n] = true;
}

}  // namespace tk
