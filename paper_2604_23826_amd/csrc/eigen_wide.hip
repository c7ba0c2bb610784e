// Finalize of more columns than one workgroup takes (24 of a correlation matrix,
// 60 of a covariance matrix) over the whole GPU: covariance, correlation and
// eigenpairs, as a sequence of launches on the handle's
// stream (finalize.hip has the one-workgroup form and the conventions).
//
// Correlation matrix (unit diagonal, so errors small against its norm are all
// that counts):
//   1. Householder reduction to tridiagonal form T.  Above 128 rows one launch
//      per column (k_house): the pending rank-two update of the last column,
//      the next column, its reflector and the product A v in a single pass over
//      the trailing rows, one wave per row; what the whole matrix needs of the
//      last product (v . p) is formed again by every workgroup, so a step is one
//      launch and no grid-wide wait.  The last 128 rows are reduced by one
//      workgroup from registers (k_tri_tail).
//   2. Eigenvalues of T by multisection: a wave per eigenvalue, a point per
//      lane, sign changes of the leading minors' recurrence (k_bisect).
//   3. Eigenvectors of T by two steps of inverse iteration from random starts,
//      a lane per eigenvector (k_invit); vectors of eigenvalues closer than
//      1e-6 ||T|| are orthogonalised within their cluster (k_orth).
//   4. Reflectors applied back, a wave per vector (k_back).
//   5. One refinement step (Ogita and Aishima, "Iterative refinement for
//      symmetric eigenvalue decomposition", 2018) with products on the FP64
//      matrix cores: R = I - V^T V and S = V^T A V correct V to
//      orthogonality and eigenvector accuracy of a few ulps (over the gap) and give
//      the eigenvalues as Rayleigh quotients.  It is also the check: a correction
//      above 1e-7, or a coupling between close eigenvalues above 10 q u ||T|| (u =
//      2^-53), rejects the result, and QL in one workgroup takes matrices of up to
//      60 columns, the Jacobi method below the others.
// Covariance matrix (may be graded): the cyclic Jacobi method, one kernel pair
// per round, until a sweep rotates nothing.  It was the only method before:
// 256 x 256 takes 2550 rounds of two launches, 27 ms.
#include <algorithm>

#include "accum_common.hpp"
#include "eigen.hpp"

namespace st {
namespace {

constexpr int kThreads = 1024;  // rotations of a Jacobi round
constexpr int kJThreads = 256;  // the other kernels
constexpr int kTail = 128;      // rows reduced by one workgroup
constexpr double kEps = 2.220446049250313e-16;
constexpr double kCluster = 1e-6;  // gap, of ||T||, below which vectors are orthogonalised together
constexpr double kNear = 1e-7;     // gap below which the refinement leaves a pair's mixture alone
constexpr double kAccept = 1e-7;   // largest correction of a refinement that squares it away
// Largest cluster that k_orth takes: one workgroup orthogonalises it vector by vector.
// Clusters of 256 take it 69 ms of 512 columns and 134 of 1024, where a whole call by
// Jacobi takes 113 and 322; of 512 columns' 511 205 ms against 65, of 1024's 1023
// 2456 against 208.  Nor does it take all but one of the vectors, as of an identity or an
// equicorrelation matrix, which the fallback decomposes in a step or two (256 columns:
// 36 ms against 1.9 and 10.8; of collinear columns 35 against 27).
constexpr int kMaxCluster = 256;
static_assert(kMaxCluster <= kJThreads, "a thread per gap in k_orth");

// Words of FinalizeLaunch::jc.
enum { J_ROT = 0, J_NONE = 1, J_LEFT = 2, J_REJECT = 3 };
enum : unsigned { NONE_NAN = 1u, NONE_N = 2u };  // J_NONE: non-finite input; n <= ddof

// ---- covariance, correlation ---------------------------------------------------

__global__ __launch_bounds__(kJThreads) void k_cov(const uint64_t* st, int p, const int32_t* sel, int q,
                                                   const uint8_t* intf, int ddof, const DevStatus* status, double* out,
                                                   unsigned* jc) {
  const Layout L = Layout::make(p);
  const int64_t n = (int64_t)st[0];
  const int first = blockIdx.x * kJThreads + threadIdx.x;
  if (first == 0) {
    double* tail = out + 4 * q + 3 * (int64_t)q * q;  // N and the status word
    tail[0] = __longlong_as_double(n);
    tail[1] = __longlong_as_double((long long)status->bits);
    tail[2] = __longlong_as_double((long long)status->parse_off);
    jc[J_ROT] = jc[J_LEFT] = jc[J_REJECT] = 0;
    jc[J_NONE] = n <= ddof ? NONE_N : 0;
  }
  if (n <= ddof) return;  // nothing is defined (the host reports it)
  double* mean = out;
  double* cov = out + q;
  const double dn = (double)(n - ddof);
  for (int idx = first; idx < q * q; idx += gridDim.x * kJThreads) {
    const int a = idx / q, b = idx % q;
    if (a > b) continue;
    const int i = sel[a], j = sel[b];  // sel ascending, so i <= j
    if (a == b)
      mean[a] = intf[i] ? exact_mean(st, L, i, n) : __longlong_as_double((long long)st[L.off_mu + i]);
    double v;
    if (intf[i] && intf[j]) v = exact_cov(st, L, i, j, n, ddof);
    else v = __longlong_as_double((long long)st[L.off_M2 + tri(p, i, j)]) / dn;
    cov[a * q + b] = v;
    cov[b * q + a] = v;
  }
}

// Correlation, and the working copy A of the matrix to decompose.
__global__ __launch_bounds__(kJThreads) void k_corr(double* out, int q, int pca_on, double* A, unsigned* jc) {
  if (jc[J_NONE] & NONE_N) return;
  const double* cov = out + q;
  double* corr = out + q + q * q;
  bool bad = false;
  for (int idx = blockIdx.x * kJThreads + threadIdx.x; idx < q * q; idx += gridDim.x * kJThreads) {
    const int a = idx / q, b = idx % q;
    const double caa = cov[a * q + a], cbb = cov[b * q + b];
    double v;
    if (caa == 0.0 || cbb == 0.0) v = __builtin_nan("");
    else if (a == b) v = 1.0;
    else v = cov[idx] / sqrt(caa * cbb);
    corr[idx] = v;
    const double x = pca_on ? cov[idx] : v;
    A[idx] = x;
    bad |= !isfinite(x);
  }
  if (bad) atomicOr(&jc[J_NONE], NONE_NAN);
}

// ---- 1: tridiagonal form --------------------------------------------------------

// Sum over the wave, in every lane.
__device__ inline double wave_sum(double v) { return lane_value(acc::wave_sum_to_lane63(v), 63); }

// Sum over the workgroup's kN waves, in every thread; buf: kN words of LDS.
template <int kN>
__device__ inline double block_sum(double v, double* buf) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) buf[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kN; ++w) t += buf[w];
  return t;
}

// Column k.  Before it, A's rows >= k hold everything but the update of column
// k - 1, whose reflector is row k - 1 of H (factor beta[k - 1]) and whose
// product is p_in; after it, rows > k hold that update and p_out = beta A v of
// column k's reflector, row k of H.  NL = ceil(q / 64) values per lane.
template <int NL>
__global__ __launch_bounds__(kJThreads) void k_house(double* __restrict__ A, int q, int k, double* __restrict__ H,
                                                     double* __restrict__ beta, double* __restrict__ d,
                                                     double* __restrict__ e, const double* __restrict__ p_in,
                                                     double* __restrict__ p_out) {
  __shared__ double sv[64 * NL], sw[64 * NL], sx[64 * NL], buf[3][kJThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int row = k + 1 + blockIdx.x * (kJThreads / 64) + (tid >> 6);
  double a[NL];  // this wave's row, loaded ahead of the reductions
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    const int j = lane + 64 * u;
    a[u] = row < q && j > k && j < q ? A[(int64_t)row * q + j] : 0.0;
  }
  constexpr int NT = (64 * NL + kJThreads - 1) / kJThreads;
  double v[NT], p[NT], x[NT];
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int j = tid + kJThreads * u;
    const bool on = j >= k && j < q;
    v[u] = on && k > 0 ? H[(int64_t)(k - 1) * q + j] : 0.0;
    p[u] = on && k > 0 ? p_in[j] : 0.0;
    x[u] = on ? A[(int64_t)k * q + j] : 0.0;
    s = __builtin_fma(v[u], p[u], s);
  }
  const double h = k > 0 ? 0.5 * beta[k - 1] * block_sum<kJThreads / 64>(s, buf[0]) : 0.0;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int j = tid + kJThreads * u;
    if (j < 64 * NL) {
      sv[j] = v[u];
      sw[j] = __builtin_fma(-h, v[u], p[u]);
    }
  }
  __syncthreads();
  const double vk = sv[k], wk = sw[k];
  double t = 0.0;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int j = tid + kJThreads * u;
    if (j < 64 * NL) {
      x[u] -= __builtin_fma(vk, sw[j], wk * sv[j]);
      sx[j] = x[u];
      if (j > k + 1) t = __builtin_fma(x[u], x[u], t);
    }
  }
  const double tail = block_sum<kJThreads / 64>(t, buf[1]);  // its barrier also publishes sx
  const double x0 = sx[k + 1];
  double v0 = 0.0, bk = 0.0, ek = x0;
  if (tail >= 1e-280) {
    const double n2 = __builtin_fma(x0, x0, tail), norm = n2 * rsqrt_f64(n2);
    v0 = x0 >= 0.0 ? x0 + norm : x0 - norm;
    bk = 1.0 / (norm * (norm + fabs(x0)));
    ek = x0 >= 0.0 ? -norm : norm;
  }
  auto refl = [&](int j) { return bk == 0.0 || j <= k ? 0.0 : (j == k + 1 ? v0 : sx[j]); };
  if (blockIdx.x == 0) {
    for (int j = tid; j < q; j += kJThreads) H[(int64_t)k * q + j] = refl(j);
    if (tid == 0) {
      beta[k] = bk;
      e[k] = ek;
      d[k] = sx[k];
    }
  }
  if (row < q) {
    const double vi = sv[row], wi = sw[row];
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int j = lane + 64 * u;
      if (j > k && j < q) {
        a[u] -= __builtin_fma(vi, sw[j], wi * sv[j]);
        A[(int64_t)row * q + j] = a[u];
        acc = __builtin_fma(a[u], refl(j), acc);
      }
    }
    acc = wave_sum(acc);
    if (lane == 0) p_out[row] = bk * acc;
  }
}

// Sum over the 16 lanes of a row of the wave, in every lane of it.
__device__ inline double row16_sum(double v) {
  v += acc::dpp_f64<0xB1, 0xF>(v);
  v += acc::dpp_f64<0x4E, 0xF>(v);
  v += acc::dpp_f64<0x124, 0xF>(v);
  return v + acc::dpp_f64<0x128, 0xF>(v);
}

// Rows o..q-1 (m <= 128 of them) in one workgroup, with the update of column
// o - 1 pending as for k_house.  Thread (r, c) of 32 x 16 holds the 4 x 8 tile of
// rows r + 32 u and columns c + 16 w in registers, so a step reads 24 words of
// the exchanged vectors from LDS for its 32 elements (a row per quad, as in
// tri_reduce, reads 64 and is bound by that: 464 us for 128 rows).  Two
// barriers a step.
constexpr int kTailThreads = 512;
__global__ __launch_bounds__(kTailThreads) void k_tri_tail(const double* __restrict__ A, int q, int o, double* H,
                                                           double* beta, double* d, double* e, const double* p_in,
                                                           const unsigned* jc) {
  if (jc[J_NONE]) return;
  __shared__ double sv[kTail], sw[kTail], s_x[2][kTail], s_p[2][kTail], buf[kTailThreads / 64];
  const int tid = threadIdx.x, r = tid >> 4, c = tid & 15, m = q - o;
  {
    double v = 0.0, p = 0.0;
    if (o > 0 && tid < m) {
      v = H[(int64_t)(o - 1) * q + o + tid];
      p = p_in[o + tid];
    }
    const double h = o > 0 ? 0.5 * beta[o - 1] * block_sum<kTailThreads / 64>(v * p, buf) : 0.0;
    if (tid < kTail) {
      sv[tid] = v;
      sw[tid] = __builtin_fma(-h, v, p);
    }
  }
  __syncthreads();
  double a[4][8];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const int i = r + 32 * u, j = c + 16 * w;
      a[u][w] = i < m && j < m ? A[(int64_t)(o + i) * q + o + j] - __builtin_fma(sv[i], sw[j], sw[i] * sv[j]) : 0.0;
    }
  for (int k = 0; k + 1 < m; ++k) {
    double *x = s_x[k & 1], *p = s_p[k & 1];
    if (r == (k & 31)) {  // row k to LDS
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (u == k >> 5) {
#pragma unroll
          for (int w = 0; w < 8; ++w) x[c + 16 * w] = a[u][w];
        }
    }
    __syncthreads();
    const double x0 = x[k + 1];
    if (tid == 0) d[o + k] = x[k];
    if (k + 2 == m) {
      if (tid == 0) e[o + k] = x0;
      break;
    }
    double v[8], vi[4], tail = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const int j = c + 16 * w;
      v[w] = j > k + 1 ? x[j] : 0.0;
      tail = __builtin_fma(v[w], v[w], tail);
    }
    tail = row16_sum(tail);
    const bool none = tail < 1e-280;  // already tridiagonal here
    const double n2 = __builtin_fma(x0, x0, tail), norm = n2 * rsqrt_f64(none ? 1.0 : n2);
    const double v0 = none ? 0.0 : (x0 >= 0.0 ? x0 + norm : x0 - norm);
    const double bk = none ? 0.0 : 1.0 / (norm * (norm + fabs(x0)));
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const int j = c + 16 * w;
      v[w] = none ? 0.0 : (j == k + 1 ? v0 : v[w]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = r + 32 * u;
      vi[u] = none || i <= k ? 0.0 : (i == k + 1 ? v0 : x[i]);
    }
    double s[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      s[u] = 0.0;
#pragma unroll
      for (int w = 0; w < 8; ++w) s[u] = __builtin_fma(a[u][w], v[w], s[u]);
      s[u] = r + 32 * u > k ? bk * row16_sum(s[u]) : 0.0;
      if (c == 0) p[r + 32 * u] = s[u];
    }
    if (tid < m) H[(int64_t)(o + k) * q + o + tid] = none || tid <= k ? 0.0 : (tid == k + 1 ? v0 : x[tid]);
    if (tid == 0) {
      beta[o + k] = bk;
      e[o + k] = none ? x0 : (x0 >= 0.0 ? -norm : norm);
    }
    __syncthreads();
    double pj[8], h = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      pj[w] = p[c + 16 * w];
      h = __builtin_fma(pj[w], v[w], h);
    }
    h = 0.5 * bk * row16_sum(h);
#pragma unroll
    for (int w = 0; w < 8; ++w) pj[w] = __builtin_fma(-h, v[w], pj[w]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double wi = __builtin_fma(-h, vi[u], s[u]);
#pragma unroll
      for (int w = 0; w < 8; ++w) a[u][w] -= __builtin_fma(vi[u], pj[w], wi * v[w]);
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 8; ++w)
      if (r + 32 * u == m - 1 && c + 16 * w == m - 1) d[q - 1] = a[u][w];
  if (tid == 0) e[q - 1] = 0.0;
  // the reflectors are zero before their own columns (rows o.. of H, columns < o)
  for (int i = tid; i < (m > 2 ? m - 2 : 0) * o; i += kTailThreads) H[(int64_t)(o + i / o) * q + i % o] = 0.0;
}

// ---- 2: eigenvalues of T --------------------------------------------------------

// Gershgorin bounds of T and their larger magnitude (at least 1e-300).
struct Bounds {
  double lo, hi, scale;
};
__device__ inline Bounds bounds_of(const double* d, const double* e, int q, double (*buf)[kJThreads / 64]) {
  double lo = __builtin_inf(), hi = -__builtin_inf();
  for (int i = threadIdx.x; i < q; i += kJThreads) {
    const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < q ? fabs(e[i]) : 0.0);
    lo = fmin(lo, d[i] - r);
    hi = fmax(hi, d[i] + r);
  }
  for (int s = 32; s > 0; s >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, s, 64));
    hi = fmax(hi, __shfl_xor(hi, s, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    buf[0][threadIdx.x >> 6] = lo;
    buf[1][threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  for (int w = 0; w < kJThreads / 64; ++w) {
    lo = fmin(lo, buf[0][w]);
    hi = fmax(hi, buf[1][w]);
  }
  return Bounds{lo, hi, fmax(fmax(fabs(lo), fabs(hi)), 1e-300)};
}

// Eigenvalue k (ascending) of T per wave, to about 2^-53 of the bounds: the
// interval shrinks 65-fold per pass.  lam[q] and, from workgroup 0, scale.
__global__ __launch_bounds__(kJThreads) void k_bisect(const double* __restrict__ d, const double* __restrict__ e,
                                                      int q, double* lam, double* scale, const unsigned* jc) {
  if (jc[J_NONE]) return;
  extern __shared__ double2 s_t[];  // d / scale, (e / scale)^2 of the coupling before it
  __shared__ double buf[2][kJThreads / 64];
  const Bounds B = bounds_of(d, e, q, buf);
  const double inv = 1.0 / B.scale;
  if (blockIdx.x == 0 && threadIdx.x == 0) *scale = B.scale;
  const int qp = (q + 7) & ~7;  // padded with rows that change no sign
  for (int i = threadIdx.x; i < qp; i += kJThreads) {
    const double c = i > 0 && i < q ? e[i - 1] * inv : 0.0;
    // a floor far below rounding keeps two minors in a row from vanishing
    s_t[i] = make_double2(i < q ? d[i] * inv : 4.0, i < q ? fmax(c * c, 1e-34) : 0.0);
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int k = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kJThreads / 64) + (threadIdx.x >> 6)));
  if (k >= q) return;
  double lo = B.lo * inv - 4e-16, hi = B.hi * inv + 4e-16;
  for (int pass = 0; pass < 9; ++pass) {
    const double x = __builtin_fma((hi - lo) * (1.0 / 65.0), (double)(lane + 1), lo);
    double pm = 0.0, pc = 1.0;
    int below = 0;  // eigenvalues below x
    for (int i = 0; i < qp; i += 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double2 t = s_t[i + u];
        const double pn = __builtin_fma(t.x - x, pc, -(t.y * pm));
        below += (uint32_t)(__double2hiint(pn) ^ __double2hiint(pc)) >> 31;
        pm = pc;
        pc = pn;
      }
      const int ex = -max(__builtin_amdgcn_frexp_exp(pm), __builtin_amdgcn_frexp_exp(pc));
      pm = ldexp(pm, ex);
      pc = ldexp(pc, ex);
    }
    // points with at most k eigenvalues below them are left of eigenvalue k
    const uint64_t left = __builtin_amdgcn_ballot_w64(below <= k);
    const int nl = ~left ? __builtin_ctzll(~left) : 64;
    const double xl = nl > 0 ? lane_value(x, nl - 1) : lo, xr = nl < 64 ? lane_value(x, nl & 63) : hi;
    lo = xl;
    hi = xr;
  }
  if (lane == 0) lam[k] = 0.5 * (lo + hi) * B.scale;
}

// ---- 3: eigenvectors of T -------------------------------------------------------

__device__ inline double start_value(uint32_t i, uint32_t col) {  // in [-1, 1), from an integer hash
  // multipliers: fractional bits of the square roots of 2, 3, 5 and 7, made odd
  uint32_t h = i * 0x6A09E667u ^ (col + 1u) * 0xBB67AE85u;
  h ^= h >> 15;
  h *= 0x3C6EF373u;
  h ^= h >> 12;
  h *= 0xA54FF53Bu;
  h ^= h >> 15;
  return (double)(int32_t)h * 0x1p-31;
}

// LU factors of T - lam I with partial pivoting, element (i, col) at i q + col:
// reciprocal pivots, two superdiagonals, multipliers, row exchanges.
struct Lu {
  double *u0, *u1, *u2, *l;
  uint8_t* sw;
};

constexpr int kBatch = 16;  // steps of a substitution whose operands are loaded together

// One step of inverse iteration for eigenvector col per lane: x := (T - lam)^-1 x.
// FIRST factors T - lam I and starts from random x (for which the forward
// substitution changes nothing).  A step grows x by 1/eps at most where pivots
// vanish once, so two steps need no scaling in between (k_back normalises; a
// result that overflowed all the same is rejected by k_correct).
template <bool FIRST>
__global__ __launch_bounds__(64) void k_invit(const double* __restrict__ d, const double* __restrict__ e, int q,
                                              const double* __restrict__ lam, const double* __restrict__ scale, Lu f,
                                              double* __restrict__ X, const unsigned* jc) {
  if (jc[J_NONE]) return;
  const int col = blockIdx.x * 64 + threadIdx.x;
  extern __shared__ double2 s_t[];  // d, e of T, two zero rows behind (FIRST)
  if constexpr (FIRST) {
    for (int i = threadIdx.x; i < q + 2; i += 64) s_t[i] = i < q ? make_double2(d[i], e[i]) : make_double2(0.0, 0.0);
    __syncthreads();
  }
  if (col >= q) return;
  if constexpr (FIRST) {
    const double w = lam[col], tiny = kEps * *scale;
    double a = s_t[0].x - w, b = s_t[0].y;  // the row being eliminated: (a, b) at (i, i + 1)
    for (int i = 0; i < q; ++i) {
      const double2 t1 = s_t[i + 1];
      const double na = s_t[i].y, nb = i + 1 < q ? t1.x - w : 0.0, nc = t1.y;
      const bool s = fabs(na) > fabs(a);
      double piv = s ? na : a;
      if (!(fabs(piv) >= tiny)) piv = copysign(tiny, piv);
      const double r = 1.0 / piv, m = (s ? a : na) * r;
      const int64_t o = (int64_t)i * q + col;
      f.u0[o] = r;
      f.u1[o] = s ? nb : b;
      f.u2[o] = s ? nc : 0.0;
      f.l[o] = m;
      f.sw[o] = s;
      a = s ? __builtin_fma(-m, nb, b) : __builtin_fma(-m, b, nb);
      b = s ? -m * nc : nc;
    }
  } else {
    double c = X[col];
    for (int i0 = 0; i0 + 1 < q; i0 += kBatch) {
      double nx[kBatch], l[kBatch];
      uint8_t sw[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int64_t o = (int64_t)min(i0 + u, q - 2) * q + col;
        nx[u] = X[o + q];
        l[u] = f.l[o];
        sw[u] = f.sw[o];
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        if (i0 + u + 1 >= q) break;
        const double top = sw[u] ? nx[u] : c, bot = sw[u] ? c : nx[u];
        X[(int64_t)(i0 + u) * q + col] = top;
        c = __builtin_fma(-l[u], top, bot);
      }
    }
    X[(int64_t)(q - 1) * q + col] = c;
  }
  double x1 = 0.0, x2 = 0.0;
  for (int i0 = q - 1; i0 >= 0; i0 -= kBatch) {
    double u0[kBatch], u1[kBatch], u2[kBatch], b[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = max(i0 - u, 0);
      const int64_t o = (int64_t)i * q + col;
      u0[u] = f.u0[o];
      u1[u] = f.u1[o];
      u2[u] = f.u2[o];
      b[u] = FIRST ? start_value(i, col) : X[o];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (i0 - u < 0) break;
      const double x = (b[u] - __builtin_fma(u1[u], x1, u2[u] * x2)) * u0[u];
      X[(int64_t)(i0 - u) * q + col] = x;
      x2 = x1;
      x1 = x;
    }
  }
}

// Classical Gram-Schmidt, twice, within the cluster that starts at eigenvalue
// blockIdx.x, if one does; a result with a cluster too large for it is rejected.
__global__ __launch_bounds__(kJThreads) void k_orth(const double* __restrict__ lam, const double* __restrict__ scale,
                                                    int q, double* X, unsigned* jc) {
  if (jc[J_NONE]) return;
  const double tol = kCluster * *scale;
  const int s = blockIdx.x;
  if (!(s + 1 < q && lam[s + 1] - lam[s] <= tol) || (s > 0 && lam[s] - lam[s - 1] <= tol)) return;
  {
    const int most = min(kMaxCluster, q - 2), t = threadIdx.x;
    if (__syncthreads_and(s + most < q && (t >= most || lam[s + t + 1] - lam[s + t] <= tol))) {
      if (t == 0) atomicOr(&jc[J_REJECT], 1u);
      return;
    }
  }
  extern __shared__ double s_x[];  // the vector, then its products with the earlier ones
  double* s_c = s_x + q;
  __shared__ double buf[2][kJThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = s; i < q && (i == s || lam[i] - lam[i - 1] <= tol); ++i) {
    for (int t = tid; t < q; t += kJThreads) s_x[t] = X[(int64_t)t * q + i];
    __syncthreads();
    for (int rep = 0; rep < 2; ++rep) {
      // a wave per product while they are few, else a thread per product
      const bool few = i - s <= 16;
      for (int j = s + wave; few && j < i; j += kJThreads / 64) {
        double c = 0.0;
        for (int t = lane; t < q; t += 64) c = __builtin_fma(X[(int64_t)t * q + j], s_x[t], c);
        c = wave_sum(c);
        if (lane == 0) s_c[j] = c;
      }
      for (int j = s + tid; !few && j < i; j += kJThreads) {
        double c = 0.0;
#pragma unroll 8
        for (int t = 0; t < q; ++t) c = __builtin_fma(X[(int64_t)t * q + j], s_x[t], c);
        s_c[j] = c;
      }
      __syncthreads();
      for (int t = wave; t < q; t += kJThreads / 64) {
        double c = 0.0;
        for (int j = s + lane; j < i; j += 64) c = __builtin_fma(X[(int64_t)t * q + j], s_c[j], c);
        c = wave_sum(c);
        if (lane == 0) s_x[t] -= c;
      }
      __syncthreads();
      double n2 = 0.0;
      for (int t = tid; t < q; t += kJThreads) n2 = __builtin_fma(s_x[t], s_x[t], n2);
      const double g = 1.0 / sqrt(block_sum<kJThreads / 64>(n2, buf[rep]));
      for (int t = tid; t < q; t += kJThreads) s_x[t] *= g;
      __syncthreads();
    }
    for (int t = tid; t < q; t += kJThreads) X[(int64_t)t * q + i] = s_x[t];
    __syncthreads();  // visible to the products with the next vector
  }
}

// ---- 4: eigenvectors of A, of unit length, one per row of Vt -------------------------------------

template <int NL>
__global__ __launch_bounds__(64) void k_back(const double* __restrict__ X, const double* __restrict__ H,
                                             const double* __restrict__ beta, int q, double* __restrict__ Vt,
                                             const unsigned* jc) {
  if (jc[J_NONE]) return;
  const int col = blockIdx.x, lane = threadIdx.x;
  double x[NL];
  double n2 = 0.0;
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    x[u] = lane + 64 * u < q ? X[(int64_t)(lane + 64 * u) * q + col] : 0.0;
    n2 = __builtin_fma(x[u], x[u], n2);
  }
  const double g = 1.0 / sqrt(wave_sum(n2));
#pragma unroll
  for (int u = 0; u < NL; ++u) x[u] *= g;
  constexpr int kAhead = 8;  // reflectors in flight
  double v[kAhead][NL], b[kAhead];
  auto fetch = [&](int k, int s) {
    const int kk = max(k, 0);
    b[s] = beta[kk];
#pragma unroll
    for (int u = 0; u < NL; ++u) v[s][u] = lane + 64 * u < q ? H[(int64_t)kk * q + lane + 64 * u] : 0.0;
  };
#pragma unroll
  for (int s = 0; s < kAhead; ++s) fetch(q - 3 - s, s);
  for (int k0 = q - 3; k0 >= 0; k0 -= kAhead) {
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {
      if (k0 - s < 0) break;
      double t = 0.0;
#pragma unroll
      for (int u = 0; u < NL; ++u) t = __builtin_fma(v[s][u], x[u], t);
      t = wave_sum(t) * b[s];
#pragma unroll
      for (int u = 0; u < NL; ++u) x[u] = __builtin_fma(-t, v[s][u], x[u]);
      fetch(k0 - s - kAhead, s);
    }
  }
#pragma unroll
  for (int u = 0; u < NL; ++u)
    if (lane + 64 * u < q) Vt[(int64_t)col * q + lane + 64 * u] = x[u];
}

// ---- 5: refinement ----------------------------------------------------------------

// C = A B (+ D), q x q: element (i, k) of A at a + i ai + k ak, (k, j) of B at
// b + k bk + j bj, C and D row-major.  A wave per 16 x 16 tile of C.
struct Gemm {
  const double *a, *b, *d;
  double* c;
  int64_t ai, ak, bk, bj;
};
typedef double d4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kJThreads) void k_gemm(Gemm g0, Gemm g1, int q) {
  const Gemm g = blockIdx.z ? g1 : g0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i0 = 32 * blockIdx.y + 16 * (wave >> 1), j0 = 32 * blockIdx.x + 16 * (wave & 1);
  const int i = i0 + (lane & 15), j = j0 + (lane & 15), kq = lane >> 4;
  const bool iv = i < q, jv = j < q;
  const double* pa = g.a + (iv ? i : 0) * g.ai + kq * g.ak;
  const double* pb = g.b + (jv ? j : 0) * g.bj + kq * g.bk;
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int k = 0; k < q; k += 32) {
    double x[8], y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int kk = k + 4 * u;
      const bool on = kk + kq < q;
      x[u] = on && iv ? pa[kk * g.ak] : 0.0;
      y[u] = on && jv ? pb[kk * g.bk] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u], y[u], acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int ci = i0 + 4 * r + kq;  // register r of lane l: element (4 r + l / 16, l % 16)
    if (ci < q && jv) g.c[(int64_t)ci * q + j] = acc[r] + (g.d ? g.d[(int64_t)ci * q + j] : 0.0);
  }
}

// Corrections E (x_j += sum_i E_ij x_i) from P = V^T V and S = V^T A V, both
// symmetrised so that E_ij + E_ji = (I - P)_ij exactly; refined eigenvalues.
__global__ __launch_bounds__(kJThreads) void k_correct(const double* __restrict__ P, const double* __restrict__ S,
                                                       int q, const double* __restrict__ scale, double* __restrict__ E,
                                                       double* __restrict__ lam, unsigned* jc) {
  bool ok = true;
  const double near = kNear * *scale, noise = 5.0 * q * kEps * *scale;
  for (int idx = blockIdx.x * kJThreads + threadIdx.x; idx < q * q; idx += gridDim.x * kJThreads) {
    const int i = idx / q, j = idx % q;
    const double r = (i == j ? 1.0 : 0.0) - 0.5 * (P[idx] + P[j * q + i]);
    const double s = 0.5 * (S[idx] + S[j * q + i]);
    const double li = S[i * q + i] / P[i * q + i], lj = S[j * q + j] / P[j * q + j];
    double x = 0.5 * r;
    if (i == j) {
      lam[i] = li;
    } else if (fabs(lj - li) > near) {
      x = __builtin_fma(lj, r, s) / (lj - li);
    } else {
      ok = ok && fabs(__builtin_fma(lj, r, s)) <= noise;
    }
    E[idx] = x;
    ok = ok && fabs(x) <= kAccept;  // false for NaN
  }
  if (!ok) atomicOr(&jc[J_REJECT], 1u);
}

// ---- outputs -----------------------------------------------------------------------

// A wave per eigenpair k: its rank (descending, ties by index), sign (entry of
// largest magnitude positive, lowest index on ties, see kTie), eigenvalue and vector.
// Eigenvalue j at lam + j ls, component j of vector k at V + j vj + k vk.
__global__ __launch_bounds__(kJThreads) void k_pairs(const double* __restrict__ lam, int ls,
                                                     const double* __restrict__ V, int64_t vj, int64_t vk, int q,
                                                     int want_vectors, double* out, const unsigned* jc) {
  if (jc[J_NONE] & NONE_N) return;
  const int k = blockIdx.x * (kJThreads / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (k >= q) return;
  double* ev = out + q + 2 * (int64_t)q * q;
  double* evec = ev + q;
  if (jc[J_NONE]) {
    for (int j = lane; j < q; j += 64) evec[(int64_t)k * q + j] = __builtin_nan("");
    if (lane == 0) ev[k] = __builtin_nan("");
    return;
  }
  const double lk = lam[(int64_t)k * ls];
  int rank = 0;
  double best = 0.0;
  for (int j = lane; j < q; j += 64) {
    const double lj = lam[(int64_t)j * ls];
    rank += (lj > lk) || (lj == lk && j < k);
    best = fmax(best, fabs(V[j * vj + k * vk]));
  }
  for (int d = 32; d > 0; d >>= 1) {
    rank += __shfl_xor(rank, d, 64);
    best = fmax(best, __shfl_xor(best, d, 64));
  }
  const double tie = kTie * best;
  int first = 2 * q;  // lowest tied index, doubled, odd where its entry is negative
  for (int j = lane; j < q; j += 64) {
    const double x = V[j * vj + k * vk];
    if (fabs(x) >= tie) first = min(first, 2 * j + (x < 0.0));
  }
  for (int d = 32; d > 0; d >>= 1) first = min(first, __shfl_xor(first, d, 64));
  if (lane == 0) ev[rank] = lk;
  if (want_vectors) {
    for (int j = lane; j < q; j += 64) {
      double x = V[j * vj + k * vk];
      if (fabs(x) >= tie) x = copysign(best, x);
      evec[(int64_t)rank * q + j] = first & 1 ? -x : x;
    }
  }
}

// Variance and cumulative percentages of the sorted eigenvalues.
__global__ __launch_bounds__(kThreads) void k_percent(double* out, int q, const unsigned* jc) {
  if (jc[J_NONE] & NONE_N) return;
  extern __shared__ double s_l[];  // eigenvalues, percentages
  double* s_v = s_l + q;
  const double* ev = out + q + 2 * (int64_t)q * q;
  double* varp = out + 2 * q + 3 * (int64_t)q * q;
  double* cump = varp + q;
  for (int k = threadIdx.x; k < q; k += kThreads) s_l[k] = ev[k];
  __syncthreads();
  double tot = 0.0;
  for (int k = 0; k < q; ++k) tot += s_l[k];
  for (int k = threadIdx.x; k < q; k += kThreads) varp[k] = s_v[k] = 100.0 * s_l[k] / tot;
  __syncthreads();
  for (int k = threadIdx.x; k < q; k += kThreads) {
    double run = 0.0;
    for (int j = 0; j <= k; ++j) run += s_v[j];
    cump[k] = run;
  }
}

// ---- Jacobi, one kernel pair per round ----------------------------------------------

// V = I, and A = src unless src is null.
__global__ __launch_bounds__(kJThreads) void k_jinit(const double* src, double* A, double* V, int q) {
  for (int idx = blockIdx.x * kJThreads + threadIdx.x; idx < q * q; idx += gridDim.x * kJThreads) {
    if (src) A[idx] = src[idx];
    V[idx] = idx / q == idx % q ? 1.0 : 0.0;
  }
}

// A and V in global memory; one round is
// k_jrot (one workgroup: the round's rotation tables, and the count of
// rotations) followed by k_japply (the 2x2 blocks of A and the rows of V,
// spread over many workgroups).  Same arithmetic as the one-workgroup loop.
__global__ __launch_bounds__(kThreads) void k_jrot(const double* __restrict__ A, int q, int m, int r,
                                                   double* tab, unsigned* jc) {
  const int npairs = m / 2;
  const RotTab R = RotTab::at(tab, npairs);
  unsigned cnt = 0;
  for (int k = threadIdx.x; k < npairs; k += blockDim.x) {
    int a, b;
    rr_pair(k, r, m, a, b);
    double c = 1.0, s = 0.0, t = 0.0, apq = 0.0;
    if (!jc[J_NONE] && b < q && jacobi_rotation(A, q, a, b, c, s, t, apq)) ++cnt;
    R.c[k] = c;
    R.s[k] = s;
    R.t[k] = t;
    R.apq[k] = apq;
    R.pair[k] = make_int2(a, b);
  }
  if (cnt) atomicAdd(&jc[J_ROT], cnt);
}

// End of a sweep: count (into jc[J_LEFT]) the pairs that would still rotate; none
// means the next sweep would change nothing.
__global__ __launch_bounds__(kJThreads) void k_jcheck(const double* __restrict__ A, int q, unsigned* jc) {
  const int64_t n = (int64_t)q * q;
  unsigned any = 0;
  for (int64_t idx = (int64_t)blockIdx.x * kJThreads + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * kJThreads) {
    const int i = (int)(idx / q), j = (int)(idx % q);
    if (i < j && rotates(A[idx], A[(int64_t)i * q + i], A[(int64_t)j * q + j])) any = 1;
  }
  if (any) atomicOr(&jc[J_LEFT], 1u);
}

__global__ __launch_bounds__(kJThreads) void k_japply(double* A, double* V, int q, int m, const double* tab) {
  const int npairs = m / 2;
  extern __shared__ double s_tab[];  // the round's tables, copied once
  for (int i = threadIdx.x; i < 5 * npairs; i += kJThreads) s_tab[i] = tab[i];
  __syncthreads();
  const RotTab R = RotTab::at(s_tab, npairs);
  const int start = blockIdx.x * kJThreads + threadIdx.x, stride = gridDim.x * kJThreads;
  jacobi_blocks(A, q, npairs, R, start, stride);
  jacobi_vectors(V, q, npairs, R, start, stride);
}

}  // namespace

int64_t finalize_scratch_words(int q) {
  if (q <= kQlQ) return 0;  // one workgroup, in LDS
  const int64_t qq = (int64_t)q * q;
  // A, V (rows of eigenvectors or Jacobi's V), H, X, four LU arrays, row
  // exchanges, vectors (d, e, beta, lam, two products, rotation tables), flags
  return 8 * qq + (qq + 7) / 8 + 8 * (int64_t)q + 5 * (((int64_t)q + 1) / 2) + 8;
}

hipError_t launch_finalize_wide(const FinalizeLaunch& F, hipStream_t s) {
  const int q = F.q;
  const int64_t qq = (int64_t)q * q;
  double* A = F.scratch;
  double* V = A + qq;
  double* H = V + qq;
  double* X = H + qq;
  Lu lu{X + qq, X + 2 * qq, X + 3 * qq, X + 4 * qq, (uint8_t*)(X + 5 * qq)};
  double* d = X + 5 * qq + (qq + 7) / 8;
  double *e = d + q, *beta = e + q, *lam = beta + q, *p0 = lam + q, *p1 = p0 + q, *scale = p1 + q, *jtab = scale + q;
  const int m = q + (q & 1), npairs = m / 2;
  unsigned* jc = (unsigned*)(jtab + 5 * npairs);
  int dev = 0, ncu = 256;
  hipError_t err = hipGetDevice(&dev);
  if (err == hipSuccess) err = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (err != hipSuccess) return err;
  const dim3 grid((unsigned)std::min<int64_t>((qq + kJThreads - 1) / kJThreads, 4 * ncu)), block(kJThreads);
  hipLaunchKernelGGL(k_cov, grid, block, 0, s, F.state, F.p, F.sel_dev, q, F.intflags_dev, F.ddof, F.status, F.out, jc);
  hipLaunchKernelGGL(k_corr, grid, block, 0, s, F.out, q, F.pca_on, A, jc);
  unsigned w[4] = {0, 0, 0, 0};
  bool done = false;
  if (!F.pca_on) {
    const double* C = F.out + q + qq;  // the correlation matrix
    auto by_width = [&](auto go) {
      if (q <= 128) go(std::integral_constant<int, 2>{});
      else if (q <= 256) go(std::integral_constant<int, 4>{});
      else if (q <= 512) go(std::integral_constant<int, 8>{});
      else go(std::integral_constant<int, 16>{});
    };
    const int o = std::max(0, q - kTail);
    by_width([&](auto nl) {
      for (int k = 0; k < o; ++k)
        hipLaunchKernelGGL(k_house<decltype(nl)::value>, dim3((q - k - 1 + 3) / 4), block, 0, s, A, q, k, H, beta, d, e,
                           k & 1 ? p1 : p0, k & 1 ? p0 : p1);
    });
    hipLaunchKernelGGL(k_tri_tail, dim3(1), dim3(kTailThreads), 0, s, A, q, o, H, beta, d, e, o & 1 ? p1 : p0, jc);
    const size_t sh_t = sizeof(double2) * (size_t)((q + 7) & ~7), sh_2 = 2 * sizeof(double) * (size_t)q;
    hipLaunchKernelGGL(k_bisect, dim3((q + 3) / 4), block, sh_t, s, d, e, q, lam, scale, jc);
    hipLaunchKernelGGL(k_invit<true>, dim3((q + 63) / 64), dim3(64), sizeof(double2) * (size_t)(q + 2), s, d, e, q, lam, scale, lu, X, jc);
    hipLaunchKernelGGL(k_orth, dim3(q), block, sh_2, s, lam, scale, q, X, jc);
    hipLaunchKernelGGL(k_invit<false>, dim3((q + 63) / 64), dim3(64), 0, s, d, e, q, lam, scale, lu, X, jc);
    hipLaunchKernelGGL(k_orth, dim3(q), block, sh_2, s, lam, scale, q, X, jc);
    by_width([&](auto nl) {
      hipLaunchKernelGGL(k_back<decltype(nl)::value>, dim3(q), dim3(64), 0, s, X, H, beta, q, V, jc);
    });
    // W = V A and P = V V^T, S = W V^T, E, V' = V + E^T V (rows of V: vectors)
    double *W = lu.u0, *P = lu.u1, *S = lu.u2, *E = lu.l;
    const unsigned nt = (unsigned)((q + 31) / 32);
    const Gemm gw{V, C, nullptr, W, q, 1, q, 1}, gp{V, V, nullptr, P, q, 1, 1, q}, gs{W, V, nullptr, S, q, 1, 1, q},
        gv{E, V, V, X, 1, q, q, 1};
    hipLaunchKernelGGL(k_gemm, dim3(nt, nt, 2), block, 0, s, gw, gp, q);
    hipLaunchKernelGGL(k_gemm, dim3(nt, nt, 1), block, 0, s, gs, gs, q);
    hipLaunchKernelGGL(k_correct, grid, block, 0, s, P, S, q, scale, E, lam, jc);
    hipLaunchKernelGGL(k_gemm, dim3(nt, nt, 1), block, 0, s, gv, gv, q);
    err = hipGetLastError();
    if (err == hipSuccess) err = hipMemcpyAsync(w, jc, sizeof w, hipMemcpyDeviceToHost, s);
    if (err == hipSuccess) err = hipStreamSynchronize(s);
    if (err != hipSuccess) return err;
    done = w[J_NONE] || !w[J_REJECT];
    if (!done && q <= kLdsQ) return launch_finalize_ql(F, s);
  }
  if (!done) {
    hipLaunchKernelGGL(k_jinit, grid, block, 0, s, F.pca_on ? nullptr : F.out + q + qq, A, V, q);
    const int64_t work = (int64_t)npairs * npairs + (int64_t)q * npairs;
    const int nwg = (int)std::max<int64_t>(1, std::min<int64_t>((work + kJThreads * kNB - 1) / (kJThreads * kNB), 4 * ncu));
    const size_t tab_shm = (size_t)npairs * 5 * sizeof(double);
    for (int sweep = 0; sweep < kMaxSweeps && err == hipSuccess; ++sweep) {
      err = hipMemsetAsync(jc + J_ROT, 0, sizeof(unsigned), s);
      for (int r = 0; r < m - 1 && err == hipSuccess; ++r) {
        hipLaunchKernelGGL(k_jrot, dim3(1), dim3(kThreads), 0, s, A, q, m, r, jtab, jc);
        hipLaunchKernelGGL(k_japply, dim3(nwg), block, tab_shm, s, A, V, q, m, jtab);
        err = hipGetLastError();
      }
      // stop when this sweep rotated nothing, or when nothing would rotate in
      // the next one (same result, one sweep earlier)
      if (err == hipSuccess) err = hipMemsetAsync(jc + J_LEFT, 0, sizeof(unsigned), s);
      if (err == hipSuccess) {
        hipLaunchKernelGGL(k_jcheck, dim3(nwg), block, 0, s, A, q, jc);
        err = hipGetLastError();
      }
      if (err == hipSuccess) err = hipMemcpyAsync(w, jc, sizeof w, hipMemcpyDeviceToHost, s);
      if (err == hipSuccess) err = hipStreamSynchronize(s);
      if (err != hipSuccess || w[J_ROT] == 0 || w[J_LEFT] == 0) break;
    }
    if (err != hipSuccess) return err;
  }
  const dim3 gk((unsigned)((q + 3) / 4));
  if (done) hipLaunchKernelGGL(k_pairs, gk, block, 0, s, lam, 1, X, (int64_t)1, (int64_t)q, q, F.want_vectors, F.out, jc);
  else hipLaunchKernelGGL(k_pairs, gk, block, 0, s, A, q + 1, V, (int64_t)q, (int64_t)1, q, F.want_vectors, F.out, jc);
  hipLaunchKernelGGL(k_percent, dim3(1), dim3(kThreads), 2 * sizeof(double) * (size_t)q, s, F.out, q, jc);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  return hipMemcpyAsync(F.host, F.out, (size_t)(4 * q + 3 * qq + 3) * sizeof(double), hipMemcpyDeviceToHost, s);
}

}  // namespace st
