// Means, covariance, correlation and PCA from the statistics alone.
//
// Section "Data Representation and Sufficient Statistics": once (N, s, X^T X)
// are known, means, covariance and correlation follow without the rows.
// Section "Numerical Considerations": the identifier column is excluded
// (column selection) and the covariance is never formed as X^T X - N mu mu^T
// in floating point: integer pairs use the exact numerator
// N C_ij - s_i s_j (256-bit) divided once with correct rounding, other pairs
// the merged centred co-moment M2 / (N - ddof).
// Section "Principal Component Analysis Results": eigenpairs of the (small,
// dense) correlation or covariance matrix in FP64.  Output as in
// Table 3: eigenvalues descending, variance %, cumulative %, loadings (one
// row per component).
//
// One workgroup does the whole job with the matrices in LDS: a correlation matrix
// of 3 to kQlQ columns by Householder reduction and implicit QL (see below), a
// smaller one, or a covariance matrix of up to kLdsQ columns, by the cyclic Jacobi
// method with the round-robin (Brent-Luk) ordering, in every round of which q/2
// disjoint rotations are computed and applied in parallel.  eigen_wide.hip takes
// the rest.
#include "common.hpp"
#include "eigen.hpp"

namespace st {
namespace {

struct Args {
  const uint64_t* state;
  int p;
  const int32_t* sel;
  int q;
  const uint8_t* intf;
  int ddof;
  int pca_on;
  int want_vectors;
  double* out;
  const DevStatus* status;
  double* host;
};

// The method: Householder and QL for a correlation matrix, Jacobi for a
// covariance matrix.  A template parameter, so that a launch fetches only the
// code it runs (kQlLarge: the matrices above kQlQ that eigen_wide.hip hands back).
enum { kQl = 0, kLdsJacobi = 1, kQlLarge = 2 };
// Correlation matrices of at most this many columns take Jacobi: their equal
// diagonal makes its one rotation exact, so both entries of either vector are equal
// at any correlation (QL, whose shift is rounded, left them 1e-8 apart at 1e-8).
constexpr int kOneRotation = 2;

// End of a sweep (after its last barrier): true when no pair would rotate,
// i.e. the next sweep would change nothing, so stopping now gives the same
// result one sweep earlier.  *cnt is workgroup-shared scratch (reset here).
__device__ inline bool converged(const double* A, int q, int tid, int nth, int* cnt) {
  if (tid == 0) *cnt = 0;
  __syncthreads();
  int any = 0;
  for (int idx = tid; idx < q * q; idx += nth) {
    const int i = idx / q, j = idx % q;
    if (i < j && rotates(A[idx], A[i * q + i], A[j * q + j])) any = 1;
  }
  if (any) atomicOr(cnt, 1);
  __syncthreads();
  return *cnt == 0;
}

// ---- correlation matrices up to kQlQ columns: Householder + implicit QL --------
//
// A correlation matrix has a unit diagonal, so a solver whose errors are small
// against its norm loses nothing on its small eigenvalues that Jacobi would
// keep (a covariance matrix may be graded, and stays with Jacobi).  The matrix
// is reduced to tridiagonal form in LDS, the reflectors are multiplied out,
// and implicit QL runs on one wave: every lane carries the scalar recurrence
// (d and e live one element per lane and are read by index across lanes), and
// lane r applies each rotation to component r of the two eigenvectors.  What
// bounds it is the chain of one rotation (about 1.2 q^2 of them), one
// reciprocal square root and a dozen dependent FMAs (360 cycles in all), where a
// Jacobi round (about 5 q of them) is three divisions, three square roots and
// two barriers.  Whole kernel with the refinement below (3 and 4 us),
// 9 x 9: 89 -> 39 us; 15 x 15: 168 -> 76 us.
constexpr int kQlThreads = 256;

// Tridiagonal form of the symmetric matrix M (q x q, global or LDS) and the
// orthogonal factor, transposed, in Zt (column j of it at Zt + j ld).  d[q],
// e[q] (e[k] couples k and k + 1) and, as scratch, H (q x ld reflectors), beta[q]
// and xp[256] in LDS.  See tri_reduce for the threads' shares; here quad i then
// holds column i of the factor.
template <int C, bool kWave>
__device__ inline void tridiagonalize(const double* M, double* Zt, double* H, int ld, int q, double* d, double* e,
                                      double* beta, double* xp, int tid) {
  const int row = tid >> 2, sub = tid & 3;
  double a[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int j = sub + 4 * c;
    a[c] = row < q && j < q ? M[row * q + j] : 0.0;
  }
  tri_reduce<C, kWave, 64>(a, H, ld, q, d, e, beta, xp, tid);
  group_sync<kWave>();
  // H_0 H_1 ... from the last reflector on
  double z[C];
#pragma unroll
  for (int c = 0; c < C; ++c) z[c] = sub + 4 * c == row ? 1.0 : 0.0;
  for (int k = q - 3; k >= 0; --k) {
    double v[C];
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = sub + 4 * c < q ? H[k * ld + sub + 4 * c] : 0.0;
    const double t = beta[k] * quad_dot<C>(v, z);
#pragma unroll
    for (int c = 0; c < C; ++c) z[c] = __builtin_fma(-t, v[c], z[c]);
  }
  if (row < q) {
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (sub + 4 * c < q) Zt[row * ld + sub + 4 * c] = z[c];
  }
  group_sync<kWave>();
}

// Implicit QL on (d, e) (one wave, q <= 63 < ld); the rotations are applied to
// the columns of the factor in Zt.  The eigenvalues replace d.
__device__ inline void implicit_ql(double* Zt, int ld, int q, double* dv, const double* ev, int lane) {
  double d = lane < q ? dv[lane] : 0.0, e = lane + 1 < q ? ev[lane] : 0.0;
  double* zp = Zt + min(lane, q);  // lanes without a component use the padding
  for (int l = 0; l < q - 1; ++l) {
    for (int it = 0; it < kMaxSweeps; ++it) {
      // first negligible coupling at or after l
      const uint64_t small = __builtin_amdgcn_ballot_w64(
          fabs(e) <= 2.220446049250313e-16 * (fabs(d) + fabs(next_lane(d))) || lane >= q - 1);
      const int m = l + __builtin_ctzll(small >> l);
      if (m == l) break;
      // Wilkinson's shift (any shift is exact; approximate operations do)
      const double dl = lane_value(d, l), el = lane_value(e, l), dm = lane_value(d, m);
      const double h = 0.5 * (lane_value(d, l + 1) - dl);
      const double h2 = __builtin_fma(h, h, el * el);
      double g = dm - dl;
      if (h2 > 1e-280) g = __builtin_fma(el * el, __builtin_amdgcn_rcp(h + copysign(h2 * rsqrt_f64(h2), h)), g);
      double s = 1.0, c = 1.0, p = 0.0, dnext = dm;  // dnext: d[i + 1] before this rotation
      double zc = zp[m * ld];
      int i = m - 1;
      double ei = lane_value(e, i), di = lane_value(d, i), zi = zp[i * ld];
#pragma unroll 2
      for (; i >= l; --i) {
        const int ip = max(i - 1, l);  // next rotation's inputs, in flight early
        const double ein = lane_value(e, ip), din = lane_value(d, ip), zin = zp[ip * ld];
        const double f = s * ei, b = c * ei;
        const double x = __builtin_fma(f, f, g * g);
        // a vanished bulge: the identity, and the next sweep splits here
        const bool none = x < 1e-280;
        const double y = rsqrt_f64(none ? 1.0 : x);
        s = none ? 0.0 : f * y;
        c = none ? 1.0 : g * y;
        const bool up = lane == i + 1;
        e = up ? (none ? 0.0 : x * y) : e;
        g = dnext - p;
        const double t = __builtin_fma(di - g, s, 2.0 * (c * b));
        p = s * t;
        d = up ? g + p : d;
        g = __builtin_fma(c, t, -b);
        zp[(i + 1) * ld] = __builtin_fma(s, zi, c * zc);
        zc = __builtin_fma(c, zi, -(s * zc));
        dnext = di;
        ei = ein;
        di = din;
        zi = zin;
      }
      zp[l * ld] = zc;
      if (lane == l) {
        d = dnext - p;
        e = g;
      }
      if (lane == m) e = 0.0;
    }
  }
  if (lane < q) dv[lane] = d;
}

// Pair idx of the q (q - 1) / 2 pairs k < l: the triangle as a rectangle, as for the
// covariances below.
__device__ inline void pair_of(int q, int idx, int& k, int& l) {
  const int len = (q - 1) | 1, r = idx / len, c = idx % len, n = q - 1;  // n rows of n .. 1 pairs
  k = c < n - r ? r : n - r - 1 + (n & 1);
  l = (c < n - r ? r + c : k + c - (n - r)) + 1;
}

// One refinement step (as in eigen_wide.hip) of the eigenvectors in the rows of
// V, by the whole workgroup: QL's rotations, a rounded root each, leave them two to
// three times as far off as Jacobi's (9 x 9: 1.0e-15 against 7.1e-16 on average).
// R = I - V V^T and S = V F V^T with F = M - I, whose diagonal is zero exactly, so
// that the products' rounding is small against the gaps also where M is near I.
// Eigenvectors i and j exchange x_ij = (mu_j R_ij + S_ij) / (mu_j - mu_i), mu the
// Rayleigh quotients on F (to d); where that is no small rotation, or the eigenvalues
// are too close to tell, only orthogonality is restored.  Returns whether an x was
// too large for its square to vanish in rounding (another step is due: gaps below
// some 1e-7).  W is scratch like V.  Every thread.
template <int C>
__device__ inline bool refine(const double* M, double* V, double* W, int ld, int q, double* d, int tid) {
  constexpr int kPairs = (16 * C * C / 2 + kQlThreads - 1) / kQlThreads;  // q <= 4 C
  constexpr int kElems = 16 * C * C / kQlThreads;
  const int qq = q * q, np = q * (q - 1) / 2;
  for (int idx = tid; idx < qq; idx += kQlThreads) {
    const int k = idx / q, j = idx % q;
    double s = 0.0;
    for (int i = 0; i < q; ++i) s = __builtin_fma(V[k * ld + i], i == j ? 0.0 : M[i * q + j], s);
    W[k * ld + j] = s;
  }
  __syncthreads();
  auto dots = [&](int k, int l, double& p, double& s) {
    p = s = 0.0;
    for (int j = 0; j < q; ++j) {
      const double v = V[l * ld + j];
      p = __builtin_fma(V[k * ld + j], v, p);
      s = __builtin_fma(W[k * ld + j], v, s);
    }
  };
  double pk = 0.0, sk = 0.0;
  if (tid < q) {
    dots(tid, tid, pk, sk);
    d[tid] = sk / pk;
  }
  __syncthreads();
  double top = 0.0;  // the spread of mu bounds |F|
  for (int k = 0; k < q; ++k) top = fmax(top, fabs(d[k]));
  double x[kPairs], y[kPairs];
  int large = 0;
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    const int idx = tid + u * kQlThreads;
    x[u] = y[u] = 0.0;
    if (idx < np) {
      int k, l;
      pair_of(q, idx, k, l);
      double p, s;
      dots(k, l, p, s);
      const double gap = d[l] - d[k];
      x[u] = y[u] = -0.5 * p;
      if (fabs(gap) > 1e-7 * top) {
        const double a = __builtin_fma(-d[l], p, s) / gap, b = __builtin_fma(-d[k], p, s) / -gap;
        const double m = fmax(fabs(a), fabs(b));
        if (m <= 0x1p-10) {
          x[u] = a;  // of vector k in l
          y[u] = b;  // of vector l in k
          large |= m > 0x1p-28;
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    const int idx = tid + u * kQlThreads;
    if (idx < np) {
      int k, l;
      pair_of(q, idx, k, l);
      W[k * ld + l] = x[u];
      W[l * ld + k] = y[u];
    }
  }
  if (tid < q) W[tid * ld + tid] = 0.5 * (1.0 - pk);
  __syncthreads();
  double v[kElems];
#pragma unroll
  for (int u = 0; u < kElems; ++u) {
    const int idx = tid + u * kQlThreads;
    v[u] = 0.0;
    if (idx < qq) {
      const int l = idx / q, j = idx % q;
      for (int k = 0; k < q; ++k) v[u] = __builtin_fma(W[k * ld + l], V[k * ld + j], v[u]);
      v[u] += V[l * ld + j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kElems; ++u) {
    const int idx = tid + u * kQlThreads;
    if (idx < qq) V[(idx / q) * ld + idx % q] = v[u];
  }
  return __syncthreads_or(large);
}

// N and the status word behind the outputs.
__device__ inline void put_tail(double* to, const uint64_t* state, const DevStatus* status) {
  to[0] = __longlong_as_double((long long)state[0]);
  to[1] = __longlong_as_double((long long)status->bits);
  to[2] = __longlong_as_double((long long)status->parse_off);
}

template <int METHOD>
__device__ inline void finalize_body(const Args& f) {
  constexpr bool QL = METHOD != kLdsJacobi;
  const Layout L = Layout::make(f.p);
  const uint64_t* st = f.state;
  const int64_t n = (int64_t)st[0];
  const int q = f.q;
  const int tid = threadIdx.x;
  const int nth = blockDim.x;  // 64 or kQlThreads, chosen by the launcher from q
  double* mean = f.out;
  double* cov = mean + q;
  double* corr = cov + (int64_t)q * q;
  double* ev = corr + (int64_t)q * q;
  double* evec = ev + q;
  double* varp = evec + (int64_t)q * q;
  double* cump = varp + q;

  __shared__ int s_flag;
  __shared__ int s_rot;
  __shared__ int s_conv;  // converged(): its own word, so that no wave reads s_rot after a reset
  const int m = q + (q & 1);  // players (a dummy when q is odd)
  const int npairs = m / 2;
  // c[npairs], s[npairs], t[npairs], apq[npairs], the round's pairs, A, V
  extern __shared__ double s_dyn[];
  const RotTab R = RotTab::at(s_dyn, npairs);
  // (QL: d, e, beta, q each, and 256 words of exchange in their place, and rows
  // padded to an odd length above q)
  double* A;
  if constexpr (QL) A = s_dyn + 3 * q + 256;
  else A = s_dyn + 5 * npairs;
  const int ld = QL ? (q + 1) | 1 : q;
  double* V = A + (int64_t)q * ld;

  // covariance undefined (the host reports it); nothing is computed, and the
  // exact divisions by n and n - ddof are never reached
  if (n <= f.ddof) return;
  // ---- means and covariance ----
  const double dn = (double)(n - f.ddof);
  for (int a = tid; a < q; a += nth) {
    const int i = f.sel[a];
    mean[a] = f.intf[i] ? exact_mean(st, L, i, n)
                        : __longlong_as_double((long long)st[L.off_mu + i]);
  }
  // q <= 1024: every index below fits 32 bits (64-bit division is a long
  // software sequence on the GPU)
  const int qq = q * q;
  // the triangle a <= b as a rectangle of (q + 1) / 2 rows of length q | 1: row r
  // is row r of the triangle followed by its row of the remaining length, so
  // that no thread idles in the exact divisions
  const int len = q | 1, ntri = (q + 1) / 2 * len;
  for (int idx = tid; idx < ntri; idx += nth) {
    const int r = idx / len, c = idx % len;
    const int a = c < q - r ? r : q - r - 1 + (q & 1);
    const int b = c < q - r ? r + c : a + c - (q - r);
    const int i = f.sel[a], j = f.sel[b];  // sel ascending, so i <= j
    double v;
    if (f.intf[i] && f.intf[j]) v = exact_cov(st, L, i, j, n, f.ddof);
    else v = __longlong_as_double((long long)st[L.off_M2 + tri(L.p, i, j)]) / dn;
    cov[(int64_t)a * q + b] = v;
    cov[(int64_t)b * q + a] = v;
  }
  __syncthreads();
  // ---- correlation ----
  for (int idx = tid; idx < qq; idx += nth) {
    const int a = idx / q, b = idx % q;
    const double caa = cov[(int64_t)a * q + a], cbb = cov[(int64_t)b * q + b];
    double v;
    if (caa == 0.0 || cbb == 0.0) v = __builtin_nan("");
    else if (a == b) v = 1.0;
    else v = cov[idx] / sqrt(caa * cbb);
    corr[idx] = v;
  }
  if (tid == 0) s_flag = 0;
  __syncthreads();
  // ---- PCA input ----
  const double* M = f.pca_on ? cov : corr;
  int bad = 0;
  for (int idx = tid; idx < qq; idx += nth) {
    const double v = M[idx];
    if (!isfinite(v)) bad = 1;
    const int i = idx / q, j = idx % q;
    if constexpr (!QL) {
      A[i * ld + j] = v;
      V[idx] = i == j ? 1.0 : 0.0;
    }
  }
  if (bad) atomicOr(&s_flag, 1);
  __syncthreads();
  if (s_flag) {
    for (int idx = tid; idx < qq; idx += nth) evec[idx] = __builtin_nan("");
    for (int a = tid; a < q; a += nth) {
      ev[a] = varp[a] = cump[a] = __builtin_nan("");
    }
    return;
  }
  if constexpr (QL) {
    double *d = s_dyn, *e = d + q, *beta = e + q, *xp = beta + q;
    static_assert(kQlQ <= 32 && kLdsQ <= 64, "eight or sixteen columns per lane of a quad, a quad per row");
    if constexpr (METHOD == kQlLarge) {
      tridiagonalize<16, false>(M, V, A, ld, q, d, e, beta, xp, tid);
    } else if (q <= 16) {  // one wave holds a quad per row
      if (tid < 64) tridiagonalize<4, true>(M, V, A, ld, q, d, e, beta, xp, tid);
    } else {
      tridiagonalize<8, false>(M, V, A, ld, q, d, e, beta, xp, tid);
    }
    if (tid < 64) implicit_ql(V, ld, q, d, e, tid);
    __syncthreads();
    for (int step = 0; step < 3; ++step) {
      bool again;
      if constexpr (METHOD == kQlLarge) again = refine<16>(M, V, A, ld, q, d, tid);
      else again = q <= 16 ? refine<4>(M, V, A, ld, q, d, tid) : refine<8>(M, V, A, ld, q, d, tid);
      if (!again) break;
    }
    if (tid < q) d[tid] += 1.0;
    __syncthreads();
  } else {
  // ---- cyclic Jacobi, round-robin ordering: q/2 disjoint rotations per round ----
  if (nth == 64 && q <= 16) {
    // One wave, at most one 2x2 block and two V row pairs per lane.  Each
    // round issues all of its loads (block, V pairs, rotation inputs) right
    // after the barrier, with the pair indices computed, not looked up; the
    // rotation tables are read once, after the second barrier.  The same
    // arithmetic as jacobi_blocks / jacobi_vectors.
    const int nblk = npairs * npairs, nv = q * npairs;
    const bool hasb = tid < nblk;
    const int bu = tid / npairs, bv = tid % npairs;
    int vrow[2], vu[2];
    bool hasv[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int idx = tid + 64 * j;
      hasv[j] = idx < nv;
      vrow[j] = idx / npairs;
      vu[j] = idx % npairs;
    }
    for (int sweep = 0; sweep < kMaxSweeps && q > 1; ++sweep) {
      if (tid == 0) s_rot = 0;
      __syncthreads();
      for (int r = 0; r < m - 1; ++r) {
        int a = 0, b = 0, c2 = 0, d2 = 0;
        double x00 = 0.0, x01 = 0.0, x10 = 0.0, x11 = 0.0;
        if (hasb) {
          rr_pair(bu, r, m, a, b);
          rr_pair(bv, r, m, c2, d2);
          x00 = A[a * q + c2];
          if (d2 < q) x01 = A[a * q + d2];
          if (b < q) x10 = A[b * q + c2];
          if (b < q && d2 < q) x11 = A[b * q + d2];
        }
        int pa[2], pb[2];
        double va[2] = {0.0, 0.0}, vb[2] = {0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          rr_pair(vu[j], r, m, pa[j], pb[j]);
          if (hasv[j] && pb[j] < q) {
            va[j] = V[vrow[j] * q + pa[j]];
            vb[j] = V[vrow[j] * q + pb[j]];
          }
        }
        if (tid < npairs) {
          int ra, rb;
          rr_pair(tid, r, m, ra, rb);
          double c = 1.0, s = 0.0, t = 0.0, apq = 0.0;
          if (rb < q && jacobi_rotation(A, q, ra, rb, c, s, t, apq)) atomicAdd(&s_rot, 1);
          R.c[tid] = c;
          R.s[tid] = s;
          R.t[tid] = t;
          R.apq[tid] = apq;
        }
        __syncthreads();
        if (hasb) {
          const double cu_ = R.c[bu], su = R.s[bu], cv_ = R.c[bv], sv = R.s[bv];
          if (su != 0.0 || sv != 0.0) {
            const double y00 = cu_ * x00 - su * x10, y10 = su * x00 + cu_ * x10;
            const double y01 = cu_ * x01 - su * x11, y11 = su * x01 + cu_ * x11;
            double z00 = cv_ * y00 - sv * y01, z01 = sv * y00 + cv_ * y01;
            double z10 = cv_ * y10 - sv * y11, z11 = sv * y10 + cv_ * y11;
            if (bu == bv && su != 0.0) {  // the rotated 2x2 block itself: exact update
              const double t = R.t[bu], apq = R.apq[bu];
              z00 = x00 - t * apq;
              z11 = x11 + t * apq;
              z01 = 0.0;
              z10 = 0.0;
            }
            A[a * q + c2] = z00;
            if (d2 < q) A[a * q + d2] = z01;
            if (b < q) A[b * q + c2] = z10;
            if (b < q && d2 < q) A[b * q + d2] = z11;
          }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (!hasv[j] || pb[j] >= q) continue;
          const double s = R.s[vu[j]];
          if (s == 0.0) continue;
          const double c = R.c[vu[j]];
          V[vrow[j] * q + pa[j]] = c * va[j] - s * vb[j];
          V[vrow[j] * q + pb[j]] = s * va[j] + c * vb[j];
        }
        __syncthreads();
      }
      if (s_rot == 0 || converged(A, q, tid, nth, &s_conv)) break;
      __syncthreads();
    }
  } else {
  for (int sweep = 0; sweep < kMaxSweeps && q > 1; ++sweep) {
    if (tid == 0) s_rot = 0;
    __syncthreads();
    for (int r = 0; r < m - 1; ++r) {
      for (int k = tid; k < npairs; k += nth) {
        int a, b;
        rr_pair(k, r, m, a, b);
        double c = 1.0, s = 0.0, t = 0.0, apq = 0.0;
        if (b < q && jacobi_rotation(A, q, a, b, c, s, t, apq)) atomicAdd(&s_rot, 1);
        R.c[k] = c;
        R.s[k] = s;
        R.t[k] = t;
        R.apq[k] = apq;
        R.pair[k] = make_int2(a, b);
      }
      __syncthreads();
      jacobi_blocks(A, q, npairs, R, tid, nth);
      jacobi_vectors(V, q, npairs, R, tid, nth);
      __syncthreads();
    }
    if (s_rot == 0 || converged(A, q, tid, nth, &s_conv)) break;
    __syncthreads();
  }
  }
  }

  // ---- sort descending (ties: lower index first), sign rule, percentages ----
  // component j of eigenvector k at V + j vj + k vk; sorted eigenvalues, the largest
  // magnitude of their vectors and their sources (complemented where the vector
  // changes sign) in LDS that is free now
  const int vj = QL ? 1 : q, vk = QL ? ld : 1;
  double* lam = QL ? s_dyn + q : s_dyn;
  double* var = QL ? s_dyn + 2 * q : s_dyn + q;
  int* src = (int*)(s_dyn + (QL ? 3 : 2) * q);
  double* top = QL ? s_dyn + 4 * q : V + qq;
  for (int k = tid; k < q; k += nth) {
    const double lk = QL ? s_dyn[k] : A[(int64_t)k * q + k];
    int rank = 0;
    double best = 0.0;
    for (int j = 0; j < q; ++j) {
      const double lj = QL ? s_dyn[j] : A[(int64_t)j * q + j];
      rank += (lj > lk) || (lj == lk && j < k);
      best = fmax(best, fabs(V[(int64_t)j * vj + (int64_t)k * vk]));
    }
    // eigenvector k's sign: largest |entry| positive (lowest index on ties)
    double lead = 0.0;
    for (int j = q - 1; j >= 0; --j) {
      const double x = V[(int64_t)j * vj + (int64_t)k * vk];
      if (fabs(x) >= kTie * best) lead = x;
    }
    lam[rank] = lk;
    top[rank] = best;
    src[rank] = lead < 0.0 ? ~k : k;
  }
  __syncthreads();
  if (f.want_vectors) {
    for (int idx = tid; idx < qq; idx += nth) {
      const int r = idx / q, j = idx % q;
      const int k = src[r] < 0 ? ~src[r] : src[r];
      double x = V[(int64_t)j * vj + (int64_t)k * vk];
      if (fabs(x) >= kTie * top[r]) x = copysign(top[r], x);
      evec[idx] = src[r] < 0 ? -x : x;
    }
  }
  double tot = 0.0;
  for (int k = 0; k < q; ++k) tot += lam[k];
  for (int k = tid; k < q; k += nth) {
    ev[k] = lam[k];
    varp[k] = var[k] = 100.0 * lam[k] / tot;
  }
  __syncthreads();
  for (int k = tid; k < q; k += nth) {
    double run = 0.0;
    for (int j = 0; j <= k; ++j) run += var[j];
    cump[k] = run;
  }
}

// The outputs go to page-locked host memory from here: a copy command and its wait
// cost more than these stores.
template <int METHOD>
__global__ __launch_bounds__(kQlThreads) void k_finalize(Args f) {
  finalize_body<METHOD>(f);
  __syncthreads();
  const int words = 4 * f.q + 3 * f.q * f.q;
  for (int i = threadIdx.x; i < words; i += blockDim.x) f.host[i] = f.out[i];
  if (threadIdx.x == 0) put_tail(f.host + words, f.state, f.status);
}

__global__ void k_raw(const uint64_t* st, int p, const uint8_t* intf, double* out) {
  // out: s_f64[p], C_f64[p*p]
  const Layout L = Layout::make(p);
  const int64_t n = (int64_t)st[0];
  const double dn = (double)n;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < p + (int64_t)p * p;
       idx += (int64_t)gridDim.x * blockDim.x) {
    if (idx < p) {
      const int i = (int)idx;
      double v;
      if (intf[i]) {
        bool neg;
        const u128 m = abs128(load_i128(st + L.off_s + 2 * i), &neg);
        v = u256_div_to_double(neg, u256_from_u128(m), u256_from_u128(1));
      } else {
        v = dn * __longlong_as_double((long long)st[L.off_mu + i]);
      }
      out[i] = v;
    } else {
      const int64_t e = idx - p;
      int i = (int)(e / p), j = (int)(e % p);
      if (i > j) {
        const int x = i;
        i = j;
        j = x;
      }
      double v;
      if (intf[i] && intf[j]) {
        bool neg;
        const u128 m = abs128(load_i128(st + L.off_C + 2 * tri(p, i, j)), &neg);
        v = u256_div_to_double(neg, u256_from_u128(m), u256_from_u128(1));
      } else {
        const double mi = __longlong_as_double((long long)st[L.off_mu + i]);
        const double mj = __longlong_as_double((long long)st[L.off_mu + j]);
        v = __longlong_as_double((long long)st[L.off_M2 + tri(p, i, j)]) + dn * mi * mj;
      }
      out[idx] = v;
    }
  }
}

}  // namespace

static Args args_of(const FinalizeLaunch& F) {
  Args a;
  a.state = F.state;
  a.p = F.p;
  a.sel = F.sel_dev;
  a.q = F.q;
  a.intf = F.intflags_dev;
  a.ddof = F.ddof;
  a.pca_on = F.pca_on;
  a.want_vectors = F.want_vectors;
  a.out = F.out;
  a.status = F.status;
  a.host = F.host;
  return a;
}

hipError_t launch_finalize_ql(const FinalizeLaunch& F, hipStream_t s) {
  const size_t q = (size_t)F.q, shm = (256 + (3 + 2 * ((q + 1) | 1)) * q) * sizeof(double);
  if (F.q <= kQlQ) hipLaunchKernelGGL(k_finalize<kQl>, dim3(1), dim3(kQlThreads), shm, s, args_of(F));
  else hipLaunchKernelGGL(k_finalize<kQlLarge>, dim3(1), dim3(kQlThreads), shm, s, args_of(F));
  return hipGetLastError();
}

hipError_t launch_finalize(const FinalizeLaunch& F, hipStream_t s) {
  if (F.q > (F.pca_on ? kLdsQ : kQlQ)) return launch_finalize_wide(F, s);
  if (!F.pca_on && F.q > kOneRotation) return launch_finalize_ql(F, s);
  // one wave for the small matrices (its barriers cost nothing)
  const size_t q = (size_t)F.q, shm = (5 * ((q + 1) / 2) + 2 * q * q + q) * sizeof(double);
  hipLaunchKernelGGL(k_finalize<kLdsJacobi>, dim3(1), dim3(F.q <= 16 ? 64 : kQlThreads), shm, s, args_of(F));
  return hipGetLastError();
}

void launch_raw(const uint64_t* state, int p, const uint8_t* intf, double* out, hipStream_t s) {
  const int64_t work = p + (int64_t)p * p;
  const unsigned blocks = (unsigned)std::min<int64_t>((work + 255) / 256, 1024);
  hipLaunchKernelGGL(k_raw, dim3(blocks), dim3(256), 0, s, state, p, intf, out);
}

}  // namespace st
