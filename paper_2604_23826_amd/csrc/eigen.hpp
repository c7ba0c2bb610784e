// Eigensolver pieces shared by the one-workgroup finalize (finalize.hip) and
// the wide one (eigen_wide.hip).
#pragma once
#include <type_traits>

#include "common.hpp"

namespace st {
namespace {

constexpr int kNB = 4;     // 2 x 2 blocks per thread and batch
constexpr int kNV = 4;     // V row pairs per thread and batch
constexpr int kMaxSweeps = 60;

// Largest correlation matrix that one workgroup decomposes by QL (finalize.hip) at
// once.  The rotation chain grows with q^2, the launches of eigen_wide.hip with little
// more than a constant: a whole finalize call takes 180 us at 24 columns by QL and 183
// at 25 by the launches; at 28 QL took 251 against 220, at 60 791 against 333.
constexpr int kQlQ = 24;
// Largest matrix decomposed in one workgroup's LDS: covariance matrices by Jacobi, and
// correlation matrices that eigen_wide.hip hands back, by QL.
constexpr int kLdsQ = 60;

// Entries of an eigenvector within kTie of its largest magnitude are ties: they
// differ by the solver's rounding only (the all-equal vector of collinear columns,
// say; up to 17 units of 2^-52 at 24 columns).  They are returned equal, and the
// one of lowest index decides the vector's sign, which so does not hang on that
// rounding.
constexpr double kTie = 1.0 - 32 * 2.220446049250313e-16;

// Round-robin schedule on m (even) players: player at position pos in round
// r (0 <= pos < m, 0 <= r < m - 1).
__device__ inline int rr_player(int pos, int r, int m) {
  if (pos == 0) return 0;
  const int x = pos - 1 + r;  // < 2 (m - 1)
  return (x >= m - 1 ? x - (m - 1) : x) + 1;
}

// The two players of pair k in round r, smaller first.
__device__ inline void rr_pair(int k, int r, int m, int& a, int& b) {
  const int x = rr_player(k, r, m), y = rr_player(m - 1 - k, r, m);
  a = min(x, y);
  b = max(x, y);
}

// Rotation tables of one round: cosine, sine, tangent, the annihilated
// element and the pair (a, b) of every pair k.
struct RotTab {
  double* c;
  double* s;
  double* t;
  double* apq;
  int2* pair;
  __device__ static RotTab at(double* base, int npairs) {
    return RotTab{base, base + npairs, base + 2 * npairs, base + 3 * npairs, (int2*)(base + 4 * npairs)};
  }
};

// Whether the element apq of the pair with diagonal entries app, aqq is
// rotated away: not when it is already negligible against them.
__device__ inline bool rotates(double apq, double app, double aqq) {
  const double tol = 2.220446049250313e-16;
  return apq != 0.0 && fabs(apq) > tol * sqrt(fabs(app * aqq));
}

// Jacobi rotation annihilating A[a][b] (a < b < q), or none (c = 1, s = 0)
// when the element is already negligible.  Returns whether it rotates.
__device__ inline bool jacobi_rotation(const double* A, int q, int a, int b, double& c, double& s, double& t,
                                       double& apq) {
  c = 1.0;
  s = t = 0.0;
  apq = A[(int64_t)a * q + b];
  const double app = A[(int64_t)a * q + a], aqq = A[(int64_t)b * q + b];
  if (rotates(apq, app, aqq)) {
    const double theta = (aqq - app) / (2.0 * apq);
    t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
    c = 1.0 / sqrt(t * t + 1.0);
    s = t * c;
    return true;
  }
  apq = 0.0;
  return false;
}

// A <- J^T A J on the 2x2 blocks idx = u * npairs + v of one round (pair u
// rows, pair v columns), idx = start, start + stride, ...  The blocks of a
// round are disjoint, so a batch is loaded before it is written; (u, v)
// advance by stride without division.
__device__ inline void jacobi_blocks(double* A, int q, int npairs, const RotTab& R, int start, int stride) {
  const int nblk = npairs * npairs;
  const int du = stride / npairs, dv = stride % npairs;
  int cu = start / npairs, cv = start % npairs;
  for (int base = start; base < nblk; base += stride * kNB) {
    double x[kNB][4];
    int ia[kNB], ib[kNB], ic[kNB], id[kNB], iu[kNB], iv[kNB];
#pragma unroll
    for (int e = 0; e < kNB; ++e) {
      iu[e] = cu;
      iv[e] = cv;
      cv += dv;
      cu += du;
      if (cv >= npairs) {
        cv -= npairs;
        ++cu;
      }
      x[e][0] = x[e][1] = x[e][2] = x[e][3] = 0.0;
      ia[e] = ib[e] = ic[e] = id[e] = 0;
      if (base + e * stride >= nblk) continue;
      const int2 pu = R.pair[iu[e]], pv = R.pair[iv[e]];
      ia[e] = pu.x;
      ib[e] = pu.y;
      ic[e] = pv.x;
      id[e] = pv.y;
      const bool bq = ib[e] < q, dq = id[e] < q;
      x[e][0] = A[(int64_t)ia[e] * q + ic[e]];
      if (dq) x[e][1] = A[(int64_t)ia[e] * q + id[e]];
      if (bq) x[e][2] = A[(int64_t)ib[e] * q + ic[e]];
      if (bq && dq) x[e][3] = A[(int64_t)ib[e] * q + id[e]];
    }
#pragma unroll
    for (int e = 0; e < kNB; ++e) {
      if (base + e * stride >= nblk) continue;
      const int u = iu[e], v = iv[e];
      const double cu_ = R.c[u], su = R.s[u], cv_ = R.c[v], sv = R.s[v];
      if (su == 0.0 && sv == 0.0) continue;
      const int a = ia[e], b = ib[e], c2 = ic[e], d2 = id[e];
      const bool bq = b < q, dq = d2 < q;
      const double x00 = x[e][0], x01 = x[e][1], x10 = x[e][2], x11 = x[e][3];
      // rows: (row a, row b) <- (c row a - s row b, s row a + c row b)
      const double y00 = cu_ * x00 - su * x10, y10 = su * x00 + cu_ * x10;
      const double y01 = cu_ * x01 - su * x11, y11 = su * x01 + cu_ * x11;
      // columns: (col c2, col d2) <- (c col c2 - s col d2, s col c2 + c col d2)
      double z00 = cv_ * y00 - sv * y01, z01 = sv * y00 + cv_ * y01;
      double z10 = cv_ * y10 - sv * y11, z11 = sv * y10 + cv_ * y11;
      if (u == v && su != 0.0) {  // the rotated 2x2 block itself: exact update
        const double t = R.t[u], apq = R.apq[u];
        z00 = x00 - t * apq;
        z11 = x11 + t * apq;
        z01 = 0.0;
        z10 = 0.0;
      }
      A[(int64_t)a * q + c2] = z00;
      if (dq) A[(int64_t)a * q + d2] = z01;
      if (bq) A[(int64_t)b * q + c2] = z10;
      if (bq && dq) A[(int64_t)b * q + d2] = z11;
    }
  }
}

// V <- V J on the entries idx = row * npairs + u, batched the same way.
__device__ inline void jacobi_vectors(double* V, int q, int npairs, const RotTab& R, int start, int stride) {
  const int nv = q * npairs;
  const int du = stride / npairs, dv = stride % npairs;
  int vr = start / npairs, vu = start % npairs;
  for (int base = start; base < nv; base += stride * kNV) {
    double va[kNV], vb[kNV];
    int jr[kNV], ju[kNV];
#pragma unroll
    for (int e = 0; e < kNV; ++e) {
      jr[e] = vr;
      ju[e] = vu;
      vu += dv;
      vr += du;
      if (vu >= npairs) {
        vu -= npairs;
        ++vr;
      }
      va[e] = vb[e] = 0.0;
      if (base + e * stride >= nv) continue;
      const int2 pu = R.pair[ju[e]];
      if (pu.y >= q) continue;  // the dummy player of odd q
      va[e] = V[(int64_t)jr[e] * q + pu.x];
      vb[e] = V[(int64_t)jr[e] * q + pu.y];
    }
#pragma unroll
    for (int e = 0; e < kNV; ++e) {
      if (base + e * stride >= nv) continue;
      const int u = ju[e];
      const double s = R.s[u];
      if (s == 0.0) continue;  // also the dummy player's pair
      const int2 pu = R.pair[u];
      const double c = R.c[u];
      V[(int64_t)jr[e] * q + pu.x] = c * va[e] - s * vb[e];
      V[(int64_t)jr[e] * q + pu.y] = s * va[e] + c * vb[e];
    }
  }
}

// Ordering point between the lanes that share the work: the whole workgroup,
// or (kWave) one wave, whose LDS accesses execute in order.
template <bool kWave>
__device__ inline void group_sync() {
  if constexpr (kWave) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

__device__ inline double lane_value(double v, int lane) {  // lane wave-uniform
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum over the four lanes of a quad, in every lane of it.
__device__ inline double quad_sum(double v) {
  auto move = [](double x, auto ctrl) {
    constexpr int c = decltype(ctrl)::value;
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), c, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), c, 0xF, 0xF, false));
  };
  v += move(v, std::integral_constant<int, 0xB1>{});  // quad_perm [1,0,3,2]
  v += move(v, std::integral_constant<int, 0x4E>{});  // quad_perm [2,3,0,1]
  return v;
}

// 1 / sqrt(x) for normal x > 0: the hardware estimate and one third-order step.
__device__ inline double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

// Lane i receives lane i + 1's value (lane 63: zero).
__device__ inline double next_lane(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xF, 0xF, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xF, 0xF, true));
}

// Sum of u[c] v[c] over the quad's columns, in every lane of it.
template <int C>
__device__ inline double quad_dot(const double (&u)[C], const double (&v)[C]) {
  double t0 = 0.0, t1 = 0.0;
#pragma unroll
  for (int c = 0; c < C; c += 2) {
    t0 = __builtin_fma(u[c], v[c], t0);
    t1 = __builtin_fma(u[c + 1], v[c + 1], t1);
  }
  return quad_sum(t0 + t1);
}

// Householder reduction of a symmetric q x q matrix held in registers: quad i
// of the threads holds row i, lane sub of it columns sub, sub + 4, ... (4 C >=
// q; kRows quads, those past q hold zeros).  Gives d[q], e[q] (e[k] couples k
// and k + 1, e[q - 1] = 0) and the reflectors: row k of H (leading dimension
// ld, zero up to column k) with its factor beta[k], k < q - 2.  xp: 4 kRows
// words of LDS.  A step exchanges row k and the product through LDS, two
// ordering points in all.  The caller orders d, e, beta and H before use.
template <int C, bool kWave, int kRows>
__device__ inline void tri_reduce(double (&a)[C], double* H, int ld, int q, double* d, double* e, double* beta,
                                  double* xp, int tid) {
  const int row = tid >> 2, sub = tid & 3;
  for (int k = 0; k + 1 < q; ++k) {
    double* xb = xp + (k & 1) * 2 * kRows;  // row k, then the product
    double* pb = xb + kRows;
    if (row == k) {
#pragma unroll
      for (int c = 0; c < C; ++c) xb[sub + 4 * c] = a[c];
    }
    group_sync<kWave>();
    const double x0 = xb[k + 1], xi = xb[row];
    if (k + 2 == q) {
      if (tid == 0) e[k] = x0;
      break;
    }
    double v[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int j = sub + 4 * c;
      const double x = xb[j];
      v[c] = j > k + 1 ? x : 0.0;
    }
    const double tail = quad_dot<C>(v, v);
    if (tail < 1e-280) {  // already tridiagonal here (as far below any rounding)
      if (row == k) {
        if (sub == 0) {
          beta[k] = 0.0;
          e[k] = x0;
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
          if (sub + 4 * c < q) H[k * ld + sub + 4 * c] = 0.0;
      }
      continue;
    }
    const double n2 = __builtin_fma(x0, x0, tail), norm = n2 * rsqrt_f64(n2);
    const double v0 = x0 >= 0.0 ? x0 + norm : x0 - norm;
    const double bk = 1.0 / (norm * (norm + fabs(x0)));
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (sub + 4 * c == k + 1) v[c] = v0;
    const bool in = row > k && row < q;
    const double av = quad_dot<C>(a, v);
    const double vi = row == k + 1 ? v0 : (in ? xi : 0.0);
    const double pi = in ? bk * av : 0.0;
    if (sub == 0) pb[row] = pi;
    group_sync<kWave>();
    double p[C];
#pragma unroll
    for (int c = 0; c < C; ++c) p[c] = pb[sub + 4 * c];
    const double h = 0.5 * bk * quad_dot<C>(p, v);
    const double wi = __builtin_fma(-h, vi, pi);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const double wj = __builtin_fma(-h, v[c], p[c]);
      a[c] -= __builtin_fma(vi, wj, wi * v[c]);
    }
    if (row == k) {
      if (sub == 0) {
        beta[k] = bk;
        e[k] = x0 >= 0.0 ? -norm : norm;
      }
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (sub + 4 * c < q) H[k * ld + sub + 4 * c] = v[c];
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (row < q && sub + 4 * c == row) d[row] = a[c];
  if (tid == 0) e[q - 1] = 0.0;
}

}  // namespace
}  // namespace st
