// Statistics with missing values (NaN), pairwise-complete: for every pair of
// columns (i, j) the rows where both are present, their count n_ij, the two
// columns' means over those rows and the centred co-moments -- the
// missing-value extension the paper names as future work (section
// "Limitations and Future Work").  Covariance and correlation of a pair use
// only its complete rows (pairwise deletion).
//
// Per block of rows, with K_i the first present value of column i from the
// block's shift row on (its own first row; blocks of less than 4096 rows: the first
// of their 4096) and, per row, d_i = x_i - K_i and v_i = 1 where x_i is present
// (d_i = v_i = 0 where it is NaN), four matrix products over the block's rows
// hold everything:
//     N = V^T V          n_ij
//     S = D^T V          S[i][j] = sum over rows with j present of d_i
//     Q = (D o D)^T V    Q[i][j] = sum over rows with j present of d_i^2
//     C = D^T D          sum of d_i d_j (zero wherever either is missing)
// S, Q and C on the FP64 matrix cores (v_mfma_f64_16x16x4, p <= 16): a lane holds
// d, d^2 and v of one column in one row of a step, its element of both operands:
// three products per 4 rows above 8 columns.  Up to 8 columns half of the A
// operand is D and half D o D, half of B V and half D, so one product gives all
// three; up to 4 columns it also takes two groups of 4 rows.  N is counted on the
// int8 matrix cores, one product per 64 rows (the presence bits of 16 steps as
// bytes).  The next steps' values are in flight while the current ones are
// multiplied.  2e6 rows of 12 FP64 columns: 215 -> 71 us (four FP64 products per
// step and no loads in flight before); the products' own time is 39 us, HBM's 27.
#include <cstring>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "runtime.hpp"

namespace st {
namespace pw {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef int i4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kMaxP = 16;
constexpr int kScan = 256;  // rows searched for a block's shift, from its shift row

// Block record: n (rows), K[16], then the four 16 x 16 tiles N, S, Q, C.
constexpr int kRecWords = 1 + kMaxP + 4 * 256;

struct Args {
  const char* colbase[kMaxP];
  int64_t colstride[kMaxP];
  int32_t dtype[kMaxP];  // STATS_F32 / STATS_F64
  int p;
  int64_t nrows, R;
  int64_t shift_low;  // see shift_row
  double* rec;
};

constexpr int kU = 8;  // steps in flight per wave

// Columns of a launch: all FP64, all FP32, or both (two words per value, the
// second re-read for FP32).
enum { K_F64 = 0, K_F32 = 1, K_MIX = 2 };
template <int KIND> struct Raw { typedef double type; };
template <> struct Raw<K_F32> { typedef float type; };
template <> struct Raw<K_MIX> { typedef uint2 type; };

template <int KIND>
__device__ inline typename Raw<KIND>::type load_raw(const char* p, bool f32) {
  if constexpr (KIND == K_MIX) return make_uint2(load_global<uint32_t>(p), load_global<uint32_t>(p + (f32 ? 0 : 4)));
  else return load_global<typename Raw<KIND>::type>(p);
}
template <int KIND>
__device__ inline double value(typename Raw<KIND>::type x, bool f32) {
  if constexpr (KIND == K_MIX)
    return f32 ? (double)__uint_as_float(x.x) : __longlong_as_double((long long)(((uint64_t)x.y << 32) | x.x));
  else return (double)x;
}

// W: columns per operand part, 16, 8 or 4 (p <= W).
template <int KIND, int W>
__global__ __launch_bounds__(kThreads) void k_pairwise(Args a) {
  typedef typename Raw<KIND>::type T;
  constexpr int NT = W == 16 ? 3 : 1;     // FP64 tiles: S, Q, C, or one with all
  constexpr int NG = W == 4 ? 2 : 1;      // row groups per product
  constexpr int kStep = 4 * NG;           // rows per step
  constexpr int kWave = kU * kStep;       // rows per wave and stage
  __shared__ double sK[kMaxP];
  __shared__ int s_first[kMaxP];
  __shared__ double red[4][NT][4][64];  // [wave][tile][register][lane]
  __shared__ int redn[4][4][64];
  const int64_t r0 = (int64_t)blockIdx.x * a.R, r1 = min(r0 + a.R, a.nrows);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q16 = lane & 15;
  const int p = a.p;
  // shift: the first present value of each column among the first rows
  const int64_t rk = shift_row(r0, a.shift_low);
  {
    const int c = tid & 15, cc = c < p ? c : 0;
    const bool f32 = a.dtype[cc] == STATS_F32;
    const int lim = (int)min((int64_t)kScan, (a.shift_low ? a.nrows : r1) - rk);
    if (tid < kMaxP) s_first[tid] = INT32_MAX;
    __syncthreads();
    for (int k = tid >> 4; k - (tid >> 4) < lim; k += 16) {
      bool found = c >= p;
      if (!found && k < lim) {
        const double x = value<KIND>(load_raw<KIND>(a.colbase[cc] + (rk + k) * a.colstride[cc], f32), f32);
        if (x == x) atomicMin(&s_first[c], k);
      }
      __syncthreads();
      found = found || s_first[c] != INT32_MAX;
      if (__syncthreads_and(found)) break;
    }
    if (tid < kMaxP) {
      double K = 0.0;
      if (tid < p && s_first[tid] != INT32_MAX)
        K = value<KIND>(load_raw<KIND>(a.colbase[tid] + (rk + s_first[tid]) * a.colstride[tid], f32), f32);
      sK[tid] = K;
    }
    __syncthreads();
  }
  const int col = q16 % W, part = W == 16 ? 0 : q16 / W % 2;  // part 1: d^2 in A, d in B
  const int rl = (lane >> 4) + (NG == 2 ? 4 * (q16 / 8) : 0);  // row of a step
  const bool cv = col < p;
  const int cc = cv ? col : 0;
  const bool f32 = a.dtype[cc] == STATS_F32;
  const int64_t stride = a.colstride[cc];
  const double K = sK[cc];
  d4 tile[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) tile[t] = (d4){0.0, 0.0, 0.0, 0.0};
  i4 tn = {0, 0, 0, 0};
  i4 bits = {0, 0, 0, 0};  // presence bytes of 16 steps
  const char* pc = a.colbase[cc] + (r0 + kWave * wave + rl) * stride;
  const int64_t step = kStep * stride, sstep = (int64_t)4 * kWave * stride;
  auto load = [&](T (&x)[kU]) {
#pragma unroll
    for (int u = 0; u < kU; ++u) x[u] = load_raw<KIND>(pc + u * step, f32);
    pc += sstep;
  };
  // half: which eight of the sixteen presence bytes these steps fill; rows at or
  // past `rows` (relative to this wave's first) are absent
  auto use = [&](const T (&x)[kU], int rows, auto half_c) {
    constexpr int half = decltype(half_c)::value;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const double y = value<KIND>(x[u], f32);
      const bool ok = cv && y == y && kStep * u + rl < rows;
      const double d = ok ? y - K : 0.0, v = ok ? 1.0 : 0.0, d2 = d * d;
      constexpr int base = half * kU;
      bits[(base + u) / 4] |= ok ? 1 << (8 * ((base + u) % 4)) : 0;
      if constexpr (NT == 3) {
        tile[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d, v, tile[0], 0, 0, 0);
        tile[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(d2, v, tile[1], 0, 0, 0);
        tile[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(d, d, tile[2], 0, 0, 0);
      } else {
        tile[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(part ? d2 : d, part ? d : v, tile[0], 0, 0, 0);
      }
    }
  };
  auto count = [&]() {
    tn = __builtin_amdgcn_mfma_i32_16x16x64_i8(bits, bits, tn, 0, 0, 0);
    bits = (i4){0, 0, 0, 0};
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  const int64_t nst = (r1 - r0) / (4 * kWave);  // whole stages
  T xa[kU], xb[kU];
  if (nst > 0) load(xa);
  for (int64_t t = 0; t < nst; t += 2) {
    if (t + 1 < nst) load(xb);
    use(xa, kWave, H0{});
    if (t + 1 < nst) {
      if (t + 2 < nst) load(xa);
      use(xb, kWave, H1{});
    }
    count();
  }
  const int64_t rb = r0 + nst * 4 * kWave + kWave * wave;  // this wave's rows of the last stage
  if (rb < r1) {
    const int rows = (int)min((int64_t)kWave, r1 - rb);
#pragma unroll
    for (int u = 0; u < kU; ++u)
      xa[u] = load_raw<KIND>(a.colbase[cc] + (rb + min(kStep * u + rl, rows - 1)) * stride, f32);
    use(xa, rows, H0{});
    count();
  }
  // the four waves' tiles, added in a fixed order
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int t = 0; t < NT; ++t) red[wave][t][k][lane] = tile[t][k];
    redn[wave][k][lane] = tn[k];
  }
  __syncthreads();
  double* out = a.rec + (int64_t)blockIdx.x * kRecWords;
  // element (x, y) of FP64 tile t: register x / 4 of lane 16 (x % 4) + y; of the
  // int32 tile: register x % 4 of lane 16 (x / 4) + y
  auto at = [&](int t, int x, int y) {
    const int k = x >> 2, l = 16 * (x & 3) + y;
    return red[0][t][k][l] + red[1][t][k][l] + red[2][t][k][l] + red[3][t][k][l];
  };
  for (int e = tid; e < W * W; e += kThreads) {
    const int i = e / W, j = e % W;
    double S = 0.0, Q = 0.0, C = 0.0;
    int n = 0;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int o = 2 * W * g;  // first operand column of the row group
      if constexpr (NT == 3) {
        S = at(0, i, j);
        Q = at(1, i, j);
        C = at(2, i, j);
      } else {
        S += at(0, o + i, o + j);
        Q += at(0, o + W + i, o + j);
        C += at(0, o + i, o + W + j);
      }
      const int k = (o + i) & 3, l = 16 * ((o + i) >> 2) + o + j;
      n += redn[0][k][l] + redn[1][k][l] + redn[2][k][l] + redn[3][k][l];
    }
    double* rec = out + 1 + kMaxP + 16 * i + j;
    rec[0] = (double)n;
    rec[256] = S;
    rec[512] = Q;
    rec[768] = C;
  }
  if (tid < kMaxP) out[1 + tid] = sK[tid];
  if (tid == 0) out[0] = (double)(r1 - r0);
}

// ---- merge: block records -> per-pair state, states -> state ----------------
//
// State of pair t = (i, j), i <= j (packed upper triangle): n, mean_i, mean_j,
// M2_ii, M2_jj, C_ij over the rows where both columns are present.  Blocks
// are combined by the pairwise update of Chan, Golub and LeVeque (the same
// update as the complete-data path), along a fixed tree, so results repeat
// bit for bit.

struct Pair {
  double n, mi, mj, m2i, m2j, c;
};

__device__ inline Pair combine(const Pair& a, const Pair& b) {
  if (b.n == 0.0) return a;
  if (a.n == 0.0) return b;
  Pair r;
  r.n = a.n + b.n;
  const double di = b.mi - a.mi, dj = b.mj - a.mj, f = a.n * b.n / r.n;
  r.mi = a.mi + di * (b.n / r.n);
  r.mj = a.mj + dj * (b.n / r.n);
  r.m2i = a.m2i + b.m2i + di * di * f;
  r.m2j = a.m2j + b.m2j + dj * dj * f;
  r.c = a.c + b.c + di * dj * f;
  return r;
}

// Pair (i, j) of block record rec: n, S_i, S_j, Q_i, Q_j, C.
__device__ inline Pair sums_of(const double* rec, int i, int j) {
  const double* N = rec + 1 + kMaxP;
  const double* S = N + 256;
  const double* Q = S + 256;
  const double* C = Q + 256;
  return Pair{N[16 * i + j], S[16 * i + j], S[16 * j + i], Q[16 * i + j], Q[16 * j + i], C[16 * i + j]};
}

// Shifted sums -> centred form, with the shifts of record rec.
__device__ inline Pair centred(const Pair& s, const double* rec, int i, int j) {
  const double* K = rec + 1;
  if (s.n == 0.0) return Pair{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  Pair r;
  r.n = s.n;
  r.mi = K[i] + s.mi / s.n;
  r.mj = K[j] + s.mj / s.n;
  r.m2i = s.m2i - s.mi * (s.mi / s.n);
  r.m2j = s.m2j - s.mj * (s.mj / s.n);
  r.c = s.c - s.mi * (s.mj / s.n);
  return r;
}

__device__ inline void pair_of(int p, int t, int& i, int& j) {
  i = 0;
  int rem = t;
  while (rem >= p - i) {
    rem -= p - i;
    ++i;
  }
  j = i + rem;
}

constexpr int kMergeThreads = 256;

// One workgroup per pair: thread k combines a contiguous range of blocks,
// then a fixed binary tree over the threads; the result is combined with the
// incoming state (cur) into next.  run > 1 (a power of two up to 16; at most 256
// records): thread b holds record b, `run` of which share their shifts and are
// added up, as the one block of 4096 rows that they were cut from, before they
// are centred (see fold_runs of the complete-data merge); the result goes to the
// thread that would have it from such blocks.
__global__ __launch_bounds__(kMergeThreads) void k_pw_merge(const double* rec, int64_t nblocks, int p,
                                                           const double* cur, double* next, int run) {
  __shared__ Pair part[kMergeThreads];
  const int t = blockIdx.x;
  int i, j;
  pair_of(p, t, i, j);
  Pair acc{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (run > 1) {
    const int b = threadIdx.x;
    const double* r = rec + (b < nblocks ? b : 0) * kRecWords;
    Pair s = sums_of(r, i, j);
    if (b >= nblocks) s = Pair{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int d = 1; d < run && d < nblocks; d <<= 1) {
      s.n += __shfl_xor(s.n, d, 64);
      s.mi += __shfl_xor(s.mi, d, 64);
      s.mj += __shfl_xor(s.mj, d, 64);
      s.m2i += __shfl_xor(s.m2i, d, 64);
      s.m2j += __shfl_xor(s.m2j, d, 64);
      s.c += __shfl_xor(s.c, d, 64);
    }
    part[b] = acc;
    __syncthreads();
    const int nr = (int)(nblocks + run - 1) / run, k = b / run;
    if (b % run == 0 && k < nr) part[(kMergeThreads * (k + 1) + nr - 1) / nr - 1] = centred(s, r, i, j);
  } else {
    const int64_t a0 = nblocks * threadIdx.x / kMergeThreads, a1 = nblocks * (threadIdx.x + 1) / kMergeThreads;
    for (int64_t b = a0; b < a1; ++b) {
      const double* r = rec + b * kRecWords;
      acc = combine(acc, centred(sums_of(r, i, j), r, i, j));
    }
    part[threadIdx.x] = acc;
  }
  __syncthreads();
  for (int s = kMergeThreads / 2; s >= 1; s >>= 1) {
    if ((int)threadIdx.x < s) part[threadIdx.x] = combine(part[threadIdx.x], part[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double* c = cur + 6 * t;
    const Pair old{c[0], c[1], c[2], c[3], c[4], c[5]};
    const Pair r = combine(old, part[0]);
    double* o = next + 6 * t;
    o[0] = r.n;
    o[1] = r.mi;
    o[2] = r.mj;
    o[3] = r.m2i;
    o[4] = r.m2j;
    o[5] = r.c;
  }
}

__global__ void k_pw_merge_states(const double* a, const double* b, double* out, int T) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const double* x = a + 6 * t;
  const double* y = b + 6 * t;
  const Pair r = combine(Pair{x[0], x[1], x[2], x[3], x[4], x[5]}, Pair{y[0], y[1], y[2], y[3], y[4], y[5]});
  double* o = out + 6 * t;
  o[0] = r.n;
  o[1] = r.mi;
  o[2] = r.mj;
  o[3] = r.m2i;
  o[4] = r.m2j;
  o[5] = r.c;
}

// n, mean (each column over its own present rows), cov and corr (p x p):
// out = [n (p*p) | mean (p) | cov (p*p) | corr (p*p)].
__global__ void k_pw_finalize(const double* st, int p, int ddof, double* out) {
  const int T = p * (p + 1) / 2;
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  int i, j;
  pair_of(p, t, i, j);
  const double* s = st + 6 * t;
  const double n = s[0];
  const double nan = __builtin_nan("");
  double* on = out;
  double* om = out + p * p;
  double* ocov = om + p;
  double* ocorr = ocov + p * p;
  on[i * p + j] = on[j * p + i] = n;
  const double cov = n > (double)ddof ? s[5] / (n - (double)ddof) : nan;
  ocov[i * p + j] = ocov[j * p + i] = cov;
  double corr = nan;
  if (s[3] > 0.0 && s[4] > 0.0) corr = i == j ? 1.0 : s[5] / sqrt(s[3] * s[4]);
  ocorr[i * p + j] = ocorr[j * p + i] = corr;
  if (i == j) om[i] = n > 0.0 ? s[1] : nan;
}

}  // namespace pw

// ---- host ----------------------------------------------------------------------

template <int KIND>
static void go_pairwise(const pw::Args& a, int64_t nblocks, hipStream_t s) {
  const dim3 grid((unsigned)nblocks), block(pw::kThreads);
  if (a.p <= 4) hipLaunchKernelGGL((pw::k_pairwise<KIND, 4>), grid, block, 0, s, a);
  else if (a.p <= 8) hipLaunchKernelGGL((pw::k_pairwise<KIND, 8>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((pw::k_pairwise<KIND, 16>), grid, block, 0, s, a);
}

static void launch_pairwise(const pw::Args& a, int64_t nblocks, hipStream_t s) {
  int n32 = 0;
  for (int c = 0; c < a.p; ++c) n32 += a.dtype[c] == STATS_F32;
  if (n32 == 0) go_pairwise<pw::K_F64>(a, nblocks, s);
  else if (n32 == a.p) go_pairwise<pw::K_F32>(a, nblocks, s);
  else go_pairwise<pw::K_MIX>(a, nblocks, s);
}

int pairwise_state_words(int p) { return 6 * p * (p + 1) / 2; }

int accumulate_pairwise(stats_ctx* h, const void* const* planes, int64_t nrows) {
  const int p = h->p;
  pw::Args a;
  memset(&a, 0, sizeof a);
  a.p = p;
  for (int c = 0; c < p; ++c) {
    const stats_column& col = h->cols[c];
    a.colbase[c] = (const char*)planes[col.plane] + col.byte_offset;
    a.colstride[c] = h->row_stride[col.plane];
    a.dtype[c] = col.dtype;
  }
  const int64_t R = block_rows_for(h, nrows);
  const int64_t max_rows = std::max<int64_t>(R, std::min<int64_t>(16384 * R, ((int64_t)1 << 28) / R * R));
  const int T = p * (p + 1) / 2;
  int64_t done = 0;
  while (done < nrows) {
    const int64_t rows = std::min(nrows - done, max_rows);
    const int64_t nblocks = (rows + R - 1) / R;
    int rc = ensure_dev(h, (void**)&h->rec, &h->rec_cap, (size_t)(nblocks * pw::kRecWords * 8));
    if (rc) return rc;
    pw::Args b = a;
    for (int c = 0; c < p; ++c) b.colbase[c] = a.colbase[c] + done * a.colstride[c];
    b.nrows = rows;
    b.R = R;
    b.shift_low = shift_low_for(h, R);
    b.rec = (double*)h->rec;
    {
      Timer t;
      t.begin(h, STATS_K_ACCUM);
      launch_pairwise(b, nblocks, h->stream);
      t.end();
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(h, e, "pairwise kernel launch");
    {
      Timer t;
      t.begin(h, STATS_K_MERGE);
      hipLaunchKernelGGL(pw::k_pw_merge, dim3((unsigned)T), dim3(pw::kMergeThreads), 0, h->stream,
                         (const double*)h->rec, nblocks, p, (const double*)h->state[h->cur],
                         (double*)h->state[h->cur ^ 1], shift_run(h, R));
      t.end();
    }
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(h, e, "pairwise merge launch");
    h->cur ^= 1;
    done += rows;
  }
  return STATS_OK;
}

void launch_pairwise_merge_states(const uint64_t* a, const uint64_t* b, uint64_t* out, int p, hipStream_t s) {
  const int T = p * (p + 1) / 2;
  hipLaunchKernelGGL(pw::k_pw_merge_states, dim3((T + 255) / 256), dim3(256), 0, s, (const double*)a,
                     (const double*)b, (double*)out, T);
}

}  // namespace st

using namespace st;

extern "C" int stats_finalize_pairwise(stats_ctx* h, int32_t ddof, int64_t* n_out, double* mean_out,
                                       double* cov_out, double* corr_out) {
  if (!h) return fail(STATS_E_ARG, "handle is NULL");
  if (h->poisoned) return fail(STATS_E_STATE, "handle is poisoned by an earlier HIP error");
  if (!(h->flags & STATS_CFG_PAIRWISE)) return fail(STATS_E_STATE, "not a pairwise (missing-value) handle");
  if (ddof < 0) return fail(STATS_E_ARG, "ddof < 0");
  const int p = h->p;
  DeviceGuard g(h->device);
  if (!g.ok) return fail(STATS_E_HIP, "hipSetDevice failed");
  const size_t words = (size_t)3 * p * p + p;
  int rc = ensure_dev(h, (void**)&h->fin_out, &h->fin_out_cap, words * 8);
  if (!rc) rc = ensure_pin(h, &h->pin_out, &h->pin_out_cap, words * 8);
  if (rc) return rc;
  const int T = p * (p + 1) / 2;
  {
    Timer t;
    t.begin(h, STATS_K_FINALIZE);
    hipLaunchKernelGGL(pw::k_pw_finalize, dim3((T + 255) / 256), dim3(256), 0, h->stream,
                       (const double*)h->state[h->cur], p, ddof, h->fin_out);
    t.end();
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(h->pin_out, h->fin_out, words * 8, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_fail(h, e, "pairwise finalize");
  collect_timings(h);
  const double* hn = (const double*)h->pin_out;
  const double* hm = hn + (size_t)p * p;
  const double* hc = hm + p;
  const double* hr = hc + (size_t)p * p;
  for (int k = 0; k < p * p; ++k) {
    if (n_out) n_out[k] = (int64_t)hn[k];
    if (cov_out) cov_out[k] = hc[k];
    if (corr_out) corr_out[k] = hr[k];
  }
  if (mean_out)
    for (int c = 0; c < p; ++c) mean_out[c] = hm[c];
  return STATS_OK;
}
