// Wide tables (p > 32 in FP64 mode, and single blocks of the split mode): block
// statistics with a dense SYRK on the FP64 matrix cores.
//
// For p columns the per-row work is p(p+1)/2 products, a real dense
// contraction X_b^T X_b over the rows of a block (section "Data
// Representation and Sufficient Statistics": X^T X accumulated in one
// streaming pass).  The block record is the same as the narrow path's (shift
// K = the block's first row, S = sum (x - K), Q = sum (x - K)(x - K)^T) and is
// merged by the same kernels.  Exact for integer columns under the same 2^53
// guard as the narrow path.  Split mode (BF16): see wide_split.hip.
//
// Tiling: columns form groups of ST = 64 or 128 (wide_group), cut into 16-column
// strips.  A workgroup owns one block of rows and one pair of groups (A, B), A <= B:
// the upper 16 x 16 tiles of a diagonal pair (at most 36, dealt over eight waves so
// that the two waves of a SIMD share them evenly), or a strip of A per wave (64: per
// two waves) against the strips of B.  Every product's accumulator stays in registers
// for the whole block, so a row is read once for p <= 128.  The next 32 rows' values
// are in flight to registers while the staged ones are multiplied; they are shifted
// into the other half of a double LDS buffer, one barrier per 32 rows.  A thread stages one column, so
// neighbouring lanes read neighbouring columns.
//
// Bound: the matrix cores (64 cycles of a SIMD per 16 x 16 x 4 product; the
// staged operands are half of what LDS can deliver).  4e6 x 101 FP64: 1.18 ms,
// 0.62 of the products' own time; 64-column groups staged element by element
// behind flat loads took 4.0 ms, one workgroup per compute unit 1.8 ms.
// Blocks are mapped to workgroup ids so that all pairs of one block run on the
// same XCD (ids congruent modulo 8), sharing its L2.
#include <type_traits>

#include "common.hpp"
#include "wide.hpp"

namespace st {
namespace wide {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kFThreads = 512;
constexpr int kFWaves = kFThreads / 64;

// Groups of ST columns (64 or 128).
template <int ST>
struct Shape {
  static constexpr int kRowStep = kFThreads / ST;   // rows staged per pass
  static constexpr int kPerThr = KR / kRowStep;     // rows of its column a thread stages
  static constexpr int kStrips = ST / 16;
  // tiles per wave, at most: of a diagonal pair, of another one
  static constexpr int kDiagMax = (kStrips * (kStrips + 1) / 2 + kFWaves - 1) / kFWaves;
  static constexpr int kOffMax = kStrips * kStrips / kFWaves;
};

// A thread's column of one group: element of row r at base + r stride.  KIND: the
// STATS_* type of every column of the launch (0: each column has its own).
template <int KIND>
struct Col {
  const char* base;
  int64_t stride, Ki;
  double K;
  int kind;
  bool valid, chk;
  __device__ inline int type() const { return KIND ? KIND : kind; }
};

// Threads without a column read column 0 and stage zeros.
template <int KIND>
__device__ inline Col<KIND> load_col(const Args& a, int c, int64_t r0) {
  const bool valid = c < a.p;
  const SlotInfo si = a.slots[valid ? c : 0];
  Col<KIND> o{si.base, si.stride, 0, 0.0, si.kind, valid, valid && si.chk};
  const char* p0 = si.base + r0 * si.stride;
  switch (o.type()) {
    case STATS_I32: o.K = (double)load_global<int32_t>(p0); break;
    case STATS_F32: o.K = (double)load_global<float>(p0); break;
    case STATS_I64:
      o.Ki = load_global<int64_t>(p0);
      o.K = (double)o.Ki;
      break;
    default: o.K = load_global<double>(p0); break;
  }
  return o;
}

// Raw values of kPerThr rows, the first at p, step bytes apart (TAIL: rows at or
// past `left` as row left - 1; left > 0).
template <int ST, bool TAIL, int KIND>
__device__ inline void load_raw(const Col<KIND>& c, const char* p, int64_t step, int left, uint64_t (&x)[Shape<ST>::kPerThr]) {
  constexpr int kRowStep = Shape<ST>::kRowStep, kPerThr = Shape<ST>::kPerThr;
  auto at = [&](int i) { return p + (TAIL ? (int64_t)min(kRowStep * i, left - 1) * c.stride : i * step); };
  if (c.type() == STATS_F64 || c.type() == STATS_I64) {
#pragma unroll
    for (int i = 0; i < kPerThr; ++i) x[i] = load_global<uint64_t>(at(i));
  } else {
#pragma unroll
    for (int i = 0; i < kPerThr; ++i) x[i] = load_global<uint32_t>(at(i));
  }
}

// Shifted values to LDS (TAIL: rows at or past `left` as zeros), added to the
// column's sum.
template <int ST, int NC, bool TAIL, int KIND>
__device__ inline void stage(const Col<KIND>& c, const uint64_t (&x)[Shape<ST>::kPerThr], int left, double* out,
                             double& sum, uint32_t& bad) {
  constexpr int kRowStep = Shape<ST>::kRowStep, kPerThr = Shape<ST>::kPerThr;
  double v[kPerThr];
  auto put = [&](auto value) {
    if (c.chk) {
#pragma unroll
      for (int i = 0; i < kPerThr; ++i) bad |= (value(x[i]) != __builtin_rint(value(x[i])));
    }
#pragma unroll
    for (int i = 0; i < kPerThr; ++i) v[i] = value(x[i]) - c.K;
  };
  switch (c.type()) {
    case STATS_F64: put([](uint64_t w) { return __longlong_as_double((long long)w); }); break;
    case STATS_F32: put([](uint64_t w) { return (double)__uint_as_float((uint32_t)w); }); break;
    case STATS_I32: put([](uint64_t w) { return (double)(int32_t)(uint32_t)w; }); break;
    default:
#pragma unroll
      for (int i = 0; i < kPerThr; ++i) v[i] = (double)((int64_t)x[i] - c.Ki);
  }
#pragma unroll
  for (int i = 0; i < kPerThr; ++i) {
    if (!c.valid || (TAIL && kRowStep * i >= left)) v[i] = 0.0;
    out[kRowStep * i * NC] = v[i];
    sum += v[i];
  }
}

// Column c's shift as the record holds it.
template <int KIND>
__device__ inline uint64_t shift_word(const Args& a, int c, const Col<KIND>& col) {
  if (!a.slots[c].isint) return (uint64_t)__double_as_longlong(col.K);
  if (col.type() == STATS_I64) return (uint64_t)col.Ki;
  return (fabs(col.K) < 4.0e18) ? (uint64_t)(int64_t)col.K : (uint64_t)0x7FFFFFFFFFFFFFFFll;
}

// One block of rows [r0, r1) and pair of groups (A, B), DIAG: A == B: this
// pair's part of the record at out.  lds: 2 KR NC doubles, NC = ST (DIAG) or
// 2 ST.  Every thread of the workgroup.
template <int ST, bool DIAG, int KIND>
__device__ inline void wide_f64_block(const Args& a, uint64_t* out, int64_t r0, int64_t r1, int A, int B,
                                      double* lds) {
  constexpr int NC = DIAG ? ST : 2 * ST;
  constexpr int NG = DIAG ? 1 : 2;
  constexpr int kRowStep = Shape<ST>::kRowStep, kPerThr = Shape<ST>::kPerThr, kStrips = Shape<ST>::kStrips;
  constexpr int NT = DIAG ? Shape<ST>::kDiagMax : Shape<ST>::kOffMax;
  const int tid = threadIdx.x, lane = tid & 63, p = a.p;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int my_c = tid % ST, my_r = tid / ST;
  Col<KIND> col[NG];
  const char* pn[NG];  // this thread's first row of the next stage to load
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    col[g] = load_col<KIND>(a, (g ? B : A) * ST + my_c, r0);
    pn[g] = col[g].base + (r0 + my_r) * col[g].stride;
  }
  // this wave's tiles: LDS columns of their operands
  const int sa = min(kStrips, (p - A * ST + 15) / 16), sb = min(kStrips, (p - B * ST + 15) / 16);
  int ta[NT] = {}, tb[NT] = {}, nt = 0;
  if constexpr (DIAG) {
    int t = 0;
    for (int i = 0; i < sa; ++i)
      for (int j = i; j < sa; ++j, ++t)
        if (t % kFWaves == wave) {
#pragma unroll
          for (int u = 0; u < NT; ++u)
            if (u == nt) {
              ta[u] = i;
              tb[u] = j;
            }
          ++nt;
        }
  } else {
    const int b0 = wave / kStrips * NT;  // 64 columns: two waves a strip of A
    nt = wave % kStrips < sa ? max(min(sb - b0, NT), 0) : 0;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      ta[u] = wave % kStrips;
      tb[u] = b0 + u;
    }
  }
  d4 acc[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) acc[u] = (d4){0.0, 0.0, 0.0, 0.0};
  double sum[NG] = {};
  uint32_t bad = 0;
  uint64_t x[NG][kPerThr];
  double* const st0 = lds + my_r * NC + my_c;
  const double* const rd0 = lds + (lane >> 4) * NC + (lane & 15);
  const int64_t nst = (r1 - r0) / KR;               // whole stages
  const int left = (int)(r1 - r0 - nst * KR) - my_r;  // this thread's rows after them: while kRowStep i < left
  // the next stage's rows into registers / from registers into half h
  auto fetch = [&](auto tail) {
    constexpr bool TAIL = decltype(tail)::value;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      // a thread with no row left re-reads the block's last one
      const char* p = TAIL && left <= 0 ? col[g].base + (r1 - 1) * col[g].stride : pn[g];
      load_raw<ST, TAIL>(col[g], p, kRowStep * col[g].stride, max(left, 1), x[g]);
      pn[g] += KR * col[g].stride;
    }
  };
  auto put = [&](auto tail, int h) {
#pragma unroll
    for (int g = 0; g < NG; ++g)
      stage<ST, NC, decltype(tail)::value>(col[g], x[g], left, st0 + h * KR * NC + g * ST, sum[g], bad);
  };
  constexpr std::false_type whole{};
  constexpr std::true_type tail{};
  if (nst > 0) {
    fetch(whole);
    put(whole, 0);
  }
  __syncthreads();
  // The stages with N tiles for this wave: a loop of its own per count, so that
  // operand reads and products schedule without branches (the waves of a
  // workgroup meet at the same barriers whatever their counts).
  auto run = [&](auto n_c) {
    constexpr int N = decltype(n_c)::value;
    auto products = [&](int h) {
      const double* rd = rd0 + h * KR * NC;
      constexpr int kAhead = DIAG ? 4 : 2;  // steps whose operands are read together
#pragma unroll kAhead
      for (int k4 = 0; k4 < KR / 4; ++k4) {
        double av[NT], bv[NT];
#pragma unroll
        for (int u = 0; u < N; ++u) {
          if (DIAG || u == 0) av[u] = rd[4 * k4 * NC + 16 * ta[u]];
          bv[u] = rd[4 * k4 * NC + (NG - 1) * ST + 16 * tb[u]];
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
          acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[DIAG ? u : 0], bv[u], acc[u], 0, 0, 0);
      }
    };
    int half = 0;
    for (int64_t t = 0; t < nst; ++t) {
      if (t + 1 < nst) fetch(whole);
      products(half);
      half ^= 1;
      if (t + 1 < nst) put(whole, half);
      __syncthreads();
    }
    if (r0 + nst * KR < r1) {
      fetch(tail);
      put(tail, half);
      __syncthreads();
      products(half);
      __syncthreads();
    }
  };
  using std::integral_constant;
  if constexpr (NT == 2) {
    if (nt == 0) run(integral_constant<int, 0>{});
    else if (nt == 1) run(integral_constant<int, 1>{});
    else run(integral_constant<int, 2>{});
  } else if constexpr (DIAG) {
    switch (nt) {
      case 0: run(integral_constant<int, 0>{}); break;
      case 1: run(integral_constant<int, 1>{}); break;
      case 2: run(integral_constant<int, 2>{}); break;
      case 3: run(integral_constant<int, 3>{}); break;
      case 4: run(integral_constant<int, 4>{}); break;
      default: run(integral_constant<int, 5>{}); break;
    }
  } else {  // strips past sb are staged as zeros
    if (nt == 0) run(integral_constant<int, 0>{});
    else if (nt == 1) run(integral_constant<int, 1>{});
    else if (nt <= 4) run(integral_constant<int, 4>{});
    else run(integral_constant<int, 8>{});
  }
  if (bad) atomicOr(&a.status->bits, ST_INEXACT);

  // ---- this pair's part of the block record ----
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    if (u >= nt) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // register r of lane l holds D[4 r + l / 16][l % 16]
      const int ga = A * ST + 16 * ta[u] + 4 * r + (lane >> 4), gb = B * ST + 16 * tb[u] + (lane & 15);
      if (ga <= gb && gb < p) out[2 + 2 * p + tri(p, ga, gb)] = (uint64_t)__double_as_longlong(acc[u][r]);
    }
  }
  if constexpr (DIAG) {
    // column sums: the row groups in order
    double* s_sum = lds;
    s_sum[my_r * ST + my_c] = sum[0];
    __syncthreads();
    const int c = A * ST + my_c;
    if (my_r == 0 && c < p) {
      double s = 0.0;
      for (int g = 0; g < kRowStep; ++g) s += s_sum[g * ST + my_c];
      out[2 + p + c] = (uint64_t)__double_as_longlong(s);
      out[2 + c] = shift_word(a, c, col[0]);
    }
    if (A == 0 && tid == 0) {
      out[0] = (uint64_t)(r1 - r0);
      out[1] = 0;
    }
  }
}

// Block and tile of a workgroup id: all tiles of one block on one XCD.
__device__ inline bool block_of_id(int64_t nblocks, int nt, int64_t* b, int* t) {
  const int64_t id = blockIdx.x, y = id / 8;
  *t = (int)(y % nt);
  *b = (y / nt) * 8 + id % 8;
  return *b < nblocks;
}

// The diagonal pairs (tiles[0 .. ng)) or the others (tiles[ng .. ntiles)) of
// every block; with ovf only of the flagged blocks.
template <int ST, bool DIAG, int KIND>
__global__ __launch_bounds__(kFThreads, DIAG || ST == 64 ? 4 : 2) void k_wide_f64(Args a, const int* ovf) {
  extern __shared__ double s_lds[];
  const int ng = (a.p + ST - 1) / ST;
  int64_t b;
  int t;
  if (!block_of_id(a.nblocks, DIAG ? ng : a.ntiles - ng, &b, &t) || (ovf && !ovf[b])) return;
  const int2 tile = a.tiles[DIAG ? t : ng + t];
  const int64_t r0 = b * a.R, r1 = min(r0 + a.R, a.nrows);
  wide_f64_block<ST, DIAG, KIND>(a, a.rec + b * rec_words(a.p), r0, r1, tile.x, tile.y, s_lds);
}

// Persistent variant for batched groups: workgroups take (row tile, pair)
// items from an atomic queue until it is empty; record slots are indexed by
// row tile, so results do not depend on which workgroup ran what.
template <int ST>
__global__ __launch_bounds__(kFThreads) void k_seg_f64(Args a, SegArgs g) {
  extern __shared__ double s_lds[];
  __shared__ int64_t s_item;
  const int64_t nitems = *g.nrowtiles * a.ntiles;
  for (;;) {
    __syncthreads();  // previous item's LDS use is over
    if (threadIdx.x == 0) s_item = (int64_t)atomicAdd(g.counter, 1ull);
    __syncthreads();
    const int64_t item = s_item;
    if (item >= nitems) break;
    const int64_t rt = item / a.ntiles;
    const int2 pair = a.tiles[item % a.ntiles];
    const SegTile tile = g.rowtiles[rt];
    uint64_t* out = a.rec + rt * rec_words(a.p);
    // (a table of groups of 128 is one group: wide_group)
    if (ST == 128 || pair.x == pair.y) wide_f64_block<ST, true, 0>(a, out, tile.r0, tile.r1, pair.x, pair.y, s_lds);
    else if constexpr (ST == 64) wide_f64_block<ST, false, 0>(a, out, tile.r0, tile.r1, pair.x, pair.y, s_lds);
  }
}

__global__ void k_zero_counter(unsigned long long* c) { *c = 0ull; }

}  // namespace wide

void wide_pairs(int p, int group, std::vector<int2>* tiles) {
  const int ng = (p + group - 1) / group;
  tiles->clear();
  for (int A = 0; A < ng; ++A) tiles->push_back(make_int2(A, A));
  for (int A = 0; A < ng; ++A)
    for (int B = A + 1; B < ng; ++B) tiles->push_back(make_int2(A, B));
}

// Column groups of the FP64 kernel.  65 to 128 columns are one group of 128 (every row
// read once).  Up to 64, half of such a group's threads would stage nothing (a call on
// 10^6 x 33 FP64 306 us, 156 in groups of 64).  Above 128, groups of 64 spread a block
// over more workgroups, each with a shorter chain of products, and pad less where
// their number is odd (5000 x 200 444 and 280 us, 4*10^6 x 160 4.6 and 3.3 ms); with as
// much padding and workgroups in plenty, groups of 128 read less (4*10^6 x 200 FP32 6.4
// and 6.7 ms, 200,000 x 1000 6.0 and 6.5).
int wide_group(int p, int64_t nblocks) {
  const int n64 = (p + 63) / 64, n128 = (p + 127) / 128;
  if (n64 == 2) return 128;
  return n64 % 2 || nblocks * n128 * (n128 + 1) / 2 <= 1024 ? 64 : 128;
}

// LDS of a pair: two stages of one group (diagonal) or two.
static constexpr size_t diag_lds(int group) { return sizeof(double) * 2 * wide::KR * group; }

static hipError_t allow_lds(const void* fn, size_t bytes) {
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int ST, int KIND>
static void go_wide(const wide::Args& a, const int* ovf, hipStream_t s) {
  const int64_t nb8 = (a.nblocks + 7) / 8 * 8;
  const int ng = (a.p + ST - 1) / ST;
  const dim3 block(wide::kFThreads);
  hipLaunchKernelGGL((wide::k_wide_f64<ST, true, KIND>), dim3((unsigned)(nb8 * ng)), block, diag_lds(ST), s, a, ovf);
  if (a.ntiles > ng) {
    (void)allow_lds((const void*)wide::k_wide_f64<ST, false, KIND>, 2 * diag_lds(ST));
    hipLaunchKernelGGL((wide::k_wide_f64<ST, false, KIND>), dim3((unsigned)(nb8 * (a.ntiles - ng))), block, 2 * diag_lds(ST), s, a, ovf);
  }
}

// kind: the STATS_* type of every column, or 0.  FP64 tables have an instance
// of their own (types told apart per thread cost the registers of a second
// workgroup per compute unit).
void launch_wide_f64(const wide::Args& a, int group, int kind, const int* ovf, hipStream_t s) {
  if (group == 64) {
    if (kind == STATS_F64) go_wide<64, STATS_F64>(a, ovf, s);
    else go_wide<64, 0>(a, ovf, s);
  } else {
    if (kind == STATS_F64) go_wide<128, STATS_F64>(a, ovf, s);
    else go_wide<128, 0>(a, ovf, s);
  }
}

void launch_seg(const wide::Args& a, const wide::SegArgs& g, int nwg, hipStream_t s) {
  const int group = wide_group(a.p, 0);
  const size_t lds = diag_lds(group) * (a.p > group ? 2 : 1);
  hipLaunchKernelGGL(wide::k_zero_counter, dim3(1), dim3(1), 0, s, g.counter);
  if (group == 64) {
    (void)allow_lds((const void*)wide::k_seg_f64<64>, lds);
    hipLaunchKernelGGL(wide::k_seg_f64<64>, dim3(nwg), dim3(wide::kFThreads), lds, s, a, g);
  } else {
    (void)allow_lds((const void*)wide::k_seg_f64<128>, lds);
    hipLaunchKernelGGL(wide::k_seg_f64<128>, dim3(nwg), dim3(wide::kFThreads), lds, s, a, g);
  }
}

}  // namespace st
