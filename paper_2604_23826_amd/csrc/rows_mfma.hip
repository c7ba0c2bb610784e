// Tables of up to 32 columns in any layout on the FP64 matrix cores, with
// every lane loading its own column (no staging, no layout or alignment rule).
//
// Serves batched groups of p <= 32 columns whose records are not the 256-byte
// ones of seg_aos64.hip, and plain tables: p <= 16 columns interleaved in one
// plane that is not 16-byte packed FP64 (FP32 rows, mixed types, odd strides),
// and 17 <= p <= 32 columns in FP64 mode.
//
// Work split: an item is a block of rows (a row tile of a group, or block k of
// a plain table).  In v_mfma_f64_16x16x4 a lane holds column (lane % 16) of
// row (lane / 16) of a 4-row step, at once its element of the A operand
// (column i, row k) and of the B operand (row k, column j); so lane l loads
// exactly that element, straight into the register the product reads.  A
// step's elements of a row-major table are consecutive rows: one coalesced
// load.  Up to 8 (4) columns, two (four) groups of 4 rows share a product,
// each in its own 8 (4) operand columns; only the diagonal blocks of the
// result are kept.  Each wave takes kU consecutive steps of a stage and has
// the next stage's loads in flight while it multiplies the current one.  Rows
// past the last whole stage take one masked stage (clamped row, zero operand).
// Columns 16..31 are a second load per step and two more products (upper
// 16 x 16 tiles (0,0), (0,1), (1,1)).
//
// Bound: a product occupies its SIMD for 64 cycles, so the chip takes 1.5e11
// rows/s at 9..16 columns (3e11 to 8, 6e11 to 4, 5e10 from 17): above HBM's
// rate for FP64 rows and for FP32 rows of 12 columns and more.  Measured per
// pass (accumulate and finish): 4096 groups of 100..10,000 ten-column FP64 rows
// (0.7 GB) 1529 -> 520 us against staging through LDS element by element, of it
// 199 in this kernel (3.6 TB/s; the smallest tile is more than a workgroup's share);
// 4e6 rows of 12 FP32 columns 416 -> 139 us against a row per lane, of it 58 in
// this kernel: 3.3 TB/s, the products (27 us) and their loads' latency.
#include "accum_common.hpp"
#include "wide.hpp"

namespace st {
namespace rowsm {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kU = 8;             // 4-row steps per wave and stage

// Columns per row group W = 16 / PK; rows per step and per stage.
template <int PK> struct Shape {
  static constexpr int W = 16 / PK;
  static constexpr int kStep = 4 * PK;
  static constexpr int kSR = 4 * kU * kStep;
};

// Element types of a launch: all columns of one type, or any mixture.
enum { K_F64 = 0, K_F32 = 1, K_I32 = 2, K_MIX = 3 };

template <int KIND> struct Raw;
template <> struct Raw<K_F64> { typedef double type; };
template <> struct Raw<K_F32> { typedef float type; };
template <> struct Raw<K_I32> { typedef int32_t type; };
template <> struct Raw<K_MIX> { typedef uint2 type; };

// One lane's column: element of row r at base + r stride.
struct Col {
  const char* base;
  int64_t stride;
  int dt;
  bool valid, chk, isint;
  double K;
  int64_t Ki;  // shift of an int64 column (subtracted as an integer)
};

template <int KIND>
__device__ inline typename Raw<KIND>::type load_raw(const Col& c, const char* p) {
  if constexpr (KIND == K_MIX) {
    // two words; the second re-reads the first for 4-byte types
    const int hoff = (c.dt == STATS_I64 || c.dt == STATS_F64) ? 4 : 0;
    return make_uint2(load_global<uint32_t>(p), load_global<uint32_t>(p + hoff));
  } else {
    return load_global<typename Raw<KIND>::type>(p);
  }
}

// Value minus shift.
template <int KIND>
__device__ inline double shifted(const Col& c, typename Raw<KIND>::type x) {
  if constexpr (KIND == K_MIX) return acc::convert(c.dt, x.x, x.y, c.K, c.Ki);
  else return (double)x - c.K;
}

template <int KIND>
__device__ inline double value(const Col& c, typename Raw<KIND>::type x) {
  if constexpr (KIND == K_MIX) return acc::convert(c.dt, x.x, x.y, 0.0, 0);
  else return (double)x;
}

template <int KIND>
__device__ inline void set_shift(Col& c, int64_t rk) {
  const typename Raw<KIND>::type x = load_raw<KIND>(c, c.base + rk * c.stride);
  c.Ki = 0;
  if constexpr (KIND == K_MIX) {
    if (c.dt == STATS_I64) {
      c.Ki = (int64_t)(((uint64_t)x.y << 32) | x.x);
      c.K = (double)c.Ki;
      return;
    }
  }
  c.K = value<KIND>(c, x);
}

template <int NT>
struct Smem {
  static constexpr int kTiles = NT == 2 ? 3 : 1;
  double acc[4][kTiles][4][64];  // per wave: tiles x registers x lanes
  double s[4][64][NT];           // per wave and lane: column sums
};

// Record of rows [r0, r1), r0 < r1, shifted by row rk, at out.  Every thread of the workgroup.
// A non-integer value of a checked column sets the record's flag word and, with
// status, the handle's status.
template <int KIND, int NT, int PK>
__device__ inline void rows_block(Col (&col)[NT], int p, int64_t r0, int64_t r1, int64_t rk, uint64_t* out,
                                  Smem<NT>& sm, DevStatus* status) {
  static_assert(NT == 1 || PK == 1, "row groups share a product only within 16 columns");
  typedef typename Raw<KIND>::type T;
  constexpr int kTiles = Smem<NT>::kTiles;
  constexpr int W = Shape<PK>::W, kStep = Shape<PK>::kStep, kSR = Shape<PK>::kSR;
  const int tid = threadIdx.x, lane = tid & 63, q16 = lane & 15, wave = tid >> 6;
  const int rl = (lane >> 4) + 4 * (q16 / W);  // this lane's row of a step
  d4 acc[kTiles];
#pragma unroll
  for (int t = 0; t < kTiles; ++t) acc[t] = (d4){0.0, 0.0, 0.0, 0.0};
  double S[NT];
  uint32_t bad = 0;
  const char* pc[NT];    // this lane's element of step 0 of the next stage to load
  int64_t s4[NT], sst[NT];
#pragma unroll
  for (int h = 0; h < NT; ++h) {
    S[h] = 0.0;
    pc[h] = col[h].base + (r0 + kU * kStep * wave + rl) * col[h].stride;
    s4[h] = kStep * col[h].stride;
    sst[h] = (int64_t)kSR * col[h].stride;
  }
  auto load = [&](T (&x)[kU][NT]) {
#pragma unroll
    for (int s = 0; s < kU; ++s)
#pragma unroll
      for (int h = 0; h < NT; ++h) x[s][h] = load_raw<KIND>(col[h], pc[h] + s * s4[h]);
#pragma unroll
    for (int h = 0; h < NT; ++h) pc[h] += sst[h];
  };
  bool anychk = false;
#pragma unroll
  for (int h = 0; h < NT; ++h) anychk |= col[h].chk;
  const bool chk = __builtin_amdgcn_ballot_w64(anychk) != 0;
  // products of one stage; rows at or past `rows` (relative to this wave's
  // first) contribute nothing
  auto use = [&](const T (&x)[kU][NT], int rows) {
#pragma unroll
    for (int s = 0; s < kU; ++s) {
      double v[NT];
#pragma unroll
      for (int h = 0; h < NT; ++h) {
        const bool on = col[h].valid && kStep * s + rl < rows;
        const double d = shifted<KIND>(col[h], x[s][h]);
        v[h] = on ? d : 0.0;
        if (chk && on && col[h].chk) bad |= acc::not_integer(value<KIND>(col[h], x[s][h]));
        S[h] += v[h];
      }
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0], v[0], acc[0], 0, 0, 0);
      if constexpr (NT == 2) {
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0], v[1], acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1], v[1], acc[2], 0, 0, 0);
      }
    }
  };
  const int64_t nst = (r1 - r0) / kSR;  // whole stages
  constexpr int kAll = kU * kStep;
  T xa[kU][NT], xb[kU][NT];
  if (nst > 0) load(xa);
#pragma unroll
  for (int h = 0; h < NT; ++h) set_shift<KIND>(col[h], rk);
  for (int64_t t = 0; t < nst; t += 2) {
    if (t + 1 < nst) load(xb);
    use(xa, kAll);
    if (t + 1 < nst) {
      if (t + 2 < nst) load(xa);
      use(xb, kAll);
    }
  }
  const int64_t rb = r0 + nst * kSR + kAll * wave;  // this wave's rows of the last stage
  if (rb < r1) {
    const int rows = (int)min((int64_t)kAll, r1 - rb);
#pragma unroll
    for (int s = 0; s < kU; ++s)
#pragma unroll
      for (int h = 0; h < NT; ++h)
        xa[s][h] = load_raw<KIND>(col[h], col[h].base + (rb + min(kStep * s + rl, rows - 1)) * col[h].stride);
    use(xa, rows);
  }

  // fixed-order sum over the waves; record
#pragma unroll
  for (int t = 0; t < kTiles; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) sm.acc[wave][t][r][lane] = acc[t][r];
#pragma unroll
  for (int h = 0; h < NT; ++h) sm.s[wave][lane][h] = S[h];
  const int anybad = __syncthreads_or((int)bad);
  for (int e = tid; e < kTiles * W * W; e += kThreads) {
    const int t = e / (W * W), i = e / W % W, j = e % W;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int g = 0; g < PK; ++g) {
        // D[a][b] is register a / 4 of lane 16 (a % 4) + b
        const int da = g * W + i, db = g * W + j;
        v += sm.acc[w][t][da >> 2][16 * (da & 3) + db];
      }
    const int ci = t == 2 ? 16 + i : i, cj = t == 0 ? j : 16 + j;
    if (ci <= cj && cj < p) out[2 + 2 * p + tri(p, ci, cj)] = (uint64_t)__double_as_longlong(v);
  }
  if (tid < W) {  // lanes 0..W-1 of wave 0 hold the columns' shifts
#pragma unroll
    for (int h = 0; h < NT; ++h) {
      const int c = 16 * h + q16;
      if (c >= p) continue;
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int k = 0; k < 4 * PK; ++k) t += sm.s[w][q16 + W * k][h];
      out[2 + p + c] = (uint64_t)__double_as_longlong(t);
      const double Kc = col[h].K;
      uint64_t kw = (uint64_t)__double_as_longlong(Kc);
      if (col[h].isint) {
        if (col[h].dt == STATS_I64) kw = (uint64_t)col[h].Ki;
        else kw = (fabs(Kc) < 4.0e18) ? (uint64_t)(int64_t)Kc : (uint64_t)0x7FFFFFFFFFFFFFFFll;
      }
      out[2 + c] = kw;
    }
  }
  if (tid == 0) {
    out[0] = (uint64_t)(r1 - r0);
    out[1] = anybad ? 1u : 0u;
    if (anybad && status) atomicOr(&status->bits, ST_INEXACT);
  }
}

// Column c of the launch's slot table; lanes without a column read column 0
// (the same addresses as lane 0's row) and contribute zeros.
__device__ inline Col col_of_slot(const wide::SlotInfo* slots, int p, int c) {
  const wide::SlotInfo si = slots[c < p ? c : 0];
  return Col{si.base, si.stride, si.kind, c < p, c < p && si.chk, (bool)si.isint, 0.0, 0};
}

// Items (row tiles of groups, or uniform blocks) from an atomic queue.
template <int KIND, int NT, int PK>
__global__ __launch_bounds__(kThreads) void k_seg_rows(wide::Args a, wide::SegArgs g) {
  __shared__ Smem<NT> sm;
  __shared__ int64_t s_item;
  Col col[NT];
#pragma unroll
  for (int h = 0; h < NT; ++h) col[h] = col_of_slot(a.slots, a.p, 16 * h + (int)(threadIdx.x % Shape<PK>::W));
  const int64_t nitems = g.tile_rows ? (g.total_rows + g.tile_rows - 1) / g.tile_rows : *g.nrowtiles;
  for (;;) {
    __syncthreads();  // previous item's LDS use is over
    if (threadIdx.x == 0) s_item = (int64_t)atomicAdd(g.counter, 1ull);
    __syncthreads();
    const int64_t item = s_item;
    if (item >= nitems) break;
    int64_t r0, r1;
    if (g.tile_rows) {
      r0 = item * g.tile_rows;
      r1 = min(r0 + g.tile_rows, g.total_rows);
    } else {
      const wide::SegTile tile = g.rowtiles[item];
      r0 = tile.r0;
      r1 = tile.r1;
    }
    rows_block<KIND, NT, PK>(col, a.p, r0, r1, shift_row(r0, g.shift_low), a.rec + item * rec_words(a.p), sm, a.status);
  }
}

__global__ void k_zero_queue(unsigned long long* c) { *c = 0ull; }

// Plain table of p <= 16 columns, descriptors in the kernel arguments (no
// device table, so no call needs memory of its own): one block per workgroup,
// slots in column order.
template <int KIND, int PK>
__global__ __launch_bounds__(kThreads) void k_rows(acc::Args a, int p) {
  __shared__ Smem<1> sm;
  const int c = (int)(threadIdx.x % Shape<PK>::W), cc = c < p ? c : 0;
  Col col[1] = {Col{a.colbase[cc], a.colstride[cc], a.dtype[cc], c < p, c < p && ((a.chkmask >> cc) & 1u),
                    (bool)((a.intmask >> cc) & 1u), 0.0, 0}};
  const int64_t r0 = (int64_t)blockIdx.x * a.R, r1 = min(r0 + a.R, a.nrows);
  rows_block<KIND, 1, PK>(col, p, r0, r1, shift_row(r0, a.shift_low), a.rec + (int64_t)blockIdx.x * rec_words(p), sm, nullptr);
}

}  // namespace rowsm

// Launch type of columns of the given STATS_* types.
static int rows_kind(const int32_t* dt, int p) {
  for (int c = 1; c < p; ++c)
    if (dt[c] != dt[0]) return rowsm::K_MIX;
  switch (dt[0]) {
    case STATS_F64: return rowsm::K_F64;
    case STATS_F32: return rowsm::K_F32;
    case STATS_I32: return rowsm::K_I32;
    default: return rowsm::K_MIX;
  }
}

template <int KIND>
static void go_seg(const wide::Args& a, const wide::SegArgs& g, int nwg, hipStream_t s) {
  const dim3 grid(nwg), block(rowsm::kThreads);
  if (a.p <= 4) hipLaunchKernelGGL((rowsm::k_seg_rows<KIND, 1, 4>), grid, block, 0, s, a, g);
  else if (a.p <= 8) hipLaunchKernelGGL((rowsm::k_seg_rows<KIND, 1, 2>), grid, block, 0, s, a, g);
  else if (a.p <= 16) hipLaunchKernelGGL((rowsm::k_seg_rows<KIND, 1, 1>), grid, block, 0, s, a, g);
  else hipLaunchKernelGGL((rowsm::k_seg_rows<KIND, 2, 1>), grid, block, 0, s, a, g);
}

void launch_seg_rows(const wide::Args& a, const wide::SegArgs& g, const int32_t* dtypes, int nwg, hipStream_t s) {
  hipLaunchKernelGGL(rowsm::k_zero_queue, dim3(1), dim3(1), 0, s, g.counter);
  switch (rows_kind(dtypes, a.p)) {
    case rowsm::K_F64: go_seg<rowsm::K_F64>(a, g, nwg, s); break;
    case rowsm::K_F32: go_seg<rowsm::K_F32>(a, g, nwg, s); break;
    case rowsm::K_I32: go_seg<rowsm::K_I32>(a, g, nwg, s); break;
    default: go_seg<rowsm::K_MIX>(a, g, nwg, s); break;
  }
}

template <int KIND>
static void go_rows(const acc::Args& a, int p, int64_t nblocks, hipStream_t s) {
  const dim3 grid((unsigned)nblocks), block(rowsm::kThreads);
  if (p <= 4) hipLaunchKernelGGL((rowsm::k_rows<KIND, 4>), grid, block, 0, s, a, p);
  else if (p <= 8) hipLaunchKernelGGL((rowsm::k_rows<KIND, 2>), grid, block, 0, s, a, p);
  else hipLaunchKernelGGL((rowsm::k_rows<KIND, 1>), grid, block, 0, s, a, p);
}

void launch_rows(const acc::Args& a, int p, int64_t nblocks, hipStream_t s) {
  switch (rows_kind(a.dtype, p)) {
    case rowsm::K_F64: go_rows<rowsm::K_F64>(a, p, nblocks, s); break;
    case rowsm::K_F32: go_rows<rowsm::K_F32>(a, p, nblocks, s); break;
    case rowsm::K_I32: go_rows<rowsm::K_I32>(a, p, nblocks, s); break;
    default: go_rows<rowsm::K_MIX>(a, p, nblocks, s); break;
  }
}

}  // namespace st
