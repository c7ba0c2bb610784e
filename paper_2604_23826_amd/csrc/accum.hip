// Host dispatch of the narrow-table reduction (p <= 16): picks the layout
// class, permutes columns into the kernel's slot order and tells the kernel
// where each slot's results go in the block record.
#include <cstring>

#include "accum_impl.hpp"

namespace st {

// Whether the columns are interleaved in one plane (row-major records): equal
// strides, all of several columns of a row within one stride.  Then the elements of
// a few rows are contiguous, which the kernel with a column per lane loads whole; a
// row per lane (k_generic) touches a line per lane and element there, and is
// kept for columns in separate planes, where it loads contiguous elements, and for
// rows of one or two elements, where most lanes would have none: a single column
// (200 million rows of a dense FP32 or int64 plane: 283 against 607 us, 350 against
// 899) and two of different types, loaded as two words each, in rows of up to 16
// bytes (100 million rows of int32 and FP32: 339 against 530 us, of int64 and FP64
// 517 against 556; FP32 twice 347 against 331, int64 twice 517 against 488, int32
// and FP32 in 32-byte rows 989 against 616).
static bool interleaved(const AccumLaunch& L) {
  if (L.p == 1) return false;
  if (L.p == 2 && L.colstride[0] <= 16 && L.dtype[0] != L.dtype[1]) return false;
  const char *lo = L.colbase[0], *hi = L.colbase[0];
  for (int c = 1; c < L.p; ++c) {
    if (L.colstride[c] != L.colstride[0]) return false;
    lo = L.colbase[c] < lo ? L.colbase[c] : lo;
    hi = L.colbase[c] > hi ? L.colbase[c] : hi;
  }
  return hi - lo < L.colstride[0];
}

bool lane_kernel(const AccumLaunch& L) { return L.kind == 0 && interleaved(L); }

int64_t launch_accum_small_p(const AccumLaunch& L, hipStream_t s) {
  const int p = L.p;
  if (p < 1 || p > 16) return -1;
  const int64_t nblocks = (L.nrows + L.block_rows - 1) / L.block_rows;
  if (nblocks <= 0) return 0;
  // slot order: for dense int32/FP64 planes, int32 columns first
  int perm[16];
  int ni = -1;
  int kind = L.kind == 1 ? ACC_AOS : (L.kind == 2 ? ACC_PLANES : ACC_GENERIC);
  if (kind == ACC_PLANES) {
    bool ok = true;
    for (int c = 0; c < p; ++c) ok = ok && (L.dtype[c] == STATS_I32 || L.dtype[c] == STATS_F64);
    if (ok) {
      int k = 0;
      for (int c = 0; c < p; ++c)
        if (L.dtype[c] == STATS_I32) perm[k++] = c;
      ni = k;
      for (int c = 0; c < p; ++c)
        if (L.dtype[c] == STATS_F64) perm[k++] = c;
    } else {
      kind = ACC_GENERIC;
    }
  }
  if (kind != ACC_PLANES)
    for (int c = 0; c < p; ++c) perm[c] = c;
  acc::Args a;
  memset(&a, 0, sizeof a);
  for (int sl = 0; sl < 16; ++sl) {
    const int c = sl < p ? perm[sl] : 0;
    a.colbase[sl] = sl < p ? L.colbase[c] : nullptr;
    a.colstride[sl] = sl < p ? L.colstride[c] : 0;
    a.dtype[sl] = sl < p ? L.dtype[c] : STATS_F64;
    if (sl < p && ((L.intmask >> c) & 1u)) a.intmask |= 1u << sl;
    if (sl < p && ((L.chkmask >> c) & 1u)) a.chkmask |= 1u << sl;
    a.kdst[sl] = (int8_t)(sl < p ? c : 0);
  }
  for (int e = 0; e < p; ++e) a.dst[e] = (int16_t)perm[e];
  int e = p;
  for (int x = 0; x < p; ++x)
    for (int y = x; y < p; ++y) {
      const int i = perm[x] < perm[y] ? perm[x] : perm[y];
      const int j = perm[x] < perm[y] ? perm[y] : perm[x];
      a.dst[e++] = (int16_t)(p + tri(p, i, j));
    }
  a.nrows = L.nrows;
  a.R = L.block_rows;
  a.shift_low = L.shift_low;
  a.rec = L.rec;
  if (kind != ACC_PLANES && (kind == ACC_GENERIC || L.nrows <= kLaneRows) && interleaved(L)) {
    launch_rows(a, p, nblocks, s);
    return nblocks;
  }
  switch (p) {
#define ST_CASE(PP) \
  case PP: launch_accum_p<PP>(a, kind, ni, nblocks, s); break;
    ST_CASE(1) ST_CASE(2) ST_CASE(3) ST_CASE(4) ST_CASE(5) ST_CASE(6) ST_CASE(7) ST_CASE(8)
    ST_CASE(9) ST_CASE(10) ST_CASE(11) ST_CASE(12) ST_CASE(13) ST_CASE(14) ST_CASE(15) ST_CASE(16)
#undef ST_CASE
  }
  return nblocks;
}

}  // namespace st
