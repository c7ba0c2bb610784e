// Text ingest fused with the reduction (p <= 16).
//
// The data start as CSV text (section "Validation and Infrastructure
// Testing"; section "Data Representation and Sufficient Statistics" on the
// cost of repeated parsing).  Here a chunk of text in HBM is parsed once, on
// the GPU, and every parsed row goes straight into the same shifted column
// sums and X^T X accumulators as the binary path; nothing is written back.
//
// Work split: workgroup w owns the lines whose first byte lies in
// [w seg, (w + 1) seg), seg a multiple of 4096 up to 40 KiB chosen per chunk
// from its mean line length (pick_text_seg); its threads find the line starts
// of their slices, then take the lines in turn, one per thread and round.  The
// workgroup stages its bytes (plus MAXLINE bytes of the next segment, for lines
// that run past the end) in LDS.  The block shift is the workgroup's first line.
//
// What bounds the kernels: instructions, 45 to 90 vector instructions a short
// integer field and some 300 a 17-digit decimal one, at two to three waves per
// SIMD (the text and the parsed rows fill LDS).  8 million ten-column Table-1
// lines (458 MB): 1050 us in the kernel with the fields unrolled (78 KiB of
// code) and a corrected FP64 division per decimal field, 525 us as it is;
// conversion of 2 million lines of eight decimals: 474 and 214 us.
//
// Fields: integer columns are decimal integers (optional sign, at most 18
// digits), parsed exactly; other columns are decimal numbers (optional sign,
// digits with an optional point, optional exponent), converted to the nearest
// FP64 value: the decimal significand w and exponent q give w * 10^q, rounded
// from a 128-bit product where that settles it (scaled_decimal), else formed as
// an exact integer ratio and divided once with correct rounding.
// The ratio's range: every |value| below 1e73 whose last written digit has
// exponent q >= -57 converts; a field beyond 2^247 (about 2.3e74) or with
// q < -57 is refused as malformed (in between, by the significand's bit
// length).  A malformed field marks
// the handle (STATS_E_PARSE, smallest byte offset) and its row is skipped.
#include <cmath>
#include <cstring>

#include "accum_common.hpp"
#include "runtime.hpp"

namespace st {
namespace text {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int UNIT = 4096;         // segments are whole units; lines are counted per unit
constexpr int SEG_MIN = 8 << 10, SEG_MAX = 40 << 10;  // bytes of line starts per workgroup (chosen per chunk)
constexpr int MAXLINE = 4096;      // longest line accepted
constexpr int MAXLS = 18 * kThreads;  // line starts in the table at a time, at most (8 KiB of two-byte lines)
constexpr int kPast = 32;          // bytes past the text that read as 0xFF

// LDS bytes of the text stage of a segment: up to 31 bytes in front (16 of the
// stream before it and the alignment), the segment, the longest line and the end mark.
constexpr int stage_bytes(int seg) { return 32 + seg + MAXLINE + kPast; }
// Dynamic LDS of the two text kernels: the stage, then the line table.
constexpr int text_lds(int seg, int maxls) { return stage_bytes(seg) + 2 * maxls; }
// Bytes of line starts per thread: an odd number of 16-byte vectors, so that
// the threads' vector reads of their slices fall on different banks.
constexpr int slice_of(int seg) { return ((seg + 16 * kThreads - 1) / (16 * kThreads) | 1) * 16; }
constexpr int SLICE_MAX = slice_of(SEG_MAX);
// Words between the parsed rows of a wave's lines: no multiple of four, against
// bank conflicts.
constexpr int row_words(int p) { return p % 4 ? p : p + 1; }

struct Args {
  const char* buf;
  int64_t nbytes;  // readable bytes
  int64_t nend;    // lines start before nend; the last one may end at nend
  int p;
  uint32_t intmask;
  int64_t base_off;  // offset of buf in the caller's stream (for messages)
  int seg;           // bytes of line starts per workgroup: a multiple of 4096, at most SEG_MAX
  int maxls;         // line starts in the table at a time, at most MAXLS
  acc::Args acc;
  DevStatus* status;
};

typedef const __attribute__((address_space(3))) unsigned char* lds_text;

// Staged text of the chunk.  The parser works on positions relative to the
// stage (32-bit); positions at or past lim read as -1.  The kPast bytes from
// lim on hold 0xFF, which is no character of a field.
struct Stage {
  lds_text s;
  int lim;  // first relative position that is not text of this chunk
};

// A thread's reader of the staged text.
struct Cur {
  const Stage* S;
  __device__ explicit Cur(const Stage& st) : S(&st) {}
  __device__ inline int at(int pos) const {
    if (pos >= S->lim) return -1;
    return S->s[pos];
  }
  // The four bytes at pos .. pos + 3 (the first in the low byte), from two
  // aligned LDS words; bytes at or past lim read as 0xFF.  pos >= 0.
  __device__ inline uint32_t word4(int pos) const {
    const int a = pos & ~3;
    const uint32_t lo = *(const __attribute__((address_space(3))) uint32_t*)(S->s + a);
    const uint32_t hi = *(const __attribute__((address_space(3))) uint32_t*)(S->s + a + 4);
    uint32_t v = __builtin_amdgcn_alignbyte(hi, lo, (uint32_t)(pos & 3));
    const int room = S->lim - pos;
    if (room < 4) v |= room <= 0 ? 0xFFFFFFFFu : (0xFFFFFFFFu << (8 * room));
    return v;
  }
};

// Leading decimal digits of a 4-byte word (first character in the low byte):
// their count k (0..4) and value.  A byte is a digit when its high nibble is
// 3 and its low nibble is below 10 (low nibble + 6 does not carry into bit 4).
__device__ inline int digit_run(uint32_t v, uint32_t* val) {
  const uint32_t m = ((v & 0xF0F0F0F0u) ^ 0x30303030u) | (((v & 0x0F0F0F0Fu) + 0x06060606u) & 0xF0F0F0F0u);
  const int k = m ? (__builtin_ctz(m) >> 3) : 4;
  // digit values moved to the top k bytes (leading zero bytes add nothing);
  // then bytes (b0 b1 b2 b3) -> (10 b0 + b1, 10 b2 + b3) -> 100 (..) + (..)
  const uint32_t y = k ? (v & 0x0F0F0F0Fu) << (8 * (4 - k)) : 0u;
  const uint32_t t = y * 10u + (y >> 8);
  *val = (t & 0xFFu) * 100u + ((t >> 16) & 0xFFu);
  return k;
}

// Decimal digits of v < 10^4 without leading zeros.
__device__ inline int sig_count(uint32_t v) {
  return (v >= 1000u) + (v >= 100u) + (v >= 10u) + (v >= 1u);
}

__device__ inline uint32_t pow10_small(int k) {  // 10^k, 1 <= k <= 4
  return k >= 3 ? (k == 4 ? 10000u : 1000u) : (k == 2 ? 100u : 10u);
}

__device__ inline int bitlen64(uint64_t v) { return v ? 64 - __builtin_clzll(v) : 0; }
__device__ inline int bitlen128(u128 v) {
  const uint64_t hi = (uint64_t)(v >> 64);
  return hi ? 128 - __builtin_clzll(hi) : bitlen64((uint64_t)v);
}

__device__ inline U256 u256_mul_small(U256 a, uint32_t m) {
  U256 r;
  u128 carry = 0;
  for (int k = 0; k < 4; ++k) {
    const u128 t = (u128)a.w[k] * m + carry;
    r.w[k] = (uint64_t)t;
    carry = t >> 64;
  }
  return r;
}

// Correctly rounded value of (w + sticky) * 2^e2 where w has 54..128 bits
// and sticky marks a nonzero remainder below the last bit of w.
__device__ inline double round_to_double(u128 w, bool sticky, int e2, bool neg) {
  const int bl = bitlen128(w);
  const int extra = bl - 53;
  uint64_t m;
  if (extra > 0) {
    const u128 low = w & (((u128)1 << extra) - 1);
    const u128 half = (u128)1 << (extra - 1);
    m = (uint64_t)(w >> extra);
    if (low > half || (low == half && (sticky || (m & 1)))) ++m;
    e2 += extra;
  } else {
    m = (uint64_t)w << (-extra);
    e2 += extra;
  }
  if (m == ((uint64_t)1 << 53)) {
    m >>= 1;
    ++e2;
  }
  const double r = ldexp((double)m, e2);
  return neg ? -r : r;
}

struct Pow5 {
  uint64_t v[28];  // 5^k, k <= 27 (5^27 < 2^63)
};
constexpr Pow5 make_pow5() {
  Pow5 t{};
  uint64_t r = 1;
  for (int k = 0; k < 28; ++k) {
    t.v[k] = r;
    r *= 5;
  }
  return t;
}
__constant__ Pow5 kPow5 = make_pow5();

__device__ inline uint64_t pow5_u64(int k) { return kPow5.v[k]; }

// Exact w * 10^q for w < 2^64 and |q| <= 27: w 5^q fits 128 bits for q > 0;
// for q < 0 the quotient w 2^k / 5^-q (k chosen for 54..56 bits) comes from
// an FP64 estimate corrected with the exact 128-bit remainder.
__device__ inline double fast_decimal(uint64_t w, int q, bool neg) {
  if (q >= 0) return round_to_double((u128)w * pow5_u64(q), false, q, neg);
  const uint64_t D = pow5_u64(-q);
  const int bw = bitlen64(w), bd = bitlen64(D);
  const int k = 55 - bw + bd;  // w 2^k has 55 + bd <= 119 bits
  const u128 N = (u128)w << k;
  const double est = (double)N / (double)D;
  uint64_t Q = (uint64_t)est;  // within a few units of floor(N / D)
  __int128 rem = (__int128)N - (__int128)((u128)Q * D);
  while (rem < 0) {
    --Q;
    rem += D;
  }
  while (rem >= (__int128)D) {
    ++Q;
    rem -= D;
  }
  return round_to_double((u128)Q, rem != 0, -k + q, neg);
}

// Exact ratio path for everything else (more than 19 digits, |q| up to 57).
__device__ __attribute__((noinline)) double slow_decimal(u128 w, int q, bool sticky, bool neg) {
  U256 num = u256_from_u128(w), den = u256_from_u128((u128)1);
  if (sticky) {
    num = u256_mul_small(num, 10u);
    num.w[0] |= 1u;  // (10 w + 1) 10^(q - 1); the low digit was 0
    --q;
  }
  if (q >= 0)
    for (int k = 0; k < q; ++k) num = u256_mul_small(num, 10u);
  else
    for (int k = 0; k < -q; ++k) den = u256_mul_small(den, 10u);
  return u256_div_to_double(neg, num, den);
}

// Parses one field starting at f; on success returns the position of the
// terminating byte (',' or '\n' or nend) and the value bits in *bits (int64
// for integer columns, FP64 otherwise).  Returns -1 - pos on malformed input.
// Decimal text keeps 38 significant digits exactly plus a sticky digit for
// any further nonzero digit, which rounds like the full expansion whenever no
// FP64 rounding midpoint lies within 1e-38 relative (always, e.g., for
// printed doubles).  Significands of up to 19 digits (every integer field and
// printed double) are gathered in 64 bits; longer ones go through
// parse_wide.
struct Parsed {
  int pos;        // terminating byte, or -1 - pos on malformed input
  uint64_t bits;  // value
};
__device__ __attribute__((noinline)) Parsed parse_wide(Stage S, int f, bool is_int);

__device__ inline double decimal_value(u128 w, int nd, int q, bool sticky, bool neg, bool* bad) {
  if (w == 0) return neg ? -0.0 : 0.0;
  if (!sticky && nd <= 19 && q >= -27 && q <= 27) return fast_decimal((uint64_t)w, q, neg);
  // range of the exact ratio: 256-bit numerator and denominator
  const int lw = bitlen128(w);
  const int qq = sticky ? q - 1 : q;
  if (qq > 0 && lw + 4 + (qq * 3402 + 1023) / 1024 > 250) *bad = true;  // log2(10) < 3402/1024
  if (qq < -57) *bad = true;
  if (*bad) return 0.0;
  return slow_decimal(w, q, sticky, neg);
}

// Digits from position i on, four per step, into w (significant digits
// counted in nd; q lowered by one per digit when frac).  Returns the character
// after the digits (-1 past the text), or kTooLong when the run would give w
// more than 19 significant digits (w, nd, i are then unspecified).
constexpr int kTooLong = -2;
__device__ inline int digit_steps(const Cur& C, int& i, uint64_t& w, int& nd, int& q, bool frac) {
  for (;;) {
    const uint32_t v = C.word4(i);
    uint32_t val;
    const int k = digit_run(v, &val);
    if (k) {
      const int sig = w ? k : sig_count(val);
      if (nd + sig > 19) return kTooLong;
      w = w * pow10_small(k) + val;
      nd += sig;
      i += k;
      if (frac) q -= k;
    }
    if (k < 4) return i >= C.S->lim ? -1 : (int)((v >> (8 * k)) & 0xFFu);
  }
}

__device__ inline int parse_field(Cur& C, int f, bool is_int, uint64_t* bits) {
  int i = f;
  int c = C.at(i);
  bool neg = false;
  if (c == '-' || c == '+') {
    neg = c == '-';
    ++i;
  }
  uint64_t w = 0;
  int nd = 0;
  int q = 0;
  const int i0 = i;
  c = digit_steps(C, i, w, nd, q, false);
  if (c == kTooLong) {
    const Parsed r = parse_wide(*C.S, f, is_int);
    *bits = r.bits;
    return r.pos;
  }
  bool digits = i > i0;
  if (is_int) {
    if (!digits || nd > 18) return -1 - i;
    if (c != ',' && c != '\n' && c != -1) return -1 - i;
    const int64_t v = (int64_t)w;
    *bits = (uint64_t)(neg ? -v : v);
    return i;
  }
  if (c == '.') {
    ++i;
    const int i1 = i;
    c = digit_steps(C, i, w, nd, q, true);
    if (c == kTooLong) {
      const Parsed r = parse_wide(*C.S, f, is_int);
      *bits = r.bits;
      return r.pos;
    }
    digits |= i > i1;
  }
  if (!digits) return -1 - i;
  if (c == 'e' || c == 'E') {
    c = C.at(++i);
    bool eneg = false;
    if (c == '-' || c == '+') {
      eneg = c == '-';
      c = C.at(++i);
    }
    int ex = 0;
    bool ed = false;
    while (c >= '0' && c <= '9') {
      ed = true;
      if (ex < 100000) ex = ex * 10 + (c - '0');
      c = C.at(++i);
    }
    if (!ed) return -1 - i;
    q += eneg ? -ex : ex;
  }
  if (c != ',' && c != '\n' && c != -1) return -1 - i;
  bool bad = false;
  const double v = decimal_value((u128)w, nd, q, false, neg, &bad);
  if (bad) return -1 - f;
  *bits = (uint64_t)__double_as_longlong(v);
  return i;
}

// The same for significands of more than 19 digits: 128-bit accumulation.
__device__ __attribute__((noinline)) Parsed parse_wide(Stage S, int f, bool is_int) {
  Cur C(S);
  Parsed out{0, 0};
  int i = f;
  int c = C.at(i);
  bool neg = false;
  if (c == '-' || c == '+') {
    neg = c == '-';
    c = C.at(++i);
  }
  u128 w = 0;
  int nd = 0;
  int q = 0;
  bool digits = false, sticky = false;
  while (c >= '0' && c <= '9') {
    digits = true;
    const int d = c - '0';
    if (w != 0 || d != 0) {
      if (nd < 38) {
        w = w * 10 + (u128)d;
        ++nd;
      } else {
        sticky |= d != 0;
        ++q;
      }
    }
    c = C.at(++i);
  }
  if (is_int) return Parsed{-1 - i, 0};  // more than 18 digits
  if (c == '.') {
    c = C.at(++i);
    while (c >= '0' && c <= '9') {
      digits = true;
      const int d = c - '0';
      if (w == 0 && d == 0) {
        --q;
      } else if (nd < 38) {
        w = w * 10 + (u128)d;
        ++nd;
        --q;
      } else {
        sticky |= d != 0;
      }
      c = C.at(++i);
    }
  }
  if (!digits) return Parsed{-1 - i, 0};
  if (c == 'e' || c == 'E') {
    c = C.at(++i);
    bool eneg = false;
    if (c == '-' || c == '+') {
      eneg = c == '-';
      c = C.at(++i);
    }
    int ex = 0;
    bool ed = false;
    while (c >= '0' && c <= '9') {
      ed = true;
      if (ex < 100000) ex = ex * 10 + (c - '0');
      c = C.at(++i);
    }
    if (!ed) return Parsed{-1 - i, 0};
    q += eneg ? -ex : ex;
  }
  if (c != ',' && c != '\n' && c != -1) return Parsed{-1 - i, 0};
  bool bad = false;
  const double v = decimal_value(w, nd, q, sticky, neg, &bad);
  if (bad) return Parsed{-1 - f, 0};
  out.pos = i;
  out.bits = (uint64_t)__double_as_longlong(v);
  return out;
}

// ---- fast path for the common field forms -----------------------------------
//
// Eight characters per step from aligned LDS words; one copy of the code for
// all fields of a line, so that it stays in the instruction cache (unrolled over
// the fields it was 78 KiB at ten columns, and fetching it was most of the time).

// 10^k, 0 <= k <= 8.
__device__ inline uint32_t pow10_upto8(int k) {
  const auto upto4 = [](int j) {
    return j == 4 ? 10000u : (uint32_t)(0x03E80064000A0001ull >> (16 * j)) & 0xFFFFu;
  };
  const int j = k < 4 ? k : 4;
  return __umul24(upto4(j), upto4(k - j));
}

// Value of four digits (the first in the low byte).
__device__ inline uint32_t four_digits(uint32_t y) {
  const uint32_t t = (y << 3) + (y << 1) + (y >> 8);  // 10 b0 + b1 in byte 0, 10 b2 + b3 in byte 2
  return __umul24(t & 0xFFu, 100u) + ((t >> 16) & 0xFFu);
}

// The leading decimal digits of the eight bytes x0, x1 (first character in the
// low byte of x0): their number, their value in *val and, when there are fewer
// than eight, the character after them in *term.
__device__ inline int digits8(uint32_t x0, uint32_t x1, uint32_t* val, uint32_t* term) {
  const auto not_digit = [](uint32_t x) {  // a bit in every byte that is no digit
    return ((x & 0xF0F0F0F0u) ^ 0x30303030u) | (((x & 0x0F0F0F0Fu) + 0x06060606u) & 0xF0F0F0F0u);
  };
  const uint32_t m0 = not_digit(x0), m1 = not_digit(x1);
  const int k = (m0 ? __builtin_ctz(m0) : m1 ? 32 + __builtin_ctz(m1) : 64) >> 3;
  const uint64_t x = (uint64_t)x1 << 32 | x0;
  // the digits moved to the top k bytes: leading zero bytes add nothing
  const uint64_t y = k ? (x & 0x0F0F0F0F0F0F0F0Full) << (64 - 8 * k) : 0ull;
  *val = __umul24(four_digits((uint32_t)y), 10000u) + four_digits((uint32_t)(y >> 32));
  *term = (uint32_t)(x >> (8 * (k & 7))) & 0xFFu;
  return k;
}

// The eight characters at pos (pos <= lim: every word read lies in the stage).
__device__ inline void chars8(const Stage& S, int pos, uint32_t* x0, uint32_t* x1) {
  const __attribute__((address_space(3))) uint32_t* b = (const __attribute__((address_space(3))) uint32_t*)(S.s + (pos & ~3));
  const uint32_t r0 = b[0], r1 = b[1], r2 = b[2], sh = (uint32_t)(pos & 3);
  *x0 = __builtin_amdgcn_alignbyte(r1, r0, sh);
  *x1 = __builtin_amdgcn_alignbyte(r2, r1, sh);
}

// The same after an optional sign at pos, which is counted in *pos.
__device__ inline bool signed_chars8(const Stage& S, int* pos, uint32_t* x0, uint32_t* x1) {
  const __attribute__((address_space(3))) uint32_t* b = (const __attribute__((address_space(3))) uint32_t*)(S.s + (*pos & ~3));
  const uint32_t r0 = b[0], r1 = b[1], r2 = b[2], r3 = b[3], sh = (uint32_t)(*pos & 3);
  const uint32_t a0 = __builtin_amdgcn_alignbyte(r1, r0, sh), a1 = __builtin_amdgcn_alignbyte(r2, r1, sh);
  const uint32_t a2 = __builtin_amdgcn_alignbyte(r3, r2, sh);
  const uint32_t c0 = a0 & 0xFFu;
  const bool neg = c0 == '-';
  const uint32_t sg = (neg || c0 == '+') ? 1u : 0u;
  *x0 = __builtin_amdgcn_alignbyte(a1, a0, sg);
  *x1 = __builtin_amdgcn_alignbyte(a2, a1, sg);
  *pos += (int)sg;
  return neg;
}

// Powers of five for the conversion, -27 <= q <= 27: 5^q = (hi:lo) 2^e with the
// top bit of the 128-bit (hi:lo) set, rounded up for q < 0, exact otherwise, and
// e = floor(q log2 5) - 127.
constexpr int kMaxPow = 27;
struct Pow5Scaled {
  uint64_t hi[2 * kMaxPow + 1], lo[2 * kMaxPow + 1];
};
constexpr Pow5Scaled make_pow5_scaled() {
  Pow5Scaled t{};
  for (int q = -kMaxPow; q <= kMaxPow; ++q) {
    uint64_t d = 1;
    for (int k = 0; k < (q < 0 ? -q : q); ++k) d *= 5;
    int bl = 0;
    while (bl < 64 && (d >> bl) != 0) ++bl;
    u128 r = 0;
    if (q >= 0) {
      r = (u128)d << (128 - bl);
    } else {
      // ceil(2^(127 + bl) / 5^-q), bit by bit
      u128 rem = 0;
      for (int b = 127 + bl; b >= 0; --b) {
        rem = 2 * rem + (b == 127 + bl ? 1 : 0);
        r <<= 1;
        if (rem >= d) {
          rem -= d;
          r |= 1;
        }
      }
      r += 1;
    }
    t.hi[q + kMaxPow] = (uint64_t)(r >> 64);
    t.lo[q + kMaxPow] = (uint64_t)r;
  }
  return t;
}
__constant__ Pow5Scaled kPow5Scaled = make_pow5_scaled();

// The table in LDS, (hi, lo) of each power side by side: the lanes of a wave read
// different entries.
constexpr int kPow5Words = 2 * (2 * kMaxPow + 1);
__device__ inline void copy_pow5(uint64_t* s) {
  for (int k = threadIdx.x; k < 2 * kMaxPow + 1; k += kThreads) {
    s[2 * k] = kPow5Scaled.hi[k];
    s[2 * k + 1] = kPow5Scaled.lo[k];
  }
}

// w 10^q (w != 0, |q| <= kMaxPow) rounded to the nearest FP64 value, ties to
// even; false when the rounding cannot be told from the 128 bits computed.
// (The idea of D. Lemire, "Number parsing at a gigabyte per second", 2021: the
// significand times a scaled power of five; the bounds below are for this
// table.)  With z = w 2^l (top bit set) and T = (hi:lo), X = z 5^q 2^-e' is the
// true value scaled like P = floor(z T / 2^64): T exceeds the exact power by
// less than one unit, so z T / 2^64 lies in [X, X + 1) and P is floor(X) or
// floor(X) + 1.  Let r be the 74 or 75 bits of P below the 53 kept and h their
// half.  r < h: X rounds down, also when r = 0 stems from floor(X) ending in
// ones (then X rounds up to the same value).  r > h + 1: X rounds up.  Only
// r = h and r = h + 1 are open (an exact tie or not); they are left to the
// exact division.  All values are normal: 10^-27 <= w 10^q < 2^64 10^27.
__device__ inline bool scaled_decimal(const uint64_t* pow5, uint64_t w, int q, bool neg, double* out) {
  const int l = __builtin_clzll(w);
  const uint64_t z = w << l;
  const u128 a = (u128)z * pow5[2 * (q + kMaxPow)];
  const u128 P = a + (uint64_t)(((u128)z * pow5[2 * (q + kMaxPow) + 1]) >> 64);
  uint64_t hi = (uint64_t)(P >> 64), lo = (uint64_t)P;
  const int top = (int)(hi >> 63);  // P has 128 bits, or 127
  const int s = 10 + top;           // bits of hi below the 53 kept
  const uint64_t m = hi >> s;
  const uint32_t rh = (uint32_t)hi & ((1u << s) - 1), half = 1u << (s - 1);
  if (rh == half && lo <= 1) return false;
  const uint64_t mr = m + (rh >= half ? 1 : 0);
  // value = m 2^(s + 64 + e), P in units of 2^e, e = floor(q log2 5) - 127 + 64 - l + q
  const int e = ((q * 152170) >> 16) - 63 - l + q + 64 + s;
  const uint64_t bits = mr + ((uint64_t)(e + 52 + 1022) << 52);  // m's top bit and a carry of the rounding add to the exponent
  *out = __longlong_as_double((long long)(bits | (neg ? 1ull << 63 : 0ull)));
  return true;
}

// Further digits at *p, eight a step, appended to *v (*nd counts them).  Past 19
// digits the field is not taken, so three steps are enough and *v may wrap.
__device__ inline void more_digits(const Stage& S, bool more, int* p, int* nd, uint64_t* v, uint32_t* c) {
  while (more) {
    uint32_t x0, x1, val;
    chars8(S, *p, &x0, &x1);
    const int k = digits8(x0, x1, &val, c);
    *v = *v * pow10_upto8(k) + val;
    *nd += k;
    *p += k;
    more = k == 8 && *nd < 24;
  }
}

// The field at f when it is followed by the byte want and has one of the common
// forms: [sign] 1..18 digits (integer columns), or [sign] digits [. digits]
// [e [sign] 1..3 digits] with 1..19 digits before the exponent and a power of
// ten of at most 10^27 either way (decimal columns).  Then it returns true with
// the position of want in *end and the value bits in *bits, exactly as
// parse_field gives them; otherwise false, and parse_field takes the field.
__device__ inline bool fast_int(const Stage& S, int f, uint32_t want, int* end, uint64_t* bits) {
  uint32_t x0, x1, val, c;
  int p = f;
  const bool neg = signed_chars8(S, &p, &x0, &x1);
  int nd = digits8(x0, x1, &val, &c);
  uint64_t v = val;
  p += nd;
  more_digits(S, nd == 8, &p, &nd, &v, &c);
  *bits = neg ? 0ull - v : v;
  *end = p;
  return (c == want) & ((uint32_t)(nd - 1) < 18u);
}

__device__ inline bool fast_decimal_field(const Stage& S, const uint64_t* pow5, int f, uint32_t want, int* end,
                                          uint64_t* bits) {
  uint32_t x0, x1, val, c;
  int p = f;
  const bool neg = signed_chars8(S, &p, &x0, &x1);
  int nd = digits8(x0, x1, &val, &c);
  uint64_t v = val;
  p += nd;
  more_digits(S, nd == 8, &p, &nd, &v, &c);
  int q = 0;
  if (c == '.') {
    ++p;
    q = nd;
    more_digits(S, true, &p, &nd, &v, &c);
    q -= nd;
  }
  bool ok = (uint32_t)(nd - 1) < 19u;
  if ((c | 0x20u) == 'e') {
    uint32_t ex;
    ++p;
    const bool eneg = signed_chars8(S, &p, &x0, &x1);
    const int k = digits8(x0, x1, &ex, &c);
    ok &= (uint32_t)(k - 1) < 3u;
    p += k;
    q += eneg ? -(int)ex : (int)ex;
  }
  ok &= (c == want) & ((uint32_t)(q + kMaxPow) <= 2u * kMaxPow);
  double d = neg ? -0.0 : 0.0;
  if (ok && v != 0) ok = scaled_decimal(pow5, v, q, neg, &d);
  *bits = (uint64_t)__double_as_longlong(d);
  *end = p;
  return ok;
}

// parse_field out of line, for the fields fast_field does not take.
__device__ __attribute__((noinline)) Parsed slow_field(Stage S, int f, bool is_int) {
  Cur C(S);
  uint64_t bits = 0;
  const int r = parse_field(C, f, is_int, &bits);
  return Parsed{r, bits};
}

// Parses the line starting at L (P fields), handing (c, value bits) of each field
// to put.  A field that the fast forms do not cover (a line that ends with the
// text among them) goes through parse_field.  Returns the position of the line's
// end ('\n' or nend), or -1 - end on a malformed line (*bad_at = the offending
// field's offset); the rest of such a line is not looked at, and put gets zeros.
template <int P, typename Put>
__device__ inline int parse_line_p(uint32_t intmask, const Stage& S, const uint64_t* pow5, int L, int* bad_at, Put put) {
  int f = L, r = L, stop = 0;
  bool bad = false;
#pragma unroll 1
  for (int c = 0; c < P; ++c) {
    const bool is_int = (intmask >> c) & 1u, last = c == P - 1;
    const uint32_t want = last ? '\n' : ',';
    uint64_t bits;
    const bool fast = is_int ? fast_int(S, f, want, &r, &bits) : fast_decimal_field(S, pow5, f, want, &r, &bits);
    if (!fast) {
      if (!bad) {
        const Parsed sp = slow_field(S, f, is_int);
        r = sp.pos;
        bits = sp.bits;
        const int term = r >= 0 ? Cur(S).at(r) : 0;
        bad = !(r >= 0 && (term == (int)want || (last && term == -1)));
        if (bad) {
          *bad_at = f;
          int e = r >= 0 ? r : -1 - r;  // skip to the end of the line
          for (;;) {
            const int ch = Cur(S).at(e);
            if (ch == '\n' || ch < 0) break;
            ++e;
          }
          stop = e;
        }
      }
      if (bad) {
        bits = 0;
        r = stop - 1;
      }
    }
    put(c, bits);
    f = r + 1;
  }
  return bad ? -1 - stop : r;
}

// Copies the text [w0r, w0r + nr) of buf into LDS on a
// 16-byte aligned origin: LDS position i holds stream byte w0r - sh + i,
// sh = the misalignment of buf + w0r, which is returned.  Every thread issues
// its aligned 16-byte loads before its first LDS write; the vectors at the
// two ends are assembled byte by byte so that nothing outside
// [buf + w0r - (w0r >= 16 ? sh : 0), buf + w0r + nr) is read (positions before
// w0r hold zeros when w0r < 16, earlier stream bytes otherwise).
__device__ inline int stage_text(const char* buf, int64_t w0r, int nr, __attribute__((address_space(3))) unsigned char* s_buf,
                                 uint64_t* s_pow5) {
  const int sh = (int)((uintptr_t)(buf + w0r) & 15u);
  const char* base = buf + w0r - sh;
  const int tot = sh + nr;
  const int nv = (tot + 15) >> 4;
  constexpr int NVT = (stage_bytes(SEG_MAX) + 15) / 16 / kThreads + 1;
  u32x4 q[NVT];
#pragma unroll
  for (int u = 0; u < NVT; ++u) {
    const int v = (int)threadIdx.x + u * kThreads;
    q[u] = (u32x4){0u, 0u, 0u, 0u};
    if (v < nv) {
      const int p0 = 16 * v;
      if (p0 + 16 <= tot && (w0r >= 16 || p0 >= sh)) {
        q[u] = *(const u32x4*)(base + p0);
      } else {
        uint32_t wd[4] = {0u, 0u, 0u, 0u};
        for (int k = 0; k < 16; ++k) {
          const int pos = p0 + k;
          if (pos >= sh && pos < tot)
            wd[k >> 2] |= (uint32_t)(unsigned char)buf[w0r + pos - sh] << (8 * (k & 3));
        }
        q[u] = (u32x4){wd[0], wd[1], wd[2], wd[3]};
      }
    }
  }
  copy_pow5(s_pow5);
#pragma unroll
  for (int u = 0; u < NVT; ++u) {
    const int v = (int)threadIdx.x + u * kThreads;
    if (v < nv) *(__attribute__((address_space(3))) u32x4*)(s_buf + 16 * v) = q[u];
  }
  return sh;
}

// Line starts of a workgroup's segment [s0r, s1r) (stage-relative; a line
// starts after '\n' or at the stream start).  Thread t finds the newlines of
// its slice (slice positions, a multiple of 16 up to SLICE_MAX) in one pass
// of 16-byte LDS reads, keeping them as a bit
// mask (a '\n' byte is a zero byte of v ^ 0x0a0a0a0a); a workgroup scan of the
// counts places lines base .. base + maxls - 1 of them in s_ls in stream order.
// Returns the number of all line starts.
// Contains barriers: every thread of the workgroup calls it.
__device__ inline int line_starts(lds_text s_buf, int64_t w0, int s0r, int s1r, int slice, int base,
                                  int maxls, unsigned short* s_ls, int* s_wsum) {
  constexpr int NV = SLICE_MAX / 16 + 1;     // 16-byte reads per slice (it may start mid-vector)
  constexpr int NM = (16 * NV + 31) / 32;    // 32-bit mask words
  const int c0 = s0r + (int)threadIdx.x * slice;
  const int c1 = min(c0 + slice, s1r);
  // newline positions m in [mlo, mhi) start the lines c0 .. c1 - 1; bit b of the
  // mask is position mb + b
  const int mlo = max(c0 - 1, 0), mhi = c1 - 1;
  const int mb = mlo & ~15;
  uint32_t nl[NM];
#pragma unroll
  for (int j = 0; j < NM; ++j) nl[j] = 0;
  int mine = 0;
  if (c0 < c1) {
    if (w0 + c0 == 0) ++mine;  // the stream's first byte
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int m16 = mb + 16 * k;
      if (m16 < mhi) {
        const u32x4 v = *(const __attribute__((address_space(3))) u32x4*)(s_buf + m16);
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t x = v[e] ^ 0x0A0A0A0Au;
          const uint32_t z = ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu);  // 0x80 per '\n'
          bits |= __builtin_amdgcn_udot4(z >> 7, 0x08040201u, 0u, false) << (4 * e);
        }
        // keep positions in [mlo, mhi)
        const int b0 = mlo - m16, b1 = mhi - m16;
        if (b0 > 0) bits &= 0xFFFFu << b0;
        if (b1 < 16) bits &= (1u << b1) - 1u;
        nl[k >> 1] |= bits << (16 * (k & 1));
      }
    }
#pragma unroll
    for (int j = 0; j < NM; ++j) mine += __builtin_popcount(nl[j]);
  }
  // workgroup exclusive scan of the counts
  int incl = mine;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
  if (lane == 63) s_wsum[wv] = incl;
  __syncthreads();
  int before = incl - mine, total = 0;
  for (int k = 0; k < kThreads / 64; ++k) {
    if (k < wv) before += s_wsum[k];
    total += s_wsum[k];
  }
  int at = before - base;
  if (c0 < c1 && at < maxls && at + mine > 0) {
    auto place = [&](int pos) {
      if ((unsigned)at < (unsigned)maxls) s_ls[at] = (unsigned short)pos;
      ++at;
    };
    if (w0 + c0 == 0) place(c0);
#pragma unroll
    for (int j = 0; j < NM; ++j) {
      uint32_t m = nl[j];
      while (m) {
        place(mb + 32 * j + __builtin_ctz(m) + 1);
        m &= m - 1;
      }
    }
  }
  __syncthreads();
  return total;
}

typedef double d4 __attribute__((ext_vector_type(4)));

// Waits for this wave's LDS accesses; also keeps the compiler from moving
// LDS accesses across it (the rows a wave stages are read by other lanes).
__device__ inline void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// What the two text kernels share: the stage and where the segment lies in it.
// Threads take the lines of the table in turn; a segment of more lines than the
// table holds refills it, window by window.
struct Lines {
  Stage S;
  int64_t w0;    // stream offset of staged byte 0
  int s0r, s1r;  // the segment, stage-relative
};

// Stages this workgroup's segment of the chunk.  Contains a barrier, and writes
// the end mark after it (line_starts does not read that far and ends in one).
__device__ inline Lines open_lines(const Args& a, __attribute__((address_space(3))) unsigned char* s_buf, uint64_t* s_pow5) {
  Lines n;
  const int64_t s0 = (int64_t)blockIdx.x * a.seg, s1 = min(s0 + (int64_t)a.seg, a.nend);
  const int64_t w0r = s0 >= 16 ? s0 - 16 : 0;  // first stream byte staged
  const int64_t w1 = min(s1 + (int64_t)MAXLINE, a.nbytes);
  // the staging origin is aligned
  n.w0 = w0r - stage_text(a.buf, w0r, (int)(w1 - w0r), s_buf, s_pow5);
  n.S = Stage{s_buf, (int)(min(a.nend, w1) - n.w0)};
  n.s0r = (int)(s0 - n.w0);
  n.s1r = (int)(s1 - n.w0);
  __syncthreads();
  if (threadIdx.x < kPast) s_buf[n.S.lim + (int)threadIdx.x] = 0xFFu;
  return n;
}

// Products on the FP64 matrix cores: each wave parses 64 lines into its own LDS
// rows; for v_mfma_f64_16x16x4f64 a lane then holds column (lane % 16) of row
// 4 m + lane / 16, at once its element of the A operand (column i, row k) and
// of the B operand (row k, column j), so 16 products give the 64 rows' upper
// triangle; absent or malformed lines count as zeros.  The column sums are kept
// per lane.  For integer columns every partial sum is an integer below 2^53
// under the guard checked by the merge, so the matrix-core sums are exact; the
// order of all sums is fixed, so results are bitwise reproducible.
template <int P>
__global__ __launch_bounds__(kThreads) void k_text(Args a) {
  constexpr int T = P * (P + 1) / 2;
  constexpr int LD = row_words(P);
  extern __shared__ __attribute__((aligned(16))) unsigned char s_buf[];  // text_lds(a.seg, a.maxls)
  __shared__ uint64_t s_rows[kWaves * 64 * LD + 16];  // per wave: 64 parsed rows, shifted
  __shared__ __attribute__((aligned(16))) uint64_t s_pow5[kPow5Words];
  __shared__ uint64_t sKb[P];
  __shared__ int s_wsum[kWaves];
  unsigned short* s_ls = (unsigned short*)(s_buf + stage_bytes(a.seg));  // line starts (stage-relative)
  static_assert(stage_bytes(SEG_MIN) >= kWaves * 5 * 64 * 8, "the final reduction reuses the text stage");
  const acc::Args& ra = a.acc;
  uint64_t* out = ra.rec + (int64_t)blockIdx.x * (2 + 2 * P + T);
  // this thread's product (register r of lane l holds D[4r + l/16][l%16]) and column in the record, looked up before they are needed
  static_assert(kThreads == 4 * 64, "one product per thread");
  const int pi = 4 * (threadIdx.x >> 6) + ((threadIdx.x & 63) >> 4), pj = threadIdx.x & 15;
  const bool prod = pi <= pj && pj < P;
  const int pdst = prod ? 2 + P + ra.dst[P + pi * P - pi * (pi - 1) / 2 + (pj - pi)] : 0;
  const int cdst = threadIdx.x < P ? 2 + P + ra.dst[threadIdx.x] : 0;
  const int kdst = threadIdx.x < P ? 2 + ra.kdst[threadIdx.x] : 0;
  __attribute__((address_space(3))) unsigned char* const text = (__attribute__((address_space(3))) unsigned char*)s_buf;
  const Lines n = open_lines(a, text, s_pow5);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, rsub = lane >> 4;
  uint64_t* wr = s_rows + wave * 64 * LD;
  d4 acc = {0.0, 0.0, 0.0, 0.0}, acc2 = {0.0, 0.0, 0.0, 0.0};  // even and odd steps
  double colsum = 0.0;
  int nrows = 0;  // of this wave
  int first_bad = INT32_MAX;
  // the value of column c less its shift, as the FP64 number the products take
  const auto shifted = [&](int c, uint64_t bits) {
    return ((a.intmask >> c) & 1u) ? (double)((int64_t)bits - (int64_t)sKb[c])
                                   : __longlong_as_double((long long)bits) - __longlong_as_double((long long)sKb[c]);
  };
  bool first = true;  // this wave's first round: the shift is not yet known
  for (int base = 0;; base += a.maxls) {
    const int total = line_starts(text, n.w0, n.s0r, n.s1r, slice_of(a.seg), base, a.maxls, s_ls, s_wsum);
    const int here = min(total - base, a.maxls);  // lines in the table
    for (int idx = threadIdx.x;; idx += kThreads) {
      const bool have = idx < here;
      // every wave runs the first round (its barrier); later rounds while a lane has a line
      if (!first && __builtin_amdgcn_ballot_w64(have) == 0) break;
      bool ok = false;
      if (have) {
        int bad_at = INT32_MAX;
        const int end = parse_line_p<P>(a.intmask, n.S, s_pow5, (int)s_ls[idx], &bad_at, [&](int c, uint64_t bits) {
          wr[lane * LD + c] = first ? bits : (uint64_t)__double_as_longlong(shifted(c, bits));
        });
        ok = end >= 0;
        if (!ok) first_bad = min(first_bad, bad_at);
      }
      if (first) {
        // block shift: the row of the workgroup's first line, zeros if it does not parse
        if (threadIdx.x == 0) {
#pragma unroll
          for (int c = 0; c < P; ++c) sKb[c] = ok ? wr[c] : 0;
        }
        __syncthreads();
        if (ok)
#pragma unroll
          for (int c = 0; c < P; ++c) wr[lane * LD + c] = (uint64_t)__double_as_longlong(shifted(c, wr[lane * LD + c]));
        first = false;
      }
      const uint64_t okm = __builtin_amdgcn_ballot_w64(ok);
      nrows += __builtin_popcountll(okm);
      if (!ok)
        for (int c = 0; c < P; ++c) wr[lane * LD + c] = 0;  // 0.0: adds nothing
      wave_lds_sync();
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        if (((okm >> (16 * h)) & 0xFFFFu) == 0) continue;  // 16 absent rows
#pragma unroll
        for (int m = 4 * h; m < 4 * h + 4; ++m) {
          // lanes of columns P and up hold some other value: only rows and columns
          // of the product that nobody reads
          const double v = __longlong_as_double((long long)wr[(4 * m + rsub) * LD + col]);
          colsum += v;
          if (m & 1) acc2 = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, acc2, 0, 0, 0);
          else acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v, v, acc, 0, 0, 0);
        }
      }
      wave_lds_sync();
    }
    if (base + a.maxls >= total) break;
    __syncthreads();  // every wave is done with the table
  }
  if (first_bad != INT32_MAX) {
    atomicMin(&a.status->parse_off, (unsigned long long)(a.base_off + n.w0 + first_bad));
    atomicOr(&a.status->bits, ST_PARSE);
  }
  if (lane == 0) s_wsum[wave] = nrows;
  __syncthreads();  // the text stage is free: it holds the per-wave sums now
  double* red = (double*)s_buf;  // [wave][4 registers + 1 sum][64 lanes]
#pragma unroll
  for (int r = 0; r < 4; ++r) red[(wave * 5 + r) * 64 + lane] = acc[r] + acc2[r];
  red[(wave * 5 + 4) * 64 + lane] = colsum;
  __syncthreads();
  if (prod) {
    double v = red[threadIdx.x];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += red[w * 5 * 64 + threadIdx.x];
    out[pdst] = (uint64_t)__double_as_longlong(v);
  }
  if (threadIdx.x < P) {
    const int c = threadIdx.x;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
#pragma unroll
      for (int k = 0; k < 4; ++k) v += red[(w * 5 + 4) * 64 + c + 16 * k];
    out[cdst] = (uint64_t)__double_as_longlong(v);
    // the shift word: the int64 value for integer columns, FP64 bits
    // otherwise, i.e. sKb as parsed
    out[kdst] = sKb[c];
  }
  if (threadIdx.x == 0) {
    uint64_t rows = 0;
    for (int w = 0; w < kWaves; ++w) rows += s_wsum[w];
    out[0] = rows;
    out[1] = 0;
  }
}

// Position after the last '\n' in [0, n), or 0 when there is none; one
// workgroup scans backwards in SEG_MAX-byte windows.
__global__ void k_last_newline(const char* buf, int64_t n, int64_t* out) {
  __shared__ unsigned long long best;
  if (threadIdx.x == 0) best = 0;
  __syncthreads();
  for (int64_t hi = n; hi > 0; hi -= SEG_MAX) {
    const int64_t lo = hi > SEG_MAX ? hi - SEG_MAX : 0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x)
      if (buf[i] == '\n') atomicMax(&best, (unsigned long long)(i + 1));
    __syncthreads();
    if (best > 0) break;
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = (int64_t)best;
}

// Newlines in a sample of [0, n), 64 windows: the 64 equal parts of it up
// to 1 MiB, else 16 KiB at the start of each 64th.  Workgroup k (1024
// threads, 16 bytes each, all loads in flight at once) writes the count of
// window k to out[k].  The chunk's mean line length sets the fused kernel's
// segment size.
constexpr int kDensWin = 64;
constexpr int kDensBytes = 16 << 10;
__global__ __launch_bounds__(1024) void k_line_density(const char* buf, int64_t n, int64_t* out) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  const int k = blockIdx.x;
  const bool all = n <= (int64_t)kDensWin * kDensBytes;
  const int64_t lo = all ? n * k / kDensWin : (n / kDensWin) * k;
  const int64_t hi = all ? n * (k + 1) / kDensWin : lo + kDensBytes;
  const int64_t i0 = lo + 16 * (int64_t)threadIdx.x;
  int c = 0;
#pragma unroll
  for (int u = 0; u < 16; ++u) c += (i0 + u < hi && buf[i0 + u] == '\n') ? 1 : 0;
  atomicAdd(&cnt, c);
  __syncthreads();
  if (threadIdx.x == 0) out[k] = cnt;
}

// ---- CSV -> fixed-width binary rows ------------------------------------------

// Line starts per unit, one wave each, read from global memory as aligned
// 16-byte vectors (a byte per load ran at 0.8 TB/s, 189 us for 150 MB of text;
// 32 us so); the bytes before the first vector and after the last one are read
// singly, so nothing outside the chunk is.  first[unit] receives the number of
// line starts in the earlier units of its group, counts[group] the group's.
constexpr int kGroup = 16;  // units per workgroup
__global__ __launch_bounds__(64 * kGroup) void k_unit_lines(const char* buf, int64_t nend, int64_t* counts, int32_t* first) {
  __shared__ int s_sum[kGroup];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t unit = (int64_t)blockIdx.x * kGroup + wave;
  const int64_t s0 = unit * UNIT;
  const int64_t s1 = min(s0 + (int64_t)UNIT, nend);
  int mine = 0;
  if (s0 < s1) {
    // newlines at m in [max(s0 - 1, 0), s1 - 1) start the lines after s0
    const char* b0 = buf + (s0 > 0 ? s0 - 1 : 0);
    const int n = (int)(buf + (s1 - 1) - b0);
    const int head = min(n, (int)(-(uintptr_t)b0 & 15u));
    const int nv = (n - head) >> 4, tail = head + 16 * nv;
    constexpr int NV = UNIT / 16 / 64 + 1;
    u32x4 q[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int v = lane + u * 64;
      q[u] = v < nv ? *(const u32x4*)(b0 + head + 16 * v) : (u32x4){0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int u = 0; u < NV; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t x = q[u][e] ^ 0x0A0A0A0Au;
        mine += __builtin_popcount(~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu));  // 0x80 per '\n'
      }
    if (lane < head) mine += b0[lane] == '\n';
    if (lane < n - tail) mine += b0[tail + lane] == '\n';
    if (s0 == 0 && lane == 0) ++mine;  // the stream's first line
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) mine += __shfl_down(mine, d, 64);
  if (lane == 0) s_sum[wave] = mine;
  __syncthreads();
  if (threadIdx.x < kGroup) {
    int before = 0;
    for (int w = 0; w < (int)threadIdx.x; ++w) before += s_sum[w];
    first[(int64_t)blockIdx.x * kGroup + threadIdx.x] = before;
    if (threadIdx.x == kGroup - 1) counts[blockIdx.x] = before + s_sum[kGroup - 1];
  }
}

// Exclusive prefix sum of counts[0 .. n) in place, the total in *total: one
// workgroup, a run of consecutive counts per thread.  Also clears the
// conversion's status.
__global__ __launch_bounds__(1024) void k_scan_counts(int64_t* counts, int64_t n, int64_t* total, DevStatus* status) {
  __shared__ int64_t s_wave[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t per = (n + 1023) / 1024, i0 = min(per * (int64_t)threadIdx.x, n), i1 = min(i0 + per, n);
  int64_t sum = 0;
#pragma unroll 8
  for (int64_t i = i0; i < i1; ++i) sum += counts[i];
  int64_t incl = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int64_t at = incl - sum;
  for (int w = 0; w < wave; ++w) at += s_wave[w];
  for (int64_t i = i0; i < i1; ++i) {
    const int64_t v = counts[i];
    counts[i] = at;
    at += v;
  }
  if (threadIdx.x == 1023) {
    *total = at;
    *status = DevStatus{0u, 0u, ~0ull};
  }
}

struct ConvArgs {
  Args t;                    // text, its line limit, p, integer mask, offsets, status
  const int64_t* group_base;  // first output row of each group of units
  const int32_t* first;       // rows of a unit's group before it
  char* out[16];             // column c of row r at out[c] + r * stride[c]
  int64_t stride[16];
  int32_t dtype[16];         // STATS_I32 / STATS_I64 / STATS_F64
};

// One parsed field into its binary column; false when the value does not fit
// the column's type (an integer beyond int32, or beyond 2^53 for FP64).
__device__ inline bool store_field(const ConvArgs& a, int c, int64_t r, uint64_t bits, bool is_int) {
  char* dst = a.out[c] + r * a.stride[c];
  switch (a.dtype[c]) {
    case STATS_I32: {
      const int64_t v = (int64_t)bits;
      if (v < INT32_MIN || v > INT32_MAX) return false;
      *(int32_t*)dst = (int32_t)v;
      return true;
    }
    case STATS_I64: *(int64_t*)dst = (int64_t)bits; return true;
    default: {
      if (is_int) {
        const int64_t v = (int64_t)bits;
        if (v > ((int64_t)1 << 53) || v < -((int64_t)1 << 53)) return false;
        *(double*)dst = (double)v;
      } else {
        *(uint64_t*)dst = bits;
      }
      return true;
    }
  }
}

// Each wave parses 64 lines into its LDS rows, then writes them out with
// neighbouring lanes on neighbouring columns, so that a row's columns leave in
// one piece (a lane storing its own row wrote 8 bytes every row stride).
template <int P>
__global__ __launch_bounds__(kThreads) void k_text_convert(ConvArgs a) {
  constexpr int LD = row_words(P);
  constexpr int CW = P <= 1 ? 1 : P <= 2 ? 2 : P <= 4 ? 4 : P <= 8 ? 8 : 16;  // lanes per row when writing
  constexpr int RW = 64 / CW;                                                 // rows per write
  extern __shared__ __attribute__((aligned(16))) unsigned char s_buf[];  // text_lds(t.seg, t.maxls)
  __shared__ uint64_t s_rows[kWaves][64 * LD];
  __shared__ __attribute__((aligned(16))) uint64_t s_pow5[kPow5Words];
  __shared__ int s_wsum[kWaves];
  const Args& t = a.t;
  unsigned short* s_ls = (unsigned short*)(s_buf + stage_bytes(t.seg));
  __attribute__((address_space(3))) unsigned char* const text = (__attribute__((address_space(3))) unsigned char*)s_buf;
  const Lines n = open_lines(t, text, s_pow5);
  const int64_t unit = (int64_t)blockIdx.x * (t.seg / UNIT);
  const int64_t base = a.group_base[unit / kGroup] + a.first[unit];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane % CW, rsub = lane / CW;
  const bool colv = col < P;
  uint64_t* wr = s_rows[wave];
  int first_bad = INT32_MAX;
  for (int w = 0;; w += t.maxls) {
    const int total = line_starts(text, n.w0, n.s0r, n.s1r, slice_of(t.seg), w, t.maxls, s_ls, s_wsum);
    const int here = min(total - w, t.maxls);  // lines in the table
    for (int idx = threadIdx.x;; idx += kThreads) {
      const bool have = idx < here;
      if (__builtin_amdgcn_ballot_w64(have) == 0) break;
      const int L = have ? (int)s_ls[idx] : 0;
      const int row = w + idx;  // this thread's line among the segment's
      bool ok = false;
      if (have) {
        int bad_at = INT32_MAX;
        const int end = parse_line_p<P>(t.intmask, n.S, s_pow5, L, &bad_at,
                                        [&](int c, uint64_t bits) { wr[lane * LD + c] = bits; });
        ok = end >= 0;
        if (!ok) first_bad = min(first_bad, L);  // reported by the line's first byte
      }
      const uint64_t okm = __builtin_amdgcn_ballot_w64(ok);
      wave_lds_sync();
#pragma unroll 4
      for (int m = 0; m < CW; ++m) {
        const int sr = m * RW + rsub;
        const int k = __shfl(row, sr, 64), Ls = __shfl(L, sr, 64);
        if (colv && ((okm >> sr) & 1u)) {
          if (!store_field(a, col, base + k, wr[sr * LD + col], (t.intmask >> col) & 1u)) first_bad = min(first_bad, Ls);
        }
      }
      wave_lds_sync();
    }
    if (w + t.maxls >= total) break;
    __syncthreads();  // every wave is done with the table
  }
  if (first_bad != INT32_MAX) {
    atomicMin(&t.status->parse_off, (unsigned long long)(t.base_off + n.w0 + first_bad));
    atomicOr(&t.status->bits, ST_PARSE);
  }
}

template <int P>
void launch_convert_p(const ConvArgs& a, int64_t nblocks, hipStream_t s) {
  hipLaunchKernelGGL(k_text_convert<P>, dim3((unsigned)nblocks), dim3(kThreads), text_lds(a.t.seg, a.t.maxls), s, a);
}

template <int P>
void launch_text_p(const Args& a, int64_t nblocks, hipStream_t s) {
  hipLaunchKernelGGL(k_text<P>, dim3((unsigned)nblocks), dim3(kThreads), text_lds(a.seg, a.maxls), s, a);
}

}  // namespace text

using namespace text;

// Rounds of 256 lines of a segment of lines of mean length ell (the line count
// taken 3 % high for the spread between segments).
static double text_rounds(double ell, int seg) { return std::ceil(seg / ell * 1.03 / kThreads); }

// Line starts in the table at a time: those of the rounds expected.  Segments of
// shorter lines than the mean go through it window by window, in whole rounds.
static int pick_maxls(double ell, int seg) {
  return ell > 0.0 ? (int)std::min<double>(MAXLS, kThreads * text_rounds(ell, seg)) : MAXLS;
}

// Segment size of the text kernels for lines of mean length ell bytes and p
// columns.  A workgroup parses its lines 256 at a time (one per thread); a last
// round with few lines takes as long as a full one, and the fixed part (staging,
// line table, final sums, record) about 1.2 rounds.  LDS (text and parsed rows)
// decides how many workgroups share a compute unit; each further one lengthens
// the others by about 18 %.  Every whole number of units from SEG_MIN to SEG_MAX is
// scored by the lines per time of a compute unit in these terms (less where a
// segment has more than 2048 lines: filling the table, a slice per thread, takes
// over then).  Ten Table-1 columns
// (57 bytes a line, 8 million lines): 24 KiB 598 us a pass, 12, 20, 28 and 40 KiB
// 703, 671, 824 and 650; thirteen decimal columns (170 bytes): 40 KiB 869,
// 24 KiB 1304.  Without a measurement: 20 KiB.
static int pick_text_seg(double ell, int p) {
  int best = 5 * UNIT;
  if (!(ell > 0.0)) return best;
  double best_score = -1.0;
  for (int seg = SEG_MIN; seg <= SEG_MAX; seg += UNIT) {
    const double lines = seg / ell;
    const double rounds = text_rounds(ell, seg);
    const int lds = text_lds(seg, pick_maxls(ell, seg)) + kThreads * row_words(p) * 8 + 1280;
    const int wgs = std::min(4, (160 << 10) / lds);
    const double score = wgs * lines / ((1.2 + rounds) * (1.0 + 0.18 * (wgs - 1))) * std::min(1.0, 2048 / (lines * 1.03));
    if (score > best_score) {
      best_score = score;
      best = seg;
    }
  }
  return best;
}

static int text_launch(stats_ctx* h, const char* dbuf, int64_t nbytes, int64_t nend, int64_t base_off) {
  const int p = h->p;
  const int seg = pick_text_seg(h->text_ell, p);
  const int64_t nblocks = (nend + seg - 1) / seg;
  if (nblocks == 0) return STATS_OK;
  const int64_t W = rec_words(p);
  // block records, then the slice totals of the merge
  const int64_t part_words = merge_slice_words(nblocks, p);
  int rc = ensure_dev(h, (void**)&h->rec, &h->rec_cap, (size_t)((nblocks * W + part_words) * 8));
  if (rc) return rc;
  Args a;
  memset(&a, 0, sizeof a);
  a.buf = dbuf;
  a.nbytes = nbytes;
  a.nend = nend;
  a.p = p;
  a.base_off = base_off;
  a.seg = seg;
  a.maxls = pick_maxls(h->text_ell, seg);
  a.status = h->status_dev;
  uint32_t intmask = 0;
  for (int c = 0; c < p; ++c)
    if (h->intf[c]) intmask |= 1u << c;
  a.intmask = intmask;
  acc::Args& x = a.acc;
  for (int c = 0; c < 16; ++c) {
    x.dtype[c] = (c < p && h->intf[c]) ? STATS_I64 : STATS_F64;
    x.kdst[c] = (int8_t)(c < p ? c : 0);
  }
  x.intmask = intmask;
  x.chkmask = 0;
  int e = p;
  for (int i = 0; i < p; ++i) x.dst[i] = (int16_t)i;
  for (int i = 0; i < p; ++i)
    for (int j = i; j < p; ++j) x.dst[e++] = (int16_t)(p + tri(p, i, j));
  x.rec = h->rec;
  {
    Timer t;
    t.begin(h, STATS_K_TEXT);
    switch (p) {
#define ST_CASE(PP) \
  case PP: launch_text_p<PP>(a, nblocks, h->stream); break;
      ST_CASE(1) ST_CASE(2) ST_CASE(3) ST_CASE(4) ST_CASE(5) ST_CASE(6) ST_CASE(7) ST_CASE(8)
      ST_CASE(9) ST_CASE(10) ST_CASE(11) ST_CASE(12) ST_CASE(13) ST_CASE(14) ST_CASE(15) ST_CASE(16)
#undef ST_CASE
    }
    t.end();
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return hip_fail(h, err, "text kernel launch");
  {
    Timer t;
    t.begin(h, STATS_K_MERGE);
    launch_merge_records(h->rec, nblocks, p, h->intf_dev, h->state[h->cur], h->state[h->cur ^ 1], h->status_dev, h->stream,
                         part_words ? h->rec + nblocks * W : nullptr);
    t.end();
  }
  err = hipGetLastError();
  if (err != hipSuccess) return hip_fail(h, err, "merge kernel launch");
  h->cur ^= 1;
  return STATS_OK;
}

}  // namespace st

using namespace st;

extern "C" int stats_accumulate_text(stats_ctx* h, const char* buf, int64_t nbytes, int32_t mem_kind,
                                     int32_t is_last, int64_t* bytes_consumed) {
  if (!h) return fail(STATS_E_ARG, "handle is NULL");
  if (h->poisoned) return fail(STATS_E_STATE, "handle is poisoned by an earlier HIP error");
  if (h->ngroups) return fail(STATS_E_STATE, "groups handle: text input is not supported");
  if (h->flags & STATS_CFG_PAIRWISE) return fail(STATS_E_STATE, "pairwise handle: text input is not supported");
  if (!bytes_consumed) return fail(STATS_E_ARG, "bytes_consumed is NULL");
  *bytes_consumed = 0;
  if (nbytes < 0) return fail(STATS_E_ARG, "nbytes < 0");
  if (h->p > 16) return fail(STATS_E_ARG, "text ingest supports p <= 16");
  if (nbytes == 0) return STATS_OK;
  if (!buf) return fail(STATS_E_ARG, "buf is NULL");
  DeviceGuard g(h->device);
  if (!g.ok) return fail(STATS_E_HIP, "hipSetDevice failed");
  const char* dbuf = buf;
  hipError_t e;
  if (mem_kind == STATS_MEM_HOST || mem_kind == STATS_MEM_HOST_PINNED) {
    int rc = ensure_dev(h, &h->aux_dev, &h->aux_cap, (size_t)nbytes);
    if (rc) return rc;
    e = hipMemcpyAsync(h->aux_dev, buf, (size_t)nbytes, hipMemcpyHostToDevice, h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "copying text to the device");
    dbuf = (const char*)h->aux_dev;
  } else if (mem_kind != STATS_MEM_DEVICE) {
    return fail(STATS_E_ARG, "unknown mem_kind");
  }
  int64_t nend = nbytes;
  // the last line end of a chunk that is not the last one, and the chunk's
  // line density (every chunk that waits for the first anyway, and a last
  // chunk when nothing was measured before)
  if (!is_last || !(h->text_ell > 0.0)) {
    int rc = ensure_dev(h, (void**)&h->raw_out, &h->raw_cap, 8 * (1 + kDensWin));
    if (rc) return rc;
    int64_t* ro = (int64_t*)h->raw_out;
    if (!is_last) hipLaunchKernelGGL(k_last_newline, dim3(1), dim3(1024), 0, h->stream, dbuf, nbytes, ro);
    hipLaunchKernelGGL(k_line_density, dim3(kDensWin), dim3(1024), 0, h->stream, dbuf, nbytes, ro + 1);
    e = hipGetLastError();
    int64_t hv[1 + kDensWin];
    hv[0] = nbytes;
    if (e == hipSuccess)
      e = hipMemcpyAsync(is_last ? hv + 1 : hv, is_last ? ro + 1 : ro, 8 * (is_last ? kDensWin : 1 + kDensWin),
                         hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "finding the last line end");
    nend = hv[0];
    int64_t lines = 0;
    for (int k = 1; k <= kDensWin; ++k) lines += hv[k];
    const int64_t counted = nbytes <= (int64_t)kDensWin * kDensBytes ? nbytes : (int64_t)kDensWin * kDensBytes;
    if (lines > 0) h->text_ell = (double)counted / (double)lines;
  }
  const int64_t base_off = h->text_offset;
  int rc = text_launch(h, dbuf, nbytes, nend, base_off);
  if (rc) return rc;
  if (mem_kind != STATS_MEM_DEVICE) {
    e = hipStreamSynchronize(h->stream);  // the staging copy may be reused by the next call
    if (e != hipSuccess) return hip_fail(h, e, "text ingest");
  }
  h->text_offset += nend;
  *bytes_consumed = nend;
  return STATS_OK;
}

extern "C" int stats_text_to_binary(stats_ctx* h, const char* buf, int64_t nbytes, int32_t mem_kind,
                                    int32_t is_last, void* const* out_planes, int64_t max_rows,
                                    int64_t* rows_out, int64_t* bytes_consumed) {
  if (!h) return fail(STATS_E_ARG, "handle is NULL");
  if (h->poisoned) return fail(STATS_E_STATE, "handle is poisoned by an earlier HIP error");
  if (h->ngroups) return fail(STATS_E_STATE, "groups handle: text conversion is not supported");
  if (!bytes_consumed || !rows_out) return fail(STATS_E_ARG, "rows_out or bytes_consumed is NULL");
  *bytes_consumed = 0;
  *rows_out = 0;
  if (nbytes < 0 || max_rows < 0) return fail(STATS_E_ARG, "nbytes or max_rows < 0");
  const int p = h->p;
  if (p > 16) return fail(STATS_E_ARG, "text conversion supports p <= 16");
  for (int c = 0; c < p; ++c) {
    const stats_column& col = h->cols[c];
    if (col.dtype == STATS_F32) return fail(STATS_E_ARG, "text conversion writes I32, I64 or F64 columns");
    if (!h->intf[c] && col.dtype != STATS_F64)
      return fail(STATS_E_ARG, "a decimal (non-integer) column must be stored as F64");
  }
  if (nbytes == 0) return STATS_OK;
  if (!buf || !out_planes) return fail(STATS_E_ARG, "buf or out_planes is NULL");
  for (int c = 0; c < p; ++c)
    if (!out_planes[h->cols[c].plane]) return fail(STATS_E_ARG, "an output plane is NULL");
  DeviceGuard g(h->device);
  if (!g.ok) return fail(STATS_E_HIP, "hipSetDevice failed");
  const char* dbuf = buf;
  hipError_t e;
  if (mem_kind == STATS_MEM_HOST || mem_kind == STATS_MEM_HOST_PINNED) {
    int rc = ensure_dev(h, &h->aux_dev, &h->aux_cap, (size_t)nbytes);
    if (rc) return rc;
    e = hipMemcpyAsync(h->aux_dev, buf, (size_t)nbytes, hipMemcpyHostToDevice, h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "copying text to the device");
    dbuf = (const char*)h->aux_dev;
  } else if (mem_kind != STATS_MEM_DEVICE) {
    return fail(STATS_E_ARG, "unknown mem_kind");
  }
  // scratch: line counts, then first rows, of the groups of units, first rows of
  // the units in them, the last line end, and a status word of its own (the
  // handle's statistics are not touched)
  const int64_t ngroups_max = (nbytes + kGroup * UNIT - 1) / (kGroup * UNIT);
  const size_t cnt_bytes = (size_t)ngroups_max * (8 + 4 * kGroup);
  const size_t need = (cnt_bytes + 255) / 256 * 256 + 256;
  int rc = ensure_dev(h, &h->conv_dev, &h->conv_cap, need);
  if (rc) return rc;
  int64_t* counts = (int64_t*)h->conv_dev;
  int32_t* first = (int32_t*)(counts + ngroups_max);
  char* tailp = (char*)h->conv_dev + (cnt_bytes + 255) / 256 * 256;
  int64_t* nend_dev = (int64_t*)tailp;
  DevStatus* cst = (DevStatus*)(tailp + 64);
  rc = ensure_pin(h, &h->pin_out, &h->pin_out_cap, 64);
  if (rc) return rc;
  int64_t* pin = (int64_t*)h->pin_out;  // number of lines, then the status
  int64_t nend = nbytes;
  if (!is_last) {
    hipLaunchKernelGGL(k_last_newline, dim3(1), dim3(1024), 0, h->stream, dbuf, nbytes, nend_dev);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&nend, nend_dev, 8, hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "finding the last line end");
  }
  if (nend == 0) return STATS_OK;
  const int64_t ngroups = (nend + kGroup * UNIT - 1) / (kGroup * UNIT);
  hipLaunchKernelGGL(k_unit_lines, dim3((unsigned)ngroups), dim3(64 * kGroup), 0, h->stream, dbuf, nend, counts, first);
  e = hipGetLastError();
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(1024), 0, h->stream, counts, ngroups, pin, cst);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_fail(h, e, "counting lines");
  const int64_t total = pin[0];
  if (total > max_rows)
    return fail(STATS_E_ARG, "the chunk holds " + std::to_string(total) + " lines, the output " +
                                 std::to_string(max_rows) + " rows");
  ConvArgs a;
  memset(&a, 0, sizeof a);
  a.t.buf = dbuf;
  a.t.nbytes = nbytes;
  a.t.nend = nend;
  a.t.p = p;
  a.t.base_off = h->text_offset;
  a.t.status = cst;
  const double ell = total > 0 ? (double)nend / (double)total : 0.0;
  a.t.seg = pick_text_seg(ell, p);
  a.t.maxls = pick_maxls(ell, a.t.seg);
  const int64_t nseg = (nend + a.t.seg - 1) / a.t.seg;
  for (int c = 0; c < p; ++c)
    if (h->intf[c]) a.t.intmask |= 1u << c;
  a.group_base = counts;
  a.first = first;
  for (int c = 0; c < p; ++c) {
    const stats_column& col = h->cols[c];
    a.out[c] = (char*)out_planes[col.plane] + col.byte_offset;
    a.stride[c] = h->row_stride[col.plane];
    a.dtype[c] = col.dtype;
  }
  switch (p) {
#define ST_CASE(PP) \
  case PP: launch_convert_p<PP>(a, nseg, h->stream); break;
    ST_CASE(1) ST_CASE(2) ST_CASE(3) ST_CASE(4) ST_CASE(5) ST_CASE(6) ST_CASE(7) ST_CASE(8)
    ST_CASE(9) ST_CASE(10) ST_CASE(11) ST_CASE(12) ST_CASE(13) ST_CASE(14) ST_CASE(15) ST_CASE(16)
#undef ST_CASE
  }
  e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(pin + 1, cst, sizeof(DevStatus), hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_fail(h, e, "text conversion");
  DevStatus st;
  memcpy(&st, pin + 1, sizeof st);
  h->text_offset += nend;
  if (st.bits & ST_PARSE)
    return fail(STATS_E_PARSE, "malformed or out-of-range field in the line starting at byte offset " +
                                   std::to_string((unsigned long long)st.parse_off));
  *rows_out = total;
  *bytes_consumed = nend;
  return STATS_OK;
}
