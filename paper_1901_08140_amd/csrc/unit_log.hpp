// Natural logarithm of x in [2^-53, 1] for the FP64 flight time -ln(1 - u)/nu'
// (eq. random_time), table-driven after P. T. P. Tang, "Table-driven implementation of the
// logarithm function in IEEE floating-point arithmetic", ACM TOMS 16 (1990):
//   x = 2^e m with m in [1, 2), and c = 1 + i/64 from the top six fraction bits of m;
//   with r = m RN(1/c) - 1 (one FMA, 0 <= r <= 2^-6),
//   ln x = e ln2 - ln RN(1/c) + log1p(r)   (exact in real arithmetic),
// the table holding RN(1/c) and -ln RN(1/c) as a sum of two doubles (hi + lo) for the 64
// values of i.  The lo part matters where e ln2 and -ln RN(1/c) nearly cancel (x just below
// 1 - 2^-7): their sum is then exact, and the table's own rounding would otherwise show.
// log1p(r) is its Taylor series to r^9 (truncation below 2^-57 relative).  Inputs within
// 2^-7 of 1 take r = x - 1 (exact) with e = 0 and no table term, so short flights keep full
// relative accuracy.  The table is built on the host in extended precision; the evaluation
// uses only IEEE-exact operations (FMA, sums), so host and
// device compute the same bits.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>

namespace swarm_impl {

constexpr int kUnitLogEntries = 64;          // table entries
constexpr int kUnitLogStride = 4;            // doubles per entry: RN(1/c), hi, lo, 0

// Table: entry i holds RN(1/c_i) and -ln RN(1/c_i) = hi + lo, c_i = 1 + i/64 (hi rounded to
// double, lo the rounded remainder, from the extended-precision logarithm).
inline void unit_log_table(double* tab) {
  for (int i = 0; i < kUnitLogEntries; ++i) {
    const double c = 1.0 + static_cast<double>(i) / 64.0;
    const double inv = 1.0 / c;
    const long double l = -logl(static_cast<long double>(inv));
    const double hi = static_cast<double>(l);
    tab[kUnitLogStride * i] = inv;
    tab[kUnitLogStride * i + 1] = hi;
    tab[kUnitLogStride * i + 2] = static_cast<double>(l - static_cast<long double>(hi));
    tab[kUnitLogStride * i + 3] = 0.0;
  }
}

// fma(a, b, c) with a constant c: on the device always the three-address form with c in a
// vector register (from fma() the compiler makes a move and the accumulating form in places,
// five moves in a trial; with c in scalar registers a lone wave was 2% slower).
__host__ __device__ inline double fma_const(double a, double b, double c) {
#ifdef __HIP_DEVICE_COMPILE__
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
#else
  return fma(a, b, c);
#endif
}

__host__ __device__ inline double unit_log(double x, const double* __restrict__ tab) {
  uint64_t bits;
  memcpy(&bits, &x, sizeof(bits));
  const uint32_t hi_word = static_cast<uint32_t>(bits >> 32);   // sign 0, exponent, 20 fraction bits
  // Within 2^-7 of 1, take m = x with exponent 0 and entry 0 (RN(1/c) = 1, no log term):
  // then r = x - 1 exactly.  Elsewhere m in [1, 2) is x with the exponent of 1.  One select, of
  // the high word that gives the exponent and the entry, serves all three (eight
  // instructions up to m, e and the entry's address, where frexp and selects took fourteen).
  const uint32_t sel = x > 0x1.fcp-1 ? 0x3ff00000u : hi_word;
  const int32_t neg_e = 1023 - static_cast<int32_t>(sel >> 20);
  // (the halves apart: a 64-bit sum takes three instructions for this one)
#ifdef __HIP_DEVICE_COMPILE__
  const double m = __hiloint2double(static_cast<int>(hi_word + (static_cast<uint32_t>(neg_e) << 20)), __double2loint(x));
#else
  const uint64_t m_bits = bits + (static_cast<uint64_t>(static_cast<uint32_t>(neg_e)) << 52);
  double m;
  memcpy(&m, &m_bits, sizeof(m));
#endif
  const double ed = -static_cast<double>(neg_e);
  // entry sel's top six fraction bits, as a byte offset
  static_assert(kUnitLogStride * sizeof(double) == 32 && kUnitLogEntries == 64);
  const double* t = reinterpret_cast<const double*>(reinterpret_cast<const char*>(tab) + ((sel >> 9) & 0x7e0u));
#ifdef __HIP_DEVICE_COMPILE__
  const double2 t01 = *reinterpret_cast<const double2*>(t);     // the table is 16-byte aligned in LDS
  const double inv = t01.x, log_hi = t01.y;
#else
  const double inv = t[0], log_hi = t[1];
#endif
  const double r = fma(m, inv, -1.0);
  double p = 1.0 / 9.0;
  p = fma_const(p, r, -1.0 / 8.0);
  p = fma_const(p, r, 1.0 / 7.0);
  p = fma_const(p, r, -1.0 / 6.0);
  p = fma_const(p, r, 1.0 / 5.0);
  p = fma_const(p, r, -1.0 / 4.0);
  p = fma_const(p, r, 1.0 / 3.0);
  p = fma(p, r, -0.5);
  const double lp = fma(r * r, p, r);                     // log1p(r)
  const double ln2_hi = 0x1.62e42fefa3800p-1;             // 42 significant bits: ed ln2_hi exact
  const double ln2_lo = 0x1.ef35793c76730p-45;
  const double hi = fma(ed, ln2_hi, log_hi);                // exact where the two terms cancel
  const double lo = fma(ed, ln2_lo, t[2] + lp);
  return hi + lo;
}

}  // namespace swarm_impl
