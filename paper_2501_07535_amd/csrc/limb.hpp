// limb.hpp - device-side multi-word modular arithmetic on 32-bit limbs (gfx950).
//
// A residue is L little-endian 32-bit limbs held in VGPRs (one lane = one
// element).  The modulus and its constants are uniform per launch and live in
// SGPRs (kernel arguments), so every word product has one SGPR operand.
//
// The paper decomposes a 2w-bit operation into w-bit operations recursively
// (Section 3, Table 1).  On gfx950 the machine word is the 32-bit VGPR lane,
// and the recursion is flattened into straight L-limb loops, unrolled at
// compile time (L is a template parameter), so no intermediate word size is
// materialised:
//   * add / subtract with carry and borrow chains (Section 2.2, rules (adc),
//     (addqdd), (subddd)) map to v_add_co_u32 / v_addc_co_u32 and
//     v_sub_co_u32 / v_subb_co_u32, with the carry bit delta held as a
//     64-bit lane mask in an SGPR pair;
//   * the conditional selects of Eqs. (saddmod) / (ssubmod) and rule
//     (moddq_add) map to v_cndmask_b32 on that mask;
//   * each 32x32->64 word product plus accumulation (rule (mulqdd)) is one
//     v_mad_u64_u32, whose carry-out feeds a third accumulator word through
//     one v_addc_co_u32 (product scanning, one column at a time).
// The instructions are written as small inline-asm statements because the
// compiler does not use the carry-out of v_mad_u64_u32 on its own; carries
// between statements travel in named SGPR-pair variables, never in VCC.
// gfx950 allows one constant-bus (SGPR) read per VALU instruction and the
// carry-in already uses it, so chained limbs take the modulus from a VGPR copy.
//
// Comparisons are canonical (>= q subtracts), not the strict comparisons
// printed in Eq. (saddmod) and Listing 1, so every output lies in [0, q).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace moma {

typedef uint32_t u32;
typedef uint64_t u64;

// A pointer that a kernel reads from memory (a batch record) is generic to the
// compiler, which then accesses it with flat loads and stores.  Those count on
// the LDS wait counter as well, so every wait for an LDS access also waits for
// the HBM accesses in flight.  The records hold device global addresses:
// reading the field as a global-space pointer lets the compiler use global
// loads and stores wherever the pointer goes.
template <class T>
__device__ __forceinline__ T* load_global_ptr(T* const* slot) {
  typedef __attribute__((address_space(1))) T* GlobalPtr;
  return (T*)*static_cast<const GlobalPtr*>(static_cast<const void*>(slot));
}

// A pointer from a uniform base (an SGPR pair, kept apart from the lane's part:
// the compiler would otherwise add the two per lane, in 64 bits) and a byte
// offset of the lane: one global access with both.
template <class T>
__device__ __forceinline__ const T& uniform_at(const void* base, u32 lane_bytes) {
  u64 b = (u64)base;
  asm volatile("" : "+s"(b));
  typedef const __attribute__((address_space(1))) char* GlobalBytes;
  typedef const __attribute__((address_space(1))) T* GlobalT;
  return *(const T*)(GlobalT)((GlobalBytes)b + lane_bytes);
}

template <class T>
__device__ __forceinline__ void uniform_put(void* base, u32 lane_bytes, const T& v) {
  u64 b = (u64)base;
  asm volatile("" : "+s"(b));
  typedef __attribute__((address_space(1))) char* GlobalBytes;
  typedef __attribute__((address_space(1))) T* GlobalT;
  *(T*)(GlobalT)((GlobalBytes)b + lane_bytes) = v;
}

// ----------------------------------------------------------------- word ops

// acc(64) += x * y; hi += carry-out.  x in a VGPR, y in a VGPR.
__device__ __forceinline__ void mac_vv(u64& acc, u32& hi, u32 x, u32 y) {
  u64 cy;
  asm("v_mad_u64_u32 %0, %1, %3, %4, %0\n\t"
      "v_addc_co_u32 %2, %1, %2, 0, %1"
      : "+v"(acc), "=&s"(cy), "+v"(hi)
      : "v"(x), "v"(y));
}

// acc(64) += x * y; hi += carry-out.  x in a VGPR, y uniform (SGPR).
__device__ __forceinline__ void mac_vs(u64& acc, u32& hi, u32 x, u32 y) {
  u64 cy;
  asm("v_mad_u64_u32 %0, %1, %3, %4, %0\n\t"
      "v_addc_co_u32 %2, %1, %2, 0, %1"
      : "+v"(acc), "=&s"(cy), "+v"(hi)
      : "v"(x), "s"(y));
}

// acc(64) += x1 * y1 + x2 * y2 with carries into hi; x in VGPRs, y1 VGPR, y2 uniform.
// One asm statement for two products halves the wait states the compiler
// inserts after every inline-asm block.
__device__ __forceinline__ void mac2_vv_vs(u64& acc, u32& hi, u32 x1, u32 y1, u32 x2, u32 y2) {
  u64 cy;
  asm("v_mad_u64_u32 %0, %1, %3, %4, %0\n\t"
      "v_addc_co_u32 %2, %1, %2, 0, %1\n\t"
      "v_mad_u64_u32 %0, %1, %5, %6, %0\n\t"
      "v_addc_co_u32 %2, %1, %2, 0, %1"
      : "+v"(acc), "=&s"(cy), "+v"(hi)
      : "v"(x1), "v"(y1), "v"(x2), "s"(y2));
}

// First products of a column: hi = carry-out (instead of hi += carry-out), so the
// carry word needs no zeroing move.
__device__ __forceinline__ void mac2_vv_vs_first(u64& acc, u32& hi, u32 x1, u32 y1, u32 x2, u32 y2) {
  u64 cy;
  asm("v_mad_u64_u32 %0, %1, %3, %4, %0\n\t"
      "v_addc_co_u32 %2, %1, 0, 0, %1\n\t"
      "v_mad_u64_u32 %0, %1, %5, %6, %0\n\t"
      "v_addc_co_u32 %2, %1, %2, 0, %1"
      : "+v"(acc), "=&s"(cy), "=&v"(hi)
      : "v"(x1), "v"(y1), "v"(x2), "s"(y2));
}

__device__ __forceinline__ void mac_vv_first(u64& acc, u32& hi, u32 x, u32 y) {
  u64 cy;
  asm("v_mad_u64_u32 %0, %1, %3, %4, %0\n\t"
      "v_addc_co_u32 %2, %1, 0, 0, %1"
      : "+v"(acc), "=&s"(cy), "=&v"(hi)
      : "v"(x), "v"(y));
}

// acc(64) += x * y with no carry-out (caller guarantees no overflow).
__device__ __forceinline__ void mad_vv(u64& acc, u32 x, u32 y) {
  u64 cy;
  asm("v_mad_u64_u32 %0, %1, %2, %3, %0" : "+v"(acc), "=s"(cy) : "v"(x), "v"(y));
}

// move the 96-bit column accumulator one word down: {acc, hi} >>= 32
__device__ __forceinline__ void shift_col(u64& acc, u32& hi) {
  acc = (acc >> 32) | ((u64)hi << 32);
  hi = 0;
}

// r = a + b over L limbs (a, b VGPR); returns the carry-out lane mask
template <int L>
__device__ __forceinline__ u64 add_vv(u32* r, const u32* a, const u32* b) {
  u64 cy;
  asm("v_add_co_u32 %0, %1, %2, %3" : "=v"(r[0]), "=s"(cy) : "v"(a[0]), "v"(b[0]));
#pragma unroll
  for (int i = 1; i < L; i++) asm("v_addc_co_u32 %0, %1, %2, %3, %1" : "=v"(r[i]), "+s"(cy) : "v"(a[i]), "v"(b[i]));
  return cy;
}

// r = a + q over L limbs (q uniform); returns the carry-out lane mask
template <int L>
__device__ __forceinline__ u64 add_vs(u32* r, const u32* a, const u32* q) {
  u64 cy;
  asm("v_add_co_u32 %0, %1, %2, %3" : "=v"(r[0]), "=s"(cy) : "v"(a[0]), "s"(q[0]));
#pragma unroll
  for (int i = 1; i < L; i++) asm("v_addc_co_u32 %0, %1, %2, %3, %1" : "=v"(r[i]), "+s"(cy) : "v"(a[i]), "v"(q[i]));
  return cy;
}

// r = a - b over L limbs (a, b VGPR); returns the borrow-out lane mask
template <int L>
__device__ __forceinline__ u64 sub_vv(u32* r, const u32* a, const u32* b) {
  u64 br;
  asm("v_sub_co_u32 %0, %1, %2, %3" : "=v"(r[0]), "=s"(br) : "v"(a[0]), "v"(b[0]));
#pragma unroll
  for (int i = 1; i < L; i++) asm("v_subb_co_u32 %0, %1, %2, %3, %1" : "=v"(r[i]), "+s"(br) : "v"(a[i]), "v"(b[i]));
  return br;
}

// r = a - q over L limbs (q uniform); returns the borrow-out lane mask
template <int L>
__device__ __forceinline__ u64 sub_vs(u32* r, const u32* a, const u32* q) {
  u64 br;
  asm("v_sub_co_u32 %0, %1, %2, %3" : "=v"(r[0]), "=s"(br) : "v"(a[0]), "s"(q[0]));
#pragma unroll
  for (int i = 1; i < L; i++) asm("v_subb_co_u32 %0, %1, %2, %3, %1" : "=v"(r[i]), "+s"(br) : "v"(a[i]), "v"(q[i]));
  return br;
}

// r[i] = mask ? x[i] : y[i] per lane
template <int L>
__device__ __forceinline__ void select(u32* r, u64 mask, const u32* x, const u32* y) {
#pragma unroll
  for (int i = 0; i < L; i++) asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(r[i]) : "v"(y[i]), "v"(x[i]), "s"(mask));
}

// ----------------------------------------------------------------- modular ops

// r = (a + b) mod q for a, b in [0, q), q < 2^(32L-1): sum, trial subtraction, select.
template <int L>
__device__ __forceinline__ void mod_add(u32* r, const u32* a, const u32* b, const u32* q) {
  u32 s[L], d[L];
  add_vv<L>(s, a, b);            // no carry-out: a + b < 2q < 2^(32L)
  u64 br = sub_vs<L>(d, s, q);   // borrow set  <=>  s < q
  select<L>(r, br, s, d);
}

// r = (a - b) mod q for a, b in [0, q): difference, add q back where it borrowed.
template <int L>
__device__ __forceinline__ void mod_sub(u32* r, const u32* a, const u32* b, const u32* q) {
  u32 d[L], e[L];
  u64 br = sub_vv<L>(d, a, b);
  add_vs<L>(e, d, q);
  select<L>(r, br, e, d);
}

// r = x mod q for x in [0, 2q): one trial subtraction.
template <int L>
__device__ __forceinline__ void reduce_once(u32* r, const u32* x, const u32* q) {
  u32 d[L];
  u64 br = sub_vs<L>(d, x, q);
  select<L>(r, br, x, d);
}

// Montgomery product t = a * b * 2^(-32L) (mod q), left in [0, 2q) (Montgomery,
// Math. Comp. 1985), product-scanning form: column i accumulates every a_j*b_{i-j}
// and m_j*q_{i-j}, then m_i = (column low word) * (-q^-1 mod 2^32) zeroes the low
// word.  Requires a*b < 4q^2 (e.g. a < 4q, b < q) and 4q <= 2^(32L); then
// t = (ab + mq) / 2^(32L) < 2q.  qinv = -q^{-1} mod 2^32.
// 2L^2 + L word products (as counted for Montgomery multiplication).
template <int L>
__device__ __forceinline__ void mont_mul_lazy(u32* t, const u32* a, const u32* b, const u32* q, u32 qinv) {
  u32 m[L];
  u64 acc = 0;
  u32 hi;
#pragma unroll
  for (int i = 0; i < L; i++) {
    if (i == 0) {
      mac_vv_first(acc, hi, a[0], b[0]);
    } else {
      mac2_vv_vs_first(acc, hi, a[0], b[i], m[0], q[i]);
#pragma unroll
      for (int j = 1; j < i; j++) mac2_vv_vs(acc, hi, a[j], b[i - j], m[j], q[i - j]);
      mac_vv(acc, hi, a[i], b[0]);
    }
    m[i] = (u32)acc * qinv;
    mac_vs(acc, hi, m[i], q[0]);
    acc = (acc >> 32) | ((u64)hi << 32);
  }
#pragma unroll
  for (int i = L; i < 2 * L; i++) {
    if (i - L + 1 < L) {
      mac2_vv_vs_first(acc, hi, a[i - L + 1], b[L - 1], m[i - L + 1], q[L - 1]);
#pragma unroll
      for (int j = i - L + 2; j < L; j++) mac2_vv_vs(acc, hi, a[j], b[i - j], m[j], q[i - j]);
      t[i - L] = (u32)acc;
      acc = (acc >> 32) | ((u64)hi << 32);
    } else {
      t[i - L] = (u32)acc;  // last column: no products left, only the carried word
    }
  }
  // t < 2q < 2^(32L): the final carry word is zero
}

// Montgomery product reduced to [0, q): a, b in [0, q).
template <int L>
__device__ __forceinline__ void mont_mul(u32* r, const u32* a, const u32* b, const u32* q, u32 qinv) {
  u32 t[L];
  mont_mul_lazy<L>(t, a, b, q, qinv);
  reduce_once<L>(r, t, q);
}

// ----------------------------------------------------------------- digit form
//
// The paper's multi-digit numbers may use any digit base z (Eq. (def_mp)).  For
// the transform's twiddle multiply, residues are re-expressed in base 2^b with
// b = 29 (28 above 28 limbs) and D digits, chosen so that a column of 2D digit
// products plus the carried word stays below 2^64.  Every word product is then
// one v_mad_u64_u32 into a 64-bit accumulator with no carry handling, which the
// compiler emits from plain C.  Operands stay in 32-bit limbs everywhere else;
// the multiply converts on the way in and out.
template <int L, bool FW = false>
struct Digits {
  static constexpr int b = digit_bits(L);
  static constexpr int D = digit_count(L, FW);
  static constexpr u32 mask = (1u << b) - 1;
};

// d = y 2^OFF in base 2^b (below 2^(b*D))
template <int L, bool FW = false, int OFF = 0>
__device__ __forceinline__ void to_digits(u32* d, const u32* y) {
  constexpr int b = Digits<L, FW>::b, D = Digits<L, FW>::D;
#pragma unroll
  for (int i = 0; i < D; i++) {
    constexpr u32 m = Digits<L, FW>::mask;
    const int pos = b * i - OFF;  // y's bit at the digit's bit 0
    if (pos < 0) {
      d[i] = pos <= -b ? 0u : (y[0] << (-pos & 31)) & m;
      continue;
    }
    const int l = pos / 32, s = pos % 32;
    u32 lo = l < L ? y[l] : 0u, hi = l + 1 < L ? y[l + 1] : 0u;
    u32 v = s ? __builtin_amdgcn_alignbit(hi, lo, s) : lo;
    d[i] = v & m;
  }
}

// t = y * w * 2^(-bD) mod q in [0, 2q), w given as digits (Montgomery form for
// R = 2^(bD)), y < 4q in 32-bit limbs (y < q for a full-width modulus, FW).
// Product scanning: column i sums every digit product y_j w_{i-j} and
// m_j q_{i-j}; m_i = (low b bits) * qinvd mod 2^b clears the low b bits, then
// the column shifts right by b.  2D^2 products.  FW: the result may reach
// 2^(32L); *top receives its bit 32L (0 or 1).
template <int L, bool FW = false>
__device__ __forceinline__ void mont_mul_digits(u32* t, const u32* y, const u32* wd, const u32* qd, u32 qinvd,
                                                u32* top = nullptr) {
  constexpr int b = Digits<L, FW>::b, D = Digits<L, FW>::D;
  constexpr u32 mask = Digits<L, FW>::mask;
  static_assert(b * D >= 32 * L - (FW ? 0 : 2), "the digits cover the result limbs");
  u32 a[D], m[D];
  to_digits<L, FW>(a, y);
  u64 acc = 0;
#pragma unroll
  for (int i = 0; i < D; i++) {
#pragma unroll
    for (int j = 0; j <= i; j++) acc += (u64)a[j] * wd[i - j];
#pragma unroll
    for (int j = 0; j < i; j++) acc += (u64)m[j] * qd[i - j];
    m[i] = ((u32)acc * qinvd) & mask;
    acc += (u64)m[i] * qd[0];
    acc >>= b;
  }
  // the upper columns give the result digits; each result limb leaves as soon
  // as its 32 bits are known (digit positions are compile-time constants), so
  // the digits are never all live at once
  u64 bits = 0;
  int nb = 0, j = 0;
#pragma unroll
  for (int i = D; i < 2 * D; i++) {
    u32 dig;
    if (i < 2 * D - 1) {
#pragma unroll
      for (int jj = i - D + 1; jj < D; jj++) acc += (u64)a[jj] * wd[i - jj] + (u64)m[jj] * qd[i - jj];
      dig = (u32)acc & mask;
      acc >>= b;
    } else {
      dig = (u32)acc;  // the last digit carries everything above
    }
    bits |= (u64)dig << nb;
    nb += b;
    while (nb >= 32 && j < L) {
      t[j++] = (u32)bits;
      bits >>= 32;
      nb -= 32;
    }
  }
  // bD is at least 32L - 2 (at least 32L for a full-width modulus), so at most
  // the top limb is still in the buffer here: its bits above bD come from the
  // last digit, which is wider than b
  if (j < L) t[j] = (u32)bits;
  if constexpr (FW) *top = (u32)bits;  // bit 32L of a full-width result below 2q
}

// Fixed-operand product (Shoup's method as in Harvey, "Faster arithmetic for
// number-theoretic transforms", J. Symb. Comp. 2014, carried to digits): the
// table holds the twiddle w < q and its scaled quotient wq = floor(w R / q),
// R = 2^(bD).  With m = floor(wq y / R),
//   t = w y - m q   lies in [0, 2q) and needs only its low D digits.
// So one product is taken from its top columns, two from their low ones: about
// 3/2 D^2 digit products, and no reduction multiply per column, against 2 D^2
// plus D multiplies for the Montgomery product scan.
//   * Quotient: columns D-2 .. 2D-2 of wq y.  The columns left out weigh less
//     than (D-2) 2^-b R together, so m is floor(w y / q) or one less whenever
//     y / R + (D-2) 2^-b < 1 (y < 4q: digit_count keeps y <= R/2).
//   * t = low digits of (w y + m nq), nq = R - q: sums only.  A column holds
//     2D digit products plus the carried word, as in the product scan.
//   * t leaves as 32-bit limbs, two instructions per digit: a digit is shifted
//     to the top of its word and one alignbit joins it with the next.
// What bounds it is the issue of v_mad_u64_u32 (about 5 cycles of a SIMD each,
// against 2.5 to 4.5 for the other integer instructions).  With the tile layout
// in LDS and the uniform addressing that came with it, against the Montgomery
// product scan: 245 instead of 306 VALU instructions per 256-bit butterfly;
// 2^20 points 126.3 -> 119.4 us at 256 bits, 1248 -> 1013 us at 1024 bits; 2^14
// points at 384 bits 39.0 -> 31.4 us.
// (Summing two columns side by side, for independent chains where a SIMD has
// only one wave, was no faster: 256 bits, 2^12 points 20.8 -> 21.1 us.)
template <int L, bool FW = false>
__device__ __forceinline__ void quot_digits(u32* m, const u32* a, const u32* wq) {
  constexpr int b = Digits<L, FW>::b, D = Digits<L, FW>::D;
  u64 acc = 0;
#pragma unroll
  for (int c = D - 2; c <= 2 * D - 2; c++) {
#pragma unroll
    for (int j = (c < D ? 0 : c - D + 1); j <= (c < D ? c : D - 1); j++) acc += (u64)a[j] * wq[c - j];
    if (c >= D) m[c - D] = (u32)acc & Digits<L, FW>::mask;
    acc >>= b;
  }
  m[D - 1] = (u32)acc;
}

// limbs of floor(value / 2^OFF), the value given as raw columns: raw[i]'s low b
// bits are digit i (the bits above are ignored, except in the last digit)
template <int L, bool FW = false, int OFF = 0>
__device__ __forceinline__ void raw_to_limbs(u32* t, const u32* raw, u32* top) {
  constexpr int b = Digits<L, FW>::b, D = Digits<L, FW>::D;
  u32 hi[D];  // the digit at the top of its word
#pragma unroll
  for (int i = 0; i < D - 1; i++) hi[i] = raw[i] << (32 - b);
#pragma unroll
  for (int j = 0; j <= L; j++) {
    if (j == L && !FW) break;
    const int pos = 32 * j + OFF, i = pos / b, s = pos % b;  // the limb's lowest bit: bit s of digit i
    u32 v;
    if (i >= D) {
      v = 0;
    } else if (i == D - 1) {
      v = raw[i] >> s;
    } else {
      // digit i from bit s up, then digit i + 1, then i + 2 where those are less than 32 bits
      const int have = 2 * b - s;
      v = __builtin_amdgcn_alignbit(raw[i + 1], hi[i], 32 - b + s);
      if (have < 32 && i + 1 < D - 1) {
        v = (hi[i] >> (32 - b + s)) | ((raw[i + 1] << (32 - b)) >> (32 - b) << (b - s));
        if (i + 2 < D) v |= raw[i + 2] << have;
      }
    }
    if (j < L)
      t[j] = v;
    else
      *top = v;
  }
}

template <int L, bool FW = false>
__device__ __forceinline__ void quot_mul(u32* t, const u32* y, const u32* w, const u32* wq, const u32* nqd,
                                         u32* top = nullptr) {
  constexpr int b = Digits<L, FW>::b, D = Digits<L, FW>::D;
  u32 a[D], m[D], raw[D];
  to_digits<L, FW>(a, y);
  quot_digits<L, FW>(m, a, wq);
  u64 acc = 0;
#pragma unroll
  for (int i = 0; i < D; i++) {
#pragma unroll
    for (int j = 0; j <= i; j++) {
      acc += (u64)a[j] * w[i - j];
      acc += (u64)m[j] * nqd[i - j];
    }
    // the last column's high word is not needed, but left to see that the
    // compiler takes a mul_lo and half an add3 in place of each v_mad_u64_u32
    if (i == D - 1) asm("" : "+v"(acc));
    raw[i] = (u32)acc;
    acc >>= b;
  }
  raw[D - 1] &= Digits<L, FW>::mask;  // t < 2q <= R: what is above is the discarded multiple of R
  raw_to_limbs<L, FW>(t, raw, top);
}

// The same product with w y by one level of Karatsuba (Eq. (mulk)) on the
// digits, of which the low D columns are needed: with y = y1 B^h + y0 and
// w = w1 B^h + w0 (B = 2^b, h = ceil(D/2)), w y = z0 + z1 B^h + ... where
// z1 = (y0 + y1)(w0 + w1) - z0 - z2.  The digit sums have b + 1 bits and need
// no carry; every product column is gathered as an exact 64-bit sum (it
// equals the schoolbook column).
template <int L>
__device__ __forceinline__ void quot_mul_kara(u32* t, const u32* y, const u32* w, const u32* wq, const u32* nqd) {
  constexpr int b = Digits<L>::b, D = Digits<L>::D, h = (D + 1) / 2, g = D - h;
  u32 a[D], m[D], raw[D], sa[h], sw[h];
  to_digits<L>(a, y);
  quot_digits<L>(m, a, wq);
#pragma unroll
  for (int i = 0; i < h; i++) {
    sa[i] = a[i] + (i < g ? a[h + i] : 0u);
    sw[i] = w[i] + (i < g ? w[h + i] : 0u);
  }
  u64 p[D];
#pragma unroll
  for (int c = 0; c < D; c++) p[c] = 0;
#pragma unroll
  for (int c = 0; c < (2 * h - 1 < D ? 2 * h - 1 : D); c++) {
    u64 z0 = 0;
#pragma unroll
    for (int i = (c < h ? 0 : c - h + 1); i <= (c < h ? c : h - 1); i++) z0 += (u64)a[i] * w[c - i];
    p[c] += z0;
    if (c + h < D) {
      u64 zm = 0, z2 = 0;
#pragma unroll
      for (int i = 0; i <= c; i++) {
        zm += (u64)sa[i] * sw[c - i];
        if (i < g && c - i < g) z2 += (u64)a[h + i] * w[h + c - i];
      }
      p[c + h] += zm - z0 - z2;  // the cross terms: exact, non-negative
    }
  }
  u64 acc = 0;
#pragma unroll
  for (int i = 0; i < D; i++) {
    acc += p[i];
#pragma unroll
    for (int j = 0; j <= i; j++) acc += (u64)m[j] * nqd[i - j];
    raw[i] = (u32)acc;
    acc >>= b;
  }
  raw[D - 1] &= Digits<L>::mask;
  raw_to_limbs<L>(t, raw, nullptr);
}

// ----------------------------------------------------------------- full width
//
// A full-width modulus (bitlen(q) > 32L - 4) leaves no headroom for the lazy
// reductions: operands stay canonical in [0, q), and a sum or a Montgomery
// product below 2q can carry out of the top limb, so that bit travels in a
// word of its own beside the L limbs (Section 5.2 names Montgomery
// multiplication for such moduli).

// r = (top 2^(32L) + t) mod q for a value below 2q (top in {0, 1}): the
// (L+1)-word trial subtraction's final borrow says whether the value is < q.
template <int L>
__device__ __forceinline__ void reduce_top(u32* r, const u32* t, u32 top, const u32* qv) {
  u32 d[L], dt;
  u64 br = sub_vv<L>(d, t, qv);
  asm("v_subb_co_u32 %0, %1, %2, 0, %1" : "=v"(dt), "+s"(br) : "v"(top));
  select<L>(r, br, t, d);
}

// r = (a + b) mod q for a, b in [0, q), q < 2^(32L) (the sum may carry out)
template <int L>
__device__ __forceinline__ void mod_add_fw(u32* r, const u32* a, const u32* b, const u32* qv) {
  u32 s[L], top;
  u64 cy = add_vv<L>(s, a, b);
  asm("v_addc_co_u32 %0, %1, 0, 0, %1" : "=v"(top), "+s"(cy));
  reduce_top<L>(r, s, top, qv);
}

// r = (a - b) mod q for a, b in [0, q): the difference wraps below zero by
// exactly 2^(32L), which adding q takes back (no headroom needed)
template <int L>
__device__ __forceinline__ void mod_sub_v(u32* r, const u32* a, const u32* b, const u32* qv) {
  u32 d[L], e[L];
  u64 br = sub_vv<L>(d, a, b);
  add_vv<L>(e, d, qv);
  select<L>(r, br, e, d);
}

// Canonical butterfly for a full-width modulus: x, y in [0, q), twiddle in
// digit form; x' = (x + wy) mod q, y' = (x - wy) mod q.
template <int L>
__device__ __forceinline__ void ct_butterfly_fw(u32* x, u32* y, const u32* w, const u32* wq, const u32* nqd,
                                                const u32* qv) {
  u32 t[L], tr[L], top;
  quot_mul<L, true>(t, y, w, wq, nqd, &top);
  reduce_top<L>(tr, t, top, qv);
  u32 s[L], d[L];
#pragma unroll
  for (int j = 0; j < L; j++) s[j] = x[j];
  mod_add_fw<L>(x, s, tr, qv);
  mod_sub_v<L>(d, s, tr, qv);
#pragma unroll
  for (int j = 0; j < L; j++) y[j] = d[j];
}

// The same with twiddle 1: (x + y, x - y) mod q.
template <int L>
__device__ __forceinline__ void ct_butterfly_one_fw(u32* x, u32* y, const u32* qv) {
  u32 s[L], d[L];
#pragma unroll
  for (int j = 0; j < L; j++) s[j] = x[j];
  mod_add_fw<L>(x, s, y, qv);
  mod_sub_v<L>(d, s, y, qv);
#pragma unroll
  for (int j = 0; j < L; j++) y[j] = d[j];
}

// Montgomery product for a full-width modulus, 32-bit limbs (the form of
// mont_mul_lazy): t = a b 2^(-32L) mod q in [0, q) for a, b in [0, q).  The
// value (ab + mq) / 2^(32L) < 2q may reach 2^(32L); its carry word is kept and
// folded into the final trial subtraction.
template <int L>
__device__ __forceinline__ void mont_mul_fw(u32* r, const u32* a, const u32* b, const u32* q, u32 qinv,
                                            const u32* qv) {
  u32 m[L], t[L];
  u64 acc = 0;
  u32 hi;
#pragma unroll
  for (int i = 0; i < L; i++) {
    if (i == 0) {
      mac_vv_first(acc, hi, a[0], b[0]);
    } else {
      mac2_vv_vs_first(acc, hi, a[0], b[i], m[0], q[i]);
#pragma unroll
      for (int j = 1; j < i; j++) mac2_vv_vs(acc, hi, a[j], b[i - j], m[j], q[i - j]);
      mac_vv(acc, hi, a[i], b[0]);
    }
    m[i] = (u32)acc * qinv;
    mac_vs(acc, hi, m[i], q[0]);
    acc = (acc >> 32) | ((u64)hi << 32);
  }
  u32 top = 0;
#pragma unroll
  for (int i = L; i < 2 * L; i++) {
    if (i - L + 1 < L) {
      mac2_vv_vs_first(acc, hi, a[i - L + 1], b[L - 1], m[i - L + 1], q[L - 1]);
#pragma unroll
      for (int j = i - L + 2; j < L; j++) mac2_vv_vs(acc, hi, a[j], b[i - j], m[j], q[i - j]);
      t[i - L] = (u32)acc;
      acc = (acc >> 32) | ((u64)hi << 32);
    } else {
      t[i - L] = (u32)acc;  // last column: only the carried words are left
      top = (u32)(acc >> 32);
    }
  }
  reduce_top<L>(r, t, top, qv);
}

// Copy uniform words into VGPRs once, opaquely, so carry chains that need the
// operand in a VGPR do not re-copy it from SGPRs at every use.
template <int L>
__device__ __forceinline__ void to_vgprs(u32* dst, const u32* src) {
#pragma unroll
  for (int i = 0; i < L; i++) asm volatile("v_mov_b32 %0, %1" : "=v"(dst[i]) : "s"(src[i]));
}

// Harvey's lazy butterfly with twiddle 1 (the first stages of a transform), with
// t = y mod 2q in [0, 2q) in place of the product w*y.
template <int L>
__device__ __forceinline__ void ct_butterfly_one(u32* x, u32* y, const u32* q2v) {
  u32 xr[L], t[L], d[L], s[L];
  u64 br = sub_vv<L>(s, x, q2v);
  select<L>(xr, br, x, s);
  br = sub_vv<L>(s, y, q2v);
  select<L>(t, br, y, s);
  add_vv<L>(x, xr, t);
  sub_vv<L>(d, xr, t);
  add_vv<L>(y, d, q2v);
}

// Lazy butterflies.  With 4 spare bits above q (and digits that cover all 32L
// bits: spare_bits, every headroom limb count but 10) a value may be anything
// in [0, 16q), and a multiplying butterfly is two additions,
//   t <- w*y in [0, g q);  x' = x + t;  y' = x - t,   g = 1 + 2^(32L-bD) + e,
// where e < (D - 2) 2^-b is what the quotient's dropped columns weigh (2^-22.9 at
// 32 limbs), as long as x stays between t and 16q - t: stages move the bounds by
// g q each way (growth_64th, in 64ths, with 1/64 for e).  Where the next stages
// would leave [0, 16q), the x of the first of them are moved to 7q and up to 1/64
// above 8q (offset_reduce): with five or six stages in a pass that is once per
// pass, against a trial subtraction of x and an addition of 2q in every butterfly
// (Harvey, "Faster arithmetic for number-theoretic transforms", J. Symb. Comp.
// 2014: values in [0, 4q)).
constexpr int spare_bits(int L) { return digit_bits(L) * digit_count(L) - 32 * L; }
constexpr u32 growth_of(int spare) { return 64 + (64 >> (spare < 0 ? 0 : spare < 6 ? spare : 6)) + 1; }
template <int L>
constexpr u32 growth_64th = growth_of(spare_bits(L));

// r = x - (f - off) q for x in [0, 16q), where f is floor(x / q) or, when x / q
// is less than 19 2^-27 above it, one less: r in [off q, (off + 1 + 19 2^-27) q)
// (the bounds of a pass take 1/64 for it).  f comes from the top 32 bits of x 2^d
// and cinv; the multiple of q is formed in signed words.
template <int L>
__device__ __forceinline__ void offset_reduce(u32* x, u32 off, const u32* qsw, u32 d, u32 cinv) {
  const u32 xt = (u32)((((u64)x[L - 1] << 32 | x[L - 2]) << d) >> 32);
  const int k = (int)(off - (__umulhi(xt, cinv) >> 26));
  u32 p[L];
  int64_t acc = 0;
#pragma unroll
  for (int i = 0; i < L; i++) {
    acc = (acc >> 32) + (int64_t)k * (int32_t)qsw[i];
    p[i] = (u32)acc;
  }
  u32 r[L];
  add_vv<L>(r, x, p);
#pragma unroll
  for (int i = 0; i < L; i++) x[i] = r[i];
}

// Harvey's form of the additions, t = w*y in [0, 2q) known:
//   x <- x mod 2q;  x' = x + t;  y' = x - t + 2q.
template <int L>
__device__ __forceinline__ void ct_lazy_tail(u32* x, u32* y, const u32* t, const u32* q2v) {
  u32 xr[L], d[L], s[L];
  u64 br = sub_vv<L>(s, x, q2v);
  select<L>(xr, br, x, s);
  add_vv<L>(x, xr, t);
  sub_vv<L>(d, xr, t);
  add_vv<L>(y, d, q2v);
}

// The additions of a lazy butterfly.  FIRST (the transform's first round, which
// starts from canonical x below what an offset needs): x' = x + t, y' = x - t + 2q.
template <int L, bool OFF, bool FIRST>
__device__ __forceinline__ void ct_tail(u32* x, u32* y, const u32* t, const u32* q2v) {
  if constexpr (!OFF) {
    ct_lazy_tail<L>(x, y, t, q2v);
  } else {
    u32 s[L], d[L];
    add_vv<L>(s, x, t);
    sub_vv<L>(d, x, t);
    if constexpr (FIRST) {
      add_vv<L>(y, d, q2v);
    } else {
#pragma unroll
      for (int i = 0; i < L; i++) y[i] = d[i];
    }
#pragma unroll
    for (int i = 0; i < L; i++) x[i] = s[i];
  }
}

// (x + y, x - y + cq) for x, y below cq: the first round's pairs with twiddle 1
template <int L>
__device__ __forceinline__ void ct_one_tail(u32* x, u32* y, const u32* cqv) {
  u32 s[L], d[L];
  add_vv<L>(s, x, y);
  sub_vv<L>(d, x, y);
  add_vv<L>(y, d, cqv);
#pragma unroll
  for (int i = 0; i < L; i++) x[i] = s[i];
}

// Multiplying butterfly, the product w y by schoolbook or (KARA) Karatsuba columns.
template <int L, bool KARA, bool OFF, bool FIRST>
__device__ __forceinline__ void ct_butterfly_mul(u32* x, u32* y, const u32* w, const u32* wq, const u32* nqd,
                                                 const u32* q2v) {
  u32 t[L];
  if constexpr (KARA)
    quot_mul_kara<L>(t, y, w, wq, nqd);
  else
    quot_mul<L>(t, y, w, wq, nqd);
  ct_tail<L, OFF, FIRST>(x, y, t, q2v);
}

// The same for a full-width modulus: t (with its carry word) reduced, then
// (x + t, x - t) mod q.
template <int L>
__device__ __forceinline__ void ct_fw_tail(u32* x, u32* y, const u32* t, u32 top, const u32* qv) {
  u32 tr[L], s[L];
  reduce_top<L>(tr, t, top, qv);
#pragma unroll
  for (int j = 0; j < L; j++) s[j] = x[j];
  mod_add_fw<L>(x, s, tr, qv);
  mod_sub_v<L>(y, s, tr, qv);
}

// Barrett multiplication (Eq. (barrett), Listing 4 generalised) in digits.  The
// first operand is scaled so that the modulus qn = q 2^(d + off) has exactly
// N = bD - 1 bits: by d in 32-bit words (W0 - bitlen(q), below 32; 0 for the
// classes' own moduli) and by a fixed `off` in the way its digits are cut, which
// puts every shift of the reduction on a digit boundary.
//   P = a 2^(d + off) b;  m = floor(floor(P / B^(D-1)) mu / B^(D+1)),
//   mu = floor(B^(2D) / qn) (its top digit takes the bits above bD, below 2^31);
//   P - m qn in [0, 2 qn): one correction, then both scalings undone.
// P has all its D^2 digit products; mu's product is taken from its columns D-1
// and up (those below weigh less than 2^-b D of m's unit) and the last one mod
// B^D: 2D^2 + 2D products, one v_mad_u64_u32 each, where the same method on
// 32-bit words took 2.5 L^2 products of two instructions.
// Bound by the issue of those products from 12 limbs on, by memory below:
// 2^24 products at 768 bits took 1534 us in words, 1202 us so.  (Up to 4 limbs the
// digits are more instructions than the words: kWordLimbsVmul.)
// m is floor(P / qn) or one less: what P loses below B^(D-1) and mu below 1
// takes off less than 2^(2-b) and 2^(W0 - bD) <= 1/2 of m's unit.
template <int L, bool FW = false>
struct BarrettC {
  static constexpr int W0 = FW ? 32 * L : 32 * L - 4;
  static constexpr int off = barrett_off(L, FW);
  u32 mu[Digits<L, FW>::D];
  u32 nqn[Digits<L, FW>::D];  // B^D - qn
  u32 qs[L];                  // q 2^d
  u32 d;
};

template <int L, bool FW = false>
__device__ __forceinline__ void barrett_mul_digits(u32* r, const u32* a, const u32* b, const BarrettC<L, FW>& c) {
  constexpr int bits = Digits<L, FW>::b, D = Digits<L, FW>::D, off = BarrettC<L, FW>::off;
  constexpr u32 mask = Digits<L, FW>::mask;
  u32 as[L];
  if (c.d == 0) {
#pragma unroll
    for (int i = 0; i < L; i++) as[i] = a[i];
  } else {
    as[0] = a[0] << c.d;
#pragma unroll
    for (int i = 1; i < L; i++) as[i] = __builtin_amdgcn_alignbit(a[i], a[i - 1], 32 - c.d);
  }
  u32 p[2 * D], m[D], raw[D];
  {
    u32 x[D], y[D];
    to_digits<L, FW, off>(x, as);
    to_digits<L, FW>(y, b);
    u64 acc = 0;
#pragma unroll
    for (int k = 0; k < 2 * D - 1; k++) {
#pragma unroll
      for (int j = (k < D ? 0 : k - D + 1); j <= (k < D ? k : D - 1); j++) acc += (u64)x[j] * y[k - j];
      p[k] = (u32)acc & mask;
      acc >>= bits;
    }
    p[2 * D - 1] = (u32)acc;
  }
  u64 acc = 0;
#pragma unroll
  for (int k = D - 1; k < 2 * D; k++) {
#pragma unroll
    for (int i = k - D + 1; i <= (k < D ? k : D); i++) acc += (u64)p[D - 1 + i] * c.mu[k - i];
    if (k > D) m[k - D - 1] = (u32)acc & mask;
    acc >>= bits;
  }
  m[D - 1] = (u32)acc;
  acc = 0;
#pragma unroll
  for (int i = 0; i < D; i++) {
    acc += p[i];
#pragma unroll
    for (int j = 0; j <= i; j++) acc += (u64)m[j] * c.nqn[i - j];
    if (i == D - 1) asm("" : "+v"(acc));  // as in quot_mul
    raw[i] = (u32)acc;
    acc >>= bits;
  }
  raw[D - 1] &= mask;
  u32 t[L], red[L], top;
  raw_to_limbs<L, FW, off>(t, raw, &top);
  if constexpr (FW)
    reduce_top<L>(red, t, top, c.qs);
  else
    reduce_once<L>(red, t, c.qs);
  if (c.d == 0) {
#pragma unroll
    for (int i = 0; i < L; i++) r[i] = red[i];
  } else {
#pragma unroll
    for (int i = 0; i < L - 1; i++) r[i] = __builtin_amdgcn_alignbit(red[i + 1], red[i], c.d);
    r[L - 1] = red[L - 1] >> c.d;
  }
}

// Constants of the form on 32-bit words, following Listings 1 and 4 generalised
// to L limbs.  The modulus is pre-scaled to qn = q * 2^d with bitlen(qn) = M = 32L-4,
// so the paper's shifts by M-2 and M+5 fall at fixed limb/bit positions:
// mu = floor(2^(2M+3) / qn) < 2^(M+4) = 2^(32L).
template <int L>
struct BarrettWordC {
  u32 qn[L];
  u32 mu[L];
  u32 d;
};

// t[0 .. M+N) = a[0 .. M) * b[0 .. N), product scanning, both operands in VGPRs
template <int M, int N>
__device__ __forceinline__ void mul_ps(u32* t, const u32* a, const u32* b) {
  u64 acc = 0;
  u32 hi = 0;
#pragma unroll
  for (int k = 0; k < M + N - 1; k++) {
#pragma unroll
    for (int i = (k < N ? 0 : k - N + 1); i <= (k < M ? k : M - 1); i++) mac_vv(acc, hi, a[i], b[k - i]);
    t[k] = (u32)acc;
    shift_col(acc, hi);
  }
  t[M + N - 1] = (u32)acc;
}

// t[0 .. 2L) = a * b by one level of Karatsuba (Eq. (mulk)), subtractive form:
// with a = a1 B^h + a0, b = b1 B^h + b0 (B = 2^32, h = ceil(L/2)),
//   a b = z2 B^(2h) + (z0 + z2 - s |a0 - a1| |b0 - b1|) B^h + z0,
//   z0 = a0 b0, z2 = a1 b1, s = sign((a0 - a1)(b0 - b1)).
// Three half-size products (3 ceil(L/2)^2 word products instead of L^2); the
// differences need no carry bit, at the price of the sign selects.
template <int L>
__device__ __forceinline__ void kara_mul(u32* t, const u32* a, const u32* b) {
  constexpr int h = (L + 1) / 2, g = L - h;  // a0, b0: h limbs; a1, b1: g <= h limbs
  u32 z0[2 * h], z2[2 * g], p[2 * h];
  mul_ps<h, h>(z0, a, b);
  mul_ps<g, g>(z2, a + h, b + h);
  u32 a1[h], b1[h], da[h], da2[h], db[h], db2[h];
#pragma unroll
  for (int i = 0; i < h; i++) {
    a1[i] = i < g ? a[h + i] : 0u;
    b1[i] = i < g ? b[h + i] : 0u;
  }
  u64 sa = sub_vv<h>(da, a, a1);  // borrow <=> a0 < a1
  sub_vv<h>(da2, a1, a);
  select<h>(da, sa, da2, da);
  u64 sb = sub_vv<h>(db, b, b1);
  sub_vv<h>(db2, b1, b);
  select<h>(db, sb, db2, db);
  mul_ps<h, h>(p, da, db);
  // mid = z0 + z2 -/+ p: a0 b1 + a1 b0 >= 0, at most 2h + 1 limbs
  constexpr int W = 2 * h + 1;
  u32 x0[W], x2[W], xp[W], m[W], mp[W], mm[W];
#pragma unroll
  for (int i = 0; i < W; i++) {
    x0[i] = i < 2 * h ? z0[i] : 0u;
    x2[i] = i < 2 * g ? z2[i] : 0u;
    xp[i] = i < 2 * h ? p[i] : 0u;
  }
  add_vv<W>(m, x0, x2);
  add_vv<W>(mp, m, xp);
  sub_vv<W>(mm, m, xp);
  select<W>(m, sa ^ sb, mp, mm);  // signs differ: the product of the differences is negative
  // t = z0 + z2 B^(2h) + mid B^h; the true value fits 2L limbs
  constexpr int T = 2 * L - h;
  u32 lo[T], mx[T];
#pragma unroll
  for (int i = 0; i < 2 * h; i++) t[i] = z0[i];
#pragma unroll
  for (int i = 0; i < 2 * g; i++) t[2 * h + i] = z2[i];
#pragma unroll
  for (int i = 0; i < T; i++) {
    lo[i] = t[h + i];
    mx[i] = i < W ? m[i] : 0u;
  }
  add_vv<T>(t + h, lo, mx);
}

// r = a*b mod q by Barrett reduction (Eq. (barrett), Listing 4 generalised):
//   a' = a*2^d, t = a'*b < qn^2, r1 = t >> (M-2), r2 = (r1*mu) >> (M+5),
//   t - r2*qn in [0, 2qn) (one correction), result = (that mod qn) >> d.
// The subtraction uses only the low L limbs, as in _dmulmod: the difference
// fits in L limbs.  KARA: the two full products (a*b, r1*mu) by one level of
// Karatsuba.
template <int L, bool KARA>
__device__ __forceinline__ void barrett_mul_words(u32* r, const u32* a, const u32* b, const BarrettWordC<L>& c) {
  // a' = a << d (a < q so a' < qn < 2^(32L-4): no overflow past L limbs)
  u32 as[L];
  if (c.d == 0) {
#pragma unroll
    for (int i = 0; i < L; i++) as[i] = a[i];
  } else {
    as[0] = a[0] << c.d;
#pragma unroll
    for (int i = 1; i < L; i++) as[i] = __builtin_amdgcn_alignbit(a[i], a[i - 1], 32 - c.d);
  }
  // t = a' * b, 2L limbs
  u32 t[2 * L];
  if constexpr (KARA) {
    kara_mul<L>(t, as, b);
  } else {
    u64 acc = 0;
    u32 hi = 0;
#pragma unroll
    for (int k = 0; k < 2 * L - 1; k++) {
#pragma unroll
      for (int i = (k < L ? 0 : k - L + 1); i <= (k < L ? k : L - 1); i++) mac_vv(acc, hi, as[i], b[k - i]);
      t[k] = (u32)acc;
      shift_col(acc, hi);
    }
    t[2 * L - 1] = (u32)acc;
  }
  // r1 = t >> (M - 2) = t >> (32(L-1) + 26): limbs L-1 .. 2L-1, bit offset 26
  u32 r1[L];
#pragma unroll
  for (int i = 0; i < L; i++) r1[i] = __builtin_amdgcn_alignbit(t[L + i], t[L - 1 + i], 26);
  // r2 = (r1 * mu) >> (M + 5) = >> (32L + 1): need product limbs L .. 2L-1 exactly
  u32 p[2 * L];
  if constexpr (KARA) {
    u32 muv[L];
    to_vgprs<L>(muv, c.mu);
    kara_mul<L>(p, r1, muv);
  } else {
    u64 acc = 0;
    u32 hi = 0;
#pragma unroll
    for (int k = 0; k < 2 * L - 1; k++) {
#pragma unroll
      for (int i = (k < L ? 0 : k - L + 1); i <= (k < L ? k : L - 1); i++) mac_vs(acc, hi, r1[i], c.mu[k - i]);
      p[k] = (u32)acc;
      shift_col(acc, hi);
    }
    p[2 * L - 1] = (u32)acc;
  }
  u32 r2[L];
#pragma unroll
  for (int i = 0; i < L - 1; i++) r2[i] = __builtin_amdgcn_alignbit(p[L + i + 1], p[L + i], 1);
  r2[L - 1] = p[2 * L - 1] >> 1;
  // low L limbs of r2 * qn
  u32 s[L];
  {
    u64 acc = 0;
    u32 hi = 0;
#pragma unroll
    for (int k = 0; k < L; k++) {
#pragma unroll
      for (int i = 0; i <= k; i++) mac_vs(acc, hi, r2[i], c.qn[k - i]);
      s[k] = (u32)acc;
      shift_col(acc, hi);
    }
  }
  u32 dlt[L], red[L];
  sub_vv<L>(dlt, t, s);               // t - r2*qn mod 2^(32L), true value in [0, 2qn)
  reduce_once<L>(red, dlt, c.qn);
  // undo the scaling: exact, the low d bits are zero
  if (c.d == 0) {
#pragma unroll
    for (int i = 0; i < L; i++) r[i] = red[i];
  } else {
#pragma unroll
    for (int i = 0; i < L - 1; i++) r[i] = __builtin_amdgcn_alignbit(red[i + 1], red[i], c.d);
    r[L - 1] = red[L - 1] >> c.d;
  }
}

}  // namespace moma
