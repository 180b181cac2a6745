// common.hpp - declarations shared by the host runtime and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

namespace moma {

constexpr int kMaxLimbs = 32;
// Digit form of the transform's multiplies: b-bit digits (b = 29, or 28 above
// 28 limbs), D of them, so that 2D products of two digits plus a carry stay
// below 2^64, and b*D >= 32L - 1, so that an operand y below 4q <= 2^(32L-2)
// is at most half of R = 2^(bD), as the fixed-operand product needs (only 20
// limbs need a digit more for that than for covering 4q).
// A full-width modulus (fw: bitlen(q) > 32L - 4) keeps canonical operands
// below q < 2^(32L); its digits cover 32L bits, and b never divides 32L, so
// again y < R / 2.
constexpr int digit_bits(int L) { return L <= 28 ? 29 : 28; }
constexpr int digit_count(int L, bool fw = false) {
  return (32 * L - (fw ? 0 : 1) + digit_bits(L) - 1) / digit_bits(L);
}
// fixed scaling of vmul's first operand (bits): q 2^(W0 - bitlen(q)) has W0 bits
// (32L, full width, or 32L - 4), and scaled once more by this it has bD - 1
constexpr int barrett_off(int L, bool fw = false) {
  return digit_bits(L) * digit_count(L, fw) - 1 - (fw ? 32 * L : 32 * L - 4);
}
// Widest limb counts whose elementwise multiplies stay on 32-bit words (vmul of
// moduli with headroom; axpy and full-width vmul): D digits take 2D^2 + 2D
// products (vmul) or about 3/2 D^2 (axpy), and with 3 to 5 of them that is more
// instructions than 2 to 4 words need, for which these calls, bound by memory,
// have little room.  2^24 elements, digits and words: vmul at 64 bits 70.6 and
// 66.5 us, 96 bits 95.5 and 93.2, 128 bits 125.5 and 124.0 (160 bits 162.9 and
// 161.7, but 2^20 of 256 bits 21.2 and 22.3); axpy at 64 bits 68.6 and 67.9, 96
// bits 96.4 and 94.0, 128 bits 127.0 and 127.2; full-width vmul at 64 bits 71.0
// and 67.0, 96 bits 97.4 and 95.9, 128 bits 126.3 and 127.0.
constexpr int kWordLimbsVmul = 4, kWordLimbs = 3;
// Words of one twiddle table entry: the quotient's digits and the twiddle's, and
// above 4 limbs up to whole 16-byte loads.  At 2 and 4 limbs that would make
// entries of 8 words for 6 and of 12 for 10, and long transforms read the whole
// table: padded and not, 2^24 points 447 and 425 us at 64 bits, 916 and 887 at 128
// (2^20: 37.0 and 38.5, 61.6 and 61.1).  Wider entries waste less, and a last load
// of 8 bytes costs what it saves or more: 2^20 points at 256 bits 112 and 115 us,
// 2^14 at 640 bits 54.4 and 56.7.
constexpr int tw_words(int L, bool fw = false) {
  const int d2 = 2 * digit_count(L, fw);
  return L <= 4 ? d2 : (d2 + 3) / 4 * 4;
}

// widest limb counts that get radix-4 / radix-8 / radix-16 register units
// (radix 4 up to 16 limbs: 4 elements of 16 limbs plus the digit multiply fit
// the 256 VGPRs of a lane at two waves per SIMD)
constexpr int kMaxLimbsRadix4 = 16;
constexpr int kMaxLimbsRadix8 = 5;
constexpr int kMaxLimbsRadix16 = 2;
// the Karatsuba form of the butterfly's multiply (Eq. (mulk)): radix-2 units,
// 2 to 24 limbs (up to 768 bits, the widths its comparison with schoolbook
// covers; its 2D - 1 live column sums cost registers the wider units lack)
constexpr int kMaxLimbsKara = 24;
// full-width moduli: radix-4 units up to 16 limbs as well
constexpr int kMaxLimbsRadix4Fw = 16;

// Constants of one modulus, sized for the largest limb count; the launchers copy
// the first L words of each array into a compile-time sized kernel argument.
struct FieldRaw {
  int L;                   // compute limbs: ceil((bitlen(q) + 4) / 32), or the storage limbs for a full-width q
  int Ls;                  // storage limbs (planes) given by the caller, >= L
  int fw;                  // full width: bitlen(q) > 32 L - 4, no headroom for lazy reduction
  uint32_t q[kMaxLimbs];
  uint32_t qinv;           // -q^{-1} mod 2^32 (Montgomery)
  uint32_t one_m[kMaxLimbs];  // 2^(32L) mod q (1 in Montgomery form)
  // vmul on words (up to kWordLimbsVmul limbs, and its Karatsuba variant); d and
  // qn's top limb, in cinv, are also the lazy butterflies' quotient estimate
  uint32_t qn[kMaxLimbs];  // q * 2^d, bitlen 32L - 4
  uint32_t mu[kMaxLimbs];  // floor(2^(2(32L-4)+3) / qn)
  uint32_t d;              // bits that q lacks to 32L - 4
  uint32_t vd;             // vmul in digits: bits that q lacks to W0 (barrett_off)
  uint32_t vmu[40];        // and its quotient constant, the top digit with the bits above bD
  uint32_t vnqn[40];       // 2^(bD) minus the scaled modulus, in digits
  uint32_t nqd[40];        // 2^(bD) - q in digits
  uint32_t qsw[kMaxLimbs]; // q in signed words: the sum of (int32) qsw[i] 2^(32 i)
  uint32_t cinv;           // floor(2^58 / (qt + 1)), qt the top 32 bits of q 2^d (2^27 <= qt < 2^28)
  uint32_t r2[kMaxLimbs];  // 2^(64L) mod q (full-width vmul on words)
};

enum BlasOp { OP_VADD = 0, OP_VSUB = 1, OP_VMUL = 2, OP_AXPY = 3 };

struct BlasArgs {
  const uint32_t* a;
  const uint32_t* b;
  uint32_t* out;
  uint64_t n;
  uint32_t alpha_m[kMaxLimbs];  // axpy: alpha 2^(32L) mod q (the word form)
  uint32_t alpha_d[40];         // alpha in digits
  uint32_t alpha_q[40];         // and its quotient floor(alpha 2^(bD) / q)
  uint32_t variant;      // vmul: 0 schoolbook products, 1 Karatsuba (L >= 2)
  uint32_t ls;           // storage planes (>= L; the planes above L are written as zero)
};

// One pass of the transform: k radix-2 stages [K, K+k) over tiles of C groups.
struct NttPass {
  uint32_t K, k, logc;
  uint64_t tiles;
};

struct NttPassArgs {
  const uint32_t* in;
  const uint32_t* in2;  // first inverse pass of a cyclic product: multiply by in2 pointwise while loading, else NULL
  uint32_t* out;
  const uint32_t* scale;  // last pass of the inverse: the factor every element takes on store, else NULL (2 D digits:
                          // its quotient's, then its own, as a twiddle's)
  const uint32_t* tw;  // twiddle table: tw_words(L) words per entry, in planes of 16 bytes (ntt_impl.hpp, Twiddle)
  uint64_t n;
  uint32_t logn, K, k, logc;
  uint32_t last;       // last pass: store canonical residues in [0, q)
  uint32_t direct;     // set by the pass launcher: the first round reads straight from `in`
  uint32_t xcd_log;    // set by the pass launcher: log2 of the neighbouring tiles kept on one XCD
};

// Consecutive workgroups go to the 8 XCDs in turn, and every XCD has an L2 of
// its own, while a tile with fewer than 32 columns reads and writes rows of
// less than a 128-byte line: its neighbours use the rest of the line.  So the
// 2^g neighbouring tiles that share their lines take workgroups 8 apart, which
// run on one XCD at about the same time, where there are 8 such groups or more.
// Measured against tile b in workgroup b: 16 columns, 256 bits, 2^16 points
// 31.3 -> 30.0 us and 2^24 2203 -> 2131 us; 4 columns, 384 bits, 2^14 points
// 39.0 -> 36.5 us; a 768-bit cyclic product of 2^16 points 341 -> 323 us.
// With fewer groups (16 tiles of 4 columns, 256 bits, 2^12 points) taking pairs
// of tiles was slower, 19.5 -> 20.5 us.
inline uint32_t xcd_group_log(uint32_t logc, uint64_t tiles) {
  const uint32_t g = logc < 5 ? 5 - logc : 0;
  return (tiles >> 3 >> g) ? g : 0;
}
// the tile of workgroup b; `tiles` is a multiple of 8 2^g or g is 0
__host__ __device__ inline uint32_t xcd_tile(uint32_t b, uint32_t g) {
  const uint32_t lo = b & ((8u << g) - 1);
  return b - lo + ((lo & 7u) << g) + (lo >> 3);
}

// Launch shape of a transform: LDS tile of 2^tile_log elements, 2^col_log
// groups per tile in multi-pass plans, threads per workgroup, stages per
// register unit (radix 2^radix_log), and the butterfly's word-product form
// (kara: one level of Karatsuba, Eq. (mulk); 0: schoolbook).
struct NttSchedule {
  uint32_t tile_log, col_log, threads, radix_log;
  uint32_t kara = 0;
};

// arithmetic of a transform kernel: lazy butterflies with the schoolbook or
// the Karatsuba digit product, or canonical ones for a full-width modulus
enum NttArith { kArithLazy = 0, kArithFull = 1, kArithKara = 2, kArithOffset = 3 };


// per-modulus constants of the digit-form multiplies
struct DigitConsts {
  uint32_t qd[40];   // q in b-bit digits (digit_count(L, fw) of them)
  uint32_t qinvd;    // -q^{-1} mod 2^b
  uint32_t adj[kMaxLimbs];  // 2^(b*D) mod q, converts a table entry to digit Montgomery form
};

// set the thread's error detail and return code
int set_error(int code, const std::string& detail);

uint32_t device_cu_count();
// launchers (return hipError_t as int)
int launch_blas(int op, const FieldRaw& f, const BlasArgs& a, hipStream_t s);
int launch_zero_planes(uint32_t* out, uint64_t n, int from_plane, int to_plane, hipStream_t s);
int launch_ntt_pass(const FieldRaw& f, const DigitConsts& dc, const NttPassArgs& a,
                    uint32_t threads, uint64_t tiles, uint32_t radix_log, uint32_t kara, hipStream_t s);
// batched transforms: one launch runs items (pass record, tile) of many plans
// (fw: full-width moduli, whose kernels and constants are of their own kind)
size_t ntt_consts_bytes(int L, bool fw);
void ntt_batch_prepare(int L, uint32_t radix_log, bool fw, size_t lds);
void ntt_fill_consts(const FieldRaw& f, const DigitConsts& dc, void* dst);
int launch_ntt_batch(int L, uint32_t radix_log, bool mul, bool variant, bool fw, uint32_t threads, size_t lds,
                     uint32_t grid, const NttPassArgs* d_passes, const void* d_consts, const uint2* d_items,
                     uint32_t nitems, hipStream_t s);
// whether a batch pass record runs the variant kernel (direct first round,
// cross-lane last stage); sets the record's `direct` flag
bool ntt_batch_variant(int L, uint32_t radix_log, uint32_t threads, NttPassArgs* a);
// largest workgroup the pass kernel for (L, radix_log) was compiled for
uint32_t ntt_max_threads(int L, uint32_t radix_log);
int launch_twiddle_gen(const FieldRaw& f, const DigitConsts& dc, uint32_t* tw, uint64_t n, uint32_t logn,
                       const uint32_t* d_ladder, hipStream_t s);


}  // namespace moma

// expand CASE(L) for every supported compute limb count
#define MOMA_FOR_EACH_L(CASE)                                                                                     \
  CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8) CASE(9) CASE(10) CASE(11) CASE(12) CASE(13)    \
  CASE(14) CASE(15) CASE(16) CASE(17) CASE(18) CASE(19) CASE(20) CASE(21) CASE(22) CASE(23) CASE(24) CASE(25)    \
  CASE(26) CASE(27) CASE(28) CASE(29) CASE(30) CASE(31) CASE(32)
