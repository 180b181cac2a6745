// ntt_impl.hpp - number theoretic transform kernels (paper Eq. (ntt),
// Section 5.3) and their per-limb-count launchers, as templates.  ntt.hip
// dispatches on the limb count at run time; the instantiations for each limb
// count live in the ntt_inst_*.hip units, so they compile in parallel.
//
// Algorithm: radix-2 Cooley-Tukey butterflies (U + V*W, U - V*W), natural-order
// input.  Stage s (s = 0 .. log2 n - 1) has 2^s blocks; block i pairs elements
// t = n / 2^(s+1) apart and multiplies by W = w_{2m}^{rev_s(i)} with m = 2^s,
// w_{2m} = w^(n/2m).  After the last stage element p holds y[rev(p)].
//
// Data movement (MI355X-first): stages are grouped into passes of k stages that
// run in LDS, so each pass reads and writes every element once in HBM.
//   * Between passes the logical element p is stored at address rev_n(p).  The
//     first pass reads natural order and writes bit-reversed; later passes read
//     and write the same addresses (in place); after the last pass address j
//     holds y[j]: the output comes out in natural order with no extra pass.
//   * A pass over stages [K, K+k) works on groups of 2^k elements that share a
//     level-K block and an offset.  A tile is C groups whose addresses are
//     consecutive (C >= 16 words per limb plane per row), so global loads and
//     stores are coalesced in every pass.
//   * Inside a tile, each thread runs radix-2^r units in registers: 2^r
//     elements spanning r consecutive stages, so LDS is read and written, and
//     the workgroup synchronised, once per r stages instead of once per stage.
//   * Twiddle table: entry m + i' (m = 2^s) holds w_{2m}^{i'} and its quotient
//     floor(w_{2m}^{i'} 2^(bD) / q), D b-bit digits each (level s stores the
//     first m powers of w_{2m}).  With that order the C
//     groups of a tile read C consecutive entries, and the first pass reads a
//     table prefix shared by every tile.
// Butterflies use lazy reduction: values stay in [0, 4q) or [0, 16q)
// (offset_applies) between stages and between passes, and the last pass stores
// canonical residues in [0, q).
#pragma once
#include <string.h>

#include <atomic>

#include "common.hpp"
#include "limb.hpp"

namespace moma {

// Which kernels take the offset form of the lazy butterflies (OFF).  It issues
// fewer additions per butterfly, but its reductions are a serial chain, while a
// wave that has its SIMD almost to itself fits Harvey's independent additions
// between its products.  So: radix-4 units from 6 limbs (2^20 points: 256 bits
// 115.6 -> 113 us, 512 bits 375 -> 315, 160 bits 71.4 -> 72), radix-2 units from
// 20 (2^16 points: 640 bits 66.3 -> 63.9 us, 1024 bits 125 -> 118; but 512 bits 46.0
// -> 51.0, 256 bits 26.4 -> 28.0); the Karatsuba kernels keep Harvey's.
constexpr bool offset_applies(int L, int R) {
  return spare_bits(L) >= 0 && ((R == 2 && L >= 6) || (R == 1 && L >= 20));
}

// constants of the offset form, in the kernels of limb counts that have it
template <int L, bool OFF>
struct OffsetC {};
template <int L>
struct OffsetC<L, true> {
  u32 qsw[L];  // q in signed words
  u32 d, cinv;  // quotient estimate (offset_reduce)
};

// FW: a full-width modulus (no headroom): canonical values, digits over 32L bits
template <int L, bool FW = false>
struct NttC : OffsetC<L, !FW && (offset_applies(L, 1) || offset_applies(L, 2))> {
  u32 q[L];
  u32 q2[L];                        // 2q (unused for a full-width modulus)
  u32 qinv;
  u32 nqd[Digits<L, FW>::D];        // 2^(bD) - q in b-bit digits (twiddle multiply)
  u32 qd[Digits<L, FW>::D];         // q in b-bit digits (pointwise product)
  u32 qinvd;                        // -q^-1 mod 2^b
};

__device__ __forceinline__ u32 rev_bits(u32 x, u32 b) { return b ? (__brev(x) >> (32 - b)) : 0u; }

// One twiddle: its quotient's digits, then its own, tw_words(L, FW) words.  The
// table holds them in 16-byte pieces, piece c of entry e at word 4 (c n + e), and
// where two words are left over, in a last plane of 8-byte ones: the lanes of a
// load read consecutive pieces, whatever the entry's length.
// `first` (the level's first entry plus the unit's, uniform) and the lane's
// offset `off` < 2^25 entries keep the lane's part of the address in 32 bits.
template <int L, bool FW = false>
struct Twiddle {
  static constexpr int D = Digits<L, FW>::D;
  u32 v[tw_words(L, FW)];
  __device__ __forceinline__ const u32* wq() const { return v; }
  __device__ __forceinline__ const u32* w() const { return v + D; }
  __device__ __forceinline__ void load(const u32* __restrict__ tw, u64 n, u64 first, u32 off) {
    // (opaque here, or the bases of a whole round are computed ahead of it and
    // spilled)
    asm volatile("" : "+s"(first));
    constexpr int S = tw_words(L, FW);
#pragma unroll
    for (int i = 0; i < S / 4; i++) {
      const uint4 t = uniform_at<uint4>(tw + 4 * (i * n + first), off << 4);
      v[4 * i] = t.x;
      v[4 * i + 1] = t.y;
      v[4 * i + 2] = t.z;
      v[4 * i + 3] = t.w;
    }
    if constexpr (S % 4) {
      const uint2 t = uniform_at<uint2>(tw + (S - 2) * n + 2 * first, off << 3);
      v[S - 2] = t.x;
      v[S - 1] = t.y;
    }
  }
};

// Tile geometry shared by the load, compute and store phases.
struct TileGeo {
  u32 k, logc, K, rows, C, E;
  u64 n, S, o0, ro, b0;
};

// Twiddle of local stage sg, local block lb of group g: table entry
// 2^(K+sg) + rev_sg(lb) 2^K + (b0 + g when K > 0).  For a unit that starts at
// stage sg0 in block lb, stage sg0 + s and sub-block i < 2^s this is the
// unit's own offset plus a uniform 2^(K+sg0+s) + rev_s(i) 2^(K+sg0).
__device__ __forceinline__ u32 tw_off(const TileGeo& t, u32 sg0, u32 lb, u32 g) {
  const u32 r = (__brev(lb) >> 1) >> (31 - sg0);  // lb < 2^sg0
  return (r << t.K) + (t.K == 0 ? 0u : (u32)t.b0 + g);
}
__device__ __forceinline__ u64 tw_first(const TileGeo& t, u32 sg0, u32 s, u32 i) {
  return (1ull << (t.K + sg0 + s)) + ((u64)rev_bits(i, s) << (t.K + sg0));
}

// A tile in LDS: element idx = row * C + group, its limbs in planes of 16-byte
// quads, then an 8-byte pair and a single word as L leaves them (4 L E bytes in
// all).  An element then takes L / 4 LDS instructions and addresses each way
// instead of L, and lanes with consecutive groups still access consecutive
// banks.  (In limb planes of single words a stage of a 256-bit radix-2 unit
// spent a third of its time on LDS: about 500 cycles until its elements were in,
// against 1340 for the butterfly; 2^12 points took 20.8 us, with quads 18.6.)
template <int L>
__device__ __forceinline__ void lds_get(u32* x, const u32* lds, u32 E, u32 idx) {
#pragma unroll
  for (int q = 0; q < L / 4; q++) {
    const uint4 v = *reinterpret_cast<const uint4*>(lds + 4 * (q * E + idx));
    x[4 * q] = v.x;
    x[4 * q + 1] = v.y;
    x[4 * q + 2] = v.z;
    x[4 * q + 3] = v.w;
  }
  if constexpr (L % 4 >= 2) {
    const uint2 v = *reinterpret_cast<const uint2*>(lds + 4 * (L / 4) * E + 2 * idx);
    x[L / 4 * 4] = v.x;
    x[L / 4 * 4 + 1] = v.y;
  }
  if constexpr (L % 2) x[L - 1] = lds[(L - 1) * E + idx];
}
template <int L>
__device__ __forceinline__ void lds_put(u32* lds, u32 E, u32 idx, const u32* x) {
#pragma unroll
  for (int q = 0; q < L / 4; q++)
    *reinterpret_cast<uint4*>(lds + 4 * (q * E + idx)) = make_uint4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
  if constexpr (L % 4 >= 2)
    *reinterpret_cast<uint2*>(lds + 4 * (L / 4) * E + 2 * idx) = make_uint2(x[L / 4 * 4], x[L / 4 * 4 + 1]);
  if constexpr (L % 2) lds[(L - 1) * E + idx] = x[L - 1];
}

// Element e of a radix-2^R unit in HBM: the lane's part of its word offset
// (element 0: row p0 of group g) and the uniform rest.  Row u lies at u S + o0 + g
// in the first pass's input and at (ro, rev_k(u), b0 + g) after it; the unit's
// rows are e 2^(k-sg0-R) apart, and e's bits reverse to rev_R(e) 2^sg0.
__device__ __forceinline__ u32 row_off(const TileGeo& t, u32 u, u32 g, bool natural) {
  return natural ? u * (u32)t.S + (u32)t.o0 + g
                 : (u32)(t.ro << (t.K + t.k)) + ((__brev(u) >> (32 - t.k)) << t.K) + (u32)t.b0 + g;
}
// one element's limbs from / to plane 0's word `first` (uniform) plus the lane's
template <int L>
__device__ __forceinline__ void hbm_get(u32* x, const u32* first, u64 n, u32 lane_bytes) {
#pragma unroll
  for (int j = 0; j < L; j++, first += n) x[j] = uniform_at<u32>(first, lane_bytes);
}
template <int L>
__device__ __forceinline__ void hbm_put(const u32* x, u32* first, u64 n, u32 lane_bytes) {
#pragma unroll
  for (int j = 0; j < L; j++, first += n) uniform_put<u32>(first, lane_bytes, x[j]);
}

// One round of R stages [sg0, sg0+R) on every radix-2^R unit of the tile.
// FIRST: the transform's first round (first pass, sg0 = 0).  There every unit
// lies in block 0, so a pair whose local block index is 0 has twiddle
// w^0 = 1 (table entry 2^s) and skips the multiply: all pairs of stage 0, half
// of stage 1, a quarter of stage 2.
// STORE: the pass's last round in a later pass (K > 0) with at least 16
// columns (and at most 10 limbs): each unit writes its finished elements straight to their HBM
// addresses (the rows of one column are consecutive across lanes, so every
// store instruction covers 64-byte runs) instead of back to LDS, so the pass
// has no separate store phase and the stores drain while other units compute.
// What the last pass does to its N elements before it stores them.  The
// inverse's factor is read here, by uniform loads, and not held in registers
// from the kernel's start.
template <int L, int AR, int N>
__device__ __forceinline__ void finish_elems(u32 (*x)[L], const NttPassArgs& a, const NttC<L, AR == kArithFull>& c) {
  constexpr bool FW = AR == kArithFull;
  if (!a.last) return;
  if (a.scale) {
    constexpr int D = Digits<L, FW>::D;
    typedef const __attribute__((address_space(4))) u32* ConstWords;
    u64 p = (u64)a.scale;
    asm volatile("" : "+s"(p));
    u32 sq[D], sd[D];
#pragma unroll
    for (int i = 0; i < D; i++) {
      sq[i] = ((ConstWords)p)[i];
      sd[i] = ((ConstWords)p)[D + i];
    }
#pragma unroll
    for (int e = 0; e < N; e++) {
      u32 y[L], top;
      quot_mul<L, FW>(y, x[e], sd, sq, c.nqd, &top);  // y in [0, 2q)
      if constexpr (FW)
        reduce_top<L>(x[e], y, top, c.q);
      else
        reduce_once<L>(x[e], y, c.q);
    }
  } else if constexpr (!FW) {  // (full-width values are canonical throughout)
#pragma unroll
    for (int e = 0; e < N; e++) {
      u32 y[L];
      if constexpr (AR == kArithOffset) {
        offset_reduce<L>(x[e], 0, c.qsw, c.d, c.cinv);  // [0, 16q) -> [0, 2q)
#pragma unroll
        for (int j = 0; j < L; j++) y[j] = x[e][j];
      } else {
        reduce_once<L>(y, x[e], c.q2);  // [0, 4q) -> [0, 2q)
      }
      reduce_once<L>(x[e], y, c.q);  // -> [0, q)
    }
  }
}

// LOADG: the pass's first round reads its elements straight from the input in
// HBM (the addresses the load phase would have filled the LDS rows from)
// instead of from LDS, so the pass has no separate load phase.
// Wide limbs, radix-2 units: registers, not instructions, bound these kernels
// (one or two waves per SIMD), so a unit reads the bottom element, forms the
// product w*y, and only then reads the top element and copies 2q (or q) into
// VGPRs for the additions; neither is live across the multiply.
constexpr int kLateLoadLimbs = 11;

// multiple of q the reduced x of a round get (offset_reduce): the most stages
// fit below and above it
constexpr u32 kOffset = 7;

template <int L, bool FIRST, bool STORE, int AR>
__device__ __forceinline__ void round_late(u32* lds, const TileGeo& t, u32 sg0, const NttPassArgs& a,
                                           const NttC<L, AR == kArithFull>& c, bool red) {
  constexpr bool FW = AR == kArithFull, OFF = AR == kArithOffset;
  const u32* __restrict__ tw = a.tw;
  const u32 k = t.k;
  const u32 B = 1u << (k - sg0);  // block size (rows) at stage sg0; the pair is B/2 rows apart
  const u32 units = t.E >> 1;
  for (u32 b = threadIdx.x; b < units; b += blockDim.x) {
    u32 g = b & (t.C - 1), v = b >> t.logc;
    u32 lb = v >> (k - sg0 - 1);
    u32 p0 = lb * B + (v & ((B >> 1) - 1));
    const u32 r0 = p0, r1 = p0 + (B >> 1);
    u32 x[L], y[L];
    if (FIRST && lb == 0) {
      // twiddle 1: no multiply
      lds_get<L>(x, lds, t.E, r0 * t.C + g);
      lds_get<L>(y, lds, t.E, r1 * t.C + g);
      u32 qv[L];
      to_vgprs<L>(qv, FW || OFF ? c.q : c.q2);
      if constexpr (FW)
        ct_butterfly_one_fw<L>(x, y, qv);
      else if constexpr (OFF)
        ct_one_tail<L>(x, y, qv);
      else
        ct_butterfly_one<L>(x, y, qv);
    } else {
      Twiddle<L, FW> w;
      u32 p[L], top = 0;
      w.load(tw, t.n, tw_first(t, sg0, 0, 0), tw_off(t, sg0, lb, g));
      lds_get<L>(y, lds, t.E, r1 * t.C + g);
      if constexpr (AR == kArithKara)
        quot_mul_kara<L>(p, y, w.w(), w.wq(), c.nqd);
      else
        quot_mul<L, FW>(p, y, w.w(), w.wq(), c.nqd, &top);
      lds_get<L>(x, lds, t.E, r0 * t.C + g);
      u32 qv[L];
      if constexpr (FIRST || !OFF) to_vgprs<L>(qv, FW ? c.q : c.q2);
      if constexpr (FW) {
        ct_fw_tail<L>(x, y, p, top, qv);
      } else {
        if constexpr (OFF && !FIRST) {
          if (red) offset_reduce<L>(x, kOffset, c.qsw, c.d, c.cinv);
        }
        ct_tail<L, OFF, FIRST>(x, y, p, qv);
      }
    }
    if constexpr (STORE) {
      const u32 dst = row_off(t, r0, g, false) << 2;
      finish_elems<L, AR, 1>(&x, a, c);
      finish_elems<L, AR, 1>(&y, a, c);
      hbm_put<L>(x, a.out, t.n, dst);
      hbm_put<L>(y, a.out + (1ull << (t.K + sg0)), t.n, dst);
    } else {
      lds_put<L>(lds, t.E, r0 * t.C + g, x);
      lds_put<L>(lds, t.E, r1 * t.C + g, y);
    }
  }
}

// AR: the kernel's arithmetic (NttArith)
// red: the x of the round's first stage are reduced before it (OFF)
template <int L, int R, bool FIRST, bool STORE, bool LOADG = false, int AR = kArithLazy>
__device__ __forceinline__ void ntt_round(u32* lds, const TileGeo& t, u32 sg0, const NttPassArgs& a,
                                          const NttC<L, AR == kArithFull>& c, bool red) {
  constexpr bool FW = AR == kArithFull, OFF = AR == kArithOffset;
  const u32* __restrict__ tw = a.tw;
  const u32 k = t.k;
  const u32 B = 1u << (k - sg0);        // block size (rows) at stage sg0
  const u32 sub = B >> R;                // row spacing of a unit's elements
  const u32 units = (t.E >> R);
  if constexpr (R == 1 && !LOADG && L >= kLateLoadLimbs) {
    round_late<L, FIRST, STORE, AR>(lds, t, sg0, a, c, red);
    return;
  }
  u32 q2v[L], q1v[L];  // 2q (lazy butterflies), or q (full width); q in the first round
  if constexpr (FIRST || !OFF) to_vgprs<L>(q2v, FW ? c.q : c.q2);
  if constexpr (FIRST && OFF) to_vgprs<L>(q1v, c.q);
  for (u32 b = threadIdx.x; b < units; b += blockDim.x) {
    u32 g = b & (t.C - 1), v = b >> t.logc;
    u32 lb = v >> (k - sg0 - R);
    u32 p0 = lb * B + (v & (sub - 1));
    u32 x[1 << R][L];
    const u32 idx0 = p0 * t.C + g, step = sub << t.logc;  // the unit's elements in LDS
    // The first stage's twiddle (one per unit) is loaded before the elements
    // where it is what a wave waits for longest: in radix-2 units, which run
    // where few waves share a SIMD (256 bits, 2^16 points 27.0 -> 26.1 us; 128
    // bits, 2^12 12.5 -> 11.5), and with LOADG, where the elements come pair by
    // pair of the first stage, (e, e + 2^(R-1)): a wave's loads complete in
    // issue order, so the first pair's butterfly can start while the later pairs
    // are still in flight; and before the branch that may reduce x (OFF).  (With radix-4 units from LDS: 2^20 points 116 -> 117 us.
    // Loaded a round ahead, before the barrier, it was 10% slower: the value
    // crosses the loop over units, and the compiler waits for it there.)
    constexpr bool EARLY = R == 1 || LOADG || OFF;
    const u32 toff = tw_off(t, sg0, lb, g);
    Twiddle<L, FW> w;
    if constexpr (EARLY && !FIRST) w.load(tw, t.n, tw_first(t, sg0, 0, 0), toff);
    if constexpr (LOADG) {
      const u32 src = row_off(t, p0, g, t.K == 0) << 2;
#pragma unroll
      for (int pp = 0; pp < (1 << R); pp++) {
        const int e = (pp >> 1) + (pp & 1) * (1 << (R - 1));
        const u64 first = t.K == 0 ? (u64)(e * sub) * t.S : (u64)rev_bits(e, R) << (t.K + sg0);
        hbm_get<L>(x[e], a.in + first, t.n, src);
      }
    } else {
#pragma unroll
      for (int e = 0; e < (1 << R); e++) lds_get<L>(x[e], lds, t.E, idx0 + e * step);
    }
    if constexpr (OFF && !FIRST) {
      if (red)
#pragma unroll
        for (int e = 0; e < (1 << (R - 1)); e++) offset_reduce<L>(x[e], kOffset, c.qsw, c.d, c.cinv);
    }
#pragma unroll
    for (int s = 0; s < R; s++) {
      const int half = 1 << (R - 1 - s);
      // block i of the 2^s the unit has at this stage: one twiddle, `half` pairs (e, e + half)
#pragma unroll
      for (int i = 0; i < (1 << s); i++) {
        // (OFF: sums without a product double the bound, so two stages of them at most)
        const bool one = FIRST && i == 0 && (!OFF || s < 2);
        if (!one && !(EARLY && s == 0)) w.load(tw, t.n, tw_first(t, sg0, s, i), toff);
#pragma unroll
        for (int e = 2 * half * i; e < 2 * half * i + half; e++) {
          if (one) {
            if constexpr (FW)
              ct_butterfly_one_fw<L>(x[e], x[e + half], q2v);
            else if constexpr (OFF)
              ct_one_tail<L>(x[e], x[e + half], s == 0 ? q1v : q2v);
            else
              ct_butterfly_one<L>(x[e], x[e + half], q2v);
          } else if constexpr (FW) {
            ct_butterfly_fw<L>(x[e], x[e + half], w.w(), w.wq(), c.nqd, q2v);
          } else {
            ct_butterfly_mul<L, AR == kArithKara, OFF, FIRST>(x[e], x[e + half], w.w(), w.wq(), c.nqd, q2v);
          }
        }
      }
    }
    if constexpr (STORE) {
      const u32 dst = row_off(t, p0, g, false) << 2;
      finish_elems<L, AR, (1 << R)>(x, a, c);
#pragma unroll
      for (int e = 0; e < (1 << R); e++) hbm_put<L>(x[e], a.out + ((u64)rev_bits(e, R) << (t.K + sg0)), t.n, dst);
    } else {
#pragma unroll
      for (int e = 0; e < (1 << R); e++) lds_put<L>(lds, t.E, idx0 + e * step, x[e]);
    }
  }
}

// Exchange of a final-stage round: a <-> the partner lane's b, where the
// partner of lane l is l ^ 32 (C = 32 groups per tile) or l ^ 16 (C = 16).
// v_permlane32_swap / v_permlane16_swap swap the upper (odd) 32- (16-) lane
// rows of the first operand with the lower (even) rows of the second.
__device__ __forceinline__ void swap_with_partner(u32& a, u32& b, bool c32) {
  if (c32) {
    auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  } else {
    auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  }
}

// The pass's last R + 1 stages [sg0, k) without an LDS round trip before the
// last one.  A radix-2^R round on stages sg0 .. k - 2 leaves element e of unit
// v at row p0 + 2e of its block (p0 = block start + (v & 1)), so the partners
// of the last stage, rows 2m and 2m + 1, sit in units v and v ^ 1: the same
// group g, in lanes C apart of one wavefront (the units of a round are laid
// out g-fastest).  Swapping the upper half of one unit's elements with the
// lower half of its partner's puts both rows of a pair in one lane: lane half
// h = v & 1 then holds pair j (elements j and j + 2^(R-1)) = rows
// 2j + 2^R h and 2j + 2^R h + 1 of the block, whose last-stage block index is
// 2^R lb + 2^(R-1) h + j.  Requires C in {16, 32}, whole wavefronts of units,
// and a round that is not the transform's first.
template <int L, int R, bool STORE, int AR>
__device__ __forceinline__ void ntt_round_last(u32* lds, const TileGeo& t, u32 sg0, const NttPassArgs& a,
                                               const NttC<L>& c, bool red) {
  constexpr bool OFF = AR == kArithOffset;
  const u32* __restrict__ tw = a.tw;
  const u32 k = t.k;
  const u32 B = 1u << (k - sg0);        // block size (rows) at stage sg0: 2^(R+1)
  const u32 units = (t.E >> R);
  const bool c32 = t.logc == 5;
  constexpr int H = 1 << (R - 1);
  u32 q2v[L];
  if constexpr (!OFF) to_vgprs<L>(q2v, c.q2);
  for (u32 b = threadIdx.x; b < units; b += blockDim.x) {
    u32 g = b & (t.C - 1), v = b >> t.logc;
    u32 lb = v >> 1;
    u32 p0 = lb * B + (v & 1u);
    const u32 toff = tw_off(t, sg0, lb, g);
    u32 x[1 << R][L];
    const u32 step = 2u << t.logc;
    Twiddle<L> w;
    if constexpr (OFF) w.load(tw, t.n, tw_first(t, sg0, 0, 0), toff);
#pragma unroll
    for (int e = 0; e < (1 << R); e++) lds_get<L>(x[e], lds, t.E, p0 * t.C + g + e * step);
    if constexpr (OFF) {
      if (red)
#pragma unroll
        for (int e = 0; e < H; e++) offset_reduce<L>(x[e], kOffset, c.qsw, c.d, c.cinv);
    }
#pragma unroll
    for (int s = 0; s < R; s++) {
      const int half = 1 << (R - 1 - s);
#pragma unroll
      for (int i = 0; i < (1 << s); i++) {
        if (!OFF || s > 0) w.load(tw, t.n, tw_first(t, sg0, s, i), toff);
#pragma unroll
        for (int e = 2 * half * i; e < 2 * half * i + half; e++)
          ct_butterfly_mul<L, false, OFF, false>(x[e], x[e + half], w.w(), w.wq(), c.nqd, q2v);
      }
    }
#pragma unroll
    for (int e = 0; e < H; e++)
#pragma unroll
      for (int j = 0; j < L; j++) swap_with_partner(x[e][j], x[e + H][j], c32);
    const u32 h = v & 1u;
#pragma unroll
    for (int jp = 0; jp < H; jp++) {
      // last-stage block 2^R lb + 2^(R-1) h + jp: h reverses to the lowest bit
      w.load(tw, t.n, tw_first(t, sg0, R, (u32)jp), toff + (h << (t.K + sg0)));
      ct_butterfly_mul<L, false, OFF, false>(x[jp], x[jp + H], w.w(), w.wq(), c.nqd, q2v);
    }
    const u32 r0 = lb * B + (h << R);
    if constexpr (STORE) {
      // row r0 + 2 jp + o: its low R bits reverse to the top of the k
      const u32 dst = row_off(t, r0, g, false) << 2;
      finish_elems<L, AR, (1 << R)>(x, a, c);
#pragma unroll
      for (int jp = 0; jp < H; jp++)
#pragma unroll
        for (int o = 0; o < 2; o++)
          hbm_put<L>(x[jp + o * H], a.out + ((u64)rev_bits(2 * jp + o, R) << (t.K + sg0 + 1)), t.n, dst);
    } else {
#pragma unroll
      for (int jp = 0; jp < H; jp++)
#pragma unroll
        for (int o = 0; o < 2; o++) lds_put<L>(lds, t.E, (r0 + 2 * jp + o) * t.C + g, x[jp + o * H]);
    }
  }
}

// One tile of one pass: stages [K, K+k) on C = 2^logc groups of 2^k elements.
// the fused store keeps a unit's finished elements live while it stores them
// (up to 10 limbs, 9 for a full-width modulus: at 11 to 16 limbs it measured
// no faster than the store from LDS)
template <int L, bool FW = false>
constexpr bool kFuseStore = L <= (FW ? 9 : 10);

template <int L, int R, int AR = kArithLazy>
__device__ __forceinline__ void round_at(u32* lds, const TileGeo& t, u32 sg0, const NttPassArgs& a,
                                         const NttC<L, AR == kArithFull>& c, bool store, bool red) {
  if constexpr (kFuseStore<L, AR == kArithFull>) {
    if (store) {
      ntt_round<L, R, false, true, false, AR>(lds, t, sg0, a, c, red);
      return;
    }
  }
  if (t.K == 0 && sg0 == 0)
    ntt_round<L, R, true, false, false, AR>(lds, t, sg0, a, c, false);
  else
    ntt_round<L, R, false, false, false, AR>(lds, t, sg0, a, c, red);
}

// Fused pointwise product of a cyclic product's first inverse pass:
// r = x * y * 2^(-bD) mod q in [0, 2q) for x, y < q (the digit-form multiply
// with y converted to digits; the last pass's scale constant carries 2^(bD)).
template <int L, int AR>
__device__ __forceinline__ void pointwise_digits(u32* r, const u32* x, const u32* y,
                                                 const NttC<L, AR == kArithFull>& c) {
  constexpr bool FW = AR == kArithFull;
  u32 yd[Digits<L, FW>::D];
  to_digits<L, FW>(yd, y);
  if constexpr (FW) {
    // canonical result for a full-width modulus
    u32 t[L], top;
    mont_mul_digits<L, true>(t, x, yd, c.qd, c.qinvd, &top);
    reduce_top<L>(r, t, top, c.q);
  } else {
    u32 t[L];
    mont_mul_digits<L>(t, x, yd, c.qd, c.qinvd);
    if constexpr (AR == kArithOffset) {
      reduce_once<L>(r, t, c.q);  // the first round's bounds start from [0, q)
    } else {
#pragma unroll
      for (int j = 0; j < L; j++) r[j] = t[j];
    }
  }
}

// MUL: the pass also multiplies its input by a.in2 element by element as it
// loads (first pass of the inverse transform inside a cyclic product).
// LASTX: the pass ends with ntt_round_last (radix-4 units only; the launcher
// sets it when fused_last_applies holds, so other launches run unchanged code).
template <int L, int R, bool MUL, bool LASTX = false, int AR = kArithLazy>
__device__ __forceinline__ void pass_tile(u32* lds, const NttPassArgs& a, const NttC<L, AR == kArithFull>& c,
                                          u64 tile) {
  constexpr bool FW = AR == kArithFull;
  constexpr int AX = AR == kArithLazy && offset_applies(L, R) ? kArithOffset : AR;
  static_assert(AR == kArithLazy || !LASTX, "only the lazy schoolbook kernels have the cross-lane variant");
  TileGeo t;
  t.k = a.k;
  t.logc = a.logc;
  t.K = a.K;
  t.C = 1u << t.logc;
  t.rows = 1u << t.k;
  t.E = t.rows << t.logc;
  t.n = a.n;
  t.S = t.n >> (t.K + t.k);
  t.o0 = t.ro = t.b0 = 0;
  if (t.K == 0) {
    t.o0 = tile << t.logc;
  } else {
    u64 per = (1ull << t.K) >> t.logc;
    t.ro = tile / per;
    t.b0 = (tile % per) << t.logc;
  }
  const u32 tid = threadIdx.x, T = blockDim.x;
  const u64 n = t.n;
  // LASTX passes without a fused product read their first round straight from HBM
  const bool direct = LASTX && !MUL && a.direct != 0;

  // ---- load (natural order in the first pass, bit-reversed storage after).
  // Up to 8 limbs each lane moves 4 consecutive words per limb: 4 groups of one
  // row when the tile has C >= 4 groups, else 4 consecutive rows of a one-pass
  // transform; wider limbs (4 L live words) take one element per lane.
  // Radix-2 units have up to half as many threads as elements; where 4 elements
  // per lane would leave threads idle, they take one each as well (256 bits:
  // 2^10 points 15.2 -> 14.5 us, 2^12 18.4 -> 17.6).
  const bool busy = R > 1 || (t.E >> 2) >= T;
  const bool vec_g = t.C >= 4 && busy, vec_u = t.C == 1 && t.S == 1 && t.rows >= 4 && busy;
  if (direct) {
    // the first round loads its own elements
  } else if (L <= 8 && (vec_g || vec_u)) {
    for (u32 e4 = tid; e4 < (t.E >> 2); e4 += T) {
      const u32 e = e4 << 2, g = e & (t.C - 1), v = e >> t.logc;
      const u32 u = t.K == 0 ? v : rev_bits(v, t.k);
      const u64 src = t.K == 0 ? (u64)u * t.S + t.o0 + g : (t.ro << (t.K + t.k)) + ((u64)v << t.K) + t.b0 + g;
      u32 x[4][L];
#pragma unroll
      for (int j = 0; j < L; j++) {
        const uint4 w = *reinterpret_cast<const uint4*>(a.in + (u64)j * n + src);
        x[0][j] = w.x; x[1][j] = w.y; x[2][j] = w.z; x[3][j] = w.w;
      }
      if constexpr (MUL) {
        u32 y[4][L], r[4][L];
#pragma unroll
        for (int j = 0; j < L; j++) {
          const uint4 z = *reinterpret_cast<const uint4*>(a.in2 + (u64)j * n + src);
          y[0][j] = z.x; y[1][j] = z.y; y[2][j] = z.z; y[3][j] = z.w;
        }
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) pointwise_digits<L, AX>(r[q4], x[q4], y[q4], c);
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) lds_put<L>(lds, t.E, u * t.C + g + q4, r[q4]);
      } else {
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) lds_put<L>(lds, t.E, u * t.C + g + q4, x[q4]);
      }
    }
  } else {
    for (u32 e = tid; e < t.E; e += T) {
      const u32 g = e & (t.C - 1), v = e >> t.logc;
      const u32 u = t.K == 0 ? v : rev_bits(v, t.k);
      const u64 src = t.K == 0 ? (u64)u * t.S + t.o0 + g : (t.ro << (t.K + t.k)) + ((u64)v << t.K) + t.b0 + g;
      u32 x[L];
#pragma unroll
      for (int j = 0; j < L; j++) x[j] = a.in[(u64)j * n + src];
      if constexpr (MUL) {
        u32 y[L], r[L];
#pragma unroll
        for (int j = 0; j < L; j++) y[j] = a.in2[(u64)j * n + src];
        pointwise_digits<L, AX>(r, x, y, c);
        lds_put<L>(lds, t.E, u * t.C + g, r);
      } else {
        lds_put<L>(lds, t.E, u * t.C + g, x);
      }
    }
  }
  if (!direct) __syncthreads();

  // ---- stages, R at a time in registers
  // later passes with 16+ columns store from the last round's registers
  const bool fuse = kFuseStore<L, FW> && t.K > 0 && t.C >= 16;
  // bounds of the values in 64ths of q (OFF): a pass starts from [0, 16q)
  // (the first from [0, q), and its first round of r stages ends below 2r q)
  u32 lo = 0, hi = 16 * 64;
  auto advance = [&](u32 stages, bool first) {
    if (AX != kArithOffset) return false;
    if (first) {
      hi = 2 * 64 * stages;
      return false;
    }
    const u32 move = stages * growth_64th<L>;
    const bool red = lo < move || hi + move > 16 * 64;
    if (red) {
      lo = kOffset * 64;
      hi = kOffset * 64 + 64 + 1;
    }
    lo -= move;
    hi += move;
    return red;
  };
  u32 sg = 0;
  while (sg < t.k) {
    u32 rem = t.k - sg;
    if constexpr (LASTX && !MUL) {
      if (direct && sg == 0) {
        const bool red = advance(R, t.K == 0);
        if (t.K == 0)
          ntt_round<L, R, true, false, true, AX>(lds, t, 0, a, c, false);
        else
          ntt_round<L, R, false, false, true, AX>(lds, t, 0, a, c, red);
        sg = R;
        __syncthreads();
        continue;
      }
    }
    if constexpr ((R == 2 || R == 3) && LASTX) {
      // the last R + 1 stages with a cross-lane exchange before the last one
      if (rem == (u32)R + 1 && (t.logc == 4 || t.logc == 5) && ((t.E >> R) & 63u) == 0 &&
          (t.E >> R) >= blockDim.x && !(t.K == 0 && sg == 0)) {
        const bool red = advance(R + 1, false);
        if constexpr (kFuseStore<L>) {
          if (fuse) {
            ntt_round_last<L, R, true, AX>(lds, t, sg, a, c, red);
            return;
          }
        }
        ntt_round_last<L, R, false, AX>(lds, t, sg, a, c, red);
        __syncthreads();
        break;
      }
    }
    const u32 rr = rem < (u32)R ? rem : (u32)R;
    const bool store = fuse && sg + rr == t.k;
    const bool red = advance(rr, t.K == 0 && sg == 0);
    if (rr == 4) {
      round_at<L, (R >= 4 ? 4 : 1), AX>(lds, t, sg, a, c, store, red);
    } else if (rr == 3) {
      round_at<L, (R >= 3 ? 3 : 1), AX>(lds, t, sg, a, c, store, red);
    } else if (rr == 2) {
      round_at<L, (R >= 2 ? 2 : 1), AX>(lds, t, sg, a, c, store, red);
    } else {
      round_at<L, 1, AX>(lds, t, sg, a, c, store, red);
    }
    sg += rr;
    if (!store) __syncthreads();
  }
  if (fuse) return;

  // ---- store (canonical residues on the last pass), 4 words per lane per limb
  const u32 logn = a.logn;
  // 4 elements of L limbs (and the scale multiply) stay in registers
  // (up to 10 limbs: at 11 to 16 limbs the 4L live words cost occupancy, and
  // 2^16-point transforms measured 3 to 10% slower)
  constexpr bool kVecStore = L <= (FW ? 9 : 10);
  if (kVecStore && t.K > 0 && vec_g) {
    // same addresses as the load: 4 consecutive groups of one row
    for (u32 e4 = tid; e4 < (t.E >> 2); e4 += T) {
      u32 e = e4 << 2;
      u32 g = e & (t.C - 1), v = e >> t.logc;
      u32 u = rev_bits(v, t.k);
      u64 dst = (t.ro << (t.K + t.k)) + ((u64)v << t.K) + t.b0 + g;
      u32 x[4][L];
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) lds_get<L>(x[q4], lds, t.E, u * t.C + g + q4);
      finish_elems<L, AX, 4>(x, a, c);
#pragma unroll
      for (int j = 0; j < L; j++)
        *reinterpret_cast<uint4*>(a.out + (u64)j * n + dst) = make_uint4(x[0][j], x[1][j], x[2][j], x[3][j]);
    }
  } else if (kVecStore && t.K == 0 && t.rows >= 4 && busy) {
    // 4 consecutive output addresses inside one group's run of 2^k
    for (u32 e4 = tid; e4 < (t.E >> 2); e4 += T) {
      u32 e = e4 << 2;
      u32 g = e >> t.k, v = e & (t.rows - 1);
      u64 dst = ((u64)rev_bits((u32)(t.o0 + g), logn - t.k) << t.k) + v;
      u32 x[4][L];
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) lds_get<L>(x[q4], lds, t.E, rev_bits(v + q4, t.k) * t.C + g);
      finish_elems<L, AX, 4>(x, a, c);
#pragma unroll
      for (int j = 0; j < L; j++)
        *reinterpret_cast<uint4*>(a.out + (u64)j * n + dst) = make_uint4(x[0][j], x[1][j], x[2][j], x[3][j]);
    }
  } else {
    for (u32 e = tid; e < t.E; e += T) {
      u32 g, v, u;
      u64 dst;
      if (t.K == 0) {
        g = e >> t.k;
        v = e & (t.rows - 1);
        u = rev_bits(v, t.k);
        dst = ((u64)rev_bits((u32)(t.o0 + g), logn - t.k) << t.k) + v;
      } else {
        g = e & (t.C - 1);
        v = e >> t.logc;
        u = rev_bits(v, t.k);
        dst = (t.ro << (t.K + t.k)) + ((u64)v << t.K) + t.b0 + g;
      }
      u32 x[L];
      lds_get<L>(x, lds, t.E, u * t.C + g);
      finish_elems<L, AX, 1>(&x, a, c);
#pragma unroll
      for (int j = 0; j < L; j++) a.out[(u64)j * n + dst] = x[j];
    }
  }
}

// Workgroup size cap per instantiation: a radix-2^R unit keeps 2^R elements of
// L limbs live, so wider units get fewer threads and more VGPRs per lane.
template <int L, int R>
struct PassTraits {
  static constexpr int live = L << R;
  static constexpr int max_threads = live <= 16 ? 1024 : (live <= 32 ? 512 : 256);
  // radix-4 units of 7 or 8 limbs need just over the 128 registers that four
  // waves per SIMD leave a lane; full-width radix-2 units of 32 limbs just over
  // the 256 of two (2^16 points 199 us with one wave, 139 with two)
  static constexpr int min_waves = R == 2 && live > 24 && live <= 32 ? 4 : (R == 1 && L == 32 ? 2 : 1);
};

// One pass of one transform: one tile per workgroup.
template <int L, int R, bool MUL, bool LASTX, int AR = kArithLazy>
__global__ __launch_bounds__((PassTraits<L, R>::max_threads), (PassTraits<L, R>::min_waves)) void ntt_pass_kernel(NttPassArgs a,
                                                                                 NttC<L, AR == kArithFull> c) {
  extern __shared__ __align__(16) u32 lds[];
  pass_tile<L, R, MUL, LASTX, AR>(lds, a, c, a.xcd_log ? xcd_tile(blockIdx.x, a.xcd_log) : blockIdx.x);
}

// Whether a pass with radix-4 units ends with ntt_round_last: its stage count
// is odd (rounds 2, 2, ..., then 3), the tile has 16 or 32 groups, the units
// fill whole wavefronts and every thread has one, and the fused round is not
// the transform's first round.  Measured against the separate radix-2 round:
// transforms 1 to 4% faster at 2^20 and 2^21 points from 64 to 256 bits; where
// a thread would have no radix-4 unit the separate round, which keeps twice as
// many threads busy, is faster.
inline bool fused_last_applies(const NttPassArgs& a, uint32_t threads, uint32_t radix_log) {
  const uint32_t r = radix_log;
  if (a.k < r + 1 || (a.k - r - 1) % r != 0 || (a.logc != 4 && a.logc != 5)) return false;
  const uint64_t units = (1ull << (a.k + a.logc)) >> r;
  return units % 64 == 0 && units >= threads && !(a.K == 0 && a.k == r + 1);
}

// One phase of a batch: items[i] = (pass record, tile); every pass record names
// its own transform (buffers, size, stages, twiddles) and its modulus constants.
// Workgroup i runs item i; items are sorted by decreasing cost, so the
// dispatcher hands out the largest tiles first.
template <int L, int R, bool MUL, bool LASTX, bool FW = false>
__global__ __launch_bounds__((PassTraits<L, R>::max_threads), (PassTraits<L, R>::min_waves)) void ntt_batch_kernel(
    const NttPassArgs* __restrict__ passes, const NttC<L, FW>* __restrict__ consts, const uint2* __restrict__ items,
    u32 nitems) {
  extern __shared__ __align__(16) u32 lds[];
  const u32 i = blockIdx.x;
  if (i >= nitems) return;
  const uint2 it = items[i];
  const NttPassArgs* rec = passes + it.x;
  NttPassArgs a = *rec;
  a.in = load_global_ptr(&rec->in);
  a.in2 = load_global_ptr(&rec->in2);
  a.out = load_global_ptr(&rec->out);
  a.tw = load_global_ptr(&rec->tw);
  const NttC<L, FW> c = consts[it.x];
  pass_tile<L, R, MUL, LASTX, FW ? kArithFull : kArithLazy>(lds, a, c, it.y);
}

// Twiddle table: entry e = 2^s + i' holds w^(i' * 2^(logn-s-1)) mod q and its quotient.
// ladder[b] = w^(2^b) * 2^(32L) mod q; the product of the ladder entries for the
// set bits of the exponent stays in Montgomery form.
// FW (full-width modulus): the products keep the carry out of the top limb.
template <int L, bool FW = false>
__global__ __launch_bounds__(256) void twiddle_kernel(u32* __restrict__ tw, u64 n, u32 logn,
                                                      const u32* __restrict__ ladder, NttC<L, FW> c,
                                                      const u32* __restrict__ one_m, const u32* __restrict__ adj) {
  u64 e = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  u32 acc[L];
#pragma unroll
  for (int j = 0; j < L; j++) acc[j] = one_m[j];
  if (e > 0) {
    u32 s = 63 - __builtin_clzll(e);
    u64 ip = e - (1ull << s);
    u64 x = ip << (logn - s - 1);
    for (u32 bit = 0; bit < logn; bit++) {
      if ((x >> bit) & 1) {
        u32 w[L], t[L];
#pragma unroll
        for (int j = 0; j < L; j++) w[j] = ladder[bit * L + j];
        if constexpr (FW)
          mont_mul_fw<L>(t, acc, w, c.q, c.qinv, c.q);
        else
          mont_mul<L>(t, acc, w, c.q, c.qinv);
#pragma unroll
        for (int j = 0; j < L; j++) acc[j] = t[j];
      }
    }
  }
  // acc = w^x 2^(32L).  Times 1 it gives w^x itself; times adj = 2^(bD) it
  // gives r = w^x R mod q (R = 2^(bD)), whose Montgomery digits
  // m = -r q^-1 mod R are floor(w^x R / q), since w^x R - r is that times q.
  constexpr int b = Digits<L, FW>::b, D = Digits<L, FW>::D, S = tw_words(L, FW);
  u32 ad[L], one[L], wm[L], wp[L], r[D], d[S];
#pragma unroll
  for (int j = 0; j < L; j++) {
    ad[j] = adj[j];
    one[j] = j == 0 ? 1u : 0u;
  }
  if constexpr (FW) {
    mont_mul_fw<L>(wm, acc, ad, c.q, c.qinv, c.q);
    mont_mul_fw<L>(wp, acc, one, c.q, c.qinv, c.q);
  } else {
    mont_mul<L>(wm, acc, ad, c.q, c.qinv);
    mont_mul<L>(wp, acc, one, c.q, c.qinv);
  }
  to_digits<L, FW>(r, wm);
  u64 carry = 0;
#pragma unroll
  for (int i = 0; i < D; i++) {
    carry += r[i];
#pragma unroll
    for (int j = 0; j < i; j++) carry += (u64)d[j] * c.qd[i - j];
    d[i] = ((u32)carry * c.qinvd) & Digits<L, FW>::mask;
    carry += (u64)d[i] * c.qd[0];
    carry >>= b;
  }
  to_digits<L, FW>(d + D, wp);
#pragma unroll
  for (int j = 2 * D; j < S; j++) d[j] = 0;
  uint4* out = reinterpret_cast<uint4*>(tw);
#pragma unroll
  for (int j = 0; j < S / 4; j++) out[j * n + e] = make_uint4(d[4 * j], d[4 * j + 1], d[4 * j + 2], d[4 * j + 3]);
  if constexpr (S % 4) reinterpret_cast<uint2*>(tw + (S - 2) * n)[e] = make_uint2(d[S - 2], d[S - 1]);
}

template <int L, bool FW = false>
inline NttC<L, FW> make_consts(const FieldRaw& f, const DigitConsts& dc) {
  NttC<L, FW> c;
  for (int j = 0; j < Digits<L, FW>::D; j++) {
    c.qd[j] = dc.qd[j];
    c.nqd[j] = f.nqd[j];
  }
  c.qinvd = dc.qinvd;
  u64 carry = 0;
  for (int j = 0; j < L; j++) {
    c.q[j] = f.q[j];
    u64 d = ((u64)f.q[j] << 1) + carry;  // 2q limb by limb (wraps for a full-width q, where it is unused)
    c.q2[j] = (u32)d;
    carry = d >> 32;
  }
  if constexpr (!FW && (offset_applies(L, 1) || offset_applies(L, 2))) {
    for (int j = 0; j < L; j++) c.qsw[j] = f.qsw[j];
    c.d = f.d;
    c.cinv = f.cinv;
  }
  c.qinv = f.qinv;
  return c;
}

template <int L, int R, bool MUL, bool LASTX, int AR = kArithLazy>
int launch_pass_LRM(const NttC<L, AR == kArithFull>& c, const NttPassArgs& pass, uint32_t threads, uint64_t tiles,
                    hipStream_t s) {
  NttPassArgs a = pass;
  a.xcd_log = xcd_group_log(a.logc, tiles);
  size_t lds = (size_t)L * ((size_t)1 << (a.k + a.logc)) * sizeof(u32);
  static std::atomic<bool> attr_set{false};  // several host threads may launch at once
  if (lds > 65536 && !attr_set.load(std::memory_order_acquire)) {
    (void)hipFuncSetAttribute((const void*)ntt_pass_kernel<L, R, MUL, LASTX, AR>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    attr_set.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((ntt_pass_kernel<L, R, MUL, LASTX, AR>), dim3((unsigned)tiles), dim3(threads), lds, s, a, c);
  return (int)hipGetLastError();
}

// (up to 8 limbs: at 10 limbs the fused round measured level at 2^20 points
// and 3% slower at 2^18)
template <int L>
constexpr bool kFusedLast = L <= 8;

// Whether a pass's first round reads its elements straight from HBM (the
// LASTX variant does when it has no fused product): 16 or 32 groups per tile
// (each load instruction then covers 64- or 128-byte runs, as the load phase's
// do), more than one round, and at least two tiles per compute unit.  Measured:
// 1 to 7% faster transforms from 64 to 256 bits at 2^19 to 2^25 points; with
// one tile per compute unit (2^18 points, 256 bits) the load phase's wider
// loads were 4% faster.
inline bool direct_load_applies(const NttPassArgs& a, uint32_t radix_log, uint64_t tiles) {
  return !a.in2 && (a.logc == 4 || a.logc == 5) && a.k > radix_log && tiles >= 2ull * device_cu_count();
}

// The batch executor's choice for one pass record: the variant kernel when the
// pass would take the cross-lane last stage or the direct first round (a batch
// launch holds many tiles, so the tile-count rule of a lone call is not applied).
inline bool batch_variant(int L, uint32_t radix_log, uint32_t threads, NttPassArgs* a) {
  if ((radix_log != 2 && radix_log != 3) || L > 8) return false;
  const bool direct = !a->in2 && (a->logc == 4 || a->logc == 5) && a->k > radix_log;
  a->direct = direct ? 1u : 0u;
  return direct || fused_last_applies(*a, threads, radix_log);
}

template <int L, int R, bool MUL>
int launch_pass_LRX(const NttC<L>& c, const NttPassArgs& a, uint32_t threads, uint64_t tiles, hipStream_t s) {
  if constexpr ((R == 2 || R == 3) && kFusedLast<L>) {
    const bool direct = direct_load_applies(a, R, tiles);
    if (direct || fused_last_applies(a, threads, R)) {
      NttPassArgs b = a;
      b.direct = direct ? 1u : 0u;
      return launch_pass_LRM<L, R, MUL, true>(c, b, threads, tiles, s);
    }
  }
  return launch_pass_LRM<L, R, MUL, false>(c, a, threads, tiles, s);
}

template <int L, int R>
int launch_pass_LR(const NttC<L>& c, const NttPassArgs& a, uint32_t threads, uint64_t tiles, hipStream_t s) {
  return a.in2 ? launch_pass_LRX<L, R, true>(c, a, threads, tiles, s)
               : launch_pass_LRX<L, R, false>(c, a, threads, tiles, s);
}

// full-width modulus: radix-2 and radix-4 units, no cross-lane variant
template <int L>
int launch_pass_fw(const FieldRaw& f, const DigitConsts& dc, const NttPassArgs& a, uint32_t threads,
                   uint64_t tiles, uint32_t radix_log, hipStream_t s) {
  NttC<L, true> c = make_consts<L, true>(f, dc);
  if (radix_log == 1)
    return a.in2 ? launch_pass_LRM<L, 1, true, false, kArithFull>(c, a, threads, tiles, s)
                 : launch_pass_LRM<L, 1, false, false, kArithFull>(c, a, threads, tiles, s);
  if constexpr (L <= kMaxLimbsRadix4Fw) {
    if (radix_log == 2)
      return a.in2 ? launch_pass_LRM<L, 2, true, false, kArithFull>(c, a, threads, tiles, s)
                   : launch_pass_LRM<L, 2, false, false, kArithFull>(c, a, threads, tiles, s);
  }
  return (int)hipErrorInvalidValue;
}

template <int L>
int launch_pass_L(const FieldRaw& f, const DigitConsts& dc, const NttPassArgs& a, uint32_t threads,
                  uint64_t tiles, uint32_t radix_log, uint32_t kara, hipStream_t s) {
  if (f.fw)
    return kara ? (int)hipErrorInvalidValue : launch_pass_fw<L>(f, dc, a, threads, tiles, radix_log, s);
  NttC<L> c = make_consts<L>(f, dc);
  if (kara) {
    // the Karatsuba butterfly: radix-2 units, 2 to 24 limbs, no cross-lane variant
    if constexpr (L >= 2 && L <= kMaxLimbsKara) {
      if (radix_log == 1)
        return a.in2 ? launch_pass_LRM<L, 1, true, false, kArithKara>(c, a, threads, tiles, s)
                     : launch_pass_LRM<L, 1, false, false, kArithKara>(c, a, threads, tiles, s);
    }
    return (int)hipErrorInvalidValue;
  }
  // register blocking is limited by the VGPR budget: 2^r elements of L limbs
  if (radix_log == 1) return launch_pass_LR<L, 1>(c, a, threads, tiles, s);
  if constexpr (L <= kMaxLimbsRadix4) {
    if (radix_log == 2) return launch_pass_LR<L, 2>(c, a, threads, tiles, s);
  }
  if constexpr (L <= kMaxLimbsRadix8) {
    if (radix_log == 3) return launch_pass_LR<L, 3>(c, a, threads, tiles, s);
  }
  if constexpr (L <= kMaxLimbsRadix16) {
    if (radix_log == 4) return launch_pass_LR<L, 4>(c, a, threads, tiles, s);
  }
  return (int)hipErrorInvalidValue;
}

template <int L, int R, bool LASTX, bool FW = false>
int launch_batch_LRX(bool mul, uint32_t threads, size_t lds, uint32_t grid, const NttPassArgs* d_passes,
                     const void* d_consts, const uint2* d_items, uint32_t nitems, hipStream_t s) {
  if (mul)
    hipLaunchKernelGGL((ntt_batch_kernel<L, R, true, LASTX, FW>), dim3(grid), dim3(threads), lds, s, d_passes,
                       (const NttC<L, FW>*)d_consts, d_items, nitems);
  else
    hipLaunchKernelGGL((ntt_batch_kernel<L, R, false, LASTX, FW>), dim3(grid), dim3(threads), lds, s, d_passes,
                       (const NttC<L, FW>*)d_consts, d_items, nitems);
  return (int)hipGetLastError();
}

template <int L, int R>
int launch_batch_LR(bool mul, bool lastx, uint32_t threads, size_t lds, uint32_t grid, const NttPassArgs* d_passes,
                    const void* d_consts, const uint2* d_items, uint32_t nitems, hipStream_t s) {
  if constexpr ((R == 2 || R == 3) && kFusedLast<L>) {
    if (lastx)
      return launch_batch_LRX<L, R, true>(mul, threads, lds, grid, d_passes, d_consts, d_items, nitems, s);
  }
  if (lastx) return (int)hipErrorInvalidValue;
  return launch_batch_LRX<L, R, false>(mul, threads, lds, grid, d_passes, d_consts, d_items, nitems, s);
}

template <int L>
int launch_batch_L(uint32_t radix_log, bool mul, bool lastx, bool fw, uint32_t threads, size_t lds, uint32_t grid,
                   const NttPassArgs* d_passes, const void* d_consts, const uint2* d_items, uint32_t nitems,
                   hipStream_t s) {
  if (fw) {
    // full-width modulus: radix-2 and radix-4 units, no cross-lane variant
    if (lastx) return (int)hipErrorInvalidValue;
    if (radix_log == 1)
      return launch_batch_LRX<L, 1, false, true>(mul, threads, lds, grid, d_passes, d_consts, d_items, nitems, s);
    if constexpr (L <= kMaxLimbsRadix4Fw) {
      if (radix_log == 2)
        return launch_batch_LRX<L, 2, false, true>(mul, threads, lds, grid, d_passes, d_consts, d_items, nitems, s);
    }
    return (int)hipErrorInvalidValue;
  }
  if (radix_log == 1)
    return launch_batch_LR<L, 1>(mul, lastx, threads, lds, grid, d_passes, d_consts, d_items, nitems, s);
  if constexpr (L <= kMaxLimbsRadix4) {
    if (radix_log == 2)
      return launch_batch_LR<L, 2>(mul, lastx, threads, lds, grid, d_passes, d_consts, d_items, nitems, s);
  }
  if constexpr (L <= kMaxLimbsRadix8) {
    if (radix_log == 3)
      return launch_batch_LR<L, 3>(mul, lastx, threads, lds, grid, d_passes, d_consts, d_items, nitems, s);
  }
  if constexpr (L <= kMaxLimbsRadix16) {
    if (radix_log == 4)
      return launch_batch_LR<L, 4>(mul, lastx, threads, lds, grid, d_passes, d_consts, d_items, nitems, s);
  }
  return (int)hipErrorInvalidValue;
}

// allow the batch kernels more than 64 KiB of dynamic LDS; called before graph
// capture so that nothing but launches is recorded
template <int L, int R>
void batch_attr_LR() {
  (void)hipFuncSetAttribute((const void*)ntt_batch_kernel<L, R, false, false>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)hipFuncSetAttribute((const void*)ntt_batch_kernel<L, R, true, false>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if constexpr ((R == 2 || R == 3) && kFusedLast<L>) {
    (void)hipFuncSetAttribute((const void*)ntt_batch_kernel<L, R, false, true>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    (void)hipFuncSetAttribute((const void*)ntt_batch_kernel<L, R, true, true>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  }
}

template <int L>
void batch_attr_L(uint32_t radix_log, bool fw) {
  if (fw) {
    const void* k[4] = {(const void*)ntt_batch_kernel<L, 1, false, false, true>,
                        (const void*)ntt_batch_kernel<L, 1, true, false, true>, nullptr, nullptr};
    if constexpr (L <= kMaxLimbsRadix4Fw) {
      k[2] = (const void*)ntt_batch_kernel<L, 2, false, false, true>;
      k[3] = (const void*)ntt_batch_kernel<L, 2, true, false, true>;
    }
    for (const void* f : k)
      if (f) (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    return;
  }
  if (radix_log == 1) batch_attr_LR<L, 1>();
  if constexpr (L <= kMaxLimbsRadix4) {
    if (radix_log == 2) batch_attr_LR<L, 2>();
  }
  if constexpr (L <= kMaxLimbsRadix8) {
    if (radix_log == 3) batch_attr_LR<L, 3>();
  }
  if constexpr (L <= kMaxLimbsRadix16) {
    if (radix_log == 4) batch_attr_LR<L, 4>();
  }
}

template <int L>
int launch_tw_L(const FieldRaw& f, const DigitConsts& dc, uint32_t* tw, uint64_t n, uint32_t logn,
                       const uint32_t* d_ladder, hipStream_t s) {
  // the ladder buffer carries one_m and then adj after the logn ladder entries
  const u32* one_m = d_ladder + (size_t)logn * L;
  const u32* adj = one_m + L;
  u64 blocks = (n + 255) / 256;
  if (f.fw) {
    NttC<L, true> c = make_consts<L, true>(f, dc);
    hipLaunchKernelGGL((twiddle_kernel<L, true>), dim3((unsigned)blocks), dim3(256), 0, s, tw, n, logn, d_ladder, c,
                       one_m, adj);
  } else {
    NttC<L> c = make_consts<L>(f, dc);
    hipLaunchKernelGGL((twiddle_kernel<L>), dim3((unsigned)blocks), dim3(256), 0, s, tw, n, logn, d_ladder, c,
                       one_m, adj);
  }
  return (int)hipGetLastError();
}

// the per-limb-count entry points, instantiated once (in ntt_inst_*.hip)
#define MOMA_NTT_DECLARE(PREFIX, LL)                                                                              \
  PREFIX template int launch_pass_L<LL>(const FieldRaw&, const DigitConsts&, const NttPassArgs&,                   \
                                        uint32_t, uint64_t, uint32_t, uint32_t, hipStream_t);                       \
  PREFIX template int launch_batch_L<LL>(uint32_t, bool, bool, bool, uint32_t, size_t, uint32_t,                  \
                                         const NttPassArgs*, const void*, const uint2*, uint32_t, hipStream_t);     \
  PREFIX template void batch_attr_L<LL>(uint32_t, bool);                                                            \
  PREFIX template int launch_tw_L<LL>(const FieldRaw&, const DigitConsts&, uint32_t*, uint64_t, uint32_t,          \
                                      const uint32_t*, hipStream_t);
#define MOMA_NTT_INSTANTIATE(LL) MOMA_NTT_DECLARE(, LL)
#define MOMA_NTT_EXTERN(LL) MOMA_NTT_DECLARE(extern, LL)

}  // namespace moma
