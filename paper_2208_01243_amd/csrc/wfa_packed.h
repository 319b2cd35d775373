// Packed 16-bit wavefront arithmetic shared by the kernels that keep two
// diagonals a word (wfa_group.hip, wfa_wide.hip).  Included inside an anonymous
// namespace of each translation unit, after wfa_common.h.
//
// Offsets are kept BIAS (32) above their value: each staged sequence has a word
// of 32 bases in front, A's before the pattern and C's before the text, so that
// an absent offset, which is negative and compares at base 0, matches nothing
// and needs no mask.  Past its end a pattern goes on with A's and a text with
// C's: a run that reaches both ends stops there.
//
// An absent mark starts at -32768 (or, where the table bound cut a candidate,
// at -32768 plus that offset, at most 16,033 more) and grows by at most one a
// score, so pairs stay below 16,000 scores, and texts and patterns at 16,000
// bases, and no mark reaches zero.  A candidate passes its table bound
// min(n, m + k) by at most one (its source was inside its own), so the cut only
// has to set its sign.
#pragma once

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// sign mask of each half
__device__ __forceinline__ uint32_t sign2(uint32_t v) {
  uint32_t r;
  asm("v_pk_ashrrev_i16 %0, 15, %1 op_sel_hi:[0,1]" : "=v"(r) : "v"(v));
  return r;
}
__device__ __forceinline__ uint32_t max2(uint32_t a, uint32_t b) { return as1(__builtin_elementwise_max(as2(a), as2(b))); }
__device__ __forceinline__ uint32_t min2(uint32_t a, uint32_t b) { return as1(__builtin_elementwise_min(as2(a), as2(b))); }
__device__ __forceinline__ uint32_t add2(uint32_t a, uint32_t b) { return as1(as2(a) + as2(b)); }
__device__ __forceinline__ uint32_t sub2(uint32_t a, uint32_t b) { return as1(as2(a) - as2(b)); }
__device__ __forceinline__ uint32_t subs2(uint32_t a, uint32_t b) {
  return as1(__builtin_elementwise_sub_sat(as2(a), as2(b)));
}
__device__ __forceinline__ uint32_t both(int32_t v) { return (uint32_t)(v & 0xffff) * 0x10001u; }
__device__ __forceinline__ uint32_t pack2(int32_t lo, int32_t hi) {
  return __builtin_amdgcn_perm((uint32_t)hi, (uint32_t)lo, 0x05040100u);
}
// a where the mask is set, else b (written out: the compiler spends an
// instruction more on the same bits)
__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(mask), "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ uint32_t bfi_v(uint32_t mask, uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(mask), "v"(a), "v"(b));
  return r;
}

// A condition that is the same in every lane, as a scalar (where the compiler
// does not see that it is, it keeps the loop's counters in vector registers).
__device__ __forceinline__ bool uniform(bool b) { return __builtin_amdgcn_readfirstlane((int)b) != 0; }

// Candidate c against its bound: c, or c with its sign set where c > lim
// (then c == lim + 1).  An absent c may have its sign set again.
__device__ __forceinline__ uint32_t cut2(uint32_t c, uint32_t lim) { return (sub2(lim, c) & 0x80008000u) | c; }

// LDS by byte address: the sequences' words are reached from 16-bit fields of
// packed offsets, whose index arithmetic the compiler otherwise lengthens.
typedef __attribute__((address_space(3))) uint32_t LdsWord;
typedef __attribute__((address_space(3))) unsigned char LdsByte;
__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)(LdsByte *)p; }

// 16 bases of a staged sequence from base i (16 i' <= i < 16 i' + 16, at word
// i' of the sequence at byte address w).
__device__ __forceinline__ uint32_t bases16(uint32_t w, uint32_t word, uint32_t shift) {
  const LdsWord *p = (const LdsWord *)(uintptr_t)(w + (word << 2));
  return __builtin_amdgcn_alignbit(p[1], p[0], shift);
}
__device__ __forceinline__ uint32_t bases16(uint32_t w, int32_t i) {
  return bases16(w, (uint32_t)i >> 4, (uint32_t)i << 1);
}
// ... from the base in the low / high half of a packed pair of indices
__device__ __forceinline__ uint32_t bases16_lo(uint32_t w, uint32_t ii) {
  uint32_t word;
  asm("v_bfe_u32 %0, %1, 4, 12" : "=v"(word) : "v"(ii));
  return bases16(w, word, ii << 1);
}
__device__ __forceinline__ uint32_t bases16_hi(uint32_t w, uint32_t ii) {
  uint32_t word;
  asm("v_lshrrev_b32 %0, 20, %1" : "=v"(word) : "v"(ii));
  return bases16(w, word, ii >> 15);
}

// Equal bases from base i of the pattern and j of the text, at most lim, 32 a
// step (a step's second half is read within the sequences' words or not at
// all).
__device__ __forceinline__ int32_t match_run(uint32_t pw, uint32_t tw, int32_t i, int32_t j, int32_t lim) {
  int32_t run = 0;
  while (run < lim) {
    const int32_t a = i + run, b = j + run, h = lim - run > 16 ? 16 : 0;
    const uint32_t d0 = bases16(pw, a) ^ bases16(tw, b);
    const uint32_t d1 = bases16(pw, a + h) ^ bases16(tw, b + h);
    run += (int32_t)(d0 ? ffbl_raw(d0) >> 1 : 16u + min(ffbl_raw(d1) >> 1, 16u));
    if (d0 | d1) break;
  }
  return min(run, lim);
}

constexpr int32_t BIAS = 32;
constexpr uint64_t ENDS_T = 0x5555555555555555ull;  // C's
// A staged word whose bases from `bases` on are replaced by `fill`.
__device__ __forceinline__ uint64_t upto(uint64_t v, int32_t bases, uint64_t fill) {
  const uint64_t in = bases >= 32 ? ~0ull : bases <= 0 ? 0ull : (1ull << (2 * bases)) - 1ull;
  return (v & in) | (fill & ~in);
}

// The origin codes of a cell as its row keeps them: X < M, I < M (sign bits of
// cx, ci), and as a source, I and D extended from it (sio, sdo): the four bits
// of each half, from bit 12 up, shifted in above the codes of earlier scores.
__device__ __forceinline__ uint32_t push_codes(uint32_t acc, uint32_t cx, uint32_t ci, uint32_t sio, uint32_t sdo) {
  const uint32_t a = bfi(0x80008000u, cx, ci >> 1), b = bfi(0x80008000u, sio, sdo >> 1);
  return bfi(0xf000f000u, bfi(0xc000c000u, a, b >> 2), acc >> 4);
}
// The codes of fewer than four scores (the last one's step in step & 3) at
// the bits they have in a full word.
__device__ __forceinline__ uint32_t settle_codes(uint32_t acc, int32_t step) {
  const uint32_t sh = 4 * (3 - (step & 3));
  return ((acc >> sh) & 0xffff0000u) | ((acc & 0xffffu) >> sh);
}

// The first 16 bases of both diagonals of a word extended (Mv: offsets, K2:
// diagonals): bits that match, halved; 0x7fff for all 16 bases.
__device__ __forceinline__ uint32_t first_run2(uint32_t pw, uint32_t tw, uint32_t Mv, uint32_t K2) {
  const uint32_t J = max2(Mv, 0u), Ii = max2(subs2(Mv, K2), 0u);
  const uint32_t da = bases16_lo(pw, Ii) ^ bases16_lo(tw, J), db = bases16_hi(pw, Ii) ^ bases16_hi(tw, J);
  uint32_t rr = pack2((int32_t)ffbl_raw(da), (int32_t)ffbl_raw(db));
  asm("v_pk_lshrrev_b16 %0, 1, %1 op_sel_hi:[0,1]" : "=v"(rr) : "v"(rr));
  return rr;
}
// The halves of F whose first run was 16 bases (rr) extended to their ends.
__device__ __forceinline__ uint32_t long_runs2(uint32_t pw, uint32_t tw, uint32_t Mv, uint32_t K2, uint32_t LIM, uint32_t rr,
                                               uint32_t F) {
  uint32_t todo = rr & 0x40004000u;
  while (todo) {
    const uint32_t sh = (todo & 0x4000u) ? 0u : 16u;
    todo &= todo - 1u;
    const int32_t f = (int32_t)(Mv >> sh) & 0xffff, l = (int32_t)(LIM >> sh) & 0xffff;
    const int32_t i = f - (int32_t)(int16_t)(K2 >> sh);
    const int32_t g = min(f + 16 + match_run(pw, tw, i + 16, f + 16, max(l - f - 16, 0)), l);
    F = sh ? pack2((int32_t)F, g) : bfi_v(0xffffu, (uint32_t)g, F);
  }
  return F;
}
