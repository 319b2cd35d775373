// Gap-affine wavefront alignment (WFA) of pairs whose wavefronts are wide, one
// pair per workgroup of T lanes (k_wfa_wide), for unit gap extension.
//
// Paper: System and Methods, "Wavefront Algorithm (WFA)" (the recurrences of
// wfa.hip, restated there) and "Data Management" (the components a step needs
// stay in fast memory).
//
// What bounds it.  The class kernel (k_wfa_lds) spends about 70 vector
// instructions a cell and streams its rings of M, I and D through the fabric
// (4.8 TB/s).  Here a lane owns C neighbouring words of two diagonals: I and D
// of the last score stay in its registers, M of the last R scores in LDS rows
// that it reads back itself; only max(M, I) and max(M, D) of the neighbouring
// lane are needed (the max commutes with the shift), which one lane shift each
// brings for all C words, and between wavefronts a word each through LDS.  About
// 31 instructions a cell, and no memory traffic but the codes.
//
// The window grows in stages: C = 1, 2, 3, ... words a lane, each until a
// wavefront could pass its edge (a wavefront of score s reaches diagonals
// -(s - o) .. s - o), so that lanes without cells cost at most about as much as
// those with.  At a change of stage I and D go through LDS to the lanes that
// own them next.  A pair that outgrows the last stage goes on by predicted
// extent to the class kernel.
//
// Arithmetic and codes: wfa_packed.h, wfa_group.hip.  Codes lie in rows of the
// stage's words, one per four scores.
//
// The walks wait until every wavefront of the workgroup has one: a walk is one
// wavefront's serial chain (a quarter of the kernel's time when it ran after
// each pair, the other wavefronts idle: 200,000 pairs of 100-10,000 bp spent 49
// of 147 ms here in it).
//
// Measured on those 200,000 pairs: 30 ms for the 55,169 that enter the narrower
// window and 86 for the 25,096 of the wider (the batch: 195 ms with the class
// kernel, 145 now).  Vector instructions issue 73 % of the time and LDS is busy
// half of it; a score's chain of ring reads, sequence reads and the barrier is
// about as long as four wavefronts' instructions for it, so that wavefronts that
// skip scores before their diagonals are reached gave 1 %, half as many words a
// lane on twice the lanes (64 registers, some spilled) lost 4 %, and extending
// the runs of all of a lane's words in one loop gave nothing.
#include <algorithm>

#include "aim_internal.h"

namespace aim {
namespace {

#include "wfa_common.h"
#include "wfa_packed.h"

// Orders LDS accesses of the workgroup (global stores are not waited for).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int C>
__device__ __forceinline__ void ld_words(const uint32_t *p, uint32_t (&v)[C]) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  if constexpr (C % 2 == 1) {
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = p[c];
  } else if constexpr (C % 4 == 0) {
#pragma unroll
    for (int c = 0; c < C; c += 4) {
      const u4 w = *reinterpret_cast<const u4 *>(p + c);
      v[c] = w.x; v[c + 1] = w.y; v[c + 2] = w.z; v[c + 3] = w.w;
    }
  } else {
#pragma unroll
    for (int c = 0; c < C; c += 2) {
      const u2 w = *reinterpret_cast<const u2 *>(p + c);
      v[c] = w.x; v[c + 1] = w.y;
    }
  }
}
template <int C>
__device__ __forceinline__ void st_words(uint32_t *p, const uint32_t (&v)[C]) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  if constexpr (C % 2 == 1) {
#pragma unroll
    for (int c = 0; c < C; ++c) p[c] = v[c];
  } else if constexpr (C % 4 == 0) {
#pragma unroll
    for (int c = 0; c < C; c += 4) *reinterpret_cast<u4 *>(p + c) = u4{v[c], v[c + 1], v[c + 2], v[c + 3]};
  } else {
#pragma unroll
    for (int c = 0; c < C; c += 2) *reinterpret_cast<u2 *>(p + c) = u2{v[c], v[c + 1]};
  }
}

// What the stages of a pair share (the same in every lane, but for the two
// sequence addresses).
struct WideState {
  int32_t m, n, par;       // par: the end diagonal's parity
  int32_t s, s_lim;        // score; last score to try
  int32_t rowW, rowX, rowO;  // ring rows (offsets in words) of score s, and of its two sources
  int32_t result;          // 0: none yet, 1: aligned, 2: past s_lim, 3: window outgrown
  bool keep;               // codes are kept
  int32_t coff;            // words of codes this pair has stored
  int32_t stage;           // words a lane of the last stage that ran
};
// A finished pair that awaits its walk.
struct WideDone {
  int32_t p, s, code, stage;  // code: its first word in the workgroup's codes
};

// The last score of the stage of c words a lane, unless it is the last stage or
// no pair of these lengths can leave it: one that fills a row of codes.
__host__ __device__ constexpr int32_t stage_end(int32_t T, int32_t c, int32_t o) { return ((T * c - 3 + o - 3) & ~3) + 3; }
// Row r of a pair's codes: its first word, and its stage.
template <int T, int CMAX>
__device__ __forceinline__ int32_t code_row(int32_t r, int32_t o, int32_t last, int32_t &stage) {
  int32_t at = r * T, c = 1;
#pragma unroll
  for (int32_t k = 1; k < CMAX; ++k) {
    // rows past the end of stage k hold T words more
    const int32_t e = (stage_end(T, k, o) + 1) / 4;
    if (k < last && r >= e) {
      at += (r - e) * T;
      c = k + 1;
    }
  }
  stage = c;
  return at;
}

constexpr int32_t GUARD = 4;  // words of LDS before and after the ring (reads past a window's edge)

// The scores of one pair in a window of T C words, until the end cell, s_lim
// or the stage's last score.  I and D of score W.s come in and go out through
// ring row `spare` (that of score W.s + 1, whose words the next score writes).
template <int T, int C, int NW>
__device__ __forceinline__ void wide_stage(WideState &W, const int32_t x, const int32_t oe, const int32_t R, uint32_t *ring, uint32_t *edge,
                           int32_t *flag, uint32_t pw, uint32_t tw, uint32_t *codes, int32_t code_cap) {
  constexpr int32_t REACH = T * C - 3;
  constexpr int32_t WAVES = T / 64;
  const int32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t pos = tid * C + (NW - T * C) / 2;  // this lane's first word in a row
  const int32_t rend = R * NW;
  // the last score of the stage: one that fills a word of codes
  const bool last_stage = T * C == NW;
  const bool unbounded = max(W.m, W.n) <= REACH;  // no wavefront of this pair leaves the window
  const int32_t s_stage = unbounded ? INT32_MAX : last_stage ? REACH + oe - 1 : stage_end(T, C, oe - 1);
  if (W.s >= s_stage) return;
  W.stage = C;
  uint32_t Iv[C], Dv[C], cacc[C], K2[C], LIM[C], TGT[C];
  const int32_t kend = W.n - W.m;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int32_t k = 2 * (tid * C + c - T * C / 2) - W.par;
    K2[c] = pack2(k, k + 1);
    LIM[c] = min2(add2(both(W.m + BIAS), K2[c]), both(W.n + BIAS));
    TGT[c] = (uint32_t)(k == kend ? W.n + BIAS : 0x7fff);
    cacc[c] = 0;
    Iv[c] = Dv[c] = ABSENT2;
  }
  if (W.s > 0) {
    // I and D of the stage before (it wrote them behind each other into the
    // rows of the next score and, the ring being longer by one, the one after)
    const int32_t r1 = W.rowW + NW == rend ? 0 : W.rowW + NW;
    ld_words<C>(ring + r1 + pos, Iv);
    ld_words<C>(ring + rend + pos, Dv);
    lds_barrier();
  }
  auto put_edges = [&](int32_t par) {
    // lane 0's I and lane 63's D, for the neighbouring wavefronts
    uint32_t *e = edge + par * 2 * (WAVES + 2) + wave + 1;
    if (lane == 0) e[0] = Iv[0];
    if (lane == 63) e[WAVES + 2] = Dv[C - 1];
  };
  put_edges(W.s & 1);
  lds_barrier();
  const int32_t npos = lane == 63 ? pos + C : pos - 1;                        // the neighbouring wavefront's word
  const int32_t nedge = lane == 63 ? wave + 2 : wave + (WAVES + 2);           // its I, or D
  while (true) {
    // score s tells of its end cell in flag[s & 1]: a wavefront that is a step
    // ahead writes the other one
    const int32_t par = W.s & 1, hitv = flag[par];
    // (uniform: every lane reads the same word)
    if (__builtin_amdgcn_readfirstlane(hitv)) { W.result = 1; break; }
    if (W.s >= W.s_lim) { W.result = 2; break; }
    if (W.s >= s_stage) break;
    ++W.s;
    W.rowW = W.rowW + NW == rend ? 0 : W.rowW + NW;
    W.rowX = W.rowX + NW == rend ? 0 : W.rowX + NW;
    W.rowO = W.rowO + NW == rend ? 0 : W.rowO + NW;
    uint32_t Mo[C], Mx[C];
    ld_words<C>(ring + W.rowO + pos, Mo);
    ld_words<C>(ring + W.rowX + pos, Mx);
    const uint32_t en = max2(ring[W.rowO + npos], edge[par * 2 * (WAVES + 2) + nedge]);
    const uint32_t An = (uint32_t)__builtin_amdgcn_update_dpp((int)en, (int)max2(Mo[0], Iv[0]), 0x130, 0xf, 0xf, false);          // wave_shl:1
    uint32_t dn = (uint32_t)__builtin_amdgcn_update_dpp((int)en, (int)max2(Mo[C - 1], Dv[C - 1]), 0x138, 0xf, 0xf, false);  // wave_shr:1
    uint32_t a = max2(Mo[0], Iv[0]);
    uint32_t F[C], Mv[C], rr[C], full = 0;
    const bool kc = W.keep;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const uint32_t up = c + 1 < C ? max2(Mo[c + 1 < C ? c + 1 : 0], Iv[c + 1 < C ? c + 1 : 0]) : An;
      const uint32_t b = max2(Mo[c], Dv[c]);
      const uint32_t I = cut2(__builtin_amdgcn_alignbit(up, a, 16), LIM[c]);
      const uint32_t D = cut2(add2(__builtin_amdgcn_alignbit(b, dn, 16), 0x00010001u), LIM[c]);
      const uint32_t X = cut2(add2(Mx[c], 0x00010001u), LIM[c]);
      const uint32_t ID = max2(I, D);
      Mv[c] = max2(X, ID);
      rr[c] = first_run2(pw, tw, Mv[c], K2[c]);
      if (kc) cacc[c] = push_codes(cacc[c], subs2(X, ID), subs2(I, D), subs2(Mo[c], Iv[c]), subs2(Mo[c], Dv[c]));
      a = up;
      dn = b;
      Iv[c] = I;
      Dv[c] = D;
      F[c] = min2(add2(Mv[c], rr[c]), LIM[c]);
      full |= rr[c];
    }
    if (full & 0x40004000u) {
#pragma unroll
      for (int c = 0; c < C; ++c) F[c] = long_runs2(pw, tw, Mv[c], K2[c], LIM[c], rr[c], F[c]);
    }
    bool hit = false;
#pragma unroll
    for (int c = 0; c < C; ++c) hit = hit || (int16_t)F[c] >= (int16_t)TGT[c];
    st_words<C>(ring + W.rowW + pos, F);
    put_edges(par ^ 1);
    if (hit) flag[par ^ 1] = 1;
    if (kc && (W.s & 3) == 3) {
      if (W.coff + T * C <= code_cap) st_words<C>(codes + W.coff + tid * C, cacc);
      else W.keep = false;
      W.coff += T * C;
    }
    lds_barrier();
  }
  if (W.result == 1 && W.keep && (W.s & 3) != 3) {
    uint32_t v[C];
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = settle_codes(cacc[c], W.s);
    if (W.coff + T * C <= code_cap) st_words<C>(codes + W.coff + tid * C, v);
    else W.keep = false;
    W.coff += T * C;
  }
  if (W.result == 0 && !last_stage) {
    const int32_t r1 = W.rowW + NW == rend ? 0 : W.rowW + NW;
    st_words<C>(ring + r1 + pos, Iv);
    st_words<C>(ring + rend + pos, Dv);
    lds_barrier();
  }
}

// An aligned pair whose codes cannot be walked: to the full-store pass with
// room for every score at its widest.  One thread.
__device__ __forceinline__ void to_full_store(const Outs &O, const WfaWide &L, int64_t p, int32_t s, int32_t m, int32_t n) {
  if (!L.need) {
    O.status[p] = ST_OVERFLOW;  // none planned: the codes of every pair are kept
    return;
  }
  const int64_t w = min(2 * (int64_t)s + 3, (int64_t)m + n + 1);
  const int64_t need = ((int64_t)s + 1) * (ENTRY + (3 * w + 1) / 2);
  L.need[p] = need;
  int c = 0;
  while (c < 3 && need > L.need_cap[c]) ++c;
  if (need > L.need_cap[3]) {
    to_long_pass(O, p, L.long_list, L.long_count);
  } else {
    L.need_list[c][atomicAdd(L.need_count[c], 1)] = (int32_t)p;
    atomicMax(L.need_max[c], (int32_t)need);
  }
}

// The walk of one finished pair by one wavefront, its sequences staged in
// `room` words of LDS where they fit.
template <int T, int CMAX>
__device__ __forceinline__ void walk_one(const Seqs &S, const Outs &O, const Scoring &P, const WfaWide &L, const WideDone d_,
                                         const uint32_t *codes_, uint32_t *tok, uint32_t *lds, int32_t room) {
  const int32_t lane = threadIdx.x & 63;
  const int32_t s = __builtin_amdgcn_readfirstlane(d_.s), last = __builtin_amdgcn_readfirstlane(d_.stage);
  const int64_t p = __builtin_amdgcn_readfirstlane(d_.p);
  const uint32_t *codes = codes_ + __builtin_amdgcn_readfirstlane(d_.code);
  const int32_t m = __builtin_amdgcn_readfirstlane(S.pat_len[p]), n = __builtin_amdgcn_readfirstlane(S.txt_len[p]);
  const int32_t par = (n - m) & 1, o = P.o, oe = P.o + 1;
  const uint64_t *gP = S.pat + S.pat_off[p], *gT = S.txt + S.txt_off[p];
  const int32_t pnw = (m + 31) >> 5, tnw = (n + 31) >> 5;
  auto code_at = [&](int32_t cs, int32_t k) -> int32_t {  // per lane
    if (cs < 1 || cs > s) return -1;
    int32_t c;
    const int32_t at = code_row<T, CMAX>(cs >> 2, o, last, c);
    const int32_t kp = k + par, q = (kp >> 1) + T * c / 2;
    if (q < 0 || q >= T * c) return -1;
    const uint32_t *row = codes + at;
    // (the furthest diagonal that a stage reaches may lie in its first or last
    // word; past those every source is absent)
    const int32_t qn = (kp & 1) ? q + 1 : q - 1;
    const uint32_t v = row[q] >> (4 * (cs & 3)), u = qn >= 0 && qn < T * c ? row[qn] >> (4 * (cs & 3)) : 0u;
    // the cell's own bits, and those of k + 1 and k - 1 as sources
    const uint32_t own = (kp & 1) ? v >> 16 : v;
    const uint32_t up = (kp & 1) ? u : v >> 16, dn = (kp & 1) ? v : u >> 16;
    return (int32_t)(((own & 8u) ? ((own & 4u) ? 2u : 1u) : 0u) | ((up & 2u) ? 0u : 4u) | ((dn & 1u) ? 0u : 8u));
  };
  bool walked;
  if (2 * (pnw + 1 + tnw + 1) <= room) {
    uint64_t *wP = reinterpret_cast<uint64_t *>(lds), *wT = wP + pnw + 1;
    for (int32_t q = lane; q <= pnw; q += 64) wP[q] = q < pnw ? gP[q] : 0ull;
    for (int32_t q = lane; q <= tnw; q += 64) wT[q] = q < tnw ? gT[q] : 0ull;
    __threadfence_block();
    auto ext = [&](int32_t k, int32_t f) {
      return extend_wave(reinterpret_cast<const uint32_t *>(wP), m, reinterpret_cast<const uint32_t *>(wT), n, k, f);
    };
    walked = walk_codes<true>(O, p, code_at, ext, P.x, oe, 1, m, n, s, tok, L.tok_cap);
  } else {
    auto ext = [&](int32_t k, int32_t f) { return extend(gP, pnw, m, gT, tnw, n, k, f); };
    walked = walk_codes<true>(O, p, code_at, ext, P.x, oe, 1, m, n, s, tok, L.tok_cap);
  }
  if (!walked && lane == 0) {
    if (L.walk_fail) atomicAdd(L.walk_fail, 1);
    O.nruns[p] = 0;
    to_full_store(O, L, p, s, m, n);
  }
}

template <int T, int CMAX>
__global__ __launch_bounds__(T, 4) void k_wfa_wide(Seqs S, Outs O, Scoring P, Work Wk, WfaWide L) {
  constexpr int32_t NW = T * CMAX;  // words of a ring row
  extern __shared__ __align__(16) unsigned char smem[];
  const int32_t tid = threadIdx.x;
  const int32_t x = P.x, oe = P.o + 1, R = L.R;
  const int32_t SW = L.seq_words + 2;
  // R rows of M and one row for the change of stage
  uint32_t *ring = (uint32_t *)smem + GUARD;
  uint32_t *edge = ring + (R + 1) * NW + GUARD;   // [2][I, D][T / 64 + 2]
  WideDone *pend = (WideDone *)(edge + 4 * (T / 64 + 2));  // T / 64
  int32_t *flag = (int32_t *)(pend + T / 64);  // [0], [1] end cell reached (odd, even scores), [2] work item, [3] progress
  uint64_t *sP = (uint64_t *)(flag + 4), *sT = sP + SW;
  uint32_t pw = lds_addr(sP), tw = lds_addr(sT);
  asm("" : "+v"(pw));
  asm("" : "+v"(tw));
  const int32_t count = Wk.count ? __builtin_amdgcn_readfirstlane(*(volatile const int32_t *)Wk.count)
                                 : (int32_t)Wk.n;
  // a workgroup the work can never reach leaves before touching the counter
  if ((int32_t)blockIdx.x >= count) return;
  constexpr int32_t WAVES = T / 64;
  // this workgroup's codes, and behind them the walks' tokens
  uint32_t *codes = L.codes + (int64_t)blockIdx.x * L.slot_words;
  uint32_t *tokens = codes + L.code_words;
  int32_t code_at0 = 0, npend = 0;  // words of codes in use, pairs in `pend`
  if (tid == 0) {
    sP[0] = 0ull;
    sT[0] = ENDS_T;
  }
  if (tid < 4 * (T / 64 + 2)) edge[tid] = ABSENT2;
  if (tid < 2 * GUARD) ring[tid < GUARD ? tid - GUARD : (R + 1) * NW + tid - GUARD] = ABSENT2;
  int32_t li = (int32_t)blockIdx.x;  // the first item is the workgroup's own
  for (;;) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the codes' stores
    __syncthreads();
    if (npend == WAVES || (npend > 0 && (li >= count || code_at0 + L.pair_words > L.code_words))) {
      // every wave's codes before the walks' loads; the acquire drops lines of
      // earlier walks from the CU's vector L1
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      const int32_t wave = tid >> 6;
      if (wave < npend) walk_one<T, CMAX>(S, O, P, L, pend[wave], codes, tokens + (int64_t)wave * L.tok_cap,
                                          ring + wave * ((R + 1) * NW / WAVES), (R + 1) * NW / WAVES);
      __syncthreads();
      npend = 0;
      code_at0 = 0;
    }
    if (li >= count) break;
    const int64_t p = Wk.idx ? (int64_t)__builtin_amdgcn_readfirstlane(Wk.idx[li]) : li;
    // the next item, on its way while this one runs
    if (tid == 0) flag[2] = (int32_t)gridDim.x + atomicAdd(Wk.counter, 1);
    if (!(O.flags && __builtin_amdgcn_readfirstlane((int32_t)O.flags[p]))) {
      WideState W;
      W.m = __builtin_amdgcn_readfirstlane(S.pat_len[p]);
      W.n = __builtin_amdgcn_readfirstlane(S.txt_len[p]);
      const int32_t m = W.m, n = W.n, kend = n - m;
      W.par = kend & 1;
      const int32_t pnw = (m + 31) >> 5, tnw = (n + 31) >> 5;
      {
        // the host sends only batches whose sequences fit the staging area
        const uint64_t *gP = S.pat + S.pat_off[p], *gT = S.txt + S.txt_off[p];
        for (int32_t q = tid; q <= pnw; q += T) sP[q + 1] = upto(q < pnw ? gP[q] : 0ull, m - 32 * q, 0ull);
        for (int32_t q = tid; q <= tnw; q += T) sT[q + 1] = upto(q < tnw ? gT[q] : 0ull, n - 32 * q, ENDS_T);
      }
      {
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        u4 *r4 = reinterpret_cast<u4 *>(ring);
        for (int32_t q = tid; q < (R + 1) * NW / 4; q += T) r4[q] = (u4)ABSENT2;
      }
      if (tid == 0) flag[0] = flag[1] = 0;
      __syncthreads();
      const int32_t ad = m > n ? m - n : n - m;
      const int32_t upper = min(x * min(m, n) + (ad ? P.o + ad : 0), (m ? P.o + m : 0) + (n ? P.o + n : 0));
      W.s_lim = min(P.max_score >= 0 ? min(P.max_score, upper) : upper, L.s_cap);
      // the length difference alone passes the threshold: rejected before any
      // score (such an end diagonal may lie outside the last window of a batch
      // whose windows the threshold bounds)
      const bool past = P.max_score >= 0 && ad > 0 && P.o + ad > P.max_score;
      W.s = 0;
      W.rowW = 0;
      W.rowX = (R - x) * NW;
      W.rowO = (R - oe) * NW;
      W.result = past ? 2 : 0;
      W.keep = P.want_cigar != 0;
      W.coff = 0;
      W.stage = 1;
      constexpr int32_t REACH = NW - 3;
      const bool out = kend < -REACH || kend > REACH;  // no window here holds the end
      if (tid == 0) {
        const int32_t f0 = match_run(pw, tw, BIAS, BIAS, min(m, n));
        // diagonal 0: the low half of its word, or the high one
        ring[NW / 2] = W.par ? (uint32_t)(f0 + BIAS) << 16 | 0x8000u : (uint32_t)(f0 + BIAS) | 0x80000000u;
        if (kend == 0 && f0 >= n) flag[0] = 1;
      }
      __syncthreads();
      if (!out && !past) {
        wide_stage<T, 1, NW>(W, x, oe, R, ring, edge, flag, pw, tw, codes + code_at0, L.pair_words);
        if constexpr (CMAX >= 2)
          if (!W.result) wide_stage<T, 2, NW>(W, x, oe, R, ring, edge, flag, pw, tw, codes + code_at0, L.pair_words);
        if constexpr (CMAX >= 3)
          if (!W.result) wide_stage<T, 3, NW>(W, x, oe, R, ring, edge, flag, pw, tw, codes + code_at0, L.pair_words);
        if constexpr (CMAX >= 4)
          if (!W.result) wide_stage<T, 4, NW>(W, x, oe, R, ring, edge, flag, pw, tw, codes + code_at0, L.pair_words);
        if constexpr (CMAX >= 5)
          if (!W.result) wide_stage<T, 5, NW>(W, x, oe, R, ring, edge, flag, pw, tw, codes + code_at0, L.pair_words);
        if constexpr (CMAX >= 6)
          if (!W.result) wide_stage<T, 6, NW>(W, x, oe, R, ring, edge, flag, pw, tw, codes + code_at0, L.pair_words);
      }
      if (!W.result) W.result = 3;
      const int32_t s = W.s;
      if (W.result == 2) {
        // past the last score to try
        W.result = past || (P.max_score >= 0 && s + 1 > P.max_score) ? 2 : s + 1 > upper ? 4 : 3;
      }
      // codes not kept: a later class may have the room
      if (W.result == 1 && P.want_cigar && !W.keep && L.my_class < L.route.nclass) W.result = 3;
      if (W.result == 3) {
        // on to a later class, with the extent the pair is predicted to need:
        // from the furthest anti-diagonal i + j any kept M offset reaches
        if (tid == 0) flag[3] = 0;
        __syncthreads();
        int32_t prog = 0;
        if (!out) {
          for (int32_t q = tid; q < R * NW; q += T) {
            const s16x2 v = as2(ring[q]);
            const int32_t k = 2 * (q % NW - NW / 2) - W.par;
            if (v.x >= 0) prog = max(prog, 2 * (v.x - BIAS) - k);
            if (v.y >= 0) prog = max(prog, 2 * (v.y - BIAS) - k - 1);
          }
          prog = wave_max_i32(prog);
          if ((tid & 63) == 0) atomicMax(&flag[3], prog);
        }
        __syncthreads();
        if (tid == 0)
          route_pair(O, L.route, L.my_class, p, predict_extent(out ? max(-kend, kend + 1) : s - P.o + 1, flag[3], m, n));
      } else {
        const bool walk = W.result == 1 && W.keep;
        if (walk) {
          if (tid == 0) pend[npend] = WideDone{(int32_t)p, s, code_at0, W.stage};
          ++npend;
          code_at0 += W.coff;
        } else if (W.result == 1 && P.want_cigar && tid == 0 && L.walk_skip) {
          atomicAdd(L.walk_skip, 1);  // codes not kept: the full-store pass walks it
        }
        if (tid == 0) {
          if (W.result == 2 || W.result == 4) {
            O.score[p] = -1;
            O.status[p] = W.result == 2 ? ST_REJECTED : ST_INVALID;
            O.nruns[p] = 0;
          } else {
            O.score[p] = s * P.unit;
            O.status[p] = ST_ALIGNED;
            if (!walk) O.nruns[p] = 0;
            if (P.want_cigar && !walk) to_full_store(O, L, p, s, m, n);
          }
        }
      }
    } else if (tid == 0) {
      O.score[p] = -1;
      O.status[p] = ST_INVALID;
      O.nruns[p] = 0;
    }
    __syncthreads();
    li = __builtin_amdgcn_readfirstlane(flag[2]);
  }
}

}  // namespace

size_t wfa_wide_lds(int32_t threads, int32_t words, int32_t R, int32_t seq_words) {
  return 4 * ((size_t)(R + 1) * threads * words + 2 * GUARD + 4 * (threads / 64 + 2) + 4 * (threads / 64) + 4) + 2 * (size_t)(seq_words + 2) * 8;
}

int64_t wfa_wide_pair_words(int32_t threads, int32_t words, int32_t o, int32_t scores) {
  int64_t w = 0;
  const int64_t rows = (int64_t)scores / 4 + 1;
  for (int32_t k = 1, from = 0; k <= words && from < rows; ++k) {
    const int64_t to = k < words ? std::min<int64_t>(rows, (stage_end(threads, k, o) + 1) / 4) : rows;
    w += (to - from) * threads * k;
    from = (int32_t)to;
  }
  return w;
}

hipError_t launch_wfa_wide(const Seqs &S, const Outs &O, const Scoring &P, const Work &Wk, const WfaWide &L, int32_t threads,
                           int32_t words, int32_t nslots, hipStream_t s) {
  const size_t lds = wfa_wide_lds(threads, words, L.R, L.seq_words);
  if (threads == 256 && words == 4)
    hipLaunchKernelGGL((k_wfa_wide<256, 4>), dim3(nslots), dim3(256), lds, s, S, O, P, Wk, L);
  else if (threads == 512 && words == 6)
    hipLaunchKernelGGL((k_wfa_wide<512, 6>), dim3(nslots), dim3(512), lds, s, S, O, P, Wk, L);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace aim
