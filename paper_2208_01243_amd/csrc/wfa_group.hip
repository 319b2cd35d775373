// Gap-affine wavefront alignment of pairs whose wavefronts are narrow, several
// pairs per 64-lane wavefront (k_wfa_group): the first pass of WFA and
// WFA-adaptive for unit gap extension (after the penalties' common divisor is
// taken out, as for 4/6/2 and edit distance).
//
// Paper: System and Methods, "Wavefront Algorithm (WFA)" (the recurrences of
// wfa.hip, restated there), its heuristic variant WFA-adaptive, and "Data
// Management" (the components a step needs stay in fast memory).
//
// What bounds it.  A score of a narrow pair is a few dozen cells: one pair
// per wavefront leaves most lanes idle and pays the step's scalar work and
// the pair's serial walk for itself alone.  (Before this kernel, 800,000
// pairs of 250 bp issued 7,500 vector and 8,700 scalar instructions a pair
// in the one-wavefront pass, and 1,000,000 adaptive pairs of 150 bp 3,200 and
// 3,500 for 91 cells; the scalar unit was busy 85 % of the time.)  So here
// - a group of G lanes holds one pair, C words of two diagonals a lane, and
//   64 / G pairs step together; everything that differs between pairs is a
//   lane value, so that a step has no scalar work per pair;
// - I and D of the last score stay in registers, M of the last R scores in a
//   ring of LDS words that only their own lane reads; the neighbouring
//   diagonals come from one lane rotate each of max(M, I) and max(M, D)
//   (the max commutes with the shift);
// - the sequences of a group's next pair are loaded while it works on this
//   one, and the queue's items are fetched up to 64 at a time;
// - the backtraces wait until up to 64 pairs have finished and then run one
//   pair per lane.
// Measured (this kernel's launches against the kernel before): 800,000 pairs of
// 250 bp 13.2 -> 5.8 ms, 1,000,000 adaptive pairs of 150 bp 12.7 -> 1.6, 100,000
// of 1 kbp 12.0 -> 3.2, 10,000 of 10 kbp 15.0 -> 6.7.  Vector instructions issue
// 65 to 85 % of the time, some 40 a score of a wavefront and over 100 with the
// reduction; 16 wavefronts per CU are best (12 and 20 to 24 a fifth slower, 32 no
// faster).
//
// Diagonals.  Word q holds diagonals 2q and 2q + 1 (low half first).  Exact
// WFA: lane l of a group holds words l C .. l C + C - 1 of a window of 2 G C
// diagonals around 0, and a pair leaves it (to the window classes, or to a
// wider group) at the first score whose wavefront could reach the window's
// edge, so no range is kept: a cell outside the wavefront computes as absent.
// WFA-adaptive: lane q mod G, with a window that follows the wavefront.
//
// Words start at diagonals of the end cell's parity, so that it lies in the
// low half of its word.
//
// Arithmetic.  Two diagonals per instruction in packed 16 bits (wfa_packed.h).
//
// Origin codes.  Four bits a cell: X < M, I < M (of the cell), and of the
// cell as a source, whether I, D were extended rather than opened from it
// (I of diagonal k - 1 and D of k + 1 read those).  The codes of four scores
// make one 32-bit word per word of diagonals, stored every fourth step of
// the wavefront at its step number: a ring of as_steps steps per wavefront,
// in which a pair owns the steps between its first and its last score.
#include "aim_internal.h"

namespace aim {
namespace {

#include "wfa_common.h"

#include "wfa_packed.h"

// The value of the next / previous lane of the group, round the group: lane
// rotates of the wavefront (64) or of the rows of 16; for groups of 32 the two
// rows' end lanes then change places.
template <int G, int WAVE, int ROW>
__device__ __forceinline__ uint32_t rotate_lane(uint32_t v, bool end) {
  if constexpr (G == 64) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, WAVE, 0xf, 0xf, true);
  const uint32_t r = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, ROW, 0xf, 0xf, true);
  if constexpr (G == 16) return r;
  // [0]: the even row of each pair in both rows, [1]: the odd row
  const auto w = __builtin_amdgcn_permlane16_swap(r, r, false, false);
  return end ? ((threadIdx.x & 16) ? w[0] : w[1]) : r;
}
template <int G>
__device__ __forceinline__ uint32_t next_lane(uint32_t v) {  // wave_rol:1, row_ror:15
  return rotate_lane<G, 0x134, 0x12f>(v, (threadIdx.x & 15) == 15);
}
template <int G>
__device__ __forceinline__ uint32_t prev_lane(uint32_t v) {  // wave_ror:1, row_ror:1
  return rotate_lane<G, 0x13c, 0x121>(v, (threadIdx.x & 15) == 0);
}

// Minimum of each half over the lanes of the group, in every lane.
template <int G>
__device__ __forceinline__ uint32_t group_min2(uint32_t v) {
  v = min2(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true));  // row_ror:8
  v = min2(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xf, 0xf, true));
  v = min2(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x122, 0xf, 0xf, true));
  v = min2(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x121, 0xf, 0xf, true));
  if constexpr (G >= 32) {
    const auto w = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min2(w[0], w[1]);
  }
  if constexpr (G >= 64) {
    const auto w = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = min2(w[0], w[1]);
  }
  return v;
}

constexpr int32_t IDLE = -1;
constexpr int32_t LOST = -2;  // (score limit) the adaptive window was outgrown

// The queue of a wavefront: items fetched together, in LDS.
struct QItem {
  int32_t p, mn;  // pair (IDLE: invalid input), lengths (pattern in the low half)
  int64_t po, to;
};
constexpr int32_t QUEUES = 64, QUEUE_STRIDE = 128;  // bytes between the queues' counters
constexpr int32_t LEAVE_AT = 16;
// A pair that goes on to another pass, and that pass's index in the route.
struct Leave {
  int32_t p, to;
};
// A finished pair that awaits its walk.
struct Done {
  int32_t p, t0, tf, g;
};

// The kernel's arguments as they lie in its argument segment.  The event code
// reads them from there when it runs: hoisted out of the score loop, as the
// compiler would have it, they do not fit the scalar registers.
typedef __attribute__((address_space(4))) const WfaGroupArgs *ArgsPtr;
__device__ __forceinline__ ArgsPtr group_args() {
  ArgsPtr a = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return a;
}

// The walk of one finished pair by one lane, over the codes kept by its
// wavefront (cleared of stale lines by the caller), then the forward replay.
template <int G, int C, bool ADAPT>
__device__ void walk_pair(ArgsPtr A, Done d, uint32_t *codes, int32_t rowmask) {
  const int64_t p = d.p;
  const int32_t m = A->S.pat_len[p], n = A->S.txt_len[p];
  const uint64_t *gP = A->S.pat + A->S.pat_off[p], *gT = A->S.txt + A->S.txt_off[p];
  const int64_t pnw = (m + 31) >> 5, tnw = (n + 31) >> 5;
  const int32_t x = A->P.x, oe = A->P.o + 1;
  uint32_t *cg = codes + d.g * (G * C);
  auto code_at = [&](int32_t tt, int32_t k) -> uint32_t {
    const int32_t kp = k + ((n - m) & 1);
    const int32_t w = ((kp >> 1) + (ADAPT ? 0 : G * C / 2)) & (G * C - 1);
    const uint32_t v = cg[((tt >> 2) & rowmask) * (64 * C) + w];
    return v >> (16 * (kp & 1) + 4 * (tt & 3));
  };
  // tokens, last op first, eight a word: the op, and 4 where a maximal run of
  // matches follows it in the alignment.  Words 0 and 1 stay in registers;
  // word w > 1 goes over codes of the pair's own last scores, which the walk
  // has passed: eight ops take at least eight scores
  uint32_t w0 = 0, w1 = 0, cur = 0;
  int32_t nt = 0, tt = d.tf, k = n - m, comp = 0;
  auto tok_at = [&](int32_t w) -> uint32_t & { return cg[(((d.tf >> 2) + 1 - w) & rowmask) * (64 * C)]; };
  bool ok = true;
  for (;;) {
    if (tt <= d.t0) {
      ok = tt == d.t0 && comp == 0 && k == 0;
      break;
    }
    uint32_t tok = 0;
    if (comp == 0) {
      const uint32_t v = code_at(tt, k);
      tok = TOK_M;
      comp = (v & 8u) ? ((v & 4u) ? OP_D : OP_I) : OP_X;
    }
    tok |= (uint32_t)comp;
    if (comp == OP_X) {
      tt -= x;
      comp = 0;
    } else {
      k += comp == OP_I ? 1 : -1;
      const uint32_t v = code_at(tt, k);
      const bool opened = !(v & (comp == OP_I ? 2u : 1u));
      tt -= opened ? oe : 1;
      if (opened) comp = 0;
    }
    cur |= tok << (4 * (nt & 7));
    if ((++nt & 7) == 0) {
      const int32_t w = (nt >> 3) - 1;
      if (w == 0) w0 = cur;
      else if (w == 1) w1 = cur;
      else tok_at(w) = cur;
      cur = 0;
    }
  }
  if (nt & 7) {
    const int32_t w = nt >> 3;
    if (w == 0) w0 = cur;
    else if (w == 1) w1 = cur;
    else tok_at(w) = cur;
  }
  // The forward replay, which meets the runs first op first: emit(r, run) for the
  // r-th, returns their number, -1 where it does not end at (m, n).
  auto replay = [&](auto emit) -> int32_t {
    int32_t nr = 0, left = nt;
    uint32_t rop = 0xffu, rlen = 0, word = 0;
    auto put = [&](uint32_t op, uint32_t len) {
      if (len == 0) return;
      if (op == rop) {
        rlen += len;
        return;
      }
      if (rlen) emit(nr, (rlen << 4) | rop);
      nr += rlen != 0;
      rop = op;
      rlen = len;
    };
    int32_t j = extend(gP, pnw, m, gT, tnw, n, 0, 0), i = j;
    put(OP_EQ, (uint32_t)j);
    while (left > 0) {
      if ((left & 7) == 0 || left == nt) {
        const int32_t w = (left - 1) >> 3;
        word = w == 0 ? w0 : w == 1 ? w1 : tok_at(w);
      }
      --left;
      const uint32_t tok = word >> (4 * (left & 7));
      const uint32_t op = tok & 3u;
      i += op != OP_D;
      j += op != OP_I;
      put(op, 1u);
      if (tok & TOK_M) {
        const int32_t f = extend(gP, pnw, m, gT, tnw, n, j - i, j);
        put(OP_EQ, (uint32_t)(f - j));
        i += f - j;
        j = f;
      }
    }
    if (rlen) emit(nr, (rlen << 4) | rop);
    nr += rlen != 0;
    return i == m && j == n ? nr : -1;
  };
  // The runs go to the end of the pair's slot, or of a reservation in the pool,
  // backwards, so that they lie there last op first, as every pass leaves them.
  // The reservation is for all that there can be, two a token and one, where that
  // is within the pair's share of the pool or the pool less than half used.  Where
  // it is not, and the runs pass the slot, a second replay lays them out the usual
  // way: the last slot_cap in the slot, the others in a reservation of their
  // number.  (With the first kind alone 10,000 unrelated pairs of 250 bp, about 170
  // runs each in a pool of 125 a pair, used that up at 261 a pair, and half were
  // re-run in place: 956 ms instead of 2; with the second for every pair past its
  // share 4,000 adaptive pairs of 10 kbp at 10 % took 8.0 ms instead of 7.1.)
  int32_t room = A->O.slot_cap;
  uint32_t *end = A->O.slot + (p + 1) * (int64_t)room;
  if (const int32_t bound = 2 * nt + 1; bound > room) {
    const int64_t pool_cap = A->O.pool_cap;
    if (bound <= A->L.pool_share || (int64_t)*(volatile unsigned long long *)A->O.pool_top + bound <= pool_cap / 2) {
      const int64_t at = (int64_t)atomicAdd(A->O.pool_top, (unsigned long long)bound);
      if (at + bound <= pool_cap) {
        end = A->O.pool + at + bound;
        room = bound;
      }
    }
  }
  const int32_t nr = ok ? replay([&](int32_t r, uint32_t run) { if (r < room) end[-1 - r] = run; }) : -1;
  if (nr > room) {
    const int32_t need = nr - room;  // (room: the slot's)
    const int64_t at = (int64_t)atomicAdd(A->O.pool_top, (unsigned long long)need);
    const bool fits = at + need <= A->O.pool_cap;
    A->O.nruns[p] = nr;
    A->O.pool_off[p] = fits ? at : -2;  // (-2: re-run in place by the compaction)
    if (fits)
      replay([&](int32_t r, uint32_t run) {
        const int32_t k = nr - 1 - r, cap = A->O.slot_cap;
        (k < cap ? A->O.slot + p * (int64_t)cap : A->O.pool + A->O.pool_off[p] - cap)[k] = run;
      });
    return;
  }
  if (nr >= 0) {
    A->O.nruns[p] = nr;
    A->O.pool_off[p] = room == A->O.slot_cap ? POOL_OFF_TAIL : (POOL_OFF_WHOLE | (end - A->O.pool)) - nr;
    return;
  }
  // cannot happen for codes that were kept and read back intact
  A->O.nruns[p] = 0;
  if (A->L.walk_fail) atomicAdd(A->L.walk_fail, 1);
  if (ADAPT || !A->L.need) {
    A->O.status[p] = ST_OVERFLOW;  // no exact fallback for a heuristic alignment, or none planned
    return;
  }
  const int64_t sc = d.tf - d.t0;
  const int64_t need = (sc + 1) * (ENTRY + (3 * (2 * sc + 3) + 1) / 2);
  A->L.need[p] = need;
  int cl = 0;
  while (cl < 3 && need > A->L.need_cap[cl]) ++cl;
  if (need > A->L.need_cap[3]) {
    if (A->L.long_list) A->L.long_list[atomicAdd(A->L.long_count, 1)] = (int32_t)p;
    else A->O.status[p] = ST_OVERFLOW;
  } else {
    A->L.need_list[cl][atomicAdd(A->L.need_count[cl], 1)] = (int32_t)p;
    atomicMax(A->L.need_max[cl], (int32_t)need);
  }
}

template <int G, int C, bool ADAPT>
__global__ __launch_bounds__(64, C == 4 ? 3 : 4) void k_wfa_group(WfaGroupArgs arg) {
  static_assert(!ADAPT || C == 1, "the adaptive window holds one word a lane");
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NG = 64 / G;
  constexpr int HALF = G * C;      // diagonals each side of 0 (exact)
  constexpr int REACH = HALF - 3;  // the furthest a wavefront may use of them
  // ended pairs that are worth the event code: two of four short reads'
  constexpr int32_t EVENT_GROUPS = NG == 4 ? 2 : 1;
  const int lane = threadIdx.x, gl = lane & (G - 1), gi = lane / G;
  const int32_t x = arg.P.x, oe = arg.P.o + 1, R = arg.L.R;
  const int32_t SW = arg.L.seq_words + 2;  // staged words per sequence, one of padding at each end
  Done *done = (Done *)smem;               // 64
  QItem *queue = (QItem *)(done + 64);     // 64
  Leave *leave = (Leave *)(queue + 64);    // LEAVE_AT
  uint64_t *seqs = (uint64_t *)(leave + LEAVE_AT);
  uint64_t *sP = seqs + (int64_t)gi * 2 * SW, *sT = sP + SW;
  // (opaque: one register each, not sums of what they are made of)
  uint32_t pw = lds_addr(sP), tw = lds_addr(sT);
  asm("" : "+v"(pw));
  asm("" : "+v"(tw));
  if (gl == 0) {
    sP[0] = 0ull;
    sT[0] = ENDS_T;
  }
  uint32_t *ring = reinterpret_cast<uint32_t *>(seqs + (int64_t)NG * 2 * SW);  // R rows of 64 C words
  uint32_t *rrow = ring + R * 64 * C;  // (adaptive) the range of each row, R rows of 64 words
  int32_t count;
  {
    ArgsPtr a = group_args();
    count = a->Wk.count ? __builtin_amdgcn_readfirstlane(*(volatile const int32_t *)a->Wk.count) : (int32_t)a->Wk.n;
  }
  // a workgroup the work can never reach leaves before touching the counter
  if ((int32_t)blockIdx.x >= count) return;
  // The work lies in up to 64 queues (item li in queue li mod nq), each with a
  // counter in a cache line of its own and a 64th of the wavefronts: up to
  // half of a wavefront's share is its own from the start, the rest comes
  // from its queue's counter, an eighth of a share at a time.  (Wavefronts
  // adding to one address take about 10 ns each, on the chip as a whole: one
  // counter made 65,536 pairs of 100 bp cost 0.64 ms, at any error rate.)
  const int32_t grid = (int32_t)gridDim.x, nq = min(grid, QUEUES), qi = (int32_t)blockIdx.x % nq;
  const int32_t qwaves = (grid - qi + nq - 1) / nq, qrank = (int32_t)blockIdx.x / nq;
  const int32_t own = max(NG, min(64, count / (2 * grid))), chunk = max(NG, min(64, count / (8 * grid)));
  const bool keep = arg.P.want_cigar != 0;
  uint32_t *codes = arg.L.codes + (int64_t)blockIdx.x * arg.L.slot_words;  // [as_steps / 4][64 C]
  const int32_t as_steps = arg.L.as_steps, rowmask = as_steps / 4 - 1;

  // the pair of this lane's group (every lane of the group holds the same)
  int32_t gp = IDLE, gm = 0, gn = 0, gt0 = 0, gslim = INT32_MAX, gdrop = 0;
  int32_t gtf = -1;  // its last score's step, once it has reached the end cell
  // words of this lane: source components of the last score, codes
  // of the running four scores, diagonals, table bounds, the end cell's
  // offset on the word that has it
  uint32_t Iv[C], Dv[C], cacc[C], K2[C], LIM[C], TGT[C];
  uint32_t DK = 0;                            // (adaptive) max(m + k, n) per half
  uint32_t rng = 0x7fff7fffu;                 // (adaptive) last score's range as (lo, -hi)
  uint32_t wlim = 0x80008000u;                // (adaptive) least (lo, -hi) the window takes
#pragma unroll
  for (int c = 0; c < C; ++c) {
    Iv[c] = Dv[c] = ABSENT2;
    cacc[c] = K2[c] = 0;
    LIM[c] = 0xffffffffu;  // idle: every offset is cut
    TGT[c] = 0x7fff;
  }
  for (int32_t r = 0; r < R; ++r) {
#pragma unroll
    for (int c = 0; c < C; ++c) ring[(r * 64 + lane) * C + c] = ABSENT2;
    if (ADAPT) rrow[r * 64 + lane] = 0x7fff7fffu;
  }
  const int32_t ad_min = arg.L.ad_min, ad_max = min(arg.L.ad_max, 0x7fff);
  uint64_t q_mask = 0;  // queue items not yet taken
  bool q_end = false, q_own = true;
  // the group's next pair and this lane's word of each of its sequences
  int32_t x_p = IDLE, x_mn = 0;
  uint64_t x_P = 0, x_T = 0;
  int32_t nf = 0, nl = 0;  // finished pairs in `done`, leaving ones in `leave`
  uint32_t dropped = 0, dropped_hi = 0;

  int32_t t = 0;  // step
  // ring rows (offsets in words) of this step, and of the two sources
  constexpr int32_t ROW = 64 * C;
  const int32_t rend = R * ROW;
  int32_t rowW = 0, rowX = (R - x) * ROW, rowO = (R - oe) * ROW;
  int32_t next_event = 0;   // step after which the event code runs
  int32_t tkeep = 0;        // first step whose codes are still needed
  bool hit = false;         // this lane's word reached the end cell
  int32_t nact = 0, npend = 0;  // groups with a pair, and those whose pair has ended
  bool first = true;

  auto set_word = [&](int c, int32_t q) {
    const int32_t kend = gn - gm, k = 2 * q - (kend & 1);
    K2[c] = pack2(k, k + 1);
    const uint32_t mk = add2(both(gm + BIAS), K2[c]), nn = both(gn + BIAS);
    LIM[c] = min2(mk, nn);
    TGT[c] = (uint32_t)(k == kend ? gn + BIAS : 0x7fff);
    if (ADAPT) DK = max2(mk, nn);
  };
  // the end of a pair: nothing it held is live any more
  auto clear_group = [&]() {
    gslim = INT32_MAX;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      LIM[c] = 0xffffffffu;
      TGT[c] = 0x7fff;
    }
    rng = 0x7fff7fffu;
    wlim = 0x80008000u;
  };
  // (adaptive) diagonals dropped of a pair that ends here, whatever its outcome
  auto count_dropped = [&]() {
    if (!ADAPT) return;
    dropped += (uint32_t)gdrop;
    dropped_hi += dropped < (uint32_t)gdrop;
  };
  // the cost of one concrete alignment bounds the optimum: all diagonal ops
  // plus one gap run for the length difference, or gap runs over both
  auto upper = [&](int32_t o) {
    const int32_t ad = gm > gn ? gm - gn : gn - gm;
    return min(x * min(gm, gn) + (ad ? o + ad : 0), (gm ? o + gm : 0) + (gn ? o + gn : 0));
  };

  for (;;) {
    // ------------------------------------------------------------- events
    // a group whose pair has reached its end cell waits until enough others
    // have (the code below costs about as much as several scores)
    if (__ballot(hit)) {
      const uint64_t hits = __ballot(hit);
      const uint64_t gmask = G == 64 ? ~0ull : (((1ull << (G & 63)) - 1ull) << (gi * G));
      const bool ends = (hits & gmask) != 0;
      if (ends) {
        gtf = t;
        hit = false;
        clear_group();
      }
      npend += (int32_t)__popcll(__ballot(ends && gl == 0));
    }
    bool again = t >= next_event || npend >= min(EVENT_GROUPS, nact);
    while (uniform(again)) {
      ArgsPtr A = group_args();
      {
        const bool ghit = gtf >= 0;
        const int32_t s = (ghit ? gtf : t) - gt0;
        const bool live = gp >= 0;
        // the ring of codes is full: the pairs that started first end here
        const bool full = live && keep && s >= as_steps - 8;
        const bool over = live && !ghit && (s >= gslim || full);
        const bool fin = live && (ghit || over);
        if (__ballot(over)) {
          // past the pair's last score: rejected, or on to the next pass
          const int32_t smax = A->P.max_score;
          const bool lost = ADAPT && gslim == LOST;
          // (a length difference alone may pass the threshold: before any score)
          const int32_t ad = gm > gn ? gm - gn : gn - gm;
          const bool rej = !lost && smax >= 0 && (s + 1 > smax || (ad > 0 && A->P.o + ad > smax));
          const bool bad = !lost && s + 1 > upper(A->P.o);  // cannot happen for exact WFA
          // (and no plan lets a pair leave the last pass)
          const bool ends = rej || bad || (ADAPT && !lost && s >= A->L.s_cap) || A->L.my_class >= A->L.route.nclass;
          const bool on = over && !ends;
          if (over && ends && gl == 0) {
            A->O.score[gp] = -1;
            A->O.status[gp] = rej ? ST_REJECTED : ST_INVALID;
            A->O.nruns[gp] = 0;
            count_dropped();
          }
          if (__ballot(on)) {
            int32_t to = 1;
            if (!ADAPT) {
              // the furthest anti-diagonal any kept M offset reaches, for
              // the prediction of the window the pair needs
              int32_t prog = 0;
              for (int32_t r = 0; r < R; ++r) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                  const s16x2 v = as2(ring[(r * 64 + lane) * C + c]), k = as2(K2[c]);
                  if (v.x >= 0) prog = max(prog, 2 * (v.x - BIAS) - k.x);
                  if (v.y >= 0) prog = max(prog, 2 * (v.y - BIAS) - k.y);
                }
              }
              for (int d = 1; d < G; d <<= 1) prog = max(prog, __shfl_xor(prog, d));
              const int32_t kend = gn - gm;
              const bool out = kend < -REACH || kend > REACH;  // left before any score
              if (on && gl == 0) {
                const int32_t pred = predict_extent(out ? max(-kend, kend + 1) : REACH + 1, out ? 0 : prog, gm, gn);
                to = A->L.my_class + 1;
                while (to < A->L.route.nclass && A->L.route.half[to] < pred) ++to;
                A->L.route.pred[gp] = pred;
              }
            }
            const uint64_t going = __ballot(on && gl == 0);
            if (on && gl == 0) leave[nl + (int32_t)__popcll(going & ((1ull << lane) - 1ull))] = Leave{gp, to};
            nl += (int32_t)__popcll(going);
          }
        }
        if (fin && ghit && gl == 0) {
          A->O.score[gp] = s * A->P.unit;
          A->O.status[gp] = ST_ALIGNED;
          if (!keep) A->O.nruns[gp] = 0;
          count_dropped();
        }
        if (keep) {
          // one entry per finished pair, in the order of the groups
          const uint64_t ended = __ballot(fin && ghit && gl == 0);
          if (ended) {
            if (fin && ghit && gl == 0)
              done[nf + (int32_t)__popcll(ended & ((1ull << lane) - 1ull))] = Done{gp, gt0, gtf, gi};
            nf += (int32_t)__popcll(ended);
          }
        }
        if (fin) {
          gp = IDLE;
          gtf = -1;
          clear_group();
        }
      }
      // ---- idle groups take their next pair, and load the one after it
      again = false;
      const uint64_t want = __ballot(gp < 0 && gl == 0);
      // (the first time there is no next pair yet)
      for (int rd = first ? 0 : 1; rd < 2; ++rd) {
        const bool start = gp < 0 && x_p >= 0;
        if (__ballot(start)) {
          if (start) {
            gp = x_p;
            gm = x_mn & 0xffff;
            gn = (x_mn >> 16) & 0xffff;
            gt0 = t;
            gdrop = 0;
            const int32_t pnw = (gm + 31) >> 5, tnw = (gn + 31) >> 5;
            if (gl <= pnw) sP[gl + 1] = upto(x_P, gm - 32 * gl, 0ull);
            if (gl <= tnw) sT[gl + 1] = upto(x_T, gn - 32 * gl, ENDS_T);
            if (max(pnw, tnw) >= G) {
              const uint64_t *gP = A->S.pat + A->S.pat_off[gp], *gT = A->S.txt + A->S.txt_off[gp];
              for (int32_t q = gl + G; q <= pnw; q += G) sP[q + 1] = upto(q < pnw ? gP[q] : 0ull, gm - 32 * q, 0ull);
              for (int32_t q = gl + G; q <= tnw; q += G) sT[q + 1] = upto(q < tnw ? gT[q] : 0ull, gn - 32 * q, ENDS_T);
            }
          }
          __syncthreads();  // (one wavefront) staged words before the reads of other lanes
          if (start) {
            const int32_t o = A->P.o, smax = A->P.max_score, kend = gn - gm;
            int32_t lim = min(upper(o), A->L.s_cap);
            if (smax >= 0) lim = min(lim, smax);
            if (smax >= 0 && kend != 0 && o + (kend < 0 ? -kend : kend) > smax) lim = -1;
            if (!ADAPT && max(gm, gn) > REACH)
              // a wavefront of score s reaches diagonals -(s - o) .. s - o
              lim = (kend < -REACH || kend > REACH) ? -1 : min(lim, REACH + o);  // (-1 stays)
            gslim = lim;
            const int32_t f0 = match_run(pw, tw, BIAS, BIAS, min(gm, gn));
            for (int32_t r = 0; r < R; ++r) {
#pragma unroll
              for (int c = 0; c < C; ++c) ring[(r * 64 + lane) * C + c] = ABSENT2;
              if (ADAPT) rrow[r * 64 + lane] = 0x7fff7fffu;
            }
            if (ADAPT) {
              const int32_t ub = -(G / 2);
              set_word(0, ub + ((gl - ub) & (G - 1)));
              wlim = pack2(2 * ub + 1 - (kend & 1), -(2 * ub + 2 * G - 2 - (kend & 1)));
              rng = 0x7fff7fffu;  // I and D of score 0 are absent: no source of score 1
              rrow[rowW + lane] = 0u;
            } else {
#pragma unroll
              for (int c = 0; c < C; ++c) set_word(c, gl * C + c - HALF / 2);
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
              Iv[c] = Dv[c] = ABSENT2;
              // the word of diagonal 0, of the pair's score 0
              if (K2[c] == 0x00010000u) ring[rowW + lane * C + c] = (uint32_t)(f0 + BIAS) | 0x80000000u;
              if (K2[c] == 0x0000ffffu) ring[rowW + lane * C + c] = (uint32_t)(f0 + BIAS) << 16 | 0x8000u;
            }
            if (kend == 0 && f0 >= gn) {
              gtf = t;
              clear_group();
            }
          }
          // (a pair that is equal to its text, or has no score to try, ends at once)
          again = __ballot(start && (gtf >= 0 || gslim <= 0)) != 0;
        }
        // the next pair of every group that has just taken one
        uint64_t todo = first || !q_end || q_mask ? want : 0ull;
        if (start) x_p = IDLE;
        while (todo) {
          const int g = (int)__builtin_ctzll(todo) / G;
          todo &= todo - 1;
          while (!q_mask && !q_end) {
            int32_t base = 0;
            if (!q_own) {
              if (lane == 0) base = atomicAdd(A->Wk.counter + qi * (QUEUE_STRIDE / 4), chunk);
              base = __builtin_amdgcn_readfirstlane(base) + own * qwaves;
            }
            const int32_t qn = (count - qi + nq - 1) / nq;  // items of this queue
            const int32_t li = qi + nq * (q_own ? lane * qwaves + qrank : base + lane);
            const int32_t cnt = q_own ? own : min(chunk, qn - base);
            // (the last fetch, when nothing is left to the counter)
            q_end = q_own ? own * qwaves >= qn : cnt <= 0;
            q_own = false;
            if (cnt > 0) {
              bool valid = false;
              if (lane < cnt && li < count) {
                const int32_t p = A->Wk.idx ? A->Wk.idx[li] : li;
                if (A->O.flags && A->O.flags[p]) {
                  A->O.score[p] = -1;
                  A->O.status[p] = ST_INVALID;
                  A->O.nruns[p] = 0;
                } else {
                  valid = true;
                  queue[lane] = QItem{p, A->S.pat_len[p] | (A->S.txt_len[p] << 16), A->S.pat_off[p], A->S.txt_off[p]};
                }
              }
              q_mask = __ballot(valid);
              __syncthreads();
            }
          }
          if (!q_mask) break;
          const int j = (int)__builtin_ctzll(q_mask);
          q_mask &= q_mask - 1;
          if (gi == g) {
            const QItem it = queue[j];
            x_p = it.p;
            x_mn = it.mn;
            x_P = x_T = 0;
            if (gl < (((it.mn & 0xffff) + 31) >> 5)) x_P = A->S.pat[it.po + gl];
            if (gl < ((((it.mn >> 16) & 0xffff) + 31) >> 5)) x_T = A->S.txt[it.to + gl];
          }
        }
        first = false;
      }
      // ---- the walks of the finished pairs
      const uint64_t busy = __ballot(gp >= 0);
      int32_t tmin = t;  // the first step a running pair needs
      {
        int32_t v = gp >= 0 ? gt0 : t;
#pragma unroll
        for (int g = 0; g < NG; ++g) tmin = min(tmin, __builtin_amdgcn_readlane(v, g * G));
      }
      if (nf > 0 && (nf > 64 - NG || !busy || t - tkeep >= as_steps - 8)) {
        // the codes of the running four scores, then every store before the
        // loads; the acquire drops lines that an earlier walk left in the
        // CU's vector L1
        if ((t & 3) != 3) {
#pragma unroll
          for (int c = 0; c < C; ++c)
            codes[((t >> 2) & rowmask) * (64 * C) + lane * C + c] = settle_codes(cacc[c], t);
        }
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (lane < nf) walk_pair<G, C, ADAPT>(A, done[lane], codes, rowmask);
        __syncthreads();
        nf = 0;
      }
      nact = (int32_t)__popcll(__ballot(gp >= 0 && gl == 0));
      npend = 0;
      if (nl > (A->L.by_length ? 0 : LEAVE_AT - NG) || (nl > 0 && !busy)) {
        // the leaving pairs to their lists, one atomic per list; at once where
        // lengths spread widely, so that the lists keep the queue's order,
        // longest first (buffered, 200,000 pairs of 100-10,000 bp lost 7 % to the
        // class kernels' last pairs)
        __syncthreads();
        const Leave v = lane < nl ? leave[lane] : Leave{IDLE, 0};
        for (int32_t c = A->L.my_class + 1; c <= A->L.route.nclass; ++c) {
          const uint64_t m = __ballot(v.to == c);
          if (!m) continue;
          int32_t at = 0;
          if (lane == 0) at = atomicAdd(A->L.route.count[c], (int32_t)__popcll(m));
          at = __builtin_amdgcn_readfirstlane(at) + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
          if (v.to == c) A->L.route.list[c][at] = v.p;
        }
        __syncthreads();
        nl = 0;
      }
      if (!busy) {
        if (ADAPT && A->L.ad_dropped && (dropped | dropped_hi))
          atomicAdd(A->L.ad_dropped, ((unsigned long long)dropped_hi << 32) | dropped);
        return;
      }
      if (nf == 0) tkeep = tmin;
      // the next event: the first pair to run out of scores, or the ring of
      // codes coming full
      next_event = keep ? tkeep + as_steps - 8 : INT32_MAX;
      {
        const int32_t v = gp >= 0 && gslim < INT32_MAX - t ? gt0 + gslim : INT32_MAX;
#pragma unroll
        for (int g = 0; g < NG; ++g) next_event = min(next_event, __builtin_amdgcn_readlane(v, g * G));
      }
    }
    if (nact == 0) continue;
    do {
    // --------------------------------------------------------------- a score
    ++t;
    rowW = rowW + ROW == rend ? 0 : rowW + ROW;
    rowX = rowX + ROW == rend ? 0 : rowX + ROW;
    rowO = rowO + ROW == rend ? 0 : rowO + ROW;
    if constexpr (ADAPT) {
      // the range over the sources, one wider at each end, inside [-m, n] (an
      // empty one stays empty: lo + (-hi) > 0)
      rng = min2(min2(rrow[rowX + lane], rrow[rowO + lane]), rng);
      rng = max2(add2(rng, 0xffffffffu), pack2(-gm, -gn));
      // the window follows the range (a pair whose recent wavefronts outgrow
      // it goes on to the next pass)
      const uint32_t under = subs2(rng, wlim) & 0x80008000u;
      if (__ballot(under != 0u)) {
        if (under != 0u) {
          uint32_t u = rng;
          for (int32_t r = 0; r < R; ++r) u = min2(u, rrow[r * ROW + lane]);  // (the oldest too: over-covers)
          const int32_t ulo = as2(u).x, uhi = -as2(u).y, par = (gn - gm) & 1;
          const int32_t ub = ((ulo + uhi) >> 2) - G / 2;
          if (ulo >= 2 * ub + 1 - par && uhi <= 2 * ub + 2 * G - 2 - par) {
            const int32_t q = ub + ((gl - ub) & (G - 1));
            if ((K2[0] & 0xffffu) != ((uint32_t)(2 * q - par) & 0xffffu)) {
              // a word new to this lane: outside every recent range
              Iv[0] = Dv[0] = ABSENT2;
              for (int32_t r = 0; r < R; ++r) ring[r * ROW + lane] = ABSENT2;
              set_word(0, q);
            }
            wlim = pack2(2 * ub + 1 - par, -(2 * ub + 2 * G - 2 - par));
          } else {
            // the group ends here: an event after this step, whose cells are
            // of no use to it
            clear_group();
            gslim = LOST;
          }
        }
        if (__ballot(gslim == LOST)) next_event = t;
      }
    }
    uint32_t Mo[C], A[C], B[C], Mx[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      Mo[c] = ring[rowO + lane * C + c];
      Mx[c] = ring[rowX + lane * C + c];
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
      A[c] = max2(Mo[c], Iv[c]);
      B[c] = max2(Mo[c], Dv[c]);
    }
    const uint32_t An = next_lane<G>(A[0]), Bp = prev_lane<G>(B[C - 1]);
    uint32_t F[C], Mv[C], rr[C];
    uint32_t full = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const uint32_t up = c + 1 < C ? A[c + 1 < C ? c + 1 : 0] : An, dn = c > 0 ? B[c > 0 ? c - 1 : 0] : Bp;
      const uint32_t I = cut2(__builtin_amdgcn_alignbit(up, A[c], 16), LIM[c]);
      const uint32_t D = cut2(add2(__builtin_amdgcn_alignbit(B[c], dn, 16), 0x00010001u), LIM[c]);
      const uint32_t X = cut2(add2(Mx[c], 0x00010001u), LIM[c]);
      const uint32_t ID = max2(I, D);
      Mv[c] = max2(X, ID);
      // extension: the first 16 bases of both diagonals by every lane
      rr[c] = first_run2(pw, tw, Mv[c], K2[c]);
      if (keep) cacc[c] = push_codes(cacc[c], subs2(X, ID), subs2(I, D), subs2(Mo[c], Iv[c]), subs2(Mo[c], Dv[c]));
      Iv[c] = I;
      Dv[c] = D;
      // (a run of 16 is done again below)
      F[c] = min2(add2(Mv[c], rr[c]), LIM[c]);
      full |= rr[c];
    }
    if (full & 0x40004000u) {
#pragma unroll
      for (int c = 0; c < C; ++c) F[c] = long_runs2(pw, tw, Mv[c], K2[c], LIM[c], rr[c], F[c]);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) hit = (c > 0 && hit) || (int16_t)F[c] >= (int16_t)TGT[c];
    if constexpr (ADAPT) {
      // the reduction: from the distance max(m - i, n - j) of each offset
      const s16x2 rv = as2(rng);
      bool red = 1 - (int32_t)rv.x - (int32_t)rv.y >= ad_min;
      if (const uint64_t hits = __ballot(hit)) {
        const uint64_t gmask = G == 64 ? ~0ull : (((1ull << (G & 63)) - 1ull) << (gi * G));
        red = red && !(hits & gmask);
      }
      if (__ballot(red)) {
        const uint32_t dist = subs2(DK, F[0]) | (sign2(F[0]) & 0x7fff7fffu);
        const uint32_t dm = group_min2<G>(min2(dist, __builtin_amdgcn_alignbit(dist, dist, 16)));
        const uint32_t thr = as1(__builtin_elementwise_add_sat(as2(dm), as2(both(ad_max))));
        const uint32_t drop = sign2(subs2(thr, dist) | F[0]);
        // the least k and the least -k of the kept diagonals (a dropped one
        // counts as 0x7fff)
        const uint32_t nk = sub2(0u, K2[0]);
        const uint32_t a = bfi_v(drop, 0x7fff7fffu, K2[0]), b = bfi_v(drop, 0x7fff7fffu, nk);
        const uint32_t ends = group_min2<G>(min2(__builtin_amdgcn_perm(b, a, 0x05040100u), __builtin_amdgcn_perm(b, a, 0x07060302u)));
        if (red && (dm & 0xffffu) != 0x7fffu) {
          const uint32_t d = sub2(ends, rng);
          gdrop += (int32_t)(d & 0xffffu) + (int32_t)(d >> 16);
          rng = ends;
          const uint32_t lo2 = __builtin_amdgcn_perm(ends, ends, 0x01000100u), nhi2 = __builtin_amdgcn_perm(ends, ends, 0x03020302u);
          const uint32_t bad = (sub2(K2[0], lo2) | sub2(nk, nhi2)) & 0x80008000u;
          F[0] |= bad;
          Iv[0] |= bad;
          Dv[0] |= bad;
        }
      }
      rrow[rowW + lane] = rng;
    }
#pragma unroll
    for (int c = 0; c < C; ++c) ring[rowW + lane * C + c] = F[c];
    if (keep && (t & 3) == 3) {
#pragma unroll
      for (int c = 0; c < C; ++c) codes[((t >> 2) & rowmask) * (64 * C) + lane * C + c] = cacc[c];
    }
    } while (uniform(t < next_event && !__ballot(hit)));
  }
}

template <int G, int C, bool ADAPT>
hipError_t launch_group(const Seqs &S, const Outs &O, const Scoring &P, const Work &Wk, const WfaGroup &L,
                        hipStream_t s) {
  hipLaunchKernelGGL((k_wfa_group<G, C, ADAPT>), dim3(L.nslots), dim3(64),
                     wfa_group_lds(G, C, ADAPT, L.R, L.seq_words), s, WfaGroupArgs{S, O, P, Wk, L});
  return hipGetLastError();
}

}  // namespace

size_t wfa_group_lds(int32_t lanes, int32_t words, bool adaptive, int32_t R, int32_t seq_words) {
  return 64 * (sizeof(Done) + sizeof(QItem)) + LEAVE_AT * sizeof(Leave) +
         (size_t)(64 / lanes) * 2 * (seq_words + 2) * 8 + (size_t)R * 64 * 4 * (words + (adaptive ? 1 : 0));
}

hipError_t launch_wfa_group(const Seqs &S, const Outs &O, const Scoring &P, const Work &Wk, const WfaGroup &L,
                            int32_t lanes, int32_t words, bool adaptive, hipStream_t s) {
  if (adaptive) {
    if (words != 1) return hipErrorInvalidValue;
    if (lanes == 16) return launch_group<16, 1, true>(S, O, P, Wk, L, s);
    if (lanes == 32) return launch_group<32, 1, true>(S, O, P, Wk, L, s);
    if (lanes == 64) return launch_group<64, 1, true>(S, O, P, Wk, L, s);
    return hipErrorInvalidValue;
  }
  if (words == 1 && lanes == 16) return launch_group<16, 1, false>(S, O, P, Wk, L, s);
  if (words == 1 && lanes == 32) return launch_group<32, 1, false>(S, O, P, Wk, L, s);
  if (words == 1 && lanes == 64) return launch_group<64, 1, false>(S, O, P, Wk, L, s);
  if (words == 2 && lanes == 64) return launch_group<64, 2, false>(S, O, P, Wk, L, s);
  if (words == 4 && lanes == 64) return launch_group<64, 4, false>(S, O, P, Wk, L, s);
  return hipErrorInvalidValue;
}

}  // namespace aim
