// GenASM: windowed bitap distance calculation with a traceback, one pair
// per lane.
//
// Paper, System and Methods, "GenASM": bitap extended with a traceback, a
// bound k on the edits, and per thread a bit-mask of the pattern per
// character, two status bit-vectors and four intermediate bit-vectors (match,
// substitution, deletion, insertion).  The library's reading (unit edits,
// windows of 64 bases with an overlap of 24, the traceback's order, the
// threshold) is the following:
//
// The pair is aligned from its end towards its start in windows of at most
// 64 pattern and 64 text bases, taken from the end of the bases still to
// align (me pattern, ne text bases).  The final window (me, ne <= 64) starts
// at the start of both sequences; any other may start anywhere on its first
// row or column.  With D(i, j) the fewest edits aligning the window's first
// i pattern and j text bases, the status vector of text position j at level
// d holds bit i - 1 = [D(i, j) <= d] for i = 1..a; the start row D(0, j) is
// implicit.  Level d at position j follows from level d at j - 1 and level
// d - 1 at j - 1 and j:
//   match        = ((R_d[j-1] << 1) | [D(0, j-1) <= d]) & PM[t_j]
//   substitution =  (R_{d-1}[j-1] << 1) | [D(0, j-1) <= d-1]
//   insertion    =  (R_{d-1}[j] << 1)   | [D(0, j) <= d-1]
//   deletion     =   R_{d-1}[j-1]
// The window's distance is the least d whose vector at j = b has bit a - 1
// set, searched up to max(a, b) (and the edits k still allows).  The
// traceback walks from (a, b) back with that budget and takes the first of:
// the previous op again if it was a gap ('I' / 'D') and still within budget;
// '='; 'X'; 'I'; 'D'.  A window other than the final commits ops until 40
// bases of either sequence are consumed or its first row or column is
// reached.  When either sequence runs out, the rest of the other is one gap.
// The score is the number of edits; more than k rejects the pair.
//
// MI355X mapping.  A lane owns a pair.  No level is built: the traceback only
// visits cells whose distance equals the edits it has left (it starts at the
// window's distance and every op keeps to an optimal continuation), and there
// the status bits it tests are the differences to the three neighbouring cells,
//   [D(i-1, j)   <= d-1]  =  vertical difference +1 at (i, j),
//   [D(i, j-1)   <= d-1]  =  horizontal difference +1,
//   [D(i-1, j-1) <= d-1]  =  diagonal difference not 0,
// which Myers' recurrence for the window's distance has in registers at every
// text position.  They are kept in LDS, as slices around the window's end
// diagonal: 8 bytes a position where no window of the wavefront has a distance
// above 10, else 12 (up to 15) or the whole vectors.  20 KiB a wavefront, two
// wavefronts a SIMD: the 40 positions that a window other than the final one is
// walked over, of the slices of 8 bytes; where a walk needs more positions than
// are kept, it goes on after another pass over the text up to those.  The
// traceback takes a run of matching bases at once and reads one entry per edit,
// all lanes together.  Work comes 64 pairs at a time.
//
// What bounds it: vector instructions (two thirds of their issue rate: 34 a text
// position, of which 10 keep the differences, and about 100 an edit).  1,000,000
// pairs of 150 bp at 4 %: 490 us; 684 with every pass's positions conditional and
// an op's run emitted in each branch of the walk; 806 with 12-byte slices in
// global memory, whose stores bound it (four wavefronts a SIMD, more were
// slower); 2,072 with sweeps that built six levels of status vectors each and
// stored them for the traceback.
#include "aim_internal.h"
#include "dev_util.h"

namespace aim {
namespace {

constexpr int32_t GW = 64;       // window bases
constexpr int32_t GC = GW - 24;  // bases a window other than the final one commits
constexpr int32_t GC_FROM = GW - GC;  // first text position whose differences the walk of a full window needs, less one
constexpr uint32_t OP_NONE = 4;

__device__ __forceinline__ uint64_t low_bits(int32_t q) {
  return q >= 64 ? ~0ull : (q <= 0 ? 0ull : ((1ull << q) - 1ull));
}

// The differences of a text position, 64 lanes' entries: three slices of 21 bits
// in 8 bytes, of 32 bits in 12, or the vectors (vertical and horizontal, then
// diagonal) in 24.
enum { KEEP_NONE = 0, KEEP_21 = 64 * 2, KEEP_32 = 64 * 3, KEEP_64 = 64 * 6 };  // words a position
constexpr int32_t KEPT_WORDS = 40 * KEEP_21;  // of LDS
constexpr int32_t MAX_21 = 10, MAX_32 = 15;   // largest distances that slices serve

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint64_t pair64(uint32_t lo, uint32_t hi) { return ((uint64_t)hi << 32) | lo; }
// First bit of a slice around the end diagonal's row e: bits e - 11 .. e + 9 (rows
// e - 10 .. e + 10), or e - 16 .. e + 15; at the vector's ends its first or last.
__device__ __forceinline__ int32_t at_21(int32_t e) { return min(max(e - 11, 0), 43); }
__device__ __forceinline__ int32_t at_32(int32_t e) { return min(max(e - 16, 0), 32); }

// D(a, b) of a window: fewest edits aligning its a pattern bases (bit planes p0,
// p1) with its b text bases (t, 16 a word), its start anchored (D(i, 0) = i,
// D(0, j) = j) or free (both 0).  Myers' bit-vector recurrence on the vertical
// deltas of one text position after another (bit i - 1: D(i, j) - D(i - 1, j) =
// +1 in pv, -1 in mv); the horizontal delta entering at the start row is +1 when
// anchored, 0 when free; bits at and above a only carry upwards and are masked
// off at the end.  Stops after position `upto`; those past `from` are kept (both the
// same in every lane).  FULL: the windows of all lanes are free and of 64 bases
// each side, and keep what their walks need; no position is conditional then, and
// slices begin at known bits.
template <int KEEP, bool FULL = false>
__device__ __forceinline__ int32_t window_pass(uint64_t p0, uint64_t p1, const uint32_t (&t)[4], int32_t a, int32_t b,
                                               bool anchored, int32_t from, int32_t upto, uint32_t *kept) {
  // (halves: v_bitop3_b32 takes any function of three words, bit by bit)
  const int32_t lane = threadIdx.x;
  uint32_t pl = anchored ? ~0u : 0u, ph_ = pl, ml = 0, mh_ = 0;
  const uint32_t pa0 = (uint32_t)p0, pa1 = (uint32_t)(p0 >> 32), pb0 = (uint32_t)p1, pb1 = (uint32_t)(p1 >> 32);
  const uint32_t hin = anchored ? 1u : 0u;
  const int32_t e0 = a - b, last = min(b, upto);
#pragma unroll FULL ? 4 : 1
  for (int32_t w = 0; FULL ? w < 4 : 16 * w < upto; ++w) {
    const int32_t tw = (int32_t)(w == 0 ? t[0] : w == 1 ? t[1] : w == 2 ? t[2] : t[3]);
#pragma unroll
    for (int32_t u = 0; u < 16; ++u) {
      const int32_t j = 16 * w + u + 1;
      if (FULL || j <= last) {
        const uint32_t t0 = (uint32_t)((tw << (31 - 2 * u)) >> 31), t1 = (uint32_t)((tw << (30 - 2 * u)) >> 31);
        const uint32_t eq0 = dev::neither_diff(pa0 ^ t0, pb0, t1), eq1 = dev::neither_diff(pa1 ^ t0, pb1, t1);
        const uint64_t sum = pair64(eq0 & pl, eq1 & ph_) + pair64(pl, ph_);
        const uint32_t xh0 = dev::xor_or((uint32_t)sum, pl, eq0), xh1 = dev::xor_or((uint32_t)(sum >> 32), ph_, eq1);
        const uint32_t hp0 = dev::or_nor(ml, xh0, pl), hp1 = dev::or_nor(mh_, xh1, ph_);  // horizontal +1
        const uint32_t z0 = xh0 | ml, z1 = xh1 | mh_;                           // diagonal 0
        const uint64_t hps = pair64(hp0, hp1) << 1, hms = pair64(pl & xh0, ph_ & xh1) << 1;
        const uint32_t hs0 = (uint32_t)hps | hin, hs1 = (uint32_t)(hps >> 32);
        pl = dev::or_nor((uint32_t)hms, eq0 | ml, hs0);
        ph_ = dev::or_nor((uint32_t)(hms >> 32), eq1 | mh_, hs1);
        ml = dev::and_or(hs0, eq0, ml);
        mh_ = dev::and_or(hs1, eq1, mh_);
        if (KEEP != KEEP_NONE && j > (FULL ? GC_FROM : from)) {
          uint32_t *q = kept + (j - 1 - (FULL ? GC_FROM : from)) * KEEP;
          if (KEEP == KEEP_21) {
            const int32_t at = at_21(FULL ? j : e0 + j);
            const uint32_t v = (uint32_t)(pair64(pl, ph_) >> at), h = (uint32_t)(pair64(hp0, hp1) >> at);
            const uint32_t z = (uint32_t)(pair64(z0, z1) >> at);
            reinterpret_cast<u32x2 *>(q)[lane] = u32x2{(v & 0x1fffffu) | h << 21, ((h >> 11) & 0x3ffu) | z << 10};
          } else if (KEEP == KEEP_32) {
            const int32_t at = at_32(e0 + j);
            q[lane] = (uint32_t)(pair64(pl, ph_) >> at);
            q[64 + lane] = (uint32_t)(pair64(hp0, hp1) >> at);
            q[128 + lane] = (uint32_t)(pair64(z0, z1) >> at);
          } else {
            reinterpret_cast<u32x4 *>(q)[lane] = u32x4{pl, ph_, hp0, hp1};
            reinterpret_cast<u32x2 *>(q + 256)[lane] = u32x2{z0, z1};
          }
        }
      }
    }
  }
  const uint64_t am = low_bits(a);
  return (anchored ? b : 0) + __popcll(pair64(pl, ph_) & am) - __popcll(pair64(ml, mh_) & am);
}

__global__ __launch_bounds__(64) void k_genasm(Seqs S, Outs O, int32_t k, int32_t want_cigar, Work Wk) {
  __shared__ __align__(16) uint32_t kept[KEPT_WORDS];
  const int lane = threadIdx.x;
  const int64_t count = Wk.count ? (int64_t)(*(volatile const int32_t *)Wk.count) : Wk.n;

  // the first 64 pairs are the wavefront's own
  for (int32_t chunk = blockIdx.x; (int64_t)chunk * 64 < count;) {
    const int64_t chunk0 = chunk;
    {
      int32_t next = 0;
      if (lane == 0) next = (int32_t)gridDim.x + atomicAdd(Wk.counter, 1);
      chunk = __shfl(next, 0);
    }
    const int64_t li = chunk0 * 64 + lane;
    const bool has = li < count;
    const int64_t p = has ? (Wk.idx ? (int64_t)Wk.idx[li] : li) : 0;
    bool live = has;
    if (has && !Wk.direct && O.flags && O.flags[p]) {
      O.score[p] = -1;
      O.status[p] = ST_INVALID;
      O.nruns[p] = 0;
      live = false;
    }
    const int32_t m = live ? S.pat_len[p] : 0, n = live ? S.txt_len[p] : 0;
    const uint64_t *pat = S.pat + (live ? S.pat_off[p] : 0);
    const uint64_t *txt = S.txt + (live ? S.txt_off[p] : 0);
    const int64_t pnw = (m + 31) >> 5, tnw = (n + 31) >> 5;
    const bool cig = live && want_cigar;
    const bool direct = Wk.direct != 0;
    const int32_t total = (cig && direct) ? O.nruns[p] : 0;
    uint32_t *dst = (cig && direct) ? O.cigar + O.cigar_off[p] : nullptr;
    RunSink sink;
    if (cig && !direct) sink.begin(O, p);
    uint32_t cur_op = 0xffu, cur_len = 0;
    int32_t nr = 0;
    int32_t me = m, ne = n, used = 0;
    uint32_t prev = OP_NONE;
    bool rej = false;
    // runs still to come, this one included, at most: one per base left, and
    // with a threshold two per edit left plus the current and a last '=' run
    auto put = [&](uint32_t op, uint32_t len, int64_t left) {
      if (!cig) return;
      if (op == cur_op) {
        cur_len += len;
        return;
      }
      if (cur_len) {
        const uint32_t run = (cur_len << 4) | cur_op;
        if (direct) {
          if (nr < total) dst[total - 1 - nr] = run;
        } else {
          int64_t more = left;
          if (k >= 0) more = min<int64_t>(more, 2 * (int64_t)(k - used) + 3);
          sink.put(nr, run, more);
        }
        ++nr;
      }
      cur_op = op;
      cur_len = len;
    };

    while (live && me > 0 && ne > 0) {
      const bool anchored = me <= GW && ne <= GW;
      const int32_t a = min(GW, me), b = min(GW, ne);
      const uint64_t plo = dev::window32(pat, pnw, me - a), phi = dev::window32(pat, pnw, me - a + 32);
      const uint64_t tlo = dev::window32(txt, tnw, ne - b), thi = dev::window32(txt, tnw, ne - b + 32);
      const uint64_t p0 = ((uint64_t)dev::even_bits(phi) << 32) | dev::even_bits(plo);
      const uint64_t p1 = ((uint64_t)dev::even_bits(phi >> 1) << 32) | dev::even_bits(plo >> 1);
      const uint64_t q0 = ((uint64_t)dev::even_bits(thi) << 32) | dev::even_bits(tlo);
      const uint64_t q1 = ((uint64_t)dev::even_bits(thi >> 1) << 32) | dev::even_bits(tlo >> 1);
      const uint32_t t[4] = {(uint32_t)tlo, (uint32_t)(tlo >> 32), (uint32_t)thi, (uint32_t)(thi >> 32)};
      int32_t lw = max(a, b);
      if (k >= 0) lw = min(lw, k - used);
      // wavefront-uniform: the longest window's text, and what is kept at first
      int32_t bmax = GW;
      if (!__any(b == GW)) {
        bmax = 0;
#pragma unroll
        for (int32_t q = GW / 2; q; q >>= 1)
          if (__any(b >= bmax + q)) bmax += q;
      }
      const bool walk = cig || !anchored;
      int32_t upto = bmax, from = max(0, bmax - KEPT_WORDS / KEEP_21), form = KEEP_21;
      int32_t dist;
      if (__all(!anchored && a == GW && b == GW)) dist = window_pass<KEEP_21, true>(p0, p1, t, GW, GW, false, GC_FROM, GW, kept);
      else if (__any(walk)) dist = window_pass<KEEP_21>(p0, p1, t, a, b, anchored, from, upto, kept);
      else dist = window_pass<KEEP_NONE>(p0, p1, t, a, b, anchored, from, upto, kept);
      if (dist > lw) {
        rej = true;
        break;
      }
      if (!walk) {
        // score only: the final window adds its distance
        used += dist;
        me = ne = 0;
        break;
      }
      if (__any(dist > MAX_21)) {
        form = __any(dist > MAX_32) ? KEEP_64 : KEEP_32;
        from = bmax;  // nothing kept yet
      }
      // ---- traceback ----
      int32_t i = a, j = b;
      auto take = [&](uint32_t op, int32_t len) {
        if (op != OP_EQ) used += len;
        if (op != OP_D) i -= len;
        if (op != OP_I) j -= len;
        put(op, (uint32_t)len, (int64_t)(me - a + i) + (ne - b + j) + 2);
        prev = op;
      };
      // Rounds: the bases that match, then one kept entry, which all lanes that
      // need one read together.
      bool done = false;
      while (true) {
        while (!done) {
          // D(i-1, j-1) = D(i, j) where the bases match, so '=' is available:
          // the bases that match from (i, j) back, within the window's walk
          int32_t lim = min(i, j);
          if (!anchored) lim = min(lim, min(GC - (a - i), GC - (b - j)));
          const int32_t up = max(i - j, 0), down = max(j - i, 0);
          const uint64_t x = ((p0 ^ (q0 << up >> down)) | (p1 ^ (q1 << up >> down))) << ((64 - i) & 63);
          const int32_t r = min(x ? __clzll(x) : 64, lim);
          const bool gap = prev == OP_I || prev == OP_D;
          if (!gap && r > 0) take(OP_EQ, r);
          done = lim <= 0 || (!gap && r == lim);
          if (done || j <= from) break;
          const uint32_t *q = kept + (j - 1 - from) * form;
          uint32_t v, h, z;  // the differences, the cell's in bit 0
          if (form == KEEP_21) {
            const u32x2 w = reinterpret_cast<const u32x2 *>(q)[lane];
            const int32_t bit = i - 1 - at_21(j + a - b);
            v = w.x >> bit;
            h = (uint32_t)(pair64(w.x, w.y) >> (21 + bit));
            z = w.y >> (10 + bit);
          } else if (form == KEEP_32) {
            const int32_t bit = i - 1 - at_32(j + a - b);
            v = q[lane] >> bit;
            h = q[64 + lane] >> bit;
            z = q[128 + lane] >> bit;
          } else {
            const u32x4 w = reinterpret_cast<const u32x4 *>(q)[lane];
            const u32x2 w2 = reinterpret_cast<const u32x2 *>(q + 256)[lane];
            v = (uint32_t)(pair64(w.x, w.y) >> (i - 1));
            h = (uint32_t)(pair64(w.z, w.w) >> (i - 1));
            z = (uint32_t)(pair64(w2.x, w2.y) >> (i - 1));
          }
          const bool ins = v & 1u, del = h & 1u;
          const bool match = gap && r > 0;
          const uint32_t other = !(z & 1u) ? OP_X : ins ? OP_I : OP_D;
          const bool on = (prev == OP_I && ins) || (prev == OP_D && del);
          take(on ? prev : match ? OP_EQ : other, !on && match ? r : 1);
        }
        if (!__any(!done)) break;
        // positions before `from`
        upto = from;
        from = max(0, upto - KEPT_WORDS / form);
        if (form == KEEP_21) window_pass<KEEP_21>(p0, p1, t, a, b, anchored, from, upto, kept);
        else if (form == KEEP_32) window_pass<KEEP_32>(p0, p1, t, a, b, anchored, from, upto, kept);
        else window_pass<KEEP_64>(p0, p1, t, a, b, anchored, from, upto, kept);
      }
      if (anchored) {
        if (i > 0) take(OP_I, i);
        else if (j > 0) take(OP_D, j);
      }
      me -= a - i;
      ne -= b - j;
    }
    if (live && !rej) {
      if (me > 0) put(OP_I, (uint32_t)me, 2);
      if (ne > 0) put(OP_D, (uint32_t)ne, 2);
      used += me + ne;
      if (k >= 0 && used > k) rej = true;
      if (!rej) put(0xfu, 0, 1);  // flush the last run
    }
    if (!live || direct) continue;
    if (cig) sink.finish();
    O.score[p] = rej ? -1 : used;
    O.status[p] = rej ? ST_REJECTED : ST_ALIGNED;
    O.nruns[p] = rej ? 0 : nr;
  }
}

}  // namespace

// wavefronts a CU holds (of LDS)
int32_t genasm_waves_per_cu() { return 160 * 1024 / (4 * KEPT_WORDS); }

hipError_t launch_genasm(const Seqs &S, const Outs &O, const Scoring &P, const Work &Wk, int32_t nblocks, hipStream_t s) {
  if (nblocks <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_genasm, dim3(nblocks), dim3(64), 0, s, S, O, P.max_score, P.want_cigar, Wk);
  return hipGetLastError();
}

}  // namespace aim
