// Sequence packing, per-pair validation, prefix scan and CIGAR compaction.
#include <algorithm>

#include "aim_internal.h"

namespace aim {
namespace {

constexpr int SCAN_BLOCK = 256, SCAN_ITEMS = 4, SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__global__ void k_pair_flags(int64_t n, int32_t max_len, const int32_t *pl, const int32_t *tl,
                             const int8_t *pf, const int8_t *tf, int8_t *flags, int64_t *pool_off,
                             ZeroSpans Z) {
  for (int k = 0; k < 3; ++k)
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < Z.n[k]; i += (int64_t)gridDim.x * blockDim.x)
      Z.p[k][i] = 0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t a = pl[i], b = tl[i];
    int8_t f = (a < 0 || b < 0 || a > max_len || b > max_len) ? 1 : 0;
    if (pf && pf[i]) f = 1;
    if (tf && tf[i]) f = 1;
    flags[i] = f;
    if (pool_off) pool_off[i] = -1;
  }
}

// words per sequence for packing
__global__ void k_word_counts(int64_t n, const int32_t *len, int32_t max_len, int32_t *cnt) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t L = len[i];
    // sequences beyond max_len are invalid pairs: give them no words so they
    // do not shift the layout of the others
    cnt[i] = (L > 0 && L <= max_len) ? (L + 31) >> 5 : 0;
  }
}

// G neighbouring lanes per sequence, each packs 8 bases (16 bits of a word) at a
// time: the sequence's last 8 bytes stand in for those past its end.  With a
// wavefront per sequence and a byte at a time two sides of 10,000 x 100 bases
// took 50 us, now 5; launch latency bounds such batches, and memory large ones.
// stride > 0: sequence s starts at word s * stride, written to woff_set
// (entries 0..n); else at woff[s].  blockIdx.y: the side.
struct PackSide {
  const uint8_t *seq;
  const int64_t *off;
  const int32_t *len;
  uint64_t *words;
  const int64_t *woff;
  int8_t *flags;
  int64_t *woff_set;
};
__global__ __launch_bounds__(256) void k_pack(int64_t n, int32_t enc, PackSide A, PackSide B, int32_t max_len,
                                              int64_t words_cap, int64_t stride, int32_t G) {
  const PackSide P = blockIdx.y ? B : A;
  const int64_t s = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / G;
  const int32_t part = threadIdx.x & (G - 1);
  bool bad = false;
  int32_t L = 0;
  if (s < n) {
    if (stride > 0 && part == 0) {
      P.woff_set[s] = s * stride;
      if (s == n - 1) P.woff_set[n] = n * stride;
    }
    L = P.len[s];
    if (L > max_len) {
      bad = true;
      L = 0;
    }
    const uint8_t *src = P.seq + (L > 0 ? P.off[s] : 0);
    const int64_t w0 = stride > 0 ? s * stride : P.woff[s];
    const int32_t pieces = L > 0 ? 4 * ((L + 31) >> 5) : 0;
    for (int32_t q = part; q < pieces; q += G) {
      const int32_t have = min(L - 8 * q, 8);  // bases of this piece (<= 0: none)
      uint64_t v = 0;
      if (have == 8) {
        __builtin_memcpy(&v, src + 8 * q, 8);
      } else if (have > 0 && L >= 8) {
        __builtin_memcpy(&v, src + L - 8, 8);
        v >>= 8 * (8 - have);
      } else {
        for (int32_t t = 0; t < have; ++t) v |= (uint64_t)src[8 * q + t] << (8 * t);
      }
      constexpr uint64_t B1 = 0x0101010101010101ull;
      uint64_t code, wrong;  // a byte each; wrong: not 0 where the byte is no base
      if (enc == 0) {
        // bits 1 and 2 tell A, C, T, G apart; what they stand for is then compared
        const uint64_t x = (v >> 1) & (3 * B1), isT = (x >> 1) & ~x & B1;
        code = x ^ ((x >> 1) & B1);
        wrong = v ^ ((0x41 * B1 | x << 1) ^ isT * 0x11);
      } else {
        code = v & (3 * B1);
        wrong = v & (0xfc * B1);
      }
      const uint64_t in = have >= 8 ? ~0ull : have > 0 ? (1ull << (8 * have)) - 1 : 0ull;
      wrong = ((((wrong & (0x7f * B1)) + 0x7f * B1) | wrong) >> 7) & B1 & in;
      bad |= wrong != 0;
      code &= in & ~(wrong * 3);
      code = (code | code >> 6) & 0x000f000f000f000full;
      code = (code | code >> 12) & 0x000000ff000000ffull;
      code |= code >> 24;
      const int64_t w = w0 + (q >> 2);
      if (w < words_cap) reinterpret_cast<uint16_t *>(P.words + w)[q & 3] = (uint16_t)code;
      else bad = true;
    }
  }
  const uint64_t any = __ballot(bad) >> ((threadIdx.x & 63) & ~(G - 1));
  if (s < n && P.flags && part == 0) P.flags[s] = (any & (G == 64 ? ~0ull : (1ull << G) - 1)) ? 1 : 0;
}

// ---- three-phase exclusive scan of int32 -> int64 ----
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_reduce(const int32_t *in, int64_t n,
                                                           int64_t *tmp) {
  __shared__ int64_t red[SCAN_BLOCK];
  const int64_t base = blockIdx.x * (int64_t)SCAN_TILE;
  int64_t s = 0;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    const int64_t i = base + (int64_t)k * SCAN_BLOCK + threadIdx.x;
    if (i < n) s += in[i];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = SCAN_BLOCK / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) tmp[blockIdx.x] = red[0];
}

// exclusive scan in place of tmp[0..nb), tmp[nb] = total; one block
__global__ __launch_bounds__(1024) void k_scan_blocks(int64_t *tmp, int64_t nb) {
  __shared__ int64_t buf[1024];
  __shared__ int64_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t b0 = 0; b0 < nb; b0 += 1024) {
    const int64_t i = b0 + threadIdx.x;
    const int64_t v = i < nb ? tmp[i] : 0;
    buf[threadIdx.x] = v;
    __syncthreads();
    for (int w = 1; w < 1024; w <<= 1) {
      const int64_t add = threadIdx.x >= w ? buf[threadIdx.x - w] : 0;
      __syncthreads();
      buf[threadIdx.x] += add;
      __syncthreads();
    }
    const int64_t incl = buf[threadIdx.x];
    if (i < nb) tmp[i] = carry + incl - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry += incl;
    __syncthreads();
  }
  if (threadIdx.x == 0) tmp[nb] = carry;
}

// tops: tmp holds the tiles' own sums (few enough to add up in each block, which
// saves a launch), else their exclusive prefixes and the total.
// tw non-null: receives the largest inclusive prefix that fits in cap, if any.
constexpr int64_t SCAN_OWN_TOPS = 2048;
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_apply(const int32_t *in, int64_t n,
                                                          const int64_t *tmp, int64_t *out,
                                                          int64_t nb, bool tops, int64_t cap, int64_t *tw) {
  __shared__ int64_t buf[SCAN_TILE];
  __shared__ int64_t sums[SCAN_BLOCK];
  int64_t before = 0;
  if (tops) {
    int64_t part = 0;
    for (int64_t k = threadIdx.x; k < blockIdx.x; k += SCAN_BLOCK) part += tmp[k];
    sums[threadIdx.x] = part;
    __syncthreads();
    for (int w = SCAN_BLOCK / 2; w > 0; w >>= 1) {
      if (threadIdx.x < w) sums[threadIdx.x] += sums[threadIdx.x + w];
      __syncthreads();
    }
    before = sums[0];
    __syncthreads();
  } else {
    before = tmp[blockIdx.x];
  }
  const int64_t base = blockIdx.x * (int64_t)SCAN_TILE;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    const int64_t i = base + (int64_t)k * SCAN_BLOCK + threadIdx.x;
    buf[k * SCAN_BLOCK + threadIdx.x] = i < n ? in[i] : 0;
  }
  __syncthreads();
  // each thread scans a contiguous run of SCAN_ITEMS, then a block scan of sums
  int64_t local[SCAN_ITEMS];
  int64_t s = 0;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    local[k] = s;
    s += buf[threadIdx.x * SCAN_ITEMS + k];
  }
  sums[threadIdx.x] = s;
  __syncthreads();
  for (int w = 1; w < SCAN_BLOCK; w <<= 1) {
    const int64_t add = threadIdx.x >= w ? sums[threadIdx.x - w] : 0;
    __syncthreads();
    sums[threadIdx.x] += add;
    __syncthreads();
  }
  const int64_t pre = before + sums[threadIdx.x] - s;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    const int64_t i = base + threadIdx.x * SCAN_ITEMS + k;
    if (i >= n) break;
    out[i] = pre + local[k];
    const int64_t incl = pre + local[k] + buf[threadIdx.x * SCAN_ITEMS + k];
    if (i + 1 == n) out[n] = incl;
    if (tw && incl <= cap && (i + 1 == n || incl + in[i + 1] > cap)) *tw = incl;  // of one i at most
  }
}

// One wavefront per `per` pairs (a power of two, at most 64), whose runs are
// one range of the output: lane by lane over the range's runs, each finding
// its pair by bisection of the pairs' offsets in LDS.  The output is written
// in order and no run waits for another, where a thread per pair copied its
// runs one by one (10,000 pairs of a thousand runs each: 10,000 serial
// chains, 0.66 ms; 1,000,000 pairs of 26 runs: 0.20 ms, now 0.08).
constexpr int SCATTER_AHEAD = 4;  // runs a lane has in flight
__global__ __launch_bounds__(64) void k_scatter(
    int64_t n, int32_t per, const int64_t *__restrict__ excl, const unsigned long long *__restrict__ tw_p,
    const int32_t *__restrict__ nruns, const uint32_t *__restrict__ slot, int32_t slot_cap,
    const uint32_t *__restrict__ pool, const int64_t *__restrict__ pool_off,
    int64_t *__restrict__ cigar_off, uint32_t *__restrict__ cigar, int32_t *spill_idx,
    int32_t *spill_count, int8_t *__restrict__ status) {
  // per pair: where its runs begin in the range, and where they lie, last op
  // first: run k at src[k], for k >= the slot's capacity at src2[k].  (64
  // pairs have fewer than 2^28 runs: at most 2 max_len + 1 each)
  __shared__ int32_t off[65];
  __shared__ const uint32_t *src[64], *src2[64];
  const int lane = threadIdx.x;
  const int64_t tw = (int64_t)*tw_p;
  const int64_t i0 = (int64_t)blockIdx.x * per, i = i0 + lane;
  const bool mine = lane < per && i < n;
  const int64_t base = excl[i0];
  const int64_t a = excl[i < n ? i : n], b = excl[i < n ? i + 1 : n];
  if (mine) {
    cigar_off[i] = a < tw ? a : tw;
    if (i + 1 == n) cigar_off[n] = tw;
  }
  const int32_t r = mine ? nruns[i] : 0;
  const uint32_t *s1 = nullptr, *s2 = nullptr;
  if (r > 0) {
    const int64_t pb = pool_off[i];
    if (b > tw) {
      status[i] = ST_OVERFLOW;
    } else if (pb >= POOL_OFF_WHOLE) {
      s1 = s2 = pool + (pb - POOL_OFF_WHOLE);
    } else if (pb <= POOL_OFF_TAIL) {
      s1 = s2 = slot + (i + 1) * (int64_t)slot_cap - r;
    } else if (r <= slot_cap || pb >= 0) {
      s1 = slot + i * (int64_t)slot_cap;
      s2 = r > slot_cap ? pool + pb - slot_cap : s1;
    } else {
      const int32_t k = atomicAdd(spill_count, 1);
      spill_idx[k] = (int32_t)i;
    }
  }
  if (lane < per) {
    src[lane] = s1;
    src2[lane] = s2;
    off[lane] = (int32_t)(a - base);
    if (lane == per - 1) off[per] = (int32_t)(b - base);
  }
  __syncthreads();
  const int32_t end = off[per];
  for (int32_t e0 = lane; e0 < end; e0 += 64 * SCATTER_AHEAD) {
    uint32_t v[SCATTER_AHEAD];
    bool have[SCATTER_AHEAD];
#pragma unroll
    for (int u = 0; u < SCATTER_AHEAD; ++u) {
      const int32_t e = min(e0 + 64 * u, end - 1);
      int p = 0;  // the last pair that begins at or before e
      for (int w = per >> 1; w > 0; w >>= 1)
        if (off[p + w] <= e) p += w;
      const int32_t k = off[p + 1] - 1 - e;
      const uint32_t *s = k < slot_cap ? src[p] : src2[p];
      have[u] = s != nullptr && e0 + 64 * u < end;
      if (have[u]) v[u] = s[k];
    }
#pragma unroll
    for (int u = 0; u < SCATTER_AHEAD; ++u)
      if (have[u]) cigar[base + e0 + 64 * u] = v[u];
  }
}

__global__ void k_zero_offsets(int64_t n, int64_t *off) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i <= n;
       i += (int64_t)gridDim.x * blockDim.x)
    off[i] = 0;
}

// ---- length buckets: counting sort of pairs, longest first ----
constexpr int NBUCKET = 128;

__device__ __forceinline__ int len_bucket(int32_t m, int32_t n) {
  // 8 buckets per octave of max(m, n); reversed so that long pairs come first
  const uint32_t L = (uint32_t)max(max(m, n), 0) + 1u;
  const int lg = 31 - __clz(L);
  const int frac = lg >= 3 ? (int)((L >> (lg - 3)) & 7u) : (int)((L << (3 - lg)) & 7u);
  const int b = min(lg * 8 + frac, NBUCKET - 1);
  return NBUCKET - 1 - b;
}

// Adds this lane's bucket (b < 0: none) to LDS counts and returns its rank: one
// atomic for the wavefront where all its lanes have the same bucket.
__device__ __forceinline__ int bucket_count(int32_t *cnt, int b) {
  const uint64_t have = __ballot(b >= 0);
  if (have == 0) return 0;
  const int b0 = __shfl(b, __ffsll((unsigned long long)have) - 1);
  if (__ballot(b == b0) != have) return b >= 0 ? atomicAdd(&cnt[b], 1) : 0;
  const int lane = threadIdx.x & 63;
  int r = 0;
  if (lane == 0) r = atomicAdd(&cnt[b0], __popcll(have));
  return __shfl(r, 0) + __popcll(have & ((1ull << lane) - 1));
}

__global__ void k_bucket_hist(int64_t n, const int32_t *pl, const int32_t *tl, int32_t *hist) {
  __shared__ int32_t h[NBUCKET];
  for (int k = threadIdx.x; k < NBUCKET; k += blockDim.x) h[k] = 0;
  __syncthreads();
  for (int64_t t0 = blockIdx.x * (int64_t)blockDim.x; t0 < n; t0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = t0 + threadIdx.x;
    bucket_count(h, i < n ? len_bucket(pl[i], tl[i]) : -1);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < NBUCKET; k += blockDim.x)
    if (h[k]) atomicAdd(&hist[k], h[k]);
}

// Per tile of blockDim pairs: ranks within the tile's buckets from LDS
// atomics, then one global atomic per non-empty bucket reserves the tile's
// range (fixed-length batches put nearly every pair in one bucket, where one
// global atomic per pair would serialise).  Every block adds up the buckets
// itself.
__global__ __launch_bounds__(256) void k_bucket_scatter(int64_t n, const int32_t *pl, const int32_t *tl,
                                                       const int32_t *hist, int32_t *cursor, int32_t *order) {
  __shared__ int32_t cnt[NBUCKET], base[NBUCKET], first[NBUCKET];
  if (threadIdx.x < NBUCKET) first[threadIdx.x] = hist[threadIdx.x];
  __syncthreads();
  for (int w = 1; w < NBUCKET; w <<= 1) {
    const int32_t add = (int)threadIdx.x >= w && threadIdx.x < NBUCKET ? first[threadIdx.x - w] : 0;
    __syncthreads();
    if (threadIdx.x < NBUCKET) first[threadIdx.x] += add;
    __syncthreads();
  }
  if (threadIdx.x < NBUCKET) first[threadIdx.x] -= hist[threadIdx.x];
  for (int64_t t0 = blockIdx.x * (int64_t)blockDim.x; t0 < n; t0 += (int64_t)gridDim.x * blockDim.x) {
    for (int k = threadIdx.x; k < NBUCKET; k += blockDim.x) cnt[k] = 0;
    __syncthreads();
    const int64_t i = t0 + threadIdx.x;
    const int b = i < n ? len_bucket(pl[i], tl[i]) : -1;
    const int r = bucket_count(cnt, b);
    __syncthreads();
    for (int k = threadIdx.x; k < NBUCKET; k += blockDim.x)
      if (cnt[k]) base[k] = first[k] + atomicAdd(&cursor[k], cnt[k]);
    __syncthreads();
    if (i < n) order[base[b] + r] = (int32_t)i;
    __syncthreads();
  }
}

// blocks of several tiles, for a tile's reservation is an atomic on one address
inline dim3 sort_grid(int64_t n) { return dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)); }
inline dim3 pack_grid(int64_t n, int32_t lanes, int sides) { return dim3((unsigned)((n + 256 / lanes - 1) / (256 / lanes)), sides); }
inline dim3 grid_for(int64_t n, int block) {
  int64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > 65536) g = 65536;
  return dim3((unsigned)g);
}

}  // namespace

size_t scan_tmp_elems(int64_t n) { return (size_t)((n + SCAN_TILE - 1) / SCAN_TILE + 2); }

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_i32, grid_for(n, 256), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

hipError_t launch_pair_flags(int64_t n, int32_t max_len, const int32_t *pl, const int32_t *tl,
                             const int8_t *pf, const int8_t *tf, int8_t *flags, int64_t *pool_off,
                             const ZeroSpans &Z, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t work = std::max({n, Z.n[0], Z.n[1], Z.n[2]});
  hipLaunchKernelGGL(k_pair_flags, grid_for(work, 256), dim3(256), 0, s, n, max_len, pl, tl, pf, tf,
                     flags, pool_off, Z);
  return hipGetLastError();
}

hipError_t launch_scan_i32(const int32_t *in, int64_t n, int64_t *out, int64_t *tmp,
                           hipStream_t s, int64_t cap, int64_t *tw) {
  const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
  if (nb == 0) {
    hipLaunchKernelGGL(k_zero_offsets, dim3(1), dim3(64), 0, s, (int64_t)0, out);
    return hipGetLastError();
  }
  const bool tops = nb <= SCAN_OWN_TOPS;
  hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, tmp);
  if (!tops) hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(1024), 0, s, tmp, nb);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, tmp, out, nb, tops, cap, tw);
  return hipGetLastError();
}

hipError_t launch_pack(int64_t n, int32_t enc, const uint8_t *seq, const int64_t *off,
                       const int32_t *len, int32_t max_len, uint64_t *words, int64_t words_cap,
                       int64_t *out_off, int8_t *flags, int64_t *scan_tmp, hipStream_t s) {
  if (n == 0) {
    hipLaunchKernelGGL(k_zero_offsets, dim3(1), dim3(64), 0, s, (int64_t)0, out_off);
    return hipGetLastError();
  }
  // word counts go into the tail of scan_tmp's companion area: reuse flags-free int32 buffer
  int32_t *cnt = (int32_t *)(scan_tmp + scan_tmp_elems(n));
  hipLaunchKernelGGL(k_word_counts, grid_for(n, 256), dim3(256), 0, s, n, len, max_len, cnt);
  hipError_t err = launch_scan_i32(cnt, n, out_off, scan_tmp, s);
  if (err != hipSuccess) return err;
  const PackSide A{seq, off, len, words, out_off, flags, nullptr};
  hipLaunchKernelGGL(k_pack, pack_grid(n, 64, 1), dim3(256), 0, s, n, enc, A, A, max_len, words_cap, (int64_t)0, 64);
  return hipGetLastError();
}

hipError_t launch_pack_strided(int64_t n, int32_t enc, const uint8_t *const seq[2], const int64_t *const off[2],
                               const int32_t *const len[2], int32_t max_len, uint64_t *const words[2],
                               int64_t words_cap, int64_t *const out_off[2], int8_t *const flags[2], hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t stride = ((int64_t)max_len + 31) / 32 > 0 ? ((int64_t)max_len + 31) / 32 : 1;
  int32_t G = 4;
  while (G < 64 && (int64_t)G * 8 < max_len) G *= 2;
  const PackSide A{seq[0], off[0], len[0], words[0], nullptr, flags[0], out_off[0]};
  const PackSide B{seq[1], off[1], len[1], words[1], nullptr, flags[1], out_off[1]};
  hipLaunchKernelGGL(k_pack, pack_grid(n, G, 2), dim3(256), 0, s, n, enc, A, B, max_len, words_cap, stride, G);
  return hipGetLastError();
}

hipError_t launch_compact(int64_t n, const Outs &O, int64_t *cigar_off, uint32_t *cigar,
                          int64_t cigar_cap, int64_t *scan_tmp, int64_t *total_written,
                          int32_t *spill_idx, int32_t *spill_count, int8_t *status,
                          hipStream_t s) {
  // scan_tmp layout: [scan blocks | excl (n+1)]
  int64_t *excl = scan_tmp + scan_tmp_elems(n);
  hipError_t err = launch_scan_i32(O.nruns, n, excl, scan_tmp, s, cigar_cap, total_written);
  if (err != hipSuccess) return err;
  unsigned long long *tw = (unsigned long long *)total_written;
  if (n > 0) {
    // 64 pairs per wavefront, fewer where that would leave the chip short of
    // wavefronts (under 4,096)
    int32_t per = 64;
    while (per > 1 && n / per < 4096) per /= 2;
    hipLaunchKernelGGL(k_scatter, dim3((unsigned)((n + per - 1) / per)), dim3(64), 0, s, n, per, excl,
                       (const unsigned long long *)tw, O.nruns, O.slot, O.slot_cap, O.pool,
                       O.pool_off, cigar_off, cigar, spill_idx, spill_count, status);
  } else {
    hipLaunchKernelGGL(k_zero_offsets, dim3(1), dim3(64), 0, s, (int64_t)0, cigar_off);
  }
  return hipGetLastError();
}

hipError_t launch_length_sort(int64_t n, const int32_t *pl, const int32_t *tl, int32_t *hist,
                              int32_t *order, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bucket_hist, sort_grid(n), dim3(256), 0, s, n, pl, tl, hist);
  hipLaunchKernelGGL(k_bucket_scatter, sort_grid(n), dim3(256), 0, s, n, pl, tl, hist, hist + NBUCKET, order);
  return hipGetLastError();
}

hipError_t launch_zero_offsets(int64_t n, int64_t *cigar_off, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_offsets, grid_for(n + 1, 256), dim3(256), 0, s, n, cigar_off);
  return hipGetLastError();
}

}  // namespace aim
