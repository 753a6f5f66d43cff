// Whole analysis of a short window (Section 4.2, Algorithm 2) by one
// workgroup, every intermediate array in LDS or registers.
//
// A short window leaves the stage-by-stage path nothing but latency: an
// analysis of 250 to 5000 tokens took 0.58 to 1.05 ms there, some 200 launches
// and 7 host synchronisations around a few microseconds of work each.  Here it
// is one launch: the window's tokens are read once and its rows written once,
// and the steps in between are separated by workgroup barriers.  Measured on
// MI355X, whole calls: 250 tokens 740 -> 45 us, 4096 tokens 960 -> 170 us, 5000
// tokens with occurrences 1181 -> 204 us, a batch of 64 windows of 250 to 5000
// tokens 4.1 ms -> 271 us.  What bounds it now is the issue rate of one compute
// unit (64 lanes per cycle) and the steps' own latency: 4096 tokens take 118 us
// of kernel time, the token ranks 8, the suffix sort 51, LCP 9, candidates 12,
// their sort 19, the greedy 19.  A first form, radix passes over every suffix in
// every round, took 162.
#include "winfused.h"
#include "device_util.h"
#include "stages.h"
#include <algorithm>

namespace apo {

namespace {

// ---------------------------------------------------------- wavefront scans
// Inclusive sum over the 64 lanes by DPP moves (no LDS round trips).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp0(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t lane_incl_sum(uint32_t v) {
  v += dpp0<0x111, 0xf>(v);
  v += dpp0<0x112, 0xf>(v);
  v += dpp0<0x114, 0xf>(v);
  v += dpp0<0x118, 0xf>(v);
  v += dpp0<0x142, 0xa>(v);
  v += dpp0<0x143, 0xc>(v);
  return v;
}
// Maximum over the lanes, in lane 63.
__device__ __forceinline__ uint32_t lane_max(uint32_t v) {
  v = max(v, dpp0<0x111, 0xf>(v));
  v = max(v, dpp0<0x112, 0xf>(v));
  v = max(v, dpp0<0x114, 0xf>(v));
  v = max(v, dpp0<0x118, 0xf>(v));
  v = max(v, dpp0<0x142, 0xa>(v));
  v = max(v, dpp0<0x143, 0xc>(v));
  return v;
}
// Value of the lane before (lane 0: 0).
__device__ __forceinline__ uint32_t lane_prev(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false);
}

__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// The lanes of `in` whose d agrees with this lane's in its low BITS bits: one
// ballot per bit.  Each step keeps a lane's bit of the mask where the ballot
// agrees with the lane's own bit (a & ~(b ^ c) in one instruction; written out,
// the compiler makes 6 instructions of a bit instead of 4).
template <int BITS>
__device__ __forceinline__ uint64_t equal_lanes(uint32_t d, uint64_t in) {
  uint32_t lo = (uint32_t)in, hi = (uint32_t)(in >> 32);
#pragma unroll
  for (int b = 0; b < BITS; b++) {
    int t = __builtin_amdgcn_sbfe((int)d, b, 1);  // 0 or -1
    asm("" : "+v"(t));  // nothing is known of t: it is compared as it is
    const uint64_t one = __builtin_amdgcn_ballot_w64(t != 0);
    lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)one, (uint32_t)t, 0x90);
    hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(one >> 32), (uint32_t)t, 0x90);
  }
  return ((uint64_t)hi << 32) | lo;
}

constexpr uint32_t kOwnRanks = 4096;     // most distinct values the stage-by-stage batch ranks per window
constexpr uint32_t kOwnPairs = 8192;     // and most distinct adjacent pairs
constexpr int kLongRounds = 18;          // the same for windows of up to kFusedLongMax tokens
static_assert((1u << (kLongRounds - 2)) >= kFusedLongMax && kLongRounds <= kMaxRounds, "the last round leaves nothing grouped");
constexpr uint32_t kLongPack = 8;        // tokens in a sort key there
constexpr int kFusedRounds = 15;         // doubling rounds of a window of up to kFusedMax tokens
static_assert((1u << (kFusedRounds - 2)) >= kFusedMax, "the last round leaves nothing grouped");
constexpr int kPosBits = 13;             // a suffix's position in its sort key
static_assert((1u << kPosBits) >= kFusedMax, "positions");
constexpr uint32_t kPackMost = 16;       // tokens in a sort key
constexpr int kMaxDigit = 7;             // radix digit bits
constexpr int kDigits = 1 << kMaxDigit;  // counter stride per wavefront

// The wavefront's number as a scalar, so that branches on it are scalar too.
__device__ __forceinline__ uint32_t wave_id() {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// Sum of the wavefronts' words before wavefront wv, and of all N (at most 64):
// one word per lane and a scan (adding up 16 words in every lane of every
// wavefront took most of the time of a step that has little else to do).
template <int N>
__device__ __forceinline__ uint32_t words_before(const uint32_t *w, uint32_t wv, uint32_t &all) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t inc = lane_incl_sum(lane < N ? w[lane] : 0u);
  all = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  return wv ? (uint32_t)__builtin_amdgcn_readlane((int)inc, (int)wv - 1) : 0u;
}

// The last word before wavefront wv's that is not kNone (0: none).
__device__ __forceinline__ uint32_t last_word(const uint32_t *w, uint32_t wv) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t v = lane < wv ? w[lane] : kNone;
  const uint64_t m = __ballot(v != kNone);
  return m ? (uint32_t)__builtin_amdgcn_readlane((int)v, 63 - __clzll((long long)m)) : 0u;
}

// The first `c` lanes (all from 64 on).
__device__ __forceinline__ uint64_t first_lanes(uint32_t c) { return c >= 64 ? ~0ull : (1ull << c) - 1ull; }

// Bits of a mask below the calling lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// One stable pass of a radix sort of m items in LDS, in place, by the digit
// digit(item) < 2^kMaxDigit.  Wavefront w holds items [w * 64 * ipt, ...).  It
// ranks its items digit by digit, 64 at a time (lanes of equal digit found by
// one ballot per bit, running counts in its row of cnt), and parks each rank
// beside the item; the digit's first place for the wavefront follows from all
// rows; then every item is read, and after a barrier written to its place.
// Only the last step, which holds MAXI items per lane in registers, is unrolled;
// with the whole pass unrolled the kernel took 97 to 128 registers instead of 79
// to 95, in the same time.
template <int NT, int MAXI, class T, class Digit, class Park, class Parked>
__device__ __forceinline__ void radix_pass(T *it, uint32_t m, int ipt, uint16_t *cnt, uint16_t *row0, Digit digit,
                                           Park park, Parked parked) {
  constexpr int NW = NT / 64;
  const uint32_t lane = threadIdx.x & 63, wv = wave_id(), base = wv * 64 * ipt;
  uint16_t *my = cnt + wv * kDigits;
  const uint16_t *row = row0 + wv * kDigits;
  my[lane] = 0;
  my[64 + lane] = 0;
  wave_order();
#pragma unroll 1
  for (uint32_t q0 = base; q0 < base + 64 * ipt && q0 < m; q0 += 64) {  // scalar
    const uint32_t k = min(q0 + lane, m - 1);
    const uint32_t d = digit(it[k]);
    const uint64_t in = first_lanes(m - q0);
    const uint64_t same = equal_lanes<kMaxDigit>(d, in);
    const uint32_t before = lanes_below(same);
    const uint32_t prev = my[d];
    wave_order();  // every lane has read before the first one of each digit writes
    if (q0 + lane < m) {
      if (before == 0) my[d] = (uint16_t)(prev + (uint32_t)__popcll(same));
      park(k, prev + before);
    }
    wave_order();
  }
  __syncthreads();
  // one digit per lane of two wavefronts: counts into first places, digit by
  // digit and wavefront by wavefront
  if (wv < 2) {  // scalar
    uint32_t c[NW], tot = 0;
#pragma unroll
    for (int w = 0; w < NW; w++) {
      c[w] = cnt[w * kDigits + threadIdx.x];
      tot += c[w];
    }
    const uint32_t inc = lane_incl_sum(tot);
    uint32_t at = inc - tot;
    if (wv == 1) {  // the lower digits' total: one word per lane again
      uint32_t low = 0;
#pragma unroll
      for (int w = 0; w < NW; w++) low += cnt[w * kDigits + lane];
      at += (uint32_t)__builtin_amdgcn_readlane((int)lane_incl_sum(low), 63);
    }
#pragma unroll
    for (int w = 0; w < NW; w++) {
      row0[w * kDigits + threadIdx.x] = (uint16_t)at;
      at += c[w];
    }
  }
  __syncthreads();
  T v[MAXI];
  uint32_t pos[MAXI];
#pragma unroll
  for (int i = 0; i < MAXI; i++)
    if (i < ipt && base + 64 * i < m) {  // scalar
      const uint32_t k = min(base + 64 * i + lane, m - 1);
      v[i] = it[k];
      pos[i] = parked(v[i], k) + row[digit(v[i])];
    }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MAXI; i++)
    if (i < ipt && base + 64 * i + lane < m) it[pos[i]] = v[i];
  __syncthreads();
}

// Place of element i of a key array that threads store IPT consecutive elements
// of: exchanging elements within a block of IPT so that 32 neighbouring threads
// storing their i-th element use 32 different banks (64-bit words); in order, a
// stride of IPT words put 4 to 8 of them on one bank, and the stores of 4096
// keys took as long as the searches (7.5 and 9.2 us in all).
template <int IPT>
__device__ __forceinline__ uint32_t spread(uint32_t i) {
  return i ^ ((i >> 5) & (IPT - 1));
}

// Sorts m distinct 64-bit keys (at most NT * IPT; ~0 pads) held IPT per
// thread into LDS (element i at spread(i)): a wavefront's own run by a network
// over its registers, then runs merged pairwise, each thread producing IPT
// consecutive outputs.  (With only a thread's own run from the network, 4096 keys
// took 19.4 us instead of 15.5.)
template <int NT, int IPT>
__device__ __forceinline__ void merge_sort(uint64_t (&x)[IPT], uint64_t *keys, uint32_t m) {
#pragma unroll 1
  for (uint32_t k = 2; k <= 64 * IPT; k <<= 1)
    lanes_merge<IPT, 32 * IPT>(x, (threadIdx.x & 63) * IPT, k, k == 64 * IPT);
  const uint32_t o0 = threadIdx.x * IPT;
#pragma unroll 1
  for (uint32_t L = 64 * IPT;; L <<= 1) {  // uniform
#pragma unroll
    for (int i = 0; i < IPT; i++)
      if (o0 + i < m) keys[spread<IPT>(o0 + i)] = x[i];
    __syncthreads();
    if (L >= m) break;
    if (o0 < m) {
      // outputs o0 .. o0 + IPT - 1 of the pair of runs A (from `base`) and B:
      // where the first of them splits the runs by binary search, then a merge
      const uint32_t base = o0 & ~(2 * L - 1), d = o0 - base;
      const uint32_t la = min(L, m - base), lb = min(L, m - base - la);
      auto at = [=](uint32_t i) { return keys[spread<IPT>(base + i)]; };  // A, then B from la on
      uint32_t lo = d > lb ? d - lb : 0, hi = min(d, la);
      while (lo < hi) {
        const uint32_t mid = (lo + hi) / 2;
        if (at(mid) < at(la + d - 1 - mid)) lo = mid + 1;
        else hi = mid;
      }
      uint32_t ia = lo, ib = d - lo;
      uint64_t u = ia < la ? at(ia) : ~0ull, v = ib < lb ? at(la + ib) : ~0ull;
#pragma unroll
      for (int i = 0; i < IPT; i++) {
        // equal only when one run is used up and the other's is ~0
        const bool fa = u < v || ib >= lb;
        x[i] = fa ? u : v;
        ia += fa ? 1u : 0u;
        ib += fa ? 0u : 1u;
        const uint64_t nx = (fa ? ia < la : ib < lb) ? at(fa ? ia : la + ib) : ~0ull;
        u = fa ? nx : u;
        v = fa ? v : nx;
      }
    }
    __syncthreads();
  }
}

__device__ __forceinline__ int bits_of(uint32_t x) { return x ? 32 - __clz((int)x) : 0; }

// Minimum of 8 words, and the last of the first `c` (1 to 8) that is below l
// (-1: none); p is 16-byte aligned.
__device__ __forceinline__ uint32_t min8(const uint16_t *p) {
  const uint4 v = *reinterpret_cast<const uint4 *>(p);
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t mn = 0xFFFFu;
#pragma unroll
  for (int q = 0; q < 4; q++) mn = min(mn, min(w[q] & 0xFFFFu, w[q] >> 16));
  return mn;
}
__device__ __forceinline__ int below8(const uint16_t *p, uint32_t c, uint32_t l) {
  const uint4 v = *reinterpret_cast<const uint4 *>(p);
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t f = 0;
#pragma unroll
  for (int q = 0; q < 8; q++) f |= ((w[q >> 1] >> (16 * (q & 1))) & 0xFFFFu) < l ? 1u << q : 0u;
  f &= (1u << c) - 1u;
  return f ? 31 - __clz((int)f) : -1;
}

// Tokens that the suffixes at x and y share, known to share `from`, `lim` being
// left of the shorter one; by a whole wavefront, 512 tokens a step.
__device__ __forceinline__ uint32_t wave_match(const uint16_t *txt, uint32_t x, uint32_t y, uint32_t lim,
                                               uint32_t from) {
  const uint32_t lane = threadIdx.x & 63;
  for (;; from += 512) {
    const uint32_t o = from + 8 * lane;
    uint32_t c = 0;
    bool stop = true;
    if (o + 8 <= lim) {
      uint64_t p0, p1, q0, q1;
      __builtin_memcpy(&p0, txt + x + o, 8);
      __builtin_memcpy(&q0, txt + y + o, 8);
      __builtin_memcpy(&p1, txt + x + o + 4, 8);
      __builtin_memcpy(&q1, txt + y + o + 4, 8);
      const uint64_t d0 = p0 ^ q0, d1 = p1 ^ q1;
      stop = (d0 | d1) != 0;
      c = d0 ? (uint32_t)__builtin_ctzll(d0) / 16 : d1 ? 4 + (uint32_t)__builtin_ctzll(d1) / 16 : 8;
    } else {
      while (o + c < lim && txt[x + o + c] == txt[y + o + c]) c++;  // fewer than 8 are left
    }
    const uint64_t b = __ballot(stop);  // the lanes before the first of them matched 8 each
    if (b) return (uint32_t)__shfl((int)(o + c), __ffsll((long long)b) - 1, 64);
  }
}

// A lower bound of the LCP at the first of a thread's `per` positions, x, with
// its predecessor y (`on`: it has one), within 8 tokens of the LCP or its end where
// that is below kAlone, the LCP itself otherwise.  Kasai's walk from zero is its
// long one: in a periodic window every thread's took up to n tokens.  A lane
// gives up after kAlone; its wavefront goes on, lane by lane from the bound that the lane
// before leaves (an LCP falls by at most one a position), so that the wavefront walks
// its span's length once.  LCP of a loop of 100 tokens over 3000, 8192, 20000 and 32768:
// 156, 257, 1106 and 1213 us before, 48, 40, 70 and 85 so.  kAlone 64: 29, 30, 50, 72, but
// a lane's turn costs more than a short walk (nested loops of 5000, the whole
// call: 229 us instead of 207); 1024: 105, 80, 144, 133.
constexpr uint32_t kAlone = 256;
__device__ __forceinline__ uint32_t first_lcp(const uint16_t *txt, bool on, uint32_t x, uint32_t y, uint32_t lim,
                                              uint32_t per) {
  uint32_t l = 0;
  bool open = on;
  while (open && l < kAlone) {
    if (l + 8 > lim) {
      open = false;
      break;
    }
    uint64_t p0, p1, q0, q1;
    __builtin_memcpy(&p0, txt + x + l, 8);
    __builtin_memcpy(&q0, txt + y + l, 8);
    __builtin_memcpy(&p1, txt + x + l + 4, 8);
    __builtin_memcpy(&q1, txt + y + l + 4, 8);
    if ((p0 ^ q0) | (p1 ^ q1)) open = false;
    else l += 8;
  }
  for (uint64_t m = __ballot(open); m; m &= m - 1) {
    const int src = __ffsll((long long)m) - 1;
    const uint32_t before = (uint32_t)__shfl((int)l, src ? src - 1 : 0, 64);
    uint32_t from = (uint32_t)__shfl((int)l, src, 64);
    if (src && before > per) from = max(from, before - per);
    const uint32_t v = wave_match(txt, (uint32_t)__shfl((int)x, src, 64), (uint32_t)__shfl((int)y, src, 64),
                                  (uint32_t)__shfl((int)lim, src, 64), from);
    if ((int)(threadIdx.x & 63) == src) l = v;
  }
  return l;
}

// Last i < k with lcp[i] < l, or -1: climbs the levels of minima of 8 until a
// block left of k holds one, then descends to it.  Windows of up to CAP tokens.
template <uint32_t CAP>
__device__ __forceinline__ uint32_t last_smaller(const uint16_t *l0, const uint16_t *l1, const uint16_t *l2,
                                                 const uint16_t *l3, uint32_t k, uint32_t l) {
  uint32_t pos = k;
  int lev = 0, f;
  for (;;) {
    if (pos == 0) return kNone;
    const uint32_t lo = (pos - 1) & ~7u;
    const uint16_t *p = lev == 0 ? l0 : lev == 1 ? l1 : lev == 2 ? l2 : l3;
    f = below8(p + lo, pos - lo, l);
    if (f >= 0) {
      f += (int)lo;
      break;
    }
    pos = lo;  // level 3 goes on down itself: CAP / 512 words at most
    if (lev < 3) {
      pos >>= 3;
      lev++;
    }
  }
  while (lev > 0) {
    lev--;
    const uint16_t *p = lev == 0 ? l0 : lev == 1 ? l1 : l2;
    f = 8 * f + below8(p + 8 * f, 8, l);
  }
  return (uint32_t)f;
}

// The sequential greedy over `tot` candidates in priority order, by one
// wavefront, 64 at a time (item(q): start | length << 16): the lowest lane with
// no marked end is accepted and knocks out the later lanes that overlap it; the
// accepted intervals are then marked in the bitmap.  keep(o, q): candidate q is
// accepted occurrence o; returns the number accepted, `na` before.
template <class Item, class Keep>
__device__ __forceinline__ uint32_t greedy_walk(uint32_t *bitmap, uint32_t tot, uint32_t na, Item item, Keep keep) {
  const uint32_t lane = threadIdx.x & 63;
#pragma unroll 1
  for (uint32_t q0 = 0; q0 < tot; q0 += 64) {
    const bool valid = q0 + lane < tot;
    const uint32_t v = item(min(q0 + lane, tot - 1));
    const uint32_t s = v & 0xFFFFu, e = s + (v >> 16) - 1u;
    const uint32_t ws = bitmap[s >> 5], we = bitmap[e >> 5];
    uint64_t pass = __ballot(valid && !((ws >> (s & 31)) & 1u) && !((we >> (e & 31)) & 1u));
    uint64_t take = 0;
    while (pass) {
      const int t = __ffsll((unsigned long long)pass) - 1;
      const uint32_t st = (uint32_t)__builtin_amdgcn_readlane((int)s, t),
                     et = (uint32_t)__builtin_amdgcn_readlane((int)e, t);  // t is uniform
      take |= 1ull << t;
      pass &= ~__ballot(valid && s <= et && e >= st);
    }
    // intervals of a few bitmap words are painted by their own lane, longer
    // ones by the whole wavefront
    const bool mine = (take >> lane) & 1ull;
    const bool own = mine && (e >> 5) - (s >> 5) < 4u;
    if (own)
      for (uint32_t x = s >> 5; x <= (e >> 5); x++) {
        uint32_t msk = kNone;
        if (x == (s >> 5)) msk &= kNone << (s & 31);
        if (x == (e >> 5)) msk &= kNone >> (31 - (e & 31));
        atomicOr(&bitmap[x], msk);
      }
    uint64_t todo = take & ~__ballot(own);
    while (todo) {
      const int t = __ffsll((unsigned long long)todo) - 1;
      todo &= todo - 1;
      const uint32_t st = (uint32_t)__builtin_amdgcn_readlane((int)s, t),
                     et = (uint32_t)__builtin_amdgcn_readlane((int)e, t);
      for (uint32_t x = (st >> 5) + lane; x <= (et >> 5); x += 64) {
        uint32_t msk = kNone;
        if (x == (st >> 5)) msk &= kNone << (st & 31);
        if (x == (et >> 5)) msk &= kNone >> (31 - (et & 31));
        atomicOr(&bitmap[x], msk);
      }
    }
    if (mine) keep(na + lanes_below(take), q0 + lane);
    na += (uint32_t)__popcll(take);
    wave_order();
  }
  return na;
}

struct Row { uint32_t start, length, count; };
struct Occ { uint32_t start, length, cand; };

struct FusedArgs {
  const void *tok;
  int bits;
  const uint64_t *off;     // batch: window offsets; null: one window of n tokens
  const uint32_t *order;   // batch: block b takes window order[b] (what is behind the windows': upload_windows)
  uint32_t windows;        // batch
  uint32_t n, min_len;
  Row *rows;               // one window: final; batch: window w's rows start at off[w] / min_len
  Occ *occ;
  uint32_t row_cap, occ_cap;
  uint64_t *spill;         // two words per token: records that find no room in LDS yet
  FusedInfo *info;         // one window
  uint32_t *win_rows;      // batch
  uint32_t *parts;         // batch: copies of the counters, added up over a share of the windows each
  uint32_t part_mask;      // their number, a power of two, - 1
};

// A batch's counters: in one copy for all its windows an atomic waits for another on
// the same words, some 100 ns a window (10^5 windows of 250 tokens 12.7 ms, now
// 4.0; 10^6 of 25 tokens 119 and 23).  A copy for 64 windows, up to kParts: the words
// of dcnt, then a word per doubling round.
constexpr uint32_t kParts = 64, kPartWords = 64;
static_assert(CNT_COUNT + kLongRounds <= kPartWords, "a part");
__device__ __forceinline__ uint32_t *part_of(const FusedArgs &a) {
  return a.parts + (blockIdx.x & a.part_mask) * kPartWords;
}

// What a window's analysis found, to the host (one window) or added to the
// batch's counters.  own: distinct tokens without the largest value.
struct Report { uint32_t sigma, own, cands, skipped, maxl, m, accepted, rows, pairs, nhist; };

__device__ __forceinline__ void report(const FusedArgs &a, uint32_t win, const Report &r, const uint32_t *hist,
                                       const uint64_t *stamp) {
  if (a.info) {
    FusedInfo &f = *a.info;
    f.sigma = a.bits == 64 ? r.sigma : 0u;
    f.cands = r.cands + r.skipped;
    f.maxl = r.maxl;
    f.m = r.m;
    f.accepted = r.accepted;
    f.rows = r.rows;
    f.nhist = r.nhist;
    for (uint32_t k = 0; k < r.nhist; k++) f.hist[k] = hist[k];
    for (int k = 0; k <= kStages; k++) f.stamp[k] = stamp[k];
    return;
  }
  a.win_rows[win] = r.rows;
  uint32_t *const cnt = part_of(a);
  atomicAdd(&cnt[CNT_NDSUM], r.sigma);
  atomicMax(&cnt[CNT_NDMAX], r.sigma);
  atomicAdd(&cnt[CNT_C], r.cands);
  atomicAdd(&cnt[CNT_CSKIP], r.skipped);
  atomicMax(&cnt[CNT_MAXL], r.maxl);
  atomicAdd(&cnt[CNT_M], r.m);
  atomicAdd(&cnt[CNT_A], r.accepted);
  atomicAdd(&cnt[CNT_NROWS], r.rows);
  // past the bounds of the stage-by-stage batch's per-window ranks and pair ranks
  if (r.own > kOwnRanks || r.pairs > kOwnPairs) {
    uint32_t g = 0;  // the window's lane
    while (g < 3 && win >= a.order[a.windows + 1 + g]) g++;
    atomicAdd(&cnt[CNT_RANGE + g], 1u);
  }
  for (uint32_t k = 0; k < r.nhist; k++)
    if (hist[k]) atomicAdd(&cnt[CNT_COUNT + k], hist[k]);
  for (int k = 0; k < kStages; k++) atomicMax(&cnt[CNT_STAGE + k], (uint32_t)(stamp[k + 1] - stamp[k]));
}

// LDS of a window of up to NT * IPT tokens.  lds holds, one phase after the other:
//   ranking: the tokens; the hash table, later the sorted distinct values
//   suffix sort: sort keys, later the list being sorted and its parked ranks;
//     token ranks (32 zero words past the end), suffix ranks, suffix order, LCP
//   candidates: records start | ID << 16 | length << 32 | parked rank << 48
template <int NT, int IPT>
struct ShortLds {
  static constexpr uint32_t CAP = NT * IPT, ROWS = NT / 64 * kDigits;
  alignas(16) unsigned char lds[CAP * 16 + 64];
  alignas(16) uint16_t rc[CAP > ROWS ? CAP : ROWS];  // distinct values' tokens; radix rows; accepted candidates
  alignas(16) uint16_t cnt[ROWS];  // radix counters; LCP minima; surviving candidates
  uint32_t bitmap[CAP / 32 + 2];   // slots that open a group; accepted positions; row openings
  uint32_t wsum[NT / 64], wsum2[NT / 64];
  uint32_t s_nd, s_top, s_zero, s_active, s_large, s_max, s_skip, s_c, s_acc, s_dup;
  uint32_t s_hist[kFusedRounds];
  uint64_t s_stamp[kStages + 1];
};

// The analysis of window `win` (n tokens from token tb on) by NT threads.
template <int NT, int IPT>
__device__ __forceinline__ void window_short(const FusedArgs &a, ShortLds<NT, IPT> &L, uint32_t win, uint64_t tb,
                                             uint32_t n) {
  constexpr int NW = NT / 64;
  constexpr uint32_t CAP = NT * IPT, SLOTS = 2 * CAP;
  constexpr uint32_t EARLY = CAP + CAP / 2 + 8;  // candidate records that fit before sa
  static_assert(CAP <= kFusedMax, "16 bytes of LDS per token, and positions and ranks in 13 bits");
  auto &lds = L.lds;
  auto &rc = L.rc;
  auto &cnt = L.cnt;
  auto &bitmap = L.bitmap;
  auto &wsum = L.wsum;
  auto &wsum2 = L.wsum2;
  auto &s_nd = L.s_nd, &s_top = L.s_top, &s_zero = L.s_zero, &s_active = L.s_active, &s_large = L.s_large;
  auto &s_max = L.s_max, &s_skip = L.s_skip, &s_c = L.s_c, &s_acc = L.s_acc, &s_dup = L.s_dup;
  auto &s_hist = L.s_hist;
  auto &s_stamp = L.s_stamp;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wv = wave_id();
  const uint64_t below = (1ull << lane) - 1ull;
  auto stamp = [&](int k) {
    if (tid == 0) s_stamp[k] = wall_clock64();
  };
  stamp(0);

  // ---- order-preserving token ranks.  Distinct values through an LDS hash
  // table (a slot holds the number of the token that claimed it, every other
  // token's entry becomes that number); the claimants' values sorted; each
  // claimant's entry becomes its rank, found by binary search.
  uint64_t *tokl = reinterpret_cast<uint64_t *>(lds);
  {
    uint32_t *tab = reinterpret_cast<uint32_t *>(lds + CAP * 8);
    if (a.bits == 64) {
      const uint64_t *t = static_cast<const uint64_t *>(a.tok) + tb;
      uint64_t v[IPT];
#pragma unroll
      for (int i = 0; i < IPT; i++) v[i] = t[min(i * NT + tid, n - 1)];
#pragma unroll
      for (int i = 0; i < IPT; i++)
        if (i * NT + tid < n) tokl[i * NT + tid] = v[i];
    } else {
      const uint32_t *t = static_cast<const uint32_t *>(a.tok) + tb;
      uint32_t v[IPT];
#pragma unroll
      for (int i = 0; i < IPT; i++) v[i] = t[min(i * NT + tid, n - 1)];
#pragma unroll
      for (int i = 0; i < IPT; i++)
        if (i * NT + tid < n) tokl[i * NT + tid] = v[i];
    }
    if (tid == 0) {
      s_nd = 0;
      s_top = 0;
      s_skip = 0;
      s_max = 0;
      s_c = 0;
      s_acc = 0;
      s_dup = 0;
    }
    if (tid < kFusedRounds) s_hist[tid] = 0;
    for (uint32_t k = 4 * tid; k < SLOTS; k += 4 * NT)
      *reinterpret_cast<uint4 *>(tab + k) = make_uint4(kNone, kNone, kNone, kNone);
    __syncthreads();
#pragma unroll 1
    for (uint32_t k = tid; k < n; k += NT) {
      const uint64_t key = tokl[k];
      uint32_t at = (uint32_t)(mix64(key) >> 40) & (SLOTS - 1);
      for (;;) {  // n <= SLOTS / 2 values: a free slot is always found
        uint32_t cur = tab[at];
        if (cur == kNone) {
          cur = atomicCAS(&tab[at], kNone, k);
          if (cur == kNone) {
            rc[atomicAdd(&s_nd, 1u)] = (uint16_t)k;
            if (key == ~0ull) s_top = 1;
            break;
          }
        }
        if (tokl[cur] == key) {
          tokl[k] = cur;  // nobody reads this token's value: it is in no slot
          break;
        }
        at = (at + 1) & (SLOTS - 1);
      }
    }
    __syncthreads();
  }
  const uint32_t D = s_nd;
  auto rank_by = [&](auto each) {
    constexpr int R = decltype(each)::value;
    uint64_t *sorted = reinterpret_cast<uint64_t *>(lds + CAP * 8);
    uint64_t x[R];
#pragma unroll
    for (int i = 0; i < R; i++) {
      const uint32_t q = tid * R + i;
      x[i] = q < D ? tokl[rc[min(q, D - 1)]] : ~0ull;
    }
    merge_sort<NT, R>(x, sorted, D);  // the table's last reads are a barrier behind
#pragma unroll 1
    for (uint32_t q = tid; q < D; q += NT) {
      const uint32_t k = rc[q];
      const uint64_t key = tokl[k];
      uint32_t lo = 0, hi = D - 1;  // sorted[lo .. hi] holds it
      while (lo < hi) {
        const uint32_t mid = (lo + hi) / 2;
        if (sorted[spread<R>(mid)] < key) lo = mid + 1;
        else hi = mid;
      }
      tokl[k] = (1ull << 63) | (lo + 1);
    }
    __syncthreads();
  };
  // one a thread where that holds them all: a merge's steps are one thread's outputs after another
  if (D <= NT) rank_by(std::integral_constant<int, 1>{});
  else rank_by(std::integral_constant<int, IPT>{});
  uint16_t *txt = reinterpret_cast<uint16_t *>(lds + CAP * 8);  // token ranks 1..D
  uint16_t *rank = txt + CAP + 32, *sa = rank + CAP, *lcp = sa + CAP;
  uint32_t *exch = reinterpret_cast<uint32_t *>(lds);
  uint16_t *rel = reinterpret_cast<uint16_t *>(lds + CAP * 4);
#pragma unroll 1
  for (uint32_t k = tid; k < n; k += NT) {
    const uint64_t e = tokl[k];
    txt[k] = (uint16_t)((e >> 63) ? e : tokl[e]);
  }
  if (tid < 32) txt[n + tid] = 0;
  __syncthreads();
  stamp(1);

  // ---- suffix array.  First every suffix sorted by as many tokens as fit in a
  // 64-bit word above its position (3 at least, kPackMost at most).
  const int ipt = (int)((n + NT - 1) / NT);
  const int tbits = bits_of(D);
  uint32_t h = min((uint32_t)((64 - kPosBits) / tbits), kPackMost);
  {
    uint64_t x[IPT];
#pragma unroll
    for (int i = 0; i < IPT; i++) x[i] = 0;
#pragma unroll 1
    for (uint32_t q = 0; q < h; q++)  // zeros past the end: h <= 32
#pragma unroll
      for (int i = 0; i < IPT; i++) x[i] = (x[i] << tbits) | txt[min(tid * IPT + i, n - 1) + q];
#pragma unroll
    for (int i = 0; i < IPT; i++) {
      const uint32_t j = tid * IPT + i;
      x[i] = j < n ? (x[i] << kPosBits) | j : ~0ull;
    }
    merge_sort<NT, IPT>(x, reinterpret_cast<uint64_t *>(lds), n);
  }
  // Groups of equal h-token prefixes: a bitmap of the slots that open one (slot
  // n counts as one), and rank[j] = the first slot of j's group.
  const uint32_t wbase = wv * 64 * ipt, wtop = min(wbase + 64 * ipt, n);  // the wavefront's slots
  {
    const uint64_t *keys = reinterpret_cast<const uint64_t *>(lds);
#pragma unroll 1
    for (uint32_t k0 = wbase; k0 < wtop; k0 += 64) {  // scalar
      const uint32_t k = min(k0 + lane, n - 1);
      const uint64_t key = keys[spread<IPT>(k)], prev = keys[spread<IPT>(k ? k - 1 : 0)];
      const uint32_t j = (uint32_t)key & ((1u << kPosBits) - 1u);
      sa[k] = (uint16_t)j;
      if (j == 0) s_zero = k;
      const uint64_t hd = __ballot(k0 + lane == 0 || k0 + lane >= n || (prev >> kPosBits) != (key >> kPosBits));
      if (lane == 0) {
        bitmap[k0 >> 5] = (uint32_t)hd;
        bitmap[(k0 >> 5) + 1] = (uint32_t)(hd >> 32);
      }
    }
    if (tid == 0 && n % 64 == 0) bitmap[n >> 5] = 1;
    __syncthreads();
#pragma unroll 1
    for (uint32_t k = tid; k < n; k += NT) {
      uint32_t x = k >> 5, w = bitmap[x] & ((2u << (k & 31)) - 1u);
      while (!w) w = bitmap[--x];  // slot 0 opens a group
      rank[sa[k]] = (uint16_t)(32 * x + 31u - (uint32_t)__clz((int)w));
    }
  }
  // Suffixes still grouped, and whether some group is large (96 slots or more;
  // up to 158 may pass): counting costs a group's size per member, the radix
  // passes about as much as a group of 100 (5000 tokens of a nested loop: 16 us a
  // round by counting, 17 to 20 by radix passes).
  uint32_t active;
  bool large;
  auto survey = [&] {
    if (tid == 0) s_active = s_large = 0;
    __syncthreads();
    if (2048 * wv < n) {  // scalar: one word per lane
      uint32_t more = 0;
      if (32 * tid < n) {
        const uint32_t w = bitmap[tid], up = 32 * tid + 32 <= n ? bitmap[tid + 1] : kNone;
        more = (uint32_t)__popc(~(w & ((w >> 1) | (up << 31))) & (uint32_t)first_lanes(n - 32 * tid));
        if (!(w | up) && 32 * tid + 64 <= n && !bitmap[tid + 2]) s_large = 1;  // 96 slots without an opening
      }
      more = lane_incl_sum(more);
      if (lane == 63 && more) atomicAdd(&s_active, more);
    }
    __syncthreads();
    active = s_active;
    large = s_large != 0;
  };
  survey();
  // Then prefix doubling of the suffixes still grouped.  While no group is
  // large a suffix finds its new group by counting its group's members with a
  // smaller second half, whose group numbers lie side by side (eight per LDS
  // read); its place in the new group is taken from a counter, any order doing.
  // Otherwise a round lists them in the order of their second halves (j = SA[k] - h over all slots k) and sorts
  // that list stably by the group of the first half.  The h shortest suffixes,
  // whose second half is empty, wrap around (j = SA[k] - h + n): the one of h
  // tokens (SA[k] = 0) is put first, the shorter ones are alone in their groups.
  uint16_t *sah = sa;  // where the suffix order is now
  while (active && h < n) {  // uniform (from n tokens on nothing can be grouped)
    const uint32_t m = active;
    if (!large) {
      uint32_t *ctr = reinterpret_cast<uint32_t *>(lds);
      uint16_t *half = reinterpret_cast<uint16_t *>(lds + CAP * 4);
      uint16_t *san = sah == sa ? half + CAP : sa;
#pragma unroll 1
      for (uint32_t k = tid; k < n; k += NT) {
        const uint32_t s = sah[k] + h;
        const uint32_t r = rank[min(s, n - 1)];
        half[k] = (uint16_t)(s < n ? r + 1 : 0);
        ctr[k] = 0;
      }
      __syncthreads();
#pragma unroll 1
      for (uint32_t k = tid; k < n; k += NT) {
        const uint32_t j = sah[k], g = rank[j];
        if ((bitmap[(g + 1) >> 5] >> ((g + 1) & 31)) & 1u) {
          san[k] = (uint16_t)j;
          continue;
        }
        uint32_t x = (k + 1) >> 5, w = bitmap[x] & (kNone << ((k + 1) & 31));
        while (!w) w = bitmap[++x];
        const uint32_t e = 32 * x + (uint32_t)__ffs((int)w) - 1u;  // the group: slots [g, e)
        typedef short pair __attribute__((ext_vector_type(2)));
        const short me = (short)half[k];
        const pair mine = {me, me};
        uint32_t less = 0;
        for (uint32_t b = g & ~7u; b < e; b += 8) {
          const uint4 v = *reinterpret_cast<const uint4 *>(half + b);
          uint32_t sg[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int q = 0; q < 4; q++)  // sign bits: below mine (values of at most 14 bits)
            sg[q] = __builtin_bit_cast(uint32_t, (pair)(__builtin_bit_cast(pair, sg[q]) - mine)) & 0x80008000u;
          if (b < g || b + 8 > e) {
            const uint32_t ok = (b < g ? 0xFFu << (g - b) : 0xFFu) & (b + 8 > e ? (1u << (e - b)) - 1u : 0xFFu);
#pragma unroll
            for (int q = 0; q < 4; q++)
              sg[q] &= ((ok >> (2 * q)) & 1u ? 0x8000u : 0u) | ((ok >> (2 * q + 1)) & 1u ? 0x80000000u : 0u);
          }
          less += (uint32_t)(__popc(sg[0]) + __popc(sg[1]) + __popc(sg[2]) + __popc(sg[3]));
        }
        rank[j] = (uint16_t)(g + less);  // this suffix's old group number was this thread's alone to read
        san[g + less + atomicAdd(&ctr[g + less], 1u)] = (uint16_t)j;
      }
      __syncthreads();
#pragma unroll 1
      for (uint32_t k0 = wbase; k0 < wtop; k0 += 64) {  // scalar
        const uint32_t k = min(k0 + lane, n - 1), j = san[k];
        if (j == 0) s_zero = k;
        const uint64_t hd = __ballot(k0 + lane >= n || rank[j] == k);
        if (lane == 0) {
          bitmap[k0 >> 5] = (uint32_t)hd;
          bitmap[(k0 >> 5) + 1] = (uint32_t)(hd >> 32);
        }
      }
      sah = san;
      h *= 2;
      survey();
      continue;
    }
    if (sah != sa) {  // uniform
      for (uint32_t k = tid; k < n; k += NT) sa[k] = sah[k];
      sah = sa;
      __syncthreads();
    }
    {
      const uint32_t first = s_zero;
      uint32_t e[IPT];
      uint64_t mk[IPT];
      uint32_t run = 0;
#pragma unroll
      for (int i = 0; i < IPT; i++) {
        mk[i] = 0;
        const uint32_t k0 = wv * 64 * ipt + 64 * i, k = min(k0 + lane, n - 1);
        if (i >= ipt || k0 >= n) continue;  // uniform
        const uint32_t s = sa[k == 0 ? first : k <= first ? k - 1 : k];
        const uint32_t j = s >= h ? s - h : s + n - h;
        const uint32_t g = rank[j];
        e[i] = j | (g << 16);
        mk[i] = __ballot(!((bitmap[(g + 1) >> 5] >> ((g + 1) & 31)) & 1u)) & first_lanes(n - k0);
        run += (uint32_t)__popcll(mk[i]);
      }
      if (lane == 0) wsum[wv] = run;
      __syncthreads();
      uint32_t all, off = words_before<NW>(wsum, wv, all);
#pragma unroll
      for (int i = 0; i < IPT; i++) {
        if ((mk[i] >> lane) & 1ull) exch[off + lanes_below(mk[i])] = e[i];
        off += (uint32_t)__popcll(mk[i]);
      }
      __syncthreads();
    }
    const int mpt = (int)((m + NT - 1) / NT);
    {
      const int gbits = bits_of(n - 1), low = gbits > kMaxDigit ? gbits / 2 : gbits;
#pragma unroll 1
      for (int shift = 0; shift < gbits; shift += low) {
        const uint32_t msk = shift ? kNone : (1u << low) - 1u;  // the upper digit takes what is left
        radix_pass<NT, IPT>(
            exch, m, mpt, cnt, rc, [=](uint32_t e) { return (e >> (16 + shift)) & msk; },
            [=](uint32_t k, uint32_t r) { rel[k] = (uint16_t)r; }, [=](uint32_t, uint32_t k) { return (uint32_t)rel[k]; });
        if (shift) break;
      }
    }
    {
      // new groups: entry q opens one when its first or second half's group
      // differs from the entry before; its slot is its distance into the old
      // group past that group's first slot
      uint64_t og[IPT], ng[IPT];
      uint32_t e[IPT];
      uint32_t lo = kNone, ln = kNone;  // the wavefront's last old and new group openings
#pragma unroll
      for (int i = 0; i < IPT; i++) {
        og[i] = ng[i] = ~0ull;
        const uint32_t q0 = wv * 64 * mpt + 64 * i, q = q0 + lane;
        if (i >= mpt || q0 >= m) continue;  // uniform
        e[i] = exch[min(q, m - 1)];
        const uint32_t s = (e[i] & 0xFFFFu) + h;
        const uint32_t r = rank[min(s, n - 1)];
        const uint32_t c = (e[i] & 0xFFFF0000u) | (s < n ? r : 0xFFFFu);
        uint32_t p = lane_prev(c);
        if (lane == 0 && q) {
          const uint32_t b = exch[q - 1], s = (b & 0xFFFFu) + h;
          p = (b & 0xFFFF0000u) | (s < n ? rank[s] : 0xFFFFu);
        }
        og[i] = __ballot(q == 0 || q >= m || (c >> 16) != (p >> 16));
        ng[i] = __ballot(q == 0 || q >= m || c != p);
        const uint64_t in = first_lanes(m - q0);
        if (og[i] & in) lo = q0 + 63u - (uint32_t)__clzll((long long)(og[i] & in));
        if (ng[i] & in) ln = q0 + 63u - (uint32_t)__clzll((long long)(ng[i] & in));
      }
      if (lane == 0) {
        wsum[wv] = lo;
        wsum2[wv] = ln;
      }
      __syncthreads();
      uint32_t co = last_word(wsum, wv), cn = last_word(wsum2, wv);
#pragma unroll
      for (int i = 0; i < IPT; i++) {
        const uint32_t q0 = wv * 64 * mpt + 64 * i;
        if (i >= mpt || q0 >= m) continue;
        const uint64_t in = first_lanes(m - q0);
        const uint64_t upto = in & (below | (1ull << lane)), uo = og[i] & upto, un = ng[i] & upto;
        if (q0 + lane < m) {
          const uint32_t ob = uo ? q0 + 63u - (uint32_t)__clzll((long long)uo) : co;
          const uint32_t nb = un ? q0 + 63u - (uint32_t)__clzll((long long)un) : cn;
          const uint32_t j = e[i] & 0xFFFFu, g = e[i] >> 16, slot = g + (q0 + lane - ob);
          sa[slot] = (uint16_t)j;
          rank[j] = (uint16_t)(g + (nb - ob));
          if (nb == q0 + lane) atomicOr(&bitmap[slot >> 5], 1u << (slot & 31));
          if (j == 0) s_zero = slot;
        }
        if (og[i] & in) co = q0 + 63u - (uint32_t)__clzll((long long)(og[i] & in));
        if (ng[i] & in) cn = q0 + 63u - (uint32_t)__clzll((long long)(ng[i] & in));
      }
      h *= 2;
      survey();  // its first barrier ends the writes above
    }
  }
  if (sah != sa) {  // uniform
    for (uint32_t k = tid; k < n; k += NT) sa[k] = sah[k];
    __syncthreads();
  }
  stamp(2);

  // ---- LCP: Kasai's walk over ipt consecutive positions per thread, eight
  // tokens per step; suffixes are all alone, so rank is the inverse of sa
  {
    const uint32_t x0 = tid * ipt, r0 = x0 < n ? rank[x0] : 0u, y0 = r0 ? sa[r0 - 1] : 0u;
    uint32_t h = first_lcp(txt, r0 != 0, x0, y0, n - (x0 > y0 ? x0 : y0), ipt);
    for (int i = 0; i < ipt; i++) {
      const uint32_t x = x0 + i;
      if (x >= n) break;
      const uint32_t r = rank[x];
      if (r == 0) {
        h = 0;
        continue;
      }
      const uint32_t y = sa[r - 1], lim = n - (x > y ? x : y);
      while (h < lim) {
        uint64_t p0, p1, q0, q1;
        __builtin_memcpy(&p0, txt + x + h, 8);
        __builtin_memcpy(&q0, txt + y + h, 8);
        __builtin_memcpy(&p1, txt + x + h + 4, 8);
        __builtin_memcpy(&q1, txt + y + h + 4, 8);
        const uint64_t d0 = p0 ^ q0, d1 = p1 ^ q1;
        if (d0 | d1) {
          h += d0 ? (uint32_t)(__ffsll((long long)d0) - 1) >> 4 : 4u + ((uint32_t)(__ffsll((long long)d1) - 1) >> 4);
          break;
        }
        h += 8;
      }
      h = h < lim ? h : lim;
      lcp[r - 1] = (uint16_t)h;
      h = h ? h - 1 : 0;
    }
    if (tid == 0) lcp[n - 1] = 0;
    if (tid < 8 && n + tid < ((n + 7) & ~7u)) lcp[n + tid] = 0xFFFF;
  }
  // minima of 8, 64 and 512 LCP values for the ID's previous-smaller-value
  // queries (0xFFFF past the end)
  uint16_t *min1 = cnt, *min2 = min1 + CAP / 8, *min3 = min2 + CAP / 64;
  static_assert(CAP / 8 + CAP / 64 + CAP / 64 <= NW * kDigits, "minima fit the radix counters");
  for (uint32_t b = tid; b < CAP / 8 + CAP / 64 + CAP / 64; b += NT) cnt[b] = 0xFFFF;
  __syncthreads();
  stamp(3);

  // ---- candidates of every adjacent pair in suffix-array order
  for (uint32_t b = tid; b < (n + 7) / 8; b += NT) min1[b] = (uint16_t)min8(lcp + 8 * b);
  __syncthreads();
  for (uint32_t b = tid; b < (n + 63) / 64; b += NT) min2[b] = (uint16_t)min8(min1 + 8 * b);
  __syncthreads();
  for (uint32_t b = tid; b < (n + 511) / 512; b += NT) min3[b] = (uint16_t)min8(min2 + 8 * b);
  __syncthreads();
  uint64_t *rec = reinterpret_cast<uint64_t *>(lds);
  {
    uint32_t mx = 0;
#pragma unroll 1
    for (uint32_t k0 = wv * 64 * ipt; k0 < wv * 64 * ipt + 64 * ipt && k0 < n; k0 += 64) {  // scalar
      const uint32_t k = k0 + lane;
      uint32_t l = 0, s1 = 0, s2 = 0, both = 0;
      bool rep = false;
      if (k < n) {
        const uint32_t x = sa[k], y = k + 1 < n ? sa[k + 1] : x, p = lcp[k];
        const uint32_t w = k ? sa[k - 1] : x, pp = k ? lcp[k - 1] : 0u;
        both = max(p, pp);
        const uint32_t lo = min(x, y), d = max(x, y) - lo;
        const bool disj = p <= d;
        if (disj) {
          l = p;
          s1 = x;
          s2 = y;
        } else {
          l = (p + d) / 2;
          l -= l % d;
          s1 = lo;
          s2 = lo + l;
        }
        if (l < a.min_len || k + 1 == n) l = 0;
        // pair k - 1 disjoint too and of equal length: its second candidate is
        // this pair's first
        rep = l && disj && k && pp == l && pp <= max(x, w) - min(x, w);
      }
      // a suffix shares 2^r tokens with a neighbour: still grouped after round r
#pragma unroll 1
      for (int r = 0; r < kFusedRounds; r++) {
        const uint64_t g = __ballot(both >> r);
        if (!g) break;  // scalar
        if (lane == 0) atomicAdd(&s_hist[r], (uint32_t)__popcll(g));
      }
      const uint64_t m2 = __ballot(l != 0), m1 = __ballot(l != 0 && !rep);
      if (!m2) continue;  // scalar
      const uint64_t id = l ? 1u + last_smaller<CAP>(lcp, min1, min2, min3, k, l) : 0u;
      // records in any order: the sort's key tells all but duplicates apart
      uint32_t q = 0;
      if (lane == 0) {
        q = atomicAdd(&s_c, (uint32_t)(__popcll(m1) + __popcll(m2)));
        atomicAdd(&s_skip, (uint32_t)(__popcll(m2) - __popcll(m1)));
      }
      q = (uint32_t)__builtin_amdgcn_readfirstlane((int)q) + lanes_below(m1) + lanes_below(m2);
      if (l) {
        const uint64_t head = (id << 16) | ((uint64_t)l << 32);
        if (!rep) {
          if (q < EARLY) rec[q] = head | s1;
          else a.spill[2 * tb + q] = head | s1;
          q++;
        }
        if (q < EARLY) rec[q] = head | s2;
        else a.spill[2 * tb + q] = head | s2;
      }
      mx = max(mx, l);
    }
    mx = lane_max(mx);
    if (lane == 63 && mx) atomicMax(&s_max, mx);
  }
  __syncthreads();  // suffix order, LCP and minima read, records written
  const uint32_t C = s_c, maxl = s_max;
  for (uint32_t k = EARLY + tid; k < C; k += NT) rec[k] = a.spill[2 * tb + k];
  for (uint32_t k = tid; k < (n + 31) / 32; k += NT) bitmap[k] = 0;
  __syncthreads();
  stamp(4);

  // ---- priority order (length desc, ID asc, start asc): a radix sort of the
  // three fields as one key
  if (C) {  // uniform
    const int pb = bits_of(n - 1), bits = bits_of(maxl - a.min_len) + 2 * pb;
    const int np = (bits + kMaxDigit - 1) / kMaxDigit;
#pragma unroll 1
    for (int p = 0; p < np; p++)
      radix_pass<NT, 2 * IPT>(
          rec, C, (int)((C + NT - 1) / NT), cnt, rc,
          [=](uint64_t v) {
            const uint64_t key = ((uint64_t)(maxl - ((uint32_t)(v >> 32) & 0xFFFFu)) << (2 * pb)) |
                                 ((uint64_t)((uint32_t)v >> 16) << pb) | ((uint32_t)v & 0xFFFFu);
            return (uint32_t)(key >> (p * kMaxDigit)) & (kDigits - 1u);
          },
          [=](uint32_t k, uint32_t r) { reinterpret_cast<uint16_t *>(rec)[4 * k + 3] = (uint16_t)r; },
          [=](uint64_t v, uint32_t) { return (uint32_t)(v >> 48); });
  }
  auto rstart = [=](uint32_t k) { return (uint32_t)reinterpret_cast<const uint16_t *>(rec)[4 * k]; };
  auto rlen = [=](uint32_t k) { return (uint32_t)reinterpret_cast<const uint16_t *>(rec)[4 * k + 2]; };
  auto same_row = [=](uint32_t k, uint32_t q) {  // equal length and ID
    return (((rec[k] ^ rec[q]) >> 16) & 0xFFFFFFFFull) == 0;
  };
  stamp(5);

  // ---- greedy selection in priority order over a bitmap of accepted
  // positions.  The workgroup drops the candidates of a chunk with a marked end
  // (exact: every interval accepted before is at least as long) and exact
  // duplicates; the first wavefront walks the few that are left, 64 at a time:
  // the lowest passing lane is accepted and knocks out the later lanes that
  // overlap it.  Chunks double from 64 candidates, since early ones are long
  // and reject most of the rest.
  uint16_t *surv = cnt, *acc = rc;
  static_assert(NT <= NW * kDigits, "a chunk's survivors fit the radix counters");
  {
    uint32_t chunk = 64;
#pragma unroll 1
    for (uint32_t p0 = 0; p0 < C; p0 += chunk, chunk = min(2 * chunk, (uint32_t)NT)) {
      const uint32_t k = p0 + tid;
      bool ok = false, dup = false;
      if (tid < chunk && k < C) {
        const uint64_t v = rec[k];
        dup = k && ((rec[k - 1] ^ v) << 16) == 0;
        const uint32_t s = (uint32_t)v & 0xFFFFu, e = s + ((uint32_t)(v >> 32) & 0xFFFFu) - 1u;
        ok = !dup && !((bitmap[s >> 5] >> (s & 31)) & 1u) && !((bitmap[e >> 5] >> (e & 31)) & 1u);
      }
      const uint64_t m = __ballot(ok), md = __ballot(dup);
      if (lane == 0) {
        wsum[wv] = (uint32_t)__popcll(m);
        if (md) atomicAdd(&s_dup, (uint32_t)__popcll(md));
      }
      __syncthreads();
      uint32_t tot;
      const uint32_t before = words_before<NW>(wsum, wv, tot);
      if (ok) surv[before + lanes_below(m)] = (uint16_t)(k - p0);
      __syncthreads();
      if (wv == 0 && tot) {
        const uint32_t na = greedy_walk(
            bitmap, tot, s_acc,
            [=](uint32_t q) {
              const uint32_t k = p0 + surv[q];
              return rstart(k) | (rlen(k) << 16);
            },
            [=](uint32_t o, uint32_t q) { acc[o] = (uint16_t)(p0 + surv[q]); });
        if (lane == 0) s_acc = na;
      }
      __syncthreads();
    }
  }
  const uint32_t A = s_acc, M = C - s_dup;
  uint32_t nhist = 1;  // doubling rounds: up to the first that leaves nothing grouped
  while (s_hist[nhist - 1]) nhist++;
  stamp(6);

  // ---- rows: occurrence o opens one when its length or ID differs from the
  // one before; its count is the distance to the next opening
  uint32_t nrows = 0;
#pragma unroll 1
  for (uint32_t o0 = 0; o0 < A; o0 += NT) {
    const uint32_t o = o0 + tid;
    const bool open = o < A && (o == 0 || !same_row(acc[o], acc[o - 1]));
    const uint64_t m = __ballot(open);
    if (lane == 0) {
      if (o0 + 64 * wv < A) {
        bitmap[(o0 >> 5) + 2 * wv] = (uint32_t)m;
        bitmap[(o0 >> 5) + 2 * wv + 1] = (uint32_t)(m >> 32);
      }
      atomicAdd(&s_nd, (uint32_t)__popcll(m));  // holds D until here, which all have read
    }
  }
  __syncthreads();
  nrows = s_nd - D;
  if (nrows <= a.row_cap && (!a.occ || A <= a.occ_cap)) {
    Row *rows = a.rows + (a.off ? tb / a.min_len : 0);
    uint32_t done = 0;  // openings in the words before
#pragma unroll 1
    for (uint32_t o0 = 0; o0 < A; o0 += NT) {
      const uint32_t o = o0 + tid;
      // openings up to o's word: the words of this pass below it
      uint32_t pre = done, tot = 0;
      for (uint32_t w = 0; w < 2 * NW && o0 + 32 * w < A; w++) {  // scalar
        const uint32_t c = (uint32_t)__popc(bitmap[(o0 >> 5) + w]);
        pre += w < (tid >> 5) ? c : 0u;
        tot += c;
      }
      done += tot;
      if (o >= A) continue;
      const uint32_t word = bitmap[o >> 5], k = acc[o];
      const uint32_t r = pre + (uint32_t)__popc(word & (2u << (o & 31)) - 1u) - 1u;
      if ((word >> (o & 31)) & 1u) {
        uint32_t next = word & ~((2u << (o & 31)) - 1u), x = o >> 5;
        while (!next && 32 * (x + 1) < A) next = bitmap[++x];
        rows[r] = Row{rstart(k), rlen(k), (next ? 32 * x + (uint32_t)__ffs((int)next) - 1u : A) - o};
      }
      if (a.occ) a.occ[o] = Occ{rstart(k), rlen(k), r};
    }
  }
  if (tid == 0) {
    stamp(7);
    // at most 8192 distinct pairs in a window of 8192 tokens
    report(a, win, Report{D, D - s_top, C, s_skip, maxl, M, A, nrows, 0, nhist}, s_hist, s_stamp);
  }
}

// ------------------------------------------------------------ longer windows
// The same analysis by one workgroup for windows of up to kFusedLongMax tokens:
// LDS holds the one array that a stage reads at random (token ranks, suffix
// ranks or LCP values, two bytes per token), the others pass through the
// window's share of the workspace, in order or scattered within it, which one
// L2 holds.
constexpr int kLongNT = 1024, kLongNW = kLongNT / 64;
constexpr int kByte = 256;                    // radix digits of 8 bits
constexpr uint64_t kFree = ~0ull;

struct LongArgs {
  FusedArgs f;
  uint16_t *txt, *sa, *rank, *lcp;  // two bytes per token, four bytes apart per window: base + 2 * offset
  uint64_t *e0, *e1;                // two words per token
  uint64_t *flags;                  // one word per token (n / 32 of them used)
  uint8_t *again;                   // batches in two launches (else null): the windows that the first one left
};

// Rank of each lane among the items of its digit d < 256 that the wavefront has
// met, `my` counting them (in: the lanes that hold an item).
template <class Cnt>
__device__ __forceinline__ uint32_t rank_lanes(Cnt *my, uint32_t d, uint64_t in) {
  const uint64_t same = equal_lanes<8>(d, in);
  const uint32_t before = lanes_below(same);
  const uint32_t prev = my[d];
  wave_order();  // every lane has read before the first one of each digit writes
  if (before == 0 && ((in >> (threadIdx.x & 63)) & 1ull)) my[d] = (Cnt)(prev + (uint32_t)__popcll(same));
  wave_order();
  return prev + before;
}

// Ranks a wavefront's items [beg, end) among its items of equal digit, in order
// (lanes of equal digit found by one ballot per bit, running counts in the
// wavefront's row of ctr): park(k, rank).  One LDS atomic per item took longer
// than this, 22 us against 10 for 30011 items, since most lanes meet on a few
// digits of a repetitive window.
template <int U, class Cnt, class Get, class Digit, class Park>
__device__ __forceinline__ void byte_rank(Cnt *my, uint32_t beg, uint32_t end, Get get, Digit digit, Park park) {
  const uint32_t lane = threadIdx.x & 63;
#pragma unroll 1
  for (uint32_t q0 = beg; q0 < end; q0 += 64 * U) {  // scalar
    decltype(get(0u)) v[U];
#pragma unroll
    for (int u = 0; u < U; u++) v[u] = get(min(q0 + 64 * u + lane, end - 1));
#pragma unroll
    for (int u = 0; u < U; u++) {
      const uint32_t q = q0 + 64 * u;
      if (q >= end) continue;  // scalar
      const uint32_t r = rank_lanes(my, digit(v[u]), first_lanes(end - q));
      if (q + lane < end) park(q + lane, r);
    }
  }
}

// Rows of counts into first places: digit by digit, wavefront by wavefront.
template <class Cnt>
__device__ __forceinline__ void byte_scan(Cnt *ctr, uint32_t *wsum) {
  const uint32_t tid = threadIdx.x, wv = wave_id();
  __syncthreads();
  uint32_t tot = 0, inc = 0;
  if (wv < kByte / 64) {
#pragma unroll 4
    for (int w = 0; w < kLongNW; w++) tot += ctr[w * kByte + tid];
    inc = lane_incl_sum(tot);
    if ((tid & 63) == 63) wsum[wv] = inc;
  }
  __syncthreads();
  if (wv < kByte / 64) {
    uint32_t base = inc - tot;
    for (uint32_t w = 0; w < wv; w++) base += wsum[w];
#pragma unroll 4
    for (int w = 0; w < kLongNW; w++) {
      const uint32_t c = ctr[w * kByte + tid];
      ctr[w * kByte + tid] = (Cnt)base;
      base += c;
    }
  }
  __syncthreads();
}

// Moves a wavefront's items to their places: put(place, item).
template <int U, class Cnt, class Get, class Digit, class Parked, class Put>
__device__ __forceinline__ void byte_move(const Cnt *my, uint32_t beg, uint32_t end, Get get, Digit digit,
                                          Parked parked, Put put) {
  const uint32_t lane = threadIdx.x & 63;
#pragma unroll 1
  for (uint32_t q0 = beg; q0 < end; q0 += 64 * U) {  // scalar
    decltype(get(0u)) v[U];
    uint32_t r[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const uint32_t k = min(q0 + 64 * u + lane, end - 1);
      v[u] = get(k);
      r[u] = parked(k);
    }
#pragma unroll
    for (int u = 0; u < U; u++)
      if (q0 + 64 * u + lane < end) put(my[digit(v[u])] + r[u], v[u]);
  }
}

// c[r]++; its value before.  The lanes of a run of one token all meet on one
// word: one of them adds for all.
__device__ __forceinline__ uint32_t count_in(uint32_t *c, uint32_t r) {
  const uint64_t act = __ballot(1);
  if (__ballot(r != (uint32_t)__builtin_amdgcn_readfirstlane((int)r)) != 0) return atomicAdd(&c[r], 1u);
  const uint32_t mine = lanes_below(act);
  uint32_t old = 0;
  if (mine == 0) old = atomicAdd(&c[r], (uint32_t)__popcll(act));
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)old) + mine;
}

// LDS of a longer window.  big holds, one after the other: the distinct tokens'
// table, their sorted list (64 KB) and ranks by slot; token ranks; suffix ranks;
// token ranks; LCP values; the survivors of a chunk of candidates.
template <uint32_t CAP>
struct LongLds {
  static constexpr uint32_t kSlots = CAP / 4;  // hash table of the distinct tokens
  static constexpr uint32_t kDistinct = CAP == kFusedLongMax ? 8192 : CAP / 16 * 3;  // most of them (the largest value aside)
  // a radix counter counts 2 * (CAP - 1) records at most
  using Cnt = std::conditional_t<(CAP > 32768), uint32_t, uint16_t>;
  alignas(16) unsigned char big[CAP * 2];
  alignas(16) Cnt ctr[kLongNW * kByte];           // radix counters; LCP minima of 8; run openings
  alignas(16) uint32_t bitmap[CAP / 32 + 2];      // as in ShortLds; LCP minima of 64 and 512
  uint32_t wsum[kLongNW], wsum2[kLongNW];
  uint32_t s_nd, s_top, s_over, s_zero, s_active, s_left, s_eighths, s_max, s_skip, s_c, s_acc, s_dup, s_pairs;
  uint32_t s_hist[kLongRounds];
  uint64_t s_stamp[kStages + 1];
  unsigned long long s_differ;
};

// FIRST: leaves a window of too many distinct tokens to the other launch.  LEAVE (see
// k_window_any): gives up a window that keeps its suffixes grouped.
template <uint32_t CAP, bool FIRST, bool LEAVE>
__device__ __forceinline__ void window_long(const LongArgs &la, LongLds<CAP> &L, uint32_t win, uint64_t tb, uint32_t n) {
  constexpr int NT = kLongNT, NW = kLongNW;
  constexpr int U = CAP > kFusedMidMax ? 8 : 4;  // steps whose reads are issued together
  constexpr uint32_t kSlots = LongLds<CAP>::kSlots, kDistinct = LongLds<CAP>::kDistinct;
  const FusedArgs &a = la.f;
  auto &big = L.big;
  auto &ctr = L.ctr;
  auto &bitmap = L.bitmap;
  auto &wsum = L.wsum;
  auto &wsum2 = L.wsum2;
  auto &s_nd = L.s_nd, &s_top = L.s_top, &s_over = L.s_over, &s_zero = L.s_zero, &s_active = L.s_active;
  auto &s_max = L.s_max, &s_skip = L.s_skip, &s_c = L.s_c, &s_acc = L.s_acc, &s_dup = L.s_dup, &s_pairs = L.s_pairs;
  auto &s_hist = L.s_hist;
  auto &s_stamp = L.s_stamp;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wv = wave_id();
  const uint64_t below = (1ull << lane) - 1ull;
  uint16_t *const gtxt = la.txt + 2 * tb, *const gsa = la.sa + 2 * tb, *const grank = la.rank + 2 * tb,
                 *const glcp = la.lcp + 2 * tb;
  uint64_t *const e0 = la.e0 + 2 * tb, *const e1 = la.e1 + 2 * tb, *const fl = la.flags + tb;
  auto stamp = [&](int k) {
    if (tid == 0) s_stamp[k] = wall_clock64();
  };
  stamp(0);
  // a wavefront's share of m items, in order
  auto seg = [](uint32_t m) { return ((m + 64 * kLongNW - 1) / (64 * kLongNW)) * 64; };
  typename LongLds<CAP>::Cnt *const my = ctr + wv * kByte;
  // ranks parked between the two halves of a radix pass (the LCP values come
  // later, and are in LDS when the candidates are sorted)
  uint16_t *const rel = glcp;
  auto park = [=](uint32_t k, uint32_t r) { rel[k] = (uint16_t)r; };
  auto parked = [=](uint32_t k) { return (uint32_t)rel[k]; };
  auto clear_row = [&] {
    if constexpr (sizeof(*my) == 4) *reinterpret_cast<uint4 *>(my + 4 * lane) = make_uint4(0, 0, 0, 0);
    else *reinterpret_cast<uint2 *>(my + 4 * lane) = make_uint2(0, 0);
    wave_order();
  };

  // An LDS hash table of distinct words, listed in e1 as they turn up, each with
  // its slot; kFree marks free slots.
  unsigned long long *const tab = reinterpret_cast<unsigned long long *>(big);
  uint16_t *const slot = reinterpret_cast<uint16_t *>(e0);      // of every token
  uint16_t *const dslot = reinterpret_cast<uint16_t *>(e1 + n);  // of every distinct word
  auto clear_table = [&] {
    if (tid == 0) s_nd = s_over = 0;
    for (uint32_t k = 2 * tid; k < kSlots; k += 2 * NT) *reinterpret_cast<ulonglong2 *>(tab + k) = make_ulonglong2(kFree, kFree);
    __syncthreads();
  };
  auto insert = [&](uint64_t key) -> uint32_t {
    uint32_t at = (uint32_t)(mix64(key) >> 40) & (kSlots - 1);
    for (int probe = 0;; probe++) {
      if (probe == (int)kSlots) {  // full (only past the limit)
        s_over = 1;
        break;
      }
      unsigned long long cur = tab[at];
      if (cur == kFree) {
        cur = atomicCAS(&tab[at], (unsigned long long)kFree, (unsigned long long)key);
        if (cur == kFree) {
          const uint32_t q = atomicAdd(&s_nd, 1u);
          if (q < kDistinct) {
            e1[q] = key;
            dslot[q] = (uint16_t)at;
          } else {
            s_over = 1;
          }
          break;
        }
      }
      if (cur == key) break;
      at = (at + 1) & (kSlots - 1);
    }
    return at;
  };
  // Sorts the table's d words; srank: their ranks from 1, by slot.
  uint16_t *const srank = reinterpret_cast<uint16_t *>(big + kDistinct * 8);
  auto rank_by = [&](auto per, uint32_t d) {
    constexpr int R = decltype(per)::value;
    uint64_t *sorted = reinterpret_cast<uint64_t *>(big);
    uint64_t x[R];
#pragma unroll
    for (int i = 0; i < R; i++) {
      const uint32_t q = tid * R + i;
      x[i] = q < d ? e1[q] : ~0ull;
    }
    merge_sort<NT, R>(x, sorted, d);  // the table's last reads are a barrier behind
#pragma unroll 1
    for (uint32_t q = tid; q < d; q += NT) {
      const uint64_t key = e1[q];
      uint32_t lo = 0, hi = d - 1;  // sorted[lo .. hi] holds it
      while (lo < hi) {
        const uint32_t mid = (lo + hi) / 2;
        if (sorted[spread<R>(mid)] < key) lo = mid + 1;
        else hi = mid;
      }
      srank[dslot[q]] = (uint16_t)(lo + 1);
    }
    __syncthreads();
  };
  // as few words a thread as hold them all: a merge's steps are one thread's
  // outputs after another (1112 words: 25 us eight a thread, 13 two a thread)
  auto rank_table = [&](uint32_t d) {
    if (d <= NT) rank_by(std::integral_constant<int, 1>{}, d);
    else if (d <= 2 * NT) rank_by(std::integral_constant<int, 2>{}, d);
    else if (d <= 4 * NT) rank_by(std::integral_constant<int, 4>{}, d);
    else rank_by(std::integral_constant<int, 8>{}, d);
  };

  // ---- token ranks: the distinct values through the table (the largest value
  // a token can have, which marks free slots, aside)
  {
    if (tid == 0) s_top = s_skip = s_max = s_c = s_acc = s_dup = s_pairs = 0;
    if (tid < kLongRounds) s_hist[tid] = 0;
    clear_table();
#pragma unroll 1
    for (uint32_t k0 = tid; k0 < n; k0 += 8 * NT) {
      uint64_t v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const uint64_t k = tb + min(k0 + u * NT, n - 1);
        v[u] = a.bits == 64 ? static_cast<const uint64_t *>(a.tok)[k] : (uint64_t) static_cast<const uint32_t *>(a.tok)[k];
      }
      if (*(volatile uint32_t *)&s_over) break;  // this window is not for this kernel
#pragma unroll
      for (int u = 0; u < 8; u++) {
        if (k0 + u * NT >= n) break;
        uint32_t at = kSlots;
        if (v[u] == kFree) s_top = 1;
        else at = insert(v[u]);
        slot[k0 + u * NT] = (uint16_t)at;
      }
    }
    __syncthreads();
    if constexpr (FIRST) {
      if (tid == 0) la.again[win] = s_over ? 1 : 0;
      if (s_over) return;  // uniform: left to the larger table
    }
  }
  uint32_t nd, D;
  const bool by_table = !s_over;  // uniform
  bool by_first = false;          // uniform: sorted by one token already
  if (by_table) {
    nd = s_nd;
    D = nd + s_top;
    rank_table(nd);
#pragma unroll 4
    for (uint32_t k = tid; k < n; k += NT) {
      const uint32_t at = slot[k];
      gtxt[k] = (uint16_t)(at == kSlots ? D : srank[at]);
    }
    __syncthreads();
  } else {
    // More distinct tokens than the table takes: positions sorted by token, a
    // radix pass for each of the four highest bytes in which the tokens differ
    // (then for all of them, should that not have put them in order), ranks
    // counted over the sorted positions.  A lone window's host tokens are read from
    // pinned memory in every pass (32768 distinct ones: the call 510 us, from the device 440,
    // stage by stage 620).
    auto token = [=](uint32_t j) {
      return a.bits == 64 ? static_cast<const uint64_t *>(a.tok)[tb + j] : (uint64_t) static_cast<const uint32_t *>(a.tok)[tb + j];
    };
    uint32_t *src = reinterpret_cast<uint32_t *>(e0), *dst = reinterpret_cast<uint32_t *>(e1);
    const uint32_t kbeg = min(wv * seg(n), n), ktop = min(kbeg + seg(n), n);
    uint64_t differ = 0;
    for (uint32_t k = kbeg + lane; k < ktop; k += 64) {
      differ |= token(k) ^ token(0);
      src[k] = k;
    }
    if (tid == 0) L.s_differ = 0;
    __syncthreads();
    if (differ) atomicOr(&L.s_differ, (unsigned long long)differ);
    __syncthreads();
    differ = L.s_differ;
    int low = 0;  // the lowest byte sorted by
    for (int sh = a.bits - 8, many = 0; sh >= 0; sh -= 8)
      if ((differ >> sh) & 255u)
        if (++many == 4) low = sh;
    uint32_t opened;
    for (;;) {  // uniform; twice at most
#pragma unroll 1
      for (int sh = low; sh < a.bits; sh += 8) {
        if (!((differ >> sh) & 255u)) continue;  // uniform
        const uint32_t *from = src;
        uint32_t *to = dst;
        auto get = [=](uint32_t k) {
          const uint32_t j = from[k];
          return j | ((uint32_t)(token(j) >> sh) & 255u) << 16;
        };
        auto dig = [](uint32_t v) { return v >> 16; };
        clear_row();
        byte_rank<U>(my, kbeg, ktop, get, dig, park);
        byte_scan(ctr, wsum);
        byte_move<U>(my, kbeg, ktop, get, dig, parked, [=](uint32_t at, uint32_t v) { to[at] = v & 0xFFFFu; });
        __syncthreads();
        dst = src;
        src = to;
      }
      if (tid == 0) s_active = 0;
      __syncthreads();
      opened = 0;
#pragma unroll 1
      for (uint32_t k0 = kbeg; k0 < ktop; k0 += 64) {  // scalar
        const uint32_t k = min(k0 + lane, n - 1);
        const uint64_t t = token(src[k]), pt = token(src[k ? k - 1 : 0]);
        if (pt > t) s_active = 1;
        const uint64_t open = __ballot(k0 + lane < ktop && (k == 0 || pt != t));
        if (lane == 0) fl[k0 >> 6] = open;
        opened += (uint32_t)__popcll(open);
      }
      if (lane == 0) wsum[wv] = opened;
      __syncthreads();
      if (!s_active || low == 0) break;  // uniform
      low = 0;
    }
    uint32_t at = words_before<NW>(wsum, wv, D);
    nd = D;
    if (D > 65535) {  // uniform: kFusedLongMax distinct tokens, more ranks than 16 bits hold, and no repeats
      if (tid == 0) {
        for (int k = 1; k <= kStages; k++) stamp(k);
        report(a, win, Report{D, D, 0, 0, 0, 0, 0, 0, n, 1}, s_hist, s_stamp);
      }
      return;
    }
    // mostly distinct ones: the positions are as good as sorted, groups of one token in them
    by_first = 2 * D >= n;
#pragma unroll 1
    for (uint32_t k0 = kbeg; k0 < ktop; k0 += 64) {  // scalar
      const uint64_t open = fl[k0 >> 6];
      const uint32_t j = src[min(k0 + lane, n - 1)];
      if (k0 + lane < ktop) {
        gtxt[j] = (uint16_t)(at + (uint32_t)__popcll(open & (below | (1ull << lane))));
        if (by_first) {
          gsa[k0 + lane] = (uint16_t)j;
          if (j == 0) s_zero = k0 + lane;
        }
      }
      at += (uint32_t)__popcll(open);
      if (lane == 0) {
        const uint64_t hd = open | ~first_lanes(n - k0);  // as below
        bitmap[k0 >> 5] = (uint32_t)hd;
        bitmap[(k0 >> 5) + 1] = (uint32_t)(hd >> 32);
      }
    }
    if (tid == 0 && n % 64 == 0) bitmap[n >> 5] = 1;
    __syncthreads();
  }
  auto load_lds = [&](const uint16_t *from) {  // n words, four a lane (windows start 4-byte aligned: two 4-byte loads)
    uint32_t *to = reinterpret_cast<uint32_t *>(big);
    const uint32_t *g = reinterpret_cast<const uint32_t *>(from);
#pragma unroll 4
    for (uint32_t k = tid; k < (n + 1) / 2; k += NT) to[k] = g[k];
    __syncthreads();
  };
  uint16_t *const txt = reinterpret_cast<uint16_t *>(big);
  uint16_t *const rank = reinterpret_cast<uint16_t *>(big);  // rank[j]: the first slot of j's group
  stamp(1);

  // ---- suffix array: every suffix first sorted by its first h tokens.  A
  // repetitive window holds few distinct words of h tokens (up to 63 bits;
  // kLongPack tokens at most): those go through the table as the tokens did, and
  // the suffixes are counted into their places (20000 tokens of a loop with 5 %
  // substitutions, 4725 words of 5: 68 us against 122 for six radix passes).  How
  // many there will be is told from the first 2048 positions and then from the second 8192
  // against the first: too many, h is lowered in proportion; mostly new ones, or
  // too many after all, and a radix sort takes as many tokens as fit above the
  // position in a 64-bit word.  So it does at once where that is three passes or
  // fewer (windows over a handful of tokens).
  const int tbits = bits_of(D);
  // (a rare token spoils h words: with mostly rare ones there are some 0.75 h D)
  uint32_t h = min(min((uint32_t)(63 / tbits), kLongPack), max(2u, kDistinct * 13 / (10 * D)));
  const uint32_t wbeg = min(wv * seg(n), n), wtop = min(wbeg + seg(n), n);  // the wavefront's tokens and slots
  bool named = !by_first && h >= 2 && min(48 / tbits, (int)kLongPack) * tbits > 24;
  bool lowered = false;
  while (named) {  // uniform; at most twice
    clear_table();
    uint32_t seen = 0, lower = 0;
#pragma unroll 1
    for (uint32_t t0 = 0; t0 < n;) {
      const uint32_t t1 = min(t0 ? t0 + 8 * NT : 2 * NT, n);
      uint64_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 1
      for (uint32_t q = 0; q < h; q++)
#pragma unroll
        for (int u = 0; u < 8; u++) {
          const uint32_t k = t0 + u * NT + tid;
          v[u] = (v[u] << tbits) | (k < t1 && k + q < n ? gtxt[k + q] : 0u);
        }
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const uint32_t k = t0 + u * NT + tid;
        if (k < t1) slot[k] = (uint16_t)insert(v[u]);
      }
      __syncthreads();
      const uint32_t now = s_nd;
      if (now > (t0 ? kDistinct : NT + NT / 4)) {
        named = false;
        break;
      }
      if (t0 == 2 * NT && !lowered) {
        const uint64_t end = now + (uint64_t)(now - seen) * (n - t1) / (t1 - t0);
        if (end > kDistinct) {
          lower = (uint32_t)(h * (uint64_t)(kDistinct - kDistinct / 8) / end);
          named = lower >= 2;
          break;
        }
      }
      __syncthreads();  // s_nd is read before it grows
      seen = now;
      t0 = t1;
    }
    __syncthreads();
    if (!lower) break;
    h = lower;
    lowered = true;
  }
  if (named) {
    const uint32_t d = s_nd;
    rank_table(d);
    uint32_t *const cnt = reinterpret_cast<uint32_t *>(big);  // the sorted list is done with
    uint32_t *const cur = cnt + kDistinct;
    static_assert(kDistinct * 8 + kSlots * 2 <= sizeof(L.big), "sorted list, or counts and cursors; ranks");
    for (uint32_t q = tid; q < kDistinct; q += NT) cnt[q] = 0;
    for (uint32_t x = tid; x <= n / 32 + 1; x += NT) bitmap[x] = 0;
    __syncthreads();
#pragma unroll 4
    for (uint32_t k = tid; k < n; k += NT) (void)count_in(cnt, srank[slot[k]] - 1u);
    __syncthreads();
    {
      constexpr int R = kDistinct / NT;
      uint32_t c[R], tot = 0, all;
#pragma unroll
      for (int i = 0; i < R; i++) tot += c[i] = cnt[tid * R + i];
      const uint32_t inc = lane_incl_sum(tot);
      if (lane == 63) wsum[wv] = inc;
      __syncthreads();
      uint32_t base = words_before<NW>(wsum, wv, all) + inc - tot;
#pragma unroll
      for (int i = 0; i < R; i++) {
        cnt[tid * R + i] = cur[tid * R + i] = base;
        if (c[i]) atomicOr(&bitmap[base >> 5], 1u << (base & 31));
        base += c[i];
      }
    }
    // the slots from n to the end of its 64 (slot n itself at least) count as openings
    if (tid == 0) {
      const uint64_t up = ~0ull << (n & 63);
      atomicOr(&bitmap[(n >> 6) * 2], n % 64 == 0 ? 1u : (uint32_t)up);
      if (n % 64) atomicOr(&bitmap[(n >> 6) * 2 + 1], (uint32_t)(up >> 32));
    }
    __syncthreads();
#pragma unroll 4
    for (uint32_t k = tid; k < n; k += NT) {
      const uint32_t r = srank[slot[k]] - 1u;
      const uint32_t at = count_in(cur, r);
      grank[k] = (uint16_t)cnt[r];
      gsa[at] = (uint16_t)k;
      if (k == 0) s_zero = at;
    }
    __syncthreads();
    load_lds(grank);
  } else if (!by_first) {
    load_lds(gtxt);
    h = min((uint32_t)(48 / tbits), kLongPack);
    auto key_of = [&](uint32_t j) {
      uint64_t key = 0;
#pragma unroll 1
      for (uint32_t q = 0; q < h; q++) key = (key << tbits) | (j + q < n ? txt[j + q] : 0u);
      return (key << 16) | j;
    };
    const int np = ((int)h * tbits + 7) / 8;
    uint64_t *src = e0, *dst = e1;
    for (uint32_t k = wbeg + lane; k < wtop; k += 64) src[k] = key_of(k);  // read back by the same wavefront
#pragma unroll 1
    for (int p = 0; p < np; p++) {
      const int sh = 16 + 8 * p;
      auto get = [=](uint32_t k) { return src[k]; };
      auto dig = [=](uint64_t v) { return (uint32_t)(v >> sh) & 255u; };
      clear_row();
      byte_rank<U>(my, wbeg, wtop, get, dig, park);
      byte_scan(ctr, wsum);
      uint64_t *to = dst;
      byte_move<U>(my, wbeg, wtop, get, dig, parked, [=](uint32_t at, uint64_t v) { to[at] = v; });
      __syncthreads();
      dst = src;
      src = to;
    }
    // groups: a bitmap of the slots that open one (slot n counts as one)
#pragma unroll 1
    for (uint32_t k0 = wbeg; k0 < wtop; k0 += 64) {  // scalar
      const uint32_t k = min(k0 + lane, n - 1);
      const uint64_t key = src[k], prev = src[k ? k - 1 : 0];
      const uint32_t j = (uint32_t)key & 0xFFFFu;
      if (k0 + lane < n) gsa[k] = (uint16_t)j;
      if (j == 0) s_zero = k;
      const uint64_t hd = __ballot(k0 + lane == 0 || k0 + lane >= n || (prev >> 16) != (key >> 16));
      if (lane == 0) {
        bitmap[k0 >> 5] = (uint32_t)hd;
        bitmap[(k0 >> 5) + 1] = (uint32_t)(hd >> 32);
      }
    }
    if (tid == 0 && n % 64 == 0) bitmap[n >> 5] = 1;
    __syncthreads();
  } else {
    h = 1;
  }
  // (both are read into registers here: the first thread sets the words again at the next survey, which has to be
  // behind a barrier of its own)
  uint32_t active;
  bool left = false;  // another window has left
  auto survey = [&] {
    if (tid == 0) {
      s_active = 0;
      if constexpr (LEAVE) L.s_left = __hip_atomic_load(part_of(a) + CNT_WFLAG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    uint32_t more = 0;
    for (uint32_t x = tid; 32 * x < n; x += NT) {
      const uint32_t w = bitmap[x], up = 32 * x + 32 <= n ? bitmap[x + 1] : kNone;
      more += (uint32_t)__popc(~(w & ((w >> 1) | (up << 31))) & (uint32_t)first_lanes(n - 32 * x));
    }
    more = lane_incl_sum(more);
    if (lane == 63 && more) atomicAdd(&s_active, more);
    __syncthreads();
    active = s_active;
    if constexpr (LEAVE) left = L.s_left != 0;
  };
  auto leave = [&] {
    if (tid == 0) {
      a.win_rows[win] = 0;
      atomicAdd(&part_of(a)[CNT_WFLAG], 1u);
    }
  };
  if constexpr (LEAVE) {  // (before the loop below, which goes back to the opening of a group for each of its suffixes)
    survey();
    // the eighths of the slots in which some group opens
    if (tid == 0) L.s_eighths = 0;
    __syncthreads();
    uint32_t m = 0;
    for (uint32_t x = tid; 32 * x < n; x += NT)
      if (bitmap[x]) m |= 1u << (256 * x / n);
    if (m) atomicOr(&L.s_eighths, m);
    __syncthreads();
    if (left || (n > kFusedLone && (active > n - n / 256 * h || L.s_eighths != 0xFFu))) {  // uniform
      leave();
      return;
    }
  }
  if (!named)
#pragma unroll 4
    for (uint32_t k = tid; k < n; k += NT) {
      uint32_t x = k >> 5, w = bitmap[x] & ((2u << (k & 31)) - 1u);
      while (!w) w = bitmap[--x];  // slot 0 opens a group
      rank[gsa[k]] = (uint16_t)(32 * x + 31u - (uint32_t)__clz((int)w));
    }
  if (tid == 0) s_nd = nd;  // (the rows are counted from there)
  survey();

  // Prefix doubling of the suffixes still grouped, listed in the order of their
  // second halves and sorted stably by the group of the first half (window_short's
  // second form): j | group << 16
  {
    uint32_t *const l0 = reinterpret_cast<uint32_t *>(e0), *const l1 = reinterpret_cast<uint32_t *>(e1);
#pragma unroll 1
    while (active && h < n) {  // uniform
      const uint32_t first = s_zero, m = active;
      uint32_t mine = 0;
#pragma unroll 1
      for (uint32_t k0 = wbeg; k0 < wtop; k0 += 256) {  // scalar
        uint32_t s[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
          const uint32_t k = min(k0 + 64 * u + lane, n - 1);
          s[u] = gsa[k == 0 ? first : k <= first ? k - 1 : k];
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
          if (k0 + 64 * u >= wtop) continue;  // scalar
          const uint32_t j = s[u] >= h ? s[u] - h : s[u] + n - h;
          const uint32_t g = rank[j];
          const uint64_t mk =
              __ballot(!((bitmap[(g + 1) >> 5] >> ((g + 1) & 31)) & 1u)) & first_lanes(wtop - k0 - 64 * u);
          if ((mk >> lane) & 1ull) l0[wbeg + mine + lanes_below(mk)] = j | (g << 16);
          mine += (uint32_t)__popcll(mk);
        }
      }
      // the wavefront's own entries first, then an even share of them all
      auto low = [](uint32_t e) { return (e >> 16) & 255u; };
      clear_row();
      byte_rank<U>(my, wbeg, wbeg + mine, [=](uint32_t q) { return l0[q]; }, low, park);
      byte_scan(ctr, wsum);
      byte_move<U>(
          my, wbeg, wbeg + mine, [=](uint32_t q) { return l0[q]; }, low, parked,
          [=](uint32_t at, uint32_t e) { l1[at] = e; });
      __syncthreads();
      const uint32_t qbeg = min(wv * seg(m), m), qtop = min(qbeg + seg(m), m);
      auto get = [=](uint32_t q) { return l1[q]; };
      auto dig = [](uint32_t e) { return e >> 24; };
      clear_row();
      byte_rank<U>(my, qbeg, qtop, get, dig, park);
      byte_scan(ctr, wsum);
      byte_move<U>(my, qbeg, qtop, get, dig, parked, [=](uint32_t at, uint32_t e) { l0[at] = e; });
      __syncthreads();
      // openings of old and new groups among the sorted entries
      uint32_t lo = kNone, ln = kNone;
#pragma unroll 1
      for (uint32_t q0 = qbeg; q0 < qtop; q0 += 256) {  // scalar
        uint32_t e[4];
#pragma unroll
        for (int u = 0; u < 4; u++) e[u] = l0[min(q0 + 64 * u + lane, m - 1)];
#pragma unroll
        for (int u = 0; u < 4; u++) {
          const uint32_t c0 = q0 + 64 * u, q = c0 + lane;
          if (c0 >= qtop) continue;  // scalar
          auto half = [&](uint32_t e) {  // the second half's group, 0 for the empty one (one past the end)
            const uint32_t s = (e & 0xFFFFu) + h, r = rank[min(s, n - 1)];
            return s < n ? r + 1 : 0u;
          };
          const uint32_t c = half(e[u]);
          uint32_t pe = lane_prev(e[u]), pc = lane_prev(c);
          if (lane == 0 && q) {
            pe = l0[q - 1];
            pc = half(pe);
          }
          const bool og = q == 0 || q >= m || (e[u] >> 16) != (pe >> 16);
          const bool ng = og || c != pc;
          const uint64_t mo = __ballot(og), mn = __ballot(ng), in = first_lanes(qtop - c0);
          if (lane == 0) {
            fl[2 * (c0 >> 6)] = mo;
            fl[2 * (c0 >> 6) + 1] = mn;
          }
          if (mo & in) lo = c0 + 63u - (uint32_t)__clzll((long long)(mo & in));
          if (mn & in) ln = c0 + 63u - (uint32_t)__clzll((long long)(mn & in));
        }
      }
      if (lane == 0) {
        wsum[wv] = lo;
        wsum2[wv] = ln;
      }
      __syncthreads();
      uint32_t co = last_word(wsum, wv), cn = last_word(wsum2, wv);
#pragma unroll 1
      for (uint32_t q0 = qbeg; q0 < qtop; q0 += 64) {  // scalar
        const uint32_t q = q0 + lane, e = l0[min(q, m - 1)];
        const uint64_t in = first_lanes(qtop - q0);
        const uint64_t og = fl[2 * (q0 >> 6)] & in, ng = fl[2 * (q0 >> 6) + 1] & in, upto = below | (1ull << lane);
        if (q < qtop) {
          const uint64_t uo = og & upto, un = ng & upto;
          const uint32_t ob = uo ? q0 + 63u - (uint32_t)__clzll((long long)uo) : co;
          const uint32_t nb = un ? q0 + 63u - (uint32_t)__clzll((long long)un) : cn;
          const uint32_t j = e & 0xFFFFu, g = e >> 16, slot = g + (q - ob);
          gsa[slot] = (uint16_t)j;
          rank[j] = (uint16_t)(g + (nb - ob));
          if (nb == q) atomicOr(&bitmap[slot >> 5], 1u << (slot & 31));
          if (j == 0) s_zero = slot;
        }
        if (og) co = q0 + 63u - (uint32_t)__clzll((long long)og);
        if (ng) cn = q0 + 63u - (uint32_t)__clzll((long long)ng);
      }
      h *= 2;
      survey();  // its first barrier ends the writes above
      if constexpr (LEAVE)
        if (left) {  // uniform
          leave();
          return;
        }
    }
  }
  {
    const uint32_t *from = reinterpret_cast<const uint32_t *>(big);
    uint32_t *g = reinterpret_cast<uint32_t *>(grank);
    for (uint32_t k = tid; k < (n + 1) / 2; k += NT) g[k] = from[k];
    __syncthreads();
  }
  stamp(2);

  // ---- LCP: Kasai's walk as in window_short, over the token ranks; the next
  // position's predecessor is read ahead (two dependent reads a position)
  load_lds(gtxt);
  {
    const uint32_t per = (n + NT - 1) / NT;
    const uint32_t x0 = min(tid * per, n), x1 = min(x0 + per, n);
    auto rank_at = [=](uint32_t x) { return (uint32_t)grank[min(x, n - 1)]; };
    auto before = [=](uint32_t r) { return (uint32_t)gsa[r ? r - 1 : 0]; };
    uint32_t r = rank_at(x0), rn = rank_at(x0 + 1), y = before(r), yn, rnn;
    uint32_t l = first_lcp(txt, x0 < n && r != 0, x0, y, n - (x0 > y ? x0 : y), per);
#pragma unroll 1
    for (uint32_t x = x0; x < x1; x++, r = rn, y = yn, rn = rnn) {
      yn = before(rn);
      rnn = rank_at(x + 2);
      if (r == 0) {
        l = 0;
        continue;
      }
      const uint32_t lim = n - (x > y ? x : y);
      bool differ = false;
      while (!differ && l + 8 <= lim) {
        uint64_t p0, p1, q0, q1;
        __builtin_memcpy(&p0, txt + x + l, 8);
        __builtin_memcpy(&q0, txt + y + l, 8);
        __builtin_memcpy(&p1, txt + x + l + 4, 8);
        __builtin_memcpy(&q1, txt + y + l + 4, 8);
        const uint64_t d0 = p0 ^ q0, d1 = p1 ^ q1;
        differ = (d0 | d1) != 0;
        l += d0 ? (uint32_t)__builtin_ctzll(d0) / 16 : d1 ? 4 + (uint32_t)__builtin_ctzll(d1) / 16 : 8;
      }
      while (!differ && l < lim && txt[x + l] == txt[y + l]) l++;  // fewer than 8 are left
      glcp[r - 1] = (uint16_t)l;
      l = l ? l - 1 : 0;
    }
    if (tid == 0) glcp[n - 1] = 0;
  }
  __syncthreads();
  uint16_t *const lcp = reinterpret_cast<uint16_t *>(big);
  load_lds(glcp);
  uint16_t *const min1 = reinterpret_cast<uint16_t *>(ctr), *const min2 = reinterpret_cast<uint16_t *>(bitmap),
                 *const min3 = min2 + CAP / 64;
  static_assert(CAP / 8 * 2 <= sizeof(ctr) && (CAP / 64 + CAP / 64) * 2 <= sizeof(bitmap), "minima fit");
  if (tid < 8 && n + tid < ((n + 7) & ~7u)) lcp[n + tid] = 0xFFFF;
  for (uint32_t b = tid; b < CAP / 8; b += NT) min1[b] = 0xFFFF;
  for (uint32_t b = tid; b < CAP / 32; b += NT) min2[b] = 0xFFFF;
  __syncthreads();
  stamp(3);

  // ---- candidates, as in window_short
  for (uint32_t b = tid; b < (n + 7) / 8; b += NT) min1[b] = (uint16_t)min8(lcp + 8 * b);
  __syncthreads();
  for (uint32_t b = tid; b < (n + 63) / 64; b += NT) min2[b] = (uint16_t)min8(min1 + 8 * b);
  __syncthreads();
  for (uint32_t b = tid; b < (n + 511) / 512; b += NT) min3[b] = (uint16_t)min8(min2 + 8 * b);
  __syncthreads();
  uint32_t mine = 0;  // the wavefront's records, in suffix-array order from 2 * wbeg on
  {
    uint32_t mx = 0, pairs = 0, skipped = 0, hist = 0;  // hist: lane r's for round r
    // suffixes of 64 slots, read once and one step ahead; the neighbours' from the other lanes
    uint32_t xs = gsa[min(wbeg + lane, n - 1)], wlast = gsa[wbeg ? min(wbeg, n) - 1 : 0], xn;
#pragma unroll 1
    for (uint32_t k0 = wbeg; k0 < wtop; k0 += 64, wlast = (uint32_t)__builtin_amdgcn_readlane((int)xs, 63), xs = xn) {  // scalar
      const uint32_t k = k0 + lane;
      xn = gsa[min(k + 64, n - 1)];
      uint32_t ys = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)xs, 0x130, 0xF, 0xF, false), ws = lane_prev(xs);
      const uint32_t next = (uint32_t)__builtin_amdgcn_readlane((int)xn, 0);
      if (lane == 63) ys = next;
      if (lane == 0) ws = wlast;
      uint32_t l = 0, s1 = 0, s2 = 0, both = 0, pp = 0;
      bool rep = false;
      if (k < n) {
        const uint32_t x = xs, y = k + 1 < n ? ys : x, p = lcp[k], w = k ? ws : x;
        pp = k ? lcp[k - 1] : 0u;
        both = max(p, pp);
        const uint32_t lo = min(x, y), d = max(x, y) - lo;
        const bool disj = p <= d;
        if (disj) {
          l = p;
          s1 = x;
          s2 = y;
        } else {
          l = (p + d) / 2;
          l -= l % d;
          s1 = lo;
          s2 = lo + l;
        }
        if (l < a.min_len || k + 1 == n) l = 0;
        rep = l && disj && k && pp == l && pp <= max(x, w) - min(x, w);
      }
#pragma unroll 1
      for (int r = 0; r < kLongRounds; r++) {
        const uint64_t g = __ballot(both >> r);
        if (!g) break;  // scalar
        hist += lane == (uint32_t)r ? (uint32_t)__popcll(g) : 0u;
      }
      pairs += (uint32_t)__popcll(__ballot(k < n && pp < 2));  // first of its two-token prefix
      const uint64_t m2 = __ballot(l != 0), m1 = __ballot(l != 0 && !rep);
      if (!m2) continue;  // scalar
      const uint64_t id = l ? 1u + last_smaller<CAP>(lcp, min1, min2, min3, k, l) : 0u;
      uint32_t q = 2 * wbeg + mine + lanes_below(m1) + lanes_below(m2);
      if (l) {
        const uint64_t head = (id << 16) | ((uint64_t)l << 32);
        if (!rep) e0[q++] = head | s1;
        e0[q] = head | s2;
      }
      mine += (uint32_t)(__popcll(m1) + __popcll(m2));
      skipped += (uint32_t)(__popcll(m2) - __popcll(m1));
      mx = max(mx, l);
    }
    mx = lane_max(mx);
    if (lane == 63 && mx) atomicMax(&s_max, mx);
    if (hist) atomicAdd(&s_hist[lane], hist);  // lanes below kLongRounds
    if (lane == 0) {
      atomicAdd(&s_pairs, pairs);
      atomicAdd(&s_skip, skipped);
      atomicAdd(&s_c, mine);
    }
  }
  __syncthreads();
  const uint32_t C = s_c, maxl = s_max;
  stamp(4);

  // ---- priority order (length desc, ID asc, start asc).  For one length the
  // ID never decreases along the suffix array, so a stable radix sort by length
  // leaves (length, ID) in order, and each run of equal ones is put in order of
  // the starts: a record's place is the number of its run's records that start
  // before it.  With a long run (128 records or more; up to 190 may pass) the
  // three fields are sorted as one key instead.
  const uint64_t *rec = e0;
  uint64_t *accs = e1;  // accepted records
  if (C) {  // uniform
    const int pb = bits_of(n - 1), lb = bits_of(maxl - a.min_len);
    const uint32_t cbeg = min(wv * seg(C), C), ctop = min(cbeg + seg(C), C);
    uint64_t *src = e0, *dst = e1;
    auto pass = [&](uint32_t beg, uint32_t end, auto dig) {
      const uint64_t *from = src;
      uint64_t *to = dst;
      auto get = [=](uint32_t k) { return from[k]; };
      clear_row();
      byte_rank<U>(my, beg, end, get, dig, park);
      byte_scan(ctr, wsum);
      byte_move<U>(my, beg, end, get, dig, parked, [=](uint32_t at, uint64_t v) { to[at] = v; });
      __syncthreads();
      dst = src;
      src = to;
    };
#pragma unroll 1
    for (int sh = 0; sh == 0 || sh < lb; sh += 8)
      pass(sh ? cbeg : 2 * wbeg, sh ? ctop : 2 * wbeg + mine,
           [=](uint64_t v) { return ((maxl - (uint32_t)(v >> 32)) >> sh) & 255u; });
    // a bitmap of the records that open a run
    uint32_t *const runs = reinterpret_cast<uint32_t *>(ctr);
    static_assert(CAP / 16 * 4 <= sizeof(ctr), "two records a token");
    if (tid == 0) s_active = 0;
#pragma unroll 1
    for (uint32_t q0 = cbeg; q0 < ctop; q0 += 64) {  // scalar
      const uint32_t k = min(q0 + lane, C - 1);
      const uint64_t open = __ballot(q0 + lane == 0 || q0 + lane >= C || (src[k] >> 16) != (src[k ? k - 1 : 0] >> 16));
      if (lane == 0) {
        runs[q0 >> 5] = (uint32_t)open;
        runs[(q0 >> 5) + 1] = (uint32_t)(open >> 32);
      }
    }
    __syncthreads();
    for (uint32_t x = tid; 32 * x + 128 <= C; x += NT)
      if (!(runs[x] | runs[x + 1] | runs[x + 2] | runs[x + 3])) s_active = 1;  // 128 records without an opening
    __syncthreads();
    if (s_active) {  // uniform
      __syncthreads();  // ... before the counters are used again
      const int bits = lb + 2 * pb;
#pragma unroll 1
      for (int sh = 0; sh < bits; sh += 8)
        pass(cbeg, ctop, [=](uint64_t v) {
          const uint64_t key = ((uint64_t)(maxl - (uint32_t)(v >> 32)) << (2 * pb)) |
                               ((uint64_t)((uint32_t)v >> 16) << pb) | ((uint32_t)v & 0xFFFFu);
          return (uint32_t)(key >> sh) & 255u;
        });
    } else {
      const uint64_t *from = src;
#pragma unroll 1
      for (uint32_t k = cbeg + lane; k < ctop; k += 64) {
        const uint64_t v = from[k];
        const uint32_t s = (uint32_t)v & 0xFFFFu;
        uint32_t x = k >> 5, w = runs[x] & ((2u << (k & 31)) - 1u);
        while (!w) w = runs[--x];  // record 0 opens a run
        const uint32_t b = 32 * x + 31u - (uint32_t)__clz((int)w);
        x = k >> 5;
        w = runs[x] & ~((2u << (k & 31)) - 1u);
        while (!w && 32 * (x + 1) < C) w = runs[++x];
        const uint32_t e = w ? min(32 * x + (uint32_t)__ffs((int)w) - 1u, C) : C;
        uint32_t at = b;
        if (e - b > 1)
#pragma unroll 4
          for (uint32_t q = b; q < e; q++) {
            const uint32_t t = (uint32_t)from[q] & 0xFFFFu;
            at += (t < s || (t == s && q < k)) ? 1u : 0u;
          }
        dst[at] = v;
      }
      __syncthreads();
      uint64_t *t = src;
      src = dst;
      dst = t;
    }
    rec = src;
    accs = dst;
  }
  for (uint32_t k = tid; k < (n + 31) / 32; k += NT) bitmap[k] = 0;
  __syncthreads();
  stamp(5);

  // ---- greedy selection, as in window_short; the survivors' intervals and numbers
  // go to LDS
  {
    uint32_t *const item = reinterpret_cast<uint32_t *>(big), *const num = item + NT;
    uint32_t chunk = 64;
    uint64_t v = rec[min(tid, C ? C - 1 : 0)], pv = tid ? rec[min(tid, C) - (C ? 1 : 0)] : 0;
#pragma unroll 1
    for (uint32_t p0 = 0; p0 < C; p0 += chunk, chunk = min(2 * chunk, (uint32_t)NT)) {
      const uint32_t k = p0 + tid, nx = min(p0 + chunk + tid, C - 1);
      const uint64_t nv = rec[nx], npv = rec[nx ? nx - 1 : 0];  // the next chunk's, ahead
      bool ok = false, dup = false;
      const uint32_t s = (uint32_t)v & 0xFFFFu, l = (uint32_t)(v >> 32), e = s + l - 1u;
      if (tid < chunk && k < C) {
        dup = k && pv == v;
        ok = !dup && !((bitmap[s >> 5] >> (s & 31)) & 1u) && !((bitmap[e >> 5] >> (e & 31)) & 1u);
      }
      const uint64_t m = __ballot(ok), md = __ballot(dup);
      if (lane == 0) {
        wsum[wv] = (uint32_t)__popcll(m);
        if (md) atomicAdd(&s_dup, (uint32_t)__popcll(md));
      }
      __syncthreads();
      uint32_t tot;
      const uint32_t before = words_before<NW>(wsum, wv, tot);
      if (ok) {
        const uint32_t q = before + lanes_below(m);
        item[q] = s | (l << 16);
        num[q] = k;
      }
      __syncthreads();
      if (wv == 0 && tot) {
        const uint32_t na = greedy_walk(
            bitmap, tot, s_acc, [=](uint32_t q) { return item[q]; },
            [=](uint32_t o, uint32_t q) { accs[o] = rec[num[q]]; });
        if (lane == 0) s_acc = na;
      }
      __syncthreads();
      v = nv;
      pv = npv;
    }
  }
  const uint32_t A = s_acc, M = C - s_dup;
  uint32_t nhist = 1;
  while (s_hist[nhist - 1]) nhist++;
  stamp(6);

  // ---- rows
  auto rstart = [=](uint64_t v) { return (uint32_t)v & 0xFFFFu; };
  auto rlen = [=](uint64_t v) { return (uint32_t)(v >> 32); };
#pragma unroll 1
  for (uint32_t o0 = 0; o0 < A; o0 += NT) {
    const uint32_t o = o0 + tid;
    const bool open = o < A && (o == 0 || (accs[o] >> 16) != (accs[o - 1] >> 16));
    const uint64_t m = __ballot(open);
    if (lane == 0) {
      if (o0 + 64 * wv < A) {
        bitmap[(o0 >> 5) + 2 * wv] = (uint32_t)m;
        bitmap[(o0 >> 5) + 2 * wv + 1] = (uint32_t)(m >> 32);
      }
      atomicAdd(&s_nd, (uint32_t)__popcll(m));  // holds nd until here, which all have read
    }
  }
  __syncthreads();
  const uint32_t nrows = s_nd - nd;
  if (nrows <= a.row_cap && (!a.occ || A <= a.occ_cap)) {
    Row *rows = a.rows + (a.off ? tb / a.min_len : 0);
    uint32_t done = 0;
#pragma unroll 1
    for (uint32_t o0 = 0; o0 < A; o0 += NT) {
      const uint32_t o = o0 + tid;
      uint32_t pre = done, tot = 0;
      for (uint32_t w = 0; w < 2 * NW && o0 + 32 * w < A; w++) {  // scalar
        const uint32_t c = (uint32_t)__popc(bitmap[(o0 >> 5) + w]);
        pre += w < (tid >> 5) ? c : 0u;
        tot += c;
      }
      done += tot;
      if (o >= A) continue;
      const uint64_t v = accs[o];
      const uint32_t word = bitmap[o >> 5];
      const uint32_t r = pre + (uint32_t)__popc(word & ((2u << (o & 31)) - 1u)) - 1u;
      if ((word >> (o & 31)) & 1u) {
        uint32_t next = word & ~((2u << (o & 31)) - 1u), x = o >> 5;
        while (!next && 32 * (x + 1) < A) next = bitmap[++x];
        rows[r] = Row{rstart(v), rlen(v), (next ? 32 * x + (uint32_t)__ffs((int)next) - 1u : A) - o};
      }
      if (a.occ) a.occ[o] = Occ{rstart(v), rlen(v), r};
    }
  }
  if (tid == 0) {
    stamp(7);
    report(a, win, Report{D, nd, C, s_skip, maxl, M, A, nrows, s_pairs, nhist}, s_hist, s_stamp);
  }
}

// The window of a workgroup: the lone one, or the next longest of the batch.
__device__ __forceinline__ uint32_t window_of(const FusedArgs &a, uint32_t &win, uint64_t &tb) {
  win = 0;
  tb = 0;
  if (!a.off) return a.n;
  win = a.order[blockIdx.x];
  tb = a.off[win] - a.off[0];
  const uint32_t n = (uint32_t)(a.off[win + 1] - a.off[win]);
  if (n < 2 && threadIdx.x == 0) {
    a.win_rows[win] = 0;
    atomicAdd(&part_of(a)[CNT_NDSUM], n);  // (0 too: the kernels took 18 registers more with a branch for it)
  }
  return n;
}

template <int NT, int IPT>
__global__ __launch_bounds__(NT) void k_window(FusedArgs a) {
  __shared__ ShortLds<NT, IPT> L;
  uint32_t win;
  uint64_t tb;
  const uint32_t n = window_of(a, win, tb);
  if (n >= 2) window_short<NT, IPT>(a, L, win, tb, n);  // uniform
}

// Windows of any length up to kFusedLongMax in one launch: in launches of their
// own the short windows of a batch would wait for its last long one.
// LEAVE, for two or three windows, some longer than kFusedLone: there a workgroup each
// is the better form for most (two of 40000 tokens, loops with 5 % substitutions, 0.93 ms,
// stage by stage 1.06; random tokens 0.55 and 18), but not for a window that keeps its
// suffixes grouped for many rounds (loops without substitutions 1.76 and 1.16, of 65536
// tokens 2.88 and 1.36; half of it one run, 65536 tokens, 3.53 and 1.81).  The first sort, by
// h <= 8 tokens, tells it: all but h in 256 suffixes are grouped (substitutions of 1 % leave
// out 2 h or more), or one group fills an eighth of the slots.  Such a window gives up,
// the others as soon as they see it, and the batch goes stage by stage, host-driven:
// 1.32, 1.61 and 2.16 ms in all, no slower than before there was the one workgroup (1.42,
// 1.65, 2.41).
template <bool LEAVE>
__global__ __launch_bounds__(kLongNT) void k_window_any(LongArgs la) {
  __shared__ union Lds {
    ShortLds<kLongNT, kFusedMax / kLongNT> s;
    LongLds<kFusedLongMax> l;
  } L;
  uint32_t win;
  uint64_t tb;
  const uint32_t n = window_of(la.f, win, tb);
  if (n > kFusedMax) window_long<kFusedLongMax, false, LEAVE>(la, L.l, win, tb, n);  // uniform
  else if (n >= 2) window_short<kLongNT, kFusedMax / kLongNT>(la.f, L.s, win, tb, n);
}

// Batches that keep the chip busy for long (fused_in_two), in two launches.  These analyses
// wait for memory, LDS and barriers 60 % of the time and issue vector
// instructions a third of it, so the windows of up to kFusedMidMax tokens run
// two to a compute unit, with half the LDS and the registers of 64 wavefronts;
// the longer ones, and those with more distinct tokens than half the table
// takes, by themselves (4096 windows of 256 to 65536 tokens: 2.1 ms of the one,
// 3.8 of the other half of the tokens).
__global__ __launch_bounds__(kLongNT, 8) void k_window_mid(LongArgs la) {
  __shared__ union Lds {
    ShortLds<kLongNT, 4> s;
    LongLds<kFusedMidMax> l;
  } L;
  static_assert(sizeof(Lds) <= 80 * 1024, "two workgroups in 160 KB");
  const uint32_t at = blockIdx.x + la.f.order[la.f.windows];  // behind the longer windows
  if (at >= la.f.windows) return;
  const uint32_t win = la.f.order[at];
  const uint64_t tb = la.f.off[win] - la.f.off[0];
  const uint32_t n = (uint32_t)(la.f.off[win + 1] - la.f.off[win]);
  if (n > 4 * kLongNT) {  // uniform
    window_long<kFusedMidMax, true, false>(la, L.l, win, tb, n);
    return;
  }
  if (threadIdx.x == 0) {
    la.again[win] = 0;
    if (n < 2) {
      la.f.win_rows[win] = 0;
      atomicAdd(&part_of(la.f)[CNT_NDSUM], n);
    }
  }
  if (n >= 2) window_short<kLongNT, 4>(la.f, L.s, win, tb, n);
}
__global__ __launch_bounds__(kLongNT) void k_window_rest(LongArgs la) {
  __shared__ LongLds<kFusedLongMax> L;
  const uint32_t win = la.f.order[blockIdx.x];
  if (blockIdx.x >= la.f.order[la.f.windows] && !la.again[win]) return;  // uniform
  const uint64_t tb = la.f.off[win] - la.f.off[0];
  window_long<kFusedLongMax, false, false>(la, L, win, tb, (uint32_t)(la.f.off[win + 1] - la.f.off[win]));
}

// The counters' copies into where finish_run reads them: dcnt, a word of rhist per
// round, and the candidates as the selection's first count.
__global__ __launch_bounds__(kPartWords) void k_sum_parts(const uint32_t *parts, uint32_t n, uint32_t *dcnt,
                                                          uint32_t *rhist, uint32_t *selcnt) {
  const uint32_t t = threadIdx.x;
  const bool most = t == CNT_NDMAX || t == CNT_MAXL || (t >= CNT_STAGE && t < CNT_STAGE + kStages);
  uint32_t v = 0;
#pragma unroll 8
  for (uint32_t p = 0; p < n; p++) {
    const uint32_t x = parts[p * kPartWords + t];
    v = most ? max(v, x) : v + x;
  }
  if (t < CNT_COUNT) dcnt[t] = t == CNT_FUSED ? 1u : v;
  else if (t < CNT_COUNT + kLongRounds) rhist[4 * (t - CNT_COUNT)] = v;
  if (t == CNT_M) selcnt[0] = v;
}

// Where each window's rows go, for batches of more than kOwnBase windows: the sums
// of the counts before it, by one workgroup (2^20 windows: 128 steps).
constexpr uint32_t kOwnBase = 4096;
__global__ __launch_bounds__(1024) void k_row_bases(const uint32_t *win_rows, uint32_t W, uint32_t *base) {
  constexpr uint32_t PER = 8;
  __shared__ uint32_t sh[1024 / 64];
  uint32_t carry = 0;
  for (uint32_t b0 = 0; b0 < W; b0 += 1024 * PER) {
    const uint32_t b = b0 + threadIdx.x * PER;
    uint32_t v[PER], loc = 0, tot;
#pragma unroll
    for (uint32_t q = 0; q < PER; q++) {
      v[q] = b + q < W ? win_rows[b + q] : 0u;
      loc += v[q];
    }
    uint32_t at = carry + block_excl_sum<1024>(loc, sh, &tot);
#pragma unroll
    for (uint32_t q = 0; q < PER; q++) {
      if (b + q < W) base[b + q] = at;
      at += v[q];
    }
    carry += tot;
    __syncthreads();  // sh is used again
  }
}

// Packs the windows' rows, each window's at row off[w] / min_len of `src`,
// into dst in window order: window w's go to the sum of the counts before it,
// which its workgroup adds up itself up to kOwnBase windows (bases null).
__global__ __launch_bounds__(256) void k_pack_rows(const Row *src, const uint64_t *off, const uint32_t *win_rows,
                                                   const uint32_t *bases, uint32_t min_len, Row *dst) {
  __shared__ uint32_t sh[4];
  const uint32_t w = blockIdx.x, c = win_rows[w];
  if (c == 0) return;  // uniform
  uint32_t base;
  if (bases) {
    base = bases[w];
  } else {
    uint32_t part = 0;
    for (uint32_t q = threadIdx.x; q < w; q += 256) part += win_rows[q];
    (void)block_excl_sum<256>(part, sh, &base);
  }
  const Row *from = src + (off[w] - off[0]) / min_len;
  for (uint32_t r = threadIdx.x; r < c; r += 256) dst[base + r] = from[r];
}

void launch(const LongArgs &la, uint32_t blocks, uint64_t longest, bool leave, hipStream_t s) {
  // the smallest workgroup that holds the longest window: fewer wavefronts per
  // barrier, and more windows per compute unit
  const FusedArgs &a = la.f;
  if (longest <= 1024) hipLaunchKernelGGL((k_window<256, 4>), dim3(blocks), dim3(256), 0, s, a);
  else if (longest <= 2048) hipLaunchKernelGGL((k_window<512, 4>), dim3(blocks), dim3(512), 0, s, a);
  else if (longest <= 4096) hipLaunchKernelGGL((k_window<1024, 4>), dim3(blocks), dim3(1024), 0, s, a);
  else if (la.again) {
    hipLaunchKernelGGL(k_window_mid, dim3(blocks), dim3(kLongNT), 0, s, la);
    hipLaunchKernelGGL(k_window_rest, dim3(blocks), dim3(kLongNT), 0, s, la);
  } else if (longest <= kFusedMax) hipLaunchKernelGGL((k_window<1024, 8>), dim3(blocks), dim3(1024), 0, s, a);
  else if (leave) hipLaunchKernelGGL(k_window_any<true>, dim3(blocks), dim3(kLongNT), 0, s, la);
  else hipLaunchKernelGGL(k_window_any<false>, dim3(blocks), dim3(kLongNT), 0, s, la);
}

LongArgs args_of(const Workspace &w) {
  LongArgs la{};
  la.f.spill = reinterpret_cast<uint64_t *>(w.crec);
  la.txt = reinterpret_cast<uint16_t *>(w.tokrank);
  la.sa = reinterpret_cast<uint16_t *>(w.sa);
  la.rank = reinterpret_cast<uint16_t *>(w.rank);
  la.lcp = reinterpret_cast<uint16_t *>(w.lcp);
  la.e0 = reinterpret_cast<uint64_t *>(w.T);  // at least four words of 64 bits per token
  la.e1 = la.e0 + 2 * w.capN;
  la.flags = reinterpret_cast<uint64_t *>(w.tmp_a);
  return la;
}

}  // namespace

void fused_window(const Workspace &w, const void *tok, int bits, uint32_t n, uint32_t min_len, void *rows,
                  uint32_t row_cap, void *occ, uint32_t occ_cap, FusedInfo *info, hipStream_t s) {
  LongArgs la = args_of(w);
  FusedArgs &a = la.f;
  a.tok = tok;
  a.bits = bits;
  a.n = n;
  a.min_len = min_len;
  a.rows = static_cast<Row *>(rows);
  a.row_cap = row_cap;
  a.occ = static_cast<Occ *>(occ);
  a.occ_cap = occ_cap;
  a.info = info;
  launch(la, 1, n, false, s);
}

void fused_read(const FusedInfo &f, uint32_t n, Workspace &w, RunInfo &info) {
  info = RunInfo{};
  info.n = n;
  info.sigma = f.sigma;
  info.cands = f.cands;
  info.maxl = f.maxl;
  info.cands_dedup = f.m;
  info.accepted = f.accepted;
  info.rows = f.rows;
  info.rounds = f.nhist;
  info.sel_rounds = f.m ? 1 : 0;
  for (uint32_t r = 0; r < f.nhist; r++) {
    info.active_sum += r == 0 ? n : f.hist[r - 1];
    w.hrhist[4 * r] = f.hist[r];
  }
  w.hsel[0] = f.m;
  w.hsel[1] = 0;
  for (int k = 0; k < kStages; k++) info.stage_ms[k] = (double)(f.stamp[k + 1] - f.stamp[k]) * 1e-5;  // 100 MHz
}

// The two launches run one after the other, so each takes its longest window's
// time at least; one launch fills the chip to its end.  Nanoseconds as measured:
// a window alone 23 a token (30 with another on its compute unit), many of them
// 34 a token and compute unit, in twos 22; and a window, however short, some 27000,
// in twos 12000, since every workgroup of a launch is of the size that its longest
// window needs.  (Windows of 256 to 65536 tokens, one launch and two: 1200 of them 1.98
// and 2.87 ms, 4096 6.5 and 5.9; of 5000 to 20000: 300 0.60 and 0.65, 600 0.98 and
// 0.78; of 250 to 8192: 1200 0.54 and 0.37, 2048 0.86 and 0.57; 200000 of 25 and one of
// 6000: 28.7 and 13.4, stage by stage 23.)  Up to 4096 tokens the single launch has the
// same workgroups.
bool fused_in_two(const uint64_t *off, uint32_t W) {
  uint64_t n[2] = {0, 0}, count[2] = {0, 0}, longest[2] = {0, 0};  // windows that share a compute unit, longer ones
  for (uint32_t k = 0; k < W; k++) {
    const uint64_t len = off[k + 1] - off[k];
    const int side = len > kFusedMidMax;
    n[side] += len;
    count[side]++;
    longest[side] = std::max(longest[side], len);
  }
  if (std::max(longest[0], longest[1]) <= 4096) return false;
  const uint64_t one = std::max(23 * std::max(longest[0], longest[1]), (34 * (n[0] + n[1]) + 27000 * (count[0] + count[1])) / 256);
  const uint64_t two = std::max(23 * longest[1], (34 * n[1] + 27000 * count[1]) / 256) +
                       std::max(30 * longest[0], (22 * n[0] + 12000 * count[0]) / 256);
  return two < one;
}

void fused_batch(Workspace &w, const void *tok, uint32_t W, uint64_t longest, bool two, uint32_t min_len,
                 hipStream_t s) {
  uint32_t *const parts = w.snap;  // (a capacity of 1024 tokens holds 12 K words)
  uint32_t nparts = 1;
  while (nparts < kParts && 64 * nparts < W) nparts *= 2;
  clear_run(nullptr, 0, CNT_COUNT, parts, nparts * kPartWords, w.selcnt, 3 * (kSelRoundCap + 2),
            reinterpret_cast<uint32_t *>(w.eng.bufs().ctr), sizeof(SortCounters) / 4, s);
  LongArgs la = args_of(w);
  FusedArgs &a = la.f;
  a.tok = tok;
  a.bits = 64;
  a.off = w.d_off;
  a.order = w.d_order;
  a.windows = W;
  a.min_len = min_len;
  a.rows = static_cast<Row *>(w.occ);  // a batch reports no occurrences: their array stages the rows
  a.row_cap = kNone;
  a.parts = parts;
  a.part_mask = nparts - 1;
  a.win_rows = w.win_rows;
  if (two) la.again = w.wflag;
  launch(la, W, longest, w.may_leave && W <= 3 && longest > kFusedLone, s);
  uint32_t *bases = W > kOwnBase ? w.d_order : nullptr;  // the order has been read, and comes with every run
  if (bases) hipLaunchKernelGGL(k_row_bases, dim3(1), dim3(1024), 0, s, w.win_rows, W, bases);
  hipLaunchKernelGGL(k_pack_rows, dim3(W), dim3(256), 0, s, static_cast<const Row *>(w.occ), w.d_off, w.win_rows, bases,
                     min_len, static_cast<Row *>(w.rows));
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(kPartWords), 0, s, parts, nparts, w.dcnt, w.rhist, w.selcnt);
}

}  // namespace apo
