// Whole analysis of a short window (Section 4.2, Algorithm 2) by one
// workgroup, every intermediate array in LDS or registers.
//
// A short window leaves the stage-by-stage path nothing but latency: an
// analysis of 250 to 5000 tokens took 0.58 to 1.05 ms there, some 200 launches
// and 7 host synchronisations around a few microseconds of work each.  Here it
// is one launch: the window's tokens are read once and its rows written once,
// and the steps in between are separated by workgroup barriers.  Measured on
// MI355X, whole calls: 250 tokens 753 -> 57 us, 4096 tokens 913 -> 211 us, 5000
// tokens with occurrences 1165 -> 261 us, a batch of 64 windows of 250 to 5000
// tokens 3973 -> 391 us.  What bounds it now is the issue rate and LDS rate of
// one compute unit (4096 tokens: suffix sort 72 us of 162, the candidates, their
// sort and the greedy 20 to 30 us each).
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
// Value of the lane before (lane 0: 0).
__device__ __forceinline__ uint32_t lane_prev(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false);
}

__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

constexpr uint32_t kOwnRanks = 4096;     // most distinct values the stage-by-stage batch ranks per window
constexpr int kFusedRounds = 15;         // doubling rounds of a window of up to kFusedMax tokens
static_assert((1u << (kFusedRounds - 2)) >= kFusedMax, "round r groups by 2^r tokens");
constexpr int kMaxDigit = 7;             // radix digit bits
constexpr int kDigits = 1 << kMaxDigit;  // counter stride per wavefront

// Stable positions of m items by one digit.  Item i of a lane is number
// wave * 64 * ipt + 64 * i + lane; pos[i] receives its place in the digit's
// order.  Each wavefront counts its items digit by digit (lanes of equal digit
// found by ballots), then adds up the digits below and the wavefronts before
// it.  One barrier inside; the caller puts one after its stores.
template <int NT, int MAXI, int DB>
__device__ __forceinline__ void digit_places(const uint32_t (&dg)[MAXI], int ipt, uint32_t m, uint16_t *cnt,
                                             uint32_t (&pos)[MAXI]) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t below = (1ull << lane) - 1ull;
  uint16_t *my = cnt + wv * kDigits;
#pragma unroll
  for (int d = 0; d < (1 << DB); d += 64) my[d + lane] = 0;
  wave_order();
  const uint32_t base = (uint32_t)(wv * 64 * ipt);
#pragma unroll
  for (int i = 0; i < MAXI; i++) {
    if (i >= ipt || base + 64 * i >= m) continue;  // uniform
    const bool valid = base + 64 * i + lane < m;
    const uint32_t d = dg[i];
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < DB; b++) {
      const uint64_t one = __ballot((d >> b) & 1u);
      same &= ((d >> b) & 1u) ? one : ~one;
    }
    const uint32_t before = (uint32_t)__popcll(same & below);
    const uint32_t prev = my[d];
    wave_order();  // every lane has read before the first one of each digit writes
    if (valid && before == 0) my[d] = (uint16_t)(prev + (uint32_t)__popcll(same));
    pos[i] = prev + before;
    wave_order();
  }
  __syncthreads();
  uint32_t tot[DB == 7 ? 2 : 1] = {0}, bef[DB == 7 ? 2 : 1] = {0};
#pragma unroll
  for (int w = 0; w < NW; w++) {
#pragma unroll
    for (int q = 0; q < (DB == 7 ? 2 : 1); q++) {
      const uint32_t c = cnt[w * kDigits + 64 * q + lane];
      tot[q] += c;
      bef[q] += w < wv ? c : 0u;
    }
  }
  const uint32_t inc0 = lane_incl_sum(tot[0]);
  const uint32_t b0 = inc0 - tot[0] + bef[0];
  uint32_t b1 = 0;
  if (DB == 7) {
    const uint32_t all0 = (uint32_t)__builtin_amdgcn_readlane((int)inc0, 63);
    b1 = all0 + lane_incl_sum(tot[DB == 7 ? 1 : 0]) - tot[DB == 7 ? 1 : 0] + bef[DB == 7 ? 1 : 0];
  }
#pragma unroll
  for (int i = 0; i < MAXI; i++) {
    if (i >= ipt || base + 64 * i >= m) continue;
    uint32_t at = (uint32_t)__shfl((int)b0, (int)(dg[i] & 63u), 64);
    if (DB == 7) {
      const uint32_t hi = (uint32_t)__shfl((int)b1, (int)(dg[i] & 63u), 64);
      at = (dg[i] & 64u) ? hi : at;
    }
    pos[i] += at;
  }
}

// The same for bits [shift, shift + nb) of key (nb <= 7, uniform).
template <int NT, int MAXI>
__device__ __forceinline__ void key_places(const uint32_t (&key)[MAXI], int shift, int nb, int ipt, uint32_t m,
                                           uint16_t *cnt, uint32_t (&pos)[MAXI]) {
  uint32_t dg[MAXI];
  const uint32_t msk = (1u << nb) - 1u;
#pragma unroll
  for (int i = 0; i < MAXI; i++) dg[i] = (key[i] >> shift) & msk;
  if (nb <= 6) digit_places<NT, MAXI, 6>(dg, ipt, m, cnt, pos);
  else digit_places<NT, MAXI, 7>(dg, ipt, m, cnt, pos);
}

__device__ __forceinline__ int bits_of(uint32_t x) { return x ? 32 - __clz((int)x) : 0; }

struct Row { uint32_t start, length, count; };
struct Occ { uint32_t start, length, cand; };

struct FusedArgs {
  const void *tok;
  int bits;
  const uint64_t *off;     // batch: window offsets; null: one window of n tokens
  const uint32_t *order;   // batch: block b takes window order[b]
  uint32_t n, min_len;
  Row *rows;               // one window: final; batch: window w's rows start at off[w] / min_len
  Occ *occ;
  uint32_t row_cap, occ_cap;
  FusedInfo *info;         // one window
  uint32_t *dcnt, *rhist, *win_rows;  // batch: counters added up over the windows
};

// NT threads, up to NT * IPT tokens.
template <int NT, int IPT>
__global__ __launch_bounds__(NT) void k_window(FusedArgs a) {
  constexpr int NW = NT / 64;
  constexpr uint32_t CAP = NT * IPT, SLOTS = 2 * CAP;
  constexpr int CI = 2 * IPT;  // candidates per thread at most
  static_assert(CAP <= kFusedMax, "16 bytes of LDS per token, and positions and ranks in 14 bits");
  // ra, rb (8 bytes per token each) hold, one phase after the other:
  //   ranking: the tokens; the hash table, later the ranks by slot
  //   suffix sort: token ranks, suffix ranks, suffix order, LCP; the exchange buffer
  //   candidate sort: start | ID << 16; length
  __shared__ __align__(16) unsigned char ra[CAP * 8 + 64], rb[CAP * 8];
  __shared__ uint16_t rc[CAP];               // slots of the distinct values; later the accepted candidates
  __shared__ uint16_t cnt[NW * kDigits];     // radix counters; later LCP minima, surviving candidates
  __shared__ uint32_t bitmap[CAP / 32];
  __shared__ uint32_t wsum[NW], wsum2[NW];
  __shared__ uint32_t s_nd, s_top, s_zero, s_single, s_max, s_skip, s_acc, s_dup;
  __shared__ uint32_t s_hist[kFusedRounds];
  __shared__ uint64_t s_stamp[kStages + 1];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint64_t below = (1ull << lane) - 1ull;

  uint32_t win = 0, n = a.n;
  uint64_t tb = 0;
  if (a.off) {
    win = a.order[blockIdx.x];
    tb = a.off[win] - a.off[0];
    n = (uint32_t)(a.off[win + 1] - a.off[win]);
    if (n < 2) {  // uniform
      if (tid == 0) {
        a.win_rows[win] = 0;
        atomicAdd(&a.dcnt[CNT_NDSUM], n);
      }
      return;
    }
  }
  auto stamp = [&](int k) {
    if (tid == 0) s_stamp[k] = wall_clock64();
  };
  stamp(0);

  // ---- order-preserving token ranks: distinct values through an LDS hash
  // table (a slot holds the number of the token that claimed it), sorted, and
  // every token's rank read from its slot
  uint64_t *tokl = reinterpret_cast<uint64_t *>(ra);
  uint32_t *tab = reinterpret_cast<uint32_t *>(rb);
  uint64_t tk[IPT];
#pragma unroll
  for (int i = 0; i < IPT; i++) {
    const uint32_t k = i * NT + tid;
    tk[i] = 0;
    if (k < n)
      tk[i] = a.bits == 64 ? static_cast<const uint64_t *>(a.tok)[tb + k]
                           : (uint64_t) static_cast<const uint32_t *>(a.tok)[tb + k];
  }
  if (tid == 0) {
    s_nd = 0;
    s_top = 0;
    s_skip = 0;
    s_max = 0;
    s_acc = 0;
    s_dup = 0;
  }
  for (uint32_t k = tid; k < SLOTS; k += NT) tab[k] = kNone;
#pragma unroll
  for (int i = 0; i < IPT; i++)
    if (i * NT + tid < n) tokl[i * NT + tid] = tk[i];
  __syncthreads();
  uint16_t slot[IPT];
#pragma unroll
  for (int i = 0; i < IPT; i++) {
    const uint32_t k = i * NT + tid;
    slot[i] = 0;
    if (k >= n) continue;
    uint32_t h = (uint32_t)(mix64(tk[i]) >> 40) & (SLOTS - 1);
    for (;;) {  // n <= SLOTS / 2 values: a free slot is always found
      uint32_t cur = tab[h];
      if (cur == kNone) {
        cur = atomicCAS(&tab[h], kNone, k);
        if (cur == kNone) {
          rc[atomicAdd(&s_nd, 1u)] = (uint16_t)h;
          if (tk[i] == ~0ull) s_top = 1;
          break;
        }
      }
      if (tokl[cur] == tk[i]) break;
      h = (h + 1) & (SLOTS - 1);
    }
    slot[i] = (uint16_t)h;
  }
  __syncthreads();
  const uint32_t D = s_nd;
  {
    // the distinct values in runs of 64, one per lane, sorted by a bitonic
    // network over lane moves; then runs merged pairwise, each value finding
    // its place by a binary search in the other run (pads: the largest value,
    // kept apart by place)
    uint32_t P = 64;
    while (P < D) P <<= 1;
    uint64_t v[IPT];
    uint32_t vs[IPT], pos[IPT];
    // register r of a thread holds value r * NT + tid while P >= NT; wavefronts
    // past P hold nothing
    const bool holds = tid < P;
    const int R = (int)((P + NT - 1) / NT);
#pragma unroll
    for (int r = 0; r < IPT; r++) {
      const uint32_t q = r * NT + tid;
      vs[r] = kNone;
      v[r] = ~0ull;
      if (r < R && q < D) {
        vs[r] = rc[q];
        v[r] = tokl[tab[vs[r]]];
      }
    }
#pragma unroll
    for (uint32_t k = 2; k <= 64; k <<= 1)
#pragma unroll
      for (uint32_t j = k >> 1; j > 0; j >>= 1)
#pragma unroll
        for (int r = 0; r < IPT; r++) {
          if (r >= R || !holds) continue;
          const uint64_t o = ((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(v[r] >> 32), (int)j, 64) << 32) |
                             (uint32_t)__shfl_xor((int)(uint32_t)v[r], (int)j, 64);
          const uint32_t os = (uint32_t)__shfl_xor((int)vs[r], (int)j, 64);
          const bool lower = (lane & j) == 0, asc = (lane & k) == 0 || k == 64;
          // pads order after every value, so equal pairs are pads and a value
          // equal to a pad (the largest token) goes first
          const bool mine_less = v[r] < o || (v[r] == o && vs[r] < os);
          const bool keep = (lower == asc) == mine_less || (v[r] == o && vs[r] == os);
          v[r] = keep ? v[r] : o;
          vs[r] = keep ? vs[r] : os;
        }
    __syncthreads();  // tokens and table read
    uint64_t *buf[2] = {reinterpret_cast<uint64_t *>(ra), reinterpret_cast<uint64_t *>(rb)};
#pragma unroll
    for (int r = 0; r < IPT; r++) {
      pos[r] = r * NT + tid;
      if (r < R && holds) buf[0][pos[r]] = v[r];
    }
    __syncthreads();
    int cb = 0;
    for (uint32_t L = 64; L < P; L <<= 1) {
      const uint64_t *src = cb ? buf[1] : buf[0];
      uint64_t *dst = cb ? buf[0] : buf[1];
#pragma unroll
      for (int r = 0; r < IPT; r++) {
        if (r >= R || !holds) continue;
        const uint32_t i = pos[r], base = i & ~(2 * L - 1), right = i & L;
        const bool rt = right != 0;
        const uint64_t x = v[r];
        const uint64_t *o = src + (right ? base : base + L);
        uint32_t c = 0;
        for (uint32_t step = L >> 1; step > 0; step >>= 1) {  // branch-free steps
          const uint64_t y = o[c + step - 1];
          c += ((y < x) | ((y == x) & rt)) ? step : 0u;
        }
        c += ((o[c] < x) | ((o[c] == x) & rt)) ? 1u : 0u;  // c <= L - 1 before this step
        pos[r] = base + (i - base - right) + c;
        dst[pos[r]] = x;
      }
      __syncthreads();
      cb ^= 1;
    }
    // ranks by slot (rb: its last use as a merge buffer is over, or it is the
    // merged list, which nothing reads)
    uint16_t *srank = reinterpret_cast<uint16_t *>(rb);
#pragma unroll
    for (int r = 0; r < IPT; r++)
      if (r < R && vs[r] != kNone) srank[vs[r]] = (uint16_t)(pos[r] + 1);
  }
  __syncthreads();
  uint16_t *txt = reinterpret_cast<uint16_t *>(ra);  // token ranks 1..D, 32 words past the end readable
  uint16_t *rank = txt + CAP + 32, *sa = rank + CAP, *lcp = sa + CAP;
  uint32_t *exch = reinterpret_cast<uint32_t *>(rb);
  {
    const uint16_t *srank = reinterpret_cast<const uint16_t *>(rb);
#pragma unroll
    for (int i = 0; i < IPT; i++)
      if (i * NT + tid < n) txt[i * NT + tid] = srank[slot[i]];
    if (tid < 32) txt[n + tid] = 0;
  }
  __syncthreads();
  stamp(1);

  // ---- suffix array by prefix doubling.  A round lists the suffixes j in the
  // order of their second halves (j = SA[k] - h) and sorts that list stably by
  // the group of the first half.  The h shortest suffixes, whose second half is
  // empty, wrap around (j = SA[k] - h + n): the one of h tokens (SA[k] = 0) is
  // put first, the shorter ones may stand anywhere, each alone in its group.
  const int ipt = (int)((n + NT - 1) / NT);
  const uint32_t kb = wv * 64 * ipt + lane;  // item i of this lane: kb + 64 * i
  uint32_t nhist = 0;
  {
    uint32_t j[IPT], key[IPT], pos[IPT];
    int kbits = bits_of(D - 1);
    uint32_t h = 0;
#pragma unroll
    for (int i = 0; i < IPT; i++) {
      j[i] = kb + 64 * i;
      key[i] = (i < ipt && j[i] < n) ? txt[j[i]] - 1u : 0u;
    }
    for (uint32_t round = 0;; round++) {
      if (round) {
        const uint32_t first = s_zero;
#pragma unroll
        for (int i = 0; i < IPT; i++) {
          const uint32_t k = kb + 64 * i;
          if (i >= ipt || k >= n) continue;
          const uint32_t s = sa[k == 0 ? first : k <= first ? k - 1 : k];
          j[i] = s >= h ? s - h : s + n - h;
          key[i] = rank[j[i]];
        }
      }
      const int lo = kbits > kMaxDigit ? (kbits + 1) / 2 : kbits;
      if (lo < kbits) {
        key_places<NT, IPT>(key, 0, lo, ipt, n, cnt, pos);
#pragma unroll
        for (int i = 0; i < IPT; i++)
          if (i < ipt && kb + 64 * i < n) exch[pos[i]] = j[i] | (key[i] << 16);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < IPT; i++)
          if (i < ipt && kb + 64 * i < n) {
            const uint32_t e = exch[kb + 64 * i];
            j[i] = e & 0xFFFFu;
            key[i] = e >> 16;
          }
        key_places<NT, IPT>(key, lo, kbits - lo, ipt, n, cnt, pos);
      } else {
        key_places<NT, IPT>(key, 0, lo, ipt, n, cnt, pos);
      }
#pragma unroll
      for (int i = 0; i < IPT; i++)
        if (i < ipt && kb + 64 * i < n) sa[pos[i]] = (uint16_t)j[i];
      __syncthreads();
      // group heads: (first half's group, second half's) differs from the slot before
      uint64_t head[IPT];
      uint32_t last = kNone;  // the wavefront's last head
#pragma unroll
      for (int i = 0; i < IPT; i++) {
        head[i] = ~0ull;
        const uint32_t k0 = wv * 64 * ipt + 64 * i;
        if (i >= ipt || k0 >= n) continue;  // uniform
        const uint32_t k = k0 + lane;
        bool hd = true;
        uint32_t c = 0;
        if (k < n) {
          const uint32_t s = sa[k];
          j[i] = s;
          if (s == 0) s_zero = k;
          if (round == 0) c = txt[s];
          else c = ((uint32_t)rank[s] << 16) | (s + h < n ? rank[s + h] : 0xFFFFu);
        }
        uint32_t p = lane_prev(c);
        if (lane == 0 && k) {
          const uint32_t s = sa[k - 1];
          if (round == 0) p = txt[s];
          else p = ((uint32_t)rank[s] << 16) | (s + h < n ? rank[s + h] : 0xFFFFu);
        }
        if (k && k < n) hd = c != p;
        head[i] = __ballot(hd);
        const uint64_t in = n - k0 >= 64 ? ~0ull : (1ull << (n - k0)) - 1ull;
        if (head[i] & in) last = k0 + 63u - (uint32_t)__clzll((long long)(head[i] & in));
      }
      if (lane == 0) {
        wsum[wv] = last;
        wsum2[wv] = (uint32_t)(head[0] & 1ull);
      }
      if (tid == 0) s_single = 0;
      __syncthreads();
      uint32_t carry = 0;
#pragma unroll
      for (int w = 0; w < NW; w++)
        if (w < (int)wv && wsum[w] != kNone) carry = wsum[w];
      const uint64_t next_first = wv + 1 < NW ? wsum2[wv + 1 < NW ? wv + 1 : 0] : 1u;
      uint32_t singles = 0;
#pragma unroll
      for (int i = 0; i < IPT; i++) {
        const uint32_t k0 = wv * 64 * ipt + 64 * i;
        if (i >= ipt || k0 >= n) continue;
        const uint64_t in = n - k0 >= 64 ? ~0ull : (1ull << (n - k0)) - 1ull;
        const uint64_t up = i + 1 < ipt ? head[i + 1 < IPT ? i + 1 : i] & 1ull : next_first;
        singles += (uint32_t)__popcll(head[i] & in & ((head[i] >> 1) | (up << 63)));
        const uint64_t upto = head[i] & in & (below | (1ull << lane));
        if (k0 + lane < n) rank[j[i]] = (uint16_t)(upto ? k0 + 63u - (uint32_t)__clzll((long long)upto) : carry);
        if (head[i] & in) carry = k0 + 63u - (uint32_t)__clzll((long long)(head[i] & in));
      }
      if (lane == 0 && singles) atomicAdd(&s_single, singles);
      __syncthreads();
      const uint32_t active = n - s_single;
      if (tid == 0) s_hist[round] = active;  // at most kFusedRounds: 2^(round - 1) < n
      nhist = round + 1;
      if (active == 0) break;  // uniform
      h = h ? 2 * h : 1;
      kbits = bits_of(n - 1);
    }
  }
  stamp(2);

  // ---- LCP: Kasai's walk over ipt consecutive positions per thread, eight
  // tokens per step; suffixes are all alone, so rank is the inverse of sa
  {
    uint32_t h = 0;
    for (int i = 0; i < ipt; i++) {
      const uint32_t x = tid * ipt + i;
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
  }
  __syncthreads();
  stamp(3);

  // ---- candidates of every adjacent pair in suffix-array order.  The minima
  // of 16 and 256 LCP values serve the ID's previous-smaller-value queries.
  uint16_t *min1 = cnt, *min2 = cnt + CAP / 16;
  static_assert(CAP / 16 + CAP / 256 <= NW * kDigits, "minima fit the radix counters");
  for (uint32_t b = tid; b < (n + 15) / 16; b += NT) {
    uint32_t mn = 0xFFFFu;
    for (uint32_t q = 0; q < 16 && b * 16 + q < n; q++) mn = min(mn, (uint32_t)lcp[b * 16 + q]);
    min1[b] = (uint16_t)mn;
  }
  __syncthreads();
  for (uint32_t b = tid; b < (n + 255) / 256; b += NT) {
    uint32_t mn = 0xFFFFu;
    for (uint32_t q = 0; q < 16 && b * 16 + q < (n + 15) / 16; q++) mn = min(mn, (uint32_t)min1[b * 16 + q]);
    min2[b] = (uint16_t)mn;
  }
  __syncthreads();
  uint32_t C = 0, maxl = 0;
  {
    uint32_t w0[CI], w1[CI], at[CI];
    uint32_t run = 0, mx = 0, skipped = 0;
#pragma unroll
    for (int i = 0; i < IPT; i++) {
      at[2 * i] = at[2 * i + 1] = kNone;
      w0[2 * i] = w0[2 * i + 1] = w1[2 * i] = w1[2 * i + 1] = 0;
      const uint32_t k0 = wv * 64 * ipt + 64 * i, k = k0 + lane;
      if (i >= ipt || k0 >= n) continue;  // uniform
      uint32_t l = 0, s1 = 0, s2 = 0;
      bool disj = false;
      if (k + 1 < n) {
        const uint32_t x = sa[k], y = sa[k + 1], p = lcp[k];
        const uint32_t lo = min(x, y), d = max(x, y) - lo;
        if (p <= d) {
          l = p;
          s1 = x;
          s2 = y;
          disj = true;
        } else {
          l = (p + d) / 2;
          l -= l % d;
          s1 = lo;
          s2 = lo + l;
        }
        if (l < a.min_len) l = 0;
      }
      // pair k - 1's length when it is disjoint too (equal lengths: its second
      // candidate is this pair's first)
      bool rep = false;
      if (l && disj && k) {
        const uint32_t x = sa[k - 1], y = sa[k], p = lcp[k - 1];
        rep = p == l && p <= max(x, y) - min(x, y);
      }
      uint32_t id = 0;
      if (l) {  // 1 + the last pair before k whose LCP is below l
        int f = (int)k - 1;
        while (f >= 0 && (f & 15) != 15 && lcp[f] >= l) f--;
        if (f >= 0 && (f & 15) == 15) {
          int b = f >> 4;
          while (b >= 0 && (b & 15) != 15 && min1[b] >= l) b--;
          if (b >= 0 && (b & 15) == 15) {
            int c = b >> 4;
            while (c >= 0 && min2[c] >= l) c--;
            b = c < 0 ? -1 : (c << 4) + 15;
            while (b >= 0 && min1[b] >= l) b--;
          }
          f = b < 0 ? -1 : (b << 4) + 15;
          while (f >= 0 && lcp[f] >= l) f--;
        }
        id = (uint32_t)(f + 1);
      }
      const uint64_t m2 = __ballot(l != 0), m1 = __ballot(l != 0 && !rep);
      uint32_t q = run + (uint32_t)__popcll(m1 & below) + (uint32_t)__popcll(m2 & below);
      if (l) {
        if (!rep) {
          at[2 * i] = q++;
          w0[2 * i] = s1 | (id << 16);
          w1[2 * i] = l;
        }
        at[2 * i + 1] = q;
        w0[2 * i + 1] = s2 | (id << 16);
        w1[2 * i + 1] = l;
      }
      run += (uint32_t)(__popcll(m1) + __popcll(m2));
      skipped += (uint32_t)(__popcll(m2) - __popcll(m1));
      mx = max(mx, l);
    }
    if (mx) atomicMax(&s_max, mx);
    if (lane == 0) {
      wsum[wv] = run;
      if (skipped) atomicAdd(&s_skip, skipped);
    }
    __syncthreads();  // suffix order, ranks, LCP and minima read
    uint32_t off = 0;
#pragma unroll
    for (int w = 0; w < NW; w++) {
      const uint32_t c = wsum[w];
      off += w < (int)wv ? c : 0u;
      C += c;
    }
    maxl = s_max;
    uint32_t *o0 = reinterpret_cast<uint32_t *>(ra);
    uint16_t *o1 = reinterpret_cast<uint16_t *>(rb);
#pragma unroll
    for (int i = 0; i < CI; i++)
      if (at[i] != kNone) {
        o0[off + at[i]] = w0[i];
        o1[off + at[i]] = (uint16_t)w1[i];
      }
  }
  for (uint32_t k = tid; k < (n + 31) / 32; k += NT) bitmap[k] = 0;
  __syncthreads();
  stamp(4);

  // ---- priority order (length desc, ID asc, start asc): a stable sort by
  // start, then ID, then length, 7 bits or fewer at a time
  uint32_t *c0 = reinterpret_cast<uint32_t *>(ra);   // start | ID << 16
  uint16_t *c1 = reinterpret_cast<uint16_t *>(rb);   // length
  if (C) {  // uniform
    const int cpt = (int)((C + NT - 1) / NT);
    const uint32_t cb = wv * 64 * cpt + lane;
    const int pb = bits_of(n - 1), lb = bits_of(maxl - a.min_len);
    for (int field = 0; field < 3; field++) {
      const int fb = field == 2 ? lb : pb;
      const int np = (fb + kMaxDigit - 1) / kMaxDigit;
      int shift = 0;
      for (int p = 0; p < np; p++) {
        const int nb = (fb - shift + (np - p) - 1) / (np - p);
        uint32_t w0[CI], w1[CI], key[CI], pos[CI];
#pragma unroll
        for (int i = 0; i < CI; i++) {
          w0[i] = w1[i] = key[i] = 0;
          if (i < cpt && cb + 64 * i < C) {
            w0[i] = c0[cb + 64 * i];
            w1[i] = c1[cb + 64 * i];
            key[i] = field == 0 ? w0[i] & 0xFFFFu : field == 1 ? w0[i] >> 16 : maxl - w1[i];
          }
        }
        key_places<NT, CI>(key, shift, nb, cpt, C, cnt, pos);
#pragma unroll
        for (int i = 0; i < CI; i++)
          if (i < cpt && cb + 64 * i < C) {
            c0[pos[i]] = w0[i];
            c1[pos[i]] = (uint16_t)w1[i];
          }
        __syncthreads();
        shift += nb;
      }
    }
  }
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
    for (uint32_t p0 = 0; p0 < C; p0 += chunk, chunk = min(2 * chunk, (uint32_t)NT)) {
      const uint32_t k = p0 + tid;
      bool ok = false, dup = false;
      if (tid < chunk && k < C) {
        const uint32_t w = c0[k], l = c1[k];
        dup = k && c0[k - 1] == w && c1[k - 1] == l;
        const uint32_t s = w & 0xFFFFu, e = s + l - 1u;
        ok = !dup && !((bitmap[s >> 5] >> (s & 31)) & 1u) && !((bitmap[e >> 5] >> (e & 31)) & 1u);
      }
      const uint64_t m = __ballot(ok), md = __ballot(dup);
      if (lane == 0) {
        wsum[wv] = (uint32_t)__popcll(m);
        if (md) atomicAdd(&s_dup, (uint32_t)__popcll(md));
      }
      __syncthreads();
      uint32_t before = 0, tot = 0;
#pragma unroll
      for (int w = 0; w < NW; w++) {
        const uint32_t c = wsum[w];
        before += w < (int)wv ? c : 0u;
        tot += c;
      }
      if (ok) surv[before + (uint32_t)__popcll(m & below)] = (uint16_t)(k - p0);
      __syncthreads();
      if (wv == 0 && tot) {
        uint32_t na = s_acc;
        for (uint32_t q0 = 0; q0 < tot; q0 += 64) {
          const bool valid = q0 + lane < tot;
          const uint32_t kk = p0 + (valid ? surv[q0 + lane] : 0u);
          const uint32_t w = c0[kk], l = c1[kk];
          const uint32_t s = w & 0xFFFFu, e = s + l - 1u;
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
          // intervals of a few bitmap words are painted by their own lane,
          // longer ones by the whole wavefront
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
          if (mine) acc[na + (uint32_t)__popcll(take & below)] = (uint16_t)kk;
          na += (uint32_t)__popcll(take);
          wave_order();
        }
        if (lane == 0) s_acc = na;
      }
      __syncthreads();
    }
  }
  const uint32_t A = s_acc, M = C - s_dup;
  stamp(6);

  // ---- rows: occurrence o opens one when its length or ID differs from the
  // one before; its count is the distance to the next row's first occurrence
  uint16_t *first = reinterpret_cast<uint16_t *>(rb) + 2 * CAP;  // above the lengths
  uint32_t nrows = 0;
  for (uint32_t o0 = 0; o0 < A; o0 += NT) {  // row count first
    const uint32_t o = o0 + tid;
    bool nr = false;
    if (o < A) {
      const uint32_t k = acc[o];
      nr = o == 0;
      if (o) {
        const uint32_t kp = acc[o - 1];
        nr = c1[k] != c1[kp] || (c0[k] >> 16) != (c0[kp] >> 16);
      }
    }
    const uint64_t m = __ballot(nr);
    if (lane == 0) wsum[wv] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t before = nrows, tot = 0;
#pragma unroll
    for (int w = 0; w < NW; w++) {
      const uint32_t c = wsum[w];
      before += w < (int)wv ? c : 0u;
      tot += c;
    }
    if (nr) first[before + (uint32_t)__popcll(m & below)] = (uint16_t)o;
    nrows += tot;
    __syncthreads();
  }
  const bool fits = nrows <= a.row_cap && (!a.occ || A <= a.occ_cap);
  if (fits) {
    Row *rows = a.rows + (a.off ? tb / a.min_len : 0);
    for (uint32_t r = tid; r < nrows; r += NT) {
      const uint32_t o = first[r], k = acc[o];
      rows[r] = Row{c0[k] & 0xFFFFu, c1[k], (r + 1 < nrows ? first[r + 1] : A) - o};
    }
    if (a.occ)
      for (uint32_t o = tid; o < A; o += NT) {
        uint32_t lo = 0, hi = nrows;  // the last row starting at or before o
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) / 2;
          if (first[mid] <= o) lo = mid;
          else hi = mid;
        }
        const uint32_t k = acc[o];
        a.occ[o] = Occ{c0[k] & 0xFFFFu, c1[k], lo};
      }
  }
  if (tid == 0) {
    stamp(7);
    if (a.info) {
      FusedInfo &f = *a.info;
      f.sigma = a.bits == 64 ? D : 0u;
      f.cands = C + s_skip;
      f.maxl = maxl;
      f.m = M;
      f.accepted = A;
      f.rows = nrows;
      f.nhist = nhist;
      for (uint32_t r = 0; r < nhist; r++) f.hist[r] = s_hist[r];
      for (int k = 0; k <= kStages; k++) f.stamp[k] = s_stamp[k];
    } else {
      a.win_rows[win] = nrows;
      atomicAdd(&a.dcnt[CNT_NDSUM], D);
      atomicMax(&a.dcnt[CNT_NDMAX], D);
      atomicAdd(&a.dcnt[CNT_C], C);
      atomicAdd(&a.dcnt[CNT_CSKIP], s_skip);
      atomicMax(&a.dcnt[CNT_MAXL], maxl);
      atomicAdd(&a.dcnt[CNT_M], M);
      atomicAdd(&a.dcnt[CNT_A], A);
      atomicAdd(&a.dcnt[CNT_NROWS], nrows);
      // a window whose ranks the stage-by-stage batch takes from the shared table
      if (D - s_top > kOwnRanks) atomicAdd(&a.dcnt[CNT_PFLAG], 1u);
      for (uint32_t r = 0; r < nhist; r++)
        if (s_hist[r]) atomicAdd(&a.rhist[4 * r], s_hist[r]);
      for (int k = 0; k < kStages; k++)
        atomicMax(&a.dcnt[CNT_STAGE + k], (uint32_t)(s_stamp[k + 1] - s_stamp[k]));
    }
  }
}

// Packs the windows' rows, each window's at row off[w] / min_len of `src`,
// into dst in window order: window w's go to the sum of the counts before it,
// which its workgroup adds up itself (a few thousand words at most).
__global__ __launch_bounds__(256) void k_pack_rows(const Row *src, const uint64_t *off, const uint32_t *win_rows,
                                                   uint32_t W, uint32_t min_len, Row *dst) {
  __shared__ uint32_t sh[4];
  const uint32_t w = blockIdx.x, c = win_rows[w];
  if (c == 0) return;  // uniform
  uint32_t part = 0;
  for (uint32_t q = threadIdx.x; q < w; q += 256) part += win_rows[q];
  uint32_t base;
  (void)block_excl_sum<256>(part, sh, &base);
  const Row *from = src + (off[w] - off[0]) / min_len;
  for (uint32_t r = threadIdx.x; r < c; r += 256) dst[base + r] = from[r];
}

void launch(const FusedArgs &a, uint32_t blocks, uint32_t longest, hipStream_t s) {
  // the smallest workgroup that holds the longest window: fewer wavefronts
  // per barrier, and more windows per compute unit
  if (longest <= 1024) hipLaunchKernelGGL((k_window<256, 4>), dim3(blocks), dim3(256), 0, s, a);
  else if (longest <= 2048) hipLaunchKernelGGL((k_window<512, 4>), dim3(blocks), dim3(512), 0, s, a);
  else if (longest <= 4096) hipLaunchKernelGGL((k_window<1024, 4>), dim3(blocks), dim3(1024), 0, s, a);
  else hipLaunchKernelGGL((k_window<1024, 8>), dim3(blocks), dim3(1024), 0, s, a);
}

}  // namespace

void fused_window(const void *tok, int bits, uint32_t n, uint32_t min_len, void *rows, uint32_t row_cap, void *occ,
                  uint32_t occ_cap, FusedInfo *info, hipStream_t s) {
  FusedArgs a{};
  a.tok = tok;
  a.bits = bits;
  a.n = n;
  a.min_len = min_len;
  a.rows = static_cast<Row *>(rows);
  a.row_cap = row_cap;
  a.occ = static_cast<Occ *>(occ);
  a.occ_cap = occ_cap;
  a.info = info;
  launch(a, 1, n, s);
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

void fused_batch(Workspace &w, const void *tok, uint32_t W, uint32_t maxwin, uint32_t min_len, hipStream_t s) {
  fill_u32(w.dcnt, CNT_COUNT, 0, s);
  fill_u32(w.rhist, 4 * (uint64_t)w.nsnap, 0, s);
  fill_u32(w.selcnt, 3 * (kSelRoundCap + 2), 0, s);
  FusedArgs a{};
  a.tok = tok;
  a.bits = 64;
  a.off = w.d_off;
  a.order = w.d_order;
  a.min_len = min_len;
  a.rows = static_cast<Row *>(w.occ);  // a batch reports no occurrences: their array stages the rows
  a.row_cap = kNone;
  a.dcnt = w.dcnt;
  a.rhist = w.rhist;
  a.win_rows = w.win_rows;
  launch(a, W, maxwin, s);
  hipLaunchKernelGGL(k_pack_rows, dim3(W), dim3(256), 0, s, static_cast<const Row *>(w.occ), w.d_off, w.win_rows, W,
                     min_len, static_cast<Row *>(w.rows));
  copy_u32(w.selcnt, w.dcnt + CNT_M, s);
}

}  // namespace apo
