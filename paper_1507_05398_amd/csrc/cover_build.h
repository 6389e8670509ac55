// cover_build.h -- graded codes (grlex, grevlex; constant weight, ranges and
// prefixes too) of distance 2, 3 or 4 for n <= 24, from a bitmap of the whole
// space instead of distance checks.  Included by greedy_code.hip.  Larger
// distances, and small codes of these: cover_windows.h.
//
// An accepted word marks the ball of radius d - 1 around it (301 words at n =
// 24, d = 3), so a candidate costs one bit and not a scan of the code.  The
// walk's order only matters among words of one weight: the levels are done in
// turn, and inside a level, where the words that can clash are at distance 2,
// in rounds: a candidate with no undecided earlier neighbour is accepted, the
// balls are marked, again until no candidate is left.  That is the sequential
// greedy (the earliest undecided candidate is always accepted), in few
// rounds: about 170 over all levels at n = 24, d = 3 for 524288 words.
//
// Words are numbered so that a level's order is the increasing order: grlex
// by value, grevlex by the complement of the reversed word.  A workgroup owns
// a slice (the top bits of the number) in LDS; a bit operation covers the 64
// candidates of a word.  The level's undecided candidates and the words
// accepted in a round go through global memory.  All workgroups are on one
// XCD, so that L2 joins them: a barrier is one atomic and a poll there (0.9
// us for 32 workgroups against 4.7 us over eight XCDs), stores need no
// write-back, and what others wrote is read past the vector L1 (relaxed
// agent-scope loads).  One barrier a round: a neighbour's candidates may be
// read before or after it has marked the last round's words.  They only
// shrink, and a candidate read too early only waits a round longer.
//
// What bounds it: the rounds, each a chain of a barrier, marks and neighbour
// reads (about 11 us at n = 20, d = 3: marks 3, reads 2.5, waiting for the
// slowest slice 4), and for the largest codes the LDS throughput of the marks
// (n = 24, d = 4: 988 words for each of 262144 code words).  Kernel time of
// this path and of the windowed screens: n = 20, d = 3 1.1 and 9 ms; n = 22,
// d = 4 2.2 and 17 ms; n = 24, d = 3 4.4 and 106 ms; n = 24, d = 4 5.9 and 64
// ms.

// Barrier of the cover team's workgroups (all on one XCD), bounded.
__device__ __forceinline__ void cover_barrier(CoverWs *ws, unsigned int team, int *abort_flag, unsigned int limit) {
  CoverLds &C = g_lds.cover;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (team == 1) return;
  if (threadIdx.x == 0) {
    C.epoch += team;
    const unsigned int target = C.epoch;
    const int aborted = ld_relaxed(abort_flag);
    __hip_atomic_fetch_add(as_global(&ws->arrived), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned int spins = 0;
    bool passed = true;
    while (__hip_atomic_load(as_global(&ws->arrived), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      __builtin_amdgcn_s_sleep(1);
      if (++spins > limit) {
        __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        passed = false;
        break;
      }
    }
    if (aborted != 0 || !passed) g_lds.abort = 1;
  }
  __syncthreads();
}

// A value another workgroup of the XCD wrote before the last barrier.
template <typename T>
__device__ __forceinline__ T cover_ld(const T *p) {
  return __hip_atomic_load(as_global(const_cast<T *>(p)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Number of a word in level order, and back (its own inverse).
__device__ __forceinline__ uint32_t cover_number(uint32_t x, int n, bool reversed) {
  const uint32_t mask = (1u << n) - 1u;
  return reversed ? (__builtin_bitreverse32(~x & mask) >> (32 - n)) : x;
}

// Bits whose index differs from a set bit's in exactly one place.
__device__ __forceinline__ unsigned long long one_off(unsigned long long t) {
  return ((t & 0x5555555555555555ull) << 1) | ((t >> 1) & 0x5555555555555555ull) |
         ((t & 0x3333333333333333ull) << 2) | ((t >> 2) & 0x3333333333333333ull) |
         ((t & 0x0f0f0f0f0f0f0f0full) << 4) | ((t >> 4) & 0x0f0f0f0f0f0f0f0full) |
         ((t & 0x00ff00ff00ff00ffull) << 8) | ((t >> 8) & 0x00ff00ff00ff00ffull) |
         ((t & 0x0000ffff0000ffffull) << 16) | ((t >> 16) & 0x0000ffff0000ffffull) | (t << 32) | (t >> 32);
}

// OR over the 16 lanes of a row.
__device__ __forceinline__ unsigned long long row_or(unsigned long long x) {
  unsigned int lo = (unsigned int)x, hi = (unsigned int)(x >> 32);
#define GC_ROW_OR(ror)                                                                        \
  lo |= (unsigned int)__builtin_amdgcn_update_dpp(0, (int)lo, 0x120 + ror, 0xf, 0xf, true);   \
  hi |= (unsigned int)__builtin_amdgcn_update_dpp(0, (int)hi, 0x120 + ror, 0xf, 0xf, true);
  GC_ROW_OR(1)
  GC_ROW_OR(2)
  GC_ROW_OR(4)
  GC_ROW_OR(8)
#undef GC_ROW_OR
  return ((unsigned long long)hi << 32) | lo;
}

// Candidates of a word (all of one index weight) with an earlier one of the
// same word at distance 2: a set bit whose index has i in place of a lower j.
__device__ __forceinline__ unsigned long long earlier_in_word(unsigned long long a) {
  constexpr unsigned long long in[6] = {0xaaaaaaaaaaaaaaaaull, 0xccccccccccccccccull, 0xf0f0f0f0f0f0f0f0ull,
                                        0xff00ff00ff00ff00ull, 0xffff0000ffff0000ull, 0xffffffff00000000ull};
  unsigned long long b = 0;
#pragma unroll
  for (int i = 1; i < 6; ++i)
#pragma unroll
    for (int j = 0; j < i; ++j) b |= (a & in[j] & ~in[i]) << ((1 << i) - (1 << j));
  return b;
}

// Marks balls in words w[0 .. K) of the slice.  Most marks of a code repeat
// others (about 36 per word of the space at n = 24, d = 4): a read is cheaper
// than the atomic it saves.
template <int K>
__device__ __forceinline__ void cover_mark(CoverLds &C, const unsigned int (&w)[K], const unsigned long long (&ball)[K]) {
  unsigned long long old[K];
#pragma unroll
  for (int q = 0; q < K; ++q) old[q] = C.dead[w[q]];
#pragma unroll
  for (int q = 0; q < K; ++q)
    if (ball[q] & ~old[q])
      __hip_atomic_fetch_or(&C.dead[w[q]], ball[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The distance to build with.  Words of one parity (a weight, or self-orthogonal)
// are at even distances: an even d is met by d - 1, whose balls have a third of
// the words (n = 24, weight 10, d = 6: 1.67 and 1.28 ms).  Not after a prefix, whose words
// may be any; and d = 2 stays.
__device__ __forceinline__ int cover_distance(const Lds &L) {
  const unsigned long long all = (2ull << L.n) - 1, even = 0x5555555555555555ull;
  const bool one_parity = (L.classes & all & even) == 0 || (L.classes & all & ~even) == 0;
  return one_parity && L.m_start == 0 && L.d > 2 ? (L.d - 1) | 1 : L.d;
}

// Builds the job's code with the first `team` workgroups of the XCD (this one
// is number `rank`); writes the words and the count.  Not inlined: the
// screens' registers are not affected.
__device__ __noinline__ void cover_team(CoverWs *ws_v, Ctl *ctl_v, unsigned int rank_v, unsigned int team_v, int *abort_v,
                                        unsigned int limit) {
  // Arguments are the same for every lane: pointers in scalar registers.
  CoverWs *const ws = uniform_ptr(ws_v);
  Ctl *const ctl = uniform_ptr(ctl_v);
  int *const abort_flag = uniform_ptr(abort_v);
  Lds &L = g_lds;
  CoverLds &C = g_lds.cover;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned int rank = __builtin_amdgcn_readfirstlane(rank_v), team = __builtin_amdgcn_readfirstlane(team_v);
  const int n = __builtin_amdgcn_readfirstlane(L.n), d = __builtin_amdgcn_readfirstlane(cover_distance(L));
  const bool rev = L.ord == GC_GREVLEX;
  const int slice_bits = __builtin_ctz(team);
  const unsigned int words = n > 6 ? 1u << (n - 6 - slice_bits) : 1u;  // words of this slice
  const int hbits = __builtin_ctz(words);                              // word-index bits of a slice
  const unsigned int high = rank << hbits;
  const unsigned long long valid = n < 6 ? (1ull << (1 << n)) - 1 : ~0ull;
  uint32_t *const code = uniform_ptr(L.code);
  const unsigned long long capacity = uniform64(L.capacity), start = uniform64(L.p_start), stop = uniform64(L.total);
  unsigned long long m = uniform64(L.m_start);
  unsigned int rounds = 0;

  // Tables, and the empty slice.
  if (tid == 0) {
    unsigned int at = 0;
    for (int j = 0; j < d; ++j) {
      C.cum[j] = at;
      at += j == 0 ? 1 : j == 1 ? hbits : j == 2 ? hbits * (hbits - 1) / 2 : hbits * (hbits - 1) * (hbits - 2) / 6;
    }
    C.cum[d] = at;
    C.epoch = 0;
  }
  for (int i = tid; i < d * 64; i += kBlock) {
    unsigned long long b = 0;
    for (int x = 0; x < 64; ++x)
      if (__builtin_popcount(x ^ (i & 63)) <= (i >> 6)) b |= 1ull << x;
    C.ball[i >> 6][i & 63] = b;
  }
  __syncthreads();
  if (tid < (int)team) {
    unsigned int place = 0;
    for (unsigned int x = 0; x < team; ++x) {
      const int a = __builtin_popcount(x), b = __builtin_popcount((unsigned int)tid);
      place += a < b || (a == b && x < (unsigned int)tid);
    }
    C.other[place] = (uint8_t)tid;
  }
  if (tid < 64) {
    unsigned long long b = 0;
    for (int x = 0; x < 64; ++x)
      if (__builtin_popcount(x) == tid - 32) b |= 1ull << x;
    C.level[tid] = b;
  }
  if (tid == 0) C.dead[kCovWords] = ~0ull;
  if (team > 1 && rank == 0 && tid < 32) ws->active[(1u << (kCovMaxN - 6)) + tid] = 0;
  // Differences of weight j, in increasing order: each finds its place by its
  // rank among the numbers of its weight (C(b, 1) + C(b', 2) + ...).
  for (unsigned int w = tid; w < words; w += kBlock) {
    const int j = __builtin_popcount(w);
    if (j < d) {
      unsigned int place = C.cum[j], k = 1;
      for (unsigned int b = w; b; b &= b - 1, ++k) {
        const unsigned int p = __builtin_ctz(b);
        place += k == 1 ? p : k == 2 ? p * (p - 1) / 2 : p * (p - 1) * (p - 2) / 6;
      }
      C.diff[place] = (uint16_t)w;
    }
    C.dead[w] = ~valid;
    if (team > 1) as_global(ws->active)[high + w] = 0;
  }
  __syncthreads();
  // Words accepted before `start` (a resumed construction): their first n
  // bits, as on the matrix screens.
  for (unsigned long long i = tid; i < m; i += kBlock) {
    const uint32_t c = cover_number(code[i] & ((1u << n) - 1u), n, rev);
    const int r = d - 1 - __builtin_popcount((c >> 6 >> hbits) ^ rank);
    if (r >= 0)
      for (unsigned int e = 0; e < C.cum[r + 1]; ++e)
        cover_mark<1>(C, {((c >> 6) ^ C.diff[e]) & (words - 1)}, {C.ball[r - __builtin_popcount(C.diff[e])][c & 63]});
  }

  unsigned int steps[kCovMaxD], places[kCovMaxD];  // by radius, for fewer than 64 differences
#pragma unroll
  for (int r = 0; r < kCovMaxD; ++r) {
    const unsigned int per = r < d ? C.cum[r + 1] : 64;
    steps[r] = per < 64 ? 64 / per : 1;
    places[r] = per < 64 ? (unsigned int)lane / per : 0;
  }
  // Marks of the words accepted in the round with parity `par` (C.cnt).  A
  // slice at distance k from this one is left a radius of r = d - 1 - k, its
  // words `per` marks each.  A lane keeps its difference (and, for small
  // `per`, its place among the 64 / per words of a step), so a mark is an
  // XOR, one LDS read and one LDS atomic.
  auto mark_slice = [&](unsigned int par, unsigned int s, int r, unsigned int part, unsigned int parts) {
    const bool own = s == rank;
    const unsigned int all = __builtin_amdgcn_readfirstlane(C.cnt[s]);
    if (all == 0) return;
    const unsigned int per = __builtin_amdgcn_readfirstlane(C.cum[r + 1]);
    const uint32_t *seg = ws->seg[par][s];
    const unsigned int step = r == 0 ? steps[0] : r == 1 ? steps[1] : r == 2 ? steps[2] : steps[3];
    const unsigned int place = r == 0 ? places[0] : r == 1 ? places[1] : r == 2 ? places[2] : places[3];
    const unsigned int chunks = (per + 63) / 64;
    if (place >= step) return;
    for (unsigned int u = part; u < chunks * parts; u += parts) {  // (difference chunk, part of the words)
      const unsigned int e = per < 64 ? (unsigned int)lane - place * per : 64 * (u / parts) + lane;
      if (e >= per) continue;
      const unsigned int diff = C.diff[e];
      const unsigned long long *ball = C.ball[r - __builtin_popcount(diff)];
      for (unsigned int k = part * step + place; k < all; k += 4 * parts * step) {
        uint32_t c[4];
        unsigned int w[4];
        unsigned long long b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const unsigned int at = umin(k + q * parts * step, all - 1);
          c[q] = own && all <= kCovOwn ? C.own[at] : cover_ld(&seg[at]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          w[q] = ((c[q] >> 6) ^ diff) & (words - 1);
          b[q] = ball[c[q] & 63];
        }
        cover_mark<4>(C, w, b);
      }
    }
  };
  auto mark_round = [&](unsigned int par) {
    mark_slice(par, rank, d - 1, wave, kWaves);
    // The slices at distance k: C(slice_bits, k) of them, shared out to the
    // waves (several waves a slice where there are fewer slices).
    unsigned int at = 1, of = (unsigned int)slice_bits;
    for (int k = 1; k < d && k <= slice_bits; ++k) {
      const unsigned int parts = of < (unsigned int)kWaves ? kWaves / of : 1;
      for (unsigned int i = wave; i < of * parts; i += kWaves)
        mark_slice(par, rank ^ C.other[at + i / parts], d - 1 - k, i % parts, parts);
      at += of;
      of = of * (unsigned int)(slice_bits - k) / (unsigned int)(k + 1);
    }
    __syncthreads();
  };
  // Bits of the level (weight k) in word w, all of one index weight.
  auto level_mask = [&](int k, unsigned int w) { return C.level[32 + k - __builtin_popcount(high + w)]; };

  unsigned int par = 0;
  bool pending = false;
  for (int w = 0; w <= n; ++w) {
    const unsigned long long at = L.tab.off[w], end = L.tab.off[w + 1];
    const unsigned long long lo = start > at ? start - at : 0, hi = stop < end ? (stop > at ? stop - at : 0) : end - at;
    if (lo >= hi) continue;
    const int k = rev ? n - w : w;  // weight of the level's numbers
    if (pending) mark_round(par ^ 1);
    pending = false;
    __syncthreads();
    // The level's candidates; positions outside [start, stop) are none.
    const unsigned long long from = lo > 0 ? unrank_weight(L.tab, lo, k, n) : 0;
    const unsigned long long to = hi < end - at ? unrank_weight(L.tab, hi, k, n) : 1ull << n;
    if (tid == 0) C.qn = C.accn = 0;
    __syncthreads();
    for (unsigned int i0 = 0; i0 < words; i0 += kBlock) {
      const unsigned int i = i0 + tid;
      unsigned long long a = 0;
      if (i < words) {
        const unsigned long long mask = level_mask(k, i), base = 64ull * (high + i);
        unsigned long long in = ~0ull;
        if (base < from) in = from - base >= 64 ? 0ull : ~0ull << (from - base);
        if (base + 64 > to) in &= to <= base ? 0ull : ~0ull >> (64 - (to - base));
        if (mask & ~in) C.dead[i] |= mask & ~in;
        a = mask & ~C.dead[i];
        C.acc[i] = 0;
        if (team > 1) as_global(ws->active)[high + i] = a;
      }
      const unsigned long long any = ballot(a != 0);
      unsigned int q = 0;
      if (lane == 0 && any) q = atomicAdd(&C.qn, (unsigned int)__builtin_popcountll(any));
      q = __builtin_amdgcn_readfirstlane(q);
      if (a) C.queue[q + __builtin_popcountll(any & lanemask_lt())] = (uint16_t)i;
    }
    __syncthreads();
    if (tid == 0 && team > 1) as_global(ws->slot[par])[rank] = C.qn;
    cover_barrier(ws, team, abort_flag, limit);
    if (L.abort) return;
    // Anything to do in any slice?  (The parity of the slots moves on with
    // every barrier: a slot is written again two barriers after it was read.)
    if (wave == 0) {
      const unsigned int left = team == 1 ? C.qn : (unsigned int)lane < team ? (unsigned int)cover_ld(&ws->slot[par][lane]) : 0u;
      const unsigned long long any = ballot(left != 0);
      if (lane == 0) C.open = any != 0;
    }
    par ^= 1;
    __syncthreads();
    bool open = C.open != 0;
    while (open) {
      // What the last round's words leave of the queued candidates.
      if (pending) {
        mark_round(par ^ 1);
        const unsigned int had = C.qn;
        __syncthreads();
        if (tid == 0) C.qn = 0;
        for (unsigned int i0 = 0; i0 < had; i0 += kBlock) {
          const unsigned int i = i0 + tid;
          unsigned int w_ = 0;
          unsigned long long a = 0;
          if (i < had) {
            w_ = C.queue[i];
            a = level_mask(k, w_) & ~C.dead[w_];
            if (team > 1) as_global(ws->active)[high + w_] = a;
          }
          __syncthreads();  // this part of the queue is read: kept entries go to places before its end
          const unsigned long long any = ballot(a != 0);
          unsigned int q = 0;
          if (lane == 0 && any) q = atomicAdd(&C.qn, (unsigned int)__builtin_popcountll(any));
          q = __builtin_amdgcn_readfirstlane(q);
          if (a) C.queue[q + __builtin_popcountll(any & lanemask_lt())] = (uint16_t)w_;
        }
      }
      if (tid == 0) {
        C.segn = C.left = 0;
        C.seg_ok = kCovSeg;
      }
      __syncthreads();
      const unsigned int queued = C.qn;
      bool left = false;
      for (unsigned int i0 = 0; i0 < queued; i0 += kBlock) {
        const unsigned int i = i0 + tid;
        const bool have = i < queued;
        const unsigned int w_ = have ? C.queue[i] : 0, H = high + w_;
        const unsigned long long a = have ? level_mask(k, w_) & ~C.dead[w_] : 0ull;
        unsigned long long free = a;
        if (d > 2 && a) {
          free &= ~earlier_in_word(a);
          // One index bit of the word moved into the bits below 64, then one
          // moved down with the same bits below 64.  Reads go out in eights
          // (past the last one: a word without candidates).
          if (free) {
            unsigned long long t = 0;
            for (unsigned int b = w_; b;) {
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                t |= ~C.dead[b ? w_ ^ (b & -b) : (unsigned int)kCovWords];
                b &= b - 1;
              }
            }
            free &= ~one_off(t & level_mask(k, w_ & (w_ - 1)));
          }
          for (unsigned int b = w_; b && free; b &= b - 1) {
            const unsigned int bi = b & -b;
            unsigned long long t = 0;
            for (unsigned int c = ~w_ & (bi - 1); c;) {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                t |= ~C.dead[c ? w_ ^ bi ^ (c & -c) : (unsigned int)kCovWords];
                c &= c - 1;
              }
            }
            free &= ~t;
          }
        }
        // The same with a slice bit: the words are another workgroup's.
        if (d > 2 && rank) {
          constexpr unsigned int none = 1u << (kCovMaxN - 6);
          unsigned long long rest = ballot(free != 0);
          if (__builtin_popcountll(rest) <= kCovShared) {
            // Few words are left: 16 lanes share one, a lane the moves into
            // one index bit (and one more past bit 16), four words at a time,
            // so that all reads of a word are out at once.
            while (rest) {
              unsigned int from_lane[4];
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                from_lane[g] = rest ? (unsigned int)__builtin_ctzll(rest) : 64u;
                rest &= rest - 1;
              }
              const int g = lane >> 4;
              const unsigned int src = g == 0 ? from_lane[0] : g == 1 ? from_lane[1] : g == 2 ? from_lane[2] : from_lane[3];
              const unsigned int gH = high + __builtin_amdgcn_ds_bpermute(4 * (src & 63), (int)w_);
              const unsigned int l = lane & 15;
              unsigned long long t1 = 0, t2 = 0;
#pragma unroll
              for (int q = 0; q < 5; ++q) {
                const unsigned int b = high & (words << q);  // uniform
                if (b == 0) continue;
                const unsigned int c = ~gH & (1u << l) & (b - 1), c2 = l < 2 ? ~gH & (0x10000u << l) & (b - 1) : 0u;
                t2 |= cover_ld(&ws->active[c && src < 64 ? gH ^ b ^ c : none]);
                t2 |= cover_ld(&ws->active[c2 && src < 64 ? gH ^ b ^ c2 : none]);
                if ((int)l == q) t1 = cover_ld(&ws->active[src < 64 ? gH ^ b : none]);
              }
              t1 = row_or(t1);
              t2 = row_or(t2) | one_off(t1);
#pragma unroll
              for (int g2 = 0; g2 < 4; ++g2) {
                const unsigned long long got =
                    ((unsigned long long)(unsigned int)__builtin_amdgcn_readlane((int)(t2 >> 32), 16 * g2) << 32) |
                    (unsigned int)__builtin_amdgcn_readlane((int)t2, 16 * g2);
                if ((unsigned int)lane == from_lane[g2]) free &= ~got;
              }
            }
          } else if (free) {
            // Each lane its own word: the moves of one bit go out with the
            // first moves of two.
            unsigned long long t = 0;
#pragma unroll
            for (int q = 0; q < 5; ++q) {
              const unsigned int b = high & (words << q);
              t |= cover_ld(&ws->active[b ? H ^ b : none]);
            }
            unsigned int left_bits = high & (high - 1), bi = high & -high, c = ~H & (bi - 1);
            do {
              unsigned long long t2 = 0;
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                t2 |= cover_ld(&ws->active[c ? H ^ bi ^ (c & -c) : none]);
                c &= c - 1;
                if (!c) {
                  bi = left_bits & -left_bits;
                  left_bits &= left_bits - 1;
                  c = ~H & (bi - 1) & (bi ? ~0u : 0u);
                }
              }
              free &= ~(t2 | one_off(t));
              t = 0;
            } while (free && (c || left_bits));
          }
        }
        if (free) {
          const unsigned int count = (unsigned int)__builtin_popcountll(free);
          unsigned int at_ = atomicAdd(&C.segn, count);
          if (at_ + count > kCovSeg) {  // no room: accepted in a later round
            atomicMin(&C.seg_ok, at_);
            free = 0;
          } else {
            C.acc[w_] |= free;
            for (unsigned long long f = free; f; f &= f - 1, ++at_) {
              const uint32_t c = 64u * H + __builtin_ctzll(f);
              if (at_ < kCovOwn) C.own[at_] = c;
              as_global(ws->seg[par][rank])[at_] = c;
            }
          }
        }
        left |= (a & ~free) != 0;
      }
      if (ballot(left) && lane == 0) C.left = 1;
      __syncthreads();
      if (tid == 0) {
        const unsigned int fresh = C.segn < C.seg_ok ? C.segn : C.seg_ok;
        const unsigned int total = C.accn + fresh;
        const unsigned long long report = ((unsigned long long)total << 32) | (fresh << 1) | C.left;
        if (team > 1) as_global(ws->slot[par])[rank] = report;
        C.accn = total;
        C.cnt[0] = fresh;      // team == 1
        C.total[0] = total;
        C.open = C.left;
      }
      cover_barrier(ws, team, abort_flag, limit);
      if (L.abort) return;
      if (team > 1 && wave == 0) {
        const unsigned long long r = (unsigned int)lane < team ? cover_ld(&ws->slot[par][lane]) : 0ull;
        const unsigned long long any = ballot((r & 1) != 0);
        if ((unsigned int)lane < team) {
          C.cnt[lane] = (unsigned int)(r & 0xffffffffu) >> 1;
          C.total[lane] = (unsigned int)(r >> 32);
        }
        if (lane == 0) C.open = any != 0;
      }
      __syncthreads();
      open = C.open != 0;
      pending = true;
      par ^= 1;
      // Every second round at the latest accepts the earliest candidate left:
      // the limit is never met, and like every wait's it ends the launch.
      if (open && ++rounds > kCovMaxRounds) {
        if (tid == 0) {
          __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          L.abort = 1;
        }
        return;
      }
    }
    if (!pending) continue;  // an empty level
    // The level's words, in increasing order of their numbers.
    unsigned long long base = m;
    unsigned long long all = 0;
    for (unsigned int s = 0; s < team; ++s) {
      if (s < rank) base += C.total[s];
      all += C.total[s];
    }
    const unsigned int per = (words + kBlock - 1) / kBlock, w0 = tid * per;
    unsigned int mine = 0;
    for (unsigned int i = w0; i < w0 + per && i < words; ++i) mine += (unsigned int)__builtin_popcountll(C.acc[i]);
    const unsigned int incl = wave_scan(mine);
    if (lane == 63) C.wsum[wave] = incl;
    __syncthreads();
    base += incl - mine;
    for (int wv = 0; wv < wave; ++wv) base += C.wsum[wv];
    for (unsigned int i = w0; i < w0 + per && i < words; ++i)
      for (unsigned long long f = C.acc[i]; f; f &= f - 1, ++base)
        if (base < capacity) as_global(code)[base] = cover_number(64u * (high + i) + __builtin_ctzll(f), n, rev);
    m += all;
    if (m > capacity) break;
    __syncthreads();
  }
  if (rank == 0 && tid == 0) {
    if (m > capacity) set_status(ctl, GC_ECAPACITY);
    ctl->m = m < capacity ? m : capacity;
    ctl->stat_rounds = rounds;
  }
}

#include "cover_windows.h"

// Windows or rounds.  Windows for larger distances, and where codes are small:
// a round passes every level (4 us, with few candidates) and decides what one
// workgroup does for itself in a window (rounds and windows: n = 10, d = 3 105
// and 56 us; n = 16, d = 4 288 and 241 us; n = 18, d = 3 739 and 706 us; n = 20,
// d = 3 1.14 and 2.47 ms; distance 2, where a level is one round: n = 9 63 and
// 61 us, n = 12 85 and 174 us).
constexpr bool cover_by_windows(int n, int d, bool self) {
  return self || d > kCovMaxD || n <= (d > 2 ? 18 : 9);
}

// A graded code by cover marks.  The team's workgroups on one XCD build it,
// while the others wait at the barrier that ends the job: as many (a power of
// two) as give each 512 words or more (rounds, n = 20, d = 3: 1.22 ms with 32
// workgroups, 1.52 ms with 8, 2.22 ms with 2; windows, n = 14, d = 5: 102 us
// with one, 120 us with 32; n = 18, d = 5 216 us with 8, 230 us with 4), by
// rounds more than one from 2048 words on (n = 16: 368 us with one, 429 us with
// two), at distance 2 256 words or more (n = 17: 179 us, with 512 231 us).
// False (alike in every workgroup) when the slices would not fit.
constexpr unsigned int cover_team_size(int n, int d, bool self, unsigned int workgroups) {
  const unsigned int words = n > 6 ? 1u << (n - 6) : 1u, most = workgroups < kCovTeam ? workgroups : kCovTeam;
  const unsigned int least = cover_by_windows(n, d, self) ? 512u : d == 2 ? 256u : words > 1024 ? 512u : 1024u;
  unsigned int team = 1;
  while (2 * team <= most && words / (2 * team) >= least) team *= 2;
  return team;
}

template <bool kSelf>
__device__ __forceinline__ bool build_cover(Lds &L, const TeamWs &W, int *abort_flag, unsigned int limit) {
  const unsigned int words = L.n > 6 ? 1u << (L.n - 6) : 1u, team = cover_team_size(L.n, L.d, kSelf, L.sub_size);
  if (words / team > (unsigned int)kCovWords) return false;
  if (L.sub_rank < team) {
    if (cover_by_windows(L.n, L.d, kSelf)) cover_window_team<kSelf>(W.cover, W.ctl, L.sub_rank, team, abort_flag, limit);
    else cover_team(W.cover, W.ctl, L.sub_rank, team, abort_flag, limit);
  }
  return true;
}
