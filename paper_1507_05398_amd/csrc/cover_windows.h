// cover_windows.h -- graded codes of distance 5 and more for n <= 24 from the
// same bitmap as cover_build.h (included by it), in windows.
//
// With a larger distance a level takes many short rounds, each a walk over
// many neighbour words.  Here the team lists the first 1024 undecided
// candidates in walk order, and every workgroup finds the greedy's choice
// among them for itself: a wave holds the conflicts inside its block of 64
// candidates, the blocks are decided in turn, and the later ones compare
// themselves with the words accepted (three instructions a pair, and of 1024
// candidates some 110 are accepted at n = 22, d = 5).  Each workgroup then
// marks the balls of the accepted words in its slice, which removes every
// candidate of the window.  One XCD-local barrier a window, after the lists.
// (With the whole conflict graph, shared out to the team, and a second
// barrier: n = 22, d = 5 884 us against 805 us, n = 10, d = 5 73 and 53 us.)
//
// Self-orthogonal codes (kSelf; every distance): a pair clashes also when its
// overlap is odd, and of the words accepted so far a basis is kept.  A new
// basis word (at most n / 2 times) removes the candidates it overlaps oddly
// from the bitmap, a word of 64 at a time.
//
// What bounds it: about 21 us a window at n = 22, d = 5 (listing 2.6, waiting
// for the busiest slice 3.5, gathering 1.7, choice 10, marks 3.4), and
// from n = 24 on the LDS throughput of the marks, uneven over the slices: a
// window's words are neighbours in the walk, so the slices near them mark
// most (slices taken from lower bits, which share the marks evenly, need a
// merge of the lists: n = 24, d = 6 2.35 ms against 2.53 ms, but n = 22, d = 5
// 1.05 ms against 0.95 ms).

// Bits 0 .. 63: which of the 64 words at `w` (broadcast reads) are closer than
// d to x.  XOR, a population count that starts at -d, and its sign shifted
// into the mask.  kSelf: or have an odd overlap with it, counted from `odd`.
template <bool kSelf>
__device__ __forceinline__ unsigned long long clash_mask(const uint32_t *w, uint32_t x, int d, unsigned int odd) {
  auto sign = [&](uint32_t y) {
    const unsigned int t = (unsigned int)(__builtin_popcount(x ^ y) - d);
    return kSelf ? t | ((__builtin_popcount(x & y) + odd) << 31) : t;
  };
  unsigned int half[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    unsigned int m = 0;
    const uint4 *v = reinterpret_cast<const uint4 *>(w + 32 * h);
#pragma unroll
    for (int q = 7; q >= 0; --q) {
      const uint4 c = v[q];
      m = __builtin_amdgcn_alignbit(m, sign(c.w), 31);
      m = __builtin_amdgcn_alignbit(m, sign(c.z), 31);
      m = __builtin_amdgcn_alignbit(m, sign(c.y), 31);
      m = __builtin_amdgcn_alignbit(m, sign(c.x), 31);
    }
    half[h] = m;
  }
  return ((unsigned long long)half[1] << 32) | half[0];
}

template <bool kSelf>
__device__ __noinline__ void cover_window_team(CoverWs *ws_v, Ctl *ctl_v, unsigned int rank_v, unsigned int team_v,
                                               int *abort_v, unsigned int limit) {
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
  const unsigned int words = n > 6 ? 1u << (n - 6 - slice_bits) : 1u;
  const int hbits = __builtin_ctz(words);
  const unsigned int high = rank << hbits;
  const unsigned long long valid = n < 6 ? (1ull << (1 << n)) - 1 : ~0ull;
  uint32_t *const code = uniform_ptr(L.code);
  const unsigned long long capacity = uniform64(L.capacity), start = uniform64(L.p_start), stop = uniform64(L.total);
  unsigned long long m = uniform64(L.m_start);
  const bool given = m > 0;  // words before `start`: any, not always of a self-orthogonal code
  // Overlap of two even words by their numbers: the bits both have, plus n
  // for complemented ones.
  const unsigned int odd = rev ? (unsigned int)n & 1u : 0u, all_bits = (1u << n) - 1u;

  // Tables: differences of the word index by weight (C(hbits, j) of weight j),
  // balls, level masks; the empty slice.
  if (tid == 0) {
    unsigned int at = 0, of = 1;
    for (int j = 0; j < 15; ++j) {
      C.wcum[j] = at;
      at += of;
      of = j < hbits ? of * (unsigned int)(hbits - j) / (unsigned int)(j + 1) : 0;
    }
    C.epoch = 0;
    C.dim = C.pick = 0;
  }
  if (tid < 8 * 64) {
    unsigned long long b = 0;
    for (int x = 0; x < 64; ++x)
      if (__builtin_popcount(x ^ (tid & 63)) < (tid >> 6)) b |= 1ull << x;
    C.wball[tid >> 6][tid & 63] = b;
  } else if (tid >= 512 && tid < 576) {
    unsigned long long b = 0;
    for (int x = 0; x < 64; ++x)
      if (__builtin_popcount(x) == tid - 512 - 32) b |= 1ull << x;
    C.level[tid - 512] = b;
  }
  __syncthreads();
  for (unsigned int w = tid; w < words; w += kBlock) {
    const int j = __builtin_popcount(w);
    // Rank among the numbers of its weight: C(b, 1) + C(b', 2) + ...
    unsigned int place = C.wcum[j], k = 1;
    for (unsigned int b = w; b; b &= b - 1, ++k) {
      const unsigned int p = __builtin_ctz(b);
      if (p >= k) place += L.tab.binom[p][k];
    }
    C.wdiff[place] = (uint16_t)w;
    C.dead[w] = ~valid;
  }
  __syncthreads();

  // Marks the balls around four numbers (uniform; `past`: distance that lies
  // past the n bits), by one wave: a lane takes a difference of the word index
  // for all of them.  Instructions bound this
  // loop, so a mark is few of them: the slice's byte offset is one XOR, the
  // ball's row one sum and one clamp (row 0, radius -1, is empty: differences
  // of too much weight need no test).
  auto mark4 = [&](const uint32_t (&c)[4], int have, const int (&past)[4]) {
    int row[4];
    unsigned int at[4], most = 0;
    unsigned int bit[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int left = d - 1 - past[q] - __builtin_popcount((c[q] >> 6 >> hbits) ^ rank), r = q < have && left >= 0 ? left : -1;
      row[q] = 64 * (r + 1);
      at[q] = (c[q] >> 6) & (words - 1);
      bit[q] = c[q] & 63;
      const unsigned int per = r < 0 ? 0u : (unsigned int)__builtin_amdgcn_readfirstlane((int)C.wcum[r + 1 < 14 ? r + 1 : 14]);
      most = per > most ? per : most;
    }
    for (unsigned int e = lane; e < most; e += 64) {
      const unsigned int diff = C.wdiff[e];
      const int weight = 64 * __builtin_popcount(diff);
      unsigned long long b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        int o = row[q] - weight;
        o = o < 0 ? 0 : o > 7 * 64 ? 7 * 64 : o;
        b[q] = (&C.wball[0][0])[o + (int)bit[q]];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        __hip_atomic_fetch_or(&C.dead[at[q] ^ diff], b[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  };
  // kSelf: candidates with an odd overlap with one of the words whose reversed
  // (grevlex) or plain bits are `b` (one a thread, 0: none) leave the bitmap;
  // the bitmap is not marked meanwhile.  The words' span is kept as a basis,
  // each vector without the top bits of those before it.
  auto keep_orthogonal = [&](uint32_t b) {
    for (;;) {
      const int dim = C.dim;
      for (int i = 0; i < dim; ++i)
        if ((b >> (31 - __builtin_clz(C.basis[i]))) & 1) b ^= C.basis[i];
      if (b) atomicMax(&C.pick, b);
      __syncthreads();
      const uint32_t pick = C.pick;
      __syncthreads();  // every wave has read it: a wave that leaves may raise the next call's at once
      if (pick == 0) break;
      if (tid == 0) {
        C.basis[dim] = pick;
        C.dim = dim + 1;
        C.pick = 0;
      }
      constexpr unsigned long long in[6] = {0xaaaaaaaaaaaaaaaaull, 0xccccccccccccccccull, 0xf0f0f0f0f0f0f0f0ull,
                                            0xff00ff00ff00ff00ull, 0xffff0000ffff0000ull, 0xffffffff00000000ull};
      unsigned long long low = rev && (__builtin_popcount(pick) & 1) ? ~0ull : 0ull;
#pragma unroll
      for (int j = 0; j < 6; ++j) low ^= (pick >> j) & 1 ? in[j] : 0ull;
      for (unsigned int i = tid; i < words; i += kBlock)
        C.dead[i] |= __builtin_popcount((high + i) & (pick >> 6)) & 1 ? ~low : low;
      __syncthreads();
    }
  };
  // Words accepted before `start`: their first n bits as on the matrix
  // screens; self-orthogonal codes count the others in the distance, as the
  // screens of the vector ALU do.
  for (unsigned long long i = 4 * wave; i < m; i += 4 * kWaves) {
    uint32_t c[4];
    int past[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t x = code[i + q < m ? i + q : i];
      c[q] = cover_number(x & all_bits, n, rev);
      past[q] = kSelf ? __builtin_popcount(x >> n) : 0;
    }
    mark4(c, m - i < 4 ? (int)(m - i) : 4, past);
  }
  __syncthreads();
  if (kSelf)
    for (unsigned long long i = 0; i < m; i += kBlock) {
      const uint32_t x = i + tid < m ? code[i + tid] & all_bits : 0u;
      keep_orthogonal(rev ? __builtin_bitreverse32(x) >> (32 - n) : x);
    }

  // Walk levels with positions in [start, stop); candidates outside are none.
  int first = n + 1, last = -1;
  unsigned int walked = 0;  // levels with candidates, by the weight of their numbers
  for (int w = 0; w <= n; ++w) {
    const unsigned long long at = L.tab.off[w], end = L.tab.off[w + 1];
    const unsigned long long lo = start > at ? start - at : 0, hi = stop < end ? (stop > at ? stop - at : 0) : end - at;
    if (lo >= hi) continue;
    if (first > n) first = w;
    last = w;
    const int k = rev ? n - w : w;
    walked |= 1u << k;
    if (lo == 0 && hi == end - at) continue;
    const unsigned long long from = lo > 0 ? unrank_weight(L.tab, lo, k, n) : 0;
    const unsigned long long to = hi < end - at ? unrank_weight(L.tab, hi, k, n) : 1ull << n;
    __syncthreads();  // the marks: a word's bits are set here without an atomic
    for (unsigned int i = tid; i < words; i += kBlock) {
      const unsigned long long base = 64ull * (high + i);
      unsigned long long in = ~0ull;
      if (base < from) in = from - base >= 64 ? 0ull : ~0ull << (from - base);
      if (base + 64 > to) in &= to <= base ? 0ull : ~0ull >> (64 - (to - base));
      C.dead[i] |= C.level[32 + k - __builtin_popcount(high + i)] & ~in;
    }
  }
  __syncthreads();

  if (walked != (2u << n) - 1u) {
    if (tid < 32) {
      unsigned long long none = 0;
      for (int j = 0; j <= 6; ++j)
        if (tid + j > n || !((walked >> (tid + j)) & 1)) none |= C.level[32 + j];
      C.none[tid] = none;
    }
    __syncthreads();
    for (unsigned int i = tid; i < words; i += kBlock) C.dead[i] |= C.none[__builtin_popcount(high + i)];
    __syncthreads();
  }
  // Clock cycles of an accepted word's marks (a third of a cycle each, the
  // ball's words even over the slices), of one comparison of 1024 candidates
  // with a word, and of listing 1024 candidates.
  unsigned int near_words = 0;
  for (int j = 0; j < d && j <= n - 6; ++j) near_words += L.tab.binom[n - 6][j];
  const unsigned int mark_cost = near_words / (3u * team), compare_cost = 48, list_cost = 8000;
  const unsigned int per = (words + kBlock - 1) / kBlock, w0 = tid * per;
  // A slice stops listing further levels once it has more than its share of a
  // window (a window takes a level only if every slice has listed it).
  const unsigned int share = umin(kCovWin, 2 * kCovWin / team);
  unsigned int windows = 0, par = 0;
  int level = first;
  while (level <= last) {
    // This slice's first undecided candidates, level by level; counted four
    // levels at a time (a lane's counts, and a wave's sums, fit 16 bits each).
    unsigned int listed = 0, levels = 0;
    bool cut = false;
    while (levels < (unsigned int)kCovLevels && level + (int)levels <= last && listed < share && !cut) {
      unsigned long long mine = 0;
      const int w4 = level + (int)levels;
      for (unsigned int i = w0; i < w0 + per && i < words; ++i) {
        const unsigned long long left = ~C.dead[i];
        const int k = 32 + (rev ? n - w4 : w4) - __builtin_popcount(high + i);
#pragma unroll
        for (int l = 0; l < 4; ++l)
          mine += (unsigned long long)__builtin_popcountll(left & C.level[rev ? k - l : k + l]) << (16 * l);
      }
      const unsigned int lo2 = wave_scan((unsigned int)mine), hi2 = wave_scan((unsigned int)(mine >> 32));
      const unsigned int buf = 16 * ((levels >> 2) & 1);
      if (lane == 63) C.sums[buf + wave] = make_uint2(lo2, hi2);
      __syncthreads();
      unsigned int at4[4] = {lo2 & 0xffffu, lo2 >> 16, hi2 & 0xffffu, hi2 >> 16}, all4[4] = {};
#pragma unroll
      for (int wv = 0; wv < kWaves; ++wv) {
        const uint2 sum = C.sums[buf + wv];
        const unsigned int of[4] = {sum.x & 0xffffu, sum.x >> 16, sum.y & 0xffffu, sum.y >> 16};
#pragma unroll
        for (int l = 0; l < 4; ++l) {
          if (wv < wave) at4[l] += of[l];
          all4[l] += of[l];
        }
      }
#pragma unroll
      for (int l = 0; l < 4; ++l) {
        if (cut || listed >= share || w4 + l > last) break;
        const unsigned int own = (unsigned int)(mine >> (16 * l)) & 0xffffu;
        unsigned int at = listed + at4[l] - own, all = all4[l];
        if (own && at < (unsigned int)kCovWin)
          for (unsigned int i = w0; i < w0 + per && i < words; ++i) {
            const int k = 32 + (rev ? n - w4 - l : w4 + l) - __builtin_popcount(high + i);
            for (unsigned long long f = C.level[k] & ~C.dead[i]; f && at < (unsigned int)kCovWin; f &= f - 1, ++at)
              as_global(ws->list[par][rank])[at] = 64u * (high + i) + __builtin_ctzll(f);
          }
        if (listed + all > (unsigned int)kCovWin) {
          all = kCovWin - listed;
          cut = true;
        }
        if (tid == 0) as_global(ws->head[par][rank])[2 + levels] = all;
        listed += all;
        ++levels;
      }
    }
    if (tid == 0) {
      as_global(ws->head[par][rank])[0] = levels;
      as_global(ws->head[par][rank])[1] = cut;
    }
    cover_barrier(ws, team, abort_flag, limit);
    if (L.abort) return;
    if (wave == 0) {
      // Candidates of every (level, slice) in walk order; a list cut short
      // ends the window, and so does a level that a slice has not listed.
      const bool in = (unsigned int)lane < team;
      const unsigned int have = in ? cover_ld(&ws->head[par][lane][0]) : (unsigned int)kCovLevels;
      const bool was_cut = in && cover_ld(&ws->head[par][lane][1]) != 0;
      unsigned int num[kCovLevels];
#pragma unroll
      for (int l = 0; l < kCovLevels; ++l) num[l] = in ? cover_ld(&ws->head[par][lane][2 + l]) : 0u;
      unsigned int before = 0, full = 0, from = 0;
      int l = 0;
#pragma unroll
      for (; l < kCovLevels; ++l) {
        if (ballot((int)have <= l)) break;  // a slice has not listed level l
        unsigned int own = num[l];
        // Slices after one whose list was cut in this level do not count.
        const unsigned long long cuts = ballot(was_cut && (int)have == l + 1);
        if (cuts && lane > (int)__builtin_ctzll(cuts)) own = 0;
        const unsigned int at = wave_scan(own);
        if (in) {
          C.run[l * kCovTeam + lane] = make_uint2(before + at - own, from);
          from += own;
        }
        before += (unsigned int)__builtin_amdgcn_readlane((int)at, 63);
        if (!cuts && before <= (unsigned int)kCovWin) full = (unsigned int)l + 1;
        if (cuts || before >= (unsigned int)kCovWin) {
          ++l;
          break;
        }
      }
      if (lane == 0) {
        C.size = before < (unsigned int)kCovWin ? before : (unsigned int)kCovWin;
        C.done_levels = full;
        C.listed = (unsigned int)l;
      }
    }
    __syncthreads();
    const unsigned int size = C.size, complete = C.done_levels;
    // A thread finds its candidate's run (the last one that begins at or before
    // it) and copies it.
    if ((unsigned int)tid < size) {
      unsigned int lo = 0, hi = C.listed * team;
      while (hi - lo > 1) {
        const unsigned int mid = (lo + hi) >> 1;
        if (C.run[(mid >> slice_bits) * kCovTeam + (mid & (team - 1))].x <= (unsigned int)tid) lo = mid;
        else hi = mid;
      }
      const unsigned int slice = lo & (team - 1);
      const uint2 run = C.run[(lo >> slice_bits) * kCovTeam + slice];
      C.cand[tid] = cover_ld(&ws->list[par][slice][run.y + (unsigned int)tid - run.x]);
    }
    __syncthreads();
    // The greedy's choice, a block of 64 candidates a wave: its wave decides a
    // block with the conflicts inside it, once those that clash with a word
    // accepted in an earlier block are out; the later ones compare themselves
    // with its words.
    const unsigned int blocks = (size + 63) / 64;
    const uint32_t x = C.cand[tid];
    unsigned long long row = 0;
    // (A basis of n / 2 words that overlap evenly: the candidates left are in
    // their span, and no pair has an odd overlap.  Given words need not.)
    const bool overlaps = kSelf && (given || 2 * C.dim < n);
    if ((unsigned int)wave < blocks)
      row = overlaps ? clash_mask<kSelf>(&C.cand[64 * wave], x, d, odd) : clash_mask<false>(&C.cand[64 * wave], x, d, odd);
    unsigned int all = 0, least = (unsigned int)tid < size ? ~0u : 0u, mixed = 0;
    for (unsigned int I = 0; I < blocks; ++I) {
      if ((unsigned int)wave == I) {
        __builtin_amdgcn_s_setprio(3);
        // The first candidate left is accepted and takes its neighbours with
        // it (itself among them).
        unsigned long long acc = 0, und = ballot(least >= (unsigned int)d && !(mixed & 1));
        while (und) {
          const int j = __builtin_ctzll(und);
          acc |= 1ull << j;
          und &= ~(((unsigned long long)(unsigned int)__builtin_amdgcn_readlane((int)(row >> 32), j) << 32) |
                   (unsigned int)__builtin_amdgcn_readlane((int)row, j));
        }
        const unsigned int got = (unsigned int)__builtin_popcountll(acc);
        if (lane == 0) C.taken[I] = got;
        if ((acc >> lane) & 1) {
          const unsigned int at = (unsigned int)__builtin_popcountll(acc & lanemask_lt());
          C.took[all + at] = C.block[I & 1][at] = x;
        } else if (acc) {
          // Up to a multiple of eight: the last one again.
          const unsigned int at = got + (unsigned int)__builtin_popcountll(~acc & lanemask_lt());
          if (at < ((got + 7) & ~7u)) C.block[I & 1][at] = (uint32_t)__builtin_amdgcn_readlane((int)x, 63 - (int)__builtin_clzll(acc));
        }
        __builtin_amdgcn_s_setprio(0);
      }
      __syncthreads();
      const unsigned int got = (unsigned int)__builtin_amdgcn_readfirstlane((int)C.taken[I]);
      all += got;
      if ((unsigned int)wave > I && (unsigned int)wave < blocks) {
        if ((unsigned int)wave == I + 1) __builtin_amdgcn_s_setprio(3);
        for (unsigned int i = 0; i < got; i += 8) {
          const uint4 *b = reinterpret_cast<const uint4 *>(&C.block[I & 1][i]);
          const uint4 t = b[0], u = b[1];
          least = umin3(least, dist(x, t.x), dist(x, t.y));
          least = umin3(least, dist(x, t.z), dist(x, t.w));
          least = umin3(least, dist(x, u.x), dist(x, u.y));
          least = umin3(least, dist(x, u.z), dist(x, u.w));
          if (overlaps)
            mixed |= (__builtin_popcount(x & t.x) + odd) | (__builtin_popcount(x & t.y) + odd) |
                     (__builtin_popcount(x & t.z) + odd) | (__builtin_popcount(x & t.w) + odd) |
                     (__builtin_popcount(x & u.x) + odd) | (__builtin_popcount(x & u.y) + odd) |
                     (__builtin_popcount(x & u.z) + odd) | (__builtin_popcount(x & u.w) + odd);
        }
      }
    }
    if (rank == 0 && (unsigned int)tid < all && m + tid < capacity)
      as_global(code)[m + tid] = cover_number(C.took[tid], n, rev);
    __syncthreads();
    m += all;
    if (m > capacity) break;
    // With few candidates left in the slice their distances to the accepted
    // words cost less than the marks (n = 24, d = 8, self-orthogonal: 0.70 ms
    // against 2.0 ms with marks alone).
    unsigned int undecided = 0, mine_at = 0;
    bool compare = false;
    // (Self-orthogonal codes count first: their slices empty soon.  n = 24, d = 6
    // 0.50 and 0.39 ms; plain ones lose 1 % by it.)
    if (all * mark_cost > list_cost + all * (kSelf ? compare_cost / kWaves : compare_cost)) {
      unsigned int mine = 0;
      for (unsigned int i = w0; i < w0 + per && i < words; ++i) mine += (unsigned int)__builtin_popcountll(~C.dead[i]);
      const unsigned int at = wave_scan(mine);
      if (lane == 63) C.wsum[wave] = at;
      __syncthreads();
      mine_at = at - mine;
#pragma unroll
      for (int wv = 0; wv < kWaves; ++wv) {
        if (wv < wave) mine_at += C.wsum[wv];
        undecided += C.wsum[wv];
      }
      const unsigned int passes = undecided / kCovWin + 1;
      const unsigned int some = kSelf && passes == 1 ? undecided | 64 : kCovWin;  // candidates of a pass
      compare = all * mark_cost > passes * (list_cost + all * compare_cost * some / kCovWin);
    }
    if (compare) {
      if (tid < 4 && all + tid < ((all + 3) & ~3u)) C.took[all + tid] = C.took[all - 1];
      // 1024 at a time, the last ones first: what they lose does not move the
      // places of those before them.
      for (unsigned int c1 = (undecided + kCovWin - 1) / kCovWin; c1 > 0; --c1) {
        const unsigned int c0 = (c1 - 1) * kCovWin;
        __syncthreads();
        unsigned int at = mine_at;
        for (unsigned int i = w0; i < w0 + per && i < words; ++i)
          for (unsigned long long f = ~C.dead[i]; f; f &= f - 1, ++at)
            if (at - c0 < (unsigned int)kCovWin) C.cand[at - c0] = 64u * (high + i) + __builtin_ctzll(f);
        __syncthreads();
        // Few candidates: several threads share one's comparisons.
        const unsigned int some = __builtin_amdgcn_readfirstlane(umin(undecided - c0, kCovWin));
        const unsigned int log = some > 64 ? 32 - (unsigned int)__builtin_clz(some - 1) : 6u, parts = kCovWin >> log;
        const unsigned int at_ = (unsigned int)tid & ((1u << log) - 1u);
        if (at_ < some) {
          const uint32_t x = C.cand[at_];
          unsigned int least = ~0u;
          for (unsigned int i = 4 * ((unsigned int)wave >> (log - 6)); i < all; i += 4 * parts) {
            const uint4 t = *reinterpret_cast<const uint4 *>(&C.took[i]);
            least = umin3(least, dist(x, t.x), dist(x, t.y));
            least = umin3(least, dist(x, t.z), dist(x, t.w));
          }
          if (least < (unsigned int)d)
            __hip_atomic_fetch_or(&C.dead[(x >> 6) & (words - 1)], 1ull << (x & 63), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    } else {
      for (unsigned int i = 4 * wave; i < all; i += 4 * kWaves) {
        const uint4 t = *reinterpret_cast<const uint4 *>(&C.took[i]);
        const uint32_t c[4] = {(uint32_t)__builtin_amdgcn_readfirstlane((int)t.x), (uint32_t)__builtin_amdgcn_readfirstlane((int)t.y),
                               (uint32_t)__builtin_amdgcn_readfirstlane((int)t.z), (uint32_t)__builtin_amdgcn_readfirstlane((int)t.w)};
        mark4(c, all - i < 4 ? (int)(all - i) : 4, {0, 0, 0, 0});
      }
    }
    __syncthreads();
    if (kSelf) keep_orthogonal((unsigned int)tid < all ? (rev ? ~C.took[tid] & all_bits : C.took[tid]) : 0u);
    level += (int)complete;
    par ^= 1;
    // Every window decides its candidates and passes levels without any: the
    // limit is never met, and like every wait's it ends the launch.
    if (++windows > kCovMaxRounds) {
      if (tid == 0) {
        __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        L.abort = 1;
      }
      return;
    }
  }
  if (rank == 0 && tid == 0) {
    if (m > capacity) set_status(ctl, GC_ECAPACITY);
    ctl->m = m < capacity ? m : capacity;
    ctl->stat_windows = windows;
  }
}
