// linear.h -- device side of the generator search for the linear greedy codes
// (gfx950).  Included by the kernels that build such codes.
//
// Greedy codes over a positional walk are linear.  Let position p hold the
// word w(p) = XOR of img[j] over the set bits j of p (lex, Gray, a B-ordering;
// the even-weight walks of the self-orthogonal lex and Gray codes), and let
// V_k be the words of the first 2^k positions.  Brualdi and Pless ("Greedy
// codes", J. Combin. Theory Ser. A 64, 1993; Conway and Sloane for lex): the
// code C of V_k is a subspace, and of the coset img[k] + V_k the walk first
// accepts the earliest word x at distance >= d from C, if there is one, and
// then exactly x + C.  (Say v in img[k] + V_k passes against C, v not in
// x + C, and let y = v + x.  y in V_k is no code word, so an earlier code word
// c has wt(y + c) < d.  At the top position bit of y + c, y has a 1.  x is the
// earliest passing word of its coset, so x has a 0 there -- otherwise the
// passing word v + c would come before x -- and v a 1, so x + c, at distance
// < d from v, comes before v and v is rejected.  With the self-orthogonal
// rule: v + c and x + c pass too, as code words overlap evenly.)  So a code is
// known from its generators, one search per position bit instead of one test
// per candidate, and its words are the XORs of generators in binary order.
//
// The search works on cosets.  The quotient V_k / C has 2^r elements; a coset
// is labelled by the r position bits that are no generator's top bit, taken
// from its earliest word, so labels ascend in walk order.  x = img[k] + (word
// of label m) passes exactly when x + C holds no word of weight < d: label m
// is free when no word z of img[k] + V_k with wt(z) < d has label(z + img[k])
// = m.  The smallest free label gives the next generator; if none is free,
// position bit k becomes label bit r.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gc_internal.h"
#include "greedy_code.h"

namespace gcimpl {

// Result of a search, in device memory.
struct LinResult {
  int ok;                          // 0: not found within the given memory (the caller screens instead)
  int dim;                         // generators
  int status;                      // GC_OK or GC_ECAPACITY
  int part;                        // k: not found, but the code of the first 2^k positions
  unsigned long long begin, end;   // words to write: code indices [begin, end)
  uint32_t gen[32];
};

// State of a search.  kWords: 64-bit words of label bitmaps held in LDS.
template <int kWords>
struct LinLds {
  unsigned long long bits[kWords];
  uint32_t img[32];   // word of position 2^j
  uint32_t gen[32];   // generators: words and positions
  uint32_t pos[32];
  uint32_t lab[32];   // label and position bit of each generator
  uint32_t top[32];
  uint32_t np[32];    // position bit of each label bit
  uint32_t q[32];     // self-orthogonal: label bits whose basis words overlap generator i oddly
  uint32_t best[2];   // smallest free label of a level, by level parity
  int k, r, dim;      // next position bit; label bits; generators
  uint32_t u;         // label of the newest unit vector (lex, Gray)
};

// Bit i of the result is bit i XOR b of x.
__device__ __forceinline__ unsigned long long xor_permute(unsigned long long x, unsigned int b) {
  if (b & 1) x = ((x & 0x5555555555555555ull) << 1) | ((x >> 1) & 0x5555555555555555ull);
  if (b & 2) x = ((x & 0x3333333333333333ull) << 2) | ((x >> 2) & 0x3333333333333333ull);
  if (b & 4) x = ((x & 0x0f0f0f0f0f0f0f0full) << 4) | ((x >> 4) & 0x0f0f0f0f0f0f0f0full);
  if (b & 8) x = ((x & 0x00ff00ff00ff00ffull) << 8) | ((x >> 8) & 0x00ff00ff00ff00ffull);
  if (b & 16) x = ((x & 0x0000ffff0000ffffull) << 16) | ((x >> 16) & 0x0000ffff0000ffffull);
  if (b & 32) x = (x << 32) | (x >> 32);
  return x;
}

// Barrier of a search's threads: one wave (its LDS operations are in order;
// only the compiler must not move them) or the whole workgroup.
template <int kThreads>
__device__ __forceinline__ void lin_sync() {
  if (kThreads == 64) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// The overlap parities of generators 0 .. dim-1 with `word`, bit i for
// generator i, in every lane.
template <typename S>
__device__ __forceinline__ uint32_t lin_overlaps(const S &L, int dim, uint32_t word) {
  const unsigned int lane = threadIdx.x & 63;
  const bool odd = (int)lane < dim && (__builtin_popcount(L.gen[lane & 31] & word) & 1);
  return (uint32_t)__builtin_amdgcn_ballot_w64(odd);
}

// Bits of `free` (labels 64 w ..) whose coset also meets the self-orthogonal
// rule: an even overlap of img[k] + (word of the label) with every generator
// (`c`: the overlaps of img[k]).  Only the lowest one is kept.
template <typename S>
__device__ __forceinline__ unsigned long long lin_first_orthogonal(const S &L, int dim, uint32_t c, unsigned int w,
                                                                   unsigned long long free) {
  while (free) {
    const unsigned int b = __builtin_ctzll(free);
    const uint32_t label = 64u * w + b;
    bool ok = true;
    for (int i = 0; i < dim && ok; ++i) ok = ((__builtin_popcount(label & L.q[i]) ^ (c >> i)) & 1) == 0;
    if (ok) return 1ull << b;
    free &= free - 1;
  }
  return 0;
}

// Smallest label with a set bit in f(w) (w < nw, label = 64 w + bit), or ~0;
// the same in every thread.  `slot` holds ~0 before the call (kThreads > 64).
template <int kThreads, typename F>
__device__ __forceinline__ uint32_t lin_min_label(unsigned int nw, uint32_t *slot, F &&f) {
  const unsigned int tid = threadIdx.x, lane = tid & 63;
  uint32_t m = ~0u;
  for (unsigned int w0 = tid - lane; w0 < nw; w0 += kThreads) {
    const unsigned int w = w0 + lane;
    const unsigned long long x = w < nw ? f(w) : 0ull;
    const unsigned long long hit = __builtin_amdgcn_ballot_w64(x != 0);
    if (hit) {
      const unsigned int l = __builtin_ctzll(hit);
      m = 64u * (w0 + l) + (uint32_t)__builtin_amdgcn_readlane((int)__builtin_ctzll(x | (1ull << 63)), (int)l);
      break;
    }
  }
  if (kThreads == 64) return m;
  if (lane == 0 && m != ~0u) atomicMin(slot, m);
  __syncthreads();
  return *slot;
}

// Records a found label (or a new label bit) of position bit k.
template <typename S>
__device__ __forceinline__ void lin_record(S &L, uint32_t m, int k, int r, int dim) {
  if (threadIdx.x != 0) return;
  if (m == ~0u) {
    L.np[r] = (uint32_t)k;
  } else {
    L.lab[dim] = m;
    L.top[dim] = (uint32_t)k;
  }
}

// Generators from their labels, one per lane of the first wave.
template <typename S>
__device__ __forceinline__ void lin_generators(S &L, int dim) {
  if ((int)threadIdx.x < dim) {
    const int i = threadIdx.x;
    uint32_t w = L.img[L.top[i]], p = 1u << L.top[i];
    for (uint32_t m = L.lab[i]; m; m &= m - 1) {
      const uint32_t b = L.np[__builtin_ctz(m)];
      w ^= L.img[b];
      p |= 1u << b;
    }
    L.gen[i] = w;
    L.pos[i] = p;
  }
}

// Levels of a lex or Gray search (plain or self-orthogonal) from L.k on,
// while the bitmaps fit `max_words` label words.  V_k is all of (the even
// words of) the first coordinates, so the low-weight words of a level are a
// unit vector plus words of weight <= d - 2 of the earlier coordinates, and
// their labels need no enumeration: A[s], the labels of the words of weight
// <= s (self-orthogonal: and of the parity of s), follow by
//   A[s] |= A[s - 1] translated by (XOR with) the new unit vector's label,
// word-parallel.  The words at index w of all A[s] lie together (stride
// `st`).  A thread updates both words of a pair w, w XOR (label / 64), so a
// level needs one barrier for the search and one for the update.  With few
// label words one wave does it alone, barrier-free.
template <int kThreads, typename S, typename Bits>
__device__ __forceinline__ void lin_levels(S &L, Bits A, unsigned int max_words, int ord, int so, int K, int D) {
  const unsigned int tid = threadIdx.x;
  const unsigned int st = (unsigned int)(D + 1) | 1u;
  const int top = so && !(D & 1) ? D - 1 : D;
  // The state is the same for every lane: scalar registers and branches.
  int k = __builtin_amdgcn_readfirstlane(L.k), r = __builtin_amdgcn_readfirstlane(L.r),
      dim = __builtin_amdgcn_readfirstlane(L.dim);
  uint32_t u = __builtin_amdgcn_readfirstlane(L.u);
  // Words w and v (= w XOR label / 64; the same word when that is 0) of every
  // A[s], largest s first, four at a time: their reads go out together.
  auto update = [&](unsigned int w, unsigned int v, unsigned int ub) {
    for (int s = D; s >= 1; s -= 4) {
      unsigned long long aw[5], av[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        const int i = s - q >= 0 ? s - q : 0;
        aw[q] = A[w * st + i];
        av[q] = A[v * st + i];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (s - q >= 1) {
          A[w * st + s - q] = aw[q] | xor_permute(av[q + 1], ub);
          if (v != w) A[v * st + s - q] = av[q] | xor_permute(aw[q + 1], ub);
        }
    }
  };
  for (; k < K; ++k) {
    const unsigned int nw = r < 6 ? 1u : 1u << (r - 6);
    if ((r + 1 < 6 ? 1u : 1u << (r - 5)) > max_words) break;
    const uint32_t t = ord == GC_GRAY ? u : 0u;  // label of (unit vector k) + img[k]
    const uint32_t c = so ? lin_overlaps(L, dim, L.img[k]) : 0u;
    const uint32_t m = __builtin_amdgcn_readfirstlane(lin_min_label<kThreads>(nw, &L.best[k & 1], [&](unsigned int w) {
      unsigned long long x = top < 0 ? ~0ull : ~xor_permute(A[(w ^ (t >> 6)) * st + top], t & 63);
      if (r < 6) x &= (1ull << (1 << r)) - 1;
      return so ? lin_first_orthogonal(L, dim, c, w, x) : x;
    }));
    const bool grew = m == ~0u;
    u = t ^ (grew ? 1u << r : m);
    if (kThreads > 64 && tid == 0) L.best[(k + 1) & 1] = ~0u;
    lin_record(L, m, k, r, dim);
    const unsigned int uw = u >> 6, ub = u & 63;
    if (grew && r >= 6) {
      // The new label bit's half starts empty: it receives the translates.
      for (unsigned int w = tid; w < nw; w += kThreads) {
        for (int s = 1; s <= D; ++s) A[(w ^ uw) * st + s] = xor_permute(A[w * st + s - 1], ub);
        A[(w ^ uw) * st] = 0;
      }
    } else if (uw == 0) {
      for (unsigned int w = tid; w < nw; w += kThreads) update(w, w, ub);
    } else {
      const int hb = 31 - __builtin_clz(uw);  // pairs: the words whose bit hb is clear
      for (unsigned int i = tid; i < nw / 2; i += kThreads) {
        const unsigned int w = ((i >> hb) << (hb + 1)) | (i & ((1u << hb) - 1u));
        update(w, w ^ uw, ub);
      }
    }
    lin_sync<kThreads>();
    if (grew) {
      if (so && (int)tid < dim) L.q[tid] |= ((c >> tid) & 1u) << r;
      ++r;
    } else {
      if (so) {  // the new generator now, and its overlaps with the label bits' words
        if (tid == 0) {
          uint32_t w = L.img[k];
          for (uint32_t b = m; b; b &= b - 1) w ^= L.img[L.np[__builtin_ctz(b)]];
          L.gen[dim] = w;
        }
        lin_sync<kThreads>();
        if (tid < 64) {
          const bool odd = (int)tid < r && (__builtin_popcount(L.img[L.np[tid & 31] & 31] & L.gen[dim]) & 1);
          const uint32_t q = (uint32_t)__builtin_amdgcn_ballot_w64(odd);
          if (tid == 0) L.q[dim] = q;
        }
      }
      ++dim;
    }
    if (so) lin_sync<kThreads>();
  }
  lin_sync<kThreads>();
  if (tid == 0) {
    L.k = k;
    L.r = r;
    L.dim = dim;
    L.u = u;
  }
}

// The same by one wave for a plain search of up to 64 labels, from the start:
// lane s holds A[s], a level is some forty instructions without LDS reads
// (n = 20, d = 4 14 us of kernel, 33 with the bitmaps in LDS).  Leaves the
// search to lin_levels where a seventh label bit is due.
template <typename S>
__device__ __forceinline__ void lin_levels_short(S &L, int ord, int K, int D) {
  const unsigned int lane = threadIdx.x;
  unsigned long long a = (int)lane <= D ? 1ull : 0ull;  // the zero word
  int k = 0, r = 0, dim = 0;
  uint32_t u = 0;
  for (; k < K; ++k) {
    const uint32_t t = ord == GC_GRAY ? u : 0u;
    const unsigned long long last = ((unsigned long long)(unsigned int)__builtin_amdgcn_readlane((int)(a >> 32), D) << 32) |
                                    (unsigned int)__builtin_amdgcn_readlane((int)a, D);
    unsigned long long x = ~xor_permute(last, t);
    if (r < 6) x &= (1ull << (1 << r)) - 1;
    if (x == 0 && r == 6) break;
    const uint32_t m = x ? (uint32_t)__builtin_ctzll(x) : ~0u;
    u = t ^ (x ? m : 1u << r);
    lin_record(L, m, k, r, dim);
    const unsigned long long below = __shfl_up(a, 1);
    if (lane > 0 && (int)lane <= D) a |= xor_permute(below, u);
    if (x) ++dim;
    else ++r;
  }
  if ((int)lane <= D) L.bits[lane] = a;
  if (lane == 0) {
    L.k = k;
    L.r = r;
    L.dim = dim;
    L.u = u;
  }
  lin_sync<64>();
}

// Whether a lex or Gray code needs a search.  Three words at distance d or more
// have 3 d differences in n coordinates, of which each takes part in two at most:
// with 3 d > 2 n there are two words, zero and the walk's first of weight d or
// more.  The first 2^k positions hold all words of the first k coordinates, so
// that is the one of d (self-orthogonal: an even number of) ones on the first
// coordinates.  (The search holds 2^(d - 1) labels for it: n = 24, d = 24 lex
// 4046 us a call with the search, 22 without, 2164 by the screens.)
__host__ __device__ constexpr bool lin_searched(int n, int d) { return 3 * d <= 2 * n; }

// Lex and Gray: the whole search by one workgroup, the bitmaps in LDS while
// they fit and then in `gbits` (global memory, gwords words).  Returns
// whether it finished.
template <int kWords>
__device__ __forceinline__ bool lin_search(LinLds<kWords> &L, int n, int d, int ord, int so,
                                           unsigned long long *gbits, unsigned int gwords) {
  const int tid = threadIdx.x, K = n - so, D = d - 2;
  const unsigned int st = (unsigned int)(D + 1) | 1u;
  const bool search = lin_searched(n, d);
  if (tid < 32) {
    const unsigned int w = 1u << tid << so, parity = so ? 1u : 0u;
    L.img[tid] = ord == GC_GRAY ? w ^ (w >> 1) : w | parity;
    L.gen[tid] = L.q[tid] = 0;
    L.np[tid] = search ? 0u : (uint32_t)tid;
  }
  if (search)
    for (int s = tid; s <= D; s += blockDim.x) L.bits[s] = 1;  // the zero word
  if (tid == 0) {
    L.k = L.r = L.dim = 0;
    L.u = 0;
    L.best[0] = L.best[1] = ~0u;
    const int weight = d + (so & d & 1), top = weight - 1 - so;
    if (!search && weight <= n) {  // the second word: `weight` ones at the low coordinates
      L.dim = 1;
      L.top[0] = (uint32_t)top;
      // Its position: ones up to the top bit (lex), or every second one (Gray).
      L.lab[0] = (ord != GC_GRAY ? ~0u : top & 1 ? 0xaaaaaaaau : 0x55555555u) & ((1u << top) - 1u);
    }
  }
  __syncthreads();
  if (search) {
    // One wave up to 256 label words (four a lane), then the workgroup.
    if (tid < 64) {
      if (!so && D >= 0) lin_levels_short(L, ord, K, D);
      lin_levels<64>(L, L.bits, kWords / st < 256 ? kWords / st : 256, ord, so, K, D);
    }
    __syncthreads();
    if (L.k < K && kWords / st > 256) lin_levels<kBlock>(L, L.bits, kWords / st, ord, so, K, D);
    __syncthreads();
    if (L.k < K && gwords / st >= (L.r < 5 ? 1u : 1u << (L.r - 5))) {
      const unsigned int held = (L.r < 6 ? 1u : 1u << (L.r - 6)) * st;
      for (unsigned int i = tid; i < held; i += kBlock) gbits[i] = L.bits[i];
      __syncthreads();
      lin_levels<kBlock>(L, gbits, gwords / st, ord, so, K, D);
    }
    __syncthreads();
  }
  lin_generators(L, L.dim);  // (of the first 2^k positions, if it did not finish)
  __syncthreads();
  return !search || L.k >= K;
}

// Words of the code at positions below `stop`: code index m has position XOR
// of pos[i] over the bits i of m, increasing with m.
template <typename S>
__device__ __forceinline__ unsigned long long lin_count_below(const S &L, unsigned long long stop) {
  if (stop == 0) return 0;
  unsigned long long m = 0, p = 0;  // the last word below `stop`, from its top bit down
  for (int i = L.dim - 1; i >= 0; --i) {
    const unsigned long long q = p ^ L.pos[i];
    if (q < stop) {
      m |= 1ull << i;
      p = q;
    }
  }
  return m + 1;
}

// Byte tables of the code: word m is the XOR of tab[j][byte j of m].
__device__ __forceinline__ void lin_word_tables(uint32_t (*tab)[256], const uint32_t *gen, int dim) {
  for (int i = threadIdx.x; i < 4 * 256; i += blockDim.x) {
    uint32_t x = 0;
    for (int j = 0; j < 8; ++j)
      if (((i >> j) & 1) && 8 * (i >> 8) + j < dim) x ^= gen[8 * (i >> 8) + j];
    tab[i >> 8][i & 255] = x;
  }
}

__device__ __forceinline__ uint32_t lin_word(const uint32_t (*tab)[256], unsigned long long m) {
  return tab[0][m & 255] ^ tab[1][(m >> 8) & 255] ^ tab[2][(m >> 16) & 255] ^ tab[3][(m >> 24) & 255];
}

// Code words [begin, end) to `code` (16-byte aligned), by threads `first`,
// first + stride, ...: four words a step, whole 16-byte stores inside.
__device__ __forceinline__ void lin_emit(const uint32_t (*tab)[256], uint32_t *code, unsigned long long begin,
                                         unsigned long long end, unsigned long long first, unsigned long long stride) {
  for (unsigned long long g = begin / 4 + first; 4 * g < end; g += stride) {
    const unsigned long long m = 4 * g;
    const uint32_t high = tab[1][(m >> 8) & 255] ^ tab[2][(m >> 16) & 255] ^ tab[3][(m >> 24) & 255];
    const uint4 low = *reinterpret_cast<const uint4 *>(&tab[0][m & 255]);
    const uint4 v = make_uint4(low.x ^ high, low.y ^ high, low.z ^ high, low.w ^ high);
    if (m >= begin && m + 4 <= end) {
      *reinterpret_cast<uint4 *>(code + m) = v;
    } else {
      if (m >= begin && m < end) code[m] = v.x;
      if (m + 1 >= begin && m + 1 < end) code[m + 1] = v.y;
      if (m + 2 >= begin && m + 2 < end) code[m + 2] = v.z;
      if (m + 3 >= begin && m + 3 < end) code[m + 3] = v.w;
    }
  }
}

}  // namespace gcimpl
