// linear.hip -- single linear codes (lex, Gray, B-ordering, self-orthogonal
// lex and Gray): one ordinary launch in which every workgroup finds the
// generators for itself and writes its part of the words (a launch more lists
// the low-weight words of a B-ordering with more than 16384; a prefix to check or bitmaps in
// global memory leave the search to one workgroup and a launch of its own).
// The mathematics is in linear.h.
//
// What bounds it: launch latency and the chain of n search levels (one wave
// while the label bitmaps are short).  One call, without and with this path:
// n = 15 d = 3 to host memory 600 and 56 us, n = 20 d = 4 3235 and 27 us,
// n = 26 d = 3 (2^21 words) 526 ms and 31 us, n = 30 d = 10 128 ms and 293 us
// (2^19 labels: the bitmaps leave LDS), a random basis at n = 23 d = 5 2698
// and 64 us.  Search and words as two launches with the result copied back
// cost 15 us more.
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>

#include "binomials.h"
#include "gc_internal.h"
#include "greedy_code.h"
#include "linear.h"

namespace gcimpl {

int acquire_workspace(size_t bytes, char **ptr, int *slot);
void release_workspace(int slot);
int workspace_host(int slot, WsHost *out);

namespace {

// Label words in LDS (128 KiB): a search with more goes on in global memory
// (lex, Gray) or is left to the screens (B-ordering).
constexpr int kLinWords = 16384;
// Global label bitmaps of a search: up to 16 MiB of the workspace pool.
constexpr size_t kLinGlobalBytes = 16u << 20;
// B-ordering: low-weight words listed per workgroup, and at most in all.  A word
// costs a search some 0.5 ns, a position of the walk the screens 0.1 ns past 0.4
// ms (random bases, by the search and by the screens: n = 20, d = 12, 784625 words
// 505 and 413 us, d = 14, 988115 words 608 and 392; n = 21, d = 10, 695859 words
// 513 and 733, d = 11, 2^20 - 1 words 678 and 609, d = 12, 1401291 words 833 and
// 573; n = 22, d = 10, 1097789 words 724 and 922, d = 11, 1744435 words 977 and
// 844).
constexpr unsigned int kSegWords = 4096;
constexpr unsigned long long max_listed(int n) {
  const unsigned long long some = (1ull << 19) + (1ull << n >> 2);
  return some < 1ull << 21 ? some : 1ull << 21;
}
// As many as a workgroup holds in registers: a search of no more keeps its
// words there (n = 23, d = 5, 10902 words: 64 us a call, 77 with a list).
constexpr int kHeld = 16;
constexpr unsigned int kMaxHeld = kHeld * kBlock;
// Given words that the searching workgroup compares with the code itself (it does
// 1024 in 0.3 us; n = 26, d = 2 Gray, 29 million words 8565 us a call, with the
// whole GPU 62).
constexpr unsigned long long kCheckAlone = 1u << 14;
constexpr int kScanBlock = 256;
constexpr int kEmitBlock = 256;

__constant__ BinomTable kBinom = make_binom();
constexpr BinomTable kHostBinom = make_binom();

struct LinArgs {
  int n, d, ord, so;
  int levels;             // position bits that occur
  unsigned long long start, stop, prefix, capacity;
  uint32_t *code;
  LinResult *res;
  unsigned long long *gbits;
  unsigned int gwords;
  unsigned int segs;      // B-ordering: segments of the word list
  unsigned int listed;    // words in it
  uint32_t *list;         // segs x kSegWords: positions of low-weight words, by top position bit
  uint32_t *offs;         // segs x 33: where each top bit's run starts in its segment
  uint32_t basis[32];     // B-ordering: b_1 .. b_n
  uint32_t inv[32];       // position of the unit vector 2^i
};

struct ScanLds {
  uint32_t inv[4][256];
  uint32_t hist[33];
};

// Byte tables of the position of a word.
template <int kThreads>
__device__ __forceinline__ void position_tables(const LinArgs &P, ScanLds &S) {
  for (int i = threadIdx.x; i < 4 * 256; i += kThreads) {
    uint32_t x = 0;
    for (int j = 0; j < 8; ++j)
      if ((i >> j) & 1) x ^= P.inv[8 * (i >> 8) + j];
    S.inv[i >> 8][i & 255] = x;
  }
}

// Positions of the words `rank` .. rank + have - 1 of those with 0 < wt < d, in
// the order weight, value (the next word of a weight by the usual bit trick).
template <int kPer, typename F>
__device__ __forceinline__ void low_words(const LinArgs &P, const ScanLds &S, unsigned int rank, unsigned int have, F &&f) {
  int s = 1;
  unsigned long long z = 0;
  if (have) {
    while (rank >= kBinom.c[P.n][s]) rank -= kBinom.c[P.n][s++];
    int left = s;
    for (int b = P.n - 1; b >= 0 && left > 0; --b) {
      const uint32_t c = kBinom.c[b][left];
      if (rank >= c) {
        z |= 1ull << b;
        rank -= c;
        --left;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (i < (int)have) {
      f(i, S.inv[0][z & 255] ^ S.inv[1][(z >> 8) & 255] ^ S.inv[2][(z >> 16) & 255] ^ S.inv[3][(z >> 24) & 255]);
      const unsigned long long low = z & (~z + 1), up = z + low;
      z = up | (((z ^ up) >> 2) >> __builtin_ctzll(low));
      if (z >> P.n) z = (1ull << ++s) - 1;  // the next weight's first word
    }
  }
}

// Segment `seg` of the list of all words z with 0 < wt(z) < d: their
// positions, sorted by top position bit (kept as a run, the bit itself
// cleared).  A thread takes consecutive words.
__device__ __forceinline__ void list_segment(const LinArgs &P, ScanLds &S, unsigned int seg) {
  const int tid = threadIdx.x;
  constexpr int kPer = kSegWords / kScanBlock;
  position_tables<kScanBlock>(P, S);
  if (tid < 33) S.hist[tid] = 0;
  __syncthreads();
  const unsigned int rank = seg * kSegWords + (unsigned int)tid * kPer;
  uint32_t p[kPer], slot[kPer];
  const unsigned int have = rank < P.listed ? (P.listed - rank < kPer ? P.listed - rank : kPer) : 0;
  low_words<kPer>(P, S, rank, have, [&](int i, uint32_t x) {
    p[i] = x;
    slot[i] = atomicAdd(&S.hist[31 - __builtin_clz(x)], 1u);
  });
  __syncthreads();
  if (tid == 0) {
    uint32_t acc = 0;
    for (int b = 0; b < 33; ++b) {
      const uint32_t c = S.hist[b];
      S.hist[b] = acc;
      P.offs[seg * 33 + b] = acc;
      acc += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (i < (int)have) {
      const int b = 31 - __builtin_clz(p[i]);
      P.list[seg * kSegWords + S.hist[b] + slot[i]] = p[i] ^ (1u << b);
    }
  }
}

__global__ void __launch_bounds__(kScanBlock) lin_list_kernel(LinArgs P) {
  __shared__ ScanLds S;
  list_segment(P, S, blockIdx.x);
}

// B-ordering: V_k is no coordinate subspace, so each low-weight word of F_2^n
// marks its label at the level of its top position bit (byte tables give the
// label of a position).  The words' positions are in registers, or listed by
// that bit in global memory.
__device__ __forceinline__ bool border_search(LinLds<kLinWords> &L, ScanLds &S, uint32_t (*lam)[256], const LinArgs &P) {
  const int tid = threadIdx.x;
  uint32_t held[kHeld];
  const bool in_registers = P.listed <= kMaxHeld;
  const unsigned int per = (P.listed + kBlock - 1) / kBlock;
  if (in_registers) {
    position_tables<kBlock>(P, S);
    __syncthreads();
    const unsigned int rank = (unsigned int)tid * per;
#pragma unroll
    for (int i = 0; i < kHeld; ++i) held[i] = 0;
    low_words<kHeld>(P, S, rank, rank < P.listed ? (P.listed - rank < per ? P.listed - rank : per) : 0u,
                     [&](int i, uint32_t x) { held[i] = x; });
  }
  if (tid < 32) L.img[tid] = P.basis[tid];
  for (int i = tid; i < 4 * 256; i += kBlock) lam[i >> 8][i & 255] = 0;
  if (tid < 2) L.best[tid] = ~0u;
  int r = 0, dim = 0, k = 0;
  uint32_t *bits32 = reinterpret_cast<uint32_t *>(L.bits);
  for (; k < P.levels; ++k) {
    const unsigned int nw = r < 6 ? 1u : 1u << (r - 6);
    if (nw > (unsigned int)kLinWords) break;
    for (unsigned int w = tid; w < nw; w += kBlock) L.bits[w] = 0;
    __syncthreads();
    auto mark = [&](uint32_t p) {
      const uint32_t l = lam[0][p & 255] ^ lam[1][(p >> 8) & 255] ^ lam[2][(p >> 16) & 255] ^ lam[3][p >> 24];
      atomicOr(&bits32[l >> 5], 1u << (l & 31));
    };
    if (in_registers) {
#pragma unroll
      for (int i = 0; i < kHeld; ++i)
        if (i < (int)per && held[i] >> k == 1) mark(held[i] ^ (1u << k));
    } else {
      for (unsigned int seg = tid >> 6; seg < P.segs; seg += kBlock / 64) {
        const uint32_t e = P.offs[seg * 33 + k + 1];
        for (uint32_t i = P.offs[seg * 33 + k] + (tid & 63); i < e; i += 64) mark(P.list[seg * kSegWords + i]);
      }
    }
    __syncthreads();
    const uint32_t m = lin_min_label<kBlock>(nw, &L.best[k & 1], [&](unsigned int w) {
      return r < 6 ? ~L.bits[w] & ((1ull << (1 << r)) - 1) : ~L.bits[w];
    });
    const uint32_t h = m == ~0u ? 1u << r : m;
    if (tid == 0) L.best[(k + 1) & 1] = ~0u;
    lin_record(L, m, k, r, dim);
    if (tid < 256 && ((tid >> (k & 7)) & 1)) lam[k >> 3][tid] = lam[k >> 3][tid ^ (1 << (k & 7))] ^ h;
    if (m == ~0u) ++r;
    else ++dim;
  }
  __syncthreads();
  if (tid == 0) L.dim = dim;
  lin_generators(L, dim);
  __syncthreads();
  return k >= P.levels;
}

// The generators, the range of code words to write, and (a resumed
// construction, one workgroup only) whether the given prefix is the code's
// beginning; with `write` the workgroup also writes its part of the words.
template <bool kBorder>
__global__ void __launch_bounds__(kBlock) lin_find_kernel(LinArgs P, unsigned long long *count, int write) {
  __shared__ LinLds<kLinWords> L;
  __shared__ __align__(16) uint32_t tab[4][256];
  __shared__ unsigned long long begin_s, end_s;
  __shared__ int ok_s;
  const int tid = threadIdx.x;
  bool ok;
  if constexpr (kBorder) {
    __shared__ ScanLds S;
    ok = border_search(L, S, tab, P);
  } else {
    ok = lin_search(L, P.n, P.d, P.ord, P.so, P.gbits, P.gwords);
  }
  if (tid == 0) {
    begin_s = ok ? lin_count_below(L, P.start) : 0;
    ok_s = ok && begin_s == P.prefix;
  }
  __syncthreads();
  if (ok_s && (P.prefix || write)) {
    lin_word_tables(tab, L.gen, L.dim);
    __syncthreads();
  }
  if (ok_s && P.prefix && P.prefix <= kCheckAlone) {
    bool same = true;
    for (unsigned long long i = tid; i < P.prefix; i += kBlock) same &= P.code[i] == lin_word(tab, i);
    if (!__syncthreads_and(same)) ok_s = 0;
    __syncthreads();
  }
  if (tid == 0) {
    const unsigned long long all = ok_s ? lin_count_below(L, P.stop) : 0;
    end_s = all < P.capacity ? all : P.capacity;
    // A search cut short leaves the rest of the walk: the words so far are written.
    const bool part = !kBorder && !write && !ok && P.start == 0 && P.prefix == 0 && 1ull << L.k < P.stop &&
                      1ull << L.dim <= P.capacity;
    if (part) end_s = 1ull << L.dim;
    if (blockIdx.x == 0) {
      P.res->part = part ? L.k : 0;
      P.res->dim = L.dim;
      P.res->status = all > P.capacity ? GC_ECAPACITY : GC_OK;
      P.res->begin = begin_s;
      P.res->end = end_s;
      P.res->ok = ok_s;
      if (write && ok_s && count) *count = end_s;
    }
  }
  if (!write) {
    if (tid < 32) P.res->gen[tid] = tid < L.dim ? L.gen[tid] : 0u;
    return;
  }
  __syncthreads();
  if (ok_s)
    lin_emit(tab, P.code, begin_s, end_s, (unsigned long long)blockIdx.x * kBlock + tid,
             (unsigned long long)gridDim.x * kBlock);
}

// Takes `ok` back where the given words are not the code's beginning.
__global__ void __launch_bounds__(kEmitBlock) lin_check_kernel(LinResult *res, const uint32_t *code,
                                                               unsigned long long prefix) {
  __shared__ __align__(16) uint32_t tab[4][256];
  if (!res->ok) return;
  lin_word_tables(tab, res->gen, res->dim);
  __syncthreads();
  bool same = true;
  const unsigned long long stride = (unsigned long long)gridDim.x * kEmitBlock;
  for (unsigned long long g = (unsigned long long)blockIdx.x * kEmitBlock + threadIdx.x; 4 * g < prefix; g += stride) {
    const unsigned long long m = 4 * g;
    if (m + 4 <= prefix) {
      const uint32_t high = tab[1][(m >> 8) & 255] ^ tab[2][(m >> 16) & 255] ^ tab[3][(m >> 24) & 255];
      const uint4 low = *reinterpret_cast<const uint4 *>(&tab[0][m & 255]);
      const uint4 v = *reinterpret_cast<const uint4 *>(code + m);
      same &= ((v.x ^ low.x ^ high) | (v.y ^ low.y ^ high) | (v.z ^ low.z ^ high) | (v.w ^ low.w ^ high)) == 0;
    } else {
      for (unsigned long long i = m; i < prefix; ++i) same &= code[i] == lin_word(tab, i);
    }
  }
  if (!same) res->ok = 0;
}

__global__ void __launch_bounds__(kEmitBlock) lin_emit_kernel(const LinResult *res, uint32_t *code,
                                                              unsigned long long *count) {
  __shared__ __align__(16) uint32_t tab[4][256];
  if (!res->ok && !res->part) return;
  lin_word_tables(tab, res->gen, res->dim);
  __syncthreads();
  lin_emit(tab, code, res->begin, res->end, (unsigned long long)blockIdx.x * kEmitBlock + threadIdx.x,
           (unsigned long long)gridDim.x * kEmitBlock);
  if (blockIdx.x == 0 && threadIdx.x == 0 && count) *count = res->end;
}

// Positions of the unit vectors: the inverse of the basis by elimination.
void invert_basis(const uint32_t *basis, int n, uint32_t *inv) {
  uint32_t v[32], tag[32];
  for (int j = 0; j < n; ++j) {
    v[j] = basis[j];
    tag[j] = 1u << j;
  }
  for (int b = 0; b < n; ++b) {
    int at = b;
    while (!((v[at] >> b) & 1)) ++at;  // the basis is independent (checked by the caller)
    std::swap(v[at], v[b]);
    std::swap(tag[at], tag[b]);
    for (int j = 0; j < n; ++j)
      if (j != b && ((v[j] >> b) & 1)) {
        v[j] ^= v[b];
        tag[j] ^= tag[b];
      }
  }
  for (int b = 0; b < n; ++b) inv[b] = tag[b];
}

size_t up256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

// The most label words of all arrays that a lex or Gray search can hold (none
// without a search): once 2^r exceeds the number of words of weight <= d - 2,
// some label is always free.
unsigned long long lin_words_most(int n, int d) {
  if (!lin_searched(n, d)) return 0;
  unsigned long long low = 1;
  for (int s = 1; s <= d - 2; ++s) low += kHostBinom.c[n - 1][s];
  unsigned long long words = 2;
  while (words * 32 < low) words *= 2;
  return words * ((unsigned int)(d > 1 ? d - 1 : 0) | 1u);
}

// The least that one holds at its last level.  The code has at most 2^m words,
// so at least K - 1 - m of the positions before the last are label bits.  (e even:
// A(2 e, e) <= 4 e, Plotkin, and A(n, e) <= 2 A(n - 1, e); for 2 e > n A(n, e) <=
// 2 floor(e / (2 e - n)); A(n, d) = A(n + 1, d + 1) for odd d.)
unsigned long long lin_words_least(int n, int d, int so) {
  if (!lin_searched(n, d)) return 0;
  const int e = d + (d & 1), N = n + (d & 1);
  unsigned long long most = greedy_code_capacity(n, d);
  most = std::min<unsigned long long>(most, 2 * e > N ? 2ull * (e / (2 * e - N)) : 4ull * e << (N - 2 * e));
  int m = 0;
  while (most >> (m + 1)) ++m;
  const int r = n - so - 1 - m;
  return (r < 5 ? 1ull : 1ull << (r - 5)) * ((unsigned int)(d > 1 ? d - 1 : 0) | 1u);
}

double linear_given_us(const Job &J) {
  // A search past the first labels: some ns a word of its bitmaps, whose number lies
  // between the bounds; self-orthogonal ones test their labels one by one.
  const double words = J.ord == GC_BORDER ? 0.0
                                          : std::sqrt((double)lin_words_least(J.n, J.d, J.so) * (double)lin_words_most(J.n, J.d));
  double us = 50.0 + 1e-3 * words + (J.so ? 0.4 * J.n * J.n : 0.0) + 1e-6 * (double)J.m_start;
  if (J.ord == GC_BORDER) {
    double listed = 0;
    for (int s = 1; s < J.d && s <= J.n; ++s) listed += kHostBinom.c[J.n][s];
    us += 100.0 + 0.5e-3 * listed;
  }
  return us;
}

bool linear_job(const Job &J) {
  return (J.ord == GC_LEX || J.ord == GC_GRAY || J.ord == GC_BORDER) && J.wclass == 0 && (J.d >= 2 || J.so) &&
         J.near_depth == 0 && J.target == 0 && J.mode == 0 && J.deep_tile == 0 && J.valu_screen == 0;
}

int run_linear(Job *J, hipStream_t stream, char *fixed, size_t fixed_bytes, float *kernel_ms, bool *built) {
  *built = false;
  const int K = J->n - J->so;
  LinArgs P;
  memset(&P, 0, sizeof(P));
  P.n = J->n;
  P.d = J->d;
  P.ord = J->ord;
  P.so = J->so;
  P.start = J->p_start;
  P.stop = J->p_stop ? J->p_stop : 1ull << K;
  // Positions below 2^k are decided by k levels; lex and Gray: they are the walk of
  // the first coordinates.
  P.levels = 0;
  while (P.levels < K && 1ull << P.levels < P.stop) ++P.levels;
  if (J->ord != GC_BORDER) P.n = std::max(1, P.levels + J->so);
  P.prefix = J->m_start;
  P.capacity = J->capacity;
  P.code = J->code;
  size_t bytes = up256(sizeof(LinResult));
  size_t off_offs = 0, off_list = 0, off_bits = bytes;
  const int dmax = std::min(J->d - 1, J->n);
  if (J->ord == GC_BORDER) {
    unsigned long long listed = 0;
    for (int s = 1; s <= dmax; ++s) listed += kHostBinom.c[J->n][s];
    if (listed > max_listed(P.n)) return GC_OK;  // the screens build it
    P.listed = (unsigned int)listed;
    P.segs = (P.listed + kSegWords - 1) / kSegWords;
    off_offs = bytes;
    off_list = off_offs + up256(sizeof(uint32_t) * 33 * P.segs);
    bytes = off_list + sizeof(uint32_t) * kSegWords * P.segs;
    memcpy(P.basis, J->basis, sizeof(P.basis));
    invert_basis(J->basis, J->n, P.inv);
  } else {
    const unsigned long long need = lin_words_most(P.n, P.d);
    if (need > (unsigned long long)kLinWords) {
      // A search that cannot end within the given memory is not begun (n = 26,
      // d = 16 lex 6.8 ms by the screens, 9.9 with a search that fails before); one
      // that turns out not to leaves the walk's last positions to the screens (n =
      // 27, d = 14 lex 9.5 ms, all of it by the screens 13.4).
      const unsigned long long room = fixed ? fixed_bytes - bytes : kLinGlobalBytes;
      if (lin_words_least(P.n, P.d, P.so) * 8 > room) return GC_OK;
      bytes += (size_t)std::min<unsigned long long>(need * 8, room);
    }
  }
  char *ws = fixed;
  int slot = -1;
  WsHost host;
  memset(&host, 0, sizeof(host));
  if (!fixed) {
    int rc = acquire_workspace(bytes, &ws, &slot);
    if (rc) return rc;
    rc = workspace_host(slot, &host);
    if (rc) {
      release_workspace(slot);
      return rc;
    }
  }
  // The result goes to pinned host memory, or (fixed workspace) is copied back.
  LinResult *const seen = reinterpret_cast<LinResult *>(host.ptr);
  P.offs = reinterpret_cast<uint32_t *>(ws + off_offs);
  P.list = reinterpret_cast<uint32_t *>(ws + off_list);
  P.gbits = reinterpret_cast<unsigned long long *>(ws + off_bits);
  P.gwords = (unsigned int)((bytes - off_bits) / 8);
  const bool one_launch = P.prefix == 0 && (J->ord == GC_BORDER || P.gwords == 0);
  P.res = one_launch && seen ? reinterpret_cast<LinResult *>(host.dev) : reinterpret_cast<LinResult *>(ws);
  // Words of the code, at most: four a thread and step.  In one launch up to a
  // workgroup per compute unit (LDS holds one), else up to four.
  const unsigned long long most = std::min<unsigned long long>(J->capacity, 1ull << K);
  const unsigned int grid = one_launch ? (unsigned int)std::min<unsigned long long>(256, most / (4 * kBlock) + 1)
                                       : (unsigned int)std::min<unsigned long long>(1024, most / (4 * kEmitBlock) + 1);
  if (seen) seen->ok = 0;
  hipError_t e = kernel_ms ? hipEventRecord(host.begin, stream) : hipSuccess;
  if (e == hipSuccess && P.listed > kMaxHeld) {
    hipLaunchKernelGGL(lin_list_kernel, dim3(P.segs), dim3(kScanBlock), 0, stream, P);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    const dim3 wgs(one_launch ? grid : 1);
    if (J->ord == GC_BORDER) hipLaunchKernelGGL(lin_find_kernel<true>, wgs, dim3(kBlock), 0, stream, P, J->count, one_launch);
    else hipLaunchKernelGGL(lin_find_kernel<false>, wgs, dim3(kBlock), 0, stream, P, J->count, one_launch);
    e = hipGetLastError();
  }
  if (e == hipSuccess && P.prefix > kCheckAlone) {
    const unsigned int groups = (unsigned int)std::min<unsigned long long>(1024, P.prefix / (4 * kEmitBlock) + 1);
    hipLaunchKernelGGL(lin_check_kernel, dim3(groups), dim3(kEmitBlock), 0, stream, P.res, J->code, P.prefix);
    e = hipGetLastError();
  }
  if (e == hipSuccess && !one_launch) {
    hipLaunchKernelGGL(lin_emit_kernel, dim3(grid), dim3(kEmitBlock), 0, stream, P.res, J->code, J->count);
    e = hipGetLastError();
  }
  if (e == hipSuccess && kernel_ms) e = hipEventRecord(host.end, stream);
  LinResult res;
  memset(&res, 0, sizeof(res));
  if (e == hipSuccess && !(one_launch && seen))
    e = hipMemcpyAsync(seen ? seen : &res, P.res, sizeof(res), hipMemcpyDeviceToHost, stream);
  const hipError_t es = hipStreamSynchronize(stream);
  if (e == hipSuccess) e = es;
  if (e == hipSuccess && kernel_ms) e = hipEventElapsedTime(kernel_ms, host.begin, host.end);
  if (e == hipSuccess && seen) res = *seen;
  if (slot >= 0 && es == hipSuccess) release_workspace(slot);
  if (e != hipSuccess) return fail(GC_EDEVICE, "linear code kernels failed: %s", hipGetErrorString(e));
  if (!res.ok) {
    if (res.part) {  // the screens go on from there
      J->p_start = 1ull << res.part;
      J->m_start = res.end;
    }
    return GC_OK;
  }
  J->out_count = res.end;
  J->status = res.status;
  J->done = 1;
  *built = true;
  return GC_OK;
}

}  // namespace gcimpl
