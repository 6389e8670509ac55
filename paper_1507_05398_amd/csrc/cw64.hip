// Constant-weight greedy codes over words of up to 64 coordinates (MI355X,
// gfx950).
//
// Section "Brief overview of the Greedy Algorithm and Codes": a
// constant-weight code takes only the vectors of weight w as candidates; the
// rule is the greedy one of section "Greedy Algorithms and Different
// Orderings" (a candidate joins the code when its Hamming distance, section
// "Hamming Distance", to every word already in the code is at least d).
// Section "Some Examples" reports such codes up to length 35, past 32-bit
// words.  Candidates are the weight-w vectors in increasing value.
//
// Two words of weight w at distance below d are those that share t =
// w - ceil(d / 2) + 1 ones, that is, a t-subset of their supports.  Where the
// t-subsets of the coordinates fit a bitmap in one workgroup's LDS and a word
// has few of them (pack_rule), cw_pack_kernel keeps that bitmap instead of
// comparing candidates with the code: see there.
//
// Otherwise one cooperative launch walks the candidates in blocks of kCands
// positions:
//   1. every workgroup unranks the block's candidates (combinatorial number
//      system) and screens them against its own slice of the committed code;
//      a clash sets the candidate's bit in a dead mask (device atomics);
//   2. grid barrier;
//   3. workgroup 0 takes the block's live candidates in order, accepts each
//      one that no word accepted earlier in the block is closer than d to
//      (the sequential rule inside the block), and appends them to the code;
//   4. grid barrier.
// The code is the sequential greedy one: a candidate is accepted exactly when
// no earlier accepted word (of an earlier block: step 1; of its own block:
// step 3) is closer than d.  This path favours simplicity over speed; the
// 32-bit windowed screen is the fast path.
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "gc_internal.h"
#include "greedy_code.h"

namespace gcimpl {

int acquire_workspace(size_t bytes, char **ptr, int *slot);
void release_workspace(int slot);
int workspace_host(int slot, WsHost *out);

namespace {

// ---- packing by t-subsets, one workgroup --------------------------------

constexpr int kPackBlock = 1024;
constexpr int kPackEach = 4;             // consecutive positions a thread filters per batch
constexpr int kPackMaxW = 8;             // weight, at most (binomials then fit 32 bits)
constexpr int kPackMaxOut = 3;           // ones left out of a t-subset, at most
constexpr unsigned int kPackSubsets = 1u << 19;  // t-subsets, at most (a 64 KiB bitmap)
constexpr unsigned int kPackOwners = 8192;
constexpr unsigned int kPackPending = kPackBlock * (kPackEach + 1);

struct PackBinomials {
  uint32_t c[kPackMaxW + 1][64];         // c[b][a] = C(a, b)
  constexpr PackBinomials() : c() {
    for (int a = 0; a < 64; ++a) c[0][a] = 1;
    for (int b = 1; b <= kPackMaxW; ++b)
      for (int a = 1; a < 64; ++a) c[b][a] = c[b][a - 1] + c[b - 1][a - 1];
  }
};
__constant__ const PackBinomials kPackBinomials{};

struct PackLds {
  uint32_t marked[kPackSubsets / 32];    // t-subsets of the code's words
  uint32_t owner[kPackOwners];           // latest claim of a t-subset (hashed): round, earliest candidate
  uint64_t pending[kPackPending];        // ring: candidates that passed the filter, in order
  uint32_t bin[kPackMaxW + 1][64];
  uint32_t wave[kPackBlock / 64];
};

struct PackParams {
  int n;
  unsigned int subsets;                  // C(n, t)
  unsigned long long total;              // C(n, w) candidate positions
  uint64_t *words;
  unsigned long long capacity;
  uint64_t *count;                       // may be null
  int *status;                           // pinned
};

constexpr int choose_small(int a, int b) { return b == 0 ? 1 : choose_small(a - 1, b - 1) * a / b; }

// Ranks (combinatorial number system) of the t-subsets of x's support, t = W -
// Out.  With k ones left out below it, one i counts as C(its place, i + 1 - k);
// a rank is a sum of such terms, each read from LDS once.
template <int W, int Out>
__device__ __forceinline__ void subset_ranks(const PackLds &L, uint64_t x, uint32_t (&r)[choose_small(W, Out)]) {
  uint32_t term[Out + 1][W];
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const int c = __builtin_ctzll(x);
    x &= x - 1;
#pragma unroll
    for (int k = 0; k <= Out; ++k) term[k][i] = i + 1 - k > 0 ? L.bin[i + 1 - k > 0 ? i + 1 - k : 0][c] : 0u;
  }
  int q = 0;
  if constexpr (Out == 1) {
#pragma unroll
    for (int a = 0; a < W; ++a) {
      uint32_t v = 0;
#pragma unroll
      for (int i = 0; i < W; ++i)
        if (i != a) v += term[i > a][i];
      r[q++] = v;
    }
  } else if constexpr (Out == 2) {
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
      for (int b = a + 1; b < W; ++b) {
        uint32_t v = 0;
#pragma unroll
        for (int i = 0; i < W; ++i)
          if (i != a && i != b) v += term[(i > a) + (i > b)][i];
        r[q++] = v;
      }
  } else {
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
      for (int b = a + 1; b < W; ++b)
#pragma unroll
        for (int c = b + 1; c < W; ++c) {
          uint32_t v = 0;
#pragma unroll
          for (int i = 0; i < W; ++i)
            if (i != a && i != b && i != c) v += term[(i > a) + (i > b) + (i > c)][i];
          r[q++] = v;
        }
  }
}

template <int N>
__device__ __forceinline__ bool any_marked(const PackLds &L, const uint32_t (&r)[N]) {
  uint32_t hit = 0;
#pragma unroll
  for (int q = 0; q < N; ++q) hit |= L.marked[r[q] >> 5] >> (r[q] & 31);
  return hit & 1u;
}

// Exclusive prefix of `mine` over the workgroup and the total; `mine` is below
// 8 and the waves' sums go through L.wave (a barrier before the next use).
__device__ __forceinline__ unsigned int pack_scan(PackLds &L, unsigned int mine, unsigned int *total) {
  const unsigned int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long below = (1ull << lane) - 1ull;
  unsigned int before = 0, all = 0;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const unsigned long long m = __ballot((mine >> b) & 1u);
    before += (unsigned int)__popcll(m & below) << b;
    all += (unsigned int)__popcll(m) << b;
  }
  if (lane == 0) L.wave[wave] = all;
  __syncthreads();
  unsigned int sum = 0;
#pragma unroll
  for (unsigned int v = 0; v < kPackBlock / 64; ++v) {
    if (v < wave) before += L.wave[v];
    sum += L.wave[v];
  }
  *total = sum;
  return before;
}

// Batches of 4096 positions: a thread decodes the first of its four, steps
// through them and drops each with a marked t-subset; the others join the
// pending ring in order.  From 1024 pending on (or at the walk's end), each
// thread takes one of the next 1024 and they are decided in rounds: an
// undecided candidate claims its t-subsets, one that holds all of its claims
// against earlier ones is accepted (nothing earlier and undecided shares a
// t-subset with it) and marks them, and those with a marked t-subset are dead.
// The earliest undecided one wins its claims in any case, hash collisions
// included, so every round decides.  Accepted words are appended in order.
//
// Bound by LDS reads of the filter (n = 30 w = 5 d = 6: 25 a position, 2 ns)
// and by barriers (n = 40 w = 4 d = 4: 200 rounds of 3).  A call, by the screens
// and here: n = 20 w = 3 d = 4 654 and 35 us, n = 40 w = 4 d = 4 18.0 ms and
// 293 us, n = 30 w = 5 d = 4 27.8 ms and 527 us, d = 6 20.5 ms and 307 us.
template <int W, int Out>
__global__ void __launch_bounds__(kPackBlock) cw_pack_kernel(PackParams P) {
  constexpr int N = choose_small(W, Out);
  __shared__ PackLds L;
  const unsigned int tid = threadIdx.x;
  for (unsigned int i = tid; i < (P.subsets + 31) / 32; i += kPackBlock) L.marked[i] = 0;
  for (unsigned int i = tid; i < kPackOwners; i += kPackBlock) L.owner[i] = 0;
  for (unsigned int i = tid; i < (kPackMaxW + 1) * 64; i += kPackBlock)
    L.bin[i / 64][i % 64] = kPackBinomials.c[i / 64][i % 64];
  __syncthreads();
  unsigned long long m = 0, p0 = 0;
  unsigned int head = 0, pend = 0;   // pending ring: first entry, entries
  unsigned int round = 0;            // below 2^22: each accepts a word, and words have distinct t-subsets
  int status = GC_OK;
  while (p0 < P.total || pend) {
    if (p0 < P.total && pend < kPackBlock) {
      const unsigned long long first = p0 + (unsigned long long)tid * kPackEach;
      uint64_t x[kPackEach];
      unsigned int live = 0;
      if (first < P.total) {
        uint64_t v = 0;
        uint32_t rest = (uint32_t)first;
        int hi = P.n;                // places below hi are left
#pragma unroll
        for (int i = W; i >= 1; --i) {
          int lo = i - 1;            // C(lo, i) = 0 <= rest < C(hi, i): the largest such lo
          while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (L.bin[i][mid] <= rest) lo = mid; else hi = mid;
          }
          rest -= L.bin[i][lo];
          v |= 1ull << lo;
          hi = lo;
        }
#pragma unroll
        for (int k = 0; k < kPackEach; ++k) {
          x[k] = v;
          if (first + k < P.total) {
            uint32_t r[N];
            subset_ranks<W, Out>(L, v, r);
            if (!any_marked(L, r)) live |= 1u << k;
            const uint64_t up = v + (v & -v);   // the next word of this weight
            v = up | (((v ^ up) >> 2) >> __builtin_ctzll(v));
          }
        }
      }
      unsigned int all;
      unsigned int at = head + pend + pack_scan(L, (unsigned int)__popc(live), &all);
#pragma unroll
      for (int k = 0; k < kPackEach; ++k)
        if ((live >> k) & 1u) {
          L.pending[at >= kPackPending ? at - kPackPending : at] = x[k];
          ++at;
        }
      pend += all;
      p0 += (unsigned long long)kPackBlock * kPackEach;
      __syncthreads();
      continue;
    }
    const unsigned int nc = pend < (unsigned int)kPackBlock ? pend : (unsigned int)kPackBlock;
    const unsigned int at = head + tid;
    uint64_t x = 0;
    uint32_t r[N];
    bool live = false, taken = false;
    if (tid < nc) {
      x = L.pending[at >= kPackPending ? at - kPackPending : at];
      subset_ranks<W, Out>(L, x, r);
      live = !any_marked(L, r);
    }
    while (__syncthreads_or(live)) {
      const uint32_t key = (++round << 10) | (kPackBlock - 1 - tid);
      if (live) {
#pragma unroll
        for (int q = 0; q < N; ++q) atomicMax(&L.owner[r[q] & (kPackOwners - 1)], key);
      }
      __syncthreads();
      if (live) {
        bool mine = true;
#pragma unroll
        for (int q = 0; q < N; ++q) mine &= L.owner[r[q] & (kPackOwners - 1)] == key;
        if (mine) {
          taken = true;
          live = false;
#pragma unroll
          for (int q = 0; q < N; ++q) atomicOr(&L.marked[r[q] >> 5], 1u << (r[q] & 31));
        }
      }
      __syncthreads();
      if (live) live = !any_marked(L, r);
    }
    unsigned int na;
    const unsigned long long to = m + pack_scan(L, taken, &na);
    if (taken && to < P.capacity) P.words[to] = x;
    m += na;
    head += nc;
    if (head >= kPackPending) head -= kPackPending;
    pend -= nc;
    __syncthreads();
    if (m > P.capacity) {
      m = P.capacity;
      status = GC_ECAPACITY;
      break;
    }
  }
  if (tid == 0) {
    if (P.count) *P.count = m;
    *P.status = status;
  }
}

using PackKernel = void (*)(PackParams);
// (With three left out of 7 or 8 the 35 and 56 ranks spill; n = 24 w = 8 d = 8
// still 5.8 ms, 141 ms by the screens.)
template <int Out>
PackKernel pack_kernel_of(int w) {
  switch (w) {
    case 2: if constexpr (Out < 2) return cw_pack_kernel<2, Out>; else return nullptr;
    case 3: if constexpr (Out < 3) return cw_pack_kernel<3, Out>; else return nullptr;
    case 4: return cw_pack_kernel<4, Out>;
    case 5: return cw_pack_kernel<5, Out>;
    case 6: return cw_pack_kernel<6, Out>;
    case 7: return cw_pack_kernel<7, Out>;
    case 8: return cw_pack_kernel<8, Out>;
    default: return nullptr;
  }
}

// ---- screens over the whole GPU -----------------------------------------

constexpr int kCwBlock = 256;                     // threads per workgroup
constexpr int kCands = 1024;                      // candidate positions per block
constexpr int kPerThread = kCands / kCwBlock;     // candidates a thread screens
constexpr unsigned long long kMaxPositions = 1ull << 32;

struct CwState {                 // device workspace (zeroed before the launch)
  unsigned long long m;          // committed words
  int status;                    // GC_OK or GC_ECAPACITY
  int pad;
  uint32_t dead[kCands / 32];    // the block's dead mask
};

struct CwParams {
  int n, w, d;
  unsigned long long total;      // C(n, w) candidate positions
  uint64_t *words;
  unsigned long long capacity;
  uint64_t *count;               // may be null
  CwState *st;
};

__device__ __forceinline__ unsigned long long ld_dev(unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The r-th weight-w vector of length n in increasing value: r is written as
// C(c_w, w) + ... + C(c_1, 1) with c_w > ... > c_1 >= 0 (combinatorial
// number system), and the vector has ones at c_1 .. c_w.
__device__ __forceinline__ uint64_t unrank(const unsigned long long (*C)[65], int n, int w, unsigned long long r) {
  uint64_t x = 0;
  int c = n;
  for (int i = w; i >= 1; --i) {
    int cc = c - 1;
    while (C[cc][i] > r) --cc;  // C(i - 1, i) = 0 <= r ends the search
    x |= 1ull << cc;
    r -= C[cc][i];
    c = cc;
  }
  return x;
}

__global__ void __launch_bounds__(kCwBlock) cw64_kernel(CwParams P) {
  __shared__ unsigned long long C[65][65];  // binomials C(a, b), a, b <= 64 (Pascal's rule)
  __shared__ uint64_t cand[kCands];         // workgroup 0: the block's candidates
  __shared__ uint64_t acc[kCands];          // workgroup 0: words accepted in this block
  __shared__ uint32_t deadw[kCands / 32];
  __shared__ unsigned long long m_s;
  __shared__ int stop_s;
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  const int tid = threadIdx.x;
  for (int a = 0; a <= 64; ++a) {
    if (tid <= 64) C[a][tid] = tid == 0 ? 1ull : (a == 0 ? 0ull : C[a - 1][tid - 1] + C[a - 1][tid]);
    __syncthreads();
  }
  const unsigned int d = (unsigned int)P.d;
  for (unsigned long long p0 = 0; p0 < P.total; p0 += kCands) {
    const unsigned int nb = (unsigned int)(P.total - p0 < (unsigned long long)kCands ? P.total - p0 : kCands);
    if (tid == 0) {
      m_s = ld_dev(&P.st->m);
      stop_s = __hip_atomic_load(&P.st->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (stop_s != 0) break;  // every workgroup reads the same state after the barrier
    const unsigned long long m = m_s;

    // 1. Screen against this workgroup's slice of code[0, m).
    uint64_t x[kPerThread];
    bool live[kPerThread];
    int nlive = 0;
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) {
      const unsigned int idx = (unsigned int)(k * kCwBlock + tid);
      live[k] = idx < nb;
      x[k] = live[k] ? unrank(C, P.n, P.w, p0 + idx) : 0ull;
      nlive += live[k];
    }
    const unsigned long long lo = m * blockIdx.x / gridDim.x, hi = m * (blockIdx.x + 1) / gridDim.x;
    for (unsigned long long j = lo; j < hi && nlive > 0; ++j) {
      const uint64_t c = P.words[j];
#pragma unroll
      for (int k = 0; k < kPerThread; ++k) {
        if (live[k] && (unsigned int)__builtin_popcountll(x[k] ^ c) < d) {
          live[k] = false;
          --nlive;
          const unsigned int idx = (unsigned int)(k * kCwBlock + tid);
          __hip_atomic_fetch_or(&P.st->dead[idx >> 5], 1u << (idx & 31), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    grid.sync();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");

    // 3. Workgroup 0: the block in order.
    if (blockIdx.x == 0) {
      for (unsigned int i = tid; i < nb; i += kCwBlock) cand[i] = unrank(C, P.n, P.w, p0 + i);
      for (int i = tid; i < kCands / 32; i += kCwBlock)
        deadw[i] = __hip_atomic_load(&P.st->dead[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      unsigned int na = 0;  // the same in every thread
      for (unsigned int i = 0; i < nb; ++i) {
        if ((deadw[i >> 5] >> (i & 31)) & 1u) continue;
        const uint64_t y = cand[i];
        bool clash = false;
        for (unsigned int a = tid; a < na; a += kCwBlock)
          clash |= (unsigned int)__builtin_popcountll(y ^ acc[a]) < d;
        if (!__syncthreads_or(clash)) {
          if (tid == 0) acc[na] = y;
          ++na;
          __syncthreads();
        }
      }
      const unsigned long long room = P.capacity > m ? P.capacity - m : 0;
      const unsigned int nput = (unsigned long long)na < room ? na : (unsigned int)room;
      for (unsigned int a = tid; a < nput; a += kCwBlock) P.words[m + a] = acc[a];
      for (int i = tid; i < kCands / 32; i += kCwBlock) P.st->dead[i] = 0;
      if (tid == 0) {
        P.st->m = m + nput;
        if (nput < na) P.st->status = GC_ECAPACITY;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    grid.sync();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  if (blockIdx.x == 0 && tid == 0 && P.count) *P.count = ld_dev(&P.st->m);
}

// C(a, b), or kMaxPositions + 1 once it exceeds kMaxPositions.  After step i
// the product is C(a - b + i, i), exact, increasing with i and at most
// 2^32 before the multiplication (so the product stays below 2^39).
unsigned long long positions(int a, int b) {
  if (b < 0 || b > a) return 0;
  if (b > a - b) b = a - b;
  unsigned long long r = 1;
  for (int i = 1; i <= b; ++i) {
    r = r * (unsigned long long)(a - b + i) / (unsigned long long)i;
    if (r > kMaxPositions) return kMaxPositions + 1;
  }
  return r;
}

// The packing kernel of (n, w, d), or null where the t-subsets outgrow LDS, a
// word has too many of them, or every two words clash or none do (t outside 1
// .. w - 1): the screens.  Inside these limits it is the faster one: a position
// costs 1 to 8 ns of one compute unit against some 145 of grid barriers.  At their
// edges, by the screens and here, ms: n = 38 w = 8 d = 8 7342 and 209, n = 48 w = 7
// d = 8 10845 and 219, n = 29 w = 8 d = 6 615 and 14.8, n = 25 w = 8 d = 4 217 and
// 4.9, n = 38 w = 7 d = 6 1869 and 30, n = 64 w = 5 d = 8 1112 and 10.3, n = 61 w =
// 5 d = 4 1404 and 14.6.
PackKernel pack_rule(int n, int w, int d, unsigned int *subsets) {
  d = d < 65 ? d : 65;  // no two words are further apart than 64 (and d + 1 stays an int)
  const int out = (d + 1) / 2 - 1, t = w - out;
  if (w > kPackMaxW || out < 1 || out > kPackMaxOut || t < 1) return nullptr;
  const unsigned long long all = positions(n, t);
  if (all > kPackSubsets) return nullptr;
  *subsets = (unsigned int)all;
  return out == 1 ? pack_kernel_of<1>(w) : out == 2 ? pack_kernel_of<2>(w) : pack_kernel_of<3>(w);
}

// Runs the packing kernel and waits for it.
int run_pack(PackKernel kernel, PackParams P, hipStream_t stream, int *status) {
  char *ws = nullptr;
  int slot = -1;
  if (int rc = acquire_workspace(256, &ws, &slot)) return rc;
  WsHost host;
  if (int rc = workspace_host(slot, &host)) {
    release_workspace(slot);
    return rc;
  }
  P.status = reinterpret_cast<int *>(host.dev);
  int *seen = reinterpret_cast<int *>(host.ptr);
  *seen = GC_ETIMEOUT;
  hipLaunchKernelGGL(kernel, dim3(1), dim3(kPackBlock), 0, stream, P);
  hipError_t e = hipGetLastError();
  const hipError_t es = hipStreamSynchronize(stream);
  if (e == hipSuccess) e = es;
  *status = *seen;
  if (es == hipSuccess) release_workspace(slot);
  if (e != hipSuccess) return fail(GC_EDEVICE, "constant-weight launch failed: %s", hipGetErrorString(e));
  return GC_OK;
}

}  // namespace
}  // namespace gcimpl

using namespace gcimpl;

extern "C" int greedy_code_cw64(int n, int w, int d, uint64_t *d_words, uint64_t capacity, uint64_t *d_count,
                                void *hip_stream) {
  if (n < 1 || n > 64) return fail(GC_EINVAL, "n = %d is outside 1..64", n);
  if (w < 0 || w > n) return fail(GC_EINVAL, "weight %d is outside 0..%d", w, n);
  if (d < 1) return fail(GC_EINVAL, "d = %d is below 1", d);
  if (!d_words && capacity) return fail(GC_EINVAL, "d_words is NULL with capacity %llu",
                                        (unsigned long long)capacity);
  if (reinterpret_cast<uintptr_t>(d_words) % 8) return fail(GC_EINVAL, "d_words is not 8-byte aligned");
  // The walk's length: at most 2^32 positions, as for the 32-bit walks.
  const unsigned long long total = positions(n, w);
  if (total > kMaxPositions) return fail(GC_EINVAL, "C(%d, %d) positions exceed 2^32", n, w);
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  int dev = 0, cus = 0, coop = 0, bpc = 0;
  if (hipGetDevice(&dev) != hipSuccess) return fail(GC_EDEVICE, "hipGetDevice failed");
  if (int rc = device_info(dev, &cus, &coop, &bpc)) return rc;
  if (!coop) return fail(GC_EDEVICE, "device %d has no cooperative launch", dev);
  unsigned int subsets = 0;
  if (const PackKernel kernel = pack_rule(n, w, d, &subsets)) {
    int status = GC_OK;
    if (int rc = run_pack(kernel, PackParams{n, subsets, total, d_words, capacity, d_count, nullptr}, stream, &status))
      return rc;
    if (status) return fail(status, "the code exceeds capacity %llu", (unsigned long long)capacity);
    return GC_OK;
  }
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, cw64_kernel, kCwBlock, 0) != hipSuccess || per_cu < 1)
    return fail(GC_EDEVICE, "the constant-weight kernel does not fit a compute unit");
  const unsigned int grid = (unsigned int)cus;  // one workgroup per CU: co-resident by the check above
  char *ws = nullptr;
  int slot = -1;
  if (int rc = acquire_workspace(sizeof(CwState), &ws, &slot)) return rc;
  CwState *st = reinterpret_cast<CwState *>(ws);
  CwParams P{n, w, d, total, d_words, capacity, d_count, st};
  void *args[] = {&P};
  hipError_t e = hipMemsetAsync(st, 0, sizeof(CwState), stream);
  if (e == hipSuccess)
    e = hipLaunchCooperativeKernel((const void *)cw64_kernel, dim3(grid), dim3(kCwBlock), args, 0, stream);
  int status = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&status, &st->status, sizeof(int), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  release_workspace(slot);
  if (e != hipSuccess) return fail(GC_EDEVICE, "constant-weight launch failed: %s", hipGetErrorString(e));
  if (status == GC_ECAPACITY) return fail(GC_ECAPACITY, "the code exceeds capacity %llu",
                                          (unsigned long long)capacity);
  return GC_OK;
}
