// greedy_code.hip -- MI355X (gfx950) greedy binary code construction.
//
// Operation (Paliwal et al., arXiv:1507.05398, section "Greedy Algorithms and
// Different Orderings"): walk the 2^n vectors of F_2^n in a fixed ordering and
// append a vector to the code C when popcount(x XOR c) >= d for every word c
// already in C (section "Hamming Distance").  The result is one ordered list.
//
// Execution model: one cooperative persistent kernel.  Its workgroups form
// teams by XCD (1, 2, 4 or 8 teams); a team pulls jobs (codes to build) from
// a queue and builds each with team-wide barriers.  A single code is a queue
// of one job on one team that spans the GPU; a batch pre-fills the queue; the
// server feeds the queue from host memory while the kernel runs.
//
// Most codes need no distance checks: the positional orderings' are linear and
// are built from their generators (linear.h), graded ones up to n = 24 from a
// bitmap of the space (cover_build.h, cover_windows.h).  Single codes of both
// have launches of their own (linear.hip, cover_kernel).  The others take the
// screens:
//
// Building one code: the ordering is cut into windows of consecutive
// positions.  For a window starting with m0 committed words:
//
//   A  near screen   every window candidate is compared with the newest
//                    `near_depth` committed words; a conflict sets the
//                    candidate's bit in the window "dead" mask.
//   C  survivors     every workgroup rebuilds the ordered survivor list in LDS
//                    (capped at kSMax; the window is cut at the cap) and the
//                    team computes the in-window conflict graph among the
//                    survivors as 64x64-bit tiles (earlier-neighbour masks).
//   D  resolve       one wave computes the lexicographically first maximal
//                    independent set of the survivor graph in position order,
//                    which is sequential greedy restricted to the window,
//                    treating survivors whose deep status is unknown as
//                    passing.
//   E  deep scan     survivors whose status is needed are compared with the
//                    older words [0, m0 - near_depth); D then runs again with
//                    the new facts.  When every tentatively accepted survivor
//                    is known to pass, the set is the greedy result for the
//                    window: it is appended to the code.
//
// The paper launched two kernels per candidate and copied |C| to the host
// each time (sections "Parallel Implementation", "Removing Wasted Threads",
// "Dynamic Parallelism"); here |C| stays on the device and one launch covers
// every position of every job.  Its "selective kernel launch" (check part of
// the code first, the rest only if that passes) becomes the near screen /
// deep scan split, reordered newest-first.
//
// Distance checks run as int8 products on the matrix cores (bits as signed
// bytes), or on the vector ALUs (self-orthogonal walks, tuning): v_xor_b32,
// v_bcnt_u32_b32 and v_min3_u32, 2.5 instructions per check.
#include <hip/hip_runtime.h>

#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "binomials.h"
#include "cover.h"
#include "gc_internal.h"
#include "greedy_code.h"
#include "linear.h"

#define GC_VERSION_STRING "greedy_code 0.2.0 (gfx950)"

namespace gcimpl {

constexpr int kWaves = kBlock / 64;                   // waves per workgroup
constexpr int kTile = 1024;                           // candidates per screen tile (16 rows of 64)
constexpr int kRows = kTile / 64;
constexpr int kSegMax = 64 * 64;                      // longest code segment staged at once (words)
constexpr int kSegLoads = kSegMax / kBlock;           // words each thread stages per segment
constexpr int kSMax = 1024;                           // survivors per window (resolve capacity)
constexpr int kNb = kSMax / 64;                       // survivor blocks of 64
constexpr int kAdjWords = 64 * kNb * (kNb + 1) / 2;   // lower-triangular block adjacency
constexpr unsigned long long kWMin = 256;
constexpr unsigned long long kWMax = 1ull << 18;
constexpr int kWordsPerThread = (int)(kWMax / 32 / kBlock);  // window mask words per thread
constexpr unsigned int kDefaultTarget = 768;         // graded orderings
constexpr unsigned int kDefaultTargetLinear = 1000;  // lex and Gray (window cut at kSMax survivors)
constexpr unsigned long long kDefaultNear = 16384;
constexpr unsigned long long kDefaultNearGray = 8192;
// Work per segment after the first, in (group of 4 rows) x (64 words) blocks
// (measured on the n=24..28 screens, matrix-core screen): short segments for a near screen over
// the newest words, where candidates die early and kills should spread
// fast; longer ones for the deep scan and for a near screen over the whole
// code, where most candidates survive long ranges.
constexpr unsigned int kNearBlocks = 16;
constexpr unsigned int kDeepBlocks = 64;
// Deep scans take segments of kFarBlocks blocks once the sweep is kFarAt
// words below the newest end of its range: most survivors that a deep scan
// kills die near that end, so deeper segments lose little to the lag of the
// kills and halve the per-segment merges.
constexpr unsigned int kFarBlocks = 128;
constexpr unsigned long long kFarAt = 1ull << 19;
constexpr unsigned int kDefaultSpin = 1u << 25;
// Near ranges (words) from which the next window's near screen overlaps the
// resolve (measured on the n=24..28 screens).
constexpr unsigned long long kEarlyMinRange = 8192;

enum : int { ST_UNKNOWN = 0, ST_PASS = 1, ST_FAIL = 2 };
enum : int { ACT_NEXT = 0, ACT_DEEP = 1, ACT_STOP = 2 };
enum : int { MODE_AUTO = 0, MODE_TENTATIVE = 1, MODE_DEEP_ALL = 2 };

// Per-team workspace, carved out of one buffer.
struct TeamWs {
  Ctl *ctl;
  unsigned long long *cur;   // kCursors range cursors (kCurLate, kCurEarly, kCurDeep)
  uint32_t *win_dead[2];     // kWMax / 32 each, by window parity
  unsigned long long *adj;   // kAdjWords
  uint32_t *deep_word;       // kSMax
  uint32_t *deep_idx;        // kSMax
  uint32_t *deep_fail;       // kSMax / 32
  uint32_t *job;             // inputs of the job being built
  LinResult *lin;            // linear codes: the generators
  unsigned long long *lin_bits;  // kLinTeamWords: label bitmaps past LDS, over `cover`
  CoverWs *cover;            // graded codes
};

constexpr size_t align256(size_t x) { return (x + 255) / 256 * 256; }
constexpr int kNearTiles = (int)(kWMax / kTile);       // tiles of a window
constexpr int kMinTile = 256;                          // smallest deep-scan tile (tuning)
constexpr int kDeepTiles = (kSMax + kMinTile - 1) / kMinTile;  // tiles of a deep list, at most
// Cursors: the near screen's late part (one per tile), its early part (one
// per tile and window parity), the deep scan's tiles.
constexpr int kCurLate = 0;
constexpr int kCurEarly = kNearTiles;
constexpr int kCurDeep = 3 * kNearTiles;
constexpr int kCursors = kCurDeep + kDeepTiles;
constexpr size_t kOffCtl = 0;
constexpr size_t kOffCur = align256(sizeof(Ctl));
constexpr size_t kOffDead = kOffCur + align256(kCursors * sizeof(unsigned long long));
constexpr size_t kDeadBytes = align256(kWMax / 32 * sizeof(uint32_t));
constexpr size_t kOffAdj = kOffDead + 2 * kDeadBytes;
constexpr size_t kOffDword = kOffAdj + align256(kAdjWords * sizeof(unsigned long long));
constexpr size_t kOffDidx = kOffDword + align256(kSMax * sizeof(uint32_t));
constexpr size_t kOffDfail = kOffDidx + align256(kSMax * sizeof(uint32_t));
// Linear codes: label bitmaps of a team's search, 16 KiB in LDS and then 3.4 MiB
// of the workspace, where a cover team's exchange is otherwise (enough for d <= 10
// at every n; a search that needs more leaves its code to the screens).
constexpr int kLinLdsWords = 2048;
constexpr size_t kOffJob = kOffDfail + align256(kSMax / 32 * sizeof(uint32_t));
constexpr size_t kOffLin = kOffJob + align256(kJobInputWords * sizeof(uint32_t));
constexpr size_t kOffCover = kOffLin + align256(sizeof(LinResult));
constexpr size_t kTeamWsBytes = kOffCover + align256(sizeof(CoverWs)) + (384u << 10);
constexpr unsigned int kLinTeamWords = (kTeamWsBytes - kOffCover) / sizeof(unsigned long long);

__host__ __device__ inline TeamWs team_ws(char *base) {
  TeamWs w;
  w.ctl = reinterpret_cast<Ctl *>(base + kOffCtl);
  w.cur = reinterpret_cast<unsigned long long *>(base + kOffCur);
  w.win_dead[0] = reinterpret_cast<uint32_t *>(base + kOffDead);
  w.win_dead[1] = reinterpret_cast<uint32_t *>(base + kOffDead + kDeadBytes);
  w.adj = reinterpret_cast<unsigned long long *>(base + kOffAdj);
  w.deep_word = reinterpret_cast<uint32_t *>(base + kOffDword);
  w.deep_idx = reinterpret_cast<uint32_t *>(base + kOffDidx);
  w.deep_fail = reinterpret_cast<uint32_t *>(base + kOffDfail);
  w.job = reinterpret_cast<uint32_t *>(base + kOffJob);
  w.lin = reinterpret_cast<LinResult *>(base + kOffLin);
  w.lin_bits = reinterpret_cast<unsigned long long *>(base + kOffCover);
  w.cover = reinterpret_cast<CoverWs *>(base + kOffCover);
  return w;
}

size_t team_workspace_bytes() { return kTeamWsBytes; }

// Candidate walk of a job: which vectors are candidates and in which order.
struct Walk {
  int n, ord;
  int so;                              // self-orthogonal: only even-weight vectors are candidates
};

// The walk is the same for every lane: its fields in scalar registers.
__device__ __forceinline__ Walk uniform_walk(const Walk &w) {
  Walk u;
  u.n = __builtin_amdgcn_readfirstlane(w.n);
  u.ord = __builtin_amdgcn_readfirstlane(w.ord);
  u.so = __builtin_amdgcn_readfirstlane(w.so);
  return u;
}

struct Tables {
  union {
    uint32_t binom[33][33];            // graded orders: C(a, b)
    uint32_t btab[4][256];             // B-ordering: XOR of the basis vectors selected by a byte of p
  };
  unsigned long long off[34];          // graded orders: candidates of the allowed weights below w
};

// Screen tile: code segment (double-buffered), candidate words and ids
// (double-buffered for compaction), per-wave conflict masks.
struct TileLds {
  alignas(16) uint32_t seg[2][kSegMax];
  uint32_t cw[2][kTile];
  uint32_t ci[2][kTile];
  alignas(16) uint32_t cx[2][kTile][8];  // matrix screens: candidate bits as 32 signed bytes, by cw order
  unsigned long long killw[kRows];     // kill mask of each row of 64 live candidates
  unsigned int wcnt[kWaves];
  unsigned long long claim[2];         // [1]: offset (from the newest end) of the next claimed segment
  uint32_t dloc[32];                   // kills found by this workgroup (the tile's dead-bit words)
  uint32_t dseen[32];                  // the tile's published dead bits, as last loaded
};

// In-window resolve (team rank 0 only).
struct ResolveLds {
  unsigned long long adj[kAdjWords];   // survivor adjacency (earlier-neighbour masks)
  unsigned long long accm[kNb];        // accepted mask per block
  uint32_t tlist[kSMax];               // tentatively accepted words
};

struct Lds {
  uint2 lut8[256];                     // byte -> its 8 bits as signed bytes (matrix screens)
  Tables tab;
  Walk walk;
  // job
  alignas(8) uint32_t in[kJobInputWords];  // its inputs (the beginning of a Job)
  int job, n, d, ord, mode;
  uint32_t *code;
  unsigned long long capacity, total, near_depth;
  unsigned long long p_start, m_start, classes;
  unsigned int target, deep_tile;
  int linear;                          // may be built from its generators
  int by_cover;                        // may be built by cover marks
  int mfma;                            // screens (other than self-orthogonal ones) on the matrix cores
  // window
  unsigned long long p0, m0, w, pe, lo;
  unsigned int s, s_tot, ndeep, round, tcount, truncated;
  unsigned int gen_seen;               // resolves of this team seen so far (generation of ctl->resolved)
  unsigned long long tk;               // phase clock (team rank 0): end of the last charged phase
  unsigned long long wfull;            // this window's positions before the cut at kSMax survivors
  unsigned long long e_p0, e_w, e_lo, e_m0;  // the early near screen done for this window (if early)
  unsigned long long nx_p0, nx_w, nx_lo, nx_m0;  // the early near screen of the next window
  unsigned int par, early, nx_early;   // window parity; 1 when [e_lo, e_m0) was screened early
  int status, action, abort;
  // team
  unsigned int xcd, xcd_members, team, team_rank, team_size, team_xcds;
  unsigned int sub_size, sub_rank;     // the team's workgroups on one XCD: their number, this one's (~0: elsewhere)
  unsigned int tgen;                   // team barriers passed (generation of the team's barrier)
  unsigned long long cnt_near, cnt_deep, cnt_pairs;   // this workgroup's executed checks
  unsigned int wsum[kWaves];
  union alignas(16) {
    struct {                           // the windowed screens
      uint32_t s1w[kSMax];             // window survivors, in position order
      uint32_t s1off[kSMax];           // their offsets from the window start
      uint8_t st[kSMax];               // deep status of each survivor (resolve only)
      union alignas(16) {
        TileLds t;
        ResolveLds r;
      } u;
    };
    LinLds<kLinLdsWords> gens;         // linear codes: the search
    uint32_t lin[4][256];              // and then the byte tables of the words
    CoverLds cover;
  };
};

// The LDS of every persistent kernel, one object: functions that are not
// inlined reach it directly (not through generic pointers).
__shared__ Lds g_lds;

// ---------------------------------------------------------------------------
// Small device helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
// min(min(a, b), c) lowers to one v_min3_u32.
__device__ __forceinline__ uint32_t umin3(uint32_t a, uint32_t b, uint32_t c) {
  return umin(umin(a, b), c);
}
__device__ __forceinline__ uint32_t dist(uint32_t a, uint32_t b) { return __builtin_popcount(a ^ b); }

__device__ __forceinline__ unsigned long long ballot(bool p) { return __ballot(p); }

// Load through a pointer known to address global memory.  A generic (flat)
// load also counts on the LDS counter until its data returns, so every LDS
// wait issued meanwhile would wait for the global access as well.
template <typename T>
__device__ __forceinline__ T gload(const T *p) {
  return *(const __attribute__((address_space(1))) T *)p;
}

// A value every lane holds alike, moved to scalar registers.
__device__ __forceinline__ unsigned long long uniform64(unsigned long long x) {
  const unsigned int lo = __builtin_amdgcn_readfirstlane((unsigned int)x);
  const unsigned int hi = __builtin_amdgcn_readfirstlane((unsigned int)(x >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

template <typename T>
__device__ __forceinline__ T *uniform_ptr(T *p) {
  return reinterpret_cast<T *>(uniform64(reinterpret_cast<unsigned long long>(p)));
}

__device__ __forceinline__ unsigned long long lanemask_lt() {
  const unsigned int l = __lane_id();
  return l ? (~0ull >> (64 - l)) : 0ull;
}

// Inclusive prefix sum over the wave (DPP moves: no LDS round trips).
__device__ __forceinline__ unsigned int wave_scan(unsigned int x) {
  x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);   // row_shr:1, 2, 4, 8
  x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);
  x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);
  x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);
  x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return x;
}

// A pointer into global memory.  Operations through it are global (not flat)
// instructions, which count only on the vector-memory counter: an atomic in
// flight does not hold up the waits for LDS reads.
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T *as_global(T *p) {
  return (__attribute__((address_space(1))) T *)p;
}

template <typename T>
__device__ __forceinline__ T ld_relaxed(T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T ld_sys(T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
template <typename T>
__device__ __forceinline__ void st_sys(T *p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ void set_status(Ctl *ctl, int code) {
  int expected = 0;
  __hip_atomic_compare_exchange_strong(&ctl->status, &expected, code, __ATOMIC_RELAXED,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void set_abort(const Params &P) {
  __hip_atomic_store(&P.dq->abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned int xcc_id() {
  unsigned int v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(v));
  return v & (kMaxXcd - 1);
}

// Bounded spin until *p != old.  Gives up after `limit` polls and raises the
// kernel-wide abort flag, so that no wait can hang the device.
__device__ __forceinline__ bool wait_change(unsigned int *p, unsigned int old, const Params &P,
                                            unsigned int limit) {
  unsigned int spins = 0;
  while (ld_relaxed(p) == old) {
    __builtin_amdgcn_s_sleep(1);
    if (++spins > limit) {
      set_abort(P);
      return false;
    }
  }
  return true;
}

// ---------------------------------------------------------------------------
// Teams and barriers
// ---------------------------------------------------------------------------

// Team of an XCD: XCD id mod nteams, or with the server's split the wide
// team 0 for ids below `split` (mod 8) and one narrow team per other XCD.
__device__ __forceinline__ unsigned int team_of(const Params &P, unsigned int x) {
  if (!P.split) return x % (unsigned int)P.nteams;
  const unsigned int r = x & 7u, w = (unsigned int)P.split;
  return r < w ? 0u : 1u + (r - w) % (unsigned int)(P.nteams - 1);
}

// One-time registration: every workgroup counts itself on its XCD, then all
// wait until the XCDs' counts add up to the grid.  No assumption is made about
// the block -> XCD mapping.  A workgroup's rank in its team follows from the
// counts of the team's lower XCDs: one atomic a workgroup, at most 32 on one
// address (with a team counter and a join counter besides, 256 workgroups each
// on one address, a launch of one code took 18 us more).
__device__ __forceinline__ void team_join(Lds &L, const Params &P) {
  if (threadIdx.x < 64) {
    Bar *B = P.bar;
    const unsigned int lane = threadIdx.x;
    const unsigned int x = xcc_id(), t = team_of(P, x);
    unsigned int xcd_rank = 0;
    if (lane == 0)
      xcd_rank = __hip_atomic_fetch_add(&B->xcd[x][2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned int members = 0, all = 0, spins = 0;
    for (;;) {
      members = lane < (unsigned int)kMaxXcd ? ld_relaxed(&B->xcd[lane][2]) : 0u;
      all = (unsigned int)__builtin_amdgcn_readlane((int)wave_scan(members), 63);
      if (all >= gridDim.x) break;
      __builtin_amdgcn_s_sleep(1);
      if (++spins > P.spin_limit) {
        if (lane == 0) set_abort(P);
        break;
      }
    }
    // The team's XCDs, and the one with the most members (the lowest of
    // several), where jobs that want one L2 are built.
    const bool ours = members > 0 && team_of(P, lane) == t;
    const unsigned int mine = ours ? members : 0u, upto = wave_scan(mine);
    unsigned int sub = 0, sub_size = 0;
    for (unsigned int i = 0; i < (unsigned int)kMaxXcd; ++i) {
      const unsigned int m = (unsigned int)__builtin_amdgcn_readlane((int)mine, (int)i);
      if (m > sub_size) {
        sub = i;
        sub_size = m;
      }
    }
    const unsigned int before = (unsigned int)__builtin_amdgcn_readlane((int)(upto - mine), (int)x);
    const unsigned int here = (unsigned int)__builtin_amdgcn_readlane((int)mine, (int)x);
    const unsigned int xcds = (unsigned int)__builtin_popcountll(ballot(ours));
    const unsigned int size = (unsigned int)__builtin_amdgcn_readlane((int)upto, 63);
    if (lane == 0) {
      L.xcd = x;
      L.xcd_members = here;
      L.team = t;
      L.team_rank = before + xcd_rank;
      L.team_size = size;
      L.team_xcds = xcds;
      L.sub_size = sub_size;
      L.sub_rank = x == sub ? xcd_rank : ~0u;
      L.tgen = 0;  // the launch starts with the barrier block cleared
      L.abort = ld_relaxed(&P.dq->abort);
    }
  }
  __syncthreads();
}

// Team-wide barrier, two levels of arrival.  Workgroups count themselves on
// their XCD's counter; the last to arrive (the XCD leader) makes the XCD's
// writes visible device-wide (release) and counts the XCD on the team
// counter; the last XCD leader bumps the team's generation.  Every workgroup
// waits for that generation to change and then acquires at agent scope
// before it reads data written elsewhere.  The counters only grow: the last
// arrival is the one that brings a count to (barriers passed + 1) x members
// (resetting them put two more round trips on the last arriver's path), and
// the generation a workgroup waits for is its own count of the barriers it
// has passed (every member passes every barrier, and none completes before
// all have arrived), so no load precedes the arrival.  The kernel-wide abort
// flag is read on arrival, so its round trip overlaps the wait (an abort
// raised meanwhile is seen at the next wait, where the workgroups still
// running time out anyway); a wait that expires aborts by itself.  Waits are
// bounded by `limit` polls.
__device__ __forceinline__ void team_barrier(Lds &L, const Params &P, unsigned int limit) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    Bar *B = P.bar;
    unsigned int *xc = &B->xcd[L.xcd][0];
    unsigned int *tc = &B->team[L.team][0];
    unsigned int *tgp = &B->team[L.team][1];
    const unsigned int tg = L.tgen;
    const int aborted = ld_relaxed(&P.dq->abort);
    const unsigned int a = __hip_atomic_fetch_add(xc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (a + 1 == (tg + 1) * L.xcd_members) {
      if (L.team_xcds == 1) {
        __hip_atomic_fetch_add(tgp, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        const unsigned int b = __hip_atomic_fetch_add(tc, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        if (b + 1 == (tg + 1) * L.team_xcds)
          __hip_atomic_fetch_add(tgp, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    const bool passed = wait_change(tgp, tg, P, limit);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __builtin_amdgcn_s_waitcnt(0);
    L.tgen = tg + 1u;
    L.abort = aborted != 0 || !passed;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Orderings: position -> word
// ---------------------------------------------------------------------------

// The r-th (from 0) n-bit integer of weight k in increasing order
// (combinatorial number system: the top bit is the largest b with
// C(b, k) <= r).
__device__ __forceinline__ uint32_t unrank_weight(const Tables &T, unsigned long long r, int k, int n) {
  uint32_t x = 0;
  for (int b = n - 1; b >= 0 && k > 0; --b) {
    const unsigned long long c = T.binom[b][k];
    if (r >= c) {
      x |= 1u << b;
      r -= c;
      --k;
    }
  }
  return x;
}

// Word at position p of the walk.  LEX: p.  GRAY: p XOR (p >> 1).  B-ordering
// (section "B-ordering Implementation"): the XOR of the basis vectors b_{j+1}
// over the set bits j of p, which lists 0, b_1, b_2, b_2+b_1, b_3, ...; the
// four bytes of p index four tables of such XORs.  Graded orders (and
// constant weight, a single allowed class): the weight class of p from the
// offsets of the allowed classes, then the rank inside the class.
// Self-orthogonal walks list only the even-weight vectors, in the same
// order: LEX takes p's bits as the top n-1 coordinates and its parity as the
// last one; GRAY takes the even positions (the reflected Gray word at q has
// the weight parity of q); graded walks allow the even classes.
__device__ __forceinline__ uint32_t position_word(const Tables &T, const Walk &K, unsigned long long p) {
  // (The shift is a scalar: a per-lane 0/1 would be hoisted out of the
  // window loop and held in a vector register.)
  const unsigned int so = (unsigned int)__builtin_amdgcn_readfirstlane(K.so != 0 ? 1 : 0);
  if (K.ord == GC_LEX) return (uint32_t)((p << so) | (so & (unsigned int)__builtin_popcountll(p)));
  if (K.ord == GC_GRAY) {
    const unsigned long long q = p << so;
    return (uint32_t)(q ^ (q >> 1));
  }
  if (K.ord == GC_BORDER)
    return T.btab[0][p & 255] ^ T.btab[1][(p >> 8) & 255] ^ T.btab[2][(p >> 16) & 255] ^ T.btab[3][(p >> 24) & 255];
  const int n = K.n;
  int w = 0;
  while (w < n && T.off[w + 1] <= p) ++w;
  const unsigned long long r = p - T.off[w];
  if (K.ord == GC_GRLEX) return unrank_weight(T, r, w, n);
  // GREVLEX: inside weight w, the r-th word is the bit-reversed complement of
  // the r-th weight-(n-w) integer (complement reverses the increasing order,
  // bit reversal turns "differs first at the top" into "at the bottom").
  const uint32_t y = unrank_weight(T, r, n - w, n);
  const uint32_t mask = n == 32 ? 0xffffffffu : ((1u << n) - 1u);
  return __builtin_bitreverse32(~y & mask) >> (32 - n);
}

__constant__ BinomTable kBinomials = make_binom();

// Fill the tables of a walk (whole workgroup): binomials and the offsets of
// the allowed weight classes (bit w of `classes`) for graded walks, the byte
// tables of the basis for a B-ordering, nothing for lex and Gray.
__device__ void init_tables(Tables &T, const Walk &K, unsigned long long classes, const uint32_t *basis) {
  const int n = K.n;
  if (K.ord == GC_LEX || K.ord == GC_GRAY) return;
  if (K.ord == GC_BORDER) {
    for (int i = threadIdx.x; i < 4 * 256; i += blockDim.x) {
      const int byte = i >> 8, v = i & 255;
      uint32_t x = 0;
      for (int j = 0; j < 8; ++j)
        if (((v >> j) & 1) && 8 * byte + j < n) x ^= basis[8 * byte + j];
      T.btab[byte][v] = x;
    }
    __syncthreads();
    return;
  }
  for (int i = threadIdx.x; i < 33 * 33; i += blockDim.x) T.binom[i / 33][i % 33] = kBinomials.c[i / 33][i % 33];
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long acc = 0;
    for (int w = 0; w < 34; ++w) {
      T.off[w] = acc;
      if (w <= n && ((classes >> w) & 1)) acc += T.binom[n][w];
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// The screen: a tile of candidates against code[a, b), whole workgroup
// ---------------------------------------------------------------------------

// Candidates of a screen: window positions (id = offset from the window
// start) or the deep list (id = index into deep_word).  `dead` holds one bit
// per id; a set bit means "closer than d to a committed word".
struct Source {
  const Tables *tab;
  Walk walk;
  unsigned long long p0;
  const uint32_t *words;  // deep list, or null for window positions
  uint32_t *dead;
  __device__ uint32_t word(uint32_t id) const {
    return words ? words[id] : position_word(*tab, walk, p0 + id);
  }
};

// Workgroup compaction: thread t offers entry t (keep, word, id); kept
// entries go densely and in order to buffer dst, and put(new position) runs
// for each of them.  Returns the count.  `between` runs after the first
// barrier (everything written to LDS before the call is visible to it).
template <typename F, typename G>
__device__ unsigned int tile_compact(TileLds &T, int dst, bool keep, uint32_t word, uint32_t id, F &&between,
                                     G &&put) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned long long m = ballot(keep);
  if (lane == 0) T.wcnt[wave] = (unsigned int)__builtin_popcountll(m);
  __syncthreads();
  between();
  unsigned int base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) base += T.wcnt[w];
    total += T.wcnt[w];
  }
  if (keep) {
    const unsigned int pos = base + (unsigned int)__builtin_popcountll(m & lanemask_lt());
    T.cw[dst][pos] = word;
    T.ci[dst][pos] = id;
    put(pos);
  }
  __syncthreads();
  return total;
}

__device__ __forceinline__ unsigned int tile_compact(TileLds &T, int dst, bool keep, uint32_t word, uint32_t id) {
  return tile_compact(T, dst, keep, word, id, [] {}, [](unsigned int) {});
}

// RG rows of 64 live candidates (rows row0 .. row0+RG-1) against the 64
// staged words of one chunk: every word broadcast from LDS serves RG
// candidates per lane, which keeps the LDS read rate below the VALU rate.
// The next four words are read while the current four are compared.  Lanes
// past `live` compare stale entries of the candidate list; the ballot drops
// them.  The rows' kills are OR-ed into the shared kill masks with LDS
// atomics that return nothing, so no wave waits on them.
//
// Self-orthogonal walks (SO) also reject a candidate with an odd number of
// common ones with a word (section "Self Orthogonal Greedy Codes
// Implementation"): the OR of the popcounts of the ANDs has bit 0 set.
template <int RG, bool SO>
__device__ __forceinline__ void rows_chunk(TileLds &T, int cur, int buf, unsigned int row0,
                                           unsigned int chunk, unsigned int live, uint32_t d) {
  const unsigned int lane = threadIdx.x & 63;
  uint32_t x[RG], acc0[RG], acc1[RG], odd[RG];
#pragma unroll
  for (int r = 0; r < RG; ++r) {
    x[r] = T.cw[cur][64u * (row0 + r) + lane];  // row0 + r < kRows
    acc0[r] = acc1[r] = 0xffffffffu;
    odd[r] = 0;
  }
  const uint4 *sp = reinterpret_cast<const uint4 *>(&T.seg[buf][64 * chunk]);
  uint4 c = sp[0];
  // Everything read before the loop is complete here, so the wait inside the
  // loop only covers the read of the current four words.
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
#pragma unroll 2
  for (int i = 0; i < 16; ++i) {
    const uint4 cn = sp[i < 15 ? i + 1 : 15];
    __builtin_amdgcn_sched_barrier(0);  // keep the read ahead of the compares
#pragma unroll
    for (int r = 0; r < RG; ++r) {
      acc0[r] = umin3(acc0[r], dist(x[r], c.x), dist(x[r], c.y));
      acc1[r] = umin3(acc1[r], dist(x[r], c.z), dist(x[r], c.w));
      if (SO) {
        odd[r] |= __builtin_popcount(x[r] & c.x) | __builtin_popcount(x[r] & c.y);
        odd[r] |= __builtin_popcount(x[r] & c.z) | __builtin_popcount(x[r] & c.w);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    c = cn;
  }
#pragma unroll
  for (int r = 0; r < RG; ++r) {
    const bool clash = umin(acc0[r], acc1[r]) < d || (SO && (odd[r] & 1u));
    const unsigned long long k = ballot(clash && 64u * (row0 + r) + lane < live);
    if (lane == 0 && k) __hip_atomic_fetch_or(&T.killw[row0 + r], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// ---- Distance screens on the matrix cores ----------------------------------
//
// With every bit written as a signed byte (+1 for 0, -1 for 1), the dot
// product of two n-bit vectors is n - 2 dist(x, c), so a candidate x is
// closer than d to a word c exactly when dot > n - 2d.  One
// v_mfma_i32_32x32x32_i8 takes 32 words (rows of A) against 32 candidates
// (columns of B) over the 32 bit positions: 1024 distances.  Lane l supplies
// row or column l % 32 and the 16 bit positions 16 (l / 32) .. + 15 as its
// 16 bytes; each lane gets back 16 dot products of its column (32 rows over
// lanes l and l + 32).  The candidate side zeroes the bytes of bits >= n.

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// Four bits of `nib` as four signed bytes: bit k -> byte k = 1 - 2 bit.
__device__ __forceinline__ uint32_t signed_bytes(uint32_t nib) {
  const uint32_t spread = (nib * 0x204081u) & 0x01010101u;  // bit k -> bit 0 of byte k
  return spread * 0xFEu + 0x01010101u;                    // 0 -> 0x01, 1 -> 0xFF, no carries
}

// A word's bits 16 h .. 16 h + 15 as the 16 bytes of a matrix operand, two
// bytes of the word looked up in the table of signed-byte expansions.
__device__ __forceinline__ v4i word_operand(const uint2 *lut8, uint32_t w, unsigned int h) {
  const uint2 lo = lut8[(w >> (16 * h)) & 255u], hi = lut8[(w >> (16 * h + 8)) & 255u];
  v4i r;
  r.x = (int)lo.x;
  r.y = (int)lo.y;
  r.z = (int)hi.x;
  r.w = (int)hi.y;
  return r;
}

__device__ __forceinline__ int max3i(int a, int b, int c) { return max(max(a, b), c); }

// Largest of the 32 dot products a lane holds for its column.
__device__ __forceinline__ int max_dot(const v16i &a, const v16i &b) {
  int m = max3i(a[0], a[1], a[2]);
  m = max3i(m, a[3], a[4]);
  m = max3i(m, a[5], a[6]);
  m = max3i(m, a[7], a[8]);
  m = max3i(m, a[9], a[10]);
  m = max3i(m, a[11], a[12]);
  m = max3i(m, a[13], a[14]);
  m = max3i(m, a[15], b[0]);
  m = max3i(m, b[1], b[2]);
  m = max3i(m, b[3], b[4]);
  m = max3i(m, b[5], b[6]);
  m = max3i(m, b[7], b[8]);
  m = max3i(m, b[9], b[10]);
  m = max3i(m, b[11], b[12]);
  m = max3i(m, b[13], b[14]);
  return max(m, b[15]);
}

// Live candidates 0 .. live-1 (columns, in groups of 32; their operands in
// cx[cur], in the order of cw[cur]) against the slen staged words of
// seg[buf] (rows, in pairs of 32-word blocks).  The segment's (word pair,
// column group) units, pair-major, are cut into one contiguous range per
// wave (they differ by at most one unit, two products); a wave builds a
// pair's operands in registers once and runs them against its groups of that
// pair.  The next group's candidate operand is read from LDS while the
// current group is compared.  Kills go into the rows' kill masks (as 32-bit
// halves) with LDS atomics that return nothing.
__device__ __forceinline__ void mfma_segment(TileLds &T, const uint2 *lut8, int cur, int buf, unsigned int live_v,
                                             unsigned int slen_v, int thr) {
  const unsigned int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, j = lane & 31;
  // Wave-uniform values in scalar registers.
  const unsigned int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned int live = __builtin_amdgcn_readfirstlane(live_v);
  const unsigned int slen = __builtin_amdgcn_readfirstlane(slen_v);
  const unsigned int groups = (live + 31) / 32, units = slen / 64 * groups;
  const unsigned int u_end = (wave + 1) * units / kWaves;
  uint32_t *kill32 = reinterpret_cast<uint32_t *>(T.killw);
  // This lane's 16 bytes of group g's operand (columns past `live` hold stale
  // operands; their results are masked): 32 candidates x 32 bytes per group.
  const v4i *ops = reinterpret_cast<const v4i *>(&T.cx[cur][j][4 * h]);
  auto group = [&](unsigned int g, const v16i &d0, const v16i &d1) {
    const unsigned long long k = __builtin_amdgcn_ballot_w64(max_dot(d0, d1) > thr);
    const unsigned int rest = live - 32 * g;  // live columns of this group (the last may be ragged)
    const uint32_t k32 = ((uint32_t)k | (uint32_t)(k >> 32)) & (rest >= 32 ? 0xffffffffu : (1u << rest) - 1u);
    if (k32 && lane == 0) __hip_atomic_fetch_or(&kill32[g], k32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  const unsigned int u_begin = wave * units / kWaves, share = u_end - u_begin;
  __builtin_amdgcn_s_setprio(3);
  for (unsigned int u = u_begin; u < u_end;) {
    const unsigned int pr = u / groups, g0 = u % groups, g1 = umin(groups, g0 + (u_end - u));
    u += g1 - g0;
    const v4i a0 = word_operand(lut8, T.seg[buf][64 * pr + j], h);
    const v4i a1 = word_operand(lut8, T.seg[buf][64 * pr + 32 + j], h);
    // Two groups per step, their operands in alternating registers; the
    // read of the next step's first operand overlaps the second group.
    const v4i *p = ops + 64 * g0;
    v4i b0 = p[0];
    unsigned int g = g0;
    for (; g + 1 < g1; g += 2, p += 128) {
      const v4i b1 = p[64];
      const v16i d0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b0, (v16i){0}, 0, 0, 0);
      const v16i d1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b0, (v16i){0}, 0, 0, 0);
      group(g, d0, d1);
      b0 = p[g + 2 < g1 ? 128 : 64];
      const v16i e0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b1, (v16i){0}, 0, 0, 0);
      const v16i e1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b1, (v16i){0}, 0, 0, 0);
      group(g + 1, e0, e1);
      // Issue priority falls as the wave's share is done, so that the waves
      // of a SIMD finish together.
      const unsigned int done4 = 4 * (u - (g1 - g - 2) - u_begin);
      if (done4 >= 3 * share) __builtin_amdgcn_s_setprio(0);
      else if (done4 >= 2 * share) __builtin_amdgcn_s_setprio(1);
      else if (done4 >= share) __builtin_amdgcn_s_setprio(2);
    }
    if (g < g1) {
      const v16i d0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, b0, (v16i){0}, 0, 0, 0);
      const v16i d1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, b0, (v16i){0}, 0, 0, 0);
      group(g, d0, d1);
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// Segment length (words, a multiple of 64) staged for `live` candidates: the
// fewer live candidates, the longer the segment, so that the work per segment
// stays near `blocks` (row group of up to 4 rows) x (64 words) blocks: 16 for
// a tile's first segment, where most candidates die early; kNearBlocks,
// kDeepBlocks or kFarBlocks afterwards, to amortise the per-segment merge.
__device__ __forceinline__ unsigned int seg_len_for(unsigned int live, unsigned int blocks) {
  const unsigned int groups = (live + 255) / 256;
  unsigned int p2 = 1;
  while (p2 < groups) p2 <<= 1;
  const unsigned int chunks = blocks / p2;
  return 64u * (chunks ? chunks : 1u);
}

// Screen candidates id0 .. id0+nc-1 of `src` (nc <= kTile, id0 a multiple of
// kTile) against code[a, b) with the whole workgroup, one of `members`
// workgroups that share this tile (this one is number `member`).  Member k
// first screens the k-th newest segment of the tile's first-segment length;
// then the members share `cursor`: each claims the next segment of the rest
// of the range, newest first (offsets count words from b), so together they
// sweep the range from the newest end.  A segment is at
// most 1/(2 members) of the range (so the last claims do not leave a few
// members with long tails) and otherwise 64..4096 words, longer as fewer
// candidates stay live (`blocks`, or `far_blocks` once the sweep is kFarAt
// words deep); it is loaded straight into one of two LDS buffers while the
// other is screened, and the waves split the (group of up to 4 rows of 64
// candidates) x (chunk of 64 words) blocks.  After every segment the kills
// are gathered into the tile's 32 dead-bit words in LDS and published with at
// most 32 atomic ORs; the same 32 words, loaded during the compute, drop the
// candidates that other members killed; the survivors are compacted.  A
// member stops when the range is exhausted or none of its candidates is live:
// it only drops dead candidates, so a claimed segment is left unscanned only
// when every candidate of the tile is dead.  The tile's dead bits are clear
// when a screen starts.  Returns the executed checks (candidate slots x
// words).
// Always inlined: called as a function, its LDS arrays would be reached
// through generic pointers (measured 15 % slower).
template <bool SO>
__device__ __forceinline__ unsigned long long tile_screen(Lds &L, const Source &src, const uint32_t *code_v, uint32_t id0,
                                          uint32_t nc_v, unsigned long long a_v, unsigned long long b_v,
                                          uint32_t d, unsigned long long *cursor, unsigned int members_v,
                                          unsigned int member_v, unsigned int blocks, unsigned int far_blocks = 0) {
  TileLds &T = L.u.t;
  const int tid = threadIdx.x, wave = tid >> 6;
  // The tile, its range and the code are the same for every lane: scalar
  // registers.
  const uint32_t *code = reinterpret_cast<const uint32_t *>(uniform64(reinterpret_cast<unsigned long long>(code_v)));
  const uint32_t nc = __builtin_amdgcn_readfirstlane(nc_v);
  const unsigned long long a = uniform64(a_v), b = uniform64(b_v);
  const unsigned int members = __builtin_amdgcn_readfirstlane(members_v);
  const unsigned int member = __builtin_amdgcn_readfirstlane(member_v);
  const unsigned long long len = b > a ? b - a : 0;
  if (len == 0 || nc == 0) return 0;
  uint32_t *dead = src.dead + (id0 >> 5);  // the tile's dead-bit words
  const int dwords = (int)((nc + 31) / 32);
  const unsigned long long share = (len / (2ull * members) + 63) & ~63ull;
  const unsigned int cap = share < 64 ? 64u : (share > (unsigned long long)kSegMax ? (unsigned)kSegMax : (unsigned)share);
  // First segments: short, so that the tile's first sweep is narrow, and
  // fixed: member k screens the k-th newest (members share one length), so
  // no claim round trip delays the start.  The cursor hands out the rest of
  // the range after them.
  unsigned int live = nc;  // all candidates are live: the tile's dead bits are clear when a screen starts
  unsigned int slen = umin(seg_len_for(live, 16), cap);
  const unsigned long long off0 = (unsigned long long)member * slen, base = (unsigned long long)members * slen;
  if (off0 >= len) return 0;
  auto claim = [&](unsigned int l) {
    return base + __hip_atomic_fetch_add(as_global(cursor), (unsigned long long)l, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
  };
  int cur = 0, buf = 0;
  unsigned long long checks = 0;
  // The segment goes from global memory straight into LDS buffer `to` (the
  // loads write LDS themselves; no registers hold the words).  A clipped
  // segment repeats its oldest word.  The words are in LDS once the issuing
  // wave's vector-memory counter drains: every wave waits for that before the
  // barrier after which the buffer is read.
  auto fetch = [&](unsigned long long o, unsigned int l, int to) {
    const unsigned long long hi = b - o, lo_s = hi > a + l ? hi - l : a;
#pragma unroll
    for (int q = 0; q < kSegLoads; ++q) {
      const unsigned long long idx = lo_s + tid + (unsigned long long)q * kBlock;
      if ((unsigned int)(tid + q * kBlock) < l)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(code + (idx < hi ? idx : hi - 1)),
                                         (__attribute__((address_space(3))) void *)&T.seg[to][q * kBlock + 64 * wave],
                                         4, 0, 0);
    }
  };
  auto fetched = [] { __builtin_amdgcn_s_waitcnt(0x0f70); };  // vmcnt(0)
  // Segment blocks at claim offset o (words below the newest end).
  auto blocks_at = [&](unsigned long long o) { return far_blocks && o >= kFarAt ? far_blocks : blocks; };

  // The first segment and the claim of the second are in flight while the
  // candidates are listed.
  fetch(off0, slen, buf);
  unsigned int next_len = umin(seg_len_for(live, blocks_at(off0)), cap);
  if (tid == 0) T.claim[1] = claim(next_len);
  bool keep = false;
  uint32_t word = 0, id = 0;
  const bool mx = !SO && __builtin_amdgcn_readfirstlane(L.mfma) != 0;
  if (tid < (int)nc) {
    id = id0 + tid;
    word = src.word(id);
    T.cw[0][tid] = word;
    T.ci[0][tid] = id;
    if (mx) {  // the candidate as 32 signed bytes, zero past bit n - 1
      uint32_t e[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int valid = L.n - 4 * q;  // bytes of this dword below bit n
        const uint32_t keep = valid >= 4 ? 0xffffffffu : (valid <= 0 ? 0u : 0xffffffffu >> (32 - 8 * valid));
        e[q] = signed_bytes((word >> (4 * q)) & 15u) & keep;
      }
      uint4 *dst = reinterpret_cast<uint4 *>(T.cx[0][tid]);
      dst[0] = make_uint4(e[0], e[1], e[2], e[3]);
      dst[1] = make_uint4(e[4], e[5], e[6], e[7]);
    }
  }
  const int thr = L.n - 2 * (int)d;  // matrix screens: a dot product above this is a clash
  if (tid < 32) T.dloc[tid] = 0;
  if (tid < kRows) T.killw[tid] = 0;
  fetched();
  __syncthreads();
  unsigned long long next_off = T.claim[1];
  // Each pass: seg[buf] holds the segment being screened, and the following
  // segment (next_off, next_len) is already claimed; it is fetched into the
  // other buffer (last read before the previous pass's first barrier) during
  // the compute, while the claim after it is in flight.  T.claim[1] is
  // rewritten only after the compaction's first barrier, when every thread
  // has read it.
  while (live > 0) {
    const bool more = next_off < len;
    if (more) fetch(next_off, next_len, buf ^ 1);  // in flight during the compute
    uint32_t seen = 0;
    if (tid < dwords)  // kills published by the other members
      seen = __hip_atomic_load(as_global(&dead[tid]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Rows go to 1, 2 or 4 groups of balanced sizes (they differ by at most
    // one; 9..12 rows make 4 groups of 2-3 rather than 3 groups of 4, so that
    // the block count of a segment, groups x chunks, stays a multiple of the
    // 16 waves), and consecutive blocks share a group: every wave gets the
    // same share of the segment.
    const unsigned int rows = (live + 63) / 64, chunks = slen / 64;
    // Self-orthogonal screens keep at most 2 rows per group (their compare
    // needs a third accumulator per row).
    const unsigned int groups = SO ? (rows > 8 ? 8u : (rows > 4 ? 4u : (rows > 2 ? 2u : 1u)))
                                   : (rows > 8 ? 4u : (rows > 4 ? 2u : 1u));
    if (mx) {
      mfma_segment(T, L.lut8, cur, buf, live, slen, thr);
      checks += 32ull * ((live + 31) / 32) * slen;
    } else {
      // A wave's issue priority drops with every block it completes, so the
      // waves of a SIMD progress together and the SIMD still has several waves
      // to interleave when the segment's blocks run out.
      __builtin_amdgcn_s_setprio(3);
      unsigned int done = 0;
      for (unsigned int blk = wave; blk < groups * chunks; blk += kWaves, ++done) {
        const unsigned int g = blk / chunks, chunk = blk % chunks;
        const unsigned int row0 = g * rows / groups, rg = (g + 1) * rows / groups - row0;
        if (!SO && rg == 4) rows_chunk<4, SO>(T, cur, buf, row0, chunk, live, d);
        else if (!SO && rg == 3) rows_chunk<3, SO>(T, cur, buf, row0, chunk, live, d);
        else if (rg == 2) rows_chunk<2, SO>(T, cur, buf, row0, chunk, live, d);
        else rows_chunk<1, SO>(T, cur, buf, row0, chunk, live, d);
        if (done == 0) __builtin_amdgcn_s_setprio(2);
        else if (done == 1) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
      }
      __builtin_amdgcn_s_setprio(0);
      checks += 64ull * rows * slen;
    }
    if (tid < 32) T.dseen[tid] = seen;
    __syncthreads();
    // Claim the segment after the next one; the atomic completes during the
    // merge and the compaction.
    const unsigned int after_len = umin(seg_len_for(live, blocks_at(next_off)), cap);
    unsigned long long after_off = len;
    if (tid == 0 && more) after_off = claim(after_len);
    bool killed = false;
    if (tid < (int)live) {
      killed = (T.killw[tid >> 6] >> (tid & 63)) & 1;
      word = T.cw[cur][tid];
      id = T.ci[cur][tid];
      if (killed) atomicOr(&T.dloc[(id - id0) >> 5], 1u << (id & 31));
    }
    keep = tid < (int)live && !killed && !((T.dseen[(id - id0) >> 5] >> (id & 31)) & 1);
    uint4 op0, op1;  // matrix screens: the candidate's operand moves with it
    if (mx && keep) {
      op0 = reinterpret_cast<const uint4 *>(T.cx[cur][tid])[0];
      op1 = reinterpret_cast<const uint4 *>(T.cx[cur][tid])[1];
    }
    // The kills are published after the compaction's first barrier, which
    // also completes the gathering in dloc and the reads of the kill masks.
    live = tile_compact(T, cur ^ 1, keep, word, id, [&] {
      if (tid < dwords) {  // one atomic per dead-bit word
        const uint32_t mine = T.dloc[tid];
        if (mine & ~T.dseen[tid])
          __hip_atomic_fetch_or(as_global(&dead[tid]), mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (tid < kRows) T.killw[tid] = 0;
      if (tid == 0) T.claim[1] = after_off;
      fetched();  // the next segment is in LDS for every wave after the barrier
    }, [&](unsigned int pos) {
      if (mx) {
        reinterpret_cast<uint4 *>(T.cx[cur ^ 1][pos])[0] = op0;
        reinterpret_cast<uint4 *>(T.cx[cur ^ 1][pos])[1] = op1;
      }
    });
    if (!more) break;
    cur ^= 1;
    buf ^= 1;
    slen = next_len;
    next_off = T.claim[1];
    next_len = after_len;
  }
  return checks;
}

// Tiles of a 2-D screen (candidate tiles x one code range) for a team: with
// fewer tiles than workgroups, workgroup r joins tile r mod tiles as its
// member r / tiles and the workgroups of a tile share its range through the
// tile's cursor; otherwise each workgroup takes tiles r, r + team_size, ...
// alone.  f(tile, members, member).
template <typename F>
__device__ __forceinline__ void for_tiles(unsigned int r_v, unsigned int ts_v, unsigned long long tiles_v, F &&f) {
  // Uniform values, in scalar registers.
  const unsigned long long ts = __builtin_amdgcn_readfirstlane(ts_v);
  const unsigned long long r = __builtin_amdgcn_readfirstlane(r_v);
  const unsigned long long tiles = uniform64(tiles_v);
  if (tiles == 0) return;
  if (tiles < ts) {
    const unsigned long long t = r % tiles;
    f(t, (unsigned int)((ts - t + tiles - 1) / tiles), (unsigned int)(r / tiles));
  } else {
    for (unsigned long long t = r; t < tiles; t += ts) f(t, 1u, 0u);
  }
}

template <typename F>
__device__ __forceinline__ void for_my_tiles(const Lds &L, unsigned long long tiles, F &&f) {
  for_tiles(L.team_rank, L.team_size, tiles, f);
}

// Length of the window after this one: aim for `target` survivors from this
// window's density (every workgroup computes it alike from its own state).
__device__ __forceinline__ unsigned long long next_window_len(const Lds &L) {
  const unsigned long long nwin = L.pe - L.p0;
  unsigned long long next;
  if (L.truncated) {
    next = nwin * 3 / 4;
  } else if (L.s_tot == 0) {
    next = 2 * L.w;
  } else {
    next = L.w * L.target / L.s_tot;
    if (next > 2 * L.w) next = 2 * L.w;
  }
  if (next < kWMin) next = kWMin;
  if (next > kWMax) next = kWMax;
  return (next + 63) & ~63ull;
}

// ---------------------------------------------------------------------------
// Phase D: in-window resolve (team rank 0)
// ---------------------------------------------------------------------------

__device__ void resolve_window(Lds &L, const TeamWs &W) {
  const int tid = threadIdx.x;
  const unsigned int s = L.s;
  const int nb = (int)((s + 63) / 64);
  const int nadj = 64 * nb * (nb + 1) / 2;
  ResolveLds &R = L.u.r;
  Ctl *ctl = W.ctl;

  if (L.round == 0 && L.mode == MODE_DEEP_ALL && L.lo > 0) {
    // Every survivor was already scanned against code[0, lo) (survivor index
    // = deep-list index): every fact is known.
    for (unsigned int j = tid; j < s; j += kBlock)
      L.st[j] = (ld_relaxed(&W.deep_fail[j >> 5]) >> (j & 31)) & 1 ? ST_FAIL : ST_PASS;
    if (tid == 0 && s > 0) ctl->stat_rounds += 1;
  } else if (L.round == 0) {
    for (unsigned int j = tid; j < s; j += kBlock) L.st[j] = L.lo == 0 ? ST_PASS : ST_UNKNOWN;
  } else {
    for (unsigned int k = tid; k < L.ndeep; k += kBlock) {
      const uint32_t word = ld_relaxed(&W.deep_fail[k >> 5]);
      L.st[W.deep_idx[k]] = (word >> (k & 31)) & 1 ? ST_FAIL : ST_PASS;
    }
  }
  // Loads issued in batches of 5 before their LDS stores, so the copy costs
  // two round trips rather than one per element.
  for (int base = 0; base < nadj; base += 5 * kBlock) {
    unsigned long long v[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const int i = base + tid + q * kBlock;
      v[q] = i < nadj ? W.adj[i] : 0ull;
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const int i = base + tid + q * kBlock;
      if (i < nadj) R.adj[i] = v[q];
    }
  }
  __syncthreads();

  if (tid < 64) {
    const unsigned int lane = tid;
    unsigned int tcount = 0, ndeep = 0;
    for (int I = 0; I < nb; ++I) {
      const unsigned int j = 64u * I + lane;
      const int base = 64 * I * (I + 1) / 2;
      const bool valid = j < s;
      const int st = valid ? L.st[j] : ST_FAIL;
      bool killed = st == ST_FAIL;
      for (int J = 0; J < I; ++J) killed |= (R.adj[base + 64 * J + lane] & R.accm[J]) != 0;
      const unsigned long long alive = ballot(!killed);
      const unsigned long long own = R.adj[base + 64 * I + lane];  // earlier neighbours in block
      // Lexicographically first maximal independent set of the block, in
      // synchronous rounds: an undecided survivor is rejected once an earlier
      // neighbour is accepted, and accepted once every earlier neighbour is
      // decided and none is accepted.  The first undecided survivor is always
      // decided, so at most 64 rounds; dependency chains are short in practice.
      unsigned long long acc = 0, und = alive;
      while (und) {
        const bool mine_und = (und >> lane) & 1;
        const bool rej = mine_und && (own & acc) != 0;
        const bool ok = mine_und && !rej && (own & und) == 0;
        const unsigned long long newacc = ballot(ok);
        und &= ~(newacc | ballot(rej));
        acc |= newacc;
      }
      if (lane == 0) R.accm[I] = acc;
      const bool mine = (acc >> lane) & 1;
      const unsigned long long need = ballot(mine && st == ST_UNKNOWN);
      if (mine) R.tlist[tcount + __builtin_popcountll(acc & lanemask_lt())] = L.s1w[j];
      if (mine && st == ST_UNKNOWN) {
        const unsigned int k = ndeep + __builtin_popcountll(need & lanemask_lt());
        W.deep_word[k] = L.s1w[j];
        W.deep_idx[k] = j;
      }
      tcount += __builtin_popcountll(acc);
      ndeep += __builtin_popcountll(need);
    }
    if (lane == 0) {
      L.tcount = tcount;
      L.ndeep = ndeep;
    }
  }
  __syncthreads();

  const unsigned int tcount = L.tcount, ndeep = L.ndeep;
  if (ndeep > 0) {
    for (unsigned int k = tid; k < (ndeep + 31) / 32; k += kBlock) W.deep_fail[k] = 0;
    if (tid < kDeepTiles) W.cur[kCurDeep + tid] = 0;
    if (tid == 0) {
      ctl->ndeep = ndeep;
      ctl->action = ACT_DEEP;
      ctl->stat_rounds += 1;
    }
    __syncthreads();
    return;
  }

  // Commit: every tentatively accepted survivor is known to pass.
  const unsigned long long m0 = L.m0;
  const unsigned long long room = L.capacity > m0 ? L.capacity - m0 : 0;
  const unsigned int nput = tcount < room ? tcount : (unsigned int)room;
  for (unsigned int k = tid; k < nput; k += kBlock) L.code[m0 + k] = R.tlist[k];

  const unsigned long long next = next_window_len(L);
  // Leave this window's dead-bit buffer, its early-screen cursors, the late
  // and deep cursors all clear for their next use (the window after the next
  // one takes this buffer; the other is being filled meanwhile by the early
  // screen of the next window).
  uint32_t *dead = (L.par ? W.win_dead[1] : W.win_dead[0]);
  for (unsigned long long k = tid; k < (L.wfull + 31) / 32; k += kBlock) dead[k] = 0;
  if (tid < kNearTiles) {
    W.cur[kCurLate + tid] = 0;
    W.cur[kCurEarly + L.par * kNearTiles + tid] = 0;
  }
  if (tid < kDeepTiles) W.cur[kCurDeep + tid] = 0;
  if (tid < kSMax / 32) W.deep_fail[tid] = 0;

  if (tid == 0) {
    ctl->stat_windows += 1;
    ctl->stat_surv += L.s;
    if (nput < tcount) {
      ctl->m = m0 + nput;
      set_status(ctl, GC_ECAPACITY);
      ctl->action = ACT_STOP;
    } else {
      ctl->m = m0 + tcount;
      ctl->p = L.pe;
      ctl->w = next;
      ctl->action = ACT_NEXT;
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Building one code with the team
// ---------------------------------------------------------------------------

template <bool SO>
__device__ __forceinline__ void build_code(Lds &L, const Params &P, const TeamWs &W) {
  const int tid = threadIdx.x;
  const unsigned int lane = tid & 63;
  const uint32_t d = (uint32_t)L.d;
  const unsigned int tw = L.team_rank * kWaves + (unsigned int)(tid >> 6);
  const unsigned int tnw = L.team_size * kWaves;
  Ctl *ctl = W.ctl;
  // Phase clock (team rank 0 only): time from the end of one team barrier to
  // the end of the next is charged to the phase in between.  The clock lives
  // in LDS: state held in registers across the window loop gets spilled.
  const bool timer = L.team_rank == 0 && tid == 0;
  if (timer) L.tk = wall_clock64();
  if (tid == 0) {
    L.par = 0;
    L.early = 0;
    // The resolve generation is stable here (the last resolve of the team's
    // previous job is behind a team barrier); from now on every workgroup
    // counts the resolves it sees.
    L.gen_seen = ld_relaxed(&ctl->resolved);
  }
  auto charge = [&](int phase) {
    if (timer) {
      const unsigned long long now = wall_clock64();
      ctl->ticks[phase] += now - L.tk;
      L.tk = now;
    }
  };

  for (;;) {
    if (tid == 0) {
      L.p0 = ld_relaxed(&ctl->p);
      L.m0 = ld_relaxed(&ctl->m);
      L.w = ld_relaxed(&ctl->w);
      L.status = ld_relaxed(&ctl->status);
      L.round = 0;
    }
    __syncthreads();
    if (L.status != 0 || L.abort || L.p0 >= L.total) break;
    // Window bounds: uniform, held in scalar registers.
    const unsigned long long p0 = uniform64(L.p0), m0 = uniform64(L.m0);
    const unsigned long long pe0 = p0 + L.w < L.total ? p0 + L.w : uniform64(L.total);
    const unsigned long long nwin = pe0 - p0;
    // The near screen covers code[lo, m0).  When the team screened this
    // window against code[e_lo, e_m0) while the previous window was being
    // resolved (early), the rest is the words that resolve accepted,
    // code[e_m0, m0); otherwise it is the newest near_depth words.
    const bool early = __builtin_amdgcn_readfirstlane(L.early) != 0;
    if (early && tid == 0 && (L.e_p0 != p0 || L.e_w != nwin)) set_status(ctl, GC_EDEVICE);  // cannot happen
    const unsigned long long lo = early ? uniform64(L.e_lo) : (m0 > L.near_depth ? m0 - L.near_depth : 0);
    const unsigned long long mid = early ? uniform64(L.e_m0) : lo;
    uint32_t *const win_dead = (L.par ? W.win_dead[1] : W.win_dead[0]);
    if (tid == 0) {
      L.lo = lo;
      L.wfull = nwin;
    }

    // ---- A: near screen of [p0, pe0) against code[mid, m0) -----------------
    if (m0 > mid) {
      const Source src{&L.tab, uniform_walk(L.walk), p0, nullptr, win_dead};
      for_my_tiles(L, (nwin + kTile - 1) / kTile, [&](unsigned long long tile, unsigned int members,
                                                      unsigned int member) {
        const unsigned long long id0 = tile * kTile;
        const uint32_t nc = (uint32_t)(nwin - id0 < (unsigned long long)kTile ? nwin - id0 : kTile);
        const unsigned long long c =
            tile_screen<SO>(L, src, L.code, (uint32_t)id0, nc, mid, m0, d, &W.cur[kCurLate + tile], members,
                            member, mid == 0 ? kDeepBlocks : kNearBlocks);
        if (tid == 0) L.cnt_near += c;
      });
    }
    team_barrier(L, P, P.spin_limit);
    charge(0);

    // ---- C: survivor list (every workgroup) and in-window pairs ------------
    {
      if (tid == 0) {
        L.truncated = 0;
        L.pe = pe0;
      }
      __syncthreads();
      // Each thread owns a contiguous run of up to kWordsPerThread mask words
      // (all loaded at once), so survivors come out in position order.
      const unsigned int nwords = (unsigned int)((nwin + 31) / 32);
      const unsigned int per = (nwords + kBlock - 1) / kBlock;
      uint32_t liveb[kWordsPerThread];
      unsigned int cnt = 0;
#pragma unroll
      for (int k = 0; k < kWordsPerThread; ++k) {
        const unsigned int wi = tid * per + k;
        liveb[k] = 0;
        if (k < (int)per && wi < nwords) {
          const uint32_t dead = ld_relaxed(&win_dead[wi]);
          const unsigned long long rem = nwin - 32ull * wi;
          const uint32_t valid = rem >= 32 ? 0xffffffffu : ((1u << rem) - 1u);
          liveb[k] = ~dead & valid;
        }
        cnt += __builtin_popcount(liveb[k]);
      }
      const unsigned int incl = wave_scan(cnt);
      if (lane == 63) L.wsum[tid >> 6] = incl;
      __syncthreads();
      unsigned int idx = incl - cnt;
      for (int wv = 0; wv < (tid >> 6); ++wv) idx += L.wsum[wv];
#pragma unroll
      for (int k = 0; k < kWordsPerThread; ++k) {
        uint32_t bits = liveb[k];
        while (bits) {
          const int bpos = __builtin_ctz(bits);
          bits &= bits - 1;
          const unsigned long long off = 32ull * (tid * per + k) + bpos;
          if (idx < (unsigned int)kSMax) {
            L.s1off[idx] = (uint32_t)off;
          } else if (idx == (unsigned int)kSMax) {
            L.pe = p0 + off;  // the window ends before the first survivor that does not fit
            L.truncated = 1;
          }
          ++idx;
        }
      }
      if (tid == 0) {
        unsigned int tot = 0;
        for (int wv = 0; wv < kWaves; ++wv) tot += L.wsum[wv];
        L.s_tot = tot;
        L.s = tot < (unsigned int)kSMax ? tot : (unsigned int)kSMax;
      }
      __syncthreads();
      // Words of the survivors, one per thread (graded orders unrank in O(n)).
      for (unsigned int k = tid; k < L.s; k += kBlock) L.s1w[k] = position_word(L.tab, uniform_walk(L.walk), p0 + L.s1off[k]);
      __syncthreads();

      const unsigned int s = L.s;
      const unsigned int nb = (s + 63) / 64;
      const unsigned int ntiles = nb * (nb + 1) / 2;
      for (unsigned long long t = tw; t < ntiles; t += tnw) {
        unsigned int I = 0;
        while ((I + 1) * (I + 2) / 2 <= t) ++I;
        const unsigned int J = (unsigned int)t - I * (I + 1) / 2;
        const unsigned int j = 64 * I + lane;
        const uint32_t xj = j < s ? L.s1w[j] : 0u;
        const unsigned int cmax = J == I ? lane : (s - 64 * J < 64 ? s - 64 * J : 64);
        unsigned long long mask = 0;
        for (unsigned int c = 0; c < 64; ++c) {
          const uint32_t y = L.s1w[64 * J + c < s ? 64 * J + c : 0];
          if (c < cmax && (dist(xj, y) < d || (SO && (__builtin_popcount(xj & y) & 1u)))) mask |= 1ull << c;
        }
        if (j >= s) mask = 0;
        W.adj[64 * (I * (I + 1) / 2) + 64 * J + lane] = mask;
        if (lane == 0) atomicAdd(&L.cnt_pairs, 64ull * 64ull);
      }
    }
    // Deep-scan-all policy: every survivor against code[0, lo) right away,
    // from this workgroup's own copy of the survivor list (no barrier needed:
    // the scan reads only the list and the committed code).
    const bool deep_now =
        __builtin_amdgcn_readfirstlane(L.mode) == MODE_DEEP_ALL && lo > 0 && __builtin_amdgcn_readfirstlane(L.s) > 0;
    if (deep_now) {
      charge(1);
      const Source src{&L.tab, uniform_walk(L.walk), 0, L.s1w, W.deep_fail};
      const unsigned int dtile = L.deep_tile;
      for_my_tiles(L, (L.s + dtile - 1) / dtile, [&](unsigned long long tile, unsigned int members,
                                                     unsigned int member) {
        const unsigned long long id0 = tile * dtile;
        const uint32_t nc = (uint32_t)(L.s - id0 < (unsigned long long)dtile ? L.s - id0 : dtile);
        const unsigned long long c =
            tile_screen<SO>(L, src, L.code, (uint32_t)id0, nc, 0, lo, d, &W.cur[kCurDeep + tile], members, member,
                        kDeepBlocks, kFarBlocks);
        if (tid == 0) L.cnt_deep += c;
      });
    }
    team_barrier(L, P, P.spin_limit);
    charge(deep_now ? 3 : 1);

    // The next window is known now: it starts at this window's cut and its
    // length follows from this window's density.  With more than one
    // workgroup in the team, the others screen it against this window's near
    // range while team rank 0 resolves (a deep-scan-all window resolves
    // once); after the resolve only the words it accepts remain to screen.
    // (Kept in LDS: values held in registers across the rounds get spilled.)
    if (tid == 0) {
      // Only when the near range is long enough for the overlap to outweigh
      // the extra screen pass it costs after the resolve, and the next window
      // has few enough tiles that each gets at least two of the workgroups
      // (without rank 0, a window of one tile per workgroup would leave one
      // of them two tiles).
      const unsigned long long nr = m0 - (m0 > L.near_depth ? m0 - L.near_depth : 0);
      const unsigned long long wn = next_window_len(L);
      const unsigned long long tiles_next = (wn + kTile - 1) / kTile;
      const bool en = L.team_size > 1 && L.mode == MODE_DEEP_ALL && L.pe < L.total && nr >= kEarlyMinRange &&
                      2 * tiles_next <= L.team_size - 1;
      L.nx_early = en ? 1u : 0u;
      L.nx_p0 = L.pe;
      L.nx_w = en ? (L.pe + wn < L.total ? wn : L.total - L.pe) : 0;
      L.nx_lo = m0 > L.near_depth ? m0 - L.near_depth : 0;
      L.nx_m0 = m0;
    }
    __syncthreads();

    // ---- D / E rounds ------------------------------------------------------
    for (;;) {
      // Only team rank 0 writes between the barrier before the resolve and
      // the next phase, so the others need not meet it: rank 0 releases its
      // writes and bumps the resolve generation, the others wait for that
      // (bounded) and acquire.
      if (L.team_rank == 0) {
        resolve_window(L, W);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0)
          __hip_atomic_fetch_add(&ctl->resolved, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        if (L.round == 0 && L.nx_early && L.nx_m0 > L.nx_lo) {
          // Early near screen of the next window, by team ranks 1.., into
          // the other dead-bit buffer with its own cursors.
          const unsigned int pn = L.par ^ 1u;
          const unsigned long long w_next = uniform64(L.nx_w), lo_next = uniform64(L.nx_lo);
          const Source src{&L.tab, uniform_walk(L.walk), uniform64(L.nx_p0), nullptr, (pn ? W.win_dead[1] : W.win_dead[0])};
          for_tiles(L.team_rank - 1, L.team_size - 1, (w_next + kTile - 1) / kTile,
                    [&](unsigned long long tile, unsigned int members, unsigned int member) {
                      const unsigned long long id0 = tile * kTile;
                      const uint32_t nc =
                          (uint32_t)(w_next - id0 < (unsigned long long)kTile ? w_next - id0 : kTile);
                      const unsigned long long c = tile_screen<SO>(
                          L, src, L.code, (uint32_t)id0, nc, lo_next, uniform64(L.nx_m0), d,
                          &W.cur[kCurEarly + pn * kNearTiles + tile], members, member,
                          lo_next == 0 ? kDeepBlocks : kNearBlocks);
                      if (tid == 0) L.cnt_near += c;
                    });
        }
        if (tid == 0) {  // the abort flag read before the wait, as at a team barrier
          const int aborted = ld_relaxed(&P.dq->abort);
          const bool passed = wait_change(&ctl->resolved, L.gen_seen, P, P.spin_limit);
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
          __builtin_amdgcn_s_waitcnt(0);
          L.abort = aborted != 0 || !passed;
        }
      }
      if (tid == 0) L.gen_seen += 1u;  // this resolve, seen by every workgroup of the team
      __syncthreads();
      charge(2);
      if (tid == 0) {
        L.action = ld_relaxed(&ctl->action);
        L.ndeep = ld_relaxed(&ctl->ndeep);
        L.status = ld_relaxed(&ctl->status);
      }
      __syncthreads();
      if (L.action != ACT_DEEP || L.status != 0 || L.abort) break;

      // ---- E: deep scan of the listed survivors against code[0, lo) --------
      {
        const unsigned long long nd = L.ndeep;
        const Source src{&L.tab, uniform_walk(L.walk), 0, W.deep_word, W.deep_fail};
        const unsigned int dtile = L.deep_tile;
        for_my_tiles(L, (nd + dtile - 1) / dtile, [&](unsigned long long tile, unsigned int members,
                                                      unsigned int member) {
          const unsigned long long id0 = tile * dtile;
          const uint32_t nc = (uint32_t)(nd - id0 < (unsigned long long)dtile ? nd - id0 : dtile);
          const unsigned long long c =
              tile_screen<SO>(L, src, L.code, (uint32_t)id0, nc, 0, lo, d, &W.cur[kCurDeep + tile], members, member,
                        kDeepBlocks, kFarBlocks);
          if (tid == 0) L.cnt_deep += c;
        });
      }
      if (tid == 0) L.round += 1;
      team_barrier(L, P, P.spin_limit);
      charge(3);
    }
    if (L.action == ACT_STOP || L.status != 0 || L.abort) break;
    if (tid == 0) {  // the next window: its early screen and its buffer parity
      L.early = L.nx_early;
      L.e_p0 = L.nx_p0;
      L.e_w = L.nx_w;
      L.e_lo = L.nx_lo;
      L.e_m0 = L.nx_m0;
      L.par ^= 1u;
    }
  }
}

// d = 1 (not self-orthogonal): every pair of distinct words is at distance
// >= 1, so the code is the walk itself from p_start on.
__device__ void emit_ordering(Lds &L, const TeamWs &W) {
  const unsigned long long m0 = L.m_start, avail = L.capacity > m0 ? L.capacity - m0 : 0;
  const unsigned long long want = L.total > L.p_start ? L.total - L.p_start : 0;
  const unsigned long long count = want < avail ? want : avail;
  const unsigned long long stride = (unsigned long long)L.team_size * kBlock;
  for (unsigned long long k = (unsigned long long)L.team_rank * kBlock + threadIdx.x; k < count; k += stride)
    L.code[m0 + k] = position_word(L.tab, uniform_walk(L.walk), L.p_start + k);
  if (L.team_rank == 0 && threadIdx.x == 0) {
    W.ctl->m = m0 + count;
    if (count < want) set_status(W.ctl, GC_ECAPACITY);
  }
}

// Generators of a linear job by one workgroup of its team.  Not inlined: the
// screens' registers are not affected.
__device__ __noinline__ void find_generators(int n, int d, int ord, unsigned long long capacity, LinResult *res,
                                             unsigned long long *bits) {
  LinLds<kLinLdsWords> &S = g_lds.gens;
  const bool ok = lin_search(S, n, d, ord, 0, bits, kLinTeamWords);
  if (threadIdx.x < 32) res->gen[threadIdx.x] = (int)threadIdx.x < S.dim ? S.gen[threadIdx.x] : 0u;
  if (threadIdx.x == 0) {
    const unsigned long long all = 1ull << S.dim;
    res->ok = ok;
    res->dim = S.dim;
    res->status = all > capacity ? GC_ECAPACITY : GC_OK;
    res->begin = 0;
    res->end = all < capacity ? all : capacity;
  }
}

// A code by the screens.  Not inlined: the registers are its own, whatever the
// kernel around it keeps and calls.  (Inlined, 45 vector registers spilled, and
// 65 beside the calls of the other builders.  n = 24, d = 3 lex 96.9 ms alone,
// 100.4 beside the calls, 92.0 here; n = 25, d = 6 grlex 9.41, 9.52 and 8.90 ms.)
template <bool SO>
__device__ __noinline__ void build_by_screens(Bar *bar_v, DevQueue *dq_v, char *ws_v, unsigned int limit_v) {
  // Arguments are the same for every lane: pointers in scalar registers.
  Params P{};
  P.bar = uniform_ptr(bar_v);
  P.dq = uniform_ptr(dq_v);
  P.spin_limit = (unsigned int)__builtin_amdgcn_readfirstlane((int)limit_v);
  build_code<SO>(g_lds, P, team_ws(uniform_ptr(ws_v)));
}

// A linear code (whole lex or Gray walk) from its generators: team rank 0
// finds them while the others wait, then the team writes the words.  False
// (alike in every workgroup) when the search did not fit its workspace.
__device__ __forceinline__ bool build_linear(Lds &L, const Params &P, const TeamWs &W) {
  if (L.team_rank == 0) find_generators(L.n, L.d, L.ord, L.capacity, W.lin, W.lin_bits);
  team_barrier(L, P, P.spin_limit);
  if (L.abort) return true;
  if (ld_relaxed(&W.lin->ok) == 0) return false;
  const unsigned long long end = ld_relaxed(&W.lin->end);
  lin_word_tables(L.lin, W.lin->gen, ld_relaxed(&W.lin->dim));
  __syncthreads();
  lin_emit(L.lin, L.code, 0, end, (unsigned long long)L.team_rank * kBlock + threadIdx.x,
           (unsigned long long)L.team_size * kBlock);
  if (L.team_rank == 0 && threadIdx.x == 0) {
    W.ctl->m = end;
    if (W.lin->status != 0) set_status(W.ctl, W.lin->status);
  }
  return true;
}

#include "cover_build.h"

// ---------------------------------------------------------------------------
// The persistent kernel: teams pull jobs until the queue is empty
// ---------------------------------------------------------------------------

// Claim the next job (team rank 0, thread 0).  Batch: a fixed count.  Server:
// wait (bounded by idle_limit polls) until the host publishes one, or stop
// when the host asks for shutdown; with the split, team 0 takes the oldest
// wide job first and the other teams only narrow ones.  Returns -1 when the
// team should stop.
__device__ int claim_job(const Params &P, unsigned int team) {
  if (P.njobs_fixed >= 0) {
    const unsigned int j =
        __hip_atomic_fetch_add(&P.dq->claimed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return j < (unsigned int)P.njobs_fixed ? (int)j : -1;
  }
  // Claim the next entry of a ring whose published count lives in host memory.
  auto take = [&](unsigned int *submitted, unsigned int *claimed, unsigned int *ring, int *out) {
    // Acquire: the entries and job descriptors the host published first.
    const unsigned int sub = __hip_atomic_load(submitted, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
    unsigned int c = ld_relaxed(claimed);
    while (c < sub) {
      if (__hip_atomic_compare_exchange_strong(claimed, &c, c + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT)) {
        *out = (int)ld_sys(&ring[c]);
        return true;
      }
    }
    return false;
  };
  unsigned int idle = 0;
  for (;;) {
    if (ld_relaxed(&P.dq->abort)) return -1;
    if (ld_sys(&P.hq->shutdown)) return -1;  // outstanding jobs are abandoned
    if (ld_sys(&P.hq->layout) != P.layout) return -1;  // the host wants other teams: it launches again
    int j = -1;
    if (P.split && team == 0 && take(&P.hq->submitted_wide, &P.dq->claimed_wide, P.ring_wide, &j)) return j;
    if (take(&P.hq->submitted, &P.dq->claimed, P.ring, &j)) return j;
    if (++idle > P.idle_limit) return -1;
    __builtin_amdgcn_s_sleep(8);
  }
}

// The job whose inputs are in L.in, for every phase of its construction.
__device__ __forceinline__ void load_job(Lds &L) {
  const int tid = threadIdx.x;
  const Job &J = *reinterpret_cast<const Job *>(L.in);
  if (tid == 0) {
    L.n = J.n;
    L.d = J.d;
    L.ord = J.ord;
    // Defaults by ordering (measured on the n=24..28 screens): graded
    // orders reject many candidates deep in the code, so they screen the
    // whole code up front; lex screens the newest 16K words and Gray the
    // newest 8K (where almost every rejected candidate meets its killer),
    // and both then deep-scan every survivor once.
    const bool graded = L.ord == GC_GRLEX || L.ord == GC_GREVLEX;
    const int mode = J.mode;
    L.mode = mode ? mode : MODE_DEEP_ALL;
    const unsigned long long nd = J.near_depth;
    L.near_depth = nd ? nd : (graded ? ~0ull : (L.ord == GC_GRAY ? kDefaultNearGray : kDefaultNear));
    const unsigned int tg = J.target;
    L.target = tg ? (tg > (unsigned int)kSMax ? (unsigned int)kSMax : (tg < 16 ? 16 : tg))
                  : (graded ? kDefaultTarget : kDefaultTargetLinear);
    L.code = J.code;
    L.capacity = J.capacity;
    const unsigned int dt = J.deep_tile;
    L.deep_tile = dt ? dt : (unsigned int)kTile;
    L.mfma = J.valu_screen == 0;
    L.linear = J.linear;
    L.by_cover = J.cover;
    const int wclass = J.wclass;
    L.walk.n = L.n;
    L.walk.ord = L.ord;
    L.walk.so = J.so;
    // Allowed weight classes of a graded walk: one class (constant
    // weight), the even ones (self-orthogonal) or all of them.
    L.classes = wclass > 0 ? 1ull << (wclass - 1) : (L.walk.so ? 0x5555555555555555ull : ~0ull);
    L.p_start = J.p_start;
    L.m_start = J.m_start;
    L.total = J.p_stop;
    L.cnt_near = L.cnt_deep = L.cnt_pairs = 0;
  }
  __syncthreads();
  init_tables(L.tab, L.walk, L.classes, J.basis);
  if (tid == 0) {
    // The walk's length: 2^n positions (2^(n-1) self-orthogonal) for the
    // positional walks, the sizes of the allowed classes for graded ones.
    const bool positional = L.ord == GC_LEX || L.ord == GC_GRAY || L.ord == GC_BORDER;
    const unsigned long long len = positional ? (1ull << (L.n - (L.walk.so ? 1 : 0))) : L.tab.off[33];
    if (L.total == 0 || L.total > len) L.total = len;
  }
  __syncthreads();
}

__device__ __forceinline__ void start_ctl(Ctl *c, const Job &J) {
  c->m = J.m_start;
  c->p = J.p_start;
  c->w = kWMin;
  c->status = 0;
  c->action = ACT_NEXT;
  c->ndeep = 0;
  c->stat_windows = c->stat_rounds = c->stat_surv = 0;
  c->stat_near = c->stat_deep = c->stat_pairs = 0;
  c->ticks[0] = c->ticks[1] = c->ticks[2] = c->ticks[3] = 0;
}

// A finished job's outputs but `done`; by one thread.
__device__ __forceinline__ void write_outputs(const Job &J, Job *out, Ctl *c) {
  // All reads first: one round trip.
  const unsigned long long m = ld_relaxed(&c->m), windows = ld_relaxed(&c->stat_windows),
                           rounds = ld_relaxed(&c->stat_rounds), survivors = ld_relaxed(&c->stat_surv),
                           near = ld_relaxed(&c->stat_near), deep = ld_relaxed(&c->stat_deep),
                           pairs = ld_relaxed(&c->stat_pairs), t0 = ld_relaxed(&c->ticks[0]),
                           t1 = ld_relaxed(&c->ticks[1]), t2 = ld_relaxed(&c->ticks[2]), t3 = ld_relaxed(&c->ticks[3]);
  const int status = ld_relaxed(&c->status);
  if (J.count) *J.count = m;
  st_sys(&out->out_count, m);
  st_sys(&out->windows, windows);
  st_sys(&out->rounds, rounds);
  st_sys(&out->survivors, survivors);
  st_sys(&out->chk_near, near);
  st_sys(&out->chk_deep, deep);
  st_sys(&out->chk_pairs, pairs);
  st_sys(&out->ticks_near, t0);
  st_sys(&out->ticks_surv, t1);
  st_sys(&out->ticks_resolve, t2);
  st_sys(&out->ticks_deep, t3);
  st_sys(&out->status, status);
  st_sys(&out->t_done, (unsigned long long)wall_clock64());
}

// Body of the persistent kernel: the team claims jobs until the queue is empty
// (batch), the host shuts it down or it stays idle too long (server).
// kLinear: jobs may be linear (batch and server; a single linear code has
// kernels of its own).
template <bool SO, bool kLinear>
__device__ __forceinline__ void persistent_body(Lds &L, const Params &P) {
  const int tid = threadIdx.x;
  if (tid < 256) L.lut8[tid] = make_uint2(signed_bytes((uint32_t)tid & 15u), signed_bytes((uint32_t)tid >> 4));
  team_join(L, P);
  // The team's workspace pointers are uniform: computed in scalar registers.
  const unsigned int team = __builtin_amdgcn_readfirstlane(L.team);
  char *const base = P.team_ws + (unsigned long long)team * P.team_ws_stride;
  const TeamWs W = team_ws(base);
  // The claim wait (server) may last up to idle_limit polls.
  const unsigned int claim_limit = P.idle_limit + P.spin_limit;

  bool screened = true;  // the window masks may hold the previous job's (or launch's) bits
  while (!L.abort) {
    // The state of the job to come, before the barrier that starts it (every
    // workgroup has left the previous job): the team's first workgroup claims
    // it and copies its inputs to the team's workspace, all words at once (the
    // job may be in host memory, where a field by field read by every
    // workgroup costs a round trip each); the window masks and cursors clear.
    if (L.team_rank == 0 && tid < 64) {
      int j = -1;
      if (tid == 0) j = claim_job(P, L.team);
      j = __builtin_amdgcn_readfirstlane(j);
      if (j >= 0) {
        const uint32_t v = ld_sys(reinterpret_cast<uint32_t *>(&P.jobs[j]) + tid);
        W.job[tid] = v;
        L.in[tid] = v;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
      if (tid == 0) {
        Ctl *c = W.ctl;
        c->job = j;
        if (j >= 0) {
          const Job &J = *reinterpret_cast<const Job *>(L.in);
          st_sys(&P.out[j].t_claim, (unsigned long long)wall_clock64());
          start_ctl(c, J);
        }
      }
    }
    if (screened) {
      for (unsigned long long k = (unsigned long long)L.team_rank * kBlock + tid; k < kWMax / 32;
           k += (unsigned long long)L.team_size * kBlock) {
        W.win_dead[0][k] = 0;
        W.win_dead[1][k] = 0;
      }
      for (unsigned long long k = (unsigned long long)L.team_rank * kBlock + tid; k < kCursors;
           k += (unsigned long long)L.team_size * kBlock)
        W.cur[k] = 0;
      if (L.team_rank == 0 && tid < kSMax / 32) W.deep_fail[tid] = 0;
      screened = false;
    }
    if (L.sub_rank == 0 && tid == 0)
      __hip_atomic_store(&W.cover->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    team_barrier(L, P, claim_limit);
    if (tid < kJobInputWords) L.in[tid] = ld_relaxed(&W.job[tid]);
    if (tid == 0) L.job = ld_relaxed(&W.ctl->job);
    __syncthreads();
    if (L.job < 0 || L.abort) break;

    const Job &J = *reinterpret_cast<const Job *>(L.in);
    load_job(L);
    if (L.d <= 1 && !L.walk.so) emit_ordering(L, W);
    else if ((!kLinear || !L.linear || !build_linear(L, P, W)) && (!L.by_cover || !build_cover<SO>(L, W, &P.dq->abort, P.spin_limit))) {
      build_by_screens<SO>(P.bar, P.dq, base, P.spin_limit);
      screened = true;
    }

    __syncthreads();
    if (tid == 0 && (L.cnt_near | L.cnt_deep | L.cnt_pairs) != 0) {  // (screens only: every workgroup on one address)
      __hip_atomic_fetch_add(&W.ctl->stat_near, L.cnt_near, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&W.ctl->stat_deep, L.cnt_deep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&W.ctl->stat_pairs, L.cnt_pairs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    team_barrier(L, P, P.spin_limit);
    if (L.abort) break;

    // Server jobs also get their words in pinned host memory: the team writes
    // them over the fabric (no copy engine or extra kernel is needed while this
    // kernel holds the GPU), then releases them at system scope before the
    // barrier that precedes `done`.
    // (A job with a status copies none, but meets the barrier: the next job's
    // start clears the status, so all must have read it.)
    if (J.host_copy != nullptr) {
      const unsigned long long m = ld_relaxed(&W.ctl->status) == 0 ? ld_relaxed(&W.ctl->m) : 0ull;
      const uint4 *src = reinterpret_cast<const uint4 *>(L.code);
      uint4 *dst = reinterpret_cast<uint4 *>(J.host_copy);
      const unsigned long long stride = (unsigned long long)L.team_size * kBlock;
      for (unsigned long long k = (unsigned long long)L.team_rank * kBlock + tid; k < m / 4; k += stride)
        dst[k] = src[k];
      for (unsigned long long k = m / 4 * 4 + (unsigned long long)L.team_rank * kBlock + tid; k < m; k += stride)
        J.host_copy[k] = L.code[k];
      // Released once per workgroup, after all of its waves' stores are done
      // (by every wave it took some 20 us), and only where words were written.
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (tid == 0 && (unsigned long long)L.team_rank * kBlock < m / 4 + 4) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
      team_barrier(L, P, P.spin_limit);
      if (L.abort) break;
    }

    // Completion: outputs first, then `done` with system-scope release, so a
    // host that sees done=1 also sees the words and the count.
    if (L.team_rank == 0 && tid == 0) {
      Job *out = &P.out[L.job];
      Ctl *c = W.ctl;
      write_outputs(J, out, c);
      // (A batch's host reads after the launch, which writes everything back.)
      if (P.njobs_fixed >= 0) st_sys(&out->done, 1u);
      else __hip_atomic_store(&out->done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_fetch_add(&P.dq->completed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (P.njobs_fixed == 1 && P.nteams == 1) break;  // a single code: no further claim
  }
}

// Three entry symbols with one body, so that profiles tell the single-code
// launches, the batch launches and the server launches apart.
__global__ void __launch_bounds__(kBlock) greedy_code_kernel(Params P) {
  persistent_body<false, false>(g_lds, P);
}

__global__ void __launch_bounds__(kBlock) greedy_batch_kernel(Params P) {
  persistent_body<false, true>(g_lds, P);
}

__global__ void __launch_bounds__(kBlock) greedy_server_kernel(Params P) {
  persistent_body<false, true>(g_lds, P);
}

// Self-orthogonal codes: the same body with the extra clash rule compiled in
// (a kernel of its own, so the plain screen's registers are unaffected).
__global__ void __launch_bounds__(kBlock) greedy_code_so_kernel(Params P) {
  persistent_body<true, false>(g_lds, P);
}

// One code by cover marks, as an ordinary launch: the workgroups of the XCD
// that the first one to arrive is on, as many as are there when that one
// closes the team.  Every member runs before it can be waited for, so the team
// needs no cooperative launch, which costs a call 50 us more (n = 1: 80 us by
// the persistent kernel, 33 us here).  Workgroups of other XCDs, and
// those that come too late, leave at once.
constexpr unsigned int kCovClosed = 1u << 16;
constexpr unsigned long long kCovJoinTicks = 2000;  // 20 us (100 MHz)

struct CoverArgs {
  Job job;
  Job *out;               // outputs; done: 1 built, 2 not (too few workgroups came on one XCD), 0 a wait expired
  char *team_ws;
  CoverCtl *ctl;          // zero between launches
  unsigned int want;      // workgroups of the team
  unsigned int spin_limit;
};

__device__ __forceinline__ void cover_join(Lds &L, const CoverArgs &A, CoverWs *ws) {
  CoverCtl *const c = A.ctl;
  const unsigned int here = xcc_id() + 1;
  unsigned int seen = 0, rank = ~0u, size = 1;
  if (gridDim.x == 1 || __hip_atomic_compare_exchange_strong(&c->xcd, &seen, here, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT) || seen == here)
    rank = gridDim.x == 1 ? 0u : __hip_atomic_fetch_add(&c->members, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (rank == 0) {
    __hip_atomic_store(&ws->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    if (gridDim.x > 1) {
      const unsigned long long t0 = wall_clock64();
      while (ld_relaxed(&c->members) < A.want && (unsigned long long)wall_clock64() - t0 < kCovJoinTicks)
        __builtin_amdgcn_s_sleep(1);
      size = __hip_atomic_fetch_or(&c->members, kCovClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&c->size, size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  } else if (rank < kCovClosed) {
    unsigned int spins = 0;
    while ((size = ld_relaxed(&c->size)) == 0) {
      __builtin_amdgcn_s_sleep(1);
      if (++spins > A.spin_limit) {
        __hip_atomic_store(&c->abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
  }
  L.sub_rank = rank < kCovClosed ? rank : ~0u;
  L.sub_size = size;
  L.abort = size == 0;
}

template <bool SO>
__global__ void __launch_bounds__(kBlock) cover_kernel(CoverArgs A) {
  Lds &L = g_lds;
  const int tid = threadIdx.x;
  const TeamWs W = team_ws(A.team_ws);
  if (tid == 0) cover_join(L, A, W.cover);
  if (tid < kJobInputWords) L.in[tid] = reinterpret_cast<const uint32_t *>(&A.job)[tid];
  __syncthreads();
  if (L.sub_rank != ~0u && !L.abort) {
    const Job &J = *reinterpret_cast<const Job *>(L.in);
    if (L.sub_rank == 0 && tid == 0) {
      st_sys(&A.out->t_claim, (unsigned long long)wall_clock64());
      start_ctl(W.ctl, J);
    }
    load_job(L);
    const bool built = build_cover<SO>(L, W, &A.ctl->abort, A.spin_limit);
    if (L.sub_rank == 0 && tid == 0 && !L.abort) {
      if (built) write_outputs(J, A.out, W.ctl);
      __hip_atomic_store(&A.ctl->built, built ? 1u : 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // The last workgroup to leave tells how it ended (a wait may have expired in
  // any of them) and clears the join state.
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0 && __hip_atomic_fetch_add(&A.ctl->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x) {
    st_sys(&A.out->done, ld_relaxed(&A.ctl->abort) ? 0u : ld_relaxed(&A.ctl->built));
    unsigned int *const w = reinterpret_cast<unsigned int *>(A.ctl);
    for (unsigned int i = 0; i < sizeof(CoverCtl) / 4; ++i)
      __hip_atomic_store(&w[i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Reset of the barrier block and the device queue before a launch (a kernel
// rather than a memset, so that it can live in captured graphs).  A server's
// queue goes on, an abort of an earlier launch included: a launch that was queued
// behind it stops at once, and the host sees the abort.
__global__ void init_kernel(Bar *bar, DevQueue *dq, int reset_queue) {
  const unsigned int i = blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned int nbar = sizeof(Bar) / sizeof(unsigned int);
  for (unsigned int k = i; k < nbar; k += gridDim.x * blockDim.x) reinterpret_cast<unsigned int *>(bar)[k] = 0;
  if (i == 0) {
    if (reset_queue) {
      dq->claimed = 0;
      dq->claimed_wide = 0;
      dq->completed = 0;
      dq->abort = 0;
    }
    dq->launches += 1;
  }
}

// Reset of the barrier block and the queue, plus the store of one job passed
// by value (the no-allocation entry point: no host-to-device copy).
__global__ void init_job_kernel(Bar *bar, DevQueue *dq, Job *dst, Job job) {
  const unsigned int i = blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned int nbar = sizeof(Bar) / sizeof(unsigned int);
  for (unsigned int k = i; k < nbar; k += gridDim.x * blockDim.x) reinterpret_cast<unsigned int *>(bar)[k] = 0;
  if (i == 0) {
    dq->claimed = 0;
    dq->claimed_wide = 0;
    dq->completed = 0;
    dq->abort = 0;
    dq->launches = 1;
    *dst = job;
  }
}

// Workspace of greedy_code_device_noalloc: barrier block, queue, one job and
// one team workspace (about 3.6 MiB), held by every device the library runs
// on until the process ends.  Host code reaches it only through the address
// hipGetSymbolAddress returns for the current device.
constexpr size_t kScratchBytes =
    align256(sizeof(Bar)) + align256(sizeof(DevQueue)) + align256(sizeof(Job)) + kTeamWsBytes;
static __device__ __align__(256) char scratch[kScratchBytes];
static __device__ CoverCtl scratch_ctl;   // its cover team's join state

// ---------------------------------------------------------------------------
// Measurement probes (the roofline's denominator and the barrier latency)
// ---------------------------------------------------------------------------

// The screen's block loop alone: every wave runs rows_chunk<4> (four rows of
// 64 candidates against a 64-word chunk) `iters` times on LDS filled with
// pseudo-random words, with d = 1 so that nothing is killed.  Each call is
// 16 * 64 lanes * 4 rows * 4 words = 16384 distance checks per wave.
__global__ void __launch_bounds__(kBlock) probe_block_loop_kernel(int iters, unsigned long long *sink) {
  __shared__ TileLds T;
  const int tid = threadIdx.x, wave = tid >> 6;
  uint32_t h = 2654435761u * (uint32_t)(blockIdx.x * kBlock + tid + 1);
  for (int i = tid; i < 2 * kSegMax; i += kBlock) {
    h ^= h << 13; h ^= h >> 17; h ^= h << 5;
    (&T.seg[0][0])[i] = h;
  }
  for (int i = tid; i < 2 * kTile; i += kBlock) {
    h ^= h << 13; h ^= h >> 17; h ^= h << 5;
    (&T.cw[0][0])[i] = h;
  }
  if (tid < kRows) T.killw[tid] = 0;
  __syncthreads();
  for (int it = 0; it < iters; ++it)
    rows_chunk<4, false>(T, 0, 0, 4u * (wave & 3), (unsigned)(wave + it) & 63u, kTile, 1u);
  __syncthreads();
  if (tid == 0) atomicAdd(sink, T.killw[0] + 1ull);
}

// The matrix screen's segment loop alone: every call screens 1024 live
// candidates against a staged segment of 1024 words (1,048,576 checks per
// workgroup) with the threshold above any dot product, so nothing is killed.
__global__ void __launch_bounds__(kBlock) probe_matrix_loop_kernel(int iters, unsigned long long *sink) {
  __shared__ TileLds T;
  __shared__ uint2 lut8[256];
  const int tid = threadIdx.x;
  uint32_t h = 2654435761u * (uint32_t)(blockIdx.x * kBlock + tid + 1);
  for (int i = tid; i < 2 * kSegMax; i += kBlock) {
    h ^= h << 13; h ^= h >> 17; h ^= h << 5;
    (&T.seg[0][0])[i] = h;
  }
  for (int i = tid; i < 2 * kTile * 8; i += kBlock) {
    h ^= h << 13; h ^= h >> 17; h ^= h << 5;
    (&T.cx[0][0][0])[i] = h & 0x01010101u;
  }
  if (tid < 256) lut8[tid] = make_uint2(signed_bytes((uint32_t)tid & 15u), signed_bytes((uint32_t)tid >> 4));
  if (tid < kRows) T.killw[tid] = 0;
  __syncthreads();
  for (int it = 0; it < iters; ++it) mfma_segment(T, lut8, 0, it & 1, (unsigned int)kTile, 1024u, 127);
  __syncthreads();
  if (tid == 0) atomicAdd(sink, T.killw[0] + 1ull);
}

// Team barriers alone: the grid joins one team and crosses `iters` barriers.
__global__ void __launch_bounds__(kBlock) probe_barrier_kernel(Params P, int iters) {
  Lds &L = g_lds;
  team_join(L, P);
  for (int i = 0; i < iters && !L.abort; ++i) team_barrier(L, P, P.spin_limit);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

thread_local std::string g_error;

int fail(int code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_error = buf;
  return code;
}

#define HIP_TRY(expr)                                                                          \
  do {                                                                                         \
    hipError_t e_ = (expr);                                                                    \
    if (e_ != hipSuccess)                                                                      \
      return fail(GC_EDEVICE, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, \
                  __LINE__);                                                                   \
  } while (0)

struct DeviceInfo {
  int cus = 0, coop = 0, blocks_per_cu = 0;
};
std::mutex g_info_mu;
DeviceInfo g_info[64];

int device_info(int dev, int *cus, int *coop, int *blocks_per_cu) {
  std::lock_guard<std::mutex> lk(g_info_mu);
  if (dev < 0 || dev >= 64) return fail(GC_EDEVICE, "device ordinal %d out of range", dev);
  DeviceInfo &di = g_info[dev];
  if (di.cus == 0) {
    HIP_TRY(hipDeviceGetAttribute(&di.cus, hipDeviceAttributeMultiprocessorCount, dev));
    HIP_TRY(hipDeviceGetAttribute(&di.coop, hipDeviceAttributeCooperativeLaunch, dev));
    int nb = 0;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, greedy_code_kernel, kBlock, 0));
    di.blocks_per_cu = nb;
  }
  *cus = di.cus;
  *coop = di.coop;
  *blocks_per_cu = di.blocks_per_cu;
  return GC_OK;
}

hipError_t launch_init(Bar *bar, DevQueue *dq, int reset_queue, hipStream_t stream) {
  hipLaunchKernelGGL(init_kernel, dim3(4), dim3(256), 0, stream, bar, dq, reset_queue);
  return hipGetLastError();
}

hipError_t launch_persistent(const Params &P, unsigned int grid, hipStream_t stream, LaunchKind kind) {
  Params copy = P;
  void *args[] = {&copy};
  const void *fn = kind == LaunchKind::kSingle     ? (const void *)greedy_code_kernel
                   : kind == LaunchKind::kSingleSO ? (const void *)greedy_code_so_kernel
                   : kind == LaunchKind::kBatch    ? (const void *)greedy_batch_kernel
                                                   : (const void *)greedy_server_kernel;
  return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kBlock), args, 0, stream);
}

unsigned long long binom_host(int a, int b) {
  if (b < 0 || b > a) return 0;
  unsigned long long c = 1;
  for (int t = 1; t <= b; ++t) c = c * (unsigned long long)(a - b + t) / (unsigned long long)t;
  return c;
}

int check_job_args(int n, int d, int ordering) {
  if (n < 1 || n > 32) return fail(GC_EINVAL, "n=%d outside [1, 32]", n);
  if (d < 1) return fail(GC_EINVAL, "d=%d must be >= 1", d);
  if (ordering < GC_LEX || ordering > GC_GREVLEX) return fail(GC_EINVAL, "unknown ordering %d", ordering);
  return GC_OK;
}

// Grid for a launch: one workgroup per compute unit unless asked otherwise.
int pick_grid(unsigned int requested, unsigned int *grid) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  int cus = 0, coop = 0, bpc = 0;
  int rc = device_info(dev, &cus, &coop, &bpc);
  if (rc) return rc;
  if (!coop) return fail(GC_EDEVICE, "device %d does not support cooperative launch", dev);
  if (bpc < 1) return fail(GC_EDEVICE, "persistent kernel does not fit on a compute unit");
  const unsigned int g = requested ? requested : (unsigned int)cus;
  if (g > (unsigned int)(cus * bpc))
    return fail(GC_EINVAL, "grid_blocks %u exceeds the co-resident limit %d", g, cus * bpc);
  *grid = g;
  return GC_OK;
}

unsigned int spin_limit_from_env() {
  unsigned int s = kDefaultSpin;
  if (const char *env = getenv("GC_SPIN_LIMIT")) s = (unsigned int)strtoul(env, nullptr, 0);
  return s;
}

// Device workspaces of the plain entry points.  A call takes a free one of
// sufficient size (allocated with hipMalloc the first time it is needed) and
// gives it back when its stream has finished with it; the library keeps them
// for reuse until the process ends and never frees them from an exit handler.
// Concurrent calls on one device get distinct workspaces.
struct WsEntry {
  int dev;
  char *ptr;
  size_t bytes;
  bool busy;
  WsHost host;     // made on the first use that wants it
};
std::mutex g_ws_mu;
std::vector<WsEntry> g_ws;

int acquire_workspace(size_t bytes, char **ptr, int *slot) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_ws_mu);
  for (size_t i = 0; i < g_ws.size(); ++i) {
    WsEntry &e = g_ws[i];
    if (!e.busy && e.dev == dev && e.bytes >= bytes) {
      e.busy = true;
      *ptr = e.ptr;
      *slot = (int)i;
      return GC_OK;
    }
  }
  const size_t rounded = (bytes + (1u << 20) - 1) & ~(size_t)((1u << 20) - 1);
  char *p = nullptr;
  const hipError_t e = hipMalloc((void **)&p, rounded);
  if (e != hipSuccess) return fail(GC_ENOMEM, "workspace of %zu bytes: %s", rounded, hipGetErrorString(e));
  g_ws.push_back(WsEntry{dev, p, rounded, true, WsHost{}});
  *ptr = p;
  *slot = (int)g_ws.size() - 1;
  return GC_OK;
}

void release_workspace(int slot) {
  std::lock_guard<std::mutex> lk(g_ws_mu);
  if (slot >= 0 && (size_t)slot < g_ws.size()) g_ws[slot].busy = false;
}

// Pinned block and events of a workspace in use (kept with it; the pool holds one
// per concurrent call).  The caller holds the workspace, so they are made outside
// the pool's lock.
int workspace_host(int slot, WsHost *out) {
  {
    std::lock_guard<std::mutex> lk(g_ws_mu);
    *out = g_ws[slot].host;
  }
  WsHost &h = *out;
  if (h.ptr && h.begin && h.end) return GC_OK;
  hipError_t e = hipSuccess;
  if (!h.ptr) {
    e = hipHostMalloc((void **)&h.ptr, kWsHostBytes, hipHostMallocCoherent | hipHostMallocMapped);
    if (e == hipSuccess && (e = hipHostGetDevicePointer((void **)&h.dev, h.ptr, 0)) != hipSuccess) {
      (void)hipHostFree(h.ptr);
      h.ptr = nullptr;
    }
  }
  if (e == hipSuccess && !h.begin) e = hipEventCreate(&h.begin);
  if (e == hipSuccess && !h.end) e = hipEventCreate(&h.end);
  std::lock_guard<std::mutex> lk(g_ws_mu);
  g_ws[slot].host = h;
  if (e != hipSuccess) return fail(GC_ENOMEM, "pinned result block: %s", hipGetErrorString(e));
  return GC_OK;
}

__global__ void clear_ctl_kernel(CoverCtl *ctl) {
  reinterpret_cast<unsigned int *>(ctl)[threadIdx.x] = 0;
}

// Join state of a cover launch of a workspace in use, kept with it as well.  The
// first use clears it on the call's own stream: the call's launch follows there,
// and the workspace is free again only once the stream is idle.
int workspace_ctl(int slot, hipStream_t stream, CoverCtl **out) {
  {
    std::lock_guard<std::mutex> lk(g_ws_mu);
    *out = g_ws[slot].host.ctl;
  }
  if (*out) return GC_OK;
  CoverCtl *ctl = nullptr;
  hipError_t e = hipMalloc((void **)&ctl, sizeof(CoverCtl));
  if (e != hipSuccess) return fail(GC_ENOMEM, "join state: %s", hipGetErrorString(e));
  hipLaunchKernelGGL(clear_ctl_kernel, dim3(1), dim3(sizeof(CoverCtl) / sizeof(unsigned int)), 0, stream, ctl);
  e = hipGetLastError();
  if (e != hipSuccess) {
    (void)hipFree(ctl);
    return fail(GC_EDEVICE, "join state: %s", hipGetErrorString(e));
  }
  std::lock_guard<std::mutex> lk(g_ws_mu);
  g_ws[slot].host.ctl = *out = ctl;
  return GC_OK;
}

// Byte layout of a launch workspace: barrier block, device queue, job table,
// then one workspace per team.
struct LaunchLayout {
  size_t off_dq, off_jobs, off_ws, bytes;
};
LaunchLayout launch_layout(int njobs, int nteams) {
  LaunchLayout l;
  l.off_dq = align256(sizeof(Bar));
  l.off_jobs = l.off_dq + align256(sizeof(DevQueue));
  l.off_ws = l.off_jobs + align256(sizeof(Job) * (size_t)njobs);
  l.bytes = l.off_ws + kTeamWsBytes * (size_t)nteams;
  return l;
}

Params launch_params(char *ws, const LaunchLayout &l, int njobs, int nteams) {
  Params P;
  memset(&P, 0, sizeof(P));
  P.jobs = P.out = reinterpret_cast<Job *>(ws + l.off_jobs);
  P.hq = nullptr;
  P.dq = reinterpret_cast<DevQueue *>(ws + l.off_dq);
  P.bar = reinterpret_cast<Bar *>(ws);
  P.njobs_fixed = njobs;
  P.nteams = nteams;
  P.spin_limit = spin_limit_from_env();
  P.idle_limit = 0;
  P.team_ws = ws + l.off_ws;
  P.team_ws_stride = kTeamWsBytes;
  return P;
}

// Run a batch of jobs on `stream` with `nteams` teams and wait for it.  A
// single job goes to the device as a kernel argument, several from the
// workspace's pinned block; the kernel writes the outputs to that block (more
// jobs than it holds are copied from and to `jobs`).
int run_batch(Job *jobs, int njobs, int nteams, unsigned int grid_req, hipStream_t stream,
              float *kernel_ms, LaunchKind kind) {
  if (njobs <= 0) return GC_OK;
  if (nteams != 1 && nteams != 2 && nteams != 4 && nteams != 8)
    return fail(GC_EINVAL, "teams must be 1, 2, 4 or 8 (got %d)", nteams);
  unsigned int grid = 0;
  int rc = pick_grid(grid_req, &grid);
  if (rc) return rc;
  const LaunchLayout lay = launch_layout(njobs, nteams);
  char *ws = nullptr;
  int slot = -1;
  rc = acquire_workspace(lay.bytes, &ws, &slot);
  if (rc) return rc;
  WsHost host;
  rc = workspace_host(slot, &host);
  if (rc) {
    release_workspace(slot);
    return rc;
  }
  Params P = launch_params(ws, lay, njobs, nteams);
  const size_t bytes = sizeof(Job) * (size_t)njobs;
  Job *const seen = bytes <= kWsHostBytes ? reinterpret_cast<Job *>(host.ptr) : nullptr;
  if (seen) {
    memcpy(seen, jobs, bytes);
    P.out = reinterpret_cast<Job *>(host.dev);
  }
  hipError_t e = hipSuccess;
  if (njobs == 1) {
    hipLaunchKernelGGL(init_job_kernel, dim3(4), dim3(256), 0, stream, P.bar, P.dq, P.jobs, jobs[0]);
    e = hipGetLastError();
  } else {
    e = hipMemcpyAsync(P.jobs, seen ? seen : jobs, bytes, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) e = launch_init(P.bar, P.dq, 1, stream);
  }
  if (e == hipSuccess && kernel_ms) e = hipEventRecord(host.begin, stream);
  if (e == hipSuccess) e = launch_persistent(P, grid, stream, kind);
  if (e == hipSuccess && kernel_ms) e = hipEventRecord(host.end, stream);
  if (e == hipSuccess && !seen) e = hipMemcpyAsync(jobs, P.jobs, bytes, hipMemcpyDeviceToHost, stream);
  // The workspace goes back to the pool only once the stream is idle.
  const hipError_t es = hipStreamSynchronize(stream);
  if (e == hipSuccess) e = es;
  if (e == hipSuccess && kernel_ms) e = hipEventElapsedTime(kernel_ms, host.begin, host.end);
  if (e == hipSuccess && seen) memcpy(jobs, seen, bytes);
  if (es == hipSuccess) release_workspace(slot);
  if (e != hipSuccess) return fail(GC_EDEVICE, "persistent kernel failed: %s", hipGetErrorString(e));
  // An expired wait ends the launch: some job is not done.
  for (int i = 0; i < njobs; ++i)
    if (!jobs[i].done) return fail(GC_ETIMEOUT, "a bounded device-side wait expired");
  return GC_OK;
}

// Builds a cover job with a launch of its own and waits for it; outputs into
// *J.  `fixed`: a workspace to use instead of the pool, with its join state
// (may be null).  *built stays false when too few workgroups came to one XCD:
// the persistent kernel then builds the code.
int run_cover(Job *J, hipStream_t stream, char *fixed, CoverCtl *fixed_ctl, float *kernel_ms, bool *built) {
  *built = false;
  int dev = 0, cus = 0, coop = 0, bpc = 0;
  HIP_TRY(hipGetDevice(&dev));
  int rc = device_info(dev, &cus, &coop, &bpc);
  if (rc) return rc;
  const LaunchLayout lay = launch_layout(1, 1);
  char *ws = fixed;
  int slot = -1;
  WsHost host{};
  if (!fixed) {
    rc = acquire_workspace(lay.bytes, &ws, &slot);
    if (rc) return rc;
    rc = workspace_host(slot, &host);
    if (rc == GC_OK) rc = workspace_ctl(slot, stream, &host.ctl);
    if (rc) {
      release_workspace(slot);
      return rc;
    }
  }
  Job *const seen = reinterpret_cast<Job *>(host.ptr);
  CoverArgs A;
  A.job = *J;
  A.job.done = 0;
  A.out = seen ? reinterpret_cast<Job *>(host.dev) : reinterpret_cast<Job *>(ws + lay.off_jobs);
  A.team_ws = ws + lay.off_ws;
  A.ctl = fixed ? fixed_ctl : host.ctl;
  A.want = cover_team_size(J->n, J->d, J->so != 0, kCovTeam);
  A.spin_limit = spin_limit_from_env();
  if (seen) *seen = A.job;
  // Workgroups go to the XCDs in turn: `want` for each of eight.
  const unsigned int grid = A.want == 1 ? 1u : std::min<unsigned int>(8 * A.want, (unsigned int)cus);
  hipError_t e = kernel_ms ? hipEventRecord(host.begin, stream) : hipSuccess;
  if (e == hipSuccess) {
    if (J->so) hipLaunchKernelGGL(cover_kernel<true>, dim3(grid), dim3(kBlock), 0, stream, A);
    else hipLaunchKernelGGL(cover_kernel<false>, dim3(grid), dim3(kBlock), 0, stream, A);
    e = hipGetLastError();
  }
  if (e == hipSuccess && kernel_ms) e = hipEventRecord(host.end, stream);
  Job res = A.job;
  if (e == hipSuccess && !seen) e = hipMemcpyAsync(&res, A.out, sizeof(Job), hipMemcpyDeviceToHost, stream);
  const hipError_t es = hipStreamSynchronize(stream);
  if (e == hipSuccess) e = es;
  if (e == hipSuccess && kernel_ms) e = hipEventElapsedTime(kernel_ms, host.begin, host.end);
  if (e == hipSuccess && seen) res = *seen;
  if (es == hipSuccess) release_workspace(slot);
  if (e != hipSuccess) return fail(GC_EDEVICE, "cover kernel failed: %s", hipGetErrorString(e));
  if (res.done == 0) return fail(GC_ETIMEOUT, "a bounded device-side wait expired");
  if (res.done != 1) return GC_OK;
  // Outputs only: the inputs of a device-side record are not kept.
  memcpy(reinterpret_cast<char *>(J) + offsetof(Job, out_count), reinterpret_cast<char *>(&res) + offsetof(Job, out_count),
         sizeof(Job) - offsetof(Job, out_count));
  *built = true;
  return GC_OK;
}

// Tunings chosen by greedy_code_tune, per device and instance.
struct TuneKey {
  int dev, n, d, ord;
  bool operator<(const TuneKey &o) const {
    if (dev != o.dev) return dev < o.dev;
    if (n != o.n) return n < o.n;
    if (d != o.d) return d < o.d;
    return ord < o.ord;
  }
};
std::mutex g_tune_mu;
std::map<TuneKey, gc_tuning> g_tuned;

bool tuned_for(int n, int d, int ordering, gc_tuning *out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  std::lock_guard<std::mutex> lk(g_tune_mu);
  auto it = g_tuned.find(TuneKey{dev, n, d, ordering});
  if (it == g_tuned.end()) return false;
  *out = it->second;
  return true;
}

void fill_job(Job *J, int n, int d, int ordering, uint32_t *words, uint64_t capacity, uint64_t *count,
              const gc_tuning *tuning) {
  gc_tuning remembered;
  if (!tuning && tuned_for(n, d, ordering, &remembered)) tuning = &remembered;
  memset(J, 0, sizeof(*J));
  J->n = n;
  J->d = job_distance(d);
  J->ord = ordering;
  J->code = words;
  J->capacity = capacity;
  J->count = reinterpret_cast<unsigned long long *>(count);
  if (tuning) {
    J->near_depth = tuning->near_depth;
    J->target = tuning->target_survivors;
    J->mode = (int)tuning->resolve_mode;
    J->deep_tile = tuning->deep_tile;
    J->valu_screen = tuning->valu_screen;
  }
}

bool cover_job(const Job &J) {
  return (J.ord == GC_GRLEX || J.ord == GC_GREVLEX) && J.n <= kCovMaxN && (J.d >= 2 || J.so) &&
         J.near_depth == 0 && J.target == 0 && J.mode == 0 && J.deep_tile == 0 && J.valu_screen == 0;
}

bool team_linear(const Job &J) {
  return linear_job(J) && J.ord != GC_BORDER && lin_words_least(J.n, J.d, 0) <= kLinTeamWords;
}

bool wide_job(const Job &J) {
  const bool one_xcd = J.cover || (J.linear && lin_words_most(J.n, J.d) <= kLinTeamWords);
  return !one_xcd && std::ldexp((double)greedy_code_capacity(J.n, J.d), J.n) >= kWideWork;
}

// About how long the screens take over a job's positions at least, us: some windows
// that grow to 2^18 positions, then those; less than half of what an even density of
// accepted words costs (graded codes accept in bursts).
static double screens_us(const Job &J) {
  const double len = (double)(J.p_stop - J.p_start), b = std::log2(std::max(len, 1.0));
  const double density = J.p_start ? std::min(1.0, (double)J.m_start / (double)J.p_start) : 0.0;
  return 90.0 + 4.0 * std::min(b, 10.0) + 27.0 * std::min(std::max(b - 10.0, 0.0), 8.0) +
         31.0 * std::max(len / 262144.0 - 1.0, 0.0) + 0.05 * density * len;
}

// About how long the marks of a cover job's given words take, with its start, us.
static double cover_given_us(const Job &J) {
  const unsigned int team = cover_team_size(J.n, J.d, J.so != 0, kCovTeam);
  const bool windows = cover_by_windows(J.n, J.d, J.so != 0);
  const double words = J.n > 6 ? (double)(1u << (J.n - 6)) / team : 1.0;
  double near_words = 0;
  for (int j = 0; j < J.d && j <= J.n - 6; ++j) near_words += (double)binom_host(J.n - 6, j);
  const double mark = near_words / (7200.0 * team) + (windows ? 0.02 : 0.0);
  return 40.0 + words * (windows ? 0.011 : 0.021) + (double)J.m_start * std::max(mark, 0.45e-3);
}

// A part of a walk after given words: the other builders pay for all of the code's
// beginning (its marks, or a search), the screens for the positions.  Both are
// estimated; without given words the others are always the faster ones.  (n = 24 d
// = 4 grevlex after 234294 words, by the screens and by marks: 1 position 106 and
// 1217 us, 2^18 577 and 1218, to the end 8.3 and 2.0 ms; n = 24 d = 8 grlex after
// 3336, to the end 0.68 and 1.16 ms; n = 24 d = 13 lex after 4 words, 1 position 90
// and 773 us, to the end 570 and 772.)
static bool part_screened(const Job &J, double other_us) { return J.m_start && other_us > screens_us(J); }

// A linear code, or one built by cover marks, uses one XCD whatever the team
// has: from four such jobs up every XCD is a team of its own (30 jobs of
// n <= 22, 4 and 8 teams: 1.37 to 1.98 and 0.95 to 1.97 ms over six job lists;
// 12 jobs of n <= 14 0.29 and 0.22 ms; 8 jobs bound by the longest the same).
// Codes built by the screens want larger teams for the largest: 4 of 64
// workgroups.
int default_teams(const Job *J, int njobs) {
  if (njobs < 4) return njobs >= 2 ? 2 : 1;
  for (int i = 0; i < njobs; ++i)
    if ((!J[i].linear && !J[i].cover) || wide_job(J[i])) return 4;
  return 8;
}

int prepare_batch(const gc_job *jobs, int njobs, Job *J, int *order) {
  for (int i = 0; i < njobs; ++i) {
    const gc_job &g = jobs[i];
    int rc = check_job_args(g.n, g.d, g.ordering);
    if (rc) return fail(GC_EINVAL, "job %d: %s", i, g_error.c_str());
    if (!g.d_words || ((uintptr_t)g.d_words & 15u) || g.capacity == 0)
      return fail(GC_EINVAL, "job %d: d_words must be a 16-byte aligned device array", i);
    fill_job(&J[i], g.n, g.d, g.ordering, g.d_words, g.capacity, g.d_count, nullptr);
    J[i].linear = team_linear(J[i]);
    J[i].cover = cover_job(J[i]);
  }
  // Teams claim jobs in queue order; the queue holds the jobs longest first
  // (by the exhaustive-scan work bound 2^n * capacity), so that the largest
  // codes do not start last and stretch the launch.
  std::vector<double> est((size_t)njobs);
  for (int i = 0; i < njobs; ++i) {
    order[i] = i;
    est[i] = std::ldexp((double)greedy_code_capacity(J[i].n, J[i].d), J[i].n);
  }
  std::stable_sort(order, order + njobs, [&](int a, int b) { return est[a] > est[b]; });
  return GC_OK;
}

int job_result(const Job &J, uint64_t capacity) {
  if (!J.done) return fail(GC_ETIMEOUT, "job did not complete");
  if (J.status == GC_ECAPACITY)
    return fail(GC_ECAPACITY, "code exceeds capacity %llu", (unsigned long long)capacity);
  if (J.status == GC_ETIMEOUT) return fail(GC_ETIMEOUT, "device barrier wait expired");
  if (J.status != 0) return fail(GC_EDEVICE, "device status %d", J.status);
  return GC_OK;
}

// Device address of `scratch` on the current device, looked up once per
// device with that device current.
std::mutex g_scratch_mu;
char *g_scratch_ptr[64];
CoverCtl *g_scratch_ctl[64];

int scratch_address(char **out, CoverCtl **ctl) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return fail(GC_EDEVICE, "device ordinal %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
    if (e == hipSuccess) e = hipGetSymbolAddress((void **)&g_scratch_ctl[dev], HIP_SYMBOL(scratch_ctl));
    if (e != hipSuccess || !ptr)
      return fail(GC_EDEVICE, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = static_cast<char *>(ptr);
  }
  *out = g_scratch_ptr[dev];
  *ctl = g_scratch_ctl[dev];
  return GC_OK;
}

// ---- generalized problems -------------------------------------------------

// Number of positions of a problem's walk (its candidates).
uint64_t positions_of(const gc_problem &p) {
  if (p.weight >= 0) return p.self_orthogonal && (p.weight & 1) ? 0 : binom_host(p.n, p.weight);
  return 1ull << (p.n - (p.self_orthogonal ? 1 : 0));
}

// Johnson bound A(n, 2e, w) <= floor(n / w * A(n - 1, 2e, w - 1)), with
// A(n, 2e, w) = A(n, 2e, n - w) and A = 1 once w < e; never above C(n, w).
uint64_t johnson_bound(int n, int e, int w) {
  if (w > n - w) w = n - w;
  if (w < e) return 1;
  const uint64_t a = johnson_bound(n - 1, e, w - 1);
  const uint64_t v = (uint64_t)n * a / (uint64_t)w, c = binom_host(n, w);
  return v < c ? v : c;
}

bool problem_plain(const gc_problem &p) {
  return p.ordering <= GC_GREVLEX && p.weight < 0 && !p.self_orthogonal;
}

int check_problem(const gc_problem *p) {
  if (!p) return fail(GC_EINVAL, "problem is NULL");
  const int n = p->n;
  if (n < 1 || n > 32) return fail(GC_EINVAL, "n=%d outside [1, 32]", n);
  if (p->d < 1) return fail(GC_EINVAL, "d=%d must be >= 1", p->d);
  if (p->ordering < GC_LEX || p->ordering > GC_BORDER) return fail(GC_EINVAL, "unknown ordering %d", p->ordering);
  if (p->self_orthogonal != 0 && p->self_orthogonal != 1)
    return fail(GC_EINVAL, "self_orthogonal must be 0 or 1 (got %d)", p->self_orthogonal);
  if (p->weight < -1 || p->weight > n) return fail(GC_EINVAL, "weight %d outside [-1, %d]", p->weight, n);
  if (p->weight >= 0 && p->ordering != GC_LEX && p->ordering != GC_GRLEX && p->ordering != GC_GREVLEX)
    return fail(GC_EINVAL, "a constant weight needs GC_LEX, GC_GRLEX or GC_GREVLEX");
  if (p->self_orthogonal && p->ordering == GC_BORDER)
    return fail(GC_EINVAL, "self_orthogonal cannot be combined with GC_BORDER");
  if (p->ordering == GC_BORDER) {
    // Independence by elimination: reduce each vector by the pivots so far;
    // a vector that reduces to zero depends on the earlier ones.
    uint32_t piv[32] = {0};
    for (int j = 0; j < n; ++j) {
      uint32_t v = p->basis[j];
      if (n < 32 && (v >> n) != 0) return fail(GC_EINVAL, "basis[%d] has bits above n", j);
      bool placed = false;
      for (int b = 31; b >= 0 && !placed; --b) {
        if (!((v >> b) & 1)) continue;
        if (piv[b]) {
          v ^= piv[b];
        } else {
          piv[b] = v;
          placed = true;
        }
      }
      if (!placed) return fail(GC_EINVAL, "basis[%d] depends on the earlier basis vectors", j);
    }
  }
  const uint64_t pos = positions_of(*p);
  const uint64_t stop = p->stop ? p->stop : pos;
  if (stop > pos) return fail(GC_EINVAL, "stop %llu beyond the walk's %llu positions", (unsigned long long)stop,
                              (unsigned long long)pos);
  if (p->start > stop) return fail(GC_EINVAL, "start %llu after stop %llu", (unsigned long long)p->start,
                                   (unsigned long long)stop);
  return GC_OK;
}

uint64_t problem_capacity(const gc_problem &p) {
  const uint64_t pos = positions_of(p);
  const uint64_t stop = p.stop ? p.stop : pos, screened = stop - p.start;
  uint64_t bound;
  if (p.d <= 1 && !p.self_orthogonal) bound = pos;
  else if (p.weight >= 0) bound = johnson_bound(p.n, (job_distance(p.d) + 1) / 2, p.weight);
  else bound = greedy_code_capacity(p.n, p.d);
  if (p.self_orthogonal && bound > (1ull << (p.n / 2))) bound = 1ull << (p.n / 2);
  if (bound > p.prefix + screened) bound = p.prefix + screened;
  return bound > p.prefix ? bound : p.prefix;
}

void fill_job_problem(Job *J, const gc_problem &p, uint32_t *words, uint64_t capacity, uint64_t *count,
                      const gc_tuning *tuning) {
  gc_tuning remembered;
  if (!tuning && problem_plain(p) && tuned_for(p.n, p.d, p.ordering, &remembered)) tuning = &remembered;
  memset(J, 0, sizeof(*J));
  J->n = p.n;
  J->d = job_distance(p.d);
  // One weight class in increasing value is the graded lexicographic walk
  // restricted to that class.
  J->ord = p.weight >= 0 && p.ordering == GC_LEX ? GC_GRLEX : p.ordering;
  J->code = words;
  J->capacity = capacity;
  J->count = reinterpret_cast<unsigned long long *>(count);
  J->wclass = p.weight >= 0 ? p.weight + 1 : 0;
  J->so = p.self_orthogonal;
  J->p_start = p.start;
  J->p_stop = p.stop ? p.stop : positions_of(p);
  J->m_start = p.prefix;
  if (p.ordering == GC_BORDER)
    for (int j = 0; j < p.n; ++j) J->basis[j] = p.basis[j];
  if (tuning) {
    J->near_depth = tuning->near_depth;
    J->target = tuning->target_survivors;
    J->mode = (int)tuning->resolve_mode;
    J->deep_tile = tuning->deep_tile;
    J->valu_screen = tuning->valu_screen;
  }
}

void copy_stats(gc_stats *stats, const Job &J, float ms) {
  if (!stats) return;
  memset(stats, 0, sizeof(*stats));
  stats->count = J.out_count;
  stats->windows = J.windows;
  stats->resolve_rounds = J.rounds;
  stats->survivors = J.survivors;
  stats->checks_near = J.chk_near;
  stats->checks_deep = J.chk_deep;
  stats->checks_pairs = J.chk_pairs;
  stats->kernel_ms = ms;
  stats->near_ms = J.ticks_near / 1e5;
  stats->survivors_ms = J.ticks_surv / 1e5;
  stats->resolve_ms = J.ticks_resolve / 1e5;
  stats->deep_ms = J.ticks_deep / 1e5;
}

}  // namespace gcimpl

using namespace gcimpl;

extern "C" {

const char *gc_last_error(void) { return g_error.c_str(); }

const char *gc_version(void) { return GC_VERSION_STRING; }

uint64_t greedy_code_capacity(int n, int d) {
  if (n < 1 || n > 32 || d < 1) return 0;
  if (d == 1) return 1ull << n;
  if (d > n) return 1;
  int nn = n, dd = d;
  if (dd % 2 == 0) {  // A(n, d) = A(n-1, d-1) for even d
    nn -= 1;
    dd -= 1;
  }
  const int t = (dd - 1) / 2;
  unsigned long long v = 0;
  for (int i = 0; i <= t; ++i) v += binom_host(nn, i);
  return (1ull << nn) / v;
}

int gc_problem_init(gc_problem *p, int n, int d, int ordering) {
  g_error.clear();
  if (!p) return fail(GC_EINVAL, "problem is NULL");
  memset(p, 0, sizeof(*p));
  p->n = n;
  p->d = d;
  p->ordering = ordering;
  p->weight = -1;
  return GC_OK;
}

uint64_t gc_problem_positions(const gc_problem *p) {
  if (check_problem(p)) return 0;
  return positions_of(*p);
}

uint64_t gc_problem_capacity(const gc_problem *p) {
  if (check_problem(p)) return 0;
  return problem_capacity(*p);
}

int greedy_code_problem_device(const gc_problem *p, uint32_t *d_words, uint64_t capacity,
                               uint64_t *d_count, void *hip_stream, const gc_tuning *tuning,
                               gc_stats *stats) {
  g_error.clear();
  int rc = check_problem(p);
  if (rc) return rc;
  if (!d_count) return fail(GC_EINVAL, "d_count is NULL");
  if (!d_words && capacity > 0) return fail(GC_EINVAL, "d_words is NULL");
  if (((uintptr_t)d_words & 15u) != 0) return fail(GC_EINVAL, "d_words must be 16-byte aligned");
  if (p->prefix > capacity) return fail(GC_EINVAL, "prefix %llu exceeds the capacity %llu",
                                        (unsigned long long)p->prefix, (unsigned long long)capacity);
  if (capacity == 0 && positions_of(*p) > 0) return fail(GC_ECAPACITY, "capacity 0 cannot hold a word");
  if (tuning && tuning->resolve_mode > 2) return fail(GC_EINVAL, "resolve_mode %u unknown", tuning->resolve_mode);
  if (tuning && tuning->deep_tile != 0 && tuning->deep_tile != 256 && tuning->deep_tile != 512 &&
      tuning->deep_tile != 1024)
    return fail(GC_EINVAL, "deep_tile %u must be 0, 256, 512 or 1024", tuning->deep_tile);
  if (tuning && tuning->valu_screen > 1) return fail(GC_EINVAL, "valu_screen %u must be 0 or 1", tuning->valu_screen);
  if (stats) memset(stats, 0, sizeof(*stats));
  hipStream_t stream = (hipStream_t)hip_stream;
  const uint64_t stop = p->stop ? p->stop : positions_of(*p);
  if (p->start >= stop) {
    // Nothing to screen: the code is the prefix.
    const unsigned long long m = p->prefix;
    hipError_t e = hipMemcpyAsync(d_count, &m, sizeof(m), hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return fail(GC_EDEVICE, "count store failed: %s", hipGetErrorString(e));
    if (stats) stats->count = m;
    return GC_OK;
  }
  Job J;
  fill_job_problem(&J, *p, d_words, capacity, d_count, tuning);
  float ms = 0.f;
  // (A linear code has words before any position but the first.)
  if (linear_job(J) && !(tuning && tuning->grid_blocks) && (J.p_start > 0) == (J.m_start > 0) &&
      !part_screened(J, linear_given_us(J))) {
    bool built = false;
    rc = run_linear(&J, stream, nullptr, 0, stats ? &ms : nullptr, &built);
    if (rc) return rc;
    if (built) {
      copy_stats(stats, J, ms);
      return job_result(J, capacity);
    }
  }
  J.cover = cover_job(J) && !(tuning && tuning->grid_blocks) && !part_screened(J, cover_given_us(J));
  if (J.cover) {
    bool built = false;
    rc = run_cover(&J, stream, nullptr, nullptr, stats ? &ms : nullptr, &built);
    if (rc) return rc;
    if (built) {
      copy_stats(stats, J, ms);
      return job_result(J, capacity);
    }
  }
  rc = run_batch(&J, 1, 1, tuning ? tuning->grid_blocks : 0, stream, stats ? &ms : nullptr,
                 p->self_orthogonal ? LaunchKind::kSingleSO : LaunchKind::kSingle);
  if (rc) return rc;
  copy_stats(stats, J, ms);
  return job_result(J, capacity);
}

int greedy_code_device_ex(int n, int d, int ordering, uint32_t *d_words, uint64_t capacity,
                          uint64_t *d_count, void *hip_stream, const gc_tuning *tuning,
                          gc_stats *stats) {
  g_error.clear();
  int rc = check_job_args(n, d, ordering);
  if (rc) return rc;
  if (capacity == 0 && d_words) return fail(GC_ECAPACITY, "capacity 0 cannot hold the zero word");
  gc_problem p;
  gc_problem_init(&p, n, d, ordering);
  return greedy_code_problem_device(&p, d_words, capacity, d_count, hip_stream, tuning, stats);
}

int greedy_code_device(int n, int d, int ordering, uint32_t *d_words, uint64_t capacity,
                       uint64_t *d_count, void *hip_stream) {
  return greedy_code_device_ex(n, d, ordering, d_words, capacity, d_count, hip_stream, nullptr, nullptr);
}

int greedy_code_device_noalloc(int n, int d, int ordering, uint32_t *d_words, uint64_t capacity,
                               uint64_t *d_count, void *hip_stream) {
  g_error.clear();
  int rc = check_job_args(n, d, ordering);
  if (rc) return rc;
  if (!d_count) return fail(GC_EINVAL, "d_count is NULL");
  if (!d_words && capacity > 0) return fail(GC_EINVAL, "d_words is NULL");
  if (((uintptr_t)d_words & 15u) != 0) return fail(GC_EINVAL, "d_words must be 16-byte aligned");
  if (capacity == 0) return fail(GC_ECAPACITY, "capacity 0 cannot hold the zero word");
  const LaunchLayout lay = launch_layout(1, 1);
  if (lay.bytes > kScratchBytes)
    return fail(GC_EINVAL, "the launch needs %zu bytes of scratch, the library holds %zu", lay.bytes,
                kScratchBytes);
  char *base = nullptr;
  CoverCtl *ctl = nullptr;
  rc = scratch_address(&base, &ctl);
  if (rc) return rc;
  Job J;
  fill_job(&J, n, d, ordering, d_words, capacity, d_count, nullptr);
  hipStream_t stream = (hipStream_t)hip_stream;
  if (linear_job(J)) {
    bool built = false;
    rc = run_linear(&J, stream, base, kScratchBytes, nullptr, &built);
    if (rc) return rc;
    if (built) return job_result(J, capacity);
  }
  J.cover = cover_job(J);
  if (J.cover) {
    bool built = false;
    rc = run_cover(&J, stream, base, ctl, nullptr, &built);
    if (rc) return rc;
    if (built) return job_result(J, capacity);
  }
  unsigned int grid = 0;
  rc = pick_grid(0, &grid);
  if (rc) return rc;
  const Params P = launch_params(base, lay, 1, 1);
  hipLaunchKernelGGL(init_job_kernel, dim3(4), dim3(256), 0, stream, P.bar, P.dq, P.jobs, J);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = launch_persistent(P, grid, stream, LaunchKind::kSingle);
  DevQueue dq;
  memset(&dq, 0, sizeof(dq));
  if (e == hipSuccess) e = hipMemcpyAsync(&J, P.jobs, sizeof(Job), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipMemcpyAsync(&dq, P.dq, sizeof(dq), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return fail(GC_EDEVICE, "persistent kernel failed: %s", hipGetErrorString(e));
  if (dq.abort) return fail(GC_ETIMEOUT, "a bounded device-side wait expired");
  return job_result(J, capacity);
}

int greedy_code_problem(const gc_problem *p, uint32_t *out_words, uint64_t *out_count) {
  g_error.clear();
  if (!out_count) return fail(GC_EINVAL, "out_count is NULL");
  int rc = check_problem(p);
  if (rc) return rc;
  const uint64_t bound = problem_capacity(*p);
  const uint64_t cap = *out_count;
  if (!out_words && cap > 0) return fail(GC_EINVAL, "out_words is NULL");
  if (p->prefix > cap) return fail(GC_EINVAL, "prefix %llu exceeds the capacity %llu",
                                   (unsigned long long)p->prefix, (unsigned long long)cap);
  const uint64_t dcap = cap < bound ? cap : bound;
  if (dcap == 0) {
    *out_count = bound;
    if (bound == 0) return GC_OK;  // no candidates and no prefix: the empty code
    return fail(GC_ECAPACITY, "capacity 0 cannot hold a word");
  }
  uint32_t *dw = nullptr;
  uint64_t *dc = nullptr;
  HIP_TRY(hipMalloc((void **)&dw, dcap * sizeof(uint32_t)));
  hipError_t e = hipMalloc((void **)&dc, sizeof(uint64_t));
  if (e == hipSuccess && p->prefix)
    e = hipMemcpy(dw, out_words, p->prefix * sizeof(uint32_t), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipFree(dw);
    if (dc) (void)hipFree(dc);
    return fail(GC_ENOMEM, "device buffers: %s", hipGetErrorString(e));
  }
  rc = greedy_code_problem_device(p, dw, dcap, dc, nullptr, nullptr, nullptr);
  if (rc == GC_OK) {
    uint64_t count = 0;
    e = hipMemcpy(&count, dc, sizeof(count), hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(out_words, dw, count * sizeof(uint32_t), hipMemcpyDeviceToHost);
    if (e != hipSuccess) rc = fail(GC_EDEVICE, "hipMemcpy failed: %s", hipGetErrorString(e));
    else *out_count = count;
  } else if (rc == GC_ECAPACITY) {
    *out_count = bound;
  }
  (void)hipFree(dw);
  (void)hipFree(dc);
  return rc;
}

int greedy_code(int n, int d, int ordering, uint32_t *out_words, uint64_t *out_count) {
  g_error.clear();
  if (!out_count) return fail(GC_EINVAL, "out_count is NULL");
  int rc = check_job_args(n, d, ordering);
  if (rc) return rc;
  gc_problem p;
  gc_problem_init(&p, n, d, ordering);
  return greedy_code_problem(&p, out_words, out_count);
}

int gc_probe_block_loop(int wgs_per_cu, int iters, double *checks_per_s) {
  g_error.clear();
  if (!checks_per_s || wgs_per_cu < 1 || wgs_per_cu > 2 || iters < 1)
    return fail(GC_EINVAL, "wgs_per_cu must be 1 or 2, iters >= 1, checks_per_s non-NULL");
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  int cus = 0;
  HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  int per_cu = 0;
  HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, probe_block_loop_kernel, kBlock, 0));
  if (per_cu < wgs_per_cu) return fail(GC_EINVAL, "only %d probe workgroups fit a compute unit", per_cu);
  char *ws = nullptr;
  int slot = -1;
  int rc = acquire_workspace(256, &ws, &slot);
  if (rc) return rc;
  unsigned long long *sink = reinterpret_cast<unsigned long long *>(ws);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  const unsigned int grid = (unsigned int)(cus * wgs_per_cu);
  // warm-up, then the timed launch
  if (e == hipSuccess) hipLaunchKernelGGL(probe_block_loop_kernel, dim3(grid), dim3(kBlock), 0, nullptr, 8, sink);
  if (e == hipSuccess) e = hipEventRecord(e0, nullptr);
  if (e == hipSuccess) hipLaunchKernelGGL(probe_block_loop_kernel, dim3(grid), dim3(kBlock), 0, nullptr, iters, sink);
  if (e == hipSuccess) e = hipGetLastError();
  if (e == hipSuccess) e = hipEventRecord(e1, nullptr);
  if (e == hipSuccess) e = hipEventSynchronize(e1);
  float ms = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  release_workspace(slot);
  if (e != hipSuccess) return fail(GC_EDEVICE, "block-loop probe failed: %s", hipGetErrorString(e));
  const double checks = (double)grid * kWaves * (double)iters * 16384.0;
  *checks_per_s = checks / (ms * 1e-3);
  return GC_OK;
}

int gc_probe_matrix_loop(int iters, double *checks_per_s) {
  g_error.clear();
  if (!checks_per_s || iters < 1) return fail(GC_EINVAL, "iters >= 1 and checks_per_s non-NULL");
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  int cus = 0;
  HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  char *ws = nullptr;
  int slot = -1;
  int rc = acquire_workspace(256, &ws, &slot);
  if (rc) return rc;
  unsigned long long *sink = reinterpret_cast<unsigned long long *>(ws);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  const unsigned int grid = (unsigned int)cus;
  if (e == hipSuccess) hipLaunchKernelGGL(probe_matrix_loop_kernel, dim3(grid), dim3(kBlock), 0, nullptr, 4, sink);
  if (e == hipSuccess) e = hipEventRecord(e0, nullptr);
  if (e == hipSuccess) hipLaunchKernelGGL(probe_matrix_loop_kernel, dim3(grid), dim3(kBlock), 0, nullptr, iters, sink);
  if (e == hipSuccess) e = hipGetLastError();
  if (e == hipSuccess) e = hipEventRecord(e1, nullptr);
  if (e == hipSuccess) e = hipEventSynchronize(e1);
  float ms = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  release_workspace(slot);
  if (e != hipSuccess) return fail(GC_EDEVICE, "matrix-loop probe failed: %s", hipGetErrorString(e));
  const double checks = (double)grid * (double)iters * 1048576.0;
  *checks_per_s = checks / (ms * 1e-3);
  return GC_OK;
}

int gc_probe_barrier(int iters, double *us_per_barrier) {
  g_error.clear();
  if (!us_per_barrier || iters < 1) return fail(GC_EINVAL, "iters >= 1 and us_per_barrier non-NULL");
  unsigned int grid = 0;
  int rc = pick_grid(0, &grid);
  if (rc) return rc;
  const LaunchLayout lay = launch_layout(0, 1);
  char *ws = nullptr;
  int slot = -1;
  rc = acquire_workspace(lay.bytes, &ws, &slot);
  if (rc) return rc;
  Params P = launch_params(ws, lay, 0, 1);
  Params copy = P;
  int it = iters;
  void *args[] = {&copy, &it};
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e == hipSuccess) e = launch_init(P.bar, P.dq, 1, nullptr);
  if (e == hipSuccess) e = hipEventRecord(e0, nullptr);
  if (e == hipSuccess)
    e = hipLaunchCooperativeKernel((const void *)probe_barrier_kernel, dim3(grid), dim3(kBlock), args, 0, nullptr);
  if (e == hipSuccess) e = hipEventRecord(e1, nullptr);
  DevQueue dq;
  memset(&dq, 0, sizeof(dq));
  if (e == hipSuccess) e = hipMemcpy(&dq, P.dq, sizeof(dq), hipMemcpyDeviceToHost);
  float ms = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (e == hipSuccess) release_workspace(slot);
  if (e != hipSuccess) return fail(GC_EDEVICE, "barrier probe failed: %s", hipGetErrorString(e));
  if (dq.abort) return fail(GC_ETIMEOUT, "a bounded device-side wait expired");
  *us_per_barrier = ms * 1e3 / iters;
  return GC_OK;
}

int greedy_code_batch(gc_job *jobs, int njobs, int teams, void *hip_stream, float *kernel_ms) {
  g_error.clear();
  if (njobs < 0 || (!jobs && njobs > 0)) return fail(GC_EINVAL, "bad job array");
  std::vector<Job> J((size_t)njobs);
  std::vector<int> order((size_t)njobs);
  int rc0 = prepare_batch(jobs, njobs, J.data(), order.data());
  if (rc0) return rc0;
  if (teams == 0) teams = default_teams(J.data(), njobs);
  std::vector<Job> Q((size_t)njobs);
  for (int k = 0; k < njobs; ++k) Q[k] = J[order[k]];
  float ms = 0.f;
  int rc = run_batch(Q.data(), njobs, teams, 0, (hipStream_t)hip_stream, &ms, LaunchKind::kBatch);
  if (kernel_ms) *kernel_ms = ms;
  for (int k = 0; k < njobs; ++k) J[order[k]] = Q[k];
  for (int i = 0; i < njobs; ++i) {
    jobs[i].count = J[i].out_count;
    jobs[i].status = J[i].done ? J[i].status : GC_ETIMEOUT;
    jobs[i].device_ms = J[i].done ? (double)(J[i].t_done - J[i].t_claim) / 1e5 : 0.0;
  }
  if (rc) return rc;
  for (int i = 0; i < njobs; ++i)
    if (jobs[i].status) return fail(jobs[i].status, "job %d failed with status %d", i, jobs[i].status);
  return GC_OK;
}


int greedy_code_tune(int n, int d, int ordering, void *hip_stream, gc_tuning *best, float *best_ms) {
  g_error.clear();
  int rc = check_job_args(n, d, ordering);
  if (rc) return rc;
  if (!best) return fail(GC_EINVAL, "best is NULL");
  memset(best, 0, sizeof(*best));
  if (best_ms) *best_ms = 0.f;
  if (d <= 1 || d > n) return GC_OK;  // the code is fixed without a search: nothing to tune
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  hipStream_t st = (hipStream_t)hip_stream;
  const uint64_t cap = greedy_code_capacity(n, d);
  // Candidates: near-screen depth (whole code, 64K, 16K or 4K newest words)
  // with either deep-scan policy; then the fastest with a larger window.
  std::vector<gc_tuning> cands = {
      {~0ull, 0, 0, 0, 0},        {65536ull, 0, 0, 2, 0}, {65536ull, 0, 0, 1, 0},
      {16384ull, 0, 0, 2, 0},     {16384ull, 0, 0, 1, 0}, {4096ull, 0, 0, 2, 0},
  };
  cands.push_back({0, 0, 0, 0, 0});  // no tuning: from the generators, by cover marks, or the defaults
  uint32_t *words = nullptr;
  HIP_TRY(hipMalloc((void **)&words, (size_t)cap * sizeof(uint32_t)));
  std::vector<uint32_t> ref, cur;
  uint64_t ref_m = 0;
  float best_t = 0.f;
  int best_i = -1;
  auto run = [&](const gc_tuning &t, float *ms, std::vector<uint32_t> &out) -> int {
    Job J;
    fill_job(&J, n, d, ordering, words, cap, nullptr, &t);
    bool built = false;
    J.cover = cover_job(J);
    int r = linear_job(J) ? run_linear(&J, st, nullptr, 0, ms, &built)
            : J.cover     ? run_cover(&J, st, nullptr, nullptr, ms, &built)
                          : GC_OK;
    if (r == GC_OK && !built) r = run_batch(&J, 1, 1, 0, st, ms, LaunchKind::kSingle);
    if (r) return r;
    r = job_result(J, cap);
    if (r) return r;
    out.resize(J.out_count);
    hipError_t e = hipMemcpyAsync(out.data(), words, J.out_count * sizeof(uint32_t), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(GC_EDEVICE, "copy of a tuning result failed: %s", hipGetErrorString(e));
    return GC_OK;
  };
  float ms = 0.f;
  rc = run(cands[0], &ms, ref);  // warm-up, also the reference output
  ref_m = ref.size();
  // The listed candidates, then refinements of the fastest so far: a larger
  // window target, then deep-scan tiles of 512 and 256 candidates.
  const size_t nrefine = 3;
  for (size_t i = 0; rc == GC_OK && i < cands.size() + nrefine; ++i) {
    gc_tuning t;
    if (i < cands.size()) {
      t = cands[i];
    } else {
      t = *best;
      if (i == cands.size()) t.target_survivors = 1000;
      else t.deep_tile = i == cands.size() + 1 ? 512 : 256;
    }
    rc = run(t, &ms, cur);
    if (rc) break;
    if (cur.size() != ref_m || memcmp(cur.data(), ref.data(), ref_m * sizeof(uint32_t)) != 0) {
      rc = fail(GC_EDEVICE, "tuning candidate %zu built a different code", i);
      break;
    }
    if (best_i < 0 || ms < best_t) {
      best_t = ms;
      best_i = (int)i;
      *best = t;
    }
  }
  (void)hipStreamSynchronize(st);
  const hipError_t ef = hipFree(words);
  if (rc) return rc;
  if (ef != hipSuccess) return fail(GC_EDEVICE, "hipFree failed: %s", hipGetErrorString(ef));
  if (best_ms) *best_ms = best_t;
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tuned[TuneKey{dev, n, d, ordering}] = *best;
  return GC_OK;
}

void greedy_code_tune_reset(void) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tuned.clear();
}

int greedy_code_batch_tune(gc_job *jobs, int njobs, void *hip_stream, int *best_teams, float *best_ms) {
  g_error.clear();
  if (!best_teams) return fail(GC_EINVAL, "best_teams is NULL");
  *best_teams = 0;
  float best_t = 0.f;
  for (int teams = 1; teams <= kMaxTeams; teams *= 2) {
    float ms = 0.f;
    const int rc = greedy_code_batch(jobs, njobs, teams, hip_stream, &ms);
    if (rc) return rc;
    if (*best_teams == 0 || ms < best_t) {
      best_t = ms;
      *best_teams = teams;
    }
  }
  if (best_ms) *best_ms = best_t;
  return GC_OK;
}

}  // extern "C"
