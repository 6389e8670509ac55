// cover.h -- storage of the cover builder (cover_build.h): graded codes from
// a bitmap of the whole space.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gcimpl {

constexpr int kCovTeam = 32;             // workgroups (slices of the space), at most
constexpr int kCovWords = 8192;          // 64-bit words of a slice, at most
constexpr int kCovMaxN = 24;             // 2^24 bits: 32 slices of 8192 words
constexpr int kCovMaxD = 4;              // by rounds; larger distances by windows
constexpr unsigned int kCovSeg = 4096;   // words a slice accepts in one round, at most
constexpr unsigned int kCovOwn = 512;
constexpr int kCovShared = 12;           // words a wave tests together with 16 lanes each, at most
constexpr unsigned int kCovMaxRounds = 1u << 19;
constexpr int kCovDiffs = 384;           // word-index differences of weight <= 3 in 13 bits: 378
constexpr int kCovWin = 1024;            // candidates of a window, at most (one a thread)
constexpr int kCovBlocks = kCovWin / 64;
constexpr int kCovLevels = 8;            // levels listed at once, at most

struct CoverLds {
  unsigned long long dead[kCovWords + 1];  // the slice: 1 = accepted, rejected or no candidate; then a word of ones
  unsigned long long level[64];          // [32 + j]: the bits of a word whose index has weight j
  unsigned int wsum[32];
  unsigned int epoch;                    // workgroups that have passed the team's barriers
  union {
    struct {                             // distance at most 4: rounds
      unsigned long long acc[kCovWords]; // accepted in the current level
      uint16_t queue[kCovWords];         // words with undecided candidates of the level
      uint16_t diff[kCovDiffs];          // word-index differences, by weight
      unsigned int cum[kCovMaxD + 1];    // differences of weight below j
      uint8_t other[kCovTeam];           // differences of slice numbers, by weight
      unsigned long long ball[kCovMaxD][64];  // ball[r][b]: bit indices within distance r of b
      unsigned int cnt[kCovTeam];        // per slice: words it accepted in the last round
      unsigned int total[kCovTeam];      // per slice: words it accepted in the level
      uint32_t own[kCovOwn];             // the first words this slice accepted in the round
      unsigned int qn, segn, seg_ok, left, accn, open;
    };
    struct {                             // larger distances: windows
      uint16_t wdiff[kCovWords];         // word-index differences, by weight
      unsigned int wcum[15];             // differences of weight below j
      unsigned long long wball[8][64];   // as ball, radius -1 (none) .. 6 (every bit)
      alignas(16) uint32_t cand[kCovWin];  // the window's candidates, in walk order
      alignas(16) uint32_t took[kCovWin];  // those accepted
      alignas(16) uint32_t block[2][64];   // those of a block of 64 candidates, up to a multiple of eight
      unsigned int taken[kCovBlocks];      // how many of each block
      uint2 run[kCovLevels * kCovTeam];    // per (level, slice): place in the window, place in its list
      unsigned long long none[32];         // [v]: bits that are no candidates in words of index weight v
      uint2 sums[32];                      // per wave: candidates of four levels, 16 bits each
      uint32_t basis[32], pick;          // self-orthogonal: a basis of the code's span
      int dim;
      unsigned int size, done_levels, listed;  // the window's candidates; levels it takes whole, and at all
    };
  };
};

// Global memory of a cover team: every exchange is within one XCD (one L2).
struct CoverWs {
  union {
    unsigned long long active[(1u << (kCovMaxN - 6)) + 32];  // undecided candidates of the level; then zeros
    struct {                                                 // windows
      uint32_t list[2][kCovTeam][kCovWin];                   // candidates a slice lists
      unsigned int head[2][kCovTeam][16];                    // levels listed, cut short?, candidates of each level
    };
  };
  uint32_t seg[2][kCovTeam][kCovSeg];                    // words accepted in a round, by slice
  unsigned long long slot[2][kCovTeam];                  // what a slice reports at a barrier
  unsigned int arrived;                                  // barrier: arrivals so far
  unsigned int pad[63];
};

// Join state of the team of a launch of its own.
struct CoverCtl {
  unsigned int xcd;       // 1 + the team's XCD; 0: none yet
  unsigned int members;   // workgroups that joined, and whether the team is closed
  unsigned int size;      // members when it was closed
  unsigned int left;      // workgroups of the launch that are done
  unsigned int built;     // 1 the code is built, 2 the team is too small
  int abort;
  unsigned int pad[58];
};

}  // namespace gcimpl
