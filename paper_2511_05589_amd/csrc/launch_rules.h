// The rules by which the launchers choose a kernel's shape, as plain functions of sizes: they hold
// nothing of the device, so that a host program can check them over their whole ranges.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define COPRIS_RULE __host__ __device__ __forceinline__
#else
#define COPRIS_RULE inline
#endif

namespace copris {

constexpr int kAttnWaves = 256 * 8;     // persistent wavefronts of the flat split kernel (8 per CU)

// Decode attention: slots (16-token pieces of a kv head) per wavefront, for a pool of `total` slots
// whose longest context has `longest` pieces.
//
// Large pools: an equal share of the slots.  A small pool has fewer slots than the chip has
// wavefronts, and two things pull at its share.  A wavefront's slots are a serial chain (about 1 us
// each while nothing hides them), so the shorter the share the better; but every cut makes a partial
// to merge, and beyond some hundred wavefronts more of them start no sooner.  Whole call in us,
// shares of 1 / 2 / 4:
//   16 sequences x 64 tokens,   12 / 2 heads   (128 slots)     8.8 /  9.4 / 10.3
//   16 sequences x ~40 tokens,  28 / 4 heads, skewed          11.2 / 13.4 / 18.6
//   4 sequences x 1000 tokens,  12 / 2 heads   (504 slots)    11.4 / 10.6 / 12.2
//   16 sequences x 300 tokens,  28 / 4 heads  (1216 slots)    12.3 / 11.9 / 12.1
//   128 sequences x 64 tokens,  28 / 4 heads  (2048 slots)    15.6 / 13.9 / 11.6
//   1 sequence x 3000 tokens,   28 / 4 heads   (752 slots)    13.9 / 11.6 / 11.8
//   1 sequence x 9000 tokens,   12 / 2 heads  (1126 slots)    22.2 / 15.9 / 13.9
//   8 sequences x 3000 tokens,  16 / 1 heads  (1504 slots)    21.3 / 14.8 / 13.4
//   128 sequences x 64 tokens,  8 / 8 heads   (4096 slots)       - / 13.7 / 16.0
// The last line: with one query head per kv head (group = 1) the partials are small, and merging them
// costs less than the chain of slots up to more slots.
constexpr int kAttnMinShare = 4;       // where there are slots for it; 8 is slower again (1 x 8192 tokens, 12 / 2 heads: 14.1 -> 16.0)
constexpr int kAttnShort = 64;
COPRIS_RULE int attn_small(int group) { return group == 1 ? 4096 : 1536; }
COPRIS_RULE int attn_share(int total, int longest, int group) {
  const int equal = total / kAttnWaves + (total % kAttnWaves != 0);
  if (equal >= kAttnMinShare) return equal;
  if (total > attn_small(group) || longest > 2 * kAttnShort) return kAttnMinShare;
  return total > 256 || longest > kAttnShort ? 2 : 1;
}
// Wavefronts that a pool whose block table admits `capacity` slots needs at most.
COPRIS_RULE int attn_most_waves(int64_t capacity, int group) {
  const int64_t in_fours = (capacity + kAttnMinShare - 1) / kAttnMinShare, in_twos = attn_small(group) / 2;
  if (capacity <= in_twos) return static_cast<int>(capacity);
  return static_cast<int>(in_fours > kAttnWaves ? kAttnWaves : (in_fours > in_twos ? in_fours : in_twos));
}

}  // namespace copris
