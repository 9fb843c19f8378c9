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

// LM head, 65 rows and more (sampling, or fewer given tokens than the 256 x 256 kernel takes): batch rows
// per row block.  The blocks share the rows evenly where that makes them narrower, 192 columns (or
// 128) multiplied instead of 256.  Where it does not, evenly shared rows only leave the last block's
// waves as long an epilogue as the others', so the blocks are full and the last one takes the rest.
// Whole sampling calls in us, blocks of 256 / shared evenly:
//   C = 330, H = 2048, V = 50257   130.3 / 116.8      C = 400, H = 2048, V = 50257   139.3 / 146.4
//   C = 384, H = 1024, V = 40000    66.5 /  59.6      C = 580, H = 2048, V = 12800    66.7 /  72.3
//   C = 160, H = 3584, V = 30000    68.1 /  57.2      C = 400, H = 1024, V = 32000    51.5 /  53.2
//   C = 160, H = 2048, V = 151936  169.5 / 153.3      C = 540, H = 1024, V = 40000    85.9 /  73.5
COPRIS_RULE int lm_row_blocks(int C) { return (C + 255) / 256; }
COPRIS_RULE int lm_block_rows(int C) {
  const int blocks = lm_row_blocks(C), even = ((C + blocks - 1) / blocks + 31) & ~31;
  return even <= 192 ? even : 256;
}
// Columns that a block multiplies: 128, 192 or 256.
COPRIS_RULE int lm_block_width(int C) {
  const int rows = lm_block_rows(C);
  return rows <= 128 ? 128 : (rows <= 192 ? 192 : 256);
}

// Row blocks of the tiles of 128 vocabulary rows.  Where the tiles of 256 columns are few, blocks of at most 128 rows put twice
// as many workgroups on the chip with half the products and half the sampler each; W is read once more, from the caches.
// With a CU for each of them that is faster (C = 129 .. 640, H = 64 .. 3584: 0.66 .. 0.99 of the time; blocks of
// 192 with H above 1024 lose where they had more than 192: 226 workgroups 1.04).  With more, two workgroups of a CU share it, and
// only a short H, whose sampler is what counts, gains (H <= 256 0.72 .. 0.98, to 1024 workgroups, but in place of one block of
// 192 columns 1.04 above 512, with H = 256 1.02 .. 1.06 from 470; more than 512 have a second round, which loses where there are
// three row blocks, up to 768 workgroups 1.00 .. 1.08, or five, up to 600 1.01 .. 1.03; H = 512 0.86 .. 1.22, H = 1024 1.05 .. 1.14;
// given tokens 0.97 .. 1.13).  Whole calls in us, 256 columns / 128:
//   C = 244, H =  512, V = 13430   25.1 / 17.0       C = 202, H = 3584, V =  4656   61.0 / 44.5     C = 256, H =  256, V = 28975   23.6 / 21.5
//   C = 476, H =  256, V =  8027   22.1 / 14.9       C = 277, H = 3584, V =  9125   54.0 / 42.9     C = 500, H =  256, V = 32500   33.8 / 27.9
//   C = 596, H = 1024, V =  5470   31.8 / 23.9       C = 250, H = 2048, V =  9230   36.5 / 30.3 (given tokens)
struct LmBlocks {
  int blocks, rows, width;             // row blocks, batch rows of each, columns that it multiplies
};
COPRIS_RULE LmBlocks lm_tile_blocks(int C, int H, int V, bool given) {
  const int narrow = (C - 1) / 128 + 1;
  const int64_t wgs = static_cast<int64_t>((V - 1) / 128 + 1) * narrow;
  const int64_t most = H <= 256 && !given ? (C <= 192 ? (H <= 192 ? 512 : 440) : 1024) : (C <= 192 && H > 1024 ? 192 : 256);
  const bool loses = wgs > 512 && ((narrow == 3 && wgs <= 768) || (narrow == 5 && wgs <= 640));
  if (C > 128 && C <= 640 && wgs <= most && !loses) return {narrow, ((C - 1) / narrow + 32) & ~31, 128};
  return {lm_row_blocks(C), lm_block_rows(C), lm_block_width(C)};
}

// Two row blocks of 256 workgroups each: workgroups i of both share a CU, and workgroup p takes the
// tiles p, p + 256, ...  Where at most half of the places have a tile more than the rest, the second block
// counts its places from the end (place = i ^ flip), so that no CU has two workgroups with the tile more.
// Where more have it, some CUs get two anyway, and the blocks no longer read the same rows of W at the same
// time: C = 330, H = 2048, dealt alike / from both ends: V = 33000 (2 of 256 places) 110.3 / 99.2 us,
// V = 100000 (14) 224.6 / 210.9, V = 40000 (57) 112.3 / 101.0, V = 45000 (96) 114.1 / 103.8, V = 50257 (137) 117.7 / 121.6,
// V = 151936 (163) 294.9 / 298.7, V = 65000 (252) 126.6 / 129.9.  (H = 512 and C = 400, 512 alike; given tokens with H = 256 gain nothing: 23.1
// from both ends, 22.0.)  With more row blocks other workgroups meet: C = 768, H = 1024, V = 32000 83.6 / 90.7.
COPRIS_RULE int lm_second_block_flip(int C, int n_tiles, int n_parts) {
  const int more = n_tiles % n_parts;
  return lm_row_blocks(C) == 2 && n_parts == 256 && more > 0 && more <= 128 ? 255 : 0;
}

// LM head, at most 64 rows: whether the skinny kernel (256 workgroups, an equal run of vocabulary rows
// each) is faster than the tiles of 128 vocabulary rows.  It is where its stream of W is long enough to
// hide the start and the last epilogue, which are longer than the tiles': with more than 32 rows twice as
// long.  The tiles have 512 workgroups, so one round of them up to V = 65536; beyond, their second round is
// as long as the first one.  Up to V = 32768 the tiles are at most one per CU and lose nothing to rounds.
// Time of the tiles over that of the skinny kernel (sampling; C = 32 / C = 64 where two are given):
//               V = 5003   20000   40000       50257         60001         75000        100000        151936
//   H =   64        0.88    0.88    0.91   0.91 / 0.87   0.92 / 0.89   0.93 / 0.92   0.95 / 0.93   0.94 / 0.93
//   H =  256        0.89    0.91    0.97   0.96 / 0.90   1.01 / 0.98   1.00 / 0.97   1.10 / 1.05   1.08 / 1.02
//   H =  512        0.93    0.95    1.06   1.07 / 0.97   1.07 / 0.99   1.10 / 1.03   1.15 / 1.08   1.12 / 1.05
//   H = 1024        0.95    0.97    1.15   1.12 / 1.06   1.06 / 1.03   1.15 / 1.09   1.14 / 1.16   1.09 / 1.12
//   H = 2048        1.03    1.01    1.12   1.04 / 1.03   1.00 / 1.00   1.23 / 1.22   1.28 / 1.33   1.09 / 1.12
// (up to 8 rows sampled, V = 5003, H = 1024: 1.02 .. 1.06; H = 1792: 1.10)
constexpr int kSkMaxRows = 64;
COPRIS_RULE bool lm_skinny_pays(int C, int H, int V, bool given) {
  const int64_t elements = static_cast<int64_t>(H) * V;
  if (C > kSkMaxRows) return false;
  if (V < 192 * 256) {                 // (fewer than six waves' worth of rows per workgroup)
    if (C > 32) return false;
    return H >= (V > 32768 || (C <= 8 && !given) ? 1024 : 1792);
  }
  if (C <= 32) return H >= 192 && elements >= 15000000;
  return H >= 256 && elements >= (V > 65536 ? 25000000 : 38000000);
}

// LM head, 65 rows and more: columns of the row blocks of the run kernel (one workgroup per CU, tiles of 256
// vocabulary rows, nothing beside a tile's sampler), or 0 where the tiles of 128 rows (two workgroups per CU, one's sampler
// beside the other's products) are as fast.
// 257 .. 320 rows fit one block of 320, which reads W once and multiplies no 384 or 512 columns: the run kernel, unless H
// is short for the sampler of a tile or V for its 256 workgroups; then it takes two blocks of 160, or none.
// Up to 256 rows the products are as many either way, and what decides is the rounds.  The tiles' 512 places are
// filled unevenly where V is more than half a round (32768) beyond a whole number of rounds: some CUs have two
// tiles, some one, and each takes as long as it does alone; the run kernel's tiles are then more than half full.  Where V is little beyond a
// whole round the run kernel's last tile is nearly empty instead.
// Time of the run kernel over that of the tiles (both with what they share as it is now), sampling / given tokens:
//   C = 65 .. 256    V = 33500          45000          50257          56000          60000
//   H =  768   100   0.93 0.90  0.99 0.99  1.00 0.98  1.00 1.00  1.03 1.02     192  0.95 0.91  0.97 0.95  0.98 0.98  0.95 0.98  1.04 1.05
//   H = 1024   128   0.89 0.85  0.98 0.98  1.03 1.02  1.02 1.07  1.09 1.10     192  0.89 0.86  0.94 0.90  0.99 0.92  0.98 0.99  1.02 0.98
//   H = 1280   128   0.83 0.77  0.89 0.84  0.92 0.87  0.94 0.90  0.97 0.92     230  0.88 0.84  0.92 0.88  0.94 0.91  0.94 0.91  0.96 0.93
//   H = 2048   100   0.83 0.80  0.95 0.95  0.97 0.96  1.00 0.99  1.01 1.00     256  0.87 0.86  0.89 0.90  0.91 0.90  0.91 0.93  0.92 0.94
//   H = 3584   100   0.73 0.73  0.80 0.85  0.84 0.82  0.88 0.87  0.91 0.90     256  0.82 0.82  0.85 0.89  0.87 0.87  0.87 0.89  0.90 0.89
//   V = 98305 .. 110000: H = 1536 .. 1792 0.88 .. 0.98 / 0.82 .. 0.94, but sampling with 256 rows 1.00 .. 1.05; H = 2048 0.94 .. 1.04 / 0.90 .. 1.03,
//   H >= 3072 (.. 131072) 0.80 .. 0.99 / 0.77 .. 0.98; 160 columns, H >= 3072, V = 66000 .. 151936 0.89 .. 0.98 / 0.86 .. 0.95
//   V <= 10000, sampling, 129 .. 256 rows: H = 64 1.00 .. 1.03, above 192 rows 0.88 .. 0.99; H = 256 0.91 .. 1.01; H = 512 .. 1024 0.87 .. 1.02
//   (.. 12288 0.90 .. 1.00; H = 64 .. 256 0.96 .. 1.08)
//   C = 257 .. 320   V <= 5000     10000, 15000    17000 .. 24000   28000 .. 30000   33000 .. 50257   65000          66000 .. 100000
//   H =  384         0.95 .. 0.99  1.02 .. 1.04    0.92 .. 1.04     0.97 .. 1.05     0.93 .. 1.06    1.06 .. 1.09   0.99 .. 1.08
//   H =  512         0.90 .. 0.98  0.99 .. 1.00    0.88 .. 0.98     0.95 .. 1.03     0.89 .. 1.02    1.04 .. 1.09   0.96 .. 1.05
//     given          0.95 .. 1.03  1.03 .. 1.07    0.87 .. 0.96     0.99 .. 1.05     0.93 .. 1.01    1.07 .. 1.08   0.96 .. 1.01
//   H =  768         0.94 .. 0.99  1.01 .. 1.03    0.88 .. 0.97     0.95 .. 1.01     0.92 .. 1.00    1.03           0.98 .. 1.04
//     given          0.95 .. 1.02  1.07 .. 1.09    0.84 .. 0.94     0.94 .. 1.01     0.90 .. 0.95    0.97 .. 1.00   0.91 .. 0.98
//   H = 1024         0.96 .. 0.98  0.99 .. 1.00    0.83 .. 0.90     0.94 .. 1.03     0.87 .. 0.96    0.86 .. 0.89   0.88 .. 1.03
//   H = 1536         0.99 .. 1.00  1.01 .. 1.07    0.79 .. 0.90     0.90 .. 0.96     0.79 .. 0.88    0.78 .. 0.79   0.81 .. 0.95
//   H = 3584         0.94 .. 0.99  0.98 .. 1.02    0.72 .. 0.82     0.84 .. 1.00     0.69 .. 0.80    0.71 .. 0.72   0.73 .. 0.86
//     (V = 13238 1.11: a block of 160 leaves four waves idle in a tile of at most 128 rows)
//     given          0.95 .. 1.02  1.00 .. 1.03    0.70 .. 0.79     0.82 .. 0.99     0.65 .. 0.76    0.63 .. 0.69   0.69 .. 0.82
//   (one block of 320 against two of 160, over the tiles: H = 1536, V = 33500 1.20 / 1.07, V = 90000 1.22 / 1.13, V = 20000 1.06 / 1.26)
//   C = 321 .. 512, sampling, V = 16385 .. 27000: H = 896 .. 1792 0.81 .. 1.02, H = 512 1.00 .. 1.11 at 400 rows; V = 28000 .. 30000: up to 384 rows
//   0.95 .. 1.09, more 0.91 .. 1.03; H >= 3072 0.76 .. 1.01 at every V above 16384
//   C = 577 .. 640, sampling, H >= 2048: 0.65 .. 1.01.  513 .. 576 rows are three row blocks of 192 to the tiles, whose 170 workgroups each
//   have whole rounds up to V = 21760, 43520, 87040: V = 22000 .. 32700 0.69 .. 0.87, V = 33000 .. 43500 1.00 .. 1.13, V = 20000 .. 21700 0.99 .. 1.13,
//   above 43520: H = 2048 0.91 .. 1.11 (above 87040 0.91 .. 1.03), H >= 2560 0.84 .. 0.98
COPRIS_RULE int lm_run_width(int C, int H, int V, bool given) {
  const bool long_rows = H >= 3072;
  if (C <= kSkMaxRows || C > 640 || (given && C >= 384)) return 0;
  if (C > 576) return H >= 2048 && V >= 20000 ? 320 : 0;
  if (C > 512) return H >= 2048 && ((V > 21760 && V <= 32768) || (V > 43520 && H >= 2560) || V > 87040) ? 320 : 0;
  if (C > 320) {
    const bool pays = V > 16384 && (long_rows || (H >= 896 && V <= (C <= 384 ? 27000 : 30000)));
    return !pays ? 0 : (C <= 384 ? 192 : 256);
  }
  if (C > 256) {
    if (V <= 16384) return !given && H >= 512 && V <= (H >= 2048 ? 10240 : 5000) ? 160 : 0;
    if (H < 1024) return given ? (H >= 640 ? 160 : 0) : (H >= 512 && V <= 52000 ? 160 : 0);
    return V > (H >= 2048 ? 28672 : 32768) && (H >= 1536 || V <= 65536 || V > 84000) ? 320 : 160;
  }
  const int width = C <= 128 ? 128 : (C <= 160 ? 160 : (C <= 192 ? 192 : 256));
  if (V <= 12288) return !given && C > 128 && H <= 1024 && (H >= 512 || V <= 10000) && (H >= 256 || C > 192) ? width : 0;
  bool pays = false;
  if (V > 32768 && V <= 65536) {
    const int most = long_rows ? 65536 : (H >= 1280 || C > 192 ? 60000 : (C > 128 ? 53000 : 44000));
    pays = H >= 768 && V <= most;
  }
  if (V > 98304 && V <= 131072) pays = long_rows || (H >= (given || C <= 192 ? 1536 : 2048) && V <= 110000);
  if (width == 160 && V > 65536) pays = pays || long_rows;
  return pays ? width : 0;
}

// The columns with which a call takes the run kernel, or 0.  Up to 12288 vocabulary rows it was the fastest of the above, but blocks of 128
// rows (lm_tile_blocks) and the small-call kernel (lm_small_tile) are faster: C = 207, H = 512, V = 6922 20.7 / 15.7 us; C = 305,
// H = 512, V = 4484 18.6 / 15.5; C = 210, H = 512, V = 1026 19.7 / 8.6.  Calls with H below 256 or fewer than 64 vocabulary rows have
// not been moved: the one that was measured, C = 200, H = 128, V = 8195, takes 16.6 where narrow blocks take 11.3.
COPRIS_RULE int lm_run_cols(int C, int H, int V, bool given) {
  return V <= 12288 && V >= 64 && H >= 256 ? 0 : lm_run_width(C, H, V, given);
}

// Vocabulary rows per workgroup of the run kernel: an equal share of as many workgroups as there are CUs for every row
// block, in whole Philox blocks, but at least kLmTileV: the workspace holds a partial per kLmTileV rows.
constexpr int kLmCUs = 256;
constexpr int kLmTileV = 64;
COPRIS_RULE int lm_run_rows(int C, int V, int width) {
  const int lanes = kLmCUs / ((C + width - 1) / width);
  const int rows = ((V - 1) / lanes + 4) & ~3;
  return rows < kLmTileV ? kLmTileV : rows;
}

// LM head, calls with few vocabulary rows (and fp32): vocabulary and batch rows of a workgroup of the small-call kernel,
// or no rows where another kernel takes the call.  max_parts: partials per row that the workspace has room for; whether the call
// is the small-call kernel's does not depend on it, only how far it may be cut: the fastest tile that fits (which of them it is
// does not change a result), or none if the workspace has no room for a partial per 64 rows.
//
// The other bf16 kernels give a workgroup 128 vocabulary rows and more and walk the hidden dimension slab by slab, so
// below 32768 rows most of the chip is idle while the call lasts as long as that chain.  Here the waves of a workgroup
// share the hidden dimension and the tile is as small as fills the chip.  A CU's requests are what
// bounds it, about 33 GB/s of rows, so a tile's time is its rows, and the estimate (ns) is
//     start + (rounds - 1) * end of a tile + rounds * (rows + cols) * pitch * 0.03,  at least the stream of W,
// against the other kernel's: start + H * slope, whatever V is.  (Tiles of 32 and 64 batch rows take down to 0.61 of the estimate where
// the hidden dimension is long.)  With a short H the tiles' ends decide, not their rows, and both sides have lines of their own:
// without them C = 76, H = 64, V = 18900 given tokens 11.5 (9.0 with tiles of 128 rows), C = 150, H = 64, V = 18500 given 14.8 / 10.6,
// C = 96, H = 64, V = 22500 14.8 / 11.9, C = 64, H = 128, V = 22500 given 11.2 / 9.5.  Whole calls in us, other kernel / small-call
// kernel with its tile (sampling):
//   C =   1, H = 3584, V =  3483   34.8 / 10.3 (16 x 16)      C =  41, H = 3584, V =  3251   40.0 / 12.7 (32 x 32)
//   C =   2, H =  256, V = 16384   12.6 /  7.2 (64 x 16)      C =  63, H = 1024, V =  3554   19.3 /  9.1 (32 x 32)
//   C =   8, H = 2048, V =  7732   25.5 / 11.8 (32 x 16)      C =  69, H =  512, V =  1885   14.7 /  7.1 (32 x 32)
//   C =  18, H = 2048, V = 13619   26.5 / 16.8 (64 x 32)      C = 126, H = 3584, V =  2572   42.7 / 15.6 (64 x 32)
//   C =  25, H = 1024, V = 24622   19.0 / 20.2, not taken     C = 192, H = 3584, V =  4804   51.1 / 23.2 (64 x 64)
//   C = 125, H = 1024, V = 10419   20.6 / 23.8, not taken     C = 387, H =  512, V =  1515   24.0 / 10.5 (64 x 64)
//   given tokens: C = 1, H = 1536, V = 3405  19.7 / 7.4;  C = 29, H = 2048, V = 6569  24.0 / 11.2;  C = 126, H = 3584, V = 6545  40.8 / 22.9
// 674 drawn calls (C = 1 .. 512, H = 64 .. 3584, V = 1000 .. 32768): at most 1.00 of the time without this kernel and the narrow blocks, 0.31 at
// best; some keep the other kernel where this one was 10 - 25 % faster.  A second round of 64 x 64 tiles is slower than the first (C = 334, H = 2048, V = 5313
// 55.7 for two, 32.7 with tiles of 128 rows), so it is priced higher.  Where the run kernel's rule takes the call it keeps it.
// fp32 against the kernel with four quarters of the hidden dimension and tiles of 64 rows: C = 8, H = 256, V = 1024 9.4 / 7.1;
// C = 4, H = 1024, V = 2994 17.0 / 9.3; C = 62, H = 3584, V = 1945 82.7 / 19.2; C = 22, H = 512, V = 109750 82.4 / 67.1; at most 1.00 of the time
// over 120 drawn calls, but with at most 8 rows and more than 32768 vocabulary rows, where that one is bound by its stream
// of W, 0.98 .. 1.06.
struct LmSmall {
  int rows, cols;
};
// Places for partials in a row of the workspace: whole 64 vocabulary rows, so that a lane of the merge loads those of 64 rows at once.
COPRIS_RULE int64_t lm_small_parts(int V, int rows) { return static_cast<int64_t>((V - 1) / kLmTileV + 1) * (kLmTileV / rows); }
constexpr int kSmMaxRows = 512;        // more batch rows: never
constexpr int kSmMaxGiven = 383;       // ... of given tokens in bf16
constexpr int kSmMaxV = 32768;         // more vocabulary rows: not in bf16
COPRIS_RULE LmSmall lm_small_tile(int C, int H, int V, bool given, bool f32, int64_t max_parts) {
  LmSmall best = {0, 0};
  if (C > kSmMaxRows || (V > kSmMaxV && (!f32 || C <= 8)) || max_parts < lm_small_parts(V, kLmTileV)) return best;
  if (!f32 && ((given && C > kSmMaxGiven) || lm_run_cols(C, H, V, given) != 0)) return best;
  const int64_t pitch = static_cast<int64_t>(H) * (f32 ? 4 : 2);
  const int64_t stream = 6000 + V * pitch / 5200;
  int64_t least = INT64_MAX;           // the other kernel
  if (!f32) {
    if (C <= 32) least = 10500 + 65 * static_cast<int64_t>(H) / 10;
    else if (C <= 64) least = 12000 + 75 * static_cast<int64_t>(H) / 10;
    else if (C <= 128) least = 11500 + 85 * static_cast<int64_t>(H) / 10;
    else if (C <= 256) least = 15200 + 137 * static_cast<int64_t>(H) / 10;
    else if (C <= 384) least = 14500 + 105 * static_cast<int64_t>(H) / 10;
    else least = 18000 + 126 * static_cast<int64_t>(H) / 10;
    if (given) least = least * 85 / 100;
    // (the lines above are for a long H; a short one takes)
    const int64_t h = H, brief = C <= 32 ? 9200 + 21 * h / 2 : (C <= 64 ? 11200 + 23 * h / 2 : 11200 + 9 * h);
    if (C <= 128 && brief - (given ? (C <= 32 ? 2000 : 3000) : 0) < least) least = brief - (given ? (C <= 32 ? 2000 : 3000) : 0);
    if (C > 128 && given && 9600 + 9 * h < least) least = 9600 + 9 * h;
    const LmBlocks tiles = lm_tile_blocks(C, H, V, given);
    if (C > 128 && tiles.width == 128) {
      least = 10800 + 9 * static_cast<int64_t>(H) - (given ? 2800 : 0);
      if (((V - 1) / 128 + 1) * tiles.blocks > 256) least = least * 5 / 4;
    }
  }
  int64_t fewest = 0;                  // workgroups of the best tile; of two as fast the one with fewer of them
  LmSmall fits = {0, 0};
  int64_t least_fits = INT64_MAX;
  for (int rows = 16; rows <= 64; rows *= 2)
    for (int cols = 16; cols <= 64; cols *= 2) {
      if ((cols > 16 && cols / 2 >= C) || (rows == 16 && cols == 64)) continue;
      const int64_t tiles = (V - 1) / rows + 1, col_blocks = (C - 1) / cols + 1, wgs = tiles * col_blocks;
      const bool alone = rows == 64 && cols == 64;                         // on its CU
      const int64_t rounds = (wgs + 255) / 256;
      if (rounds > (1 << 13)) continue;                                    // (a grid has fewer than 2^32 threads)
      int64_t cost = (alone ? 6400 : 5200) + (rounds - 1) * (alone ? 5000 : 1100) + rounds * (rows + cols) * pitch * (alone && rounds > 1 ? 4 : 3) / 100;
      if (cost < stream) cost = stream;
      // With a short H more tiles than CUs cost what their ends do, on one CU side by side; a tile that has its CU alone waits where an
      // XCD has more than its 32 CUs' (84 tiles in 3 column blocks are 252 workgroups, 33 of them on four XCDs).
      int64_t ends = (given ? 5200 : 6000) + 1600 * rounds;
      if (alone) ends = (given ? 7200 : 8000) + ((tiles + 7) / 8 * col_blocks > 32 * rounds ? 2500 : 0);
      ends += 6 * static_cast<int64_t>(H);
      if (!f32 && (alone || rounds > (cols == 16 ? 2 : 1)) && cost < ends) cost = ends;
      if (cost < least || (cost == least && wgs < fewest)) {
        least = cost;
        fewest = wgs;
        best = {rows, cols};
      }
      if (lm_small_parts(V, rows) <= max_parts && cost <= least_fits) {    // (at the same cost the one with fewer partials)
        least_fits = cost;
        fits = {rows, cols};
      }
    }
  return best.rows == 0 || lm_small_parts(V, best.rows) <= max_parts ? best : fits;
}
// Most places for partials, rows x partials of each, that calls with up to M rows of given tokens have where they are the small-call
// kernel's.  Its tile is the same for the rows 16 i + 1 .. 16 i + 16 (test_most_partials_of_small_calls).
COPRIS_RULE int64_t lm_small_most_parts(int M, int H, int V, bool f32) {
  int64_t most = 0;
  if (V > kSmMaxV && !f32) return most;
  const int rows = f32 ? kSmMaxRows : kSmMaxGiven;
  for (int m = M < rows ? M : rows; m > 0; m = (m - 1) & ~15) {
    const LmSmall t = lm_small_tile(m, H, V, true, f32, INT64_MAX);
    const int64_t parts = t.rows != 0 ? m * lm_small_parts(V, t.rows) : 0;
    if (parts > most) most = parts;
  }
  return most;
}

// LM head, 384 given tokens and more: the 256 x 256 kernel's row blocks and lanes, one workgroup per CU.  A last row
// block that is not full costs as much as a full one, so it takes another width from the run kernel where that
// is faster: 128 or 160 columns, or 320 in place of a full block and up to 64 rows more.  (192 columns: M = 448 0.97 .. 1.10,
// M = 690 0.98 .. 1.03; not taken.)  The last block's lanes are then as many as make it finish with the others, by the
// time of a whole tile relative to one of 256 columns: 0.6, 0.65 and 1.25, where the mixtures were fastest among
// weights in steps of 0.1; a run of r rows takes its whole tiles and a part of one for the rest.
// The estimate leaves out the start of a lane and the end of its tiles, so it is not enough by itself (time of the mixture
// over that of full blocks only; M = 390 .. 8200, H = 64 .. 3584, V = 5003 .. 151936):
//   lanes of one tile, before                             0.91 .. 1.17
//   of two, and still two                                 0.92 .. 1.19; one then 0.71 .. 1.01, but 160 columns with H = 64 1.05
//   more, 128 or 160 columns, estimated gain 3 % and more 0.77 .. 1.03
//   more, 320 columns: H = 64 1.09 .. 1.49, H = 256 0.94 .. 1.25; H = 512 from 16 % on 0.90 .. 1.00, else 0.93 .. 1.13;
//     H = 768 and 1024 from 7 % on 0.87 .. 1.02, else 0.97 .. 1.04, but with three or four tiles that become fewer 0.84 .. 0.99;
//     H >= 2048 0.77 .. 1.02
// (900 drawn calls of M = 385 .. 4250: at most 1.05, 1.00 in the middle.)
// Full blocks only / mixed, in us: M = 777, H = 2048, V = 151936 543 / 459, H = 3584, V = 20011 139 / 113; M = 390, H = 3584, V = 100000
// 358 / 288; M = 600, H = 256, V = 75000 43.7 / 38.7; M = 1600, H = 2048, V = 20011 136 / 124; M = 2100, H = 3584, V = 151936 2037 / 1926.
struct LmGivenPlan {
  int full, lanes, lane_units;         // row blocks of 256, lanes of each, 64-row blocks of the vocabulary per lane
  int width, rest_lanes, rest_rows;    // columns of the last block (0: there is none), its lanes and vocabulary rows per lane
};
// Thousandths of a whole tile's time at 256 x 256 columns.
COPRIS_RULE int64_t lm_full_cost(int units) {
  const int left = units % 4;
  return units / 4 * INT64_C(1000) + (left == 0 ? 0 : (left == 3 ? 800 : 650));
}
COPRIS_RULE int64_t lm_rest_cost(int rows, int width) {
  const int64_t whole = width == 128 ? 600 : (width == 160 ? 650 : 1250);
  const int left = rows % 256;
  return rows / 256 * whole + (left == 0 ? 0 : (width == 128 && left <= 128 ? whole * 7 / 10 : whole));
}
COPRIS_RULE LmGivenPlan lm_given_plan(int M, int H, int V) {
  const int blocks = (M - 1) / 256 + 1, units = (V - 1) / 64 + 1, last = M - (blocks - 1) * 256;
  LmGivenPlan p = {blocks, 1, 0, 0, 0, 0};
  const int even = kLmCUs / blocks < 1 ? 1 : kLmCUs / blocks;
  p.lane_units = (units + even - 1) / even;
  p.lanes = (units - 1) / p.lane_units + 1;
  if (last > 160 || blocks > 64) return p;
  const int width = last <= 64 ? 320 : (last <= 128 ? 128 : 160);
  const int full = width == 320 ? blocks - 2 : blocks - 1;
  LmGivenPlan mixed = p;
  int64_t best = lm_full_cost(p.lane_units);
  for (int lanes = even; lanes * full < kLmCUs; ++lanes) {
    const int lane_units = (units + lanes - 1) / lanes, used = (units - 1) / lane_units + 1;
    const int left = kLmCUs - full * used;
    int rows = ((V - 1) / left + 4) & ~3;
    if (rows < kLmTileV) rows = kLmTileV;
    const int64_t a = lm_full_cost(lane_units), b = lm_rest_cost(rows, width), cost = a > b ? a : b;
    if (cost < best) {
      best = cost;
      mixed = {full, used, lane_units, width, (V - 1) / rows + 1, rows};
    }
  }
  const bool fewer_tiles = (mixed.lane_units + 3) / 4 < (p.lane_units + 3) / 4;
  if (p.lane_units <= 8 && (!fewer_tiles || (width == 160 && H < 256))) return p;
  int percent = 97;
  if (width == 320) percent = H < 512 ? 0 : (H < 768 ? 84 : (H >= 2048 || (H >= 1024 && fewer_tiles && p.lane_units <= 16) ? 97 : 93));
  return 100 * best < percent * lm_full_cost(p.lane_units) ? mixed : p;
}

// Re-prefill attention: what is known of the sequences is their number B, their tokens T and a bound of their lengths.
// Tokens of the longest chain of steps: the bound, if it can be a length (bound <= T, or one sequence); a looser one says
// nothing, and the longest is at least T / B long.
COPRIS_RULE int64_t prefill_chain(int B, int64_t T, int max_seqlen) {
  return max_seqlen <= T ? max_seqlen : (B == 1 ? T : T / B);
}
// n / d as n * ceil(2^32 / d) / 2^32: exact for n * d < 2^32 (the product exceeds n / d by less than n * d / 2^32 / d).
struct Divisor {
  uint32_t d;
  uint64_t inverse;
  COPRIS_RULE uint32_t divide(uint32_t n) const { return static_cast<uint32_t>((n * inverse) >> 32); }
};
COPRIS_RULE Divisor divisor(uint32_t d) { return {d, ((UINT64_C(1) << 32) + d - 1) / d}; }
// The flat grid of a call: workgroups of per_wg units that the sequences can need, a list for each residue of the kv heads
// modulo 2^part_shift and its XCDs in turn.  0: the sequences are too many to be searched by every workgroup, or the
// workgroups for one dimension of a grid.
constexpr int kXcdShift = 3, kXcds = 1 << kXcdShift;
COPRIS_RULE int xcd_part_shift(int Hkv) { return Hkv % 8 == 0 ? 3 : (Hkv % 4 == 0 ? 2 : (Hkv % 2 == 0 ? 1 : 0)); }
COPRIS_RULE int64_t prefill_flat_grid(int B, int64_t T, int Hkv, int group, int64_t wgs_max, int tile, int per_wg) {
  const int shift = xcd_part_shift(Hkv);
  // a sequence of n tokens has ceil(n / tile) tiles and ceil(tiles * group / per_wg) workgroups per kv head
  const int64_t bound = wgs_max * B, exist = ((T / tile + B) * group) / per_wg + B;
  const int64_t list = (exist < bound ? exist : bound) * (Hkv >> shift);
  const int lanes = kXcds >> shift;
  const int64_t wgs = (list + lanes - 1) / lanes * kXcds;
  return B <= 256 && wgs < (INT64_C(1) << 22) && Hkv <= 512 ? wgs : 0;
}
struct PrefillGrid {
  int flat, B, part_shift;
  Divisor group, heads;            // query heads per kv head; kv heads of a residue
};
COPRIS_RULE PrefillGrid prefill_grid(int B, int Hkv, int group, bool flat) {
  const int shift = flat ? xcd_part_shift(Hkv) : 0;
  return {flat, B, shift, divisor(static_cast<uint32_t>(group)), divisor(static_cast<uint32_t>(Hkv >> shift))};
}
// Workgroup shapes: four units of 32 queries or of 16 (two workgroups per CU), or two groups of waves on two or four units
// of 16, which have a CU to themselves and half the chain.  The shape is the one with the smallest estimate
//     start + max(chain * step, workgroups / 256 * (steps of a workgroup * load + each)),
// and a quarter of a chain where workgroups that have a CU to themselves are more than there are CUs;
// the steps of a workgroup being half of what lies between the mean length and the longest.  The constants (ns) are fitted to
// 400 drawn calls (1 .. 40 sequences of 1 .. 8192 tokens, ten head counts) in all shapes, with an error of 12 .. 15 %, and moved
// to where the choice loses least: it took 1.011 times the time of the best on average, 1.31 at most.  (That was with one softmax state
// per wave.)  Whole call in us, whole / half / 2 x 2 / 2 x 4, with the states that prefill_sums asks for where the shape can hold them:
//   32 tokens, 12 / 2 heads                            7.9 /  5.9 /  5.5 /  6.7
//   512 tokens, 12 / 2 heads                          15.7 / 12.0 / 10.0 / 12.0
//   356 + 942 tokens, 12 / 2 heads                    23.2 / 17.7 / 19.0 / 16.5
//   3 x 600 tokens, 8 / 8 heads                       18.5 / 14.9 / 19.2 / 14.9
//   2000 tokens, 12 / 2 heads                         39.7 / 31.1 / 36.4 / 26.4
//   1000 tokens, 28 / 4 heads                         24.4 / 20.2 / 30.7 / 22.1
//   4 x 100 tokens, 28 / 4 heads                       9.4 /  7.8 / 10.7 /  8.6
//   2000 + 500 + 300 tokens, 16 / 4 heads             42.7 / 34.3 / 56.6 / 40.3
//   2 x 3000 tokens, 8 / 8 heads                      63.6 / 55.9 / 86.4 / 62.2
//   3 x 900 tokens, 28 / 4 heads                      33.4 / 34.8 / 73.1 / 50.0
//   24 x 300 tokens, 28 / 4 heads                     50.2 / 56.1 / 133  / 93.9
// (A group of four units of 32 queries more, 2 x 4 x 32, was best in 4 of the 400 calls, by 5 % in the middle; not taken.)
enum PrefillShape { kPrefillWhole, kPrefillHalf, kPrefill2x2, kPrefill2x4 };
struct PrefillCost {
  int queries, units, groups;          // of a unit; of a workgroup; of a unit
  int start, step, load, each;
};
constexpr PrefillCost kPrefillCost[4] = {{32, 4, 1, 6600, 690, 450, 5200}, {16, 4, 1, 4850, 440, 290, 3200},
                                         {16, 2, 2, 5050, 260, 220, 2900}, {16, 4, 2, 6300, 240, 290, 4300}};
COPRIS_RULE PrefillShape prefill_shape(int B, int64_t T, int Hq, int max_seqlen) {
  const int64_t chain_tok = prefill_chain(B, T, max_seqlen), chain = (chain_tok + 31) / 32;
  const int64_t twice_steps = (T / B * 11 + chain_tok * 9) / 640 + 1;      // twice the mean steps of a workgroup
  PrefillShape best = kPrefillWhole;
  if ((T / 32 + B) * Hq > (1 << 20)) return best;                          // (and no product below overflows)
  int64_t least = INT64_MAX;
  for (int s = 0; s < 4; ++s) {
    const PrefillCost c = kPrefillCost[s];
    const int64_t wgs = (T / c.queries * 2 + B) * Hq / (2 * c.units);      // (half a tile more per sequence)
    const int64_t long_chain = chain * c.step, all = wgs * (c.load * twice_steps / 2 + c.each) / 256;
    const int64_t second = c.groups == 2 && wgs > 256 ? long_chain / 4 : 0;
    const int64_t cost = c.start + (long_chain > all ? long_chain : all) + second;
    if (cost < least) {
      least = cost;
      best = static_cast<PrefillShape>(s);
    }
  }
  return best;
}

// Sums that the keys of a query are shared out to, step i to sum i % sums, each with a softmax reference of its own: 4, 2 or 1.
// The weights are rounded to bf16 against their sum's reference, so the sums decide the result, and more of them, whose references lie
// nearer to their weights, are more exact (1e-3 of the result, its own rounding being 1.6; 1 / 2 / 4 sums):
//   100 tokens 1.89 / 1.85 / 1.84     300 2.00 / 1.96 / 1.92     900 2.08 / 2.03 / 1.99     2500 2.10 / 2.07 / 2.03
// They do not follow the workgroup's shape, which is chosen for its time: a shape with fewer groups of waves than sums keeps several
// per wave (prefill_plan), one with more has as many as groups.  The lines are where two and four groups of waves paid when each had a CU's
// whole chain to itself; moving them changes results.
COPRIS_RULE int prefill_sums(int B, int64_t T, int Hq, int group, int max_seqlen) {
  const int64_t units = (T / 32 + B) * Hq;
  const int64_t launched = ((static_cast<int64_t>(max_seqlen) + 31) / 32) * B * Hq;
  const int64_t steps = (prefill_chain(B, T, max_seqlen) + 31) / 32;
  if (launched - units > (B == 1 ? 250 : 100) * steps) return 1;
  if (units <= 256 && launched <= 512) return 4;
  if (units <= 512 && (launched <= 600 || 5 * launched <= 8 * units)) return steps > (group == 1 ? 18 : 24) ? 4 : 2;
  return units <= 2048 && units <= (units <= 1728 ? 36 : 24) * steps ? 2 : 1;
}

// The shape of prefill_shape, unless its waves cannot hold the sums: two states of 32 queries do not fit a wave's registers, nor do
// four of 16 (one sequence of 151 tokens, 32 / 4 heads: 9.4 us with spills, 8.0 as 2 x 2).  A second state costs up to 0.8 us (two
// sequences of 942 + 356 tokens, 12 / 2 heads: 15.7 / 16.5 us; 172 + 115, 16 / 4: 7.7 / 8.0).
struct PrefillPlan {
  PrefillShape shape;
  int sums;                            // of a wave
};
COPRIS_RULE PrefillPlan prefill_plan(int B, int64_t T, int Hq, int group, int max_seqlen) {
  const int64_t most_steps = ((max_seqlen < T ? max_seqlen : T) + 31) / 32;
  int sums = prefill_sums(B, T, Hq, group, max_seqlen);
  while (sums > 1 && sums / 2 >= most_steps) sums /= 2;                    // (the others would stay empty)
  PrefillShape shape = prefill_shape(B, T, Hq, max_seqlen);
  if (shape == kPrefillWhole && sums > 1) shape = kPrefillHalf;
  if (shape == kPrefillHalf && sums > 2) shape = kPrefill2x2;
  const int groups = kPrefillCost[shape].groups;
  return {shape, sums > groups ? sums / groups : 1};
}

}  // namespace copris
