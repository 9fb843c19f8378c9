// Re-prefill of resumed partial trajectories: causal attention over packed
// variable-length sequences, filling the sequences' KV pages on the way
// (Section 4, "Prioritized Resumption": buffered partial trajectories are continued in the
// next rollout stage; Section 5.3 names their re-prefilling as a cost of high concurrency).
//
// bf16, head_dim 128, page 16.  The unit of work is (query head, tile of query tokens): one wave, the tile as NB blocks
// of 16 queries (NB = 2, or 1 in calls that leave wave slots idle).  The units of a (sequence, kv head) are numbered
// tile-major (unit u = tile u / g, head u % g of the kv head's g query heads); a workgroup is four consecutive ones (or two),
// so its waves need the same K/V rows: the workgroup walks the sequence's K/V once, in 32-token steps (two pages), up to
// the last of its tiles, and a wave whose own tile is over only keeps fetching.  Late units first.
// A step's K and V rows (8 KB each) are fetched once by all waves together with LDS-direct loads into rings of four
// buffers (the XOR swizzle is applied by choosing which global granule a lane fetches) and read by every wave in operand
// layout.  Per block of 16 queries:
//     S^T[token][query] = K[token][:] . Q[query][:]           2 x 4 x mfma 16x16x32 (16 tokens each)
//     O^T[d][query]    += V^T[d][token] . P^T[token][query]   8 x mfma 16x16x32 (all 32 tokens)
// The value product's k-slot (g, e) is token 4g+e of the first page for e < 4 and token 4g+e-4 of the second page for
// e >= 4, which is exactly how the two score tiles leave the weights in a lane and how the transposing LDS read delivers
// V - both operands are two register pairs put side by side, nothing moves between lanes.  Max / sum / rescale of a query
// live in the lane that owns it.  Only the last step needs the causal mask.
//
// What bounds it.  A product takes 16 clocks of the matrix pipe and a vector instruction 4 of the vector pipe, an
// exponential 12 (two waves per SIMD, csrc/chip_rates.hip); a wave alone issues a vector instruction every 8.  Per wave
// and step of 32 queries that is 512 clocks of products and about 600 of vector issue, so the two have to run beside each
// other.  Therefore a wave multiplies the scores of its next step while it forms the weights of this one (one product, one
// exponential at a time), and reads its next K operands and requests rows while it multiplies the values; the steps are
// unrolled over the ring, so that operand addresses are immediates; the other workgroup of the CU fills what is left.
// 16 sequences of 513 .. 16897 tokens, 28 / 4 heads: 2690 us with the score, softmax and value parts one after the other
// and a grid per sequence, 2440 with parts, rings and grid as they are here, which came in one step and were not timed apart
// (1.16 PFLOP/s, 1390 W of the board's 1400 at 1.9 GHz; 2314 and 1990 on zeros, where power is no limit).
//
// Where a workgroup works.  The grid is flat over the workgroups that the lengths need, and the kv heads are dealt to the
// XCDs (Place): 8 / 8 heads, 40 x 2048 tokens 661 -> 474 us, whose rows every XCD pulled through its own L2 before;
// 30 x 60 tokens with a bound of 4096 45 -> 9.2, most of whose workgroups had nothing to do.
//
// LDS reads are inline instructions with explicit waits: the compiler cannot tell which
// LDS-direct load fills which buffer and would wait for all of them before any LDS read.
#include <type_traits>

#include "copris_device.h"
#include "copris_internal.h"

namespace copris {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kD = 128;
constexpr int kP = 16;
constexpr int kPageGranules = kP * kD * 2 / 16;   // 256 16-byte granules of K (and of V) per page
constexpr int kSubs = 2;                          // pages per step
constexpr int kStepTok = kSubs * kP;              // 32 tokens per step (a tile's own tokens lie in one step)
constexpr int kStepGranules = kSubs * kPageGranules;   // 512 granules of K (and of V) per step
constexpr int kHalfBytes = kStepGranules * 16;    // 8 KB: a step's K rows (or V rows)
constexpr int kRing = 4;                          // ring buffers of K rows, and of V rows, per group
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kSlack = 6.0f;   // scores may exceed the softmax reference by 2^kSlack
constexpr float kBig = 64.0f;    // = 2^kSlack

// A workgroup is GROUPS groups of UNITS waves, one unit (query head, tile of 16 * NB query tokens) per wave of a group; a wave
// keeps SUMS softmax states, step i of its group in state i % SUMS.
template <int GROUPS, int UNITS, int NB, int SUMS> struct Shape {
  static constexpr int kTileQ = 16 * NB;
  static constexpr int kUnits = UNITS;
  static constexpr int kThreads = 64 * GROUPS * UNITS;
  static constexpr int kRows = kStepTok / kUnits;          // K and V rows of a step that a wave fetches
  static constexpr int kGroupLds = 2 * kRing * kHalfBytes;
  static constexpr int kState = NB * (8 * 64 * 16 + 64 * 8); // bytes of a softmax state of a wave: O, then (m, l)
  static constexpr int kRings = GROUPS * kGroupLds, kStates = GROUPS == 1 ? 0 : GROUPS * UNITS * SUMS * kState;
  static constexpr int kLds = kRings > kStates ? kRings : kStates;   // 64 KB (two workgroups per CU); two groups: 128 KB, or 136
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  uint32_t r;
  asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(lo), "v"(hi));
  return r;
}

// LDS position (in 16-byte granules) of granule c of token row `row` of a page (conflict-free
// for the row-wise fills and for both operand read patterns).
__device__ __forceinline__ int swz_k(int row, int c) { return row * 16 + (c ^ (row & 15)); }
__device__ __forceinline__ int swz_v(int row, int c) { return row * 16 + (c ^ ((row & 7) << 1)); }

template <int OFF>
__device__ __forceinline__ u32x4 lds_read128(uint32_t addr) {
  u32x4 x;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(x) : "v"(addr), "n"(OFF) : "memory");
  return x;
}
// the transposing read: four 16-bit elements of four rows, delivered in MFMA operand order
template <int OFF>
__device__ __forceinline__ s16x4 lds_read_tr16(uint32_t addr) {
  s16x4 x;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(x) : "v"(addr), "n"(OFF) : "memory");
  return x;
}

// A buffer of `bytes` bytes: loads past its end give zeros and reach no memory.  (The descriptor's type and its
// builtins exist in the device compilation only.)
#if defined(__HIP_DEVICE_COMPILE__)
typedef __amdgpu_buffer_rsrc_t BufferRsrc;
#else
typedef int BufferRsrc;
#endif
__device__ __forceinline__ BufferRsrc buffer_rsrc(const void* p, uint32_t bytes) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
#else
  (void)p; (void)bytes;
  return 0;
#endif
}
// 16 bytes per lane from `offset` to dst + 16 * lane in LDS
__device__ __forceinline__ void buffer_load_lds16(BufferRsrc rsrc, char* dst, uint32_t offset) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst, 16, offset, 0, 0, 0);
#else
  (void)rsrc; (void)dst; (void)offset;
#endif
}

template <int N>
__device__ __forceinline__ void wait_loads() {   // at most N of this wave's loads may still be in flight
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// What a workgroup works on: the units first .. first + UNITS of sequence b (tokens s0 .. s0 + len) and kv head kvh.
// first < 0: nothing.
struct Place {
  int b, kvh, first, s0, len;
};
// Workgroups that a sequence of len tokens needs per kv head
template <class S>
__device__ __forceinline__ int workgroups_of(int len, const PrefillGrid& pg) {
  return ((max(len, 0) + S::kTileQ - 1) / S::kTileQ * pg.group.d + S::kUnits - 1) / S::kUnits;
}
// A grid of (workgroups of the longest sequence, kv heads, sequences); the last units of a sequence (the long chains) first.
template <class S>
__device__ __forceinline__ Place place_grid(const int32_t* __restrict__ cu_seqlens, const PrefillGrid& pg) {
  Place p;
  p.b = blockIdx.z;
  p.kvh = blockIdx.y;
  p.s0 = cu_seqlens[p.b];
  p.len = cu_seqlens[p.b + 1] - p.s0;
  p.first = (workgroups_of<S>(p.len, pg) - 1 - static_cast<int>(blockIdx.x)) * S::kUnits;
  return p;
}
// A flat grid over the workgroups that the sequences need, sequence after sequence.  Workgroups go to the XCDs in turn, so
// the kv heads are dealt to the XCDs: an XCD's L2 serves 1 / gcd(Hkv, 8) of them, and the workgroups that walk the same rows
// at the same time share it.  The sequence is found from the lanes' lengths: one per lane, or four in larger batches.
template <class S>
__device__ __forceinline__ Place place_flat(const int32_t* __restrict__ cu_seqlens, const PrefillGrid& pg) {
  const int lane = threadIdx.x & (kWave - 1);
  const int x = static_cast<int>(blockIdx.x) & (kXcds - 1);
  // place in the list of the kv heads of this XCD's residue, and in that of one of them
  const uint32_t j = ((blockIdx.x / kXcds) << (kXcdShift - pg.part_shift)) + static_cast<uint32_t>(x >> pg.part_shift);
  const uint32_t q = pg.heads.divide(j);
  Place p;
  p.kvh = (x & ((1 << pg.part_shift) - 1)) + static_cast<int>((j - q * pg.heads.d) << pg.part_shift);
  p.b = p.s0 = p.len = 0;
  p.first = -1;
  int left = static_cast<int>(q);
  if (pg.B <= kWave) {
    const int i = min(lane, pg.B - 1);
    const int s0 = cu_seqlens[i], len = cu_seqlens[i + 1] - s0;
    const int n = lane < pg.B ? workgroups_of<S>(len, pg) : 0;
    const int upto = wave_prefix_sum(n);
    const uint64_t beyond = __builtin_amdgcn_ballot_w64(upto > left);
    if (beyond != 0) {
      const int l = __builtin_ctzll(beyond);
      p.b = l;
      p.first = (__builtin_amdgcn_readlane(upto, l) - 1 - left) * S::kUnits;
      p.s0 = __builtin_amdgcn_readlane(s0, l);
      p.len = __builtin_amdgcn_readlane(len, l);
    }
  } else {
    int at[5], n[4];
#pragma unroll
    for (int e = 0; e < 5; ++e) at[e] = cu_seqlens[min(4 * lane + e, pg.B)];
#pragma unroll
    for (int e = 0; e < 4; ++e) n[e] = workgroups_of<S>(at[e + 1] - at[e], pg);
    const int sum = (n[0] + n[1]) + (n[2] + n[3]), upto = wave_prefix_sum(sum);
    const uint64_t beyond = __builtin_amdgcn_ballot_w64(upto > left);
    if (beyond != 0) {
      const int l = __builtin_ctzll(beyond);
      left -= __builtin_amdgcn_readlane(upto, l) - __builtin_amdgcn_readlane(sum, l);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ne = __builtin_amdgcn_readlane(n[e], l), a0 = __builtin_amdgcn_readlane(at[e], l);
        if (p.first < 0 && left < ne) {
          p.b = 4 * l + e;
          p.first = (ne - 1 - left) * S::kUnits;
          p.s0 = a0;
          p.len = __builtin_amdgcn_readlane(at[e + 1], l) - a0;
        }
        left -= ne;
      }
    }
  }
  return p;
}

template <int GROUPS, int UNITS, int NB, int SUMS>
__device__ __forceinline__ void prefill_attn_body(
    char* __restrict__ smem, const uint16_t* __restrict__ q, const u32x4* __restrict__ k, const u32x4* __restrict__ v,
    const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ block_table,
    u32x4* __restrict__ k_cache, u32x4* __restrict__ v_cache, uint16_t* __restrict__ out,
    float* __restrict__ lse, PrefillGrid pg, int Hq, int Hkv, int max_pages,
    float scale_log2e) {
  using S = Shape<GROUPS, UNITS, NB, SUMS>;
  constexpr int kTileQ = S::kTileQ, kProducts = 8 * NB;     // products of a step's scores: pages x blocks x 4
  const int g = static_cast<int>(pg.group.d);
  const Place at = pg.flat ? place_flat<S>(cu_seqlens, pg) : place_grid<S>(cu_seqlens, pg);
  if (at.first < 0) return;
  const int b = at.b, kvh = at.kvh, s0 = at.s0, len = at.len;
  const int n_tiles = (len + kTileQ - 1) / kTileQ, units = n_tiles * g;      // unit u: tile u / g, head u % g
  // the last step of the workgroup: that of its last unit's tile
  const int last_step = static_cast<int>(pg.group.divide(min(at.first + UNITS, units) - 1)) * kTileQ / kStepTok;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = GROUPS == 1 ? wave_id : wave_id % S::kUnits;   // within its group
  const int grp = GROUPS == 1 ? 0 : wave_id / S::kUnits;
  const int n = lane & 15;        // N index of both products: the query within a block
  const int bq = lane >> 4;       // k-group of the MFMA operand layouts
  const int unit = __builtin_amdgcn_readfirstlane(at.first + wave);
  const bool computes = unit < units;                                // else the wave only moves data
  const int tile = computes ? static_cast<int>(pg.group.divide(unit)) : 0;
  const int head = kvh * g + (unit - tile * g);
  const int q0 = tile * kTileQ;                      // first query token of the tile
  const int own_step = q0 / kStepTok;                // the step with the tile's own tokens
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  // Q^T operands: lane (n, bq) holds Q[query n of block nb][32*kk + 8*bq .. +8]; queries past
  // the end of the sequence are zero
  bf16x8 qf[NB][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int tq = q0 + 16 * nb + n;
    const u32x4* qrow =
        reinterpret_cast<const u32x4*>(q + (static_cast<size_t>(s0 + tq) * Hq + head) * kD);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      u32x4 x = {0u, 0u, 0u, 0u};
      if (computes && tq < len) x = qrow[kk * 4 + bq];
      qf[nb][kk] = __builtin_bit_cast(bf16x8, x);
    }
  }

  // ---- LDS-direct fetch of one step's K rows, or V rows, into a ring buffer ----
  // A wave moves kRows rows of its group's: kRows / 4 instructions of four rows x 256 bytes.  LDS
  // position lane%16 of row kRows*wave + 4*j + lane/16 takes the global granule that the swizzle maps
  // there.  The loads carry the range of the step's rows that the sequence has: rows past its end (they
  // are masked below) read as zeros, steps past it reach no memory.
  const size_t row_pitch = static_cast<size_t>(Hkv) * (kD * 2);
  const char* kbase = reinterpret_cast<const char*>(k) + (static_cast<size_t>(s0) * Hkv + kvh) * (kD * 2);
  const char* vbase = reinterpret_cast<const char*>(v) + (static_cast<size_t>(s0) * Hkv + kvh) * (kD * 2);
  uint32_t ld_k[S::kRows / 4], ld_v[S::kRows / 4];   // byte offset of the lane's granule in the step's rows
#pragma unroll
  for (int j = 0; j < S::kRows / 4; ++j) {
    const int row = S::kRows * wave + (lane >> 4) + 4 * j;
    ld_k[j] = static_cast<uint32_t>(row) * static_cast<uint32_t>(row_pitch) + static_cast<uint32_t>((lane & 15) ^ (row & 15)) * 16;
    ld_v[j] = static_cast<uint32_t>(row) * static_cast<uint32_t>(row_pitch) + static_cast<uint32_t>((lane & 15) ^ ((row & 7) << 1)) * 16;
  }
  // (The groups' steps alternate; each group has rings of its own: K buffers, then V buffers.)
  char* const ring = smem + grp * S::kGroupLds;
  // A stream of the group's steps: where the next one's rows begin, and the tokens from there to the sequence's end.
  struct Stream {
    const char* p;
    int left;
  };
  const size_t stride = static_cast<size_t>(GROUPS * kStepTok) * row_pitch;
  Stream ks = {kbase + static_cast<size_t>(grp * kStepTok) * row_pitch, len - grp * kStepTok};
  Stream vs = {vbase + static_cast<size_t>(grp * kStepTok) * row_pitch, len - grp * kStepTok};
  auto rows_of = [&](Stream& st) __attribute__((always_inline)) {
    // (the product before the comparison: as max(min(..)) the compiler clamps in a vector register)
    const uint32_t bytes = static_cast<uint32_t>(min(st.left, kStepTok)) * static_cast<uint32_t>(row_pitch);
    const BufferRsrc rsrc = buffer_rsrc(st.p, st.left > 0 ? bytes : 0u);
    st.p += stride;
    st.left -= GROUPS * kStepTok;
    return rsrc;
  };
  constexpr int kHalfLoads = S::kRows / 4;
  auto load_k = [&](const BufferRsrc rsrc, const int slot, const int j) __attribute__((always_inline)) {
    buffer_load_lds16(rsrc, ring + slot * kHalfBytes + (S::kRows * wave) * 256 + j * 1024, ld_k[j]);
  };
  auto load_v = [&](const BufferRsrc rsrc, const int slot, const int j) __attribute__((always_inline)) {
    buffer_load_lds16(rsrc, ring + (kRing + slot) * kHalfBytes + (S::kRows * wave) * 256 + j * 1024, ld_v[j]);
  };
  auto fetch_k = [&](const int slot) __attribute__((always_inline)) {
    const BufferRsrc rsrc = rows_of(ks);
#pragma unroll
    for (int j = 0; j < kHalfLoads; ++j) load_k(rsrc, slot, j);
  };
  auto fetch_v = [&](const int slot) __attribute__((always_inline)) {
    const BufferRsrc rsrc = rows_of(vs);
#pragma unroll
    for (int j = 0; j < kHalfLoads; ++j) load_v(rsrc, slot, j);
  };

  // operand read addresses inside a ring buffer (bytes)
  const uint32_t ring0 = lds0 + static_cast<uint32_t>(grp * S::kGroupLds);
  uint32_t k_off[4], v_off[8];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) k_off[kk] = ring0 + swz_k(n, 4 * kk + bq) * 16;
  {
    const int vrow = 4 * bq + (n >> 2);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
      v_off[dt] = ring0 + kRing * kHalfBytes + swz_v(vrow, 2 * dt + ((n & 3) >> 1)) * 16 + (n & 1) * 8;
  }

  struct State {
    float m[NB], l[NB];
    f32x4 o[NB][8];
  } state[SUMS];
#pragma unroll
  for (int e = 0; e < SUMS * NB; ++e) {
    State& st = state[e / NB];
    st.m[e % NB] = -INFINITY;
    st.l[e % NB] = 0.0f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) st.o[e % NB][dt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }

  // K rows of a step as the A operand (token = lane & 15), read once for both query blocks: a page's
  // 4 KB are 16 rows.  SLOT: the ring slot where it is known at compile time (an immediate offset), else -1.
  auto read_k = [&](u32x4 (&kf)[kSubs][4], const int kk, auto slotc, const int slot) __attribute__((always_inline)) {
    constexpr int OFF = decltype(slotc)::value < 0 ? 0 : decltype(slotc)::value * kHalfBytes;
    const uint32_t at = decltype(slotc)::value < 0 ? static_cast<uint32_t>(slot * kHalfBytes) : 0u;
    kf[0][kk] = lds_read128<OFF>(at + k_off[kk]);
    kf[1][kk] = lds_read128<OFF + kPageGranules * 16>(at + k_off[kk]);
  };
  auto wait_k = [&](u32x4 (&kf)[kSubs][4]) __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(kf[0][0]), "+v"(kf[0][1]), "+v"(kf[0][2]), "+v"(kf[0][3]), "+v"(kf[1][0]),
                 "+v"(kf[1][1]), "+v"(kf[1][2]), "+v"(kf[1][3])::"memory");
  };
  // The i-th product of a step's scores: 2 * NB independent chains.  This lane gets query n of block nb,
  // tokens 4*bq .. 4*bq+3 of page sub.
  auto score = [&](const int i, const u32x4 (&kf)[kSubs][4], f32x4 (&sc)[kSubs][NB]) __attribute__((always_inline)) {
    const int kk = i / (2 * NB), sub = i / NB % 2, nb = i % NB;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    sc[sub][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[sub][kk]), qf[nb][kk],
                                                          kk == 0 ? zero : sc[sub][nb], 0, 0, 0);
  };

  u32x4 kf[kSubs][4];       // K operands of the step after the one whose weights are formed
  f32x4 t[kSubs][NB];        // scores of that step, raw: the scale rides on the exponent's fma

  // Step i of the wave (its K/V step GROUPS * i + grp): the scores of step i + 1 are multiplied while the weights of
  // step i are formed, and the K rows of step i + 2 are read while the values of step i are multiplied.  last: the
  // wave's last step; it carries the causal mask and the end of the sequence (a block whose queries all lie before a
  // page's tokens is fully masked there: its weights are exp2(-inf - m) = 0).
  // (k_fill, v_fill: the ring buffers that the step's requests fill; V's go out first.)
  auto compute = [&](const int i, State& st, const int k_slot, const int v_slot, const int k_fill, const int v_fill, auto lastc,
                     auto kslotc, auto vslotc) __attribute__((always_inline)) {
    constexpr bool kLast = decltype(lastc)::value;
    BufferRsrc rsrc;
    // the step's requests, spread over eight places
    auto request = [&](const int place) __attribute__((always_inline)) {
      constexpr int kPer = 2 * kHalfLoads / 8 < 1 ? 1 : 2 * kHalfLoads / 8, kEvery = 8 / (2 * kHalfLoads) < 1 ? 1 : 8 / (2 * kHalfLoads);
      if (place % kEvery != 0) return;
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const int j = place / kEvery * kPer + e;
        if (j == 0) rsrc = rows_of(vs);
        if (j == kHalfLoads) rsrc = rows_of(ks);
        if (j < kHalfLoads) load_v(rsrc, v_fill, j);
        else load_k(rsrc, k_fill, j - kHalfLoads);
      }
    };
    // V^T operands: as the A operand through the transposing read (per page the lane gets rows
    // 4*bq + n/4 .. of columns 16*dt + 4*(n%4) .. +3), the two pages' halves side by side.
    s16x4 vf[8][2];
    auto read_v = [&](const int dt) __attribute__((always_inline)) {
      constexpr int OFF = decltype(vslotc)::value < 0 ? 0 : decltype(vslotc)::value * kHalfBytes;
      const uint32_t at = decltype(vslotc)::value < 0 ? static_cast<uint32_t>(v_slot * kHalfBytes) : 0u;
      vf[dt][0] = lds_read_tr16<OFF>(at + v_off[dt]);
      vf[dt][1] = lds_read_tr16<OFF + kPageGranules * 16>(at + v_off[dt]);
    };
    if (kLast) {
#pragma unroll
      for (int sub = 0; sub < kSubs; ++sub)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int tq = q0 + 16 * nb + n;
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            const int tk = (GROUPS * i + grp) * kStepTok + sub * kP + 4 * bq + rr;
            t[sub][nb][rr] = (tk <= tq && tk < len) ? t[sub][nb][rr] : -INFINITY;
          }
        }
    }
    // The running reference m of a query only has to keep the weights in range, so it is
    // left alone while no score of the step exceeds it by more than kSlack (in log2 units):
    // the step then needs no maximum, no exchange between lanes and no rescaling of the
    // state.  The weights are formed against the old reference first; if one of them is
    // above 2^kSlack (then so is the lane's sum of them - the test - and also while m is
    // still -inf), the references that have to move are moved and the weights formed again.
    f32x4 next[kSubs][NB];
    float w[NB][kSubs][4], add[NB];
    auto weight = [&](const int e) __attribute__((always_inline)) {
      const int nb = e >> 3, sub = (e >> 2) & 1, rr = e & 3;
      w[nb][sub][rr] = __builtin_amdgcn_exp2f(__builtin_fmaf(t[sub][nb][rr], scale_log2e, -st.m[nb]));
    };
    auto sum = [&](const int nb) __attribute__((always_inline)) {
      add[nb] = ((w[nb][0][0] + w[nb][0][1]) + (w[nb][0][2] + w[nb][0][3])) +
                ((w[nb][1][0] + w[nb][1][1]) + (w[nb][1][2] + w[nb][1][3]));
    };
#pragma unroll
    for (int e = 0; e < kProducts; ++e) {
      if (!kLast) score(e, kf, next);
      if (e < 8) read_v(e);
      weight(e);
      if (NB == 2 && e == 8) sum(0);
      if (!kLast) __builtin_amdgcn_sched_barrier(0);
    }
    sum(NB - 1);
    // (written so that a NaN sum - a masked score against m = -inf - also takes the branch)
    const bool grow = !(add[0] <= kBig && add[NB - 1] <= kBig);
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
      float alpha[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float mx = fmaxf(fmaxf(t[0][nb][0], t[0][nb][1]), fmaxf(t[0][nb][2], t[0][nb][3]));
#pragma unroll
        for (int sub = 1; sub < kSubs; ++sub)
          mx = fmaxf(mx, fmaxf(fmaxf(t[sub][nb][0], t[sub][nb][1]), fmaxf(t[sub][nb][2], t[sub][nb][3])));
        mx *= scale_log2e;                         // (the scale is positive: max commutes with it)
        mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
        // only a query whose own scores outgrew its reference moves it, so a query's
        // arithmetic does not depend on the other queries of the wave
        const float m_new = (mx > st.m[nb] + kSlack) ? mx : st.m[nb];
        alpha[nb] = __builtin_amdgcn_exp2f(st.m[nb] - m_new);
        st.m[nb] = m_new;
        st.l[nb] *= alpha[nb];
      }
#pragma unroll
      for (int e = 0; e < 8 * NB; ++e) st.o[e >> 3][e & 7] *= alpha[e >> 3];
#pragma unroll
      for (int e = 0; e < kProducts; ++e) weight(e);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) sum(nb);
    }
    // weights of the step's 32 tokens as the B operand of the 32-deep value product:
    // the first page's four in k-slots 0..3, the second page's in 4..7
    bf16x8 pf[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      st.l[nb] += add[nb];
      pf[nb] = __builtin_bit_cast(
          bf16x8, u32x4{pack_bf16x2(w[nb][0][0], w[nb][0][1]), pack_bf16x2(w[nb][0][2], w[nb][0][3]),
                        pack_bf16x2(w[nb][1][0], w[nb][1][1]), pack_bf16x2(w[nb][1][2], w[nb][1][3])});
    }
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(vf[0][0]), "+v"(vf[0][1]), "+v"(vf[1][0]), "+v"(vf[1][1]), "+v"(vf[2][0]), "+v"(vf[2][1]),
                   "+v"(vf[3][0]), "+v"(vf[3][1]), "+v"(vf[4][0]), "+v"(vf[4][1]), "+v"(vf[5][0]), "+v"(vf[5][1]),
                   "+v"(vf[6][0]), "+v"(vf[6][1]), "+v"(vf[7][0]), "+v"(vf[7][1])::"memory");
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      const s16x4 v0 = vf[dt][0], v1 = vf[dt][1];
      const s16x8 vv = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
      const bf16x8 va = __builtin_bit_cast(bf16x8, vv);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) st.o[nb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pf[nb], st.o[nb][dt], 0, 0, 0);
      if (!kLast && dt < 4) read_k(kf, dt, kslotc, k_slot);
      if (!kLast) request(dt);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (!kLast) {
#pragma unroll
      for (int e = 0; e < 2 * NB; ++e) t[e / NB][e % NB] = next[e / NB][e % NB];
      __builtin_amdgcn_sched_barrier(0);
      wait_k(kf);
    }
  };

  // A group's steps: `steps` in all, of which this wave computes the first `mine`.
  const int steps = last_step / GROUPS + 1;
  const int mine = computes && own_step >= grp ? (own_step - grp) / GROUPS + 1 : 0;
  // In step i the rows of V(i + kRing - 1) and K(i + kRing + 1) are requested, in this order, into the buffers of
  // V(i - 1) and K(i + 1), which every wave has read before the barrier that precedes step i; behind that barrier
  // V(i) and K(i + 2) have landed.  A wave's loads complete in issue order.
  auto wait_next = [&]() __attribute__((always_inline)) {
    wait_loads<4 * kHalfLoads>();      // those of the last two steps
    asm volatile("s_barrier" ::: "memory");
  };
  fetch_k(0);
  if (steps > 1) {
    fetch_k(1);
    fetch_v(0);
    fetch_k(2);
    fetch_v(1);
    fetch_k(3);
    wait_loads<4 * kHalfLoads>();
  } else {
    fetch_v(0);
    wait_loads<0>();
  }
  // The rows of a tile whose unit of head 0 is in this workgroup go to the sequence's pages (each row is written by exactly
  // one workgroup; slots past the end of the sequence are left alone).  They are requested behind the first steps' rows and
  // stored beside the first products.
  constexpr int kTileGranules = NB * kPageGranules, kMoves = 2 * kTileGranules / S::kThreads;
  u32x4 own[UNITS][kMoves];
  int32_t page[UNITS][kMoves];
  auto copies = [&](const int u) __attribute__((always_inline)) {      // the tile of that unit, or -1
    const int t0 = static_cast<int>(pg.group.divide(at.first + u));
    return at.first + u < units && t0 * g == at.first + u ? t0 : -1;
  };
#pragma unroll
  for (int u = 0; u < UNITS; ++u) {
    const int ct = copies(u);
    if (ct < 0) continue;
#pragma unroll
    for (int j = 0; j < kMoves; ++j) {
      const int m = tid + j * S::kThreads, gi = m & (kTileGranules - 1);   // K rows, then V rows; token gi >> 4, granule gi & 15
      const int tok = min(ct * kTileQ + (gi >> 4), len - 1);
      own[u][j] = (m < kTileGranules ? k : v)[(static_cast<size_t>(s0 + tok) * Hkv + kvh) * (kD * 2 / 16) + (m & 15)];
      page[u][j] = block_table[static_cast<size_t>(b) * max_pages + tok / kP];
    }
  }
  asm volatile("s_barrier" ::: "memory");
  // (Q is older than these rows.  Named here, where it has landed, it is not waited for behind the younger loads.)
#pragma unroll
  for (int e = 0; e < 4 * NB; ++e) asm volatile("" : "+v"(qf[e >> 2][e & 3]));
  if (mine > 0) {
    u32x4 kf0[kSubs][4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) read_k(kf0, kk, std::integral_constant<int, 0>{}, 0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) read_k(kf, kk, std::integral_constant<int, 1>{}, 0);
    asm volatile("s_waitcnt lgkmcnt(8)" : "+v"(kf0[0][0]), "+v"(kf0[0][1]), "+v"(kf0[0][2]), "+v"(kf0[0][3]), "+v"(kf0[1][0]),
                 "+v"(kf0[1][1]), "+v"(kf0[1][2]), "+v"(kf0[1][3])::"memory");
#pragma unroll
    for (int e = 0; e < kProducts; ++e) score(e, kf0, t);
    wait_k(kf);
  }
#pragma unroll
  for (int u = 0; u < UNITS; ++u) {
    const int ct = copies(u);
    if (ct < 0) continue;
#pragma unroll
    for (int j = 0; j < kMoves; ++j) {
      const int m = tid + j * S::kThreads, gi = m & (kTileGranules - 1);
      const size_t dst = (static_cast<size_t>(page[u][j]) * Hkv + kvh) * kPageGranules + (gi & (kPageGranules - 1));
      if (ct * kTileQ + (gi >> 4) < len) (m < kTileGranules ? k_cache : v_cache)[dst] = own[u][j];
    }
  }
  if (steps > 1) {
    wait_loads<2 * kHalfLoads>();
    asm volatile("s_barrier" ::: "memory");
    fetch_v(2);
    fetch_k(0);
  }

  constexpr std::integral_constant<int, -1> kAny{};
  int i = 0;
  auto fixed = [&](auto pc) __attribute__((always_inline)) {
    constexpr int p = decltype(pc)::value;
    compute(i + p, state[p % SUMS], 0, 0, (p + 1) % kRing, (p + 3) % kRing, std::false_type{},
            std::integral_constant<int, (p + 2) % kRing>{}, std::integral_constant<int, p>{});
    wait_next();
  };
  static_assert(kRing == 4 && kRing % SUMS == 0, "the steps below");
  for (; i + 4 < mine; i += 4) {
    fixed(std::integral_constant<int, 0>{});
    fixed(std::integral_constant<int, 1>{});
    fixed(std::integral_constant<int, 2>{});
    fixed(std::integral_constant<int, 3>{});
  }
  auto slot = [&](const int of) __attribute__((always_inline)) { return of & (kRing - 1); };
  while (i + 1 < mine) {
#pragma unroll
    for (int e = 0; e < SUMS; ++e) {                     // (i % SUMS == e)
      if (e > 0 && i + 1 >= mine) break;
      compute(i, state[e], slot(i + 2), slot(i), slot(i + 1), slot(i + 3), std::false_type{}, kAny, kAny);
      wait_next();
      ++i;
    }
  }
  auto fetch_step = [&]() __attribute__((always_inline)) {
    fetch_v(slot(i + 3));
    fetch_k(slot(i + 1));
  };
  if (i < mine) {
    const bool more = i + 1 < steps;         // another wave has further steps
    if (more) fetch_step();
#pragma unroll
    for (int e = 0; e < SUMS; ++e)
      if (SUMS == 1 || i % SUMS == e) compute(i, state[e], 0, slot(i), 0, 0, std::true_type{}, kAny, kAny);
    if (more) wait_next();
    ++i;
  }
  // a step after the wave's own tile (another wave of the workgroup still needs the rows), or a wave without a unit: it
  // fetches and waits with the others; nobody waits behind the last step (every wave passes the same number of barriers)
  for (; i + 1 < steps; ++i) {
    fetch_step();
    wait_next();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (the loads past the last step land before the LDS is given back)

  // normalise and store: lane (n, bq) owns d = 16*dt + 4*bq + r of query n
  auto store = [&](const int nb, const int dt, const f32x4& x, const float inv) __attribute__((always_inline)) {
    const int tq = q0 + 16 * nb + n;
    if (tq >= len) return;
    *reinterpret_cast<uint2*>(out + (static_cast<size_t>(s0 + tq) * Hq + head) * kD + 4 * bq + 16 * dt) =
        make_uint2(pack_bf16x2(x[0] * inv, x[1] * inv), pack_bf16x2(x[2] * inv, x[3] * inv));
  };
  auto finish = [&](const int nb, const float m, float l) __attribute__((always_inline)) {   // -> 1 / the query's sum
    l += __shfl_xor(l, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    const int tq = q0 + 16 * nb + n;
    if (lse != nullptr && grp == 0 && bq == 0 && tq < len)
      lse[static_cast<size_t>(s0 + tq) * Hq + head] = (m + __builtin_amdgcn_logf(l)) * kLn2;
    return 1.0f / l;
  };
  // The states of a query's keys are put together in the order of their first steps.  One without a step (m = -inf) would weigh
  // 0 and is passed over; the first has seen token 0, so the common reference is finite.
  auto weights = [](float& m, float& l, const float m1, const float l1, float& w0, float& w1) __attribute__((always_inline)) {
    const float m_all = fmaxf(m, m1);
    w0 = __builtin_amdgcn_exp2f(m - m_all);
    w1 = __builtin_amdgcn_exp2f(m1 - m_all);
    m = m_all;
    l = __builtin_fmaf(w0, l, w1 * l1);
  };
  auto mix = [](f32x4& x, const float w0, const float w1, const f32x4& y) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = __builtin_fmaf(w0, x[r], w1 * y[r]);
  };
  if constexpr (GROUPS == 1) {
    if (!computes) return;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      State& all = state[0];
#pragma unroll
      for (int e = 1; e < SUMS; ++e) {
        if (e > own_step) break;
        float w0, w1;
        weights(all.m[nb], all.l[nb], state[e].m[nb], state[e].l[nb], w0, w1);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) mix(all.o[nb][dt], w0, w1, state[e].o[nb][dt]);
      }
      const float inv = finish(nb, all.m[nb], all.l[nb]);
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) store(nb, dt, all.o[nb][dt], inv);
    }
  } else {
    // ... by all waves of a unit, each an equal part of the head dimension (by the first group's alone it took 128 vector
    // instructions per other group of 32 queries, 1.3 us for four): a wave hands the others their parts of its states, and all of
    // its (m, l).  State a of the unit is state a / GROUPS of group a % GROUPS.
    constexpr int kDt = 8 / GROUPS, kAll = GROUPS * SUMS;
    __syncthreads();                       // every load has landed and every buffer has been read
    char* const states = smem + wave * kAll * S::kState;
    auto hand = [&](auto group) __attribute__((always_inline)) {
      constexpr int G = decltype(group)::value;
#pragma unroll
      for (int s = 0; s < SUMS; ++s) {
        char* const to = states + (s * GROUPS + G) * S::kState;
#pragma unroll
        for (int e = 0; e < 8 * NB; ++e)
          if ((e & 7) / kDt != G) reinterpret_cast<f32x4*>(to)[e * 64 + lane] = state[s].o[e >> 3][e & 7];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          reinterpret_cast<float2*>(to + NB * 8 * 64 * 16)[nb * 64 + lane] = make_float2(state[s].m[nb], state[s].l[nb]);
      }
    };
    auto take = [&](auto group) __attribute__((always_inline)) {
      constexpr int G = decltype(group)::value;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float2 ml[kAll];
        f32x4 o[kAll][kDt];
#pragma unroll
        for (int a = 0; a < kAll; ++a) {
          const char* const from = states + a * S::kState;
          const State& own = state[a / GROUPS];
          if (a % GROUPS == G) ml[a] = make_float2(own.m[nb], own.l[nb]);
          else ml[a] = reinterpret_cast<const float2*>(from + NB * 8 * 64 * 16)[nb * 64 + lane];
#pragma unroll
          for (int e = 0; e < kDt; ++e) {
            const int dt = kDt * G + e;
            o[a][e] = a % GROUPS == G ? own.o[nb][dt] : reinterpret_cast<const f32x4*>(from)[(8 * nb + dt) * 64 + lane];
          }
        }
        float m = ml[0].x, l = ml[0].y;
#pragma unroll
        for (int a = 1; a < kAll; ++a) {
          if (a > own_step) break;
          float w0, w1;
          weights(m, l, ml[a].x, ml[a].y, w0, w1);
#pragma unroll
          for (int e = 0; e < kDt; ++e) mix(o[0][e], w0, w1, o[a][e]);
        }
        const float inv = finish(nb, m, l);
#pragma unroll
        for (int e = 0; e < kDt; ++e) store(nb, kDt * G + e, o[0][e], inv);
      }
    };
    static_assert(GROUPS == 2, "the two branches");
    if (computes && grp == 0) hand(std::integral_constant<int, 0>{});
    if (computes && grp == 1) hand(std::integral_constant<int, 1>{});
    __syncthreads();
    if (computes && grp == 0) take(std::integral_constant<int, 0>{});
    if (computes && grp == 1) take(std::integral_constant<int, 1>{});
  }
}

#define COPRIS_PREFILL_KERNEL(NAME, GROUPS, UNITS, NB, WAVES)                                            \
  template <int SUMS>                                                                                    \
  __global__ __launch_bounds__(GROUPS * 256)                                                           \
  __attribute__((amdgpu_waves_per_eu(WAVES, 2))) void NAME(                                            \
      const uint16_t* __restrict__ q, const u32x4* __restrict__ k, const u32x4* __restrict__ v,        \
      const int32_t* __restrict__ cu_seqlens, const int32_t* __restrict__ block_table,                 \
      u32x4* __restrict__ k_cache, u32x4* __restrict__ v_cache, uint16_t* __restrict__ out,            \
      float* __restrict__ lse, PrefillGrid pg, int Hq, int Hkv, int max_pages, float scale_log2e) {    \
    __shared__ __attribute__((aligned(1024))) char smem[Shape<GROUPS, UNITS, NB, SUMS>::kLds];         \
    prefill_attn_body<GROUPS, UNITS, NB, SUMS>(smem, q, k, v, cu_seqlens, block_table, k_cache, v_cache, out, \
                                               lse, pg, Hq, Hkv, max_pages, scale_log2e);              \
  }
// (two workgroups per CU: 256 registers per lane)
COPRIS_PREFILL_KERNEL(prefill_attn_kernel, 1, 4, 2, 2)
// For calls that do not fill the chip with these (prefill_shape says which shape a call takes): units of 16 queries, which
// have half the instructions per step; and two groups of waves per unit, group i taking the steps i, i + 2, ... from rings of
// its own, the softmax states put together at the end.  (One sequence of 4000 tokens, one head, us: 69.8 whole, 31.2 and 35.4 in
// two groups; 42.1 in four groups of 32 queries, whose rings of two buffers were too short for the rows to arrive.)
// The bounds of two groups allow eight waves also where there are four: with 512 registers for a wave the compiler keeps the
// accumulators in the other register file and moves them at every use (172 + 115 tokens, 16 / 4 heads: 8.8 us / 8.1).
COPRIS_PREFILL_KERNEL(prefill_attn_half_kernel, 1, 4, 1, 2)
COPRIS_PREFILL_KERNEL(prefill_attn_split2x2_kernel, 2, 2, 1, 1)
COPRIS_PREFILL_KERNEL(prefill_attn_split2x4_kernel, 2, 4, 1, 1)
#undef COPRIS_PREFILL_KERNEL

}  // namespace

bool prefill_attn_supported(int Hq, int Hkv, int D, int page_size, int dtype) {
  if (dtype != 1 || D != kD || page_size != kP || Hq % Hkv != 0) return false;
  const int g = Hq / Hkv;
  return g >= 1 && g <= 8;
}

int launch_prefill_attn(const void* q, const void* k, const void* v, const int32_t* cu_seqlens,
                        const int32_t* block_table, void* k_cache, void* v_cache, void* out,
                        float* lse, int B, int64_t T, int Hq, int Hkv, int max_pages, int max_seqlen,
                        float scale, hipStream_t stream) {
  const int g = Hq / Hkv;
  const float scale_log2e = scale * kLog2e;
  const PrefillPlan plan = prefill_plan(B, T, Hq, g, max_seqlen);
  const int per_wg = kPrefillCost[plan.shape].units, tile = kPrefillCost[plan.shape].queries;
  const int64_t wgs_max = (static_cast<int64_t>((max_seqlen - 1) / tile + 1) * g + per_wg - 1) / per_wg;      // of a sequence and kv head
  const int64_t wgs = prefill_flat_grid(B, T, Hkv, g, wgs_max, tile, per_wg);
  const dim3 grid = wgs > 0 ? dim3(static_cast<unsigned>(wgs)) : dim3(static_cast<unsigned>(wgs_max), Hkv, B);
  const PrefillGrid pg = prefill_grid(B, Hkv, g, wgs > 0);
#define COPRIS_PREFILL(KERNEL, THREADS, SUMS)                                                               \
  COPRIS_PRE(#KERNEL);                                                                                      \
  hipLaunchKernelGGL(KERNEL<SUMS>, grid, dim3(THREADS), 0, stream, static_cast<const uint16_t*>(q),         \
                     static_cast<const u32x4*>(k), static_cast<const u32x4*>(v), cu_seqlens, block_table,   \
                     static_cast<u32x4*>(k_cache), static_cast<u32x4*>(v_cache), static_cast<uint16_t*>(out), \
                     lse, pg, Hq, Hkv, max_pages, scale_log2e);                                             \
  COPRIS_POST(#KERNEL)
  switch (10 * plan.shape + plan.sums) {
    case 10 * kPrefillHalf + 1: COPRIS_PREFILL(prefill_attn_half_kernel, 256, 1); break;
    case 10 * kPrefillHalf + 2: COPRIS_PREFILL(prefill_attn_half_kernel, 256, 2); break;
    case 10 * kPrefill2x2 + 1: COPRIS_PREFILL(prefill_attn_split2x2_kernel, 256, 1); break;
    case 10 * kPrefill2x2 + 2: COPRIS_PREFILL(prefill_attn_split2x2_kernel, 256, 2); break;
    case 10 * kPrefill2x4 + 1: COPRIS_PREFILL(prefill_attn_split2x4_kernel, 512, 1); break;
    case 10 * kPrefill2x4 + 2: COPRIS_PREFILL(prefill_attn_split2x4_kernel, 512, 2); break;
    default: COPRIS_PREFILL(prefill_attn_kernel, 256, 1); break;
  }
#undef COPRIS_PREFILL
  return 0;
}

}  // namespace copris
