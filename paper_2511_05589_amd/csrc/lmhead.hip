// LM-head projection fused with log-softmax, Gumbel-max sampling and the chosen
// token's log-probability (the per-token log-prob under the generating policy that
// the buffer keeps: Section 4, Eq. 6; sampler settings: Table 4).
//
// The V logits of a row are never written out.  Every (row, vocabulary tile) pair
// produces one small partial
//     m    = max_v z_v                s = sum_v exp(z_v - m)
//     best = max_v (z_v + G_v)        idx, z = its vocabulary index and raw logit
// and a merge kernel combines the partials of a row: lse = m + ln s,
// logprob = z_best - lse.  Ties on the perturbed score go to the lowest index, in
// the tiles and in the merge, so the result does not depend on the tiling.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <utility>

#include "copris_device.h"
#include "copris_internal.h"

namespace copris {

struct LmPartial {
  float m, s, best, z;
  int32_t idx;
};

constexpr int kLmTileC = 16;      // batch rows per workgroup (generic kernel)
constexpr int kLmBK = 256;        // hidden-dim slab staged in LDS

static inline size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// (score, idx) ordering: larger score first, then lower index.
__device__ __forceinline__ bool better(float sa, int ia, float sb, int ib) {
  return sa > sb || (sa == sb && ia < ib);
}

__device__ __forceinline__ void combine(LmPartial& a, const LmPartial& o) {
  const float m = fmaxf(a.m, o.m);
  // exp(-inf - m) = 0 handles empty partials (m = -inf, s = 0) as long as m is finite
  const float sa = a.m == -INFINITY ? 0.0f : a.s * __expf(a.m - m);
  const float sb = o.m == -INFINITY ? 0.0f : o.s * __expf(o.m - m);
  a.m = m;
  a.s = sa + sb;
  if (better(o.best, o.idx, a.best, a.idx)) {
    a.best = o.best;
    a.idx = o.idx;
    a.z = o.z;
  }
}

// Two neighbouring runs of vocabulary rows.  The same bits with the two exchanged, and wherever it is called.
__device__ __forceinline__ void join(LmPartial& a, const LmPartial& o) {
#pragma clang fp contract(off)
  const float m = fmaxf(a.m, o.m);
  const float sa = a.m == -INFINITY ? 0.0f : a.s * __expf(a.m - m);
  const float sb = o.m == -INFINITY ? 0.0f : o.s * __expf(o.m - m);
  a.m = m;
  a.s = sa + sb;
  if (better(o.best, o.idx, a.best, a.idx)) {
    a.best = o.best;
    a.idx = o.idx;
    a.z = o.z;
  }
}

__device__ __forceinline__ LmPartial wave_combine(LmPartial p) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    LmPartial q;
    q.m = __shfl_xor(p.m, o, kWave);
    q.s = __shfl_xor(p.s, o, kWave);
    q.best = __shfl_xor(p.best, o, kWave);
    q.z = __shfl_xor(p.z, o, kWave);
    q.idx = __shfl_xor(p.idx, o, kWave);
    combine(p, q);
  }
  return p;
}

// One logit -> a single-element partial.
__device__ __forceinline__ LmPartial logit_partial(float z, int v, uint32_t word) {
  LmPartial p;
  p.m = z;
  p.s = 1.0f;
  p.best = z + gumbel_from_uniform(word_to_uniform(word));
  p.z = z;
  p.idx = v;
  return p;
}

__device__ __forceinline__ LmPartial empty_partial() {
  LmPartial p;
  p.m = -INFINITY;
  p.s = 0.0f;
  p.best = -INFINITY;
  p.z = 0.0f;
  p.idx = 0x7fffffff;
  return p;
}

// --------------------------------------------------------------------------
// generic kernel (bf16 whose hidden size the matrix-core kernels do not take; vector ALU): wave w of
// a workgroup owns batch rows 4w..4w+3 of the 16-row block, lane l owns vocabulary row tile*64 + l.
// --------------------------------------------------------------------------
__device__ __forceinline__ void load_bf16x8(const uint16_t* p, float (&x)[8]) {
  const uint4 v = *reinterpret_cast<const uint4*>(p);
  x[0] = bf16lo_to_f32(v.x); x[1] = bf16hi_to_f32(v.x);
  x[2] = bf16lo_to_f32(v.y); x[3] = bf16hi_to_f32(v.y);
  x[4] = bf16lo_to_f32(v.z); x[5] = bf16hi_to_f32(v.z);
  x[6] = bf16lo_to_f32(v.w); x[7] = bf16hi_to_f32(v.w);
}

// Logit z of vocabulary entry v of batch row c as a partial.  GIVEN: no sampling; the partial that
// holds vocabulary entry target[c] carries its logit (best = +inf marks it, so the same combine
// picks it up).
template <bool GIVEN>
__device__ __forceinline__ LmPartial tile_partial(float z, int v, int c, const int64_t* seq_id, const int32_t* step,
                                                  const int32_t* target, uint32_t key0, uint32_t key1) {
  if (GIVEN) {
    const bool hit = v == target[c];
    LmPartial p;
    p.m = z;
    p.s = 1.0f;
    p.z = z;
    p.best = hit ? INFINITY : -INFINITY;
    p.idx = hit ? v : 0x7fffffff;
    return p;
  }
  const uint64_t sid = static_cast<uint64_t>(seq_id[c]);
  const Philox4 x = philox4x32_10(static_cast<uint32_t>(v) >> 2, static_cast<uint32_t>(step[c]),
                                  static_cast<uint32_t>(sid), static_cast<uint32_t>(sid >> 32), key0, key1);
  const int sel = v & 3;
  const uint32_t word = sel == 0 ? x.x : (sel == 1 ? x.y : (sel == 2 ? x.z : x.w));
  return logit_partial(z, v, word);
}

template <bool GIVEN>
__global__ __launch_bounds__(256) void lmhead_generic_kernel(
    const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight, const int64_t* __restrict__ seq_id,
    const int32_t* __restrict__ step, const int32_t* __restrict__ target, uint32_t key0,
    uint32_t key1, float inv_temperature, LmPartial* __restrict__ part, int C, int H, int V,
    int n_tiles) {
  __shared__ float s_h[kLmTileC][kLmBK];
  const int tile = blockIdx.x, cb = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int v = tile * kLmTileV + lane;
  const bool v_ok = v < V;
  const uint16_t* wrow = weight + static_cast<size_t>(v_ok ? v : 0) * H;
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};

  for (int k0 = 0; k0 < H; k0 += kLmBK) {
    const int kn = min(kLmBK, H - k0);
    __syncthreads();
    for (int e = tid; e < kLmTileC * kn; e += 256) {
      const int r = e / kn, k = e - r * kn;
      const int c = cb * kLmTileC + r;
      s_h[r][k] = c < C ? bf16_to_f32(hidden[static_cast<size_t>(c) * H + k0 + k]) : 0.0f;
    }
    __syncthreads();
    if (v_ok) {
      for (int k = 0; k < kn; k += 8) {
        float x[8];
        load_bf16x8(wrow + k0 + k, x);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[r] = fmaf(s_h[4 * wave + r][k + j], x[j], acc[r]);
        }
      }
    }
  }

#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = cb * kLmTileC + 4 * wave + r;
    if (c >= C) continue;   // uniform across the wave
    LmPartial p = empty_partial();
    if (v_ok) p = tile_partial<GIVEN>(acc[r] * inv_temperature, v, c, seq_id, step, target, key0, key1);
    p = wave_combine(p);
    if (lane == 0) part[static_cast<size_t>(c) * n_tiles + tile] = p;
  }
}

// --------------------------------------------------------------------------
// fp32 kernel: full-precision matrix products (mfma 16x16x4 fp32).
//
// A workgroup of 16 waves takes 64 vocabulary rows (one partial per batch row, as in the generic
// kernel) against 16 * NB batch rows: four vocabulary groups of 16 rows x four quarters of the hidden
// dimension.  Lane (i, b) of a product holds element b of row i, so a lane fetches 16-byte granules
// 4j + b of its vocabulary row and of its batch rows and feeds four products with each; the operands
// come straight from memory, kDeep granules of each in flight.  The quarters' sums are added in
// order, and then every wave forms the partials of NB batch rows with one vocabulary entry per lane.
// Small shapes are bound by the chain of latencies (16 products deep per quarter here, where a wave
// of the vector-ALU kernel walked the whole hidden dimension with four entries in flight):
// whole calls, C = 8, H = 256, V = 1024: 20.4 -> 10.8 us; C = 64, H = 1024, V = 32768: 283 -> 100;
// C = 2, H = 3584, V = 100000: 1020 -> 272.
// --------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kF32Threads = 1024;

template <bool GIVEN, int NB>
__global__ __launch_bounds__(kF32Threads) void lmhead_f32_kernel(
    const float* __restrict__ hidden, const float* __restrict__ weight, const int64_t* __restrict__ seq_id,
    const int32_t* __restrict__ step, const int32_t* __restrict__ target, uint32_t key0, uint32_t key1,
    float inv_temperature, LmPartial* __restrict__ part, int C, int H, int V, int n_tiles) {
  constexpr int kPitch = kLmTileV + 4;
  constexpr int kDeep = NB == 1 ? 4 : 2;
  __shared__ __attribute__((aligned(16))) float s_z[4][16 * NB][kPitch];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int vg = wave & 3, kq = wave >> 2;             // vocabulary group, quarter of the hidden dimension
  const int n = lane & 15, b = lane >> 4;
  const int tile = blockIdx.x, c0 = blockIdx.y * 16 * NB;
  const int granules = H / 4;                          // of a row
  const int steps = (granules + 3) / 4;                // four granules (16 elements) of a row per step
  const int j0 = steps * kq / 4, j1 = steps * (kq + 1) / 4;
  const float4* wrow = reinterpret_cast<const float4*>(weight + static_cast<size_t>(min(tile * kLmTileV + 16 * vg + n, V - 1)) * H);
  const float4* hrow[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
    hrow[i] = reinterpret_cast<const float4*>(hidden + static_cast<size_t>(min(c0 + 16 * i + n, C - 1)) * H);
  f32x4 acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  for (int j = j0; j < j1; j += kDeep) {
    float4 x[kDeep], y[kDeep][NB];
#pragma unroll
    for (int u = 0; u < kDeep; ++u) {
      const int gr = 4 * (j + u) + b, at = gr < granules ? gr : 0;
      x[u] = wrow[at];
#pragma unroll
      for (int i = 0; i < NB; ++i) y[u][i] = hrow[i][at];
    }
#pragma unroll
    for (int u = 0; u < kDeep; ++u) {
      // past the quarter or the row: nothing (both sides zero, so that no infinity meets a zero)
      const bool in = j + u < j1 && 4 * (j + u) + b < granules;
      if (!in) x[u] = zero;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const float4 h = in ? y[u][i] : zero;
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u].x, h.x, acc[i], 0, 0, 0);
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u].y, h.y, acc[i], 0, 0, 0);
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u].z, h.z, acc[i], 0, 0, 0);
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u].w, h.w, acc[i], 0, 0, 0);
      }
    }
  }
  // lane (n, b): vocabulary rows 16*vg + 4b .. +3 of batch row 16*i + n
#pragma unroll
  for (int i = 0; i < NB; ++i)
    *reinterpret_cast<float4*>(&s_z[kq][16 * i + n][16 * vg + 4 * b]) = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
  __syncthreads();
  const int v = tile * kLmTileV + lane;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int c = c0 + 16 * i + wave;
    if (c >= C) continue;   // uniform across the wave
    const float dot = ((s_z[0][16 * i + wave][lane] + s_z[1][16 * i + wave][lane]) + s_z[2][16 * i + wave][lane]) +
                      s_z[3][16 * i + wave][lane];
    LmPartial p = empty_partial();
    if (v < V) p = tile_partial<GIVEN>(dot * inv_temperature, v, c, seq_id, step, target, key0, key1);
    p = wave_combine(p);
    if (lane == 0) part[static_cast<size_t>(c) * n_tiles + tile] = p;
  }
}

// --------------------------------------------------------------------------
// matrix-core kernel (bf16, H % 32 == 0).
//
// Z^T[v][c] = W[v][:] . hidden[c][:] with the VOCABULARY as the M side of
// mfma_f32_32x32x16_bf16 and the batch as the N side: a lane's 16 accumulators of a
// 32x32 block are then 4 runs of 4 consecutive vocabulary entries of ONE batch row,
// i.e. exactly one Philox block (4 words) per run, and the row's running
// log-sum-exp / arg-max state lives in that lane.
//
// A workgroup (4 waves) owns a 128 (vocab) x 256 (batch) tile and walks the hidden
// dimension in slabs of 64 (128-byte row segments: full cache lines).  Workgroups are
// persistent over vocabulary tiles and keep their per-row state across tiles, so W is
// streamed from HBM exactly once and only gridDim.x partials per row reach the merge.
// Two workgroups share a CU, so one's epilogue (vector ALU) overlaps the other's
// products (matrix cores) and loads.
//
// Sampling without a second logarithm: argmax_v (z_v - ln E_v), E_v = -ln u_v, is
// argmin_v E_v / exp(z_v - m); the exponential is the one the log-sum-exp needs
// anyway, and candidates are compared by cross-multiplication of logarithms to base 2
// (log u_v * p_best > log u_best * p_v), rescaling p_best whenever the running max moves.
// --------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMfBM = 128;       // vocabulary rows per tile
constexpr int kMfBN = 256;       // batch rows per workgroup
constexpr int kMfBK = 64;        // hidden-dim slab (128 bytes of a row)
constexpr int kMfMaxGrid = 512;  // persistent workgroups along the vocabulary (2 per CU)
constexpr float kLn2f = 0.6931471805599453f, kLog2ef = 1.4426950408889634f;

// The running maximum is an accumulator, and exp(z - m) = exp2((accumulator - maximum) * scale) with
// scale = log2(e) / temperature: three instructions, whose rounding is relative to the distance from the maximum.  The
// maximum's own exponential is 1 and its logit rounds like the chosen one's, so that a row's log-prob is never above 0.
// (exp2(fma(accumulator, scale, -maximum * scale)) is one instruction fewer, but then the rounding of scale counts by the
// size of the logits: a log-prob was 3e-6 off for logits around 30 at temperature 0.55, now 1e-6; up to 3e-5 above 0 at
// temperature 0.1 where one token has all the weight, now 0.  Whole calls before / now, in us: C = 256, H = 3584,
// V = 151936 300.5 / 298.0; C = 301, H = 2048, V = 50257 85.0 / 85.0; 8192 given tokens 6496 / 6466.)
struct LmLaneState {
  float m, s;        // running max (an accumulator) and sum of the exponentials
  float l_best;      // log2(u) of the current best candidate (-inf: none yet)
  float p_best;      // its exponential
  float a_best;      // its accumulator
  int idx;
};

// log2(e) / temperature, finite where 1 / temperature is
__device__ __forceinline__ float lm_scale(float inv_temperature) {
  constexpr float kLog2eLo = 1.92596299e-8f;     // log2(e) - kLog2ef
  return fminf(__builtin_fmaf(inv_temperature, kLog2ef, inv_temperature * kLog2eLo), 3.402823466e38f);
}
__device__ __forceinline__ float lm_exp(float a, float m, float scale) { return __builtin_amdgcn_exp2f((a - m) * scale); }

// LDS position (in 16-byte granules) of granule g (0..7) of row `row` of a [rows][64]
// bf16 slab.  Sixteen lanes that read one granule column of sixteen consecutive rows
// touch sixteen different 4-bank groups.
__device__ __forceinline__ int lm_swz(int row, int g) { return row * 8 + (g ^ ((row >> 1) & 7)); }

// Masks the accumulators of a block whose vocabulary entries lie past the end (accumulator r is entry
// vbase + 8*(r/4) + r%4).
__device__ __forceinline__ void lm_mask_block(f32x16& acc, int vbase, int V) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (vbase + 8 * (r >> 2) + (r & 3) >= V) acc[r] = -INFINITY;
}

// The sampler: 25 vector instructions per entry (of a Philox block's 99, 18 are 64-bit multiplications and 19
// three-input exclusive ors).  It is bound by their number: two waves of a SIMD issue one each in turn.  35 instructions
// (exclusive ors by pairs, the uniform through a conversion, the temperature and the base of the exponential
// multiplied apart, a mask test per entry) against 24 (see above) took 171 cycles per entry and SIMD where nothing else ran; whole calls
// C = 64, H = 1536, V = 151936 92 -> 89.5 us, C = 301, H = 2048, V = 50257 118.4 -> 115.4,
// C = 256, H = 3584, V = 151936 302.5 -> 299.1.
__device__ __forceinline__ void lm_epilogue_block(f32x16& acc, LmLaneState& st, int vbase, int V, bool tail,
                                                  float scale, uint32_t step_c, uint32_t sid_lo, uint32_t sid_hi,
                                                  uint32_t key0, uint32_t key1) {
  if (tail) lm_mask_block(acc, vbase, V);
  float am = acc[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) am = fmaxf(am, acc[r]);
  const float m_new = fmaxf(st.m, am);
  if (m_new == -INFINITY) return;            // nothing valid seen so far (vocabulary tail)
  const float alpha = lm_exp(st.m, m_new, scale);  // 0 on the first block (m = -inf)
  st.s *= alpha;
  st.p_best *= alpha;
  st.m = m_new;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int vq = vbase + 8 * q;
    const Philox4 x = philox4x32_10(static_cast<uint32_t>(vq) >> 2, step_c, sid_lo, sid_hi, key0, key1);
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float p = lm_exp(acc[4 * q + j], m_new, scale);   // 0 for masked entries
      st.s += p;
      const float l = __builtin_amdgcn_logf(word_to_uniform(w[j]));   // log2(u) < 0
      // strictly better only: on an exact tie the earlier (lower) index stays
      if (l * st.p_best > st.l_best * p) {
        st.l_best = l;
        st.p_best = p;
        st.a_best = acc[4 * q + j];
        st.idx = vq + j;
      }
    }
  }
}

// Same block, no sampling: running log-sum-exp, and the logit of vocabulary entry `target`
// if this lane holds it.
__device__ __forceinline__ void lm_given_block(f32x16& acc, LmLaneState& st, int vbase, int V, bool tail, float scale,
                                               int target) {
  if (tail) lm_mask_block(acc, vbase, V);
  float am = acc[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) am = fmaxf(am, acc[r]);
  const float m_new = fmaxf(st.m, am);
  if (m_new == -INFINITY) return;
  st.s *= lm_exp(st.m, m_new, scale);
  st.m = m_new;
  float s = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) s += lm_exp(acc[r], m_new, scale);
  st.s += s;
  const int d = target - vbase;                  // entry vbase + 8q + j sits in accumulator 4q + j
  if (d >= 0 && d < 32 && (d & 4) == 0 && target < V) {
    const int sel = (d >> 3) * 4 + (d & 3);
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (r == sel) st.a_best = acc[r];
    st.idx = target;
  }
}

// A lane's running state as a partial.
template <bool GIVEN>
__device__ __forceinline__ LmPartial state_partial(const LmLaneState& st, float inv_temperature) {
  LmPartial p;
  p.m = st.m * inv_temperature;
  p.s = st.s;
  p.z = st.a_best * inv_temperature;
  p.idx = st.idx;
  // perturbed score z + G with G = -ln(E), E = -ln u = -l_best * ln 2
  if (GIVEN) {
    p.best = st.idx == 0x7fffffff ? -INFINITY : INFINITY;
  } else {
    p.best = st.idx == 0x7fffffff ? -INFINITY : p.z - logf(st.l_best * -kLn2f);
  }
  return p;
}
// ... combined with the other k-half of the wave (lane ^ 32).
template <bool GIVEN>
__device__ __forceinline__ LmPartial lane_partial(const LmLaneState& st, float inv_temperature) {
  LmPartial p = state_partial<GIVEN>(st, inv_temperature);
  LmPartial o;
  o.m = __shfl_xor(p.m, 32, kWave);
  o.s = __shfl_xor(p.s, 32, kWave);
  o.best = __shfl_xor(p.best, 32, kWave);
  o.z = __shfl_xor(p.z, 32, kWave);
  o.idx = __shfl_xor(p.idx, 32, kWave);
  combine(p, o);
  return p;
}

// ---- memory pipeline of the matrix-core kernel --------------------------------
// Both operands reach LDS through LDS-direct loads (global_load_lds_dwordx4: each
// lane's 16 bytes land at base + 16*lane, no registers in between), so the data in
// flight lives in LDS rings:
//   W       [128 rows][64 k] slabs of 16 KB, ring of two, issued a slab and a half ahead (a
//           slab's slot is given away as soon as every wave has its operands in registers);
//   hidden  [128 rows][64 k] units of 16 KB - the two batch halves of a slab are
//           consumed one after the other against the same W slab - ring of three,
//           issued two units (one slab) ahead.
// Every wave issues a quarter of each slab and unit, one load at a time between the matrix
// products.  The outstanding-load counter of a wave retires in order, so the issue order is
// chosen such that what a wait needs is always older than what may stay in flight: per slab
// d hidden (d+1, half 0), then W(d+2), and after the middle barrier hidden (d+1, half 1).  The
// compiler cannot count LDS-direct loads per buffer (it would drain them all before any LDS
// read), so the operand reads are inline ds_read_b128 and every wait is explicit.  80 KB of LDS per workgroup: two workgroups fill a CU's 160 KB.
constexpr int kLmStreamOnce = 2;                    // cache policy of the W loads: non-temporal (every byte is read once)
constexpr int kNW = 2;                              // W ring slabs
constexpr int kNH = 3;                              // hidden ring units
constexpr int kSlab = 128 * kMfBK * 2;              // 16 KB: a W slab or a hidden unit
constexpr int kHRing = kNW * kSlab;                 // hidden ring starts here
constexpr int kMfLds = kHRing + kNH * kSlab;        // 80 KB

template <int OFF>
__device__ __forceinline__ u32x4 lds_read128(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
// (Waits on these reads are inline "s_waitcnt lgkmcnt(N)" statements that tie the operands
// which must have arrived, so that no use can be scheduled above the wait.)

template <int N>
__device__ __forceinline__ void wait_loads() {   // at most N of this wave's loads may still be in flight
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// two k-steps' hidden operands have arrived, N LDS reads may still be under way
template <int N, int NT>
__device__ __forceinline__ void lds_wait_b(u32x4 (&p)[NT], u32x4 (&q)[NT]) {
  if constexpr (NT == 2) {
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(p[0]), "+v"(p[1]), "+v"(q[0]), "+v"(q[1]) : "n"(N) : "memory");
  } else {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(p[0]), "+v"(q[0]) : "n"(N) : "memory");
  }
}

// Timing probes (never defined in the product build; `python -m paper_2511_05589_amd.build
// --define NAME --out other.so` builds one, bench.py --lib times it; the results of such a
// build are wrong by design, every access stays in bounds and every loop ends):
//   COPRIS_LM_PROBE_NO_MFMA      the matrix products become one scalar multiply-add each
//   COPRIS_LM_PROBE_NO_EPILOGUE  no log-sum-exp / sampling after a tile
//   COPRIS_LM_PROBE_NO_W_LOADS   the W stream is not requested (operands are whatever LDS holds)
//   COPRIS_LM_PROBE_NO_H_LOADS   the hidden stream is not requested
//   COPRIS_LM_PROBE_W_FROM_L2    every workgroup re-reads the first two vocabulary tiles
// They separate what bounds the kernel: the memory pipeline alone, the products alone, the
// lead of the W stream.
#if defined(COPRIS_LM_PROBE_NO_MFMA)
#define COPRIS_LM_MFMA(fa, fb, c) ((c)[0] += static_cast<float>((fa)[0]) * static_cast<float>((fb)[0]), (c))
#else
#define COPRIS_LM_MFMA(fa, fb, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb, c, 0, 0, 0)
#endif

// (Batches of up to 64 rows mostly take lmhead_skinny_kernel below.)
// HALVES = 2: 256 batch rows per workgroup (two halves of 128 against every W slab), W ring
// of two slabs, hidden ring of three units; NT1 = 1: the second half has only 64 rows (192 in all).
// HALVES = 1 (C <= 128): only the first half
// exists, so there is no second half of products, loads and barrier; the hidden ring needs two
// units and the W ring gets three slabs (a slab is requested two slabs ahead).
template <bool GIVEN, int HALVES, int NT1>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void lmhead_mfma_kernel(
    const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight,
    const int64_t* __restrict__ seq_id, const int32_t* __restrict__ step,
    const int32_t* __restrict__ target, uint32_t key0, uint32_t key1, float inv_temperature,
    LmPartial* __restrict__ part, int C, int H, int V, int block_rows, int n_tiles, int n_parts, int flip) {
  __shared__ __attribute__((aligned(1024))) char smem[kMfLds];
  const int tid = threadIdx.x, lane = tid & 63;
  const float scale = lm_scale(inv_temperature);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wq = wave & 1;     // vocabulary half; 64-row block of a batch half
  const int l32 = lane & 31, kb = lane >> 5;
  // this workgroup's batch rows, and its place among those that share the tiles out (flip: see
  // lm_second_block_flip; with one tile each the blocks share it through the L2)
  const int c0 = blockIdx.y * block_rows, c_end = min(C, c0 + block_rows);
  const int place = blockIdx.x ^ (blockIdx.y * flip);
  const int nkd = H / kMfBK;                   // slabs per tile
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const uint32_t pitch = static_cast<uint32_t>(H) * 2u;
  constexpr int kRingW = HALVES == 2 ? kNW : 3;        // W ring slabs
  constexpr int kRingH = HALVES == 2 ? kNH : 2;        // hidden ring units
  constexpr int kHBase = kRingW * kSlab;               // hidden ring starts here
  static_assert(kHBase + kRingH * kSlab <= kMfLds, "rings exceed the workgroup's LDS");

  // operand read offsets inside a slab / unit (bytes); it / nt add 32 rows = 4096 bytes
  uint32_t a_off[4], b_off[4], b1_off[4];
#pragma unroll
  for (int k16 = 0; k16 < 4; ++k16) {
    a_off[k16] = lm_swz(64 * wm + l32, 2 * k16 + kb) * 16;
    b_off[k16] = lm_swz(64 * wq + l32, 2 * k16 + kb) * 16;
    b1_off[k16] = lm_swz(32 * NT1 * wq + l32, 2 * k16 + kb) * 16;   // second half
  }

  // ---- loader cursors (wave-uniform) ----
  const int my_tiles = place < n_tiles ? (n_tiles - 1 - place) / gridDim.x + 1 : 0;
  const int total = my_tiles * nkd;            // W slabs this workgroup consumes (hidden units: 2x)
  // Every wave moves a quarter of every W slab and of every hidden unit: rows 32*wave ..
  // 32*wave+31, four instructions of 8 rows x 128 bytes.  LDS position 64*chunk + lane of a
  // slab holds (row 8*chunk + lane/8, stored granule lane%8); the lane fetches the global
  // granule that the swizzle maps there: (row>>1)&7 = lane>>4 for even chunks, +4 for odd
  // ones, i.e. bit 6 of the byte offset flips for odd j.
  const int ld_row = 32 * wave + (lane >> 3);                // + 8*j
  const uint32_t ld_g = ((lane & 7) ^ (lane >> 4)) * 16;
  int w_tile = place, w_kd = 0, w_ring = 0;             // W cursor (tile, slab) and ring slot
  int h_n = 0, h_kd = 0, h_ring = 0;                         // hidden units issued so far (half = h_n & 1), slab, slot
  const char* wbase = reinterpret_cast<const char*>(weight);
  const char* hbase = reinterpret_cast<const char*>(hidden);
  // Rows past V re-read the last vocabulary row (masked in the epilogue); rows past C
  // duplicate the last batch row (never used).
  // one of the four loads of this wave's quarter of the W slab / hidden unit at the cursor
  auto w_load = [&](int j) __attribute__((always_inline)) {
    char* dst = smem + w_ring * kSlab + (4 * wave + j) * 1024;
    const uint32_t koff = static_cast<uint32_t>(w_kd) * (kMfBK * 2) + ld_g;
#if defined(COPRIS_LM_PROBE_W_FROM_L2)
    const int v = min((w_tile & 1) * kMfBM + ld_row + 8 * j, V - 1);
#else
    const int v = min(w_tile * kMfBM + ld_row + 8 * j, V - 1);
#endif
#if !defined(COPRIS_LM_PROBE_NO_W_LOADS)
    __builtin_amdgcn_global_load_lds(wbase + (static_cast<uint32_t>(v) * pitch + (koff ^ ((j & 1) * 64))), dst,
                                     16, 0, kLmStreamOnce);
#else
    (void)v; (void)koff; (void)dst;
#endif
  };
  auto w_advance = [&]() __attribute__((always_inline)) {
    w_ring = w_ring + 1 == kRingW ? 0 : w_ring + 1;
    if (++w_kd == nkd) {
      w_kd = 0;
      w_tile += gridDim.x;
    }
  };
  // (a second half of 64 rows is two loads per wave, rows 16*wave ..)
  auto h_load = [&](int j, auto halfc) __attribute__((always_inline)) {
    constexpr int kHalf = decltype(halfc)::value, kPer = kHalf == 1 ? 2 * NT1 : 4;
    char* dst = smem + kHBase + h_ring * kSlab + (kPer * wave + j) * 1024;
    const uint32_t koff = static_cast<uint32_t>(h_kd) * (kMfBK * 2) + ld_g;
    // (128 * kHalf from the unit counter where registers are short: as a constant it makes the rows'
    // eight addresses loop invariants, which do not fit)
    const int first = HALVES == 2 && NT1 == 2 ? 128 * (h_n & 1) : 128 * kHalf;
    const int c = min(c0 + first + (kPer == 4 ? ld_row : 16 * wave + (lane >> 3)) + 8 * j, C - 1);
#if !defined(COPRIS_LM_PROBE_NO_H_LOADS)
    __builtin_amdgcn_global_load_lds(hbase + (static_cast<uint32_t>(c) * pitch + (koff ^ ((j & 1) * 64))), dst,
                                     16, 0, 0);
#else
    (void)c; (void)koff; (void)dst;
#endif
  };
  auto h_advance = [&]() __attribute__((always_inline)) {
    h_ring = h_ring + 1 == kRingH ? 0 : h_ring + 1;
    if ((HALVES == 1 || (h_n & 1)) && ++h_kd == nkd) h_kd = 0;
    ++h_n;
  };
  auto issue_w = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) w_load(j);
    w_advance();
  };
  using Half0 = std::integral_constant<int, 0>;
  using Half1 = std::integral_constant<int, 1>;
  auto issue_h = [&](auto halfc) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < (decltype(halfc)::value == 1 ? 2 * NT1 : 4); ++j) h_load(j, halfc);
    h_advance();
  };
  // batch row of state i (2*half + nt) of this lane
  auto state_row = [&](int i) __attribute__((always_inline)) {
    return c0 + 128 * (i >> 1) + (i >> 1 ? 32 * NT1 : 64) * wq + 32 * (i & 1) + l32;
  };

  // this lane owns the batch rows state_row(2*half + nt); their stream keys stay in registers (a global load inside the tile loop would drain
  // the prefetch queue)
  constexpr int kStates = HALVES == 1 ? 2 : 2 + NT1;
  LmLaneState st[kStates];
  uint32_t step_c[kStates], sid_lo[kStates], sid_hi[kStates];
#pragma unroll
  for (int i = 0; i < kStates; ++i) {
    st[i] = LmLaneState{-INFINITY, 0.0f, -INFINITY, 0.0f, 0.0f, 0x7fffffff};
    const int c = state_row(i);
    if (GIVEN) {   // step_c holds the row's given token
      step_c[i] = c < c_end ? static_cast<uint32_t>(target[c]) : 0xffffffffu;
      sid_lo[i] = sid_hi[i] = 0;
    } else {
      const uint64_t sid = c < c_end ? static_cast<uint64_t>(seq_id[c]) : 0;
      step_c[i] = c < c_end ? static_cast<uint32_t>(step[c]) : 0;
      sid_lo[i] = static_cast<uint32_t>(sid);
      sid_hi[i] = static_cast<uint32_t>(sid >> 32);
    }
  }

  // prologue = the loads of "slabs -2 and -1".  A wave's loads complete in issue order, and
  // that order is, per slab d: hidden (d+1, half 0), W(d+2) | hidden (d+1, half 1).  So at the
  // top of slab d the wave may leave its newest loads (W(d+1), four, and hidden (d, 1)) in flight
  // and knows hidden (d, 0) has landed; at mid-slab it may leave the eight issued since the
  // top and knows W(d+1) and hidden (d, 1) have.
  // (HALVES = 1: per slab d hidden (d+1), W(d+3); at the top of slab d the newest four loads,
  // W(d+2), may stay in flight and hidden (d), W(d+1) have landed.)
  if (total > 0) {
    if (HALVES == 2) {
      issue_w();
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // W(0): the first slab reads it before any barrier of the loop
      issue_h(Half0{});
      issue_w();
      issue_h(Half1{});
    } else {
      issue_w();
      issue_w();
      issue_h(Half0{});
      issue_w();
      asm volatile("s_waitcnt vmcnt(12)" ::: "memory");  // W(0)
    }
  }
  asm volatile("s_barrier" ::: "memory");

  int ring = 0, hring = 0;                     // W / hidden ring slots being consumed
  for (int tile = place; tile < n_tiles; tile += gridDim.x) {
    const int v0 = tile * kMfBM;
    f32x16 acc[2][2][2];                       // [batch half][it][nt]
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i >> 2][(i >> 1) & 1][i & 1][r] = 0.0f;

    if constexpr (HALVES == 1) {
      for (int kd = 0; kd < nkd; ++kd) {
        const uint32_t wb = lds0 + ring * kSlab;
        ring = ring + 1 == kRingW ? 0 : ring + 1;
        u32x4 a[4][2];
#pragma unroll
        for (int k16 = 0; k16 < 4; ++k16) {
          a[k16][0] = lds_read128<0>(wb + a_off[k16]);
          a[k16][1] = lds_read128<4096>(wb + a_off[k16]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(a[0][0]), "+v"(a[0][1]), "+v"(a[1][0]), "+v"(a[1][1]), "+v"(a[2][0]),
                       "+v"(a[2][1]), "+v"(a[3][0]), "+v"(a[3][1])::"memory");
        // ---- top: hidden unit (d) and W(d+1) have landed; every wave holds W(d)'s operands ----
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        asm volatile("s_barrier" ::: "memory");
        const uint32_t hb = lds0 + kHBase + hring * kSlab;
        hring = hring + 1 == kRingH ? 0 : hring + 1;
        u32x4 b[4][2];
#pragma unroll
        for (int k16 = 0; k16 < 4; ++k16) {
          b[k16][0] = lds_read128<0>(hb + b_off[k16]);
          b[k16][1] = lds_read128<4096>(hb + b_off[k16]);
        }
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) {
          if (grp == 0) {
            asm volatile("s_waitcnt lgkmcnt(4)" : "+v"(b[0][0]), "+v"(b[0][1]), "+v"(b[1][0]), "+v"(b[1][1])::"memory");
          } else {
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(b[2][0]), "+v"(b[2][1]), "+v"(b[3][0]), "+v"(b[3][1])::"memory");
          }
#pragma unroll
          for (int m = 0; m < 8; ++m) {
            const int k16 = 2 * grp + (m >> 2), it = (m >> 1) & 1;
            const bf16x8 fa = __builtin_bit_cast(bf16x8, a[k16][it]);
            const bf16x8 fb = __builtin_bit_cast(bf16x8, b[k16][m & 1]);
            acc[0][it][m & 1] = COPRIS_LM_MFMA(fa, fb, acc[0][it][m & 1]);
            if (m & 1) {   // hidden (d+1) into the slot of (d-1), then W(d+3) into the slot of W(d)
              const int q = 4 * grp + (m >> 1);                                   // 0 .. 7
              __builtin_amdgcn_sched_barrier(0);
              if (q < 4) {
                h_load(q, Half0{});
                if (q == 3) h_advance();
              } else {
                w_load(q - 4);
                if (q == 7) w_advance();
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
    } else
    for (int kd = 0; kd < nkd; ++kd) {
      // The W operands of the slab go to registers BEFORE the top barrier (the slab has been
      // in LDS, for every wave, since the middle barrier of the slab before), so that barrier
      // also says "every wave holds its operands": the slot of W(d) is free from there on and
      // W(d+2) is requested right away - a slab is on its way for a slab and a half although
      // the ring holds only two.
      const uint32_t wb = lds0 + ring * kSlab;
      ring ^= 1;
      u32x4 a[4][2];
#pragma unroll
      for (int k16 = 0; k16 < 4; ++k16) {
        a[k16][0] = lds_read128<0>(wb + a_off[k16]);
        a[k16][1] = lds_read128<4096>(wb + a_off[k16]);
      }
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(a[0][0]), "+v"(a[0][1]), "+v"(a[1][0]), "+v"(a[1][1]), "+v"(a[2][0]),
                     "+v"(a[2][1]), "+v"(a[3][0]), "+v"(a[3][1])::"memory");
      // ---- top: hidden unit (d, half 0) has landed ----
      wait_loads<4 + 2 * NT1>();
      asm volatile("s_barrier" ::: "memory");   // ... for every wave; all are done with slab d-1
      auto half_slab = [&](auto halfc) __attribute__((always_inline)) {
        constexpr int half = decltype(halfc)::value, kNt = half == 1 ? NT1 : 2;
        if (half == 1) {
          // ---- middle: W(d+1) and hidden unit (d, half 1) have landed ----
          wait_loads<8>();
          asm volatile("s_barrier" ::: "memory");             // all are done with unit (d, half 0)
        }
        const uint32_t hb = lds0 + kHBase + hring * kSlab;
        hring = hring + 1 == kRingH ? 0 : hring + 1;
        // all hidden operands of the half at once, then its products in two groups of eight (of
        // four where the half has 64 rows): one wait per group instead of one per four
        u32x4 b[4][kNt];
#pragma unroll
        for (int k16 = 0; k16 < 4; ++k16) {
          b[k16][0] = lds_read128<0>(hb + (half == 1 && NT1 == 1 ? b1_off[k16] : b_off[k16]));
          if constexpr (kNt == 2) b[k16][1] = lds_read128<4096>(hb + (half == 1 && NT1 == 1 ? b1_off[k16] : b_off[k16]));
        }
#pragma unroll
        for (int grp = 0; grp < 2; ++grp) {
          if (grp == 0) lds_wait_b<2 * kNt>(b[0], b[1]);
          else lds_wait_b<0>(b[2], b[3]);
#pragma unroll
          for (int m = 0; m < 4 * kNt; ++m) {
            const int k16 = 2 * grp + m / (2 * kNt), it = m / kNt % 2, nt = m % kNt;
            const bf16x8 fa = __builtin_bit_cast(bf16x8, a[k16][it]);
            const bf16x8 fb = __builtin_bit_cast(bf16x8, b[k16][nt]);
            acc[half][it][nt] = COPRIS_LM_MFMA(fa, fb, acc[half][it][nt]);
            // The loads a wave issues per slab go out one at a time between the products.  Issued
            // in a bunch they keep every wave of the CU at the issue stage while the address unit
            // works through them, and the matrix pipes idle meanwhile; spread out they cost the
            // products nothing.  First half: hidden (d+1, half 0) (its slot is free since the top
            // barrier), then W(d+2) (likewise); second half: hidden (d+1, half 1) (the middle
            // barrier has freed the slot of (d, half 0)).  Past the last slab the loads re-read
            // clamped rows into ring slots nobody reads any more.
            if (half == 0 && (m & 1)) {
              const int q = 4 * grp + (m >> 1);                                   // 0 .. 7
              __builtin_amdgcn_sched_barrier(0);
              if (q < 4) {
                h_load(q, Half0{});
                if (q == 3) h_advance();
              } else {
                w_load(q - 4);
                if (q == 7) w_advance();
              }
              __builtin_amdgcn_sched_barrier(0);
            } else if (half == 1 && m % 4 == 1) {
              const int q = kNt * grp + (m >> 2);                                 // 0 .. 2 * NT1 - 1
              __builtin_amdgcn_sched_barrier(0);
              h_load(q, Half1{});
              if (q == 2 * NT1 - 1) h_advance();
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      };
      half_slab(Half0{});
      half_slab(Half1{});
    }

    const bool tail = v0 + kMfBM > V;   // only the last tile can hold rows past V
    // written out per batch block: the unrolled body is too large for the unroll pragma
    auto epilogue = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;       // state index = 2*half + nt
      const int c = state_row(i);
#if defined(COPRIS_LM_PROBE_NO_EPILOGUE)
      if (c < c_end) {   // keep the accumulators alive, nothing else
        st[i].s += acc[i >> 1][0][i & 1][0] + acc[i >> 1][1][i & 1][15];
        st[i].m = 0.0f;
        st[i].idx = v0;
      } else
#endif
      if (c < c_end && GIVEN) {
        lm_given_block(acc[i >> 1][0][i & 1], st[i], v0 + 64 * wm + 4 * kb, V, tail, scale,
                       static_cast<int>(step_c[i]));
        lm_given_block(acc[i >> 1][1][i & 1], st[i], v0 + 64 * wm + 32 + 4 * kb, V, tail, scale, static_cast<int>(step_c[i]));
      } else if (c < c_end) {
        lm_epilogue_block(acc[i >> 1][0][i & 1], st[i], v0 + 64 * wm + 4 * kb, V, tail, scale, step_c[i], sid_lo[i], sid_hi[i], key0, key1);
        lm_epilogue_block(acc[i >> 1][1][i & 1], st[i], v0 + 64 * wm + 32 + 4 * kb, V, tail, scale, step_c[i], sid_lo[i], sid_hi[i], key0, key1);
      }
    };
    epilogue(std::integral_constant<int, 0>{});
    epilogue(std::integral_constant<int, 1>{});
    if constexpr (HALVES == 2) {
      epilogue(std::integral_constant<int, 2>{});
      if constexpr (NT1 == 2) epilogue(std::integral_constant<int, 3>{});
    }
  }

  // lane state -> partial; combine the two k-halves of a wave, then the two vocabulary
  // halves.  The exchange buffer reuses the ring memory: all slabs have been consumed.
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  LmPartial(*s_part)[kMfBN / 2] = reinterpret_cast<LmPartial(*)[kMfBN / 2]>(smem);
#pragma unroll
  for (int i = 0; i < kStates; ++i) {
    LmPartial p = lane_partial<GIVEN>(st[i], inv_temperature);
    if (wm == 1 && kb == 0) s_part[wq][32 * i + l32] = p;
    __syncthreads();
    if (wm == 0 && kb == 0) {
      combine(p, s_part[wq][32 * i + l32]);
      const int c = state_row(i);
      if (c < c_end) part[static_cast<size_t>(c) * n_parts + blockIdx.x] = p;
    }
    __syncthreads();
  }
}

// --------------------------------------------------------------------------
// matrix-core kernel for at most 64 batch rows.
//
// With so few rows the kernel is its W stream, and what counts is that the stream never stops.
// One workgroup of eight waves per CU takes 32 vocabulary rows per wave against all 32 * NT batch
// rows: [256 rows][64 k] slabs of W (32 KB) and [32 * NT rows][64 k] slabs of the hidden state,
// both in rings of four (all of the CU's LDS).  A CU's loads return in the order they were issued,
// whichever wave issued them, so a hidden slab that is requested later than W but needed sooner
// would drain the W requests with it: both streams run the same four slabs ahead, and two to three
// slabs (64 .. 96 KB of W per CU) stay in flight.  Both operands of a slab go to registers before
// the slab's one barrier, which therefore frees both slots.
// A workgroup owns a contiguous run of `rows` vocabulary rows, the same for all, in tiles of equal
// height: the stream ends everywhere at once and asks for the same bytes per slab throughout
// (128-row tiles dealt out whole leave the last round to a third of the chip).  The rows that a
// tile lacks to 256 re-read its last row (from the cache) and are masked.
// The epilogue of a tile is spread over the slabs of the next one, a Philox block (four vocabulary
// entries of one batch row) at a time: its ~30 vector instructions per entry would otherwise stop
// the workgroup's loads.
// --------------------------------------------------------------------------
// every LDS read of the slab's operands has arrived
template <int NT>
__device__ __forceinline__ void lds_arrived(u32x4 (&a)[4], u32x4 (&b)[4][NT]) {
  asm volatile("s_waitcnt lgkmcnt(0)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0][0]), "+v"(b[1][0]), "+v"(b[2][0]),
                 "+v"(b[3][0])::"memory");
  if constexpr (NT == 2)
    asm volatile("" : "+v"(b[0][1]), "+v"(b[1][1]), "+v"(b[2][1]), "+v"(b[3][1])::"memory");
}

// The accumulators a of vocabulary entries vq .. vq+3 (-inf: none) into the state, with the block's random words from draw().
template <typename Draw>
__device__ __forceinline__ void lm_sample_words(const float (&a)[4], LmLaneState& st, int vq, float scale, const Draw& draw) {
  const float m_new = fmaxf(st.m, fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])));
  if (m_new == -INFINITY) return;
  const float alpha = lm_exp(st.m, m_new, scale);
  st.s *= alpha;
  st.p_best *= alpha;
  st.m = m_new;
  const Philox4 x = draw();
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float p = lm_exp(a[j], m_new, scale);                     // 0 for masked entries
    st.s += p;
    const float l = __builtin_amdgcn_logf(word_to_uniform(w[j]));   // log2(u) < 0
    if (l * st.p_best > st.l_best * p) {                            // (see lm_epilogue_block)
      st.l_best = l;
      st.p_best = p;
      st.a_best = a[j];
      st.idx = vq + j;
    }
  }
}
// One Philox block of a tile: the accumulators of vocabulary entries vq .. vq+3 (vq % 4 == 0),
// of which those at or past v_end are masked where the vocabulary (or a tile) ends inside a block.
__device__ __forceinline__ void lm_sample_quad(float (&a)[4], LmLaneState& st, int vq, int v_end,
                                               bool ragged, float scale, uint32_t step_c, uint32_t sid_lo,
                                               uint32_t sid_hi, uint32_t key0, uint32_t key1) {
  if (ragged) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (vq + j >= v_end) a[j] = -INFINITY;
  }
  lm_sample_words(a, st, vq, scale, [&]() __attribute__((always_inline)) {
    return philox4x32_10(static_cast<uint32_t>(vq) >> 2, step_c, sid_lo, sid_hi, key0, key1);
  });
}
__device__ __forceinline__ void lm_given_quad(float (&a)[4], LmLaneState& st, int vq, int v_end,
                                              bool ragged, float scale, int target) {
  if (ragged) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (vq + j >= v_end) a[j] = -INFINITY;
  }
  const float m_new = fmaxf(st.m, fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])));
  if (m_new == -INFINITY) return;
  float p[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) p[j] = lm_exp(a[j], m_new, scale);
  st.s = st.s * lm_exp(st.m, m_new, scale) + ((p[0] + p[1]) + (p[2] + p[3]));
  st.m = m_new;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (target == vq + j && target < v_end) {
      st.a_best = a[j];
      st.idx = target;
    }
  }
}

constexpr int kSkBM = 256;                             // vocabulary rows per tile, at most
constexpr int kSkMaxGrid = 256;                        // one workgroup per CU
constexpr int kSkRing = 4;
constexpr int kSkSlab = kSkBM * kMfBK * 2;             // 32 KB
constexpr int kSkLds = kSkRing * (kSkSlab + kSkMaxRows * kMfBK * 2);   // 160 KB

template <bool GIVEN, int NT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void lmhead_skinny_kernel(
    const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight,
    const int64_t* __restrict__ seq_id, const int32_t* __restrict__ step,
    const int32_t* __restrict__ target, uint32_t key0, uint32_t key1, float inv_temperature,
    LmPartial* __restrict__ part, int C, int H, int V, int rows, int height, int n_parts) {
  constexpr int kHUnit = 32 * NT * kMfBK * 2;          // bytes of a hidden slab
  constexpr int kHBase = kSkRing * kSkSlab;
  constexpr int kWLoads = 4;                           // loads per wave and slab: W ...
  constexpr int kLoads = kWLoads + 1;                  // ... and hidden
  static_assert(32 * NT <= kSkMaxRows, "rings exceed the workgroup's LDS");
  __shared__ __attribute__((aligned(1024))) char smem[kSkLds];
  const int tid = threadIdx.x, lane = tid & 63;
  const float scale = lm_scale(inv_temperature);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, kb = lane >> 5;
  const int nkd = H / kMfBK;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const uint32_t pitch = static_cast<uint32_t>(H) * 2u;
  const int v_begin = blockIdx.x * rows, v_end = min(v_begin + rows, V);   // (v_begin < V: the launcher's grid)

  uint32_t a_off[4], b_off[4];
#pragma unroll
  for (int k16 = 0; k16 < 4; ++k16) {
    a_off[k16] = lm_swz(32 * wave + l32, 2 * k16 + kb) * 16;
    b_off[k16] = lm_swz(l32, 2 * k16 + kb) * 16;       // a further 32 rows add 4096 bytes
  }

  // this lane owns batch rows 32*nt + l32; their keys are here before the pipeline starts
  LmLaneState st[NT];
  uint32_t step_c[NT], sid_lo[NT], sid_hi[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    st[i] = LmLaneState{-INFINITY, 0.0f, -INFINITY, 0.0f, 0.0f, 0x7fffffff};
    const int c = 32 * i + l32;
    if (GIVEN) {   // step_c holds the row's given token
      step_c[i] = c < C ? static_cast<uint32_t>(target[c]) : 0xffffffffu;
      sid_lo[i] = sid_hi[i] = 0;
    } else {
      const uint64_t sid = c < C ? static_cast<uint64_t>(seq_id[c]) : 0;
      step_c[i] = c < C ? static_cast<uint32_t>(step[c]) : 0;
      sid_lo[i] = static_cast<uint32_t>(sid);
      sid_hi[i] = static_cast<uint32_t>(sid >> 32);
    }
  }

  // ---- loaders: an instruction moves 8 rows x 128 bytes; LDS position 64*chunk + lane holds (row
  // 8*chunk + lane/8, stored granule lane%8), see lm_swz ((row>>1)&7 = lane>>4, +4 in odd chunks)
  const uint32_t ld_g = ((lane & 7) ^ (lane >> 4)) * 16;
  int ld_tile = v_begin, ld_kd = 0, ld_slot = 0;       // cursor of both streams
  const char* wbase = reinterpret_cast<const char*>(weight);
  const char* hbase = reinterpret_cast<const char*>(hidden);
  // W: wave w moves chunks 4w .. 4w+3.  Hidden: chunk w, or w mod 4 where there are only four (two
  // waves then write the same bytes).
  auto load = [&](int j) __attribute__((always_inline)) {
    const uint32_t koff = static_cast<uint32_t>(ld_kd) * (kMfBK * 2) + ld_g;
    if (j < kWLoads) {
      const int chunk = kWLoads * wave + j;
      const int v = min(min(ld_tile + 8 * chunk + (lane >> 3), ld_tile + height - 1), v_end - 1);
      __builtin_amdgcn_global_load_lds(wbase + (static_cast<uint32_t>(v) * pitch + (koff ^ ((j & 1) * 64))),
                                       smem + ld_slot * kSkSlab + chunk * 1024, 16, 0, kLmStreamOnce);
    } else {
      const int chunk = wave & (4 * NT - 1);
      const int c = min(8 * chunk + (lane >> 3), C - 1);           // rows past C duplicate the last row (unused)
      __builtin_amdgcn_global_load_lds(hbase + (static_cast<uint32_t>(c) * pitch + (koff ^ ((chunk & 1) * 64))),
                                       smem + kHBase + ld_slot * kHUnit + chunk * 1024, 16, 0, 0);
    }
  };
  // Past the run's last slab the loads re-read clamped rows into slots nobody reads any more.
  auto advance = [&]() __attribute__((always_inline)) {
    ld_slot = (ld_slot + 1) & (kSkRing - 1);
    if (++ld_kd == nkd) {
      ld_kd = 0;
      ld_tile += height;
    }
  };
  // prologue: the rings are filled; the first slab has landed at the barrier
  for (int d = 0; d < kSkRing; ++d) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) load(j);
    advance();
  }
  wait_loads<(kSkRing - 1) * kLoads>();
  asm volatile("s_barrier" ::: "memory");

  // the finished tile whose epilogue is under way: its accumulators, first row and end
  f32x16 done[NT];
  int done_v0 = v_begin, done_end = v_begin;           // (nothing yet: every entry is masked)
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) done[i][r] = 0.0f;
  constexpr int kPieces = 4 * NT;
  auto piece = [&](auto pc) __attribute__((always_inline)) {
    constexpr int i = decltype(pc)::value / 4, q = decltype(pc)::value % 4;
    const int vq = done_v0 + 32 * wave + 4 * kb + 8 * q;       // accumulators 4q .. 4q+3 of block i
    if (32 * i + l32 < C && vq < done_end) {
      float z[4] = {done[i][4 * q], done[i][4 * q + 1], done[i][4 * q + 2], done[i][4 * q + 3]};
      const bool ragged = (done_end & 3) != 0;
      if (GIVEN) lm_given_quad(z, st[i], vq, done_end, ragged, scale, static_cast<int>(step_c[i]));
      else lm_sample_quad(z, st[i], vq, done_end, ragged, scale, step_c[i], sid_lo[i], sid_hi[i], key0, key1);
    }
  };
  auto pieces = [&](int from, int to) __attribute__((always_inline)) {
    for (int p = from; p < to; ++p) {
      switch (p) {
        case 0: piece(std::integral_constant<int, 0>{}); break;
        case 1: piece(std::integral_constant<int, 1>{}); break;
        case 2: piece(std::integral_constant<int, 2>{}); break;
        case 3: piece(std::integral_constant<int, 3>{}); break;
        case 4: piece(std::integral_constant<int, 4 % kPieces>{}); break;
        case 5: piece(std::integral_constant<int, 5 % kPieces>{}); break;
        case 6: piece(std::integral_constant<int, 6 % kPieces>{}); break;
        case 7: piece(std::integral_constant<int, 7 % kPieces>{}); break;
      }
    }
  };
  const int per_slab = (kPieces + nkd - 1) / nkd;

  int slot = 0;
  for (int v0 = v_begin; v0 < v_end; v0 += height) {
    f32x16 acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.0f;
    for (int kd = 0; kd < nkd; ++kd) {
      const uint32_t wb = lds0 + slot * kSkSlab, hb = lds0 + kHBase + slot * kHUnit;
      slot = (slot + 1) & (kSkRing - 1);
      u32x4 a[4], b[4][NT];
#pragma unroll
      for (int k16 = 0; k16 < 4; ++k16) {
        a[k16] = lds_read128<0>(wb + a_off[k16]);
        b[k16][0] = lds_read128<0>(hb + b_off[k16]);
        if (NT == 2) b[k16][NT - 1] = lds_read128<4096>(hb + b_off[k16]);
      }
      lds_arrived(a, b);
      // the next slab has landed (the two after it may be in flight) ...
      wait_loads<(kSkRing - 2) * kLoads>();
      asm volatile("s_barrier" ::: "memory");   // ... for every wave, and all hold this slab's operands
      // the loads into the freed slot go out between the products
#pragma unroll
      for (int m = 0; m < 4 * NT; ++m) {
        const int k16 = m / NT, nt = m % NT;
        acc[nt] = COPRIS_LM_MFMA(__builtin_bit_cast(bf16x8, a[k16]), __builtin_bit_cast(bf16x8, b[k16][nt]), acc[nt]);
        __builtin_amdgcn_sched_barrier(0);
        if (NT == 1 || m < kLoads) load(m);
        if (NT == 1 && m == 3) load(4);
        __builtin_amdgcn_sched_barrier(0);
      }
      advance();
      const int first = kd * per_slab;
      if (first < kPieces) pieces(first, min(first + per_slab, kPieces));
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) done[i] = acc[i];
    done_v0 = v0;
    done_end = min(v0 + height, v_end);
  }
  // the last tile's epilogue has nothing to hide behind: a block at a time, which leaves the
  // compiler sixteen entries to interleave
  const bool tail = done_v0 + 32 * wave + 32 > done_end;
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    if (32 * i + l32 < C) {
      const int vbase = done_v0 + 32 * wave + 4 * kb;
      if (GIVEN) {
        lm_given_block(done[i], st[i], vbase, done_end, tail, scale, static_cast<int>(step_c[i]));
      } else {
        lm_epilogue_block(done[i], st[i], vbase, done_end, tail, scale, step_c[i], sid_lo[i], sid_hi[i],
                          key0, key1);
      }
    }
  }

  // lane state -> partial; combine the two k-halves of a wave, then the waves' vocabulary
  // rows.  The exchange buffer reuses the ring memory: all slabs have been consumed.
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  LmPartial(*s_part)[32 * NT] = reinterpret_cast<LmPartial(*)[32 * NT]>(smem);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    LmPartial p = lane_partial<GIVEN>(st[i], inv_temperature);
    if (kb == 0) s_part[wave][32 * i + l32] = p;
  }
  __syncthreads();
  if (tid < 32 * NT && tid < C) {
    LmPartial p = s_part[0][tid];
    for (int w = 1; w < 8; ++w) combine(p, s_part[w][tid]);
    part[static_cast<size_t>(tid) * n_parts + blockIdx.x] = p;
  }
}

// --------------------------------------------------------------------------
// matrix-core kernel for micro-batches of given tokens (many row blocks).
//
// With hundreds of row blocks the work is a plain dense contraction and what counts is
// bytes moved into LDS per flop.  One 8-wave workgroup per CU owns a 256 (vocab) x 256
// (batch) tile - 64 KB of operands per 64-wide slab of the hidden dimension instead of
// the 96 KB that two 128 x 256 workgroups move for the same flops - and the whole 160 KB
// of LDS is one pipeline: W slabs [256][64] in a ring of three (issued three slabs ahead),
// hidden slabs [256][64] in a ring of two.  Every wave issues its eighth of both slabs,
// the hidden part first, so that its in-order load counter can wait for the hidden slab
// while the younger W slab stays in flight.  The one barrier per slab sits before the last
// eight products of the slab, after all of the slab's LDS reads: the refill and the first
// operand reads of the next slab are issued there and overlap those products.
// No sampler here: the epilogue is the running log-sum-exp and the given token's logit.
// --------------------------------------------------------------------------
constexpr int kGmBM = 256;                          // vocabulary rows per tile
constexpr int kGmBN = 256;                          // batch rows per workgroup
constexpr int kGmSlab = 256 * kMfBK * 2;            // 32 KB
constexpr int kGmNW = 3;                            // W ring slabs (issued three ahead)
constexpr int kGmNH = 2;                            // hidden ring slabs
constexpr int kGmHRing = kGmNW * kGmSlab;           // the hidden ring starts here
constexpr int kGmLds = kGmHRing + kGmNH * kGmSlab;  // 160 KB
constexpr int kGmMinRows = 384;                     // below this the 128-row kernel is used

template <int N>
__device__ __forceinline__ void lds_wait6(u32x4 (&a)[4], u32x4 (&b)[2]) {
  asm volatile("s_waitcnt lgkmcnt(%6)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1])
               : "n"(N)
               : "memory");
}

// lane_id: which run of lane_units * 64 vocabulary rows; c0: the block's first batch row.
__device__ __forceinline__ void lm_gemm_given_body(
    char* __restrict__ smem, const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight,
    const int32_t* __restrict__ target, float inv_temperature, LmPartial* __restrict__ part, int c0, int C, int H, int V,
    int lane_id, int lane_units, int n_parts) {
  const int tid = threadIdx.x, lane = tid & 63;
  const float scale = lm_scale(inv_temperature);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wq = wave & 3;     // vocabulary rows 64*rb + 32*wm ..; 64-row batch block
  const int l32 = lane & 31, kb = lane >> 5;
  const int nkd = H / kMfBK;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const uint32_t pitch = static_cast<uint32_t>(H) * 2u;

  // A lane owns a contiguous run of lane_units * 64 vocabulary rows, the same for all (the last
  // one's may be shorter): whole tiles, then one of one to three row blocks of 64 where they are left.
  // Dealt out as whole tiles the last round would run as long as any other: 2.5 rounds instead of 3
  // at M = 2000, V = 20011 and 9.5 instead of 10 at M = 777, V = 151936.
  const int v_begin = lane_id * lane_units * 64, v_end = min(v_begin + lane_units * 64, V);

  // operand read offsets inside a slab (bytes); each further row block of W adds 64 rows = 8192
  // bytes, of the hidden state 32 rows = 4096
  uint32_t a_off[4], b_off[4];
#pragma unroll
  for (int k16 = 0; k16 < 4; ++k16) {
    a_off[k16] = lm_swz(32 * wm + l32, 2 * k16 + kb) * 16;
    b_off[k16] = lm_swz(64 * wq + l32, 2 * k16 + kb) * 16;
  }

  // ---- loader cursors (wave-uniform).  Wave w moves rows 32w .. 32w+31 of every slab:
  // four instructions of 8 rows x 128 bytes; LDS position 64*chunk + lane holds (row
  // 8*chunk + lane/8, stored granule lane%8) and the lane fetches the global granule the
  // swizzle maps there ((row>>1)&7 = lane>>4 for even chunks, +4 for odd ones).
  const int total = (v_end - v_begin + kGmBM - 1) / kGmBM * nkd;   // slabs this workgroup consumes
  const int ld_row = 32 * wave + (lane >> 3);
  const uint32_t ld_g = ((lane & 7) ^ (lane >> 4)) * 16;
  int w_row = v_begin, w_kd = 0, w_slot = 0;
  int h_kd = 0, h_slot = 0;
  const char* wbase = reinterpret_cast<const char*>(weight);
  const char* hbase = reinterpret_cast<const char*>(hidden);
  // one of the four loads of this wave's eighth of the W / hidden slab at the cursor
  auto w_load = [&](int j) __attribute__((always_inline)) {
    char* dst = smem + w_slot * kGmSlab + (4 * wave + j) * 1024;
    const uint32_t koff = static_cast<uint32_t>(w_kd) * (kMfBK * 2) + ld_g;
    const int v = min(w_row + ld_row + 8 * j, v_end - 1);   // rows past the run re-read its last row (masked or skipped later)
    __builtin_amdgcn_global_load_lds(wbase + (static_cast<uint32_t>(v) * pitch + (koff ^ ((j & 1) * 64))), dst,
                                     16, 0, 0);
  };
  auto w_advance = [&]() __attribute__((always_inline)) {
    w_slot = w_slot + 1 == kGmNW ? 0 : w_slot + 1;
    if (++w_kd == nkd) {
      w_kd = 0;
      w_row += kGmBM;
    }
  };
  auto h_load = [&](int j) __attribute__((always_inline)) {
    char* dst = smem + kGmHRing + h_slot * kGmSlab + (4 * wave + j) * 1024;
    const uint32_t koff = static_cast<uint32_t>(h_kd) * (kMfBK * 2) + ld_g;
    const int c = min(c0 + ld_row + 8 * j, C - 1);               // rows past C duplicate the last row (unused)
    __builtin_amdgcn_global_load_lds(hbase + (static_cast<uint32_t>(c) * pitch + (koff ^ ((j & 1) * 64))), dst,
                                     16, 0, 0);
  };
  auto h_advance = [&]() __attribute__((always_inline)) {
    h_slot = h_slot + 1 == kGmNH ? 0 : h_slot + 1;
    if (++h_kd == nkd) h_kd = 0;
  };
  // Load k (0..7) of the set a barrier opens: the hidden slab first, then the W slab.  Past the workgroup's last slab the loads re-read clamped rows into ring slots
  // nobody reads any more, so none of them needs a condition.
  auto load_one = [&](int k) __attribute__((always_inline)) {
    if (k < 4) {
      h_load(k & 3);
      if ((k & 3) == 3) h_advance();
    } else {
      w_load(k & 3);
      if ((k & 3) == 3) w_advance();
    }
  };

  // this lane owns batch rows c0 + 64*wq + 32*nt + l32; their given tokens are fetched
  // before the pipeline starts (the prologue's wait covers them)
  LmLaneState st[2];
  int tgt[2];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    st[nt] = LmLaneState{-INFINITY, 0.0f, -INFINITY, 0.0f, 0.0f, 0x7fffffff};
    const int c = c0 + 64 * wq + 32 * nt + l32;
    tgt[nt] = c < C ? target[c] : -1;
  }

  // prologue: slab 0 of both streams and slab 1 of W land; then the steady order
  // begins - after the barrier that ends slab d, the hidden slab d+2 and the W
  // slab d+3 go out, one load at a time between the matrix products of the next 32
  // (issued in a bunch they keep all eight waves at the issue stage while the address unit
  // works through them, and the matrix pipes idle).  The first two loads of the set that the
  // prologue's barrier opens go out here, the other six with the products of slab 0.
  for (int k = 0; k < 4; ++k) load_one(k);          // hidden slab 0
  for (int k = 4; k < 8; ++k) load_one(k);          // W slab 0
  for (int k = 4; k < 8; ++k) load_one(k);          // W slab 1
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  load_one(0);
  load_one(1);

  u32x4 a[2][4], b[2][2];
  int wslot = 0, hslot = 0;                     // ring slots of the slab being consumed
  uint32_t wb = lds0, hb = lds0 + kGmHRing;
  auto read_operands = [&](auto bufc, auto k16c) __attribute__((always_inline)) {
    constexpr int buf = decltype(bufc)::value, k16 = decltype(k16c)::value;
    a[buf][0] = lds_read128<0>(wb + a_off[k16]);
    a[buf][1] = lds_read128<8192>(wb + a_off[k16]);
    a[buf][2] = lds_read128<16384>(wb + a_off[k16]);
    a[buf][3] = lds_read128<24576>(wb + a_off[k16]);
    b[buf][0] = lds_read128<0>(hb + b_off[k16]);
    b[buf][1] = lds_read128<4096>(hb + b_off[k16]);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  read_operands(I0{}, I0{});
  // they arrive before the loop begins, and a next tile's before its epilogue: where a tile's loops begin the compiler may
  // move them to other registers, which it must not do with a read under way
  lds_wait6<0>(a[0], b[0]);

  int d = 0;
  for (int v0 = v_begin; v0 < v_end; v0 += kGmBM) {
    const int blocks = min(4, (v_end - v0 + 63) / 64);     // row blocks of the tile
    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i >> 1][i & 1][r] = 0.0f;
    // eight products from operand buffer `buf` (two per row block); if `issue`, loads FIRST and
    // FIRST+1 of the open set go out after the second and the sixth of them
    auto products = [&](auto fullc, auto bufc, auto firstc, const bool issue) __attribute__((always_inline)) {
      constexpr bool kFull = decltype(fullc)::value;
      constexpr int buf = decltype(bufc)::value, kFirst = decltype(firstc)::value;
      const bf16x8 fb0 = __builtin_bit_cast(bf16x8, b[buf][0]);
      const bf16x8 fb1 = __builtin_bit_cast(bf16x8, b[buf][1]);
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        const bf16x8 fa = __builtin_bit_cast(bf16x8, a[buf][rb]);
        if (kFull || rb < blocks) {
          acc[rb][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb0, acc[rb][0], 0, 0, 0);
          acc[rb][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb1, acc[rb][1], 0, 0, 0);
        }
        if (rb == 0 || rb == 2) {
          __builtin_amdgcn_sched_barrier(0);
          if (issue) load_one(kFirst + (rb >> 1));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    using L0 = std::integral_constant<int, 0>;
    using L2 = std::integral_constant<int, 2>;
    using L4 = std::integral_constant<int, 4>;
    using L6 = std::integral_constant<int, 6>;

    auto slabs = [&](auto fullc) __attribute__((always_inline)) {
    for (int kd = 0; kd < nkd; ++kd, ++d) {
      read_operands(I1{}, I1{});
      lds_wait6<6>(a[0], b[0]);
      products(fullc, I0{}, L2{}, true);
      read_operands(I0{}, I2{});
      lds_wait6<6>(a[1], b[1]);
      products(fullc, I1{}, L4{}, true);
      read_operands(I1{}, I3{});
      lds_wait6<6>(a[0], b[0]);
      products(fullc, I0{}, L6{}, true);
      // every LDS read of slab d is complete; the other operand buffer is tied as well so
      // that the products just issued from it stay above this wait
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(a[1][0]), "+v"(a[1][1]), "+v"(a[1][2]), "+v"(a[1][3]), "+v"(b[1][0]),
                     "+v"(b[1][1]), "+v"(a[0][0]), "+v"(a[0][1]), "+v"(a[0][2]), "+v"(a[0][3]),
                     "+v"(b[0][0]), "+v"(b[0][1])::"memory");
      const bool more = d + 1 < total;
      if (more) {
        // slab d+1 has landed (this wave's part: only W slab d+2, the newest
        // four loads, is younger) ...
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        asm volatile("s_barrier" ::: "memory");   // ... for every wave, and all are done reading slab d
        wslot = wslot + 1 == kGmNW ? 0 : wslot + 1;
        hslot = hslot + 1 == kGmNH ? 0 : hslot + 1;
        wb = lds0 + wslot * kGmSlab;
        hb = lds0 + kGmHRing + hslot * kGmSlab;
        read_operands(I0{}, I0{});                // first operands of slab d+1, under the products below
      }
      products(fullc, I1{}, L0{}, more);                 // with the first two loads into the slots of slab d
    }
    };
    if (blocks == 4) slabs(std::true_type{});
    else slabs(std::false_type{});
    lds_wait6<0>(a[0], b[0]);   // (as before the loop)

    const bool tail = v0 + kGmBM > v_end;   // only a run's last tile can hold rows past it
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const int c = c0 + 64 * wq + 32 * nt + l32;
      if (c < C) {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
          if (rb < blocks)
            lm_given_block(acc[rb][nt], st[nt], v0 + 64 * rb + 32 * wm + 4 * kb, v_end, tail, scale,
                           tgt[nt]);
      }
    }
  }

  // lane state -> partial; combine the two k-halves of a wave, then the two vocabulary
  // halves.  The exchange buffer reuses the ring memory: all slabs have been consumed.
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  LmPartial(*s_part)[64] = reinterpret_cast<LmPartial(*)[64]>(smem);
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    LmPartial p = lane_partial<true>(st[nt], inv_temperature);
    if (wm == 1 && kb == 0) s_part[wq][32 * nt + l32] = p;
    __syncthreads();
    if (wm == 0 && kb == 0) {
      combine(p, s_part[wq][32 * nt + l32]);
      const int c = c0 + 64 * wq + 32 * nt + l32;
      if (c < C) part[static_cast<size_t>(c) * n_parts + lane_id] = p;
    }
    __syncthreads();
  }
}

// --------------------------------------------------------------------------
// matrix-core kernel for 65 .. 640 batch rows whose W stream fills whole tiles (lm_run_width).
//
// One workgroup of eight waves per CU multiplies 256 vocabulary rows, 32 per wave, by a block of
// 128 .. 320 batch rows, and owns an equal contiguous run of vocabulary rows.  Per 64-deep slab of the hidden
// dimension a CU moves 32 KB of W and 128 bytes per batch row: at 320 rows 288 bytes per vocabulary row, where
// two workgroups of 128 x 192 move 512 for 384.
// What bounded the tiles is how early a slab of W can be requested.  A CU's loads return in the order they
// were issued, so a slab of W that is requested before a hidden slab has to land before it, and its lead is
// what the hidden slab's is: with rings of three (W) and two (hidden) slabs, the hidden one first, a slab takes 2.0 us
// (HBM latency under load 2.2), with two and two at 320 rows 2.5.  Therefore:
//   W        private to a wave: its 32 rows of a slab go to its registers (16) when the slab begins, and the
//            request for the slab kRingW later goes into the same 4 KB right away, without a barrier;
//   hidden   in the rest of the LDS, three or four slabs deep; at 320 rows there is room for two, and a slab's hidden
//            part is requested before its W, so that what the next slab waits for has only the W of a slab earlier ahead of it.
// A slab takes 1.9 us at 320 rows, 2000 of 3700 cycles of it products; a wave waits for its loads less than 1 % of its
// time, at barriers a sixth.  With all waves on whole columns a hidden operand is read from LDS by every wave,
// 36 reads of 1 KB per 32 products at 256 rows: a third of the LDS's time.  At H = 3584 the products leave the board at
// its power cap (1.6 - 1.7 GHz on normal data).
// Both operands come by buffer loads: rows past the run or past C are out of range, move nothing and read
// as zeros, whose products draw less power than those of a repeated row (2 - 5 % of the time where a third is padding).
// A run's last tile of at most 128 rows is shared out differently: four waves along the vocabulary, two along the
// columns (SPLIT; 0.7 of a whole tile's time, 1.1 with four idle waves).
// The sampler follows a tile's last slab; the rows' states stay in the lanes where registers allow it, else
// they go to one thread per batch row through the slot of the tile's last hidden slab.
// Whole sampling calls in us, tiles of 128 rows / run kernel:
//   C = 280, H = 2048, V = 50257    113.3 /  85.1       C = 320, H = 3584, V = 151936   485.4 / 352.3
//   C = 160, H = 3584, V =  45000    98.5 /  75.2       C = 100, H = 3584, V =  50257    83.2 /  69.8
//   C = 256, H = 2048, V =  50257    79.9 /  72.4       C = 320, H = 1536, V =  20000    50.0 /  40.4
// --------------------------------------------------------------------------
constexpr int kRunBM = 256;                           // vocabulary rows per tile, 32 per wave
constexpr int kRunSlab = kRunBM * kMfBK * 2;          // 32 KB: a slab of W

// f(0), f(1), ... f(N - 1) with constants
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
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
template <int POLICY>
__device__ __forceinline__ void buffer_load_lds16(BufferRsrc rsrc, char* dst, uint32_t offset) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, dst, 16, offset, 0, 0, POLICY);
#else
  (void)rsrc; (void)dst; (void)offset;
#endif
}

// 16 bytes per lane from `offset` + `at`
__device__ __forceinline__ u32x4 buffer_load16(BufferRsrc rsrc, uint32_t offset, int at) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_raw_buffer_load_b128(rsrc, static_cast<int>(offset), at, 0);
#else
  (void)rsrc; (void)offset; (void)at;
  return u32x4{};
#endif
}

// A register that an LDS read fills: no use of it moves above this point.
__device__ __forceinline__ void tie(u32x4& x) { asm volatile("" : "+v"(x)::"memory"); }

// NT blocks of 32 batch rows, products in groups of GN blocks; ring slots of W slabs and of hidden slabs.
template <int NT, int GN, int RW, int RH>
struct LmRun {
  static constexpr int kNT = NT, kGN = GN, kRingW = RW, kRingH = RH;
  static constexpr int kCols = 32 * NT;
  static constexpr int kHSlab = kCols * kMfBK * 2;         // bytes of a hidden slab
  static constexpr int kGroups = 4 * NT / GN;              // groups of products per slab
  static constexpr int kHLoads = (NT + 1) / 2, kWLoads = 4, kLoads = kHLoads + kWLoads;   // per wave and slab
  static constexpr int kHBase = RW * kRunSlab;
  static constexpr bool kCarry = NT <= 6;
  static constexpr bool kSplits = NT % 2 == 0;             // tiles of at most 128 rows share the columns out as well
  static constexpr bool kKeysInLds = NT > 8;
  static constexpr int kKeyBase = kHBase + RH * kHSlab;
  static constexpr int kLds = kKeyBase + (kKeysInLds ? kCols * 16 : 0);
  // waves that can hand their rows' states over at a time (20 bytes each) in a hidden slab's slot
  static constexpr int kFlushWaves = kHSlab / (kCols * 20) >= 8 ? 8 : (kHSlab / (kCols * 20) >= 4 ? 4 : 2);
  // The set of loads of slab d is W(d + RW) and hidden (d + RH - 1), W first unless the hidden ring is shallow.  When
  // slab d + 1 begins, hidden (d + 1) of set d + 2 - RH and W(d + 1) of set d + 1 - RW have to have landed: this many newer
  // loads may still be in flight.
  static constexpr bool kHFirst = RH == 2;
  static constexpr int kInFlightH = (RH - 2) * kLoads + (kHFirst ? kWLoads : 0);
  static constexpr int kInFlightW = (RW - 1) * kLoads + (kHFirst ? 0 : kHLoads);
  static constexpr int kInFlight = kInFlightH < kInFlightW ? kInFlightH : kInFlightW;
  static_assert((kHFirst ? RW == 2 : RW <= RH - 1 && RH <= RW + 2) && NT % GN == 0 && kGroups % 2 == 0 && kLds <= 160 * 1024,
                "rings: the sets before the first slab have to be whole where they are counted");
};
using LmRun128 = LmRun<4, 4, 3, 4>;
using LmRun160 = LmRun<5, 5, 2, 4>;
using LmRun192 = LmRun<6, 3, 2, 4>;
using LmRun256 = LmRun<8, 4, 2, 3>;
using LmRun320 = LmRun<10, 5, 2, 2>;


// lane_id: which run of lane_rows vocabulary rows; c0: the block's first batch row.
template <bool GIVEN, typename S>
__device__ __forceinline__ void lm_run_body(
    char* __restrict__ smem, const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight,
    const int64_t* __restrict__ seq_id, const int32_t* __restrict__ step, const int32_t* __restrict__ target, uint32_t key0,
    uint32_t key1, float inv_temperature, LmPartial* __restrict__ part, int c0, int C, int H, int V, int lane_id,
    int lane_rows, int n_parts) {
  constexpr int NT = S::kNT, GN = S::kGN, GPK = NT / GN;
  const int tid = threadIdx.x, lane = tid & 63;
  const float scale = lm_scale(inv_temperature);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, kb = lane >> 5;
  const int nkd = H / kMfBK;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const uint32_t pitch = static_cast<uint32_t>(H) * 2u;
  const int v_begin = lane_id * lane_rows, v_end = min(v_begin + lane_rows, V);

  // operand read addresses in the first slot of either ring; a further block of 32 batch rows adds 4096 bytes
  uint32_t a_off[4], b_off[4];
#pragma unroll
  for (int k16 = 0; k16 < 4; ++k16) {
    a_off[k16] = lds0 + lm_swz(32 * wave + l32, 2 * k16 + kb) * 16;
    b_off[k16] = lds0 + S::kHBase + lm_swz(l32, 2 * k16 + kb) * 16;
  }

  // this lane's batch rows are c0 + 32*nt + l32; their keys (or given tokens, in key_a) are here before the
  // pipeline starts, in registers or, where there are too many, in LDS
  LmLaneState st[S::kCarry ? NT : 1];
  uint32_t key_a[S::kKeysInLds ? 1 : NT], sid_lo[S::kKeysInLds ? 1 : NT], sid_hi[S::kKeysInLds ? 1 : NT];
  auto fetch_keys = [&](int c, uint32_t& ka, uint32_t& lo, uint32_t& hi) __attribute__((always_inline)) {
    ka = GIVEN ? 0xffffffffu : 0u;
    lo = hi = 0;
    if (c < C) {
      if (GIVEN) {
        ka = static_cast<uint32_t>(target[c]);
      } else {
        const uint64_t sid = static_cast<uint64_t>(seq_id[c]);
        ka = static_cast<uint32_t>(step[c]);
        lo = static_cast<uint32_t>(sid);
        hi = static_cast<uint32_t>(sid >> 32);
      }
    }
  };
  if constexpr (S::kKeysInLds) {
    if (tid < S::kCols) {
      u32x4 kv = {0, 0, 0, 0};
      uint32_t ka, lo, hi;
      fetch_keys(c0 + tid, ka, lo, hi);
      kv[0] = ka; kv[1] = lo; kv[2] = hi;
      reinterpret_cast<u32x4*>(smem + S::kKeyBase)[tid] = kv;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  } else {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      fetch_keys(c0 + 32 * nt + l32, key_a[nt], sid_lo[nt], sid_hi[nt]);
      asm volatile("" : "+v"(key_a[nt]), "+v"(sid_lo[nt]), "+v"(sid_hi[nt]));
    }
  }
#pragma unroll
  for (int nt = 0; nt < (S::kCarry ? NT : 1); ++nt) st[nt] = LmLaneState{-INFINITY, 0.0f, -INFINITY, 0.0f, 0.0f, 0x7fffffff};
  LmPartial mine = empty_partial();   // !kCarry: thread i owns the state of batch row i between tiles

  // ---- loader cursors (wave-uniform).  An instruction moves 8 rows x 128 bytes; LDS position 64*chunk + lane holds
  // (row 8*chunk + lane/8, stored granule lane%8), see lm_swz ((row>>1)&7 = lane>>4, +4 in odd chunks).
  // W: chunks 4w .. 4w+3 of a slab by wave w, its own rows.  Hidden: chunks w, 8 + w, ...
  const uint32_t ld_gw = ((lane & 7) ^ (lane >> 4)) * 16;
  const uint32_t ld_gh = ld_gw ^ (64 * (wave & 1));
  int w_row = v_begin, w_kd = 0, w_slot = 0;
  auto split_tile = [&](int v0) __attribute__((always_inline)) {   // the tile at v0 is shared out by columns as well
    return S::kSplits && v_end - v0 <= kRunBM / 2 && v0 < v_end; };
  int w_up = split_tile(v_begin) ? 32 * (wave & 4) : 0;   // the rows that the wave's lie above their place in a whole tile
  int h_kd = 0, h_slot = 0;
  // (a row past the run, or past C, is out of its buffer's range)
  const BufferRsrc wrsrc = buffer_rsrc(weight, static_cast<uint32_t>(v_end) * pitch);
  const BufferRsrc hrsrc = buffer_rsrc(hidden, static_cast<uint32_t>(C) * pitch);
  // (a lane's offset in the first two W loads and in the first hidden load; the other loads' rows follow at
  // distances that are the same for the whole wave)
  const uint32_t w_off0 = static_cast<uint32_t>(32 * wave + (lane >> 3)) * pitch + ld_gw;
  const uint32_t w_off1 = static_cast<uint32_t>(32 * wave + 8 + (lane >> 3)) * pitch + (ld_gw ^ 64);
  const uint32_t h_off = static_cast<uint32_t>(c0 + 8 * wave + (lane >> 3)) * pitch + ld_gh;
  auto w_load = [&](int j) __attribute__((always_inline)) {
    char* dst = smem + w_slot * kRunSlab + (4 * wave + j) * 1024;
    const uint32_t at = static_cast<uint32_t>(w_row - w_up + 16 * (j >> 1)) * pitch + static_cast<uint32_t>(w_kd) * (kMfBK * 2);
    buffer_load_lds16<kLmStreamOnce>(wrsrc, dst, ((j & 1) ? w_off1 : w_off0) + at);
    if (j == 3) {
      w_slot = w_slot + 1 == S::kRingW ? 0 : w_slot + 1;
      if (++w_kd == nkd) {
        w_kd = 0;
        w_row += kRunBM;
        w_up = split_tile(w_row) ? 32 * (wave & 4) : 0;
      }
    }
  };
  auto h_load = [&](int j) __attribute__((always_inline)) {
    // (an odd number of 32-row blocks leaves half a load: two waves move the same rows)
    const int chunk = 8 * j + (2 * j + 1 == NT ? (wave & 3) : wave);
    char* dst = smem + S::kHBase + h_slot * S::kHSlab + chunk * 1024;
    const uint32_t at = static_cast<uint32_t>(8 * (chunk - wave)) * pitch + static_cast<uint32_t>(h_kd) * (kMfBK * 2);
    buffer_load_lds16<0>(hrsrc, dst, h_off + at);
    if (j == S::kHLoads - 1) {
      h_slot = h_slot + 1 == S::kRingH ? 0 : h_slot + 1;
      if (++h_kd == nkd) h_kd = 0;
    }
  };
  // load i of a slab's set
  auto load_one = [&](int i) __attribute__((always_inline)) {
    if (S::kHFirst ? i >= S::kHLoads : i < S::kWLoads) w_load(S::kHFirst ? i - S::kHLoads : i);
    else h_load(S::kHFirst ? i : i - S::kWLoads);
  };

  // prologue: the sets of the slabs before the first one, as far as there is something in them
  {
    constexpr int kFirst = S::kRingW > S::kRingH - 1 ? S::kRingW : S::kRingH - 1;
    static_for<kFirst>([&](auto vc) __attribute__((always_inline)) {
      constexpr int v = decltype(vc)::value - kFirst;
      constexpr bool kW = v >= -S::kRingW, kH = v - 1 + S::kRingH >= 0;
      for (int i = 0; i < S::kLoads; ++i) {
        const bool hidden_part = S::kHFirst ? i < S::kHLoads : i >= S::kWLoads;
        if (hidden_part ? kH : kW) load_one(i);
      }
    });
  }

  u32x4 a[4], b[2][GN];
  int wslot = S::kRingW - 1, hslot = S::kRingH - 1;             // ring slots of the slab being consumed (advanced on entry)
  uint32_t wb = 0, hb = 0;
  f32x16 acc[NT];
  // what a wave does in a tile: nothing but its loads; its 32 rows by all columns; its 32 of 128 rows by half of them
  using Idle = std::integral_constant<int, 0>;
  using Whole = std::integral_constant<int, 1>;
  using Split = std::integral_constant<int, 2>;
  // group g of a slab's products: column blocks n0 .. n0 + count - 1 of depth 16 * k16
  auto read_b = [&](auto modec, auto gc) __attribute__((always_inline)) {
    constexpr bool kSplit = decltype(modec)::value == 2;
    constexpr int g = decltype(gc)::value, per = kSplit ? 1 : GPK, n = kSplit ? NT / 2 : GN, k16 = g / per, n0 = g % per * n;
    static_for<n>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      b[g & 1][i] = lds_read128<(n0 + i) * 4096>(hb + b_off[k16]);
    });
  };
  auto read_a = [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    a[k] = lds_read128<0>(wb + a_off[k]);
  };
  // operand buffer `buf` has arrived (and the operands `k` of W), N later LDS reads may be under way
  auto arrived = [&](auto bufc, auto kc, auto nc) __attribute__((always_inline)) {
    constexpr int buf = decltype(bufc)::value, k = decltype(kc)::value, n = decltype(nc)::value;
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(n) : "memory");
#pragma unroll
    for (int i = 0; i < GN; ++i) tie(b[buf][i]);
    tie(a[k]);
  };
  using I0 = std::integral_constant<int, 0>;
  // the next slab: it has landed for every wave, which are all done with the one before it
  auto enter = [&](auto modec, uint32_t columns) __attribute__((always_inline)) {
    wait_loads<S::kInFlight>();
    asm volatile("s_barrier" ::: "memory");
    hslot = hslot + 1 == S::kRingH ? 0 : hslot + 1;
    hb = hslot * S::kHSlab + columns;
    wslot = wslot + 1 == S::kRingW ? 0 : wslot + 1;
    wb = wslot * kRunSlab;
    if constexpr (decltype(modec)::value != 0) {
      static_for<3>(read_a);
      read_b(modec, I0{});
    }
  };
  for (int v0 = v_begin; v0 < v_end; v0 += kRunBM) {
    const bool split = split_tile(v0);
    const int vw = v0 + 32 * (split ? wave & 3 : wave);   // the wave's first row in this tile ...
    const bool active = vw < v_end;                       // ... if it has one
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.0f;
    auto slabs = [&](auto modec) __attribute__((always_inline)) {
      constexpr int kMode = decltype(modec)::value;
      constexpr bool kSplit = kMode == 2;
      constexpr int per = kSplit ? 1 : GPK, n = kSplit ? NT / 2 : GN, groups = 4 * per;
      const uint32_t columns = kSplit ? static_cast<uint32_t>(wave >> 2) * (NT / 2 * 4096) : 0;
      enter(modec, columns);
      if constexpr (kMode != 0) {
        arrived(I0{}, I0{}, I0{});
        tie(a[1]);
        tie(a[2]);
      }
      for (int kd = 0; kd < nkd; ++kd) {
        // group g's products; the set's loads go out between those of all groups but the last
        auto products = [&](auto gc) __attribute__((always_inline)) {
          constexpr int g = decltype(gc)::value, k16 = g / per, n0 = g % per * n;
          constexpr int P = (groups - 1) * n, L = S::kLoads;
#pragma unroll
          for (int m = 0; m < n; ++m) {
            if (kMode != 0)
              acc[n0 + m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[k16]),
                                                                    __builtin_bit_cast(bf16x8, b[g & 1][m]), acc[n0 + m], 0, 0, 0);
            if (g < groups - 1) {
#pragma unroll
              for (int i = 0; i < L; ++i)
                if (g * n + m == (2 * i + 1) * P / (2 * L)) {
                  __builtin_amdgcn_sched_barrier(0);
                  load_one(i);
                  __builtin_amdgcn_sched_barrier(0);
                }
            }
          }
        };
        static_for<groups - 1>([&](auto gc) __attribute__((always_inline)) {
          constexpr int g = decltype(gc)::value;
          if constexpr (kMode != 0) {
            if constexpr (g == 0) read_a(std::integral_constant<int, 3>{});
            read_b(modec, std::integral_constant<int, g + 1>{});
            arrived(std::integral_constant<int, (g & 1)>{}, std::integral_constant<int, g / per>{}, std::integral_constant<int, n>{});
            if constexpr (g == 0) {
              tie(a[1]);
              tie(a[2]);
              tie(a[3]);
            }
          }
          products(gc);
        });
        if constexpr (kMode != 0) arrived(std::integral_constant<int, 1>{}, std::integral_constant<int, 3>{}, I0{});
        // every operand of this slab is in registers; the last group is multiplied under the next slab's first reads
        if (kd + 1 < nkd) enter(modec, columns);
        products(std::integral_constant<int, groups - 1>{});
      }
    };
    if (!active) slabs(Idle{});
    else if (!S::kSplits || !split) slabs(Whole{});
    else {
      if constexpr (S::kSplits) {
        slabs(Split{});
        if (wave & 4) {   // its columns are the upper half
#pragma unroll
          for (int i = 0; i < NT / 2; ++i) acc[NT / 2 + i] = acc[i];
        }
      }
    }

    LmPartial flushed[S::kCarry ? 1 : NT];
    static_for<NT>([&](auto ntc) __attribute__((always_inline)) {
      constexpr int nt = decltype(ntc)::value, si = S::kCarry ? nt : 0, ki = S::kKeysInLds ? 0 : nt;
      if (!S::kCarry) st[0] = LmLaneState{-INFINITY, 0.0f, -INFINITY, 0.0f, 0.0f, 0x7fffffff};
      const int c = c0 + 32 * nt + l32;
      if constexpr (S::kKeysInLds) {
        u32x4 kv = lds_read128<nt * 512>(lds0 + S::kKeyBase + l32 * 16);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(kv)::"memory");
        key_a[0] = kv[0]; sid_lo[0] = kv[1]; sid_hi[0] = kv[2];
      }
      if (active && c < C && (!split || nt / (NT / 2) == wave >> 2)) {
        const bool tail = vw + 32 > v_end;
        if (GIVEN) lm_given_block(acc[nt], st[si], vw + 4 * kb, v_end, tail, scale, static_cast<int>(key_a[ki]));
        else
          lm_epilogue_block(acc[nt], st[si], vw + 4 * kb, v_end, tail, scale, key_a[ki], sid_lo[ki], sid_hi[ki], key0, key1);
      }
      if constexpr (!S::kCarry) flushed[nt] = lane_partial<GIVEN>(st[0], inv_temperature);
    });
    if constexpr (!S::kCarry) {
      constexpr int F = S::kFlushWaves;
      LmPartial(*s_x)[S::kCols] = reinterpret_cast<LmPartial(*)[S::kCols]>(smem + S::kHBase + hslot * S::kHSlab);
      asm volatile("s_barrier" ::: "memory");   // every wave has left the tile's last slab, whose slot this is
#pragma unroll
      for (int ph = 0; ph < 8 / F; ++ph) {
        if (wave / F == ph && kb == 0)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) s_x[wave % F][32 * nt + l32] = flushed[nt];
        __syncthreads();
        if (tid < S::kCols)
          for (int w = 0; w < F; ++w) combine(mine, s_x[w][tid]);
        __syncthreads();
      }
    }
  }

  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if constexpr (S::kCarry) {
    LmPartial(*s_part)[S::kCols] = reinterpret_cast<LmPartial(*)[S::kCols]>(smem);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const LmPartial p = lane_partial<GIVEN>(st[nt], inv_temperature);
      if (kb == 0) s_part[wave][32 * nt + l32] = p;
    }
    __syncthreads();
    if (tid < S::kCols) {
      mine = s_part[0][tid];
      for (int w = 1; w < 8; ++w) combine(mine, s_part[w][tid]);
    }
  }
  if (tid < S::kCols && c0 + tid < C) part[static_cast<size_t>(c0 + tid) * n_parts + lane_id] = mine;
}

// grid = (row blocks, vocabulary lanes): the blocks of a lane run together and share its rows of W through the caches
template <bool GIVEN, typename S>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void lmhead_run_kernel(
    const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight, const int64_t* __restrict__ seq_id,
    const int32_t* __restrict__ step, const int32_t* __restrict__ target, uint32_t key0, uint32_t key1,
    float inv_temperature, LmPartial* __restrict__ part, int C, int H, int V, int lane_rows, int n_parts) {
  __shared__ __attribute__((aligned(1024))) char smem[S::kLds];
  lm_run_body<GIVEN, S>(smem, hidden, weight, seq_id, step, target, key0, key1, inv_temperature, part,
                        blockIdx.x * S::kCols, C, H, V, blockIdx.y, lane_rows, n_parts);
}

// grid = (row blocks, vocabulary lanes): consecutive workgroups (which the dispatcher deals out
// to the XCDs in turn) differ in the row block, so one XCD's L2 sees few row blocks
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void lmhead_gemm_given_kernel(
    const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight, const int32_t* __restrict__ target,
    float inv_temperature, LmPartial* __restrict__ part, int C, int H, int V, int lane_units, int n_parts) {
  __shared__ __attribute__((aligned(1024))) char smem[kGmLds];
  lm_gemm_given_body(smem, hidden, weight, target, inv_temperature, part, blockIdx.x * kGmBN, C, H, V, blockIdx.y,
                     lane_units, n_parts);
}

// Row blocks of 256 and a last one of another width (lm_given_plan): the first full * lanes workgroups are those
// of the whole blocks, ordered as above, the others the last block's.
template <typename S>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void lmhead_gemm_rest_kernel(
    const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight, const int32_t* __restrict__ target,
    float inv_temperature, LmPartial* __restrict__ part, int C, int H, int V, int full, int lanes, int lane_units,
    int rest_rows, int n_parts) {
  __shared__ __attribute__((aligned(1024))) char smem[kGmLds > S::kLds ? kGmLds : S::kLds];
  const int id = blockIdx.x;
  if (id < full * lanes) {
    lm_gemm_given_body(smem, hidden, weight, target, inv_temperature, part, id % full * kGmBN, C, H, V, id / full, lane_units,
                       n_parts);
  } else {
    lm_run_body<true, S>(smem, hidden, weight, nullptr, nullptr, target, 0, 0, inv_temperature, part, full * kGmBN, C, H, V,
                         id - full * lanes, rest_rows, n_parts);
  }
}

// --------------------------------------------------------------------------
// small-call kernel (bf16 with H % 64 == 0, fp32 with H % 16 == 0): calls whose tiles of 128 vocabulary rows and more would
// leave most of the chip idle (lm_small_tile).
//
// A workgroup of eight waves takes 16 * NV vocabulary rows against 16 * NC batch rows, and its waves share the HIDDEN
// dimension: wave w multiplies run w of the k-steps (64 bytes of a row), so the chain is an eighth of the row.
// Operands come straight from memory, DEEP steps of each in flight in a wave's registers: lane (n, b) of a product holds granule b
// of row n, which is the same in both operands, so fp32 feeds four products with a granule and bf16 one.  The buffer loads
// take the lane's row from a register and the step from a scalar, so that a step has no address arithmetic and a wave fits
// 128 registers (two workgroups per CU; 64 x 64: one; two or three of the bf16 64 x 32 kernels' spill).  The runs' sums are added in
// order through LDS, and then every thread has one Philox block of a column (two at 64 x 64), whose words it drew while the first
// operands were on their way; the lanes of a column meet by DPP.
// The tile follows what fills the chip and what the workspace has room for, the result does not: 16 rows of a column have one maximum,
// and sixteens are joined by pairs to 64 rows, here or, from smaller tiles, by the merge (join, the same arithmetic in both; one maximum
// per tile was 0.25 .. 0.5 us faster with 16 and 32 rows: C = 1, H = 1024, V = 3554 6.5 / 6.8).
// What bounds it: a CU's requests.  In operand order neighbouring lanes fetch from different rows, and a load of 64 such pieces
// of 16 bytes takes 64 clocks (33 GB/s).  With 32 batch rows and more (kGather) four neighbouring lanes fetch 64 bytes of one
// row instead and the operands are put in order by a lane permutation through LDS: C = 41, H = 3584, V = 3251 18.6 -> 12.7 us; C = 126,
// H = 3584, V = 2572 25.0 -> 15.3; C = 192, H = 3584, V = 4804 32.9 -> 22.9; C = 48, H = 1024, V = 7868 11.6 -> 9.7; fp32 C = 62, H = 3584, V = 1945
// 25.8 -> 18.4 (C = 66, H = 64, V = 1380 6.6 -> 7.1).  With 16 batch rows the permutation costs more than the few requests: C = 6, H = 1024,
// V = 6703 8.4 -> 9.3.  Requesting both halves of a
// 128-byte line one behind the other, and twice as many steps in flight with one workgroup per CU, gave nothing; W loaded
// non-temporally loses the line's other half (C = 2, H = 3584, V = 9482 19.7 -> 25.4); the
// sampler's counters loaded after the products cost 2 us (C = 2, H = 256, V = 1117: 9.0 -> 6.5, 11.8 with tiles of 128
// rows).  Times of whole calls are at lm_small_tile.
// --------------------------------------------------------------------------
constexpr int kSmThreads = 512, kSmRuns = kSmThreads / kWave;
constexpr int kSmStep = 64;                          // bytes of a row in a k-step

// The value of another lane: STEP 0 and 1 within four lanes, 2 between the halves of eight, 3 between the halves of sixteen.
template <int STEP>
__device__ __forceinline__ int lane_swap(int x) {
  constexpr int kCtrl[4] = {0xb1, 0x4e, 0x141, 0x140};   // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror
  return __builtin_amdgcn_update_dpp(0, x, kCtrl[STEP], 0xf, 0xf, false);
}
template <int STEP>
__device__ __forceinline__ float lane_swap(float x) { return __int_as_float(lane_swap<STEP>(__float_as_int(x))); }

template <typename T, bool GIVEN, int NV, int NC, int DEEP>
__global__ __launch_bounds__(kSmThreads) __attribute__((amdgpu_waves_per_eu(NV * NC > 8 ? 2 : 4, NV * NC > 8 ? 2 : 4)))
void lmhead_small_kernel(
    const T* __restrict__ hidden, const T* __restrict__ weight, const int64_t* __restrict__ seq_id,
    const int32_t* __restrict__ step, const int32_t* __restrict__ target, uint32_t key0, uint32_t key1,
    float inv_temperature, LmPartial* __restrict__ part, int C, int H, int V, int col_blocks, int n_tiles, int part_pitch) {
  constexpr int kRows = 16 * NV, kCols = 16 * NC, kPitch = kRows + 4;
  constexpr int kQuads = kRows / 4;                   // Philox blocks of a column
  constexpr bool kGather = NC > 1;
  constexpr int kSwaps = NV == 4 ? 4 : (NV == 2 ? 3 : 2);   // exchanges that bring a column's lanes together; two: those of 16 rows
  constexpr int kEach = (kCols * kQuads + kSmThreads - 1) / kSmThreads;   // ... of a thread
  __shared__ __attribute__((aligned(16))) float s_z[kSmRuns][kCols][kPitch];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  // the column blocks of a tile run one after the other on one XCD
  const int turn = blockIdx.x >> 3;
  const int tile = turn / col_blocks * 8 + (blockIdx.x & 7), c0 = turn % col_blocks * kCols;
  if (tile >= n_tiles) return;
  const int v0 = tile * kRows;
  const int n = lane & 15, b = lane >> 4;
  const uint32_t pitch = static_cast<uint32_t>(H) * sizeof(T);
  const int steps = static_cast<int>(pitch / kSmStep);
  const int j0 = steps * wave / kSmRuns, j1 = steps * (wave + 1) / kSmRuns;   // the wave's k-steps
  // the sampler's counters and the words drawn from them, or the given token, of the thread's entries
  const int quad = tid & (kQuads - 1), col0 = tid / kQuads;
  uint32_t sid_lo[kEach], sid_hi[kEach], at_step[kEach];
  int given[kEach];
  const bool samples = wave * kWave < kCols * kQuads;
  if (samples) {
#pragma unroll
    for (int e = 0; e < kEach; ++e) {
      const int c = min(c0 + col0 + e * (kSmThreads / kQuads), C - 1);
      if (GIVEN) {
        given[e] = target[c];
      } else {
        const uint64_t sid = static_cast<uint64_t>(seq_id[c]);
        sid_lo[e] = static_cast<uint32_t>(sid);
        sid_hi[e] = static_cast<uint32_t>(sid >> 32);
        at_step[e] = static_cast<uint32_t>(step[c]);
      }
    }
  }
  // row and 16-byte granule of a k-step that the lane fetches
  const int row = kGather ? lane >> 2 : n, granule = kGather ? lane & 3 : b;
  uint32_t woff[NV], hoff[NC];
#pragma unroll
  for (int i = 0; i < NV; ++i)
    woff[i] = static_cast<uint32_t>(min(v0 + 16 * i + row, V - 1)) * pitch + 16u * granule;
#pragma unroll
  for (int i = 0; i < NC; ++i)
    hoff[i] = static_cast<uint32_t>(min(c0 + 16 * i + row, C - 1)) * pitch + 16u * granule;
  const BufferRsrc wr = buffer_rsrc(weight, static_cast<uint32_t>(V) * pitch);
  const BufferRsrc hr = buffer_rsrc(hidden, static_cast<uint32_t>(C) * pitch);
  u32x4 x[DEEP][NV], y[DEEP][NC];
  f32x4 acc[NV][NC];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int k = 0; k < NC; ++k) acc[i][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto load = [&](auto stage, int j) __attribute__((always_inline)) {
    constexpr int U = decltype(stage)::value;
#pragma unroll
    for (int i = 0; i < NV; ++i) x[U][i] = buffer_load16(wr, woff[i], j * kSmStep);
#pragma unroll
    for (int i = 0; i < NC; ++i) y[U][i] = buffer_load16(hr, hoff[i], j * kSmStep);
  };
  const int from = 4 * (4 * n + b);                   // lane 4 n + b has fetched what lane (n, b) of a product holds
  auto operand = [&](const u32x4& x) __attribute__((always_inline)) {
    if (!kGather) return x;
    u32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(x[e])));
    return y;
  };
  auto multiply = [&](auto stage) __attribute__((always_inline)) {
    constexpr int U = decltype(stage)::value;
    u32x4 hid[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) hid[k] = operand(y[U][k]);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const u32x4 w = operand(x[U][i]);
      if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int k = 0; k < NC; ++k)
          acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, hid[k]),
                                                              acc[i][k], 0, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int k = 0; k < NC; ++k)
            acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[e]), __uint_as_float(hid[k][e]), acc[i][k], 0, 0, 0);
      }
    }
  };
  int j = j0;
  if (j1 - j0 >= 2 * DEEP) {
    // (no branch around a load, so that the compiler's counts of those in flight are exact)
    static_for<DEEP>([&](auto u) __attribute__((always_inline)) { load(u, j0 + u.value); });
    for (; j + 2 * DEEP <= j1; j += DEEP)
      static_for<DEEP>([&](auto u) __attribute__((always_inline)) {
        multiply(u);
        load(u, j + DEEP + u.value);
      });
  } else {
    static_for<DEEP>([&](auto u) __attribute__((always_inline)) {
      if (j0 + u.value < j1) load(u, j0 + u.value);
    });
  }
  Philox4 words[kEach] = {};
  if (!GIVEN && samples) {
#pragma unroll
    for (int e = 0; e < kEach; ++e)
      words[e] = philox4x32_10(static_cast<uint32_t>(v0 / 4 + quad), at_step[e], sid_lo[e], sid_hi[e], key0, key1);
  }
  static_for<DEEP>([&](auto u) __attribute__((always_inline)) {
    if (j + u.value < j1) multiply(u);
    if (j + DEEP + u.value < j1) load(u, j + DEEP + u.value);
  });
  static_for<DEEP>([&](auto u) __attribute__((always_inline)) {
    if (j + DEEP + u.value < j1) multiply(u);
  });
  // lane (n, b): vocabulary rows 16 i + 4 b .. + 3 of column 16 k + n
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int k = 0; k < NC; ++k) *reinterpret_cast<f32x4*>(&s_z[wave][16 * k + n][16 * i + 4 * b]) = acc[i][k];
  __syncthreads();
  if (!samples) return;
  const float scale = lm_scale(inv_temperature);
#pragma unroll
  for (int e = 0; e < kEach; ++e) {
    const int col = col0 + e * (kSmThreads / kQuads), c = c0 + col;
    f32x4 z = *reinterpret_cast<const f32x4*>(&s_z[0][col][4 * quad]);
#pragma unroll
    for (int r = 1; r < kSmRuns; ++r) z += *reinterpret_cast<const f32x4*>(&s_z[r][col][4 * quad]);
    const int vq = v0 + 4 * quad;
    float a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = sizeof(T) == 2 ? z[i] : z[i] * inv_temperature;
      if (vq + i >= V) a[i] = -INFINITY;
    }
    // one maximum for 16 rows of the column
    float m = fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3]));
    if (sizeof(T) == 2) m = fmaxf(m, -INFINITY);       // (not a number only in fp32: as in the other kernels)
    static_for<2>([&](auto s) __attribute__((always_inline)) { m = fmaxf(m, lane_swap<s.value>(m)); });
    LmPartial p;
    if constexpr (sizeof(T) == 2) {
      LmLaneState st{m, 0.0f, -INFINITY, 0.0f, 0.0f, 0x7fffffff};
      if (GIVEN) lm_given_quad(a, st, vq, V, false, scale, given[e]);
      else lm_sample_words(a, st, vq, scale, [w = words[e]]() __attribute__((always_inline)) { return w; });
      p = state_partial<GIVEN>(st, inv_temperature);
    } else {
      p = empty_partial();
      p.m = m;
      const uint32_t word[4] = {words[e].x, words[e].y, words[e].z, words[e].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p.s += a[i] == -INFINITY ? 0.0f : __expf(a[i] - m);
        const int v = vq + i;
        const float best = GIVEN ? (v == given[e] ? INFINITY : -INFINITY) : a[i] + gumbel_from_uniform(word_to_uniform(word[i]));
        if (v < V && (!GIVEN || v == given[e]) && better(best, v, p.best, p.idx)) {
          p.best = best;
          p.z = a[i];
          p.idx = v;
        }
      }
    }
    static_for<2>([&](auto s) __attribute__((always_inline)) {
      p.s += lane_swap<s.value>(p.s);
      const float best = lane_swap<s.value>(p.best), logit = lane_swap<s.value>(p.z);
      const int idx = lane_swap<s.value>(p.idx);
      if (better(best, idx, p.best, p.idx)) {
        p.best = best;
        p.z = logit;
        p.idx = idx;
      }
    });
    static_for<kSwaps - 2>([&](auto i) __attribute__((always_inline)) {
      constexpr int s = 2 + i.value;
      LmPartial o;
      o.m = lane_swap<s>(p.m);
      o.s = lane_swap<s>(p.s);
      o.best = lane_swap<s>(p.best);
      o.z = lane_swap<s>(p.z);
      o.idx = lane_swap<s>(p.idx);
      join(p, o);
    });
    if (quad == 0 && c < C) part[static_cast<size_t>(c) * part_pitch + tile] = p;
  }
}

// --------------------------------------------------------------------------
// merge: one wavefront per batch row over its partials, four where there are more than kMergeAlone.
//
// It is a chain of latencies: launch, one round trip to memory (four partials per lane in flight), one maximum for the
// row, one exponential per partial against it, sums and the best score by DPP.  With four waves per row, every lane's
// partials and every exchange combined with two exponentials of their own, and a barrier, whole calls took, in us, before / now:
// given tokens M = 4164, H = 256, V = 5269 31.3 / 26.5, M = 8192, H = 256, V = 20011 113.1 / 103.1; sampling within what runs differ by:
// C = 64, H = 1536, V = 151936 92.4 / 90.7, C = 301, H = 2048, V = 50257 93.0 / 92.0.  With 2374 partials of a row (C = 5, H = 72, V = 151936) 30.0 / 27.7,
// and 30.3 with one wavefront.
// --------------------------------------------------------------------------
// (Rows from `rest` on have n_rest partials, in rows of n_tiles like the others.)  PER neighbouring partials are joined first: those of
// the small-call kernel's tiles, to the 64 rows of its largest.
constexpr int kMergeAlone = 1024;
template <int WAVES, int PER>
__global__ __launch_bounds__(WAVES * kWave) void lmhead_merge_kernel(const LmPartial* __restrict__ part,
                                                             int n_tiles, int n_all, int rest, int n_rest,
                                                             int32_t* __restrict__ token,
                                                             float* __restrict__ logprob,
                                                             float* __restrict__ lse) {
  constexpr int kDeep = 4;
  const int c = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1);
  const LmPartial* row = part + static_cast<size_t>(c) * n_tiles;
  LmPartial p = empty_partial();
  const int n_parts = c < rest ? n_all : n_rest, n = (n_parts - 1) / PER + 1;
  for (int t = tid; t < n; t += kDeep * WAVES * kWave) {
    LmPartial q[kDeep];
    if constexpr (PER == 1) {
#pragma unroll
      for (int u = 0; u < kDeep; ++u) q[u] = row[min(t + u * WAVES * kWave, n - 1)];
    } else {
      typedef unsigned int Words __attribute__((ext_vector_type(PER)));
      static_assert(sizeof(LmPartial) == 5 * sizeof(unsigned int), "PER partials are five loads");
      alignas(16) LmPartial x[kDeep][PER];
#pragma unroll
      for (int u = 0; u < kDeep; ++u)
        if (u == 0 || t - tid + u * WAVES * kWave < n) {       // (all lanes or none)
#pragma unroll
          for (int e = 0; e < 5; ++e)                          // (whole groups have places in the workspace)
            reinterpret_cast<Words*>(&x[u])[e] = reinterpret_cast<const Words*>(row + static_cast<size_t>(min(t + u * WAVES * kWave, n - 1)) * PER)[e];
        }
#pragma unroll
      for (int u = 0; u < kDeep; ++u) {
        if (u != 0 && t - tid + u * WAVES * kWave >= n) continue;
#pragma unroll
        for (int e = 1; e < PER; ++e)
          if ((t + u * WAVES * kWave) * PER + e >= n_parts) x[u][e] = empty_partial();
#pragma unroll
        for (int e = 0; e < PER; e += 2) join(x[u][e], x[u][e + 1]);
        if constexpr (PER == 4) join(x[u][0], x[u][2]);
        q[u] = x[u][0];
      }
    }
    const float before = p.m;
#pragma unroll
    for (int u = 0; u < kDeep; ++u) {
      if (t + u * WAVES * kWave >= n) q[u] = empty_partial();
      p.m = fmaxf(p.m, q[u].m);
    }
    // an empty partial (m = -inf) weighs nothing, whatever the maximum is
    p.s = before == -INFINITY ? p.s : p.s * __expf(before - p.m);
#pragma unroll
    for (int u = 0; u < kDeep; ++u) {
      p.s += q[u].m == -INFINITY ? 0.0f : q[u].s * __expf(q[u].m - p.m);
      if (better(q[u].best, q[u].idx, p.best, p.idx)) {
        p.best = q[u].best;
        p.idx = q[u].idx;
        p.z = q[u].z;
      }
    }
  }
  float m = p.m;
  static_for<4>([&](auto k) __attribute__((always_inline)) { m = fmaxf(m, lane_swap<k.value>(m)); });
  m = fmaxf(m, __shfl_xor(m, 16, kWave));
  m = fmaxf(m, __shfl_xor(m, 32, kWave));
  p.s = p.m == -INFINITY ? p.s : p.s * __expf(p.m - m);
  p.m = m;
  auto take = [&](float best, int idx, float z) __attribute__((always_inline)) {
    if (better(best, idx, p.best, p.idx)) {
      p.best = best;
      p.idx = idx;
      p.z = z;
    }
  };
  static_for<4>([&](auto k) __attribute__((always_inline)) {
    p.s += lane_swap<k.value>(p.s);
    take(lane_swap<k.value>(p.best), lane_swap<k.value>(p.idx), lane_swap<k.value>(p.z));
  });
#pragma unroll
  for (int o = 16; o <= 32; o *= 2) {
    p.s += __shfl_xor(p.s, o, kWave);
    take(__shfl_xor(p.best, o, kWave), __shfl_xor(p.idx, o, kWave), __shfl_xor(p.z, o, kWave));
  }
  if constexpr (WAVES > 1) {
    __shared__ LmPartial s_part[WAVES];
    if (lane == 0) s_part[tid / kWave] = p;
    __syncthreads();
    if (tid == 0) {
#pragma unroll
      for (int w = 1; w < WAVES; ++w) combine(p, s_part[w]);
    }
  }
  if (tid == 0) {
    // m + ln s in fp64, the logarithm of the mantissa alone (at most 1, so good to 6e-8) in fp32: logf is
    // 3.2e-7 too small on average over 1 .. 10^4, as much as all other roundings of a row together
    const double l = static_cast<double>(p.m) +
                     (static_cast<double>(__builtin_amdgcn_frexp_expf(p.s)) +
                      static_cast<double>(__builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(p.s)))) * 0.69314718055994531;
    if (token != nullptr) token[c] = p.idx;
    // no candidate at all (a given token outside [0, V)): not a number
    logprob[c] = p.idx == 0x7fffffff ? __int_as_float(0x7fc00000) : static_cast<float>(static_cast<double>(p.z) - l);
    if (lse != nullptr) lse[c] = static_cast<float>(l);
  }
}

// True if the matrix-core kernels take the shape (they address both operands with 32-bit
// byte offsets).
static bool lm_use_mfma(int C, int H, int V, int dtype) {
  return dtype == 1 && H % kMfBK == 0 && static_cast<uint64_t>(V) * H * 2 < (1ull << 32) &&
         static_cast<uint64_t>(C) * H * 2 < (1ull << 32);
}
// Micro-batches of given tokens go to the 256 x 256 kernel.
static bool lm_use_gemm(int C, int H, int V, int dtype, bool given) {
  return given && C >= kGmMinRows && lm_use_mfma(C, H, V, dtype);
}

// At most 64 rows: the skinny kernel, where it pays.
static bool lm_use_skinny(int C, int H, int V, int dtype, bool given) {
  return lm_use_mfma(C, H, V, dtype) && lm_skinny_pays(C, H, V, given);
}
// Vocabulary rows per workgroup of the skinny kernel: an equal share for the resident workgroups,
// in whole Philox blocks, but at least kLmTileV (a shorter run is all pipeline start).  Its tiles:
// as few as cover the run, of equal height.
static int lm_skinny_height(int rows) {
  const int tiles = (rows + kSkBM - 1) / kSkBM;
  return ((rows + tiles - 1) / tiles + 3) & ~3;
}
static int lm_skinny_rows(int V) {
  const int rows = (((V + kSkMaxGrid - 1) / kSkMaxGrid) + 3) & ~3;
  return rows < kLmTileV ? kLmTileV : rows;
}

// Columns of the run kernel's row blocks; 0: another kernel takes the call.
static int lm_use_run(int C, int H, int V, int dtype, bool given) {
  return lm_use_mfma(C, H, V, dtype) ? lm_run_cols(C, H, V, given) : 0;
}
// Tile of the small-call kernel, for a workspace with room for max_parts partials per row; no rows: another kernel
// takes the call.
static bool lm_small_takes(int C, int H, int V, int dtype) {
  const int64_t pitch = static_cast<int64_t>(H) * (dtype == 0 ? 4 : 2), most = ((1ll << 32) - 1) / pitch;   // (bytes of a buffer)
  return pitch % (dtype == 0 ? kSmStep : 2 * kSmStep) == 0 && V <= most && C <= most;
}
static LmSmall lm_use_small(int C, int H, int V, int dtype, bool given, int64_t max_parts) {
  if (!lm_small_takes(C, H, V, dtype)) return {0, 0};
  return lm_small_tile(C, H, V, given, dtype == 0, max_parts);
}
// Partials per row.  Matrix-core kernels: the grid is (parts, row blocks) with
// parts * blocks <= the resident workgroups (512, or 256 for the 256 x 256 kernel) where
// possible, so that the workgroups that run at the same time walk the same vocabulary tiles
// (W comes from HBM once and is shared through the caches) and each keeps its rows' state
// across all of its tiles.
static int lm_parts(int C, int H, int V, int dtype, bool given, int64_t max_parts) {
  if (const LmSmall sm = lm_use_small(C, H, V, dtype, given, max_parts); sm.rows != 0) return static_cast<int>(lm_small_parts(V, sm.rows));
  if (!lm_use_mfma(C, H, V, dtype)) return (V - 1) / kLmTileV + 1;
  if (const int width = lm_use_run(C, H, V, dtype, given)) return (V - 1) / lm_run_rows(C, V, width) + 1;
  if (lm_use_skinny(C, H, V, dtype, given)) return (V - 1) / lm_skinny_rows(V) + 1;
  if (lm_use_gemm(C, H, V, dtype, given)) {
    const LmGivenPlan p = lm_given_plan(C, H, V);
    return p.lanes > p.rest_lanes ? p.lanes : p.rest_lanes;
  }
  const int n_tiles = (V + kMfBM - 1) / kMfBM;
  int parts = kMfMaxGrid / lm_tile_blocks(C, H, V, given).blocks;
  parts = parts < 1 ? 1 : parts;
  return parts < n_tiles ? parts : n_tiles;
}

// Partials per row that a workspace of `bytes` bytes has room for.
static int64_t lm_room(size_t bytes, int C) {
  return static_cast<int64_t>(std::min<size_t>(bytes, size_t{1} << 40) / (static_cast<size_t>(C) * sizeof(LmPartial)));
}
constexpr int64_t kLmAnyParts = INT64_MAX;

// The sampling call: a partial per 64 vocabulary rows is what it needs; with the rest it may cut smaller tiles.
size_t lm_workspace_need(int C, int V) {
  return align256(static_cast<size_t>(C) * ((V - 1) / kLmTileV + 1) * sizeof(LmPartial));
}
size_t lm_workspace_bytes(int C, int H, int V) {
  size_t most = lm_workspace_need(C, V);
  for (int dtype : {0, 1})
    if (lm_use_small(C, H, V, dtype, false, kLmAnyParts).rows != 0)
      most = std::max(most, align256(static_cast<size_t>(C) * lm_parts(C, H, V, dtype, false, kLmAnyParts) * sizeof(LmPartial)));
  return most;
}

static size_t lm_token_bytes(int M, int H, int V, int dtype, int64_t max_parts) {
  return align256(static_cast<size_t>(M) * lm_parts(M, H, V, dtype, true, max_parts) * sizeof(LmPartial));
}
// What a call cannot do without (the small-call kernel is taken where there is more).
size_t lm_token_workspace_need(int M, int H, int V, int dtype) { return lm_token_bytes(M, H, V, dtype, 0); }

// What M positions need, or any smaller number: fewer rows may be cut into more parts, and a program
// sizes its workspace for its largest micro-batch.
size_t lm_token_workspace_bytes(int M, int H, int V, int dtype) {
  size_t most = lm_token_workspace_need(M, H, V, dtype);
  if (lm_small_takes(1, H, V, dtype))
    most = std::max(most, align256(static_cast<size_t>(lm_small_most_parts(M, H, V, dtype == 0)) * sizeof(LmPartial)));
  if (!lm_use_mfma(M, H, V, dtype)) return most;   // (a part per 64 vocabulary rows: as many as there can be)
  // the parts per row are constant between these numbers of rows
  const int ends[] = {8, 32, kSkMaxRows, 128, 160, 192, 256, 320, kGmMinRows - 1};
  for (int m : ends)
    if (m < M) most = std::max(most, lm_token_workspace_need(m, H, V, dtype));
  for (int64_t m = kMfBN; m < M; m += kMfBN)
    for (int rest : {0, 64, 128, 160})
      if (m + rest < M) most = std::max(most, lm_token_workspace_need(static_cast<int>(m + rest), H, V, dtype));
  return most;
}

// Both modes: target == nullptr samples (seq_id / step / seed), else scores the given tokens.
static int launch_lmhead(const void* hidden, const void* weight, const int64_t* seq_id,
                         const int32_t* step, const int32_t* target, uint64_t seed,
                         float temperature, int32_t* token, float* logprob, float* lse,
                         void* workspace, size_t workspace_bytes, int C, int H, int V, int dtype,
                         hipStream_t stream) {
  LmPartial* part = static_cast<LmPartial*>(workspace);
  const int64_t room = lm_room(workspace_bytes, C);
  const uint32_t key0 = static_cast<uint32_t>(seed), key1 = static_cast<uint32_t>(seed >> 32);
  const float inv_t = 1.0f / temperature;
  const bool given = target != nullptr;
  const LmSmall sm = lm_use_small(C, H, V, dtype, given, room);
  const int n_parts = static_cast<int>(sm.rows != 0 ? lm_small_parts(V, sm.rows) : lm_parts(C, H, V, dtype, given, 0));
  int n_all = n_parts, rest = C, n_rest = 0;   // partials of a row; first row that has n_rest of them
  if (sm.rows != 0) {
    const int col_blocks = (C - 1) / sm.cols + 1;
    n_all = (V - 1) / sm.rows + 1;
    const dim3 grid((n_all + 7) / 8 * 8 * col_blocks);
    COPRIS_PRE("lmhead_small_kernel");
#define COPRIS_LM_SMALL(T, G, NV, NC, D)                                                                    \
  hipLaunchKernelGGL((lmhead_small_kernel<T, G, NV, NC, D>), grid, dim3(kSmThreads), 0, stream,             \
                     static_cast<const T*>(hidden), static_cast<const T*>(weight), seq_id, step, target,    \
                     key0, key1, inv_t, part, C, H, V, col_blocks, n_all, n_parts)
#define COPRIS_LM_SMALLS(T, G)                                                  \
  switch (100 * sm.rows + sm.cols) {                                            \
    case 1616: COPRIS_LM_SMALL(T, G, 1, 1, 8); break;                           \
    case 3216: COPRIS_LM_SMALL(T, G, 2, 1, 6); break;                           \
    case 6416: COPRIS_LM_SMALL(T, G, 4, 1, 4); break;                           \
    case 1632: COPRIS_LM_SMALL(T, G, 1, 2, 6); break;                           \
    case 3232: COPRIS_LM_SMALL(T, G, 2, 2, 4); break;                           \
    case 6432: COPRIS_LM_SMALL(T, G, 4, 2, 3); break;                           \
    case 3264: COPRIS_LM_SMALL(T, G, 2, 4, 2); break;                           \
    default: COPRIS_LM_SMALL(T, G, 4, 4, 4); break;                             \
  }
    if (dtype == 0 && given) {
      COPRIS_LM_SMALLS(float, true);
    } else if (dtype == 0) {
      COPRIS_LM_SMALLS(float, false);
    } else if (given) {
      COPRIS_LM_SMALLS(uint16_t, true);
    } else {
      COPRIS_LM_SMALLS(uint16_t, false);
    }
#undef COPRIS_LM_SMALLS
#undef COPRIS_LM_SMALL
    COPRIS_POST("lmhead_small_kernel");
  } else if (const int width = lm_use_run(C, H, V, dtype, given)) {
    const dim3 grid((C + width - 1) / width, n_parts);
    COPRIS_PRE("lmhead_run_kernel");
#define COPRIS_LM_RUN(G, S)                                                                              \
  hipLaunchKernelGGL((lmhead_run_kernel<G, S>), grid, dim3(512), 0, stream,                              \
                     static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(weight), seq_id, \
                     step, target, key0, key1, inv_t, part, C, H, V, lm_run_rows(C, V, width), n_parts)
#define COPRIS_LM_RUNS(G)                              \
  if (width == 128) COPRIS_LM_RUN(G, LmRun128);        \
  else if (width == 160) COPRIS_LM_RUN(G, LmRun160);   \
  else if (width == 192) COPRIS_LM_RUN(G, LmRun192);   \
  else if (width == 256) COPRIS_LM_RUN(G, LmRun256);   \
  else COPRIS_LM_RUN(G, LmRun320)
    if (given) {
      COPRIS_LM_RUNS(true);
    } else {
      COPRIS_LM_RUNS(false);
    }
#undef COPRIS_LM_RUNS
#undef COPRIS_LM_RUN
    COPRIS_POST("lmhead_run_kernel");
  } else if (lm_use_gemm(C, H, V, dtype, given)) {
    const LmGivenPlan p = lm_given_plan(C, H, V);
    if (p.width == 0) {
      COPRIS_PRE("lmhead_gemm_given_kernel");
      hipLaunchKernelGGL(lmhead_gemm_given_kernel, dim3(p.full, p.lanes), dim3(512), 0, stream,
                         static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(weight),
                         target, inv_t, part, C, H, V, p.lane_units, n_parts);
      COPRIS_POST("lmhead_gemm_given_kernel");
    } else {
      rest = p.full * kGmBN;
      n_all = p.lanes;
      n_rest = p.rest_lanes;
      COPRIS_PRE("lmhead_gemm_rest_kernel");
#define COPRIS_LM_REST(S)                                                                                 \
  hipLaunchKernelGGL((lmhead_gemm_rest_kernel<S>), dim3(p.full * p.lanes + p.rest_lanes), dim3(512), 0,   \
                     stream, static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(weight),  \
                     target, inv_t, part, C, H, V, p.full, p.lanes, p.lane_units, p.rest_rows, n_parts)
      if (p.width == 128) COPRIS_LM_REST(LmRun128);
      else if (p.width == 160) COPRIS_LM_REST(LmRun160);
      else COPRIS_LM_REST(LmRun320);
#undef COPRIS_LM_REST
      COPRIS_POST("lmhead_gemm_rest_kernel");
    }
  } else if (lm_use_skinny(C, H, V, dtype, given)) {
    const int rows = lm_skinny_rows(V);
    COPRIS_PRE("lmhead_skinny_kernel");
#define COPRIS_LM_SKINNY(G, NT)                                                                          \
  hipLaunchKernelGGL((lmhead_skinny_kernel<G, NT>), dim3(n_parts), dim3(512), 0, stream,                 \
                     static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(weight), seq_id, \
                     step, target, key0, key1, inv_t, part, C, H, V, rows, lm_skinny_height(rows), n_parts)
    if (given && C <= 32) COPRIS_LM_SKINNY(true, 1);
    else if (given) COPRIS_LM_SKINNY(true, 2);
    else if (C <= 32) COPRIS_LM_SKINNY(false, 1);
    else COPRIS_LM_SKINNY(false, 2);
#undef COPRIS_LM_SKINNY
    COPRIS_POST("lmhead_skinny_kernel");
  } else if (lm_use_mfma(C, H, V, dtype)) {
    const int n_tiles = (V + kMfBM - 1) / kMfBM;
    const LmBlocks rows = lm_tile_blocks(C, H, V, given);
    const dim3 grid(n_parts, rows.blocks);
    COPRIS_PRE("lmhead_mfma_kernel");
#define COPRIS_LM_MFMA_LAUNCH(G, HV, NT1)                                                                \
  hipLaunchKernelGGL((lmhead_mfma_kernel<G, HV, NT1>), grid, dim3(256), 0, stream,                        \
                     static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(weight), seq_id, \
                     step, target, key0, key1, inv_t, part, C, H, V, block_rows, n_tiles, n_parts, flip)
    const int block_rows = rows.rows, width = rows.width;
    const int flip = lm_second_block_flip(C, n_tiles, n_parts);
    if (given) {
      if (width == 128) COPRIS_LM_MFMA_LAUNCH(true, 1, 2);
      else if (width == 192) COPRIS_LM_MFMA_LAUNCH(true, 2, 1);
      else COPRIS_LM_MFMA_LAUNCH(true, 2, 2);
    } else {
      if (width == 128) COPRIS_LM_MFMA_LAUNCH(false, 1, 2);
      else if (width == 192) COPRIS_LM_MFMA_LAUNCH(false, 2, 1);
      else COPRIS_LM_MFMA_LAUNCH(false, 2, 2);
    }
#undef COPRIS_LM_MFMA_LAUNCH
    COPRIS_POST("lmhead_mfma_kernel");
  } else if (dtype == 0) {
    // (up to 16 rows the second half of a 32-row block would be padding)
    COPRIS_PRE("lmhead_f32_kernel");
#define COPRIS_LM_F32(G, NB)                                                                              \
  hipLaunchKernelGGL((lmhead_f32_kernel<G, NB>), dim3(n_parts, (C + 16 * NB - 1) / (16 * NB)),            \
                     dim3(kF32Threads), 0, stream, static_cast<const float*>(hidden),                     \
                     static_cast<const float*>(weight), seq_id, step, target, key0, key1, inv_t, part, C, \
                     H, V, n_parts)
    if (given && C <= 16) COPRIS_LM_F32(true, 1);
    else if (given) COPRIS_LM_F32(true, 2);
    else if (C <= 16) COPRIS_LM_F32(false, 1);
    else COPRIS_LM_F32(false, 2);
#undef COPRIS_LM_F32
    COPRIS_POST("lmhead_f32_kernel");
  } else {
    const dim3 grid(n_parts, (C + kLmTileC - 1) / kLmTileC);
#define COPRIS_LM_GENERIC(G)                                                                      \
  hipLaunchKernelGGL((lmhead_generic_kernel<G>), grid, dim3(256), 0, stream,            \
                     static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(weight), seq_id, step,  \
                     target, key0, key1, inv_t, part, C, H, V, n_parts)
    COPRIS_PRE("lmhead_generic_kernel");
    if (given) COPRIS_LM_GENERIC(true);
    else COPRIS_LM_GENERIC(false);
#undef COPRIS_LM_GENERIC
    COPRIS_POST("lmhead_generic_kernel");
  }
  COPRIS_PRE("lmhead_merge_kernel");
  const int per = sm.rows != 0 ? kLmTileV / sm.rows : 1;
#define COPRIS_LM_MERGE(PER)                                                                                              \
  if ((n_parts - 1) / PER < kMergeAlone)                                                                                  \
    hipLaunchKernelGGL((lmhead_merge_kernel<1, PER>), dim3(C), dim3(kWave), 0, stream, part, n_parts, n_all, rest, n_rest, \
                       token, logprob, lse);                                                                              \
  else                                                                                                                    \
    hipLaunchKernelGGL((lmhead_merge_kernel<4, PER>), dim3(C), dim3(4 * kWave), 0, stream, part, n_parts, n_all, rest,     \
                       n_rest, token, logprob, lse)
  switch (per) {
    case 1: COPRIS_LM_MERGE(1); break;
    case 2: COPRIS_LM_MERGE(2); break;
    default: COPRIS_LM_MERGE(4); break;
  }
#undef COPRIS_LM_MERGE
  COPRIS_POST("lmhead_merge_kernel");
  return 0;
}

int launch_lmhead_logprob(const void* hidden, const void* weight, const int64_t* seq_id,
                          const int32_t* step, uint64_t seed, float temperature, int32_t* token,
                          float* logprob, float* lse, void* workspace, size_t workspace_bytes, int C, int H, int V,
                          int dtype, hipStream_t stream) {
  return launch_lmhead(hidden, weight, seq_id, step, nullptr, seed, temperature, token, logprob, lse,
                       workspace, workspace_bytes, C, H, V, dtype, stream);
}

// --------------------------------------------------------------------------
// The sampling call for callers that cannot allocate: the per-(row, part) partials live in a
// file-scope device array instead of a caller workspace.  Every GPU the library runs on holds
// its own copy of the array at its own address; the address is looked up once per device.
// --------------------------------------------------------------------------
constexpr size_t kLmScratchBytes = 4u << 20;
static __device__ __align__(256) unsigned char scratch[kLmScratchBytes];

size_t lm_noalloc_scratch_limit() { return kLmScratchBytes; }

size_t lm_noalloc_scratch_needed(int C, int H, int V, int dtype) {
  return static_cast<size_t>(C) * lm_parts(C, H, V, dtype, false, lm_room(kLmScratchBytes, C)) * sizeof(LmPartial);
}

// Device address of this GPU's copy of `scratch` (nullptr + *err set on failure).
static void* lm_scratch_on_current_device(hipError_t* err) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptrs[kMaxDevices] = {};
  int dev = -1;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= kMaxDevices) {
    *err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (ptrs[dev] == nullptr) {
    void* p = nullptr;
    *err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (*err != hipSuccess) return nullptr;
    ptrs[dev] = p;
  }
  return ptrs[dev];
}

int launch_lmhead_logprob_noalloc(const void* hidden, const void* weight, const int64_t* seq_id,
                                  const int32_t* step, uint64_t seed, float temperature,
                                  int32_t* token, float* logprob, float* lse, int C, int H, int V,
                                  int dtype, hipStream_t stream) {
  hipError_t err = hipSuccess;
  void* ws = lm_scratch_on_current_device(&err);
  if (ws == nullptr) {
    set_error_detail("hipGetSymbolAddress(scratch)", err);
    return kErrLaunch;
  }
  return launch_lmhead(hidden, weight, seq_id, step, nullptr, seed, temperature, token, logprob, lse, ws,
                       kLmScratchBytes, C, H, V, dtype, stream);
}

int launch_lmhead_token_logprob(const void* hidden, const void* weight, const int32_t* tokens,
                                float temperature, float* logprob, float* lse, void* workspace,
                                size_t workspace_bytes, int M, int H, int V, int dtype, hipStream_t stream) {
  return launch_lmhead(hidden, weight, nullptr, nullptr, tokens, 0, temperature, nullptr, logprob,
                       lse, workspace, workspace_bytes, M, H, V, dtype, stream);
}

}  // namespace copris
