// Learning the quantisation step sizes (Section 4.1, "Efficient distillation", taken layer by layer; the
// straight-through estimator of Section 3 for Eq. 1): per output channel j, on calibration activations X,
//
//     r_tj = sum_i x_ti (Dtilde_ji(s_j) - Delta_ji)        L_j = 1/2 sum_t r_tj^2
//     g_j  = sum_t r_tj p_tj,   p_tj = sum_{i not salient} x_ti D_ji,   D_ji = (u_ji - z) - [inside] Delta_ji / s_j
//
// With E_ji = (Dtilde_ji - Delta_ji) / s_j -- (u - z) - Delta / s at low-bit columns, whether clamped or not, and
// (fp16(Delta) - Delta) / s at salient columns -- both sums are dense contractions over the input channels with the
// same activations: r = s X E^T and p = X D^T, where D equals E inside the grid, u - z where the weight is clamped
// and 0 at salient columns.  The kernel builds E and D on the fly from the fp32 delta (never stored), as bf16
// matrix-core operands, and multiplies both with X.
#include "mes_internal.h"

#include <cmath>

namespace mes {
namespace {


typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;

constexpr int kRows = 64;      // output channels per workgroup: 4 row tiles of 16, one generated by each wavefront
constexpr int kTokBlock = 256; // tokens per workgroup: 4 groups of 64, one multiplied by each wavefront
constexpr int kStepCols = 128; // input channels between two barriers: 4 blocks of 32 (one matrix instruction deep)

struct StepParams {
  const float* delta;       // [d_out, d_in] fp32
  const float* step;        // [d_out]
  const uint32_t* salmask;  // [d_in_pad / 32] bit i of word i / 32 set: column i is salient
  const u32x4* xt;          // activations as matrix-core fragments: [d_in_pad / 32][n_tq][64 lanes] x 16 bytes
  float* partial;           // [n_tg][2][d_out_pad]: per 64-token group, loss and gradient sums of every row
  f32x4* tiles;             // split columns only: every workgroup's accumulator tiles, [split][row group][token block][thread][32]
  int d_in, d_out, d_out_pad, n_tokens, n_tq, n_steps, steps_per_split, n_split;
};

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const bf16x2 h = __builtin_convertvector(f32x2{a, b}, bf16x2);   // round to nearest even
  return __builtin_bit_cast(uint32_t, h);
}

// x [n_tokens, d_in] bf16 row-major -> fragment order: block (kb, tq) holds, for lane l, the 8 values
// x[16 tq + (l & 15)][32 kb + 8 (l >> 4) ...]; zero beyond the last token and the last column.
// The first block writes the salient-column mask instead: one bit per column, set for the columns in sidx (a launch of
// its own took 4 us).
__global__ __launch_bounds__(256) void k_tile_x(const uint16_t* __restrict__ x, int n_tokens, int d_in, int n_tq, u32x4* __restrict__ xt,
                                                const int32_t* __restrict__ sidx, int k, int n_words, uint32_t* __restrict__ mask) {
  if (blockIdx.x == 0) {
    for (int w = threadIdx.x; w < n_words; w += 256) mask[w] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < k; i += 256) {
      const int c = sidx[i];
      if (c >= 0 && c < 32 * n_words) atomicOr(&mask[c >> 5], 1u << (c & 31));
    }
    return;
  }
  const int lane = threadIdx.x & 63;
  const size_t blk = (size_t)(blockIdx.x - 1) * 4 + (threadIdx.x >> 6);
  const int tq = (int)(blk % n_tq), kb = (int)(blk / n_tq);
  const int t = 16 * tq + (lane & 15), c = 32 * kb + 8 * (lane >> 4);
  u32x4 v = {0, 0, 0, 0};
  if (t < n_tokens && c < d_in) v = *reinterpret_cast<const u32x4*>(x + (size_t)t * d_in + c);
  xt[blk * 64 + lane] = v;
}

// E and D for 8 consecutive input channels of one row, as two packed bf16 operands.
// The code decision is exact: m = floor(w / s) (or the nearest integer, ties to even, on Eq. 1's grid) is first
// estimated from the rounded quotient pushed slightly upwards, then corrected with one fused multiply-add whose
// sign is that of the exact w - m s.  SALIENT: bit e of sal8 marks column e as salient (kept in fp16, no slope).
// Written stage by stage over the 8 channels: each channel is a chain of a dozen dependent instructions, and a
// builder is the only wavefront of its SIMD that issues vector arithmetic, so the 8 chains have to be interleaved
// for the vector unit not to sit waiting on its own results.
template <int BITS, bool EQ1, bool SALIENT>
__device__ __forceinline__ void make_operands(const f32x4 lo, const f32x4 hi, float s, float inv_s, uint32_t sal8,
                                              u32x4& e_out, u32x4& d_out) {
  constexpr float kHalf = (float)(1 << (BITS - 1));
  // + 0.0f turns a weight of -0.0 into +0.0: the sign-bit test below must see "w - m s < 0" false for it
  const float w[8] = {lo[0] + 0.0f, lo[1] + 0.0f, lo[2] + 0.0f, lo[3] + 0.0f, hi[0] + 0.0f, hi[1] + 0.0f, hi[2] + 0.0f, hi[3] + 0.0f};
  float v[8], m[8], r[8], mc[8], E[8], D[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = w[e] * inv_s;
#pragma unroll
  for (int e = 0; e < 8; ++e) m[e] = __builtin_fmaf(__builtin_fabsf(v[e]), 0x1p-21f, v[e]);
  if constexpr (EQ1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) m[e] += 0.5f;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) m[e] = __builtin_floorf(m[e]);
  if constexpr (!EQ1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = __builtin_fmaf(-m[e], s, w[e]);               // w - m s
    // m -= (r < 0): the sign bit spread over the word selects the bits of 1.0f (no condition register involved)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      m[e] -= __uint_as_float((uint32_t)((int32_t)__float_as_uint(r[e]) >> 31) & 0x3f800000u);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = __builtin_fmaf(0.5f - m[e], s, w[e]);         // w - (m - 1/2) s
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float hm = 0.5f * m[e];
      const bool odd = __builtin_floorf(hm) != hm;
      m[e] -= (r[e] < 0.0f || (r[e] == 0.0f && odd)) ? 1.0f : 0.0f;
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) mc[e] = __builtin_fminf(__builtin_fmaxf(m[e], -kHalf), kHalf - 1.0f);
  // E = (u - z) - w / s;  D = E inside the grid, u - z where clamped: m and mc are integers, so min(|m - mc|, 1) is
  // 0 inside and 1 outside and D = E + (w / s) min(|m - mc|, 1).  b = 1: the code never depends on s, D = u - z.
#pragma unroll
  for (int e = 0; e < 8; ++e) E[e] = (EQ1 ? mc[e] : mc[e] + 0.5f) - v[e];
  if constexpr (BITS > 1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) D[e] = __builtin_fmaf(v[e], __builtin_fminf(__builtin_fabsf(m[e] - mc[e]), 1.0f), E[e]);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) D[e] = mc[e] + 0.5f;
  }
  if constexpr (SALIENT) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if ((sal8 >> e) & 1u) {
        E[e] = ((float)(_Float16)w[e] - w[e]) * inv_s;
        D[e] = 0.0f;
      }
    }
  }
  e_out = u32x4{pack_bf16(E[0], E[1]), pack_bf16(E[2], E[3]), pack_bf16(E[4], E[5]), pack_bf16(E[6], E[7])};
  d_out = u32x4{pack_bf16(D[0], D[1]), pack_bf16(D[2], D[3]), pack_bf16(D[4], D[5]), pack_bf16(D[6], D[7])};
}

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// What a lane holds after the contractions, per row tile and token tile tt: rows 4 g .. 4 g + 3 at token n of
// x E^T (accR) and x D^T (accP).  For one row tile (first row j16): forms r = s accR, sums r^2 and r p over the
// lane's 4 token tiles, then over the 16 lanes that share g (the 16 tokens of a tile), and stores the sums of this
// 64-token group.
__device__ __forceinline__ void store_tile_sums(const StepParams& p, const f32x4 (&accR)[4], const f32x4 (&accP)[4],
                                                int j16, int tg, int n, int g) {
  float* pl = p.partial + (size_t)tg * 2 * p.d_out_pad;
  float* pg = pl + p.d_out_pad;
  const int j = j16 + 4 * g;
  f32x4 sv = {0, 0, 0, 0};
  if (j < p.d_out) sv = *reinterpret_cast<const f32x4*>(p.step + j);   // d_out % 4 == 0
  f32x4 ls = {0, 0, 0, 0}, gs = {0, 0, 0, 0};
#pragma unroll
  for (int tt = 0; tt < 4; ++tt) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float r = (sv[v] > 0.0f ? sv[v] : 0.0f) * accR[tt][v];
      ls[v] += r * r;
      gs[v] += r * accP[tt][v];
    }
  }
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      ls[v] += __shfl_xor(ls[v], off, 64);
      gs[v] += __shfl_xor(gs[v], off, 64);
    }
  }
  if (n == 0) {
    *reinterpret_cast<f32x4*>(pl + j) = ls;
    *reinterpret_cast<f32x4*>(pg + j) = gs;
  }
}

__device__ __forceinline__ void store_group_sums(const StepParams& p, const f32x4 (&accR)[4][4], const f32x4 (&accP)[4][4],
                                                 int j0, int tg, int n, int g) {
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) store_tile_sums(p, accR[rt], accP[rt], j0 + 16 * rt, tg, n, g);
}

// Grid: (d_out_pad / 64, token blocks of 64 NM tokens, n_split); NM + 4 wavefronts in two roles, every SIMD hosting
// one builder and NM / 4 multipliers.
//   builders (the last 4 wavefronts): builder r streams the fp32 delta of row tile r (16 output channels) from
//     memory, two steps of 128 input channels ahead, and builds the operands E and D of the next step into the idle
//     LDS buffer -- vector arithmetic only;
//   multipliers (wavefronts 0 .. NM - 1): every one multiplies all 4 row tiles of the current step (from LDS) with
//     its own 64 tokens, whose activations come straight from memory in fragment order -- matrix instructions only.
// NM = 8 (512 tokens per workgroup: the operands of a mini-batch of calibration tokens are built once; 3 wavefronts
// per SIMD, 168 registers each) or NM = 4 (256 tokens).
// Activations reach a multiplier through a ring in LDS that is its own: asynchronous copies (memory -> LDS, no
// registers) run kXAhead k blocks ahead of the matrix instructions -- a cached load takes longer than the 32 matrix
// instructions of a k block, so a request made only one block ahead would leave the matrix core waiting.
// So the vector unit and the matrix core of a SIMD are fed by different wavefronts and run side by side, and no
// wavefront ever waits on a mix of near (activations, cached) and far (delta, streamed) loads.  One barrier per
// step.  With n_split > 1 (few rows: not enough workgroups otherwise) a workgroup covers a share of the input
// channels and leaves its accumulators to k_step_reduce.
//
// Addresses are clamped instead of guarded: rows past the end repeat the last row and are never reported, columns
// past the end meet activations that are zero, steps past the end rebuild the last step into the idle buffer, a
// token group that is all padding is multiplied like any other.
// The barrier between two steps of the contraction: waits for this wavefront's LDS traffic only.  (__syncthreads()
// would also wait for the memory loads in flight -- the delta values a builder has just requested for a later step,
// the activation copies a multiplier keeps ahead of itself -- a full memory round trip per step.)
__device__ __forceinline__ void step_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int BITS, bool EQ1, int NM>
__global__ __launch_bounds__(64 * (NM + 4), 1) void k_step_grad(const StepParams p) {
  __shared__ __attribute__((aligned(16))) u32x4 afrag[2][4][4][2][64];   // [buffer][row tile][k block][E, D][lane]
  constexpr int XD = NM == 8 ? 3 : 4;                   // ring depth in k blocks: 96 / 64 KiB for all multipliers
  __shared__ __attribute__((aligned(16))) u32x4 xring[NM][XD][4][64];    // [multiplier][slot][token tile][lane]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int j0 = blockIdx.x * kRows;
  const int ks0 = blockIdx.z * p.steps_per_split;
  const int ks1 = ks0 + p.steps_per_split < p.n_steps ? ks0 + p.steps_per_split : p.n_steps;

  if (wave >= NM) {
    // ---- builder: row j0 + 16 rt + n, columns 8 g .. 8 g + 7 of every 32-column block
    const int rt = wave - NM;
    int jrow = j0 + 16 * rt + n;
    const bool row_ok = jrow < p.d_out;
    jrow = row_ok ? jrow : p.d_out - 1;
    float s = row_ok ? p.step[jrow] : 0.0f;
    s = s > 0.0f ? s : 0.0f;
    const float inv_s = s > 0.0f ? 1.0f / s : 0.0f;     // a dead row builds harmless finite operands; its sums are dropped
    const float* drow = p.delta + (size_t)jrow * p.d_in;
    const int c_last = p.d_in - 8;
    f32x4 dl[2][4][2];                                   // delta values of the next two steps to build
    uint32_t sw[2][4];                                   // ... and their salient-column masks: requested together, so
                                                         // that no step waits on a load younger than its delta values
    auto load_delta = [&](int slot, int ks, int kb) {
      ks = ks < ks1 ? ks : ks1 - 1;
      int c = kStepCols * ks + 32 * kb + 8 * g;
      c = c < c_last ? c : c_last;
      dl[slot][kb][0] = *reinterpret_cast<const f32x4*>(drow + c);
      dl[slot][kb][1] = *reinterpret_cast<const f32x4*>(drow + c + 4);
      sw[slot][kb] = p.salmask[4 * ks + kb];
    };
    auto build = [&](int slot, int ks, int kb) {        // dl[slot][kb] (of step ks) -> LDS buffer ks & 1
      const int buf = ks & 1;                           // a step past the end repeats the last one, into the idle buffer
      const uint32_t word = sw[slot][kb];
      const uint32_t sal8 = (word >> (8 * g)) & 0xffu;
      u32x4 ev, dv;
      if (word == 0)                                      // the usual case: none of the 32 columns is salient
        make_operands<BITS, EQ1, false>(dl[slot][kb][0], dl[slot][kb][1], s, inv_s, 0, ev, dv);
      else
        make_operands<BITS, EQ1, true>(dl[slot][kb][0], dl[slot][kb][1], s, inv_s, sal8, ev, dv);
      afrag[buf][rt][kb][0][lane] = ev;
      afrag[buf][rt][kb][1][lane] = dv;
    };
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) load_delta(0, ks0, kb);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) load_delta(1, ks0 + 1, kb);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      build(0, ks0, kb);
      load_delta(0, ks0 + 2, kb);
    }
    __syncthreads();
    // iteration ks builds step ks + 1 (slot alternates 1, 0, 1, ...) and requests step ks + 3 into the same slot
    for (int ks = ks0; ks < ks1; ks += 2) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        build(1, ks + 1, kb);
        load_delta(1, ks + 3, kb);
      }
      step_barrier();
      if (ks + 1 >= ks1) break;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        build(0, ks + 2, kb);
        load_delta(0, ks + 4, kb);
      }
      step_barrier();
    }
    return;
  }

  // ---- multiplier: 64-token group tg, all 4 row tiles
  const int tg = NM * blockIdx.y + wave;
  // activations: k block b (counted from this workgroup's first) goes to ring slot b % XD; blocks past the last
  // one repeat it (requested, never multiplied)
  const char* xbase = reinterpret_cast<const char*>(p.xt + ((size_t)4 * tg) * 64);
  const size_t x_stride = (size_t)p.n_tq * 1024;        // bytes between k blocks
  const int kbg_last = 4 * ks1 - 1;
  auto request_x = [&](int kbg, int slot) {             // 4 copies of 1 KiB: lane l moves 16 bytes
    const char* src = xbase + (size_t)(kbg < kbg_last ? kbg : kbg_last) * x_stride;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      const uint32_t l = (uint32_t)(uintptr_t)&xring[wave][slot][tt][0];
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                   : : "v"((uint32_t)lane * 16u), "s"(src + tt * 1024), "s"(l) : "memory", "m0");
    }
  };
  f32x4 accR[4][4], accP[4][4];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) { accR[rt][tt] = f32x4{0, 0, 0, 0}; accP[rt][tt] = f32x4{0, 0, 0, 0}; }
  // the copies are this wavefront's only memory loads, 4 per k block, completed in order: "at most 4 (XD - 1)
  // outstanding" means the oldest requested block has arrived
  constexpr int kXAhead = 2;                             // copies run two k blocks ahead
#pragma unroll
  for (int b = 0; b < kXAhead; ++b) request_x(4 * ks0 + b, b);
  int slot = 0;                                          // ring slot of the block read next
  // One k block of one step: all 4 row tiles (operands read from LDS one row tile, 8 matrix instructions, ahead of
  // their use) times the 4 token tiles in xb.
  u32x4 ae[2], ad[2];
  auto multiply_block = [&](int cur, int kb, const u32x4 (&xb)[4]) {
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      constexpr int kNone = -1;
      const int rn = rt < 3 ? rt + 1 : 0, kn = rt < 3 ? kb : (kb < 3 ? kb + 1 : kNone);
      if (kn != kNone) {
        ae[(rt + 1) & 1] = afrag[cur][rn][kn][0][lane];
        ad[(rt + 1) & 1] = afrag[cur][rn][kn][1][lane];
      }
      __builtin_amdgcn_sched_barrier(0);                 // keep the reads above ahead of the matrix instructions below
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        accR[rt][tt] = mfma_bf16(ae[rt & 1], xb[tt], accR[rt][tt]);
        accP[rt][tt] = mfma_bf16(ad[rt & 1], xb[tt], accP[rt][tt]);
      }
    }
  };
  // Ring -> registers for k block kbg: request block kbg + 2 first, into the slot that held kbg - 1 (XD = 3) or
  // kbg - 2 (XD = 4); either way a block whose reads were waited for before it was multiplied.
  auto ring_to_regs = [&](int kbg, u32x4 (&dst)[4]) {
    const int ahead = slot + kXAhead < XD ? slot + kXAhead : slot + kXAhead - XD;
    request_x(kbg + kXAhead, ahead);
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(4 * kXAhead) : "memory");
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) dst[tt] = xring[wave][slot][tt][lane];
    slot = slot + 1 < XD ? slot + 1 : 0;
  };
  if constexpr (NM == 8) {
    // 168 registers: one set of activation registers, filled right before use (the SIMD's other multiplier covers
    // the wait)
    __syncthreads();
    for (int ks = ks0; ks < ks1; ++ks) {
      const int cur = ks & 1;
      ae[0] = afrag[cur][0][0][0][lane];
      ad[0] = afrag[cur][0][0][1][lane];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        u32x4 xb[4];
        ring_to_regs(4 * ks + kb, xb);
        multiply_block(cur, kb, xb);
      }
      step_barrier();
    }
  } else {
    // 256 registers: two sets, the next block's activations leave the ring while this block is multiplied
    u32x4 xb[2][4];
    ring_to_regs(4 * ks0, xb[0]);
    __syncthreads();
    for (int ks = ks0; ks < ks1; ++ks) {
      const int cur = ks & 1;
      ae[0] = afrag[cur][0][0][0][lane];
      ad[0] = afrag[cur][0][0][1][lane];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        ring_to_regs(4 * ks + kb + 1, xb[(kb + 1) & 1]);   // (past the last block: a repeat that is never multiplied)
        multiply_block(cur, kb, xb[kb & 1]);
      }
      step_barrier();
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");     // the surplus copies must land before the LDS is given back

  if (p.n_split > 1) {   // this workgroup saw a share of the input channels only: leave the tiles, in thread order
    constexpr int NT = 64 * NM;
    f32x4* t = p.tiles + ((((size_t)blockIdx.z * gridDim.x + blockIdx.x) * gridDim.y + blockIdx.y) * 32) * NT + threadIdx.x;
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        t[(size_t)((rt * 4 + tt) * 2) * NT] = accR[rt][tt];
        t[(size_t)((rt * 4 + tt) * 2 + 1) * NT] = accP[rt][tt];
      }
    return;
  }
  store_group_sums(p, accR, accP, j0, tg, n, g);
}

// Split columns only: adds the accumulator tiles of the splits (in split order) and finishes like the multiplier
// wavefronts of the main kernel.  Grid (row groups, token blocks, 4 row tiles), NM wavefronts laid out like those.
template <int NM>
__global__ __launch_bounds__(64 * NM) void k_step_reduce(const StepParams p) {
  constexpr int NT = 64 * NM;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rt = blockIdx.z;
  f32x4 accR[4], accP[4];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt) { accR[tt] = f32x4{0, 0, 0, 0}; accP[tt] = f32x4{0, 0, 0, 0}; }
  for (int sp = 0; sp < p.n_split; ++sp) {
    const f32x4* t = p.tiles + ((((size_t)sp * gridDim.x + blockIdx.x) * gridDim.y + blockIdx.y) * 32) * NT + threadIdx.x;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      accR[tt] += t[(size_t)((rt * 4 + tt) * 2) * NT];
      accP[tt] += t[(size_t)((rt * 4 + tt) * 2 + 1) * NT];
    }
  }
  store_tile_sums(p, accR, accP, blockIdx.x * kRows + 16 * rt, NM * blockIdx.y + wave, lane & 15, lane >> 4);
}

// loss_j = 1/2 sum over token groups (in order), grad_j likewise; rows with a step that is not positive report 0.
__global__ void k_step_finish(const float* __restrict__ partial, const float* __restrict__ step, int n_tg, int d_out,
                              int d_out_pad, float* __restrict__ loss, float* __restrict__ grad) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d_out) return;
  float l = 0.0f, gsum = 0.0f;
  for (int tg = 0; tg < n_tg; ++tg) {
    l += partial[(size_t)tg * 2 * d_out_pad + j];
    gsum += partial[(size_t)tg * 2 * d_out_pad + d_out_pad + j];
  }
  const bool alive = step[j] > 0.0f;
  loss[j] = alive ? 0.5f * l : 0.0f;
  grad[j] = alive ? gsum : 0.0f;
}

__global__ void k_adamw(float* __restrict__ step, const float* __restrict__ grad, float* __restrict__ m,
                        float* __restrict__ v, int n, float lr, float beta1, float beta2, float eps, float decay,
                        float corr1, float corr2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = grad[i];
  const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
  const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  step[i] = step[i] * decay - lr * (mi / corr1) / (__builtin_sqrtf(vi / corr2) + eps);
}

struct StepLayout {
  size_t xt_at, mask_at, partial_at, tiles_at, total;
  int d_in_pad, d_out_pad, n_tq, n_tg, n_split, steps_per_split, nm, n_tb;
};

StepLayout step_layout(int d_in, int d_out, int n_tokens) {
  StepLayout L;
  L.d_in_pad = ceil_to(d_in, kStepCols);
  L.d_out_pad = ceil_to(d_out, kRows);
  const int n_blocks = (n_tokens + kTokBlock - 1) / kTokBlock;
  L.n_tq = 16 * n_blocks;
  L.n_tg = 4 * n_blocks;
  size_t at = 0;
  L.xt_at = at;
  at += (size_t)(L.d_in_pad / 32) * L.n_tq * 1024;
  L.mask_at = at;
  at += ((size_t)(L.d_in_pad / 32) * 4 + 255) / 256 * 256;
  L.partial_at = at;
  at += (size_t)L.n_tg * 2 * L.d_out_pad * 4;
  // One workgroup (8 wavefronts with 256 registers each) per compute unit, 256 units: with fewer workgroups
  // than that the input channels are split.
  const int n_steps = L.d_in_pad / kStepCols;
  // 512 tokens per workgroup when that pads the batch no further than 256 would, else 256
  const bool wide = n_tokens > kTokBlock && n_blocks % 2 == 0;
  L.nm = wide ? 8 : 4;
  L.n_tb = wide ? n_blocks / 2 : n_blocks;
  const long base = (long)(L.d_out_pad / kRows) * L.n_tb;
  int want = base > 0 ? (int)(256 / base) : 1;
  want = want < 1 ? 1 : (want > 8 ? 8 : want);
  L.steps_per_split = (n_steps + want - 1) / want;
  if (L.steps_per_split < 4) L.steps_per_split = n_steps < 4 ? n_steps : 4;
  L.n_split = (n_steps + L.steps_per_split - 1) / L.steps_per_split;
  at = (at + 255) / 256 * 256;
  L.tiles_at = at;
  if (L.n_split > 1) at += (size_t)L.n_split * base * 32 * (64 * L.nm) * 16;
  L.total = at < 256 ? 256 : at;
  return L;
}

template <int BITS, int NM>
hipError_t launch_grid_variants(const StepParams& p, bool eq1, dim3 grid, hipStream_t s) {
  if constexpr (BITS > 1) {
    if (eq1) { k_step_grad<BITS, true, NM><<<grid, 64 * (NM + 4), 0, s>>>(p); return hipGetLastError(); }
  }
  k_step_grad<BITS, false, NM><<<grid, 64 * (NM + 4), 0, s>>>(p);
  return hipGetLastError();
}

template <int NM>
hipError_t launch_bits(const StepParams& p, int bits, bool eq1, dim3 grid, hipStream_t s) {
  switch (bits) {
    case 1: return launch_grid_variants<1, NM>(p, false, grid, s);
    case 2: return launch_grid_variants<2, NM>(p, eq1, grid, s);
    case 3: return launch_grid_variants<3, NM>(p, eq1, grid, s);
    default: return launch_grid_variants<4, NM>(p, eq1, grid, s);
  }
}

}  // namespace

size_t step_grad_workspace_bytes(int d_in, int d_out, int n_tokens) { return step_layout(d_in, d_out, n_tokens).total; }

hipError_t launch_step_grad(const float* delta, int d_in, int d_out, const int32_t* sidx, int k, int bits, int grid,
                            const float* step, const void* x, int n_tokens, float* loss, float* grad, void* ws,
                            hipEvent_t ev_start, hipEvent_t ev_stop, hipStream_t s) {
  const StepLayout L = step_layout(d_in, d_out, n_tokens);
  char* w = reinterpret_cast<char*>(ws);
  StepParams p;
  p.delta = delta;
  p.step = step;
  p.salmask = reinterpret_cast<const uint32_t*>(w + L.mask_at);
  p.xt = reinterpret_cast<const u32x4*>(w + L.xt_at);
  p.partial = reinterpret_cast<float*>(w + L.partial_at);
  p.d_in = d_in;
  p.d_out = d_out;
  p.d_out_pad = L.d_out_pad;
  p.n_tokens = n_tokens;
  p.n_tq = L.n_tq;
  p.n_steps = L.d_in_pad / kStepCols;
  p.tiles = reinterpret_cast<f32x4*>(w + L.tiles_at);
  p.n_split = L.n_split;
  p.steps_per_split = L.steps_per_split;
  hipError_t e;
  if (n_tokens > 0) {
    const size_t n_blk = (size_t)(L.d_in_pad / 32) * L.n_tq;   // a multiple of 4
    k_tile_x<<<(unsigned)(n_blk / 4) + 1, 256, 0, s>>>(reinterpret_cast<const uint16_t*>(x), n_tokens, d_in, L.n_tq,
                                                        reinterpret_cast<u32x4*>(w + L.xt_at), sidx, k, L.d_in_pad / 32,
                                                        reinterpret_cast<uint32_t*>(w + L.mask_at));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const dim3 g(L.d_out_pad / kRows, L.n_tb, L.n_split);
    if (ev_start && (e = hipEventRecord(ev_start, s)) != hipSuccess) return e;
    const bool eq1 = grid == MES_GRID_EQ1;
    e = L.nm == 8 ? launch_bits<8>(p, bits, eq1, g, s) : launch_bits<4>(p, bits, eq1, g, s);
    if (e != hipSuccess) return e;
    if (L.n_split > 1) {
      if (L.nm == 8) k_step_reduce<8><<<dim3(g.x, g.y, 4), 512, 0, s>>>(p);
      else k_step_reduce<4><<<dim3(g.x, g.y, 4), 256, 0, s>>>(p);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (ev_stop && (e = hipEventRecord(ev_stop, s)) != hipSuccess) return e;
  }
  k_step_finish<<<(d_out + 255) / 256, 256, 0, s>>>(p.partial, step, n_tokens > 0 ? L.n_tg : 0, d_out, L.d_out_pad, loss, grad);
  return hipGetLastError();
}

hipError_t launch_adamw(float* step, const float* grad, float* m, float* v, int n, int t, float lr, float beta1,
                        float beta2, float eps, float weight_decay, hipStream_t s) {
  const double c1 = 1.0 - pow((double)beta1, (double)t), c2 = 1.0 - pow((double)beta2, (double)t);
  const float decay = (float)(1.0 - (double)lr * (double)weight_decay);
  k_adamw<<<(n + 255) / 256, 256, 0, s>>>(step, grad, m, v, n, lr, beta1, beta2, eps, decay, (float)c1, (float)c2);
  return hipGetLastError();
}

}  // namespace mes
