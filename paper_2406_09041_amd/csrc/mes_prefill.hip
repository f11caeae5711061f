// Long token segments (prefill): one product per expert, y_e = x_e (W + Delta~_e)^T  -- Eq. 4 before it is
// decoupled.  With hundreds of tokens on one expert the layer is a dense contraction bound by the matrix cores,
// not by weight bytes, and streaming the weights once per 64 tokens (the decode kernel) wastes both.  Here the
// expert's effective weight is formed in registers, never in memory: per 16 x 32 block, bf16(W + (u - z) s) from
// the tiled base weight and the packed codes, as the A operand of the bf16 matrix instruction.  Salient input
// channels store code 0, so the main product carries (0 - z) s for them; a short second part of the contraction,
// over the gathered salient activations, adds bf16(Delta_S + z s) (Delta_S: the stored fp16 values).
// The rounding of the operands to bf16 adds a relative error of about 2^-9 / sqrt(3) to y, the same size as the
// rounding of y itself.
#include <type_traits>

#include "mes_internal.h"
#include "mes_prefill_plan.h"

namespace mes {
namespace {

typedef __attribute__((__vector_size__(16))) uint32_t u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;

constexpr int kWaves = 8;
constexpr int kMaxGridY = 65535;     // token blocks of one launch
static_assert(kRowPad == 64, "row_tiles() of the plan");

// Per layer of a call; per segment (= per expert with a long segment): codes, step, sal.
struct PrefillLinear {
  const u32x4* base;        // tiled base weight: block (chunk c, row tile jt) = [4 k blocks][64 lanes] x 16 bytes
  uint16_t* y;              // bf16 [T, d_out]
  const uint32_t* codes[kMaxSegs];   // packed codes: block (c, jt) = 64 * bits words
  const float* step[kMaxSegs];       // [d_out]
  const u32x4* sal[kMaxSegs];        // salient tile: ((jt * n_sb + sb) * 64 + lane) x 8 fp16
  int d_out, n_jt;
  int rg_begin, rg_end;     // its row groups among the launch's
};

struct PrefillParams {
  PrefillLinear lin[MES_MAX_FUSED];
  int t_begin[kMaxSegs], t_end[kMaxSegs];   // a segment's rows of x and y
  int tile0[kMaxSegs];                      // its first token tile in xt
  Blocks blocks;            // the token blocks
  const u32x4* xt;          // the segments' activations in fragment order: [k block][token tile][64 lanes] x 16 bytes,
                            // k blocks 0 .. 4 n_chunks - 1 the input channels, then 4 n_ssteps per layer of gathered salient ones
  f32x4* tiles;             // split contraction only: accumulator tiles, [split][row group][token block][4 RT][thread]
  int n_rg, n_blk, n_chunks, n_sb, n_ssteps, n_tq, steps_per_split, n_split;
  float z;
};

// Token tiles a wavefront takes of a block: of up to 16 tiles four columns of wavefronts share the tokens, and the two of a
// column the k blocks; of more, eight.
__host__ __device__ constexpr int wave_tiles(int tiles) { return tiles > 24 ? 4 : tiles > 16 ? 3 : (tiles + 3) / 4; }

// What a workgroup's start depends on, from the arguments in one trip: one after the other, as the compiler has it, each is
// another 0.3 us of a call.
struct Place {
  TokenBlock tb;
  int l, n_chunks, n_ssteps, steps_per_split;
};
__device__ __forceinline__ Place place_of(const PrefillParams& p, int rg, int blk) {
  auto now = [](int& v) { asm volatile("" : "+s"(v)); };
  BlockEntry e = p.blocks.list[blk < kMaxBlocks ? blk : 0];
  int n_list = p.blocks.n_list, rg_end[MES_MAX_FUSED - 1];
  Place at{{}, 0, p.n_chunks, p.n_ssteps, p.steps_per_split};
#pragma unroll
  for (int i = 0; i + 1 < MES_MAX_FUSED; ++i) rg_end[i] = p.lin[i].rg_end;
  now(e.tile0); now(e.shape); now(n_list); now(at.n_chunks); now(at.n_ssteps); now(at.steps_per_split);
#pragma unroll
  for (int i = 0; i + 1 < MES_MAX_FUSED; ++i) {            // (of layers that are not there: all the launch's row groups)
    now(rg_end[i]);
    at.l += rg >= rg_end[i] ? 1 : 0;
  }
  at.tb = blk < n_list ? token_block(e) : unlisted_block(p.blocks, blk - n_list);
  return at;
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const bf16x2 h = __builtin_convertvector(f32x2{a, b}, bf16x2);   // round to nearest even
  return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The barrier between two steps: waits for this wavefront's LDS traffic only.  (__syncthreads() would also wait for
// the memory loads in flight: weights and activations of later steps, a full memory round trip per step.)
__device__ __forceinline__ void step_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Loads as (wave-uniform address) + (32-bit lane offset).
typedef __attribute__((address_space(1))) const char global_char;
__device__ __forceinline__ u32x4 load128(uint64_t uniform, uint32_t off) {
  return *reinterpret_cast<__attribute__((address_space(1))) const u32x4*>(reinterpret_cast<global_char*>(uniform) + off);
}
__device__ __forceinline__ uint32_t load32(uint64_t uniform, uint32_t off) {
  return *reinterpret_cast<__attribute__((address_space(1))) const uint32_t*>(reinterpret_cast<global_char*>(uniform) + off);
}
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}
// A lane offset of this step: the compiler cannot widen it to 64 bits ahead of the loop, which would take the loads off the
// scalar base + 32-bit offset form and cost vector arithmetic and registers.
__device__ __forceinline__ uint32_t here(uint32_t v) { asm volatile("" : "+v"(v)); return v; }

struct TileParams {
  const uint16_t* x;
  const int32_t* sidx[MES_MAX_FUSED][kMaxSegs];
  int t_begin[kMaxSegs], t_end[kMaxSegs], tile0[kMaxSegs];
  int n_seg, k, d_in, n_chunks, n_ssteps, n_tq;
  int u_begin, n_units;     // this launch writes the units u_begin .. u_begin + n_units - 1 (see below)
  u32x4* xt;
};

// The segments' rows of x -> fragment order.  A wavefront writes one unit of one token tile tq: unit u < n_chunks are the four
// k blocks of input channels 128 u .. 128 u + 127, the units behind them, 4 n_ssteps per layer, one k block of 32 of the
// layer's salient channels each.  Block (kb, tq), lane l: token 16 tq' + (l & 15) of the segment that tq belongs to (tq'
// counted from the segment's first tile); the 8 input channels 32 kb + 8 (l >> 4) .., or the 8 salient channels of that
// segment's expert with ranks 32 kb + 8 (l >> 4) ..; zero beyond the segment's last token, the last channel or rank.
// Bound by memory latency: a lane has four loads in flight, the wavefront 256 bytes of each of 16 rows.  (Gathers take a
// cycle per lane and a second trip: four k blocks of them in one wavefront were the launch's last to end, 1536 tokens x 4096
// channels, 128 salient ones, 19.5 us against 9.7.  The stored ranks are padded to 128: gathering the padding as well took
// 64000 tokens x 512 channels, 8 salient ones, 2.5 to 4 us of a call of 54, small calls 0.5 us.)
__global__ __launch_bounds__(256) void k_prefill_tile_x(const TileParams p) {
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const long w = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= (long)p.n_units * p.n_tq) return;
  const int tq = (int)(w / p.n_units), u = p.u_begin + (int)(w - (long)tq * p.n_units);
  int sg = 0;
#pragma unroll
  for (int i = 1; i < kMaxSegs; ++i) sg += (i < p.n_seg && tq >= p.tile0[i]) ? 1 : 0;
  const int t = p.t_begin[sg] + 16 * (tq - p.tile0[sg]) + (lane & 15);
  const bool live = t < p.t_end[sg];
  const uint16_t* row = p.x + (size_t)(live ? t : p.t_begin[sg]) * p.d_in;
  if (u < p.n_chunks) {
    u32x4 v[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      const int c = 128 * u + 32 * kb + 8 * g;     // d_in % 8 == 0
      v[kb] = *reinterpret_cast<const u32x4*>(row + (c < p.d_in ? c : p.d_in - 8));
      if (!live || c >= p.d_in) v[kb] = u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) p.xt[((size_t)(4 * u + kb) * p.n_tq + tq) * 64 + lane] = v[kb];
  } else {
    const int l = (u - p.n_chunks) / (4 * p.n_ssteps), r0 = 32 * (u - p.n_chunks - 4 * l * p.n_ssteps) + 8 * g;
    const int32_t* sidx = p.sidx[l][sg];
    uint32_t h[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (live && r0 < p.k) {                              // (lanes of ranks past the last one have nothing to gather)
      int c[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) c[q] = sidx[r0 + q < p.k ? r0 + q : p.k - 1];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const bool valid = r0 + q < p.k && (uint32_t)c[q] < (uint32_t)p.d_in;   // a corrupt list can never address outside the row
        h[q] = row[valid ? c[q] : 0];
        if (!valid) h[q] = 0;
      }
    }
    p.xt[((size_t)(3 * p.n_chunks + u) * p.n_tq + tq) * 64 + lane] =
        u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
  }
}

// What a wavefront keeps in flight of a later step's weights: its NOP of the step's 4 RT operands.
template <int BITS, int NOP>
struct StepData {
  u32x4 w[NOP];                                // base fragment (main step) or 8 fp16 salient values (salient step)
  uint32_t lo[NOP], hi[BITS >= 3 ? NOP : 1];   // code words
};

// One workgroup's share of the launch: RT row tiles (16 output channels each) of row group rg of a layer x one token block,
// the steps st0 .. st1 - 1.  A step is 128 input channels (or 128 salient ranks), 4 k blocks.  All eight wavefronts do both
// halves of the work:
//   multiply: every wavefront has token tiles of its own (TT of them) and takes all RT operands of its k blocks from LDS;
//     activations come straight from memory, already in fragment order, XD - 1 k blocks ahead.  KS = 1: all 4 k blocks of a
//     step, 8 x TT token tiles per workgroup.  KS = 2 (blocks of up to 16 tiles, but see SHORT): wavefronts w and w + 4 share the token tiles
//     and take two k blocks each; the sums meet in LDS at the end.  So both wavefronts of a SIMD multiply, whatever the block.
//   build: wavefront w forms the operands (row tiles w / 4 + 2 i, k block w % 4) of the next step in the idle LDS buffer,
//     bf16(W + (u - z) s) from a base fragment and a code word that were asked for a step before.  The vector instructions
//     for it are dealt out between the matrix instructions.
// Both wavefronts of a SIMD thereby have matrix instructions ready most of the time, and a weight is formed once per 512
// tokens; a workgroup with builders and multipliers as roles of different wavefronts formed it once per 256, had one
// multiplier per SIMD and lost that one's waits.
template <int BITS, int RT, int TT, int KS>
__device__ __forceinline__ void multiply_rows(const PrefillParams& p, const PrefillLinear& L, int l, const TokenBlock& tb, u32x4* lds,
                                              int wave, int rg, int blk, int st0, int st1) {
  constexpr int NOP = (4 * RT + kWaves - 1) / kWaves;
  constexpr int NBW = 4 / KS;                            // k blocks of a step this wavefront multiplies
  constexpr int OPB = NOP / NBW;                         // operands built under one of them
  // Sets of activation fragments: what the registers hold (512 of them per lane and SIMD, two wavefronts) with nothing put aside
  // in the main loop.  (The last steps of the bodies of 4 tiles and 8 rows do put 20 to 55 registers aside.  A third set at 3 and
  // 4 bits with 8 rows had scratch accesses in every main step: 4096 tokens of 4 experts on 14336 -> 4096, 3 / 4 bits 466 / 460
  // us, with two sets 446 / 452; at 1 and 2 bits two sets instead of three are 4 % slower, and so are blocks of 17 to 24 tiles at 3
  // and 4 bits, by 1 to 2 %: 13248 -> 8048, 491 + 567 tokens, 3 bits, 276 us with two, 271 with three.)
  constexpr int XD = TT == 0 ? 1 : TT <= 2 ? 4 : KS == 2 ? 2 : (RT == 7 ? (BITS <= 2 ? 4 : 3) : BITS <= 2 || TT == 3 ? 3 : 2);
  constexpr int U = NBW % XD == 0 ? 1 : (2 * NBW) % XD == 0 ? 2 : 3;   // steps until the sets come round
  static_assert((U * NBW) % XD == 0, "the sets are named at compile time");
  static_assert(NOP % NBW == 0, "every k block has the same number of operands to build");
  constexpr int TA = TT > 0 ? TT : 1;
  constexpr int kBuf = RT * 4 * 1024, kSpare = 2 * kBuf;
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int half = KS == 2 ? wave >> 2 : 0, col = KS == 2 ? wave & 3 : wave;
  const uint32_t lane16 = (uint32_t)lane * 16u;
  const int sg = tb.sg;
  char* const ldsc = reinterpret_cast<char*>(lds);

  // ---- weights
  const int bkb = wave & 3, brt = wave >> 2;
  const int n_jt = L.n_jt, n_sb = p.n_sb, n_chunks = p.n_chunks;
  const float z = p.z;
  uint32_t jt[NOP];
  float s[NOP];
#pragma unroll
  for (int i = 0; i < NOP; ++i) {                        // stored matrices are padded to whole groups of 4 row tiles: a last
    const int j = RT * (rg - L.rg_begin) + brt + 2 * i;  // group may repeat tiles (its rows are never stored)
    jt[i] = j < n_jt ? j : n_jt - 1;
    const int row = 16 * (int)jt[i] + n;
    s[i] = L.step[sg][row < L.d_out ? row : L.d_out - 1];
  }
  // the code block's lane 16 kb + n owns columns 32 kb + 8 g + 0 .. 7 of row n
  uint32_t wl = lane16, co = (BITS == 1 ? 16 * bkb + n : 2 * (16 * bkb + n) + (g >> 1)) * 4u;
  uint32_t coh = BITS == 3 ? 512u + (16 * bkb + n) * 4u : 512u + co;
  const uint64_t codes = reinterpret_cast<uint64_t>(L.codes[sg]);
  const uint64_t base = reinterpret_cast<uint64_t>(L.base) + bkb * 1024;
  const uint64_t sal = reinterpret_cast<uint64_t>(L.sal[sg]);
  using SD = StepData<BITS, NOP>;
  uint64_t w_at, c_at;                                   // where the weights of the step asked for next are
  uint32_t w_mul;
  auto aim = [&](int st) {
    st = st < st1 ? st : st1 - 1;
    const bool main_step = st < n_chunks;                // (a salient step re-reads code words it never uses)
    const uint32_t c = main_step ? st : n_chunks - 1;
    int sb = 4 * (st - n_chunks) + bkb;
    sb = sb < n_sb ? sb : n_sb - 1;                      // past the last salient block: repeated, zeroed when built
    c_at = uniform64(codes + (uint64_t)c * (uint32_t)(n_jt * 256 * BITS));
    const uint64_t wm = base + (uint64_t)c * (uint32_t)n_jt * 4096, ws = sal + (uint64_t)(uint32_t)sb * 1024;
    w_at = uniform64(main_step ? wm : ws);
    w_mul = __builtin_amdgcn_readfirstlane(main_step ? 4096 : n_sb * 1024);
  };
  auto fetch = [&](SD& d, int i) {
    d.w[i] = load128(w_at + (uint64_t)jt[i] * w_mul, wl);
    const uint64_t cw = c_at + jt[i] * (256u * BITS);
    d.lo[i] = load32(cw, co);
    if constexpr (BITS >= 3) d.hi[i] = load32(cw, coh);
  };
  auto store_operand = [&](int i, int buf, const u32x4& v) {
    const int rt = brt + 2 * i;                          // (odd RT: half of the wavefronts have one operand less, and put
    const int at = 2 * i + 1 < RT || rt < RT ? buf * kBuf + (rt * 4 + bkb) * 1024 : kSpare;   // theirs where nobody reads)
    *reinterpret_cast<u32x4*>(ldsc + at + lane16) = v;
  };
  // An operand's way from weights and codes to LDS, in parts of one to three vector instructions: 0 the code fields, 1 .. 16
  // four parts for each pair of values, 17 the store, 18 the request for the same place's weights of the step after next.
  constexpr int kParts = 19;
  u32x4 out;
  uint32_t c0, c1;
  float nzs, v0, v1, w1;
  auto fp4 = [](uint32_t v, int q) -> f32x2 {            // byte q's two code fields, u / 2 as fp4 numbers, times two
    switch (q) {
      case 0: return __builtin_bit_cast(f32x2, __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(v, 2.0f, 0));
      case 1: return __builtin_bit_cast(f32x2, __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(v, 2.0f, 1));
      case 2: return __builtin_bit_cast(f32x2, __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(v, 2.0f, 2));
      default: return __builtin_bit_cast(f32x2, __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(v, 2.0f, 3));
    }
  };
  auto build_part = [&](SD& d, int i, int part, int buf) {
    if (part == 0) {
      nzs = -(z * s[i]);
      c0 = BITS == 1 ? (d.lo[i] >> g) & 0x11111111u : (d.lo[i] >> (2 * (g & 1))) & 0x33333333u;
      if constexpr (BITS >= 3) {                         // whole codes, the even columns' in the bytes of c0, the odd ones' in c1
        const uint32_t c = c0 | (BITS == 3 ? (d.hi[i] >> g) & 0x11111111u : (d.hi[i] >> (2 * (g & 1))) & 0x33333333u) << 2;
        c0 = c & 0x0f0f0f0fu;
        c1 = (c >> 4) & 0x0f0f0f0fu;
      }
    } else if (part <= 16) {
      const int q = (part - 1) >> 2;
      const uint32_t ww = d.w[i][q];
      switch ((part - 1) & 3) {
        case 0:
          if constexpr (BITS >= 3) {
            v0 = (float)((c0 >> (8 * q)) & 0xffu);
            v1 = (float)((c1 >> (8 * q)) & 0xffu);
          } else {
            const f32x2 u = fp4(c0, q);
            v0 = u[0]; v1 = u[1];
          }
          break;
        case 1: v0 = __builtin_fmaf(v0, s[i], nzs); v1 = __builtin_fmaf(v1, s[i], nzs); break;   // (u - z) s
        case 2: v0 = bf16_lo(ww) + v0; w1 = bf16_hi(ww); break;
        default: out[q] = pack_bf16(v0, w1 + v1); break;
      }
    } else if (part == 17) {
      store_operand(i, buf, out);
    } else {
      fetch(d, i);
    }
  };
  auto build_any = [&](SD& d, int i, int st, int buf) {  // a whole operand of any step (past the last: repeated, never read)
    st = st < st1 ? st : st1 - 1;
    if (st < n_chunks) {
#pragma unroll
      for (int part = 0; part < 17; ++part) build_part(d, i, part, buf);
    } else {
      out = u32x4{0, 0, 0, 0};
      if (4 * (st - n_chunks) + bkb < n_sb) {            // ranks past k hold 0 and meet activations that are 0
        const float zs = z * s[i];
        const f16x8 h = __builtin_bit_cast(f16x8, d.w[i]);
#pragma unroll
        for (int q = 0; q < 4; ++q) out[q] = pack_bf16((float)h[2 * q] + zs, (float)h[2 * q + 1] + zs);
      }
    }
    store_operand(i, buf, out);
  };

  // ---- activations: this wavefront's k blocks one after the other, the last one repeated
  const uint64_t x_stride = tile_offset(p.n_tq);         // from a k block to the next
  const uint64_t x_jump = (uint64_t)(4 * p.n_ssteps * l) * x_stride;   // over the other layers' salient channels
  uint32_t toff[TA];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {                      // tiles past the block's last one repeat it, and are not stored
    const int t = TT * col + tt;                         // (offsets within the block: a launch may have more than 2^22 tiles)
    toff[tt] = __builtin_amdgcn_readfirstlane((uint32_t)(t < tb.tiles ? t : tb.tiles - 1) * (uint32_t)kTileBytes);
  }
  u32x4 xb[XD][TA];
  uint64_t x_at = uniform64(reinterpret_cast<uint64_t>(p.xt) + tile_offset(tb.tile0) + (uint64_t)(4 * st0 + NBW * half) * x_stride +
                            (st0 >= n_chunks ? x_jump : 0));
  int x_left = (st1 - st0) * NBW - 1, x_cross = (n_chunks - st0) * NBW;   // blocks behind the next one; until the salient ones
  auto request_x = [&](int j, int set) {                 // j: the block's number among those of its step
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) xb[set][tt] = load128(x_at + toff[tt], wl);
    const uint64_t by = (KS == 2 && j == NBW - 1 ? 3 * x_stride : x_stride) + (--x_cross == 0 ? x_jump : 0);
    x_at += x_left > 0 ? by : 0;
    --x_left;
  };

  f32x4 acc[RT][TA];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) acc[rt][tt] = f32x4{0, 0, 0, 0};

  SD sd;
  {
    SD s0;
    aim(st0);
#pragma unroll
    for (int i = 0; i < NOP; ++i) fetch(s0, i);
    aim(st0 + 1);
    if constexpr (TT > 0) {
#pragma unroll
      for (int j = 0; j < XD - 1 - NBW; ++j) request_x(j % NBW, j);
    }
    // in the loop's order, so that the loop's waits let the same loads stay in flight in its first round
#pragma unroll
    for (int b = 0; b < NBW; ++b) {
      if constexpr (TT > 0)
        if (b - NBW + XD - 1 >= 0) request_x((b + XD - 1) % NBW, b - NBW + XD - 1);
#pragma unroll
      for (int o = 0; o < OPB; ++o) fetch(sd, b * OPB + o);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < NOP; ++i) build_any(s0, i, st0, st0 & 1);
  }
  step_barrier();

  // One step: multiplies the operands of step st, builds those of st + 1, asks for the weights of st + 2.  MAIN: step st + 1
  // is one of the main steps.  u: the step's number modulo U.
  auto step = [&](auto main_step, int u, int st) {
    constexpr bool MAIN = decltype(main_step)::value;
    aim(st + 2);
    wl = here(wl); co = here(co);
    if constexpr (BITS >= 3) coh = here(coh);
    const int nbuf = (st + 1) & 1;
    const char* cur = ldsc + (st & 1) * kBuf + (half * NBW) * 1024 + lane16;
    auto a_at = [&](int b, int rt) { return *reinterpret_cast<const u32x4*>(cur + (rt * 4 + b) * 1024); };
    u32x4 a[2];                                          // operands are read from LDS one row tile ahead of their use
    if constexpr (TT > 0) a[0] = a_at(0, 0);
#pragma unroll
    for (int b = 0; b < NBW; ++b) {
      if constexpr (TT > 0) request_x((b + XD - 1) % NBW, (u * NBW + b + XD - 1) % XD);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if constexpr (TT > 0) {
          const int at = b * RT + rt, next = at + 1;
          if (next < NBW * RT) a[next & 1] = a_at(next / RT, next % RT);
          __builtin_amdgcn_sched_barrier(0);             // keep the read above ahead of the matrix instructions below
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) {
            acc[rt][tt] = mfma_bf16(a[at & 1], xb[(u * NBW + b) % XD][tt], acc[rt][tt]);
            if constexpr (MAIN) {
              constexpr int P = OPB * kParts, M = RT * TT;
              const int m = rt * TT + tt;
#pragma unroll
              for (int pp = P * m / M; pp < P * (m + 1) / M; ++pp) build_part(sd, b * OPB + pp / kParts, pp % kParts, nbuf);
              __builtin_amdgcn_sched_barrier(0);         // and the parts where they were dealt to
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (MAIN) {
          if (TT == 0 && rt == 0) {
#pragma unroll
            for (int pp = 0; pp < OPB * kParts; ++pp) build_part(sd, b * OPB + pp / kParts, pp % kParts, nbuf);
          }
        } else {
#pragma unroll
          for (int o = 0; o < OPB; ++o)
            if (rt == 2 + 2 * o) {
              build_any(sd, b * OPB + o, st + 1, nbuf);
              fetch(sd, b * OPB + o);
            }
        }
      }
    }
    step_barrier();
  };
  int st = st0;
  for (; st + U < st1 && st + U < n_chunks; st += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) step(std::true_type{}, u, st + u);
  }
  for (; st < st1; st += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (st + u >= st1) break;
      step(std::false_type{}, u, st + u);
    }
  }

  if constexpr (TT == 0) return;
  if constexpr (KS == 2) {                               // the other half's sums (the operands are done with)
    f32x4* xch = reinterpret_cast<f32x4*>(lds) + (size_t)col * (RT * TT * 64);
    if (half == 1) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) xch[(rt * TT + tt) * 64 + lane] = acc[rt][tt];
    }
    __syncthreads();
    if (half == 1) return;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) acc[rt][tt] += xch[(rt * TT + tt) * 64 + lane];
  }
  if (p.n_split > 1) {   // this workgroup saw a share of the contraction only: leave the tiles, in thread order
    constexpr int NT = 64 * kWaves;
    f32x4* t = p.tiles + (((size_t)blockIdx.z * p.n_rg + rg) * p.n_blk + blk) * (RT * 4) * NT + threadIdx.x;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) t[(size_t)(rt * 4 + tt) * NT] = acc[rt][tt];
    return;
  }
  // this lane holds, per row tile and token tile, rows 4 g .. 4 g + 3 at token n
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int j = 16 * (RT * (rg - L.rg_begin) + rt) + 4 * g;
    if (j >= L.d_out) continue;                          // d_out % 4 == 0
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int tile = TT * col + tt;
      const int t = p.t_begin[sg] + 16 * (tb.tile0 + tile - p.tile0[sg]) + n;
      if (tile < tb.tiles && t < p.t_end[sg]) {
        const f32x4 o = acc[rt][tt];
        uint2 pk;
        pk.x = pack_bf16(o[0], o[1]);
        pk.y = pack_bf16(o[2], o[3]);
        *reinterpret_cast<uint2*>(L.y + (size_t)t * L.d_out + j) = pk;
      }
    }
  }
}

// Grid: (row groups of 16 RT output channels of all layers of the call, token blocks of up to 512 tokens, n_split); 512
// threads, one workgroup per compute unit.
// What bounds it: 1536 tokens of 3 experts on 4096 -> 14336, 2 bits, 181 us (before, with roles, 209): the matrix pipes are busy for 54 %
// of a workgroup's time (56 to 64 % in full blocks of 8 row tiles), 2.55 GB leave the L2s.  Without activation loads 168, without
// weight and code loads 162, without the operands' arithmetic 167; on zero activations, with less power, 155.
// SHORT: launches of short contractions, no block of more than 16 tiles, n_split = 1.  Blocks of 13 to 16 tiles take eight
// columns of two tiles there: the operands are read from LDS twice as often, but there are no sums to exchange at the end, about 1 us.
// (784 tokens x 7448, 3 / 13 / 25 / 33 / 49 steps, four columns 20.3 / 36.6 / 59.0 / 76.7 / 104.6 us, eight 19.4 / 34.7 / 58.5 /
// 77.2 / 105.2; 490 x 12992, 1 bit, 3 / 17 / 33 / 49 steps 20.5 / 45.5 / 77.5 / 105.3 against 19.6 / 45.2 / 77.6 / 111.4.  Of 9 to
// 12 tiles eight columns would leave two without tokens: slower from 5 steps on, 1470 x 4096, 3 bits, 22.0 against 22.3; in
// split contractions the exchange is not what counts, 1024 x 1024 on 1024 channels 18.9 against 19.9.  Kernels of their
// own: one more body in the others moves their spilled registers about, up to 20 % at 3 bits.)
constexpr int kShortSteps = 20;
template <int BITS, int RT, bool SHORT>
__global__ __launch_bounds__(64 * kWaves) void k_prefill_fused(const PrefillParams p) {
  // two operand buffers of 4 RT KiB and, behind them, the operand too many; at the end 16 RT KiB of sums (KS = 2)
  __shared__ __attribute__((aligned(16))) u32x4 lds[RT * 4 * 4 * 64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rg = blockIdx.x, blk = blockIdx.y;
  const Place at = place_of(p, rg, blk);
  const int n_steps = at.n_chunks + at.n_ssteps;
  const int st0 = blockIdx.z * at.steps_per_split;
  const int st1 = st0 + at.steps_per_split < n_steps ? st0 + at.steps_per_split : n_steps;
  const int l = at.l;
  const PrefillLinear& L = p.lin[l];
  const TokenBlock tb = at.tb;
  if constexpr (SHORT) {
    if (tb.tiles > 12) {
      if (2 * wave >= tb.tiles) multiply_rows<BITS, RT, 0, 1>(p, L, l, tb, lds, wave, rg, blk, st0, st1);   // builds only
      else multiply_rows<BITS, RT, 2, 1>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
    } else if (tb.tiles > 8) {
      multiply_rows<BITS, RT, 3, 2>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
    } else if (tb.tiles > 4) {
      multiply_rows<BITS, RT, 2, 2>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
    } else {
      multiply_rows<BITS, RT, 1, 2>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
    }
  } else if (tb.tiles > 16) {
    const int tt = wave_tiles(tb.tiles);
    if (tt * wave >= tb.tiles) multiply_rows<BITS, RT, 0, 1>(p, L, l, tb, lds, wave, rg, blk, st0, st1);   // builds only
    else if (tt == 4) multiply_rows<BITS, RT, 4, 1>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
    else multiply_rows<BITS, RT, 3, 1>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
  } else if (tb.tiles > 12) {
    multiply_rows<BITS, RT, 4, 2>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
  } else if (tb.tiles > 8) {
    multiply_rows<BITS, RT, 3, 2>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
  } else if (tb.tiles > 4) {
    multiply_rows<BITS, RT, 2, 2>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
  } else {
    multiply_rows<BITS, RT, 1, 2>(p, L, l, tb, lds, wave, rg, blk, st0, st1);
  }
}

// Split contraction only: y = sum over splits (in split order) of the accumulator tiles, rounded to bf16.
// Grid (row groups, token blocks, 4 RT tiles), wavefronts laid out like those of the main kernel that hold sums; one tile (row tile
// rt = z / 4, token tile tt = z % 4) of each per workgroup.
template <int RT>
__global__ __launch_bounds__(64 * kWaves) void k_prefill_reduce(const PrefillParams p) {
  constexpr int NT = 64 * kWaves;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15, g = lane >> 4;
  const int rg = blockIdx.x, blk = blockIdx.y, rt = blockIdx.z >> 2, tt = blockIdx.z & 3;
  const Place at = place_of(p, rg, blk);
  const TokenBlock tb = at.tb;
  const int TT = wave_tiles(tb.tiles), tile = TT * wave + tt;
  if (tt >= TT || tile >= tb.tiles) return;
  const PrefillLinear& L = p.lin[at.l];
  f32x4 o = {0, 0, 0, 0};
  for (int sp = 0; sp < p.n_split; ++sp)
    o += p.tiles[((((size_t)sp * p.n_rg + rg) * p.n_blk + blk) * (RT * 4) + blockIdx.z) * NT + threadIdx.x];
  const int j = 16 * (RT * (rg - L.rg_begin) + rt) + 4 * g;
  const int t = p.t_begin[tb.sg] + 16 * (tb.tile0 + tile - p.tile0[tb.sg]) + n;
  if (j < L.d_out && t < p.t_end[tb.sg]) {
    uint2 pk;
    pk.x = pack_bf16(o[0], o[1]);
    pk.y = pack_bf16(o[2], o[3]);
    *reinterpret_cast<uint2*>(L.y + (size_t)t * L.d_out + j) = pk;
  }
}

template <int BITS>
hipError_t launch_fused(const PrefillParams& p, int rt, dim3 grid, hipStream_t s) {
  const int most = longest(p.blocks);
  const bool brief = p.n_split == 1 && p.steps_per_split <= kShortSteps && most > 12 && most <= 16;
  if (rt == 7) {
    if (brief) k_prefill_fused<BITS, 7, true><<<grid, 64 * kWaves, 0, s>>>(p);
    else k_prefill_fused<BITS, 7, false><<<grid, 64 * kWaves, 0, s>>>(p);
  } else {
    if (brief) k_prefill_fused<BITS, 8, true><<<grid, 64 * kWaves, 0, s>>>(p);
    else k_prefill_fused<BITS, 8, false><<<grid, 64 * kWaves, 0, s>>>(p);
  }
  return hipGetLastError();
}

}  // namespace

// Scratch for the long segments of a call of up to max_tokens tokens: their activations in fragment order (input
// channels, then up to d_in gathered salient ones; room for every segment padded to whole blocks of 256 tokens, at most
// max_tokens / 192 segments) and, for a split contraction, the accumulator tiles: a split happens only while
// splits x row groups x token blocks stays within 256 workgroups, each leaving 128 rows x 512 tokens x 4 bytes.
size_t prefill_scratch_bytes(int d_in, int max_tokens) {
  const size_t tok_pad = (size_t)max_tokens + (size_t)256 * (max_tokens / 192 + 1);
  const size_t xt = tok_pad * (size_t)(ceil_to(d_in, kColPad) + ceil_to(ceil_to(d_in, kSalPad), 128)) * 2;
  const size_t tiles = (size_t)kMaxWorkgroups * 128 * 512 * 4;
  return (xt + 255) / 256 * 256 + tiles;
}

// y rows of the n_seg long segments seg_experts[i] (expert numbers; rows seg[e] .. seg[e + 1]) of the n_linears layers
// of a call (they read the same x and routing), each layer with its own experts' deltas, up to kMaxSegs segments per
// launch.  All layers share a launch (their row groups one after the other) while the scratch holds every layer's gathered
// salient activations behind the input channels; else each has its own, the gathered activations in the same place one
// after the other (the launches are stream-ordered).
// scratch: prefill_scratch_bytes(d_in, >= all their tokens).
// ev_start / ev_stop (measurement hook, may be null): recorded immediately before the first fused kernel (only while
// *first_kernel is set, which this clears) and immediately after every fused kernel and its reduction.
hipError_t launch_prefill_segments(const mes_linear* lin, int n_linears, const int* seg_experts, int n_seg,
                                   const int32_t* seg, const void* x, void* scratch, hipEvent_t ev_start,
                                   hipEvent_t ev_stop, bool* first_kernel, hipStream_t s) {
  char* ws = reinterpret_cast<char*>(scratch);
  const mes_delta& d = lin[0].experts[seg_experts[0]];   // d_in, bits, grid and k are the same for all experts and layers
  const int n_chunks = ceil_to(d.d_in, kColPad) / 128, n_ssteps = (ceil_to(d.k, kSalPad) / 32 + 3) / 4, steps = n_chunks + n_ssteps;
  const bool together = n_linears * n_ssteps <= ceil_to(ceil_to(d.d_in, kSalPad), 128) / 128;
  const int per_launch = together ? n_linears : 1;
  for (int first = 0; first < n_seg; first += kMaxSegs) {
    const int ns = n_seg - first < kMaxSegs ? n_seg - first : kMaxSegs;
    PrefillParams p;
    TileParams tp;
    int seg_tiles[kMaxSegs], n_tq = 0;
    for (int i = 0; i < kMaxSegs; ++i) {
      const int e = seg_experts[first + (i < ns ? i : 0)];
      p.t_begin[i] = tp.t_begin[i] = seg[e];
      p.t_end[i] = tp.t_end[i] = seg[e + 1];
      p.tile0[i] = tp.tile0[i] = n_tq;
      if (i < ns) n_tq += seg_tiles[i] = (seg[e + 1] - seg[e] + 15) / 16;
    }
    p.xt = reinterpret_cast<const u32x4*>(ws);
    p.n_chunks = n_chunks;
    p.n_sb = ceil_to(d.k, kSalPad) / 32;
    p.n_ssteps = n_ssteps;
    p.n_tq = n_tq;
    p.z = d.grid == MES_GRID_SYM ? (float)(1 << (d.bits - 1)) - 0.5f : (float)(1 << (d.bits - 1));
    const size_t xt_bytes = (size_t)4 * (n_chunks + per_launch * n_ssteps) * n_tq * 1024;
    p.tiles = reinterpret_cast<f32x4*>(ws + (xt_bytes + 255) / 256 * 256);
    tp.x = reinterpret_cast<const uint16_t*>(x);
    tp.n_seg = ns;
    tp.k = d.k;
    tp.d_in = d.d_in;
    tp.n_chunks = n_chunks;
    tp.n_ssteps = n_ssteps;
    tp.n_tq = n_tq;
    tp.xt = reinterpret_cast<u32x4*>(ws);
    for (int l0 = 0; l0 < n_linears; l0 += per_launch) {
      int d_outs[MES_MAX_FUSED];
      for (int l = 0; l < MES_MAX_FUSED; ++l) {
        const mes_linear& src = lin[l0 + (l < per_launch ? l : 0)];   // unused entries repeat the first (never selected)
        PrefillLinear& L = p.lin[l];
        L.base = reinterpret_cast<const u32x4*>(src.w_base_tiled);
        L.y = reinterpret_cast<uint16_t*>(src.y);
        for (int i = 0; i < kMaxSegs; ++i) {
          const mes_delta& de = src.experts[seg_experts[first + (i < ns ? i : 0)]];
          L.codes[i] = reinterpret_cast<const uint32_t*>(de.codes);
          L.step[i] = de.step;
          L.sal[i] = reinterpret_cast<const u32x4*>(de.salient);
          tp.sidx[l][i] = de.salient_idx;
        }
        L.d_out = d_outs[l] = src.experts[seg_experts[first]].d_out;
        L.n_jt = ceil_to(L.d_out, kRowPad) / 16;
      }
      hipError_t e = hipSuccess;
      // the input channels, the same for every layer of the call, go with the first launch
      tp.u_begin = l0 == 0 ? 0 : n_chunks;
      tp.n_units = n_chunks + 4 * per_launch * n_ssteps - tp.u_begin;
      if (tp.n_units > 0) {
        const long waves = (long)tp.n_units * n_tq;
        k_prefill_tile_x<<<(unsigned)((waves + 3) / 4), 256, 0, s>>>(tp);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      PrefillPlan pl;
      prefill_plan(pl, seg_tiles, ns, d_outs, per_launch, steps);
      p.n_split = pl.n_split;
      p.steps_per_split = pl.steps_per_split;
      p.blocks = pl.blocks;
      p.n_blk = count(pl.blocks);
      p.n_rg = 0;
      for (int l = 0; l < MES_MAX_FUSED; ++l) {
        p.lin[l].rg_begin = p.n_rg;
        if (l < per_launch) p.n_rg += (p.lin[l].n_jt + pl.rt - 1) / pl.rt;
        p.lin[l].rg_end = p.n_rg;
      }
      for (int left = p.n_blk; left > 0;) {
        const int blocks = left < kMaxGridY ? left : kMaxGridY;
        const dim3 grid(p.n_rg, blocks, pl.n_split);
        if (ev_start && *first_kernel && (e = hipEventRecord(ev_start, s)) != hipSuccess) return e;
        *first_kernel = false;
        switch (d.bits) {
          case 1: e = launch_fused<1>(p, pl.rt, grid, s); break;
          case 2: e = launch_fused<2>(p, pl.rt, grid, s); break;
          case 3: e = launch_fused<3>(p, pl.rt, grid, s); break;
          default: e = launch_fused<4>(p, pl.rt, grid, s); break;
        }
        if (e != hipSuccess) return e;
        if (pl.n_split > 1) {
          if (pl.rt == 7) k_prefill_reduce<7><<<dim3(p.n_rg, p.n_blk, 28), 64 * kWaves, 0, s>>>(p);
          else k_prefill_reduce<8><<<dim3(p.n_rg, p.n_blk, 32), 64 * kWaves, 0, s>>>(p);
          if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if (ev_stop && (e = hipEventRecord(ev_stop, s)) != hipSuccess) return e;
        left -= blocks;
        if (left > 0) p.blocks = behind(p.blocks, blocks);
      }
    }
  }
  return hipSuccess;
}

}  // namespace mes
