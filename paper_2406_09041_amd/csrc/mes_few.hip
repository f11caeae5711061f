// The serving hot path for a handful of tokens (Eq. 4, as in mes_linear.hip) in ONE launch: no preparation of the
// activations before it, no reduction of split columns after it.
//
// A call of one decoded token moves 38 MB through a 4096 x 4096 layer, 8 us at the rate of a large copy; the
// three launches of the streaming path, each with its own start-up, took 22 us for it; this one takes 13.4.  With one or two
// 16-token tiles the activations are so few that every workgroup can afford to prepare them for itself:
//   - a workgroup owns 16 output channels (of two layers if they are a gated pair) and ALL the columns; its wavefronts
//     deal the 128-column chunks among themselves, each with its own accumulators, and meet in LDS at the end, where
//     the sums are added in wavefront order: the result does not depend on timing;
//   - every wavefront reads its chunk's activations straight from x (bf16 operands as they are), and makes their fp8
//     pieces in registers (about 170 vector instructions per chunk and token tile, hidden behind the weights' way from
//     memory) with a trip through its own corner of LDS to bring the bytes into the operand's column order;
//   - several chunks' weights, code words and activations per wavefront are in flight from the start.
// The products are those of the streaming kernel (the same instructions on the same operands); only the order in
// which the fp32 sums are taken differs.
#include "mes_linear_common.h"

namespace mes {
namespace {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

template <int BITS>
__device__ __forceinline__ CodeRegs<BITS> ld_codes(const char* blk, int lane) {
  CodeRegs<BITS> r;
  typedef __attribute__((address_space(1))) const uint32_t g32;
  typedef __attribute__((address_space(1))) const u32x2 g64;
  if constexpr (BITS == 1) {
    r.lo[0] = *reinterpret_cast<g32*>(gptr(blk) + (uint32_t)lane * 4u);
  } else {
    const u32x2 v = *reinterpret_cast<g64*>(gptr(blk) + (uint32_t)lane * 8u);
    r.lo[0] = v[0]; r.lo[1] = v[1];
    if constexpr (BITS == 3) r.hi[0] = *reinterpret_cast<g32*>(gptr(blk) + 512 + (uint32_t)lane * 4u);
    if constexpr (BITS == 4) {
      const u32x2 h = *reinterpret_cast<g64*>(gptr(blk) + 512 + (uint32_t)lane * 8u);
      r.hi[0] = h[0]; r.hi[1] = h[1];
    }
  }
  return r;
}

// Numbers pass between the lanes of one wavefront through LDS without a barrier.  The hardware keeps a wavefront's LDS
// accesses in order; this has the compiler keep them in order too (no instruction, no wait).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

constexpr int kFewWaves = 8;    // per workgroup
constexpr int kFewPairs = 64;   // salient pairs a launch takes (half of them for each layer of a gated pair)

// What a wavefront keeps in flight for one chunk.
template <int BITS, int NA, int TT>
struct FewChunk {
  u32x4 w[4];               // base weights of the row tile
  CodeRegs<BITS> c[NA];     // code words, per slot
  u32x4 x[TT][4];           // activations: block kb of tile tt, lane 16 g + n: x[16 tt + n][32 kb + 8 g + 0..7]
};

// Grid: the row tiles of all the layers (of one layer of a gated pair).  NA slots at most, TT token tiles, NW
// wavefronts, AHEAD chunks in flight per wavefront.
template <int BITS, int NA, int TT, int NW, int AHEAD>
__global__ __launch_bounds__(64 * NW) void k_few_tokens(const LinearParams p, int team_log) {
  __shared__ __attribute__((aligned(16))) char fp8_lds[NW][TT * 4096];   // per wavefront: [tile][piece][half][lane][16]
  __shared__ __attribute__((aligned(16))) u32x4 sal_lds[kFewPairs][64];  // gathered activations of the salient pairs
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the team's layer and row tile (a gated pair: two teams, one per layer, on the same row tile) and this wavefront's
  // place in the team
  const int team_waves = 1 << team_log, team = wave >> team_log, kw = wave & (team_waves - 1);
  const int teams = p.pair ? NW >> (team_log + 1) : NW >> team_log;   // row tiles of a layer per workgroup, of one layer unless a pair
  int l = 0, jt = blockIdx.x;
  if (p.pair) {
    l = team & 1;
    jt = jt * teams + (team >> 1);
  } else {
    while (l + 1 < p.n_linears) {
      const int wgs = (((p.lin[l].d_out + 15) >> 4) + teams - 1) / teams;
      if (jt < wgs) break;
      jt -= wgs;
      ++l;
    }
    jt = jt * teams + team;
  }
  const int n_tiles = (p.lin[l].d_out + 15) >> 4;
  const bool live = jt < n_tiles;                           // teams past the last row tile keep the barriers company
  jt = live ? jt : n_tiles - 1;
  const PerLinear& L = p.lin[l];
  // Steps, wanted at the end, when a load would be waited for: lane 4 a + q brings slot a's for rows 4 q .. 4 q + 3
  // (unused slots alias slot 0); the lookup of the pointer goes first, so that it is not queued behind the weights.
  // (4096 x 4096, 2 bits, 8 tokens of as many experts: 21.7 -> 21.2 us against steps loaded when they are needed; the
  // 16-slot bodies have no registers for it: at 3 bits 3 of them spilled, 12 experts 35.3 -> 37.8 us.)
  constexpr bool kStepsEarly = NA < kMaxSlots;
  const float* const step_at = L.step[kStepsEarly ? lane >> 2 : 0];

  // Salient channels: every pair (visit, 32 ranks) has 1 KiB of activations, gathered once for the workgroup into LDS
  // (for each layer of a gated pair: they have salient sets of their own), and 1 KiB of weights per row tile.  The
  // wavefronts of a layer deal the gathers among themselves; the indices of the first few
  // are requested behind the first chunk's weights, their activations once all the first weights are asked for (the gathers
  // wait for their indices; 5600 -> 1000, 4 bits, 128 channels, 17.9 -> 16.8 us against indices first and the gathers before the
  // second chunk), and they go to LDS when the stream is over.  The 16-slot bodies at 2 and 3 bits keep indices first and
  // gathers before the second chunk: two chunks of theirs are so many loads that the gathers come too late behind them (4096 ->
  // 6144, 3 bits, 9 experts 44.0 against 46.7 us; 4096 x 4096, 2 bits, 9 experts 25.9 against 26.8, 16 experts 33.9 against 33.1;
  // 30 calls 1.4 % faster on average).
  constexpr bool kGathersFirst = NA == kMaxSlots && BITS >= 2;
  const int n_pairs = p.n_vis * p.n_sb, n_sb = p.n_sb;
  // visit of a pair = pair / n_sb, by a multiplication (the dozen divisions took about 1 % of a call): the reciprocal in 16 bits
  // is too large by less than 2^-16, and pair times that less than 1 / n_sb, as pair and n_sb are at most kFewPairs
  const int inv_sb = n_sb > 0 ? (65535 + n_sb) / n_sb : 0;
  auto visit_of = [&](int pair) { return pair * inv_sb >> 16; };
  const int gw = p.pair ? (team >> 1) * team_waves + kw : wave, gathers = p.pair ? NW / 2 : NW;
  u32x4 (*const sal_at)[64] = p.pair && l ? sal_lds + kFewPairs / 2 : sal_lds;
  constexpr int kGather = 4, kEarly = 2;                   // pairs per wavefront gathered, and weights of pairs requested, up front
  int sal_idx[kGather][8];
  auto request_indices = [&](int pair, int (&idx)[8]) {
    const int v = visit_of(pair);
    const int32_t* si = L.sidx[p.vis_info[v] & 0xff];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int r = 32 * (pair - v * n_sb) + 8 * g + e;
      idx[e] = si[r < p.k ? r : p.k - 1];
    }
  };

  const char* const x_at = keep(reinterpret_cast<const char*>(p.x + (size_t)p.t0 * p.d_in));
  uint32_t x_off[TT];       // lanes past the last token read the group's first: their columns of the products are never stored
  uint32_t slot_tok[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    x_off[tt] = p.t0 + 16 * tt + n < p.T ? (uint32_t)(16 * tt + n) * (uint32_t)p.d_in * 2u : 0u;
    slot_tok[tt] = p.tok_slot[16 * tt + n];
  }
  const char* base_at = keep(L.w_base + (size_t)jt * 4096);
  const uint32_t base_stride = keep((uint32_t)L.n_jt * 4096u);
  const char* code_at[NA];
#pragma unroll
  for (int a = 0; a < NA; ++a) code_at[a] = keep(L.codes[a] + (size_t)jt * code_block_bytes(BITS));
  const uint32_t code_stride = keep((uint32_t)L.n_jt * (uint32_t)code_block_bytes(BITS));
  const int d_in = keep(p.d_in), n_chunks = keep(p.n_chunks);

  using Chunk = FewChunk<BITS, NA, TT>;
  Chunk buf[AHEAD];
  auto x_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(x_at), 0, (p.T - p.t0) * p.d_in * 2, 0x00020000);
  auto request = [&](Chunk& b, int c) {
    const int cw = c < n_chunks ? c : n_chunks - 1;       // weights of a chunk past the last one: repeated
    const char* src = base_at + (size_t)cw * base_stride;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) b.w[kb] = ld128(src + kb * 1024, (uint32_t)lane * 16u);
#pragma unroll
    for (int a = 0; a < NA; ++a) b.c[a] = ld_codes<BITS>(code_at[a] + (size_t)cw * code_stride, lane);   // (unused slots alias slot 0)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        // the buffer descriptor's bounds check makes columns past the end (d_in % 8 == 0) and chunks past the last one zero
        const int col = kChunk * c + 32 * kb + 8 * g;
        b.x[tt][kb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, col < d_in ? (int)(x_off[tt] + 2u * (uint32_t)col) : -16, 0, 0));
      }
  };
  f32x4 acc_base[TT], acc_raw[TT];
  float rs[TT];             // this lane's share of the sum of its token's activations
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) { acc_base[tt] = f32x4{0, 0, 0, 0}; acc_raw[tt] = f32x4{0, 0, 0, 0}; rs[tt] = 0.0f; }

  char* const my_fp8 = fp8_lds[wave];
  auto multiply = [&](const Chunk& b) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      // largest magnitude of the token's chunk: bf16 magnitudes compare like integers, two to a word
      u16x2 m2 = {0, 0};
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(u16x2, b.x[tt][kb][e] & 0x7fff7fffu));
      uint32_t m = m2[0] > m2[1] ? m2[0] : m2[1];
      m = max(m, (uint32_t)__shfl_xor((int)m, 16));         // the token's four lanes
      m = max(m, (uint32_t)__shfl_xor((int)m, 32));
      const int s = chunk_exponent(__uint_as_float(m << 16));
      wave_lds_fence();                                     // the other lanes have read the last chunk's pieces
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        float xv[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          xv[2 * e] = __uint_as_float(b.x[tt][kb][e] << 16);
          xv[2 * e + 1] = __uint_as_float(b.x[tt][kb][e] & 0xffff0000u);
          rs[tt] += xv[2 * e] + xv[2 * e + 1];
        }
        asm volatile("" : "+v"(rs[tt]));                    // added up here and now, not when the sum is needed
        // columns 32 kb + 8 g + e  ->  half = kb / 2, lane group 2 (kb % 2) + g / 2, bytes 8 (g % 2) + e
        int hw[2], lw[2];
        split_fp8(xv, s, hw, lw);
        char* dst = my_fp8 + tt * 4096 + (kb >> 1) * 1024 + (16 * (2 * (kb & 1) + (g >> 1)) + n) * 16 + 8 * (g & 1);
        *reinterpret_cast<u32x2*>(dst) = u32x2{(uint32_t)hw[0], (uint32_t)hw[1]};
        *reinterpret_cast<u32x2*>(dst + 2048) = u32x2{(uint32_t)lw[0], (uint32_t)lw[1]};
        __builtin_amdgcn_sched_barrier(0);                  // one block's temporaries at a time
      }
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) acc_base[tt] = mfma_bf16(b.w[kb], b.x[tt][kb], acc_base[tt]);
      wave_lds_fence();                                     // ... and written this one's
      v8i piece[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const u32x4 h0 = lds128(my_fp8, tt * 4096 + q * 2048 + lane * 16), h1 = lds128(my_fp8, tt * 4096 + q * 2048 + 1024 + lane * 16);
        piece[q] = v8i{(int)h0[0], (int)h0[1], (int)h0[2], (int)h0[3], (int)h1[0], (int)h1[1], (int)h1[2], (int)h1[3]};
      }
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        if (a >= p.tile_first[tt] && a <= p.tile_last[tt]) {
          const int sc = slot_tok[tt] == (uint32_t)a ? 128 + s : 0;   // 2^-127 for the tokens of other experts
          mfma_fp4_fp8_pair(acc_raw[tt], dequant_lo<BITS>(b.c[a]), piece[0], piece[1], sc);
          if constexpr (BITS >= 3) mfma_fp4_fp8_pair(acc_raw[tt], dequant_hi(b.c[a]), piece[0], piece[1], sc, BITS == 4 ? 129 : 127);
        }
      }
    }
  };

  // This wavefront's chunks: kw, kw + team_waves, ...
  const int mine = kw < n_chunks ? (n_chunks - kw + team_waves - 1) / team_waves : 0;
  auto chunk_at = [&](int i) { return kw + team_waves * i; };
  auto request_first_indices = [&] {
    if (n_pairs > 0) {
#pragma unroll
      for (int q = 0; q < kGather; ++q)
        if (gw + gathers * q < n_pairs) request_indices(gw + gathers * q, sal_idx[q]);
    }
  };
  auto request_other_chunks = [&] {
#pragma unroll
    for (int u = 1; u < AHEAD; ++u) request(buf[u], chunk_at(u));
  };
  if constexpr (kGathersFirst) request_first_indices();
  request(buf[0], chunk_at(0));
  if constexpr (!kGathersFirst) {
    request_first_indices();
    request_other_chunks();
  }
  const int st_j = 16 * jt + 4 * (lane & 3);
  typedef __attribute__((address_space(1))) const f32x4 gf4;   // (a generic load would count as an LDS access as well)
  f32x4 st_v = {0, 0, 0, 0};
  if constexpr (kStepsEarly) st_v = *reinterpret_cast<gf4*>(gptr(step_at + (st_j < L.d_out ? st_j : 0)));
  uint32_t sal_h[kGather][8];
  typedef __attribute__((address_space(1))) const uint16_t g16;
  auto request_gather = [&](int pair, const int (&idx)[8], uint32_t (&h)[8]) {
    const int info = p.vis_info[visit_of(pair)], a = info & 0xff, tl = 16 * (info >> 8) + n;
    if (tl < p.lo[a] || tl >= p.hi[a]) return;              // other experts' tokens: zero when they are stored
    const uint32_t row_off = (uint32_t)tl * (uint32_t)d_in * 2u;
#pragma unroll
    for (int e = 0; e < 8; ++e)   // a corrupt list cannot address outside the row
      h[e] = *reinterpret_cast<g16*>(gptr(x_at) + row_off + 2u * min((uint32_t)idx[e], (uint32_t)(d_in - 1)));
  };
  // (the activations of other experts' tokens and of ranks past k count as zero)
  auto store_gather = [&](int pair, const uint32_t (&h)[8]) {
    const int v = visit_of(pair), info = p.vis_info[v], a = info & 0xff, tl = 16 * (info >> 8) + n, r0 = 32 * (pair - v * n_sb) + 8 * g;
    const bool inm = tl >= p.lo[a] && tl < p.hi[a];
    u32x4 x;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      x[q] = (inm && r0 + 2 * q < p.k ? h[2 * q] : 0u) | (inm && r0 + 2 * q + 1 < p.k ? h[2 * q + 1] << 16 : 0u);
    sal_at[pair][lane] = x;
  };
  if (n_pairs > 0) {
#pragma unroll
    for (int q = 0; q < kGather; ++q)
      if (gw + gathers * q < n_pairs) request_gather(gw + gathers * q, sal_idx[q], sal_h[q]);
  }
  if constexpr (kGathersFirst) request_other_chunks();
  // weights of one pair and the row's step of its expert, as loaded; pairs past the last one repeat it
  struct PairLoad { u32x4 d; float step; };
  PairLoad pl[kEarly];
  auto request_pair = [&](int pair, PairLoad& o) {
    pair = pair < n_pairs ? pair : n_pairs - 1;
    const int v = visit_of(pair), a = p.vis_info[v] & 0xff;
    o.d = ld128(L.sal[a] + ((size_t)jt * n_sb + (pair - v * n_sb)) * 1024, (uint32_t)lane * 16u);
    const int row_n = 16 * jt + n;
    o.step = L.step[a][row_n < L.d_out ? row_n : L.d_out - 1];   // (rows past the end are never stored)
  };
  // acc_base += (D + z step) x as two bf16 pieces, exactly as the streaming kernel has it
  auto multiply_pair = [&](int pair, const PairLoad& o) {
    const int tile = p.vis_info[visit_of(pair)] >> 8;
    const u32x4 x = sal_at[pair][lane];
    const f16x8 dh = __builtin_bit_cast(f16x8, o.d);
    const float zs = p.z * o.step;
    u32x4 hi, lo;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float f0 = (float)dh[2 * q] + zs, f1 = (float)dh[2 * q + 1] + zs;
      const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{f0, f1}, bf16x2));   // round to nearest even
      hi[q] = h;
      lo[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{f0 - __uint_as_float(h << 16), f1 - __uint_as_float(h & 0xffff0000u)}, bf16x2));
    }
    f32x4 t = mfma_bf16(hi, x, f32x4{0, 0, 0, 0});
    t = mfma_bf16(lo, x, t);
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc_base[tt][v] += tt == tile ? t[v] : 0.0f;
  };
  if (n_pairs > 0) {
#pragma unroll
    for (int q = 0; q < kEarly; ++q) request_pair(kw + team_waves * q, pl[q]);
  }

  // The stream.  Every load of the loop body is issued whatever the data (weights of chunks past the last one repeat
  // it) and no branch goes around a load: the compiler then knows how many younger loads may stay in flight at each wait.
  int i = 0;
  for (; i + AHEAD < mine; i += AHEAD) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      multiply(buf[u]);
      __builtin_amdgcn_sched_barrier(0);
      request(buf[u], chunk_at(i + u + AHEAD));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) {
    if (i + u < mine) multiply(buf[u]);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (n_pairs > 0) {
#pragma unroll
    for (int q = 0; q < kGather; ++q)
      if (gw + gathers * q < n_pairs) store_gather(gw + gathers * q, sal_h[q]);
    for (int pair = gw + gathers * kGather; pair < n_pairs; pair += gathers) {
      request_indices(pair, sal_idx[0]);
      request_gather(pair, sal_idx[0], sal_h[0]);
      store_gather(pair, sal_h[0]);
    }
    __syncthreads();
  }
  for (int pair = kw; pair < n_pairs; pair += kEarly * team_waves) {
#pragma unroll
    for (int q = 0; q < kEarly; ++q) {
      if (pair + q * team_waves < n_pairs) multiply_pair(pair + q * team_waves, pl[q]);
      request_pair(pair + (kEarly + q) * team_waves, pl[q]);
    }
  }

  // Zero point and step, then the sum over the wavefronts.  The matrix instructions issued from assembly blocks get
  // the wait states a result needs before vector instructions may read it.
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  f32x4 stepv[TT];                                          // (tokens past the last one have no slot and are never stored)
  if constexpr (kStepsEarly) {
    wave_lds_fence();                                       // this wavefront is done with its fp8 pieces
    *reinterpret_cast<f32x4*>(my_fp8 + (lane >> 2) * 64 + (lane & 3) * 16) = st_v;
    wave_lds_fence();
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) stepv[tt] = *reinterpret_cast<const f32x4*>(my_fp8 + (slot_tok[tt] & (kMaxSlots - 1)) * 64 + g * 16);
  } else {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int j = 16 * jt + 4 * g;
      stepv[tt] = f32x4{0, 0, 0, 0};
      if (slot_tok[tt] != 0xffu && j < L.d_out) stepv[tt] = *reinterpret_cast<const f32x4*>(L.step[slot_tok[tt]] + j);
    }
  }
  __syncthreads();                                          // ... and every wavefront, and with its steps
  f32x4* const part = reinterpret_cast<f32x4*>(&fp8_lds[0][0]);   // [wavefront][tile][lane]
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    float r = rs[tt] + __shfl_xor(rs[tt], 16);
    r += __shfl_xor(r, 32);
    f32x4 o;
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = acc_base[tt][v] + stepv[tt][v] * (acc_raw[tt][v] - p.z * r);
    part[(wave * TT + tt) * 64 + lane] = o;
  }
  __syncthreads();
  if (!live || kw > 0 || (p.pair && (team & 1))) return;    // the team's (pair's) first wavefront finishes the row tile
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    f32x4 o = {0, 0, 0, 0};
    for (int w = 0; w < team_waves; ++w) o += part[((wave + w) * TT + tt) * 64 + lane];
    if (p.pair) {
      f32x4 up = {0, 0, 0, 0};
      for (int w = 0; w < team_waves; ++w) up += part[((wave + team_waves + w) * TT + tt) * 64 + lane];
      o = gated(o, up);
    }
    const int t = p.t0 + 16 * tt + n, j = 16 * jt + 4 * g;
    if (t < p.T && j < L.d_out) {
      uint2 pk;
      pk.x = pack_bf16(o[0], o[1]);
      pk.y = pack_bf16(o[2], o[3]);
      *reinterpret_cast<uint2*>(L.y + (size_t)t * L.d_out + j) = pk;
    }
  }
}

template <int BITS>
void launch_slots(const LinearParams& p, int grid, int team_log, int mine, hipStream_t s) {
  constexpr int NT = 64 * kFewWaves;
  if (p.tiles == 2) {
    if (p.n_act <= 1) k_few_tokens<BITS, 1, 2, kFewWaves, 2><<<grid, NT, 0, s>>>(p, team_log);
    else if (p.n_act <= 4) k_few_tokens<BITS, 4, 2, kFewWaves, 2><<<grid, NT, 0, s>>>(p, team_log);
    else if constexpr (BITS < 3) k_few_tokens<BITS, 8, 2, kFewWaves, 2><<<grid, NT, 0, s>>>(p, team_log);
  } else if (p.n_act <= 1) {
    if (mine == 1) k_few_tokens<BITS, 1, 1, kFewWaves, 1><<<grid, NT, 0, s>>>(p, team_log);
    else if (mine < 4) k_few_tokens<BITS, 1, 1, kFewWaves, 2><<<grid, NT, 0, s>>>(p, team_log);
    else k_few_tokens<BITS, 1, 1, kFewWaves, 4><<<grid, NT, 0, s>>>(p, team_log);
  } else if (p.n_act <= 4) {
    if (mine == 1) k_few_tokens<BITS, 4, 1, kFewWaves, 1><<<grid, NT, 0, s>>>(p, team_log);
    else if (mine < 4) k_few_tokens<BITS, 4, 1, kFewWaves, 2><<<grid, NT, 0, s>>>(p, team_log);
    else k_few_tokens<BITS, 4, 1, kFewWaves, BITS >= 3 ? 3 : 4><<<grid, NT, 0, s>>>(p, team_log);
  } else if (p.n_act <= 8) {
    k_few_tokens<BITS, 8, 1, kFewWaves, 2><<<grid, NT, 0, s>>>(p, team_log);
  } else if constexpr (BITS < 4) {
    k_few_tokens<BITS, 16, 1, kFewWaves, 2><<<grid, NT, 0, s>>>(p, team_log);
  }
}

}  // namespace

// Wavefronts per row tile (as a power of two) and workgroups of a launch.  One workgroup runs per compute unit;
// the teams are as large as fills the 256 of them once, a second round of workgroups pays the start-up again (about 3.5
// chunks' worth).
struct FewPlan { int team_log, grid, mine; };   // mine: chunks per wavefront

static FewPlan few_plan(const LinearParams& p) {
  FewPlan f{0, 0, 0};
  double best = 1e30;
  for (int t = p.pair ? 2 : 3; t >= 0; --t) {
    const int teams = (kFewWaves >> t) / (p.pair ? 2 : 1), mine = ((p.n_chunks - 1) >> t) + 1;
    int wgs = 0;
    for (int l = 0; l < (p.pair ? 1 : p.n_linears); ++l) wgs += ((p.lin[l].d_out + 15) / 16 + teams - 1) / teams;
    const double cost = (double)((wgs + 255) / 256) * (mine + 3.5);
    if (cost < best) { best = cost; f.team_log = t; f.grid = wgs; f.mine = mine; }
  }
  return f;
}

// Token groups the kernel can take: one or two token tiles whose experts' code words fit the registers (one tile: 16
// experts, at 4 bits 8; two tiles: 8 experts, at 3 and 4 bits 4), salient pairs that fit their place in LDS, 32-bit offsets
// into x.
bool few_tokens_fits(const LinearParams& p) {
  if (p.tiles > 2 || p.n_vis * p.n_sb > (p.pair ? kFewPairs / 2 : kFewPairs) || p.d_in > (1 << 24)) return false;
  return p.tiles == 2 ? p.n_act <= (p.bits < 3 ? 8 : 4) : p.n_act <= 8 || p.bits < 4;
}

// Expected time of a group here, us: per round of workgroups a start-up, per chunk the multiplications and the
// preparation of the activations (which every row tile's wavefronts do again, per tile of tokens), and the
// wavefronts' shares of the salient pairs; plus a share of the weights' way from memory.  The terms are those of the
// kernel, the numbers least squares over 1800 calls (d_in and d_out from 256 to 14336, one layer, two or three, gated
// pairs, 1 to 32 tokens, 1 to 16 experts, 1 to 4 bits, up to 128 salient channels); 11 % off on 1135 others, 4 % of it too
// high: the kernel has become faster since.
double few_tokens_us(const LinearParams& p) {
  const FewPlan f = few_plan(p);
  const int rounds = (f.grid + 255) / 256, more = p.tiles - 1;
  const double pairs = (double)(p.n_vis * p.n_sb) / (1 << f.team_log);
  return 0.4 + rounds * (6.1 + 1.3 * more + f.mine * (0.9 + 0.13 * p.n_act + 1.1 * more) + pairs) + 0.28 * weights_us(p);
}

hipError_t launch_few_tokens(const LinearParams& p, hipStream_t s) {
  const FewPlan f = few_plan(p);
  switch (p.bits) {
    case 1: launch_slots<1>(p, f.grid, f.team_log, f.mine, s); break;
    case 2: launch_slots<2>(p, f.grid, f.team_log, f.mine, s); break;
    case 3: launch_slots<3>(p, f.grid, f.team_log, f.mine, s); break;
    default: launch_slots<4>(p, f.grid, f.team_log, f.mine, s); break;
  }
  return hipGetLastError();
}

}  // namespace mes
