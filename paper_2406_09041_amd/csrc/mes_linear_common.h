// What the streaming kernels (mes_linear.hip) and the one-launch kernel for few tokens (mes_few.hip) share: the kernel
// arguments of a token group, the code-word formats as matrix operands, small conversions.
#pragma once

#include "mes_internal.h"

namespace mes {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
typedef int v8i __attribute__((ext_vector_type(8)));
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;

constexpr int kChunk = 128;                     // columns per chunk (one fp4 x fp8 MFMA deep)
constexpr int kStageVec = 2048;                 // 16-byte slots of activations per chunk
constexpr int kStageBytes = kStageVec * 16 + 1024;  // + a block of per-token numbers (block scales, sums)
constexpr int kStageFp8 = 16384;                // byte offset of the fp8 pieces inside a stage
constexpr int kStageScale = 32768;              // byte offset of the scales inside a stage
constexpr int kStageSum = 32768 + 256;          // byte offset of the tokens' sums over the chunk's columns
constexpr int kStageBlocks = 33;                // 1 KiB blocks the main kernel copies to LDS per chunk
constexpr int kStageLds = 32 * 1024;            // LDS bytes of a stage's operand images; its 33rd block sits apart (see k_delta_linear)
constexpr int kMaxSlots = 16;                   // experts with tokens in one token group (the host cuts groups accordingly)
constexpr int kMaxVisits = kMaxSlots + 3;       // (expert, 16-token tile) pairs in one group

constexpr int kMaxSplits = 32;                  // workgroups that may share one row group's columns

constexpr int kMaxLinears = MES_MAX_FUSED;    // linear layers one launch serves (they read the same activations)

// Per linear layer: where its weights, outputs and its share of the workspace are.  Per-expert arrays are indexed by slot.
struct PerLinear {
  const char* w_base;
  uint16_t* y;
  u32x4* xs;        // workspace: salient activations per visit, bf16 as gathered  [visit][k_pad/32][64 lanes]
  const char* codes[kMaxSlots];
  const float* step[kMaxSlots];
  const char* sal[kMaxSlots];
  const int32_t* sidx[kMaxSlots];
  int d_out, n_jt;
  int rg_begin, rg_end;   // its row groups among the launch's
};

// Kernel arguments.
struct LinearParams {
  const uint16_t* x;
  char* xt;         // workspace: one stage per chunk (see prepare_item), shared by the linears
  f32x4* partial;   // workspace: [row group][nsplit][4 tiles][threads of a workgroup] partial result tiles (split columns only)
  PerLinear lin[kMaxLinears];
  int16_t lo[kMaxSlots], hi[kMaxSlots];   // tokens [lo, hi) of the group belong to the slot's expert
  uint8_t tok_slot[kTokGroup];            // slot of every token of the group, 0xFF past the last token
  int vis_info[kMaxVisits + 1];           // visits (slot, tile) in tile-major order: slot | tile << 8
  int tile_first[4], tile_last[4];        // slots that own tokens of 16-token tile tt: tile_first[tt] .. tile_last[tt]
  int d_in, n_linears, n_chunks, n_sb, k, T, t0, n_act, n_vis, nsplit, bits;
  int16_t c_split[kMaxSplits + 1];        // workgroup sp of a row group covers the chunks c_split[sp] .. c_split[sp + 1]
  int tiles;                              // 16-token tiles of the group that hold tokens
  int n_stage_items, n_items;             // preparation items: tiles * n_chunks stage items, then n_linears * n_vis gathers
  float z;
  // Gated pair (see launch_delta_linear): lin[0] is the gate, lin[1] the up projection of an MLP block.  The first
  // half of a workgroup's wavefronts owns row tiles of the gate, the second half the same row tiles of the up
  // projection, and the workgroup writes SiLU(gate) * up to lin[0].y instead of the two results.
  int pair;
};

// The linear a row group belongs to.
__device__ __forceinline__ int linear_of(const LinearParams& p, int rg) {
  int l = 0;
#pragma unroll
  for (int i = 0; i + 1 < kMaxLinears; ++i) l += (i + 1 < p.n_linears && rg >= p.lin[i].rg_end) ? 1 : 0;
  return l;
}


__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// acc += A x (Bhi + Blo) [+ Ah x (Bhi + Blo)], fp4 (A, four registers) x fp8 E4M3 (B, eight registers each),
// B scaled per lane by 2^(scale_b - 127).  Written as instructions with the accumulator tied to itself: these
// updates sit in loops and wave-uniform branches, and only a tied operand keeps the compiler from copying
// whole accumulator sets from block to block.  The compiler does not know what the block contains, so the
// block itself provides the two wait states the hardware needs between a vector-ALU write of an operand
// register and a matrix instruction reading it.  (Same opcode, same register as source C and destination:
// back-to-back issue needs no further wait states.)
// scale_a is A's block scale byte: 127 for 2^0; the high plane of 4-bit codes takes 129 (its codes count four times).
__device__ __forceinline__ void mfma_fp4_fp8_pair(f32x4& acc, u32x4 a, v8i bhi, v8i blo, int scale_b, int scale_a = 127) {
  asm volatile("s_nop 1\n\t"
               "v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %4, %5 op_sel_hi:[0,0,0] cbsz:4\n\t"
               "v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %3, %0, %4, %5 op_sel_hi:[0,0,0] cbsz:4"
               : "+v"(acc) : "v"(a), "v"(bhi), "v"(blo), "v"(scale_a), "v"(scale_b));
}

// Code words of one slot for one (chunk, row tile): LW low words per lane and HW words of high bits (b = 3: one
// word, the third bit; b = 4: two words, the high two bits laid out like the low two).
template <int BITS> struct Codec;
template <> struct Codec<2> { static constexpr int LW = 2, HW = 0; };
template <> struct Codec<1> { static constexpr int LW = 1, HW = 0; };
template <> struct Codec<3> { static constexpr int LW = 2, HW = 1; };
template <> struct Codec<4> { static constexpr int LW = 2, HW = 2; };

template <int BITS>
struct CodeRegs {
  uint32_t lo[Codec<BITS>::LW];
  uint32_t hi[Codec<BITS>::HW > 0 ? Codec<BITS>::HW : 1];
};

// Bytes of one (chunk, row tile) block of a slot's codes.
__host__ __device__ constexpr int code_block_bytes(int bits) { return 256 * bits; }

template <int BITS>
// `blk` is the same in all lanes and the lane offset an unsigned 32-bit number: the load then takes its
// address as (scalar base) + (vector offset) and needs no 64-bit vector arithmetic.
__device__ __forceinline__ void load_codes(const char* blk, int lane, CodeRegs<BITS>& r) {
  if constexpr (BITS == 1) {
    r.lo[0] = *reinterpret_cast<const uint32_t*>(blk + (uint32_t)lane * 4u);
  } else {
    const u32x2 v = *reinterpret_cast<const u32x2*>(blk + (uint32_t)lane * 8u);
    r.lo[0] = v[0]; r.lo[1] = v[1];
    if constexpr (BITS == 3) r.hi[0] = *reinterpret_cast<const uint32_t*>(blk + 512 + (uint32_t)lane * 4u);
    if constexpr (BITS == 4) {
      const u32x2 h = *reinterpret_cast<const u32x2*>(blk + 512 + (uint32_t)lane * 8u);
      r.hi[0] = h[0]; r.hi[1] = h[1];
    }
  }
}

// Low code bits as an fp4 A operand (values u / 2, or (u mod 4) / 2 for b = 3).
template <int BITS>
__device__ __forceinline__ u32x4 dequant_lo(const CodeRegs<BITS>& r) {
  u32x4 a;
  if constexpr (BITS == 1) {
    const uint32_t w = r.lo[0];
    a[0] = w & 0x11111111u; a[1] = (w >> 1) & 0x11111111u; a[2] = (w >> 2) & 0x11111111u; a[3] = (w >> 3) & 0x11111111u;
  } else {
    const uint32_t w0 = r.lo[0], w1 = r.lo[1];
    a[0] = w0 & 0x33333333u; a[1] = (w0 >> 2) & 0x33333333u; a[2] = w1 & 0x33333333u; a[3] = (w1 >> 2) & 0x33333333u;
  }
  return a;
}

// High code bit (b = 3) as an fp4 A operand: nibble 0h00 = 2 h = (4 h) / 2.
__device__ __forceinline__ u32x4 dequant_hi(const CodeRegs<3>& r) {
  const uint32_t w = r.hi[0];
  u32x4 a;
  a[0] = (w << 2) & 0x44444444u; a[1] = (w << 1) & 0x44444444u; a[2] = w & 0x44444444u; a[3] = (w >> 1) & 0x44444444u;
  return a;
}

// High two code bits (b = 4) as an fp4 A operand: values h / 2; the matrix instruction scales them by four.
__device__ __forceinline__ u32x4 dequant_hi(const CodeRegs<4>& r) {
  const uint32_t w0 = r.hi[0], w1 = r.hi[1];
  return u32x4{w0 & 0x33333333u, (w0 >> 2) & 0x33333333u, w1 & 0x33333333u, (w1 >> 2) & 0x33333333u};
}

// Two fp32 values -> bf16 bits, round to nearest even (one instruction; the rounding written out in integers, with its
// branch for NaN, was 20 per value).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// SiLU(gate) * up, element by element, in fp32: SiLU(v) = v / (1 + e^-v).
__device__ __forceinline__ f32x4 gated(f32x4 gate, f32x4 up) {
  f32x4 h;
#pragma unroll
  for (int v = 0; v < 4; ++v) h[v] = gate[v] / (1.0f + expf(-gate[v])) * up[v];
  return h;
}

// Activations as fp8: a token's values of one chunk are scaled by 2^-s, s = exponent(amax) - 7, which puts the largest
// into [128, 256); clamped so that 128 + s is a valid scale byte.  Non-finite activations give non-finite outputs
// either way.
__device__ __forceinline__ int chunk_exponent(float amax) {
  int s = (int)((__float_as_uint(amax) >> 23) & 0xffu) - 127 - 7;
  if (amax == 0.0f) s = 0;
  return s < -126 ? -126 : (s > 120 ? 120 : s);
}

// hi = x 2^-s rounded to the E4M3 grid (to nearest: the hardware conversion), lo = what is left, on the same grid;
// eight values, four per word.
__device__ __forceinline__ void split_fp8(const float (&xv)[8], int s, int (&hw)[2], int (&lw)[2]) {
  const float inv = __uint_as_float((uint32_t)(127 - s) << 23);   // 2^-s
  hw[0] = hw[1] = lw[0] = lw[1] = 0;
  // (the half of the word a conversion writes or reads is part of the instruction: spelled out, not looped)
#define MES_SPLIT_PAIR(E, W, UPPER)                                                                   \
  {                                                                                                   \
    const float s0 = xv[E] * inv, s1 = xv[E + 1] * inv;                                               \
    hw[W] = __builtin_amdgcn_cvt_pk_fp8_f32(s0, s1, hw[W], UPPER);                                    \
    const auto back = __builtin_amdgcn_cvt_pk_f32_fp8(hw[W], UPPER);                                  \
    lw[W] = __builtin_amdgcn_cvt_pk_fp8_f32(s0 - back[0], s1 - back[1], lw[W], UPPER);                \
  }
  MES_SPLIT_PAIR(0, 0, false)
  MES_SPLIT_PAIR(2, 0, true)
  MES_SPLIT_PAIR(4, 1, false)
  MES_SPLIT_PAIR(6, 1, true)
#undef MES_SPLIT_PAIR
}

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Loads are written as (wave-uniform pointer) + (32-bit unsigned lane offset): the pointer then lives in
// scalar registers and one vector register per lane serves every stream.
// The pointers are declared to be device (global) memory: one that has been through keep() has lost the
// compiler's knowledge of that, and a generic load would also count as an LDS access.
typedef __attribute__((address_space(1))) const char global_char;
__device__ __forceinline__ global_char* gptr(const void* q) { return reinterpret_cast<global_char*>(reinterpret_cast<uintptr_t>(q)); }
__device__ __forceinline__ u32x4 ld128(const void* uniform_ptr, uint32_t lane_off) {
  return *reinterpret_cast<__attribute__((address_space(1))) const u32x4*>(gptr(uniform_ptr) + lane_off);
}


__device__ __forceinline__ u32x4 lds128(const char* stage, int off) { return *reinterpret_cast<const u32x4*>(stage + off); }

// A value read from the kernel's argument block is kept in a register from here on.  Left alone the compiler treats
// such a value as free to fetch again (it is constant memory) wherever scalar registers run short, i.e. all over
// the streaming loop; every such fetch is a scalar memory load, and while one is in flight every wait for an LDS
// read of the wavefront has to be a wait for everything, which takes the pipelining out of the operand reads.
template <class V>
__device__ __forceinline__ V keep(V v) {
  asm volatile("" : "+s"(v));
  return v;
}

// 16 bytes from a device address held in a lane's registers (a global load, not a generic one: a generic load
// would also count as an LDS access and make every wait for an operand read wait for memory as well).
typedef __attribute__((address_space(1))) const u32x4 global_u32x4;
__device__ __forceinline__ u32x4 ld128_at(uint64_t addr) { return *reinterpret_cast<global_u32x4*>(addr); }

// The group's weights at 5 TB/s, us.
inline double weights_us(const LinearParams& p) {
  double row_tiles = 0;
  for (int l = 0; l < p.n_linears; ++l) row_tiles += (p.lin[l].d_out + 15) / 16;
  return row_tiles * p.n_chunks * (4096.0 + (double)p.n_act * code_block_bytes(p.bits)) / 5e6;
}

// The one-launch path for a token group of one or two tiles (mes_few.hip): whether the kernel can take the group, the
// time it is expected to need, the launch.
bool few_tokens_fits(const LinearParams& p);
double few_tokens_us(const LinearParams& p);
hipError_t launch_few_tokens(const LinearParams& p, hipStream_t s);

}  // namespace mes
