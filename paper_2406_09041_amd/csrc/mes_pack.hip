// Offline kernels: re-tiling of the base weight, compression of one expert's delta
// (Eq. 1 per output channel, fp16 salient columns -- Section 4.1), its inverse for tests,
// and the salient-channel selection of Eq. 2.  None of these is on the serving path; all of them are bound by the
// bytes of the delta matrix, with results that are exact (codes) or summed in fp64 (scores).
#include "mes_internal.h"

#include <hip/hip_fp16.h>

namespace mes {
namespace {

__device__ __forceinline__ bool is_salient(const int32_t* sidx, int k, int col, int* pos) {
  int lo = 0, hi = k;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    int v = sidx[mid];
    if (v < col) lo = mid + 1; else hi = mid;
  }
  if (lo < k && sidx[lo] == col) { if (pos) *pos = lo; return true; }
  return false;
}

__device__ __forceinline__ double zero_point(int bits, int grid) {
  return grid == MES_GRID_SYM ? (double)(1 << (bits - 1)) - 0.5 : (double)(1 << (bits - 1));
}

// Eq. 1 with an unsigned code: SYM takes the cell index floor(t), EQ1 rounds half to even.
__device__ __forceinline__ uint32_t quant_code(float w, float step, int bits, int grid) {
  const int half = 1 << (bits - 1);
  if (!(step > 0.0f)) return (uint32_t)half;
  double t = (double)w / (double)step;
  double u;
  if (grid == MES_GRID_SYM) {
    u = floor(t) + (double)half;
    u = fmin(fmax(u, 0.0), (double)(2 * half - 1));
  } else {
    u = fmin(fmax(rint(t), (double)-half), (double)(half - 1)) + (double)half;
  }
  return (uint32_t)(int)u;
}

// ---- base weight tiling --------------------------------------------------------------------------

__global__ void k_pack_base(const uint16_t* __restrict__ w, int d_in, int d_out, int n_kb, size_t n_slots,
                            uint4* __restrict__ out) {
  size_t slot = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= n_slots) return;
  // slot = ((c * n_jt + jt) * 4 + kb) * 64 + lane: chunk-major
  int lane = (int)(slot & 63);
  size_t blk = slot >> 6;
  int kb = (int)(blk & 3);
  blk >>= 2;
  const int n_jt = (d_out + 63) / 64 * 4;
  int jt = (int)(blk % n_jt);
  int c = (int)(blk / n_jt);
  int row = 16 * jt + (lane & 15);
  int col = 128 * c + 32 * kb + 8 * (lane >> 4);
  uint4 v = make_uint4(0, 0, 0, 0);
  if (row < d_out && col < d_in) v = *reinterpret_cast<const uint4*>(w + (size_t)row * d_in + col);
  out[slot] = v;
}

__global__ void k_unpack_base(const uint4* __restrict__ t, int d_in, int d_out, int n_kb, size_t n_slots,
                              uint16_t* __restrict__ w) {
  size_t slot = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= n_slots) return;
  int lane = (int)(slot & 63);
  size_t blk = slot >> 6;
  int kb = (int)(blk & 3);
  blk >>= 2;
  const int n_jt = (d_out + 63) / 64 * 4;
  int jt = (int)(blk % n_jt);
  int c = (int)(blk / n_jt);
  int row = 16 * jt + (lane & 15);
  int col = 128 * c + 32 * kb + 8 * (lane >> 4);
  if (row < d_out && col < d_in) *reinterpret_cast<uint4*>(w + (size_t)row * d_in + col) = t[slot];
}

// ---- delta compression -----------------------------------------------------------------------------

// ---- a code without the fp64 division --------------------------------------------------------------
// quant_code() decides floor(w / s) (or the nearest integer, ties to even) on the fp64 quotient, which is the exact
// decision: w and s have 24 significant bits, so a quotient of magnitude >= 1 that is no integer (or half integer) is
// further than 2^-49 from one, which fp64 resolves.  The same decision in fp32: m is estimated from the rounded
// quotient (reciprocal and product err by less than 2^-22 relative) pushed upwards by 2^-21, so that it is the right
// integer or one more, and corrected with one fused multiply-add whose sign is that of the exact w - m s (nothing
// underflows while s is far from the ends of fp32's range).  Returns the clamped m, -2^(b-1) <= m < 2^(b-1), as a
// float; infinities clamp and NaN gives the lowest code, as quant_code() has it.
__device__ __forceinline__ bool fast_step(float s) { return s >= 0x1p-100f && s <= 0x1p100f; }

template <int BITS, bool EQ1>
__device__ __forceinline__ float clamped_cell(float w, float s, float inv_s) {
  constexpr float kHalf = (float)(1 << (BITS - 1));
  const float v = w * inv_s;
  float m = __builtin_fmaf(__builtin_fabsf(v), 0x1p-21f, v);
  if constexpr (EQ1) {
    m = __builtin_floorf(m + 0.5f);
    const float r = __builtin_fmaf(0.5f - m, s, w);          // w - (m - 1/2) s
    const float hm = 0.5f * m;
    const bool odd = __builtin_floorf(hm) != hm;
    m -= (r < 0.0f || (r == 0.0f && odd)) ? 1.0f : 0.0f;
  } else {
    m = __builtin_floorf(m);
    const float r = __builtin_fmaf(-m, s, w);                // w - m s
    m -= r < 0.0f ? 1.0f : 0.0f;
  }
  return __builtin_fminf(__builtin_fmaxf(m, -kHalf), kHalf - 1.0f);
}

// Four consecutive floats.  The caller's matrix need not be 16-byte aligned (its rows are multiples of 32 bytes).
__device__ __forceinline__ float4 load4(const float* p, bool aligned) {
  if (aligned) return *reinterpret_cast<const float4*>(p);
  return make_float4(p[0], p[1], p[2], p[3]);
}

__device__ __forceinline__ float max4(float m, float4 v) {
  return fmaxf(fmaxf(fmaxf(m, fabsf(v.x)), fmaxf(fabsf(v.y), fabsf(v.z))), fabsf(v.w));
}

__device__ __forceinline__ float wave_max(float m) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) m = fmaxf(m, __shfl_xor(m, off));
  return m;
}

__device__ __forceinline__ float maxabs_step(float m, int bits, bool eq1) {
  const double div = eq1 ? (double)(1 << (bits - 1)) - 1.0 : (double)(1 << (bits - 1)) - 0.5;
  return (float)((double)m / div);
}

// Salient selection: Eq. 1's initialisation max|X| / D over the whole row, one block per output channel.
__global__ __launch_bounds__(256) void k_row_maxabs(const float* __restrict__ delta, int d_in, int bits, int grid,
                                                    bool aligned, float* __restrict__ step_out) {
  const float* r = delta + (size_t)blockIdx.x * d_in;
  float m = 0.0f;
  for (int c = 4 * threadIdx.x; c < d_in; c += 1024) m = max4(m, load4(r + c, aligned));
  __shared__ float red[4];
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) step_out[blockIdx.x] = maxabs_step(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])), bits, grid == MES_GRID_EQ1);
}

// b = 1: step = 2 mean|w| over the non-salient columns.  The fp64 sum runs over a row's columns in ascending order
// (the stored step is the rounding of exactly that sum), so the columns of a row cannot be shared out; the rows can:
// wavefront 0 of a block sums 64 rows, one per lane, out of LDS, while all four wavefronts bring in the next 64
// columns.  A salient column counts as + 0, which leaves the sum as it is.
__global__ __launch_bounds__(256) void k_row_meanabs(const float* __restrict__ delta, int d_in, int d_out,
                                                     const int32_t* __restrict__ sidx, int k, bool aligned,
                                                     float* __restrict__ step_out) {
  __shared__ float tile[2][64][65];
  const int tid = threadIdx.x, lane = tid & 63;
  const int row_l = tid >> 2, c_l = 16 * (tid & 3);
  const int row = 64 * blockIdx.x + row_l;
  const float* r = delta + (size_t)(row < d_out ? row : d_out - 1) * d_in;
  float4 v[4];
  auto load = [&](int c0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = c0 + c_l + 4 * i;
      v[i] = c < d_in ? load4(r + c, aligned) : make_float4(0, 0, 0, 0);   // d_in % 8 == 0
    }
  };
  load(0);
  int pos = 0;                                             // salient indices before this thread's columns
  double tot = 0.0;
  for (int c0 = 0, buf = 0; c0 < d_in; c0 += 64, buf ^= 1) {
    float a[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) { a[4 * i] = v[i].x; a[4 * i + 1] = v[i].y; a[4 * i + 2] = v[i].z; a[4 * i + 3] = v[i].w; }
    while (pos < k && sidx[pos] < c0 + c_l) ++pos;
    uint32_t sal = 0;
    for (int q = pos; q < k; ++q) {
      const int e = sidx[q] - (c0 + c_l);
      if (e < 0 || e >= 16) break;
      sal |= 1u << e;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) tile[buf][row_l][c_l + e] = (sal >> e) & 1u ? 0.0f : fabsf(a[e]);
    load(c0 + 64);
    __syncthreads();
    // one barrier per tile: the buffer written next was last read before this barrier
    if (tid < 64) {
      const int n = d_in - c0 < 64 ? d_in - c0 : 64;
#pragma unroll 8
      for (int e = 0; e < n; ++e) tot += (double)tile[buf][lane][e];
    }
  }
  const int out = 64 * blockIdx.x + lane, cnt = d_in - k;
  if (tid < 64 && out < d_out) step_out[out] = cnt > 0 ? (float)(2.0 * (tot / (double)cnt)) : 0.0f;
}

// Where the code of (row, col) is stored (see mes.h, "codes").  Blocks of 16 rows x 128 columns, chunk-major;
// inside a block lane = 16 g + r owns the 32 columns 32 g + e, e = 8 q + pp.
struct CodeLoc {
  size_t lo_word;   // index of the 32-bit word holding the low bits (all bits for b = 1, 2)
  int lo_shift;
  size_t hi_word;   // b = 3: word holding the high bit; b = 4: word holding the high two bits
  int hi_shift;
};

__device__ __forceinline__ CodeLoc code_location(int bits, int n_jt, int row, int col) {
  const int jt = row >> 4, r = row & 15;
  const int c = col >> 7, g = (col >> 5) & 3, e = col & 31, q = e >> 3, pp = e & 7;
  const int lane = 16 * g + r;
  const size_t blk = ((size_t)c * n_jt + jt) * (64 * bits);
  CodeLoc L;
  if (bits == 1) {
    L.lo_word = blk + lane;
    L.lo_shift = 4 * pp + q;
    L.hi_word = 0; L.hi_shift = 0;
  } else {
    L.lo_word = blk + lane * 2 + (q >> 1);
    L.lo_shift = 4 * pp + 2 * (q & 1);
    if (bits == 4) {   // a second 2-bit block
      L.hi_word = blk + 128 + lane * 2 + (q >> 1);
      L.hi_shift = 4 * pp + 2 * (q & 1);
    } else {
      L.hi_word = blk + 128 + lane;
      L.hi_shift = 4 * pp + q;
    }
  }
  return L;
}

struct PackParams {
  const float* delta;
  const int32_t* sidx;
  const float* step_in;     // GIVEN: the caller's steps (may be step_out); MEANABS: step_out, already written
  float* step_out;
  uint32_t* codes;
  uint16_t* sal;
  int* flag;                // set to 1 by block 0 if the salient list is not strictly ascending inside [0, d_in), else to 0
  int d_in, d_out, k, n_jt, n_chunks, n_sb, policy;
  bool aligned;             // delta is 16-byte aligned
};

// The value of the lane `CTRL` names (a permutation inside every 8 lanes) or'ed to this lane's.
template <int CTRL>
__device__ __forceinline__ uint32_t or_lanes(uint32_t v) {
  return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppMirror8 = 0x141;   // quad_perm [1,0,3,2], [2,3,0,1]; row_half_mirror

// Compression of one output channel per block, in one pass over the delta: the row is read once into registers
// (4 NV values per thread), its largest non-salient magnitude gives the step, the codes are formed from the registers,
// the fp16 salient values are picked out of the row.  Rows and columns of padding are written as zeros, so nothing
// has to be cleared before.
// Bound by the bytes of the delta matrix: 4096 x 14336 at 2 bits in 62 us (4.0 TB/s; six launches that read the row
// twice, searched the salient list for every element and divided in fp64: 719 us).
// A thread owns 4 consecutive columns per pass (16-byte loads, coalesced); the 8 threads of a 32-column group or
// their bits together through lane permutations and the first of them stores the group's words (see mes.h, "codes").
// The 16 rows of a row tile share every 128-byte line of code words, so their blocks are given ids 8 apart: those go
// to one XCD at about the same time, and its L2 holds whole lines when it writes them back.
// NV = 0: rows longer than 64 values per thread; the row is read a second time instead.
template <int BITS, bool EQ1, int NT, int NV>
__global__ __launch_bounds__(NT) void k_pack_rows(const PackParams p) {
  constexpr int kNW = NT / 64;
  __shared__ uint32_t mask[NV > 0 ? NT * NV / 8 : 1];      // one bit per column: salient
  __shared__ float red[kNW];
  const int tid = threadIdx.x, b = blockIdx.x;
  const int jt = (b >> 7) * 8 + (b & 7), r = (b >> 3) & 15, row = 16 * jt + r;
  if (jt >= p.n_jt) return;                                // row tiles are dealt in eights
  const bool real = row < p.d_out;
  const float* drow = p.delta + (size_t)(real ? row : 0) * p.d_in;
  float4 v[NV > 0 ? NV : 1];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = 4 * (i * NT + tid);
    v[i] = real && c < p.d_in ? load4(drow + c, p.aligned) : make_float4(0, 0, 0, 0);
  }
  bool bad = false;
  if (p.k > 0) {
    if constexpr (NV > 0) {
      for (int w = tid; w < NT * NV / 8; w += NT) mask[w] = 0;
      __syncthreads();
    }
    int mine = 0;
    for (int i = tid; i < p.k; i += NT) {
      const int c = p.sidx[i];
      const bool in = c >= 0 && c < p.d_in;
      mine |= !in || (i > 0 && p.sidx[i - 1] >= c);
      if constexpr (NV > 0) { if (in) atomicOr(&mask[c >> 5], 1u << (c & 31)); }
    }
    bad = __syncthreads_or(mine) != 0;
  }
  if (b == 0 && tid == 0) *p.flag = bad ? 1 : 0;
  // the salient bits of the 4 columns from c on
  auto salient4 = [&](int c) -> uint32_t {
    if (p.k == 0) return 0;
    if constexpr (NV > 0) return (mask[c >> 5] >> (c & 31)) & 15u;
    uint32_t m = 0;
    for (int e = 0; e < 4; ++e) m |= is_salient(p.sidx, p.k, c + e, nullptr) ? 1u << e : 0u;
    return m;
  };
  auto values = [&](int i, int c) -> float4 {
    if constexpr (NV > 0) return v[i];
    return real && c < p.d_in ? load4(drow + c, p.aligned) : make_float4(0, 0, 0, 0);
  };
  const int n_pass = NV > 0 ? NV : (p.d_in + 4 * NT - 1) / (4 * NT);

  float s = 0.0f;
  if (p.policy == MES_STEP_MAXABS) {
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < n_pass; ++i) {
      const int c = 4 * (i * NT + tid);
      float4 a = values(i, c);
      const uint32_t sal = c < p.d_in ? salient4(c) : 0;
      if (sal) {
        if (sal & 1) a.x = 0.0f;
        if (sal & 2) a.y = 0.0f;
        if (sal & 4) a.z = 0.0f;
        if (sal & 8) a.w = 0.0f;
      }
      m = max4(m, a);
    }
    m = wave_max(m);
    if (kNW > 1) {
      if ((tid & 63) == 0) red[tid >> 6] = m;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kNW; ++w) m = fmaxf(m, red[w]);
    }
    s = maxabs_step(m, BITS, EQ1);
  } else if (real) {
    s = p.step_in[row];
    if (p.policy == MES_STEP_GIVEN) s = s > 0.0f ? s : 0.0f;
  }
  __syncthreads();                                         // step_in may be step_out: every thread has read it
  if (real && tid == 0 && p.policy != MES_STEP_MEANABS) p.step_out[row] = s;

  const bool fast = fast_step(s);
  const float inv_s = fast ? 1.0f / s : 0.0f;
  constexpr float kHalf = (float)(1 << (BITS - 1));
  const int li = tid & 7;                                  // this thread's columns inside its group of 32: 4 li ..
  const int q = li >> 1, p0 = 4 * (li & 1);
#pragma unroll
  for (int i = 0; i < n_pass; ++i) {
    const int c = 4 * (i * NT + tid);
    const float4 a = values(i, c);
    const float w[4] = {a.x, a.y, a.z, a.w};
    const uint32_t skip = real && c < p.d_in ? salient4(c) : 15u;
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t u;
      if (fast) u = (uint32_t)(int)(clamped_cell<BITS, EQ1>(w[e], s, inv_s) + kHalf);
      else u = quant_code(w[e], s, BITS, EQ1 ? MES_GRID_EQ1 : MES_GRID_SYM);
      u = (skip >> e) & 1u ? 0u : u;
      if constexpr (BITS == 1) lo |= u << (4 * e);
      else lo |= (u & 3u) << (4 * e);
      if constexpr (BITS >= 3) hi |= (u >> 2) << (4 * e);
    }
    lo <<= 4 * p0 + (BITS == 1 ? q : 2 * (q & 1));
    if constexpr (BITS >= 3) hi <<= 4 * p0 + (BITS == 3 ? q : 2 * (q & 1));
    lo = or_lanes<kDppXor2>(or_lanes<kDppXor1>(lo));       // the 16 columns of four lanes
    if constexpr (BITS >= 3) hi = or_lanes<kDppXor2>(or_lanes<kDppXor1>(hi));
    uint32_t lo2 = 0, hi2 = 0;                             // two-word planes: the other 16 columns' word
    if constexpr (BITS == 1) lo = or_lanes<kDppMirror8>(lo);
    else lo2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, kDppMirror8, 0xf, 0xf, true);
    if constexpr (BITS == 3) hi = or_lanes<kDppMirror8>(hi);
    if constexpr (BITS == 4) hi2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, kDppMirror8, 0xf, 0xf, true);
    const int chunk = c >> 7, lane = 16 * ((c >> 5) & 3) + r;
    if (li == 0 && chunk < p.n_chunks) {
      uint32_t* blk = p.codes + ((size_t)chunk * p.n_jt + jt) * (64 * BITS);
      if constexpr (BITS == 1) blk[lane] = lo;
      else *reinterpret_cast<uint2*>(blk + 2 * lane) = make_uint2(lo, lo2);
      if constexpr (BITS == 3) blk[128 + lane] = hi;
      if constexpr (BITS == 4) *reinterpret_cast<uint2*>(blk + 128 + 2 * lane) = make_uint2(hi, hi2);
    }
  }

  // fp16 salient values of this row: rank rc sits in block rc / 32, lane 16 ((rc / 8) % 4) + r, element rc % 8.  With
  // a list that failed the check nothing is gathered (an index is an address only if the whole list is valid).
  for (int rc = tid; rc < 32 * p.n_sb; rc += NT) {
    uint16_t h = 0;
    if (real && !bad && rc < p.k) h = __half_as_ushort(__float2half_rn(drow[p.sidx[rc]]));
    p.sal[(((size_t)jt * p.n_sb + (rc >> 5)) * 64 + 16 * ((rc >> 3) & 3) + r) * 8 + (rc & 7)] = h;
  }
}

__device__ __forceinline__ uint32_t load_code(const uint32_t* codes, int bits, int n_jt, int row, int col) {
  const CodeLoc L = code_location(bits, n_jt, row, col);
  if (bits == 1) return (codes[L.lo_word] >> L.lo_shift) & 1u;
  const uint32_t lo = (codes[L.lo_word] >> L.lo_shift) & 3u;
  if (bits == 2) return lo;
  return lo | (((codes[L.hi_word] >> L.hi_shift) & (bits == 4 ? 3u : 1u)) << 2);
}

__global__ void k_unpack_delta(const uint32_t* __restrict__ codes, const float* __restrict__ step,
                               const uint16_t* __restrict__ sal, const int32_t* __restrict__ sidx, int d_in,
                               int d_out, int k, int bits, int grid, int n_ks, int n_sb,
                               float* __restrict__ delta_hat, uint8_t* __restrict__ codes_out) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)d_in * d_out) return;
  int row = (int)(idx / d_in), col = (int)(idx % d_in);
  int pos = 0;
  if (is_salient(sidx, k, col, &pos)) {
    int jt = row >> 4, r = row & 15, sb = pos >> 5, g = (pos >> 3) & 3, e = pos & 7;
    uint16_t hb = sal[(((size_t)(jt * n_sb + sb) * 64) + 16 * g + r) * 8 + e];
    if (delta_hat) delta_hat[idx] = __half2float(__ushort_as_half(hb));
    if (codes_out) codes_out[idx] = 0xFF;
    return;
  }
  uint32_t u = load_code(codes, bits, n_ks, row, col);
  if (codes_out) codes_out[idx] = (uint8_t)u;
  if (delta_hat) delta_hat[idx] = (float)(((double)u - zero_point(bits, grid)) * (double)step[row]);
}

// ---- salient selection (Eq. 2) ------------------------------------------------------------------------
// score_i = (sum_t x_ti^2) * (sum_j (D_ji - Dhat_ji)^2): the same number as the double sum of Eq. 2,
// since x_ti factors out of each squared term.
// A block owns 16 input channels (64-byte pieces of every row) and all the rows: 256 row lanes of 4 threads, 4
// channels per thread, fp64 sums per thread, added up over the row lanes in a fixed order that is the same for every
// channel (equal columns get equal scores).  (u - z) s is exact in fp64 (half integers of few bits times 24 bits), so
// the fused multiply-add below is the rounded difference D - Dhat itself.
// Bound by the bytes of the delta, in 64-byte pieces: 4096 x 4096 in 16 us (4.2 TB/s; one thread per channel
// walking all the rows with an fp64 division each: 1448 us).  Neighbouring blocks share 128-byte lines: their ids go to one XCD.
template <int BITS, bool EQ1>
__global__ __launch_bounds__(1024) void k_scores(const float* __restrict__ delta, const float* __restrict__ xc, int n,
                                                 int d_in, int d_out, const float* __restrict__ step, bool aligned,
                                                 bool x_aligned, double* __restrict__ score, double* __restrict__ score_out,
                                                 int* __restrict__ rank) {
  const int strips = (d_in + 15) / 16, per_xcd = (strips + 7) / 8;
  const int strip = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (strip >= strips) return;                             // (the strips are dealt to the 8 XCDs evenly)
  const int tid = threadIdx.x, rl = tid >> 2, c = 16 * strip + 4 * (tid & 3);
  const bool in = c < d_in;                                // d_in % 8 == 0
  double err[4] = {0, 0, 0, 0}, xs[4] = {0, 0, 0, 0};
  if (in) {
    const float* col = delta + c;
#pragma unroll 4
    for (int j = rl; j < d_out; j += 256) {
      const float4 a = load4(col + (size_t)j * d_in, aligned);
      const float w[4] = {a.x, a.y, a.z, a.w};
      const float s = step[j];
      const double sd = (double)s;
      if (fast_step(s)) {
        const float inv_s = __builtin_amdgcn_rcpf(s);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float level = clamped_cell<BITS, EQ1>(w[e], s, inv_s) + (EQ1 ? 0.0f : 0.5f);
          const double d = __builtin_fma(-(double)level, sd, (double)w[e]);
          err[e] = __builtin_fma(d, d, err[e]);
        }
      } else {
        const double z = zero_point(BITS, EQ1 ? MES_GRID_EQ1 : MES_GRID_SYM);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double d = (double)w[e] - ((double)quant_code(w[e], s, BITS, EQ1 ? MES_GRID_EQ1 : MES_GRID_SYM) - z) * sd;
          err[e] = __builtin_fma(d, d, err[e]);
        }
      }
    }
    const float* xcol = xc + c;
#pragma unroll 4
    for (int t = rl; t < n; t += 256) {
      const float4 a = load4(xcol + (size_t)t * d_in, x_aligned);
      const float w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) xs[e] = __builtin_fma((double)w[e], (double)w[e], xs[e]);
    }
  }
  __shared__ double sum[2][16][16];                        // [err, xs][wavefront][channel]
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#pragma unroll
    for (int off = 4; off < 64; off <<= 1) {
      err[e] += __shfl_xor(err[e], off);
      xs[e] += __shfl_xor(xs[e], off);
    }
    if ((tid & 63) < 4) {
      sum[0][tid >> 6][4 * (tid & 3) + e] = err[e];
      sum[1][tid >> 6][4 * (tid & 3) + e] = xs[e];
    }
  }
  __syncthreads();
  if (tid < 16 && 16 * strip + tid < d_in) {
    double te = 0.0, tx = 0.0;
    for (int w = 0; w < 16; ++w) { te += sum[0][w][tid]; tx += sum[1][w][tid]; }
    score[16 * strip + tid] = tx * te;
    if (score_out) score_out[16 * strip + tid] = tx * te;
    rank[16 * strip + tid] = 0;                            // for k_rank to add to
  }
}

// rank[i] += channels among this wavefront's share that come before channel i (a larger score, or the same one at a lower
// index).  A block ranks 64 channels, one per lane; the channels compared with are dealt to the 4 wavefronts of gridDim.y
// blocks, are the same for all lanes and come through scalar loads.  The shares add up with integer atomics (k_scores
// cleared the sums): the result does not depend on their order.  4096 channels with 16 blocks per 64 channels: 6 us, one block
// of 16 wavefronts 14 us (64 blocks leave most of the chip idle), the same through LDS 27 us, one thread per channel
// comparing with all of them 281 us.
__global__ __launch_bounds__(256) void k_rank(const double* __restrict__ score, int d_in, int* __restrict__ rank_out) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = 64 * blockIdx.x, i = i0 + lane;
  const double s = score[i < d_in ? i : d_in - 1];
  const int shares = 4 * gridDim.y, per = (d_in + shares - 1) / shares, share = 4 * blockIdx.y + wave;
  const int lo = share * per < d_in ? share * per : d_in, hi = lo + per < d_in ? lo + per : d_in;
  const int a = lo > i0 ? lo : (i0 < hi ? i0 : hi);        // [lo, a): before the block's channels, [b, hi): after them
  const int b = a > i0 + 64 ? a : (i0 + 64 < hi ? i0 + 64 : hi);
  int rank = 0;
#pragma unroll 8
  for (int o = lo; o < a; ++o) rank += score[o] >= s;
  for (int o = a; o < b; ++o) {
    const double so = score[o];
    rank += (so > s) || (so == s && o < i);
  }
#pragma unroll 8
  for (int o = b; o < hi; ++o) rank += score[o] > s;
  __shared__ int part[4][64];
  part[wave][lane] = rank;
  __syncthreads();
  if (wave == 0 && i < d_in) atomicAdd(rank_out + i, part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane]);
}

// The chosen channels (fewer than k come before them) in ascending order: one block, 1024 channels at a time, positions by
// counting lane masks (4096 channels: 4 us; every thread counting the chosen ones before it: 198 us).
__global__ __launch_bounds__(1024) void k_compact(const int* __restrict__ rank, int d_in, int k, int32_t* __restrict__ idx_out) {
  __shared__ int count[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int before = 0;
  for (int base = 0, buf = 0; base < d_in; base += 1024, buf ^= 1) {
    const int i = base + tid;
    const bool c = i < d_in && rank[i] < k;
    const unsigned long long m = __ballot(c);
    if (lane == 0) count[buf][wave] = __popcll(m);
    __syncthreads();
    int pos = before + __popcll(m & ((1ull << lane) - 1ull));
    for (int w = 0; w < 16; ++w) {
      const int cw = count[buf][w];
      pos += w < wave ? cw : 0;
      before += cw;
    }
    if (c && pos < k) idx_out[pos] = i;   // more than k can only be chosen when scores are NaN
  }
}

inline unsigned blocks_for(size_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_pack_base(const uint16_t* w, int d_in, int d_out, uint16_t* out, hipStream_t s) {
  int n_kb = ceil_to(d_in, kColPad) / 32;
  size_t n_slots = (size_t)(ceil_to(d_out, kRowPad) / 16) * n_kb * 64;
  k_pack_base<<<blocks_for(n_slots, 256), 256, 0, s>>>(w, d_in, d_out, n_kb, n_slots, reinterpret_cast<uint4*>(out));
  return hipGetLastError();
}

hipError_t launch_unpack_base(const uint16_t* t, int d_in, int d_out, uint16_t* out, hipStream_t s) {
  int n_kb = ceil_to(d_in, kColPad) / 32;
  size_t n_slots = (size_t)(ceil_to(d_out, kRowPad) / 16) * n_kb * 64;
  k_unpack_base<<<blocks_for(n_slots, 256), 256, 0, s>>>(reinterpret_cast<const uint4*>(t), d_in, d_out, n_kb, n_slots, out);
  return hipGetLastError();
}

// Plain streaming copy, 16 bytes per thread and iteration: the yardstick the HBM byte counters are scaled by.
__global__ __launch_bounds__(256) void k_copy_probe(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

hipError_t launch_copy_probe(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 16;
  if (n == 0) return hipSuccess;
  k_copy_probe<<<(unsigned)(blocks_for(n, 256) < 8192 ? blocks_for(n, 256) : 8192), 256, 0, s>>>(
      reinterpret_cast<const uint4*>(src), reinterpret_cast<uint4*>(dst), n);
  return hipGetLastError();
}

namespace {

// Threads per block and values per thread of k_pack_rows by row length: 64 threads up to 1024 columns, 256 beyond,
// and registers for the whole row up to 16384 columns.
template <int BITS, bool EQ1>
void launch_pack_rows(const PackParams& p, hipStream_t s) {
  const unsigned grid = (unsigned)((p.n_jt + 7) / 8 * 8 * 16);
  const int cols = kColPad * p.n_chunks;                   // padding columns get code 0
  if (cols <= 1024) k_pack_rows<BITS, EQ1, 64, 4><<<grid, 64, 0, s>>>(p);
  else if (cols <= 4096) k_pack_rows<BITS, EQ1, 256, 4><<<grid, 256, 0, s>>>(p);
  else if (cols <= 8192) k_pack_rows<BITS, EQ1, 256, 8><<<grid, 256, 0, s>>>(p);
  else if (cols <= 16384) k_pack_rows<BITS, EQ1, 256, 16><<<grid, 256, 0, s>>>(p);
  else k_pack_rows<BITS, EQ1, 256, 0><<<grid, 256, 0, s>>>(p);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

hipError_t launch_pack_delta(const float* delta, int d_in, int d_out, const int32_t* sidx, int k, int bits,
                             int grid, int policy, const float* step_in, uint32_t* codes, float* step_out,
                             uint16_t* sal, int* flag, hipStream_t s) {
  hipError_t e;
  PackParams p;
  p.delta = delta;
  p.sidx = sidx;
  p.step_in = policy == MES_STEP_MEANABS ? step_out : step_in;
  p.step_out = step_out;
  p.codes = codes;
  p.sal = sal;
  p.flag = flag;
  p.d_in = d_in;
  p.d_out = d_out;
  p.k = k;
  p.n_jt = ceil_to(d_out, kRowPad) / 16;
  p.n_chunks = ceil_to(d_in, kColPad) / kColPad;
  p.n_sb = ceil_to(k, kSalPad) / 32;
  p.policy = policy;
  p.aligned = aligned16(delta);
  if (policy == MES_STEP_MEANABS) {
    k_row_meanabs<<<blocks_for(d_out, 64), 256, 0, s>>>(delta, d_in, d_out, sidx, k, p.aligned, step_out);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const bool eq1 = grid == MES_GRID_EQ1;
  switch (bits) {
    case 1: launch_pack_rows<1, false>(p, s); break;
    case 2: eq1 ? launch_pack_rows<2, true>(p, s) : launch_pack_rows<2, false>(p, s); break;
    case 3: eq1 ? launch_pack_rows<3, true>(p, s) : launch_pack_rows<3, false>(p, s); break;
    default: eq1 ? launch_pack_rows<4, true>(p, s) : launch_pack_rows<4, false>(p, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_unpack_delta(const mes_delta& d, float* delta_hat, uint8_t* codes_out, hipStream_t s) {
  int pi = ceil_to(d.d_in, kColPad);
  int n_ks = ceil_to(d.d_out, kRowPad) / 16;   // row tiles
  int n_sb = ceil_to(d.k, kSalPad) / 32;
  size_t n = (size_t)d.d_in * d.d_out;
  k_unpack_delta<<<blocks_for(n, 256), 256, 0, s>>>(reinterpret_cast<const uint32_t*>(d.codes), d.step,
                                                    reinterpret_cast<const uint16_t*>(d.salient), d.salient_idx, d.d_in,
                                                    d.d_out, d.k, d.bits, d.grid, n_ks, n_sb, delta_hat, codes_out);
  return hipGetLastError();
}

hipError_t launch_select(const float* delta, const float* xc, int n, int d_in, int d_out, int bits, int grid,
                         int policy, int k, int32_t* idx_out, double* score_out, void* ws, hipStream_t s) {
  // workspace: double score[d_in] | float step[d_out] | int rank[d_in]
  char* p = reinterpret_cast<char*>(ws);
  double* score = reinterpret_cast<double*>(p);
  p += (size_t)ceil_to(d_in, 32) * sizeof(double);
  float* step = reinterpret_cast<float*>(p);
  p += (size_t)ceil_to(d_out, 64) * sizeof(float);
  int* rank = reinterpret_cast<int*>(p);
  const bool aligned = aligned16(delta), x_aligned = aligned16(xc), eq1 = grid == MES_GRID_EQ1;
  hipError_t e;
  if (policy == MES_STEP_MEANABS) k_row_meanabs<<<blocks_for(d_out, 64), 256, 0, s>>>(delta, d_in, d_out, nullptr, 0, aligned, step);
  else k_row_maxabs<<<d_out, 256, 0, s>>>(delta, d_in, bits, grid, aligned, step);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const unsigned strips = ((unsigned)((d_in + 15) / 16) + 7) / 8 * 8;
  auto scores = [&](auto kernel) { kernel<<<strips, 1024, 0, s>>>(delta, xc, n, d_in, d_out, step, aligned, x_aligned, score, score_out, rank); };
  switch (bits) {
    case 1: scores(k_scores<1, false>); break;
    case 2: eq1 ? scores(k_scores<2, true>) : scores(k_scores<2, false>); break;
    case 3: eq1 ? scores(k_scores<3, true>) : scores(k_scores<3, false>); break;
    default: eq1 ? scores(k_scores<4, true>) : scores(k_scores<4, false>); break;
  }
  if ((e = hipGetLastError()) != hipSuccess || k == 0) return e;
  k_rank<<<dim3(blocks_for(d_in, 64), 16), 256, 0, s>>>(score, d_in, rank);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_compact<<<1, 1024, 0, s>>>(rank, d_in, k, idx_out);
  return hipGetLastError();
}

}  // namespace mes
