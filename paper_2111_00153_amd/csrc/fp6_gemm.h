// FP6 tile kernel of librmsmp (gfx950): the mixed-scheme GEMM / implicit-im2col convolution with 4-bit
// activations on v_mfma_scale_f32_32x32x64_f8f6f4, at the 6-bit rate of the matrix cores (twice the
// int8 rate), with exact integer results.
//
// Why it is exact.  Every operand is an integer that a 6-bit float holds: an activation code 0..15 is
// the E2M3 bit pattern of the same number (value code / 8); Fixed-4 levels (|q| <= 7) and PoT-4 levels
// (0, +-1, .., +-64) are E3M2 numbers (value q / 4); a Fixed-8 level is 16 h + l with |h|, |l| <= 8,
// two E3M2 numbers.  The accumulators of the tile kernel hold 1/32 of integers (4 and 8 are made up for in the row's
// multiplier, 16 when the two sums of a Fixed-8 tile are added, or as a block scale where they share an accumulator), those of the split kernel, which gives the instruction these
// factors as block scales, integers.  Layers are packed for this
// kernel only if 15 * sum_k (|16 h| + |l|) of every row stays below 2^24: then every partial sum, in
// whatever order the hardware adds, is an integer that fp32 holds.  (That the instruction
// keeps such sums exact whatever the mix of products is measured, not promised: the tests hold it
// against integers with the largest and the smallest levels in one instruction, odd sums and both
// signs, just below 2^24.)
//
// Weights are stored a second time in operand form when a layer is packed (0.75 bytes a weight, 1.5 in
// tiles with Fixed-8 rows): the K loop has no weight decode at all, where the int8 kernels spend up to
// 11 vector instructions per 8 PoT codes.  The operand of 32 rows x 64 k is 64 lanes x 16 bytes
// followed by 64 lanes x 8 bytes: two coalesced reads.  k runs over (tap, block of 32 channels), a
// tap's channels padded to whole blocks with zero weights, so that one 16-byte read of an activation
// tensor is one lane's half-fragment whatever the channel count.
//
// Activations go from memory to LDS as 6-bit fragments in lane order (nine vector instructions widen
// 16 nibbles to 16 fields), double-buffered, 128 k at a time, one barrier per 128 k; they are shared by
// the waves of a work-group, whose weights come straight from the L2 into registers.
#pragma once
#include <hip/hip_runtime.h>

#include "device_common.h"

namespace rmsmp {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef unsigned fp6_v4u __attribute__((ext_vector_type(4)));
typedef unsigned fp6_v2u __attribute__((ext_vector_type(2)));

constexpr int FP6_FRAG = 1536;  // bytes of one operand: 32 rows (or columns) x 64 k x 6 bits
// An activation operand in LDS: the 16-byte parts of its lanes 0..31, those of lanes 32..63, then the 8-byte parts
// the same way.  The gaps of 64 bytes and the pitch (128 bytes beyond a multiple of 256) put the four parts that
// neighbouring staging threads write, two halves of two operands, side by side in the banks.
constexpr int FP6_LDS_HALF = 512 + 64, FP6_LDS_TAIL = FP6_LDS_HALF + 512, FP6_LDS_TAIL_HALF = 256 + 64;
constexpr int FP6_LDS_FRAG = FP6_LDS_TAIL + FP6_LDS_TAIL_HALF + 256;
static_assert(FP6_LDS_FRAG % 256 == 128, "see above");

struct Fp6Args {
  const uint8_t* w;       // fragments: [tile][64-deep K step][hi, lo parts of a Fixed-8 tile][FP6_FRAG]
  const int32_t* p_meta;
  const void* X;
  void* Y;
  const float* bias;
  int32_t M, N;           // rows; columns (output pixels)
  int32_t n_tiles, n_single;  // weight tiles; those stored in one part (the others, at the end, in two)
  int32_t pairs;          // what a tile kernel's waves are given (fp6_pair)
  int32_t nsteps;         // 64-deep K steps
  int32_t ld;             // bytes of one input column (pixel)
  uint32_t x_bytes, y_bytes;
  int32_t gx, gy;         // column blocks, row blocks of the grid
  int32_t by_rows;        // see fp6_block
  float act_scale, out_inv_scale;
  int32_t zp, relu, out_kind, out_zero_point;
  int32_t last_rows;      // live rows of the last tile
  int32_t whole_lines;    // 32 columns of a 32-bit output row are a line of 128 bytes
  // convolutions
  int32_t CB;             // 32-channel blocks of a tap
  struct Div {
    uint32_t magic;       // ceil(2^(32 + shift) / d); 0 for d == 1
    int32_t shift;
  } by_cb, by_kw, by_hw, by_ow;
  int32_t KW, H, W, OHW, OW, stride, pad;
  GeluTable gelu;         // break points of GELU output (out_kind 3)
  GeluBins bins;          // the same cut into bins, for the tile kernel
};

// n / d for 0 <= n < 2^31
__device__ __forceinline__ int fp6_div(int n, const Fp6Args::Div& d) { return d.magic ? (int)(__umulhi((uint32_t)n, d.magic) >> d.shift) : n; }

struct Fp6Frag {
  v4i a;
  v2i b;
};
__device__ __forceinline__ v8i fp6_operand(const Fp6Frag& f) {
  v8i r;
  r[0] = f.a[0], r[1] = f.a[1], r[2] = f.a[2], r[3] = f.a[3], r[4] = f.b[0], r[5] = f.b[1];
  r[6] = 0, r[7] = 0;
  return r;
}
// acc += weights (E3M2, unit 1/4) x activations (E2M3, unit 1/8), in units of 1/32.  Without block scales: they are an
// instruction word and registers of their own, with which the loops below spilled (256 x 128 outputs of a 3x3 layer, 144 to 144
// channels, 16 images of 57 x 57: 24.2 -> 18.5 us).
__device__ __forceinline__ v16f fp6_mfma(const Fp6Frag& w, const Fp6Frag& x, v16f acc) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp6_operand(w), fp6_operand(x), acc, 3, 2, 0, 0, 0, 0);
}

// acc += 16 x weights x activations: hi parts, in the accumulators of the lo parts
__device__ __forceinline__ v16f fp6_mfma_hi(const Fp6Frag& w, const Fp6Frag& x, v16f acc) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp6_operand(w), fp6_operand(x), acc, 3, 2, 0, 0x83838383, 0, 0x7f7f7f7f);
}

// Sixteen 4-bit codes (two words, eight nibbles each) to sixteen 6-bit fields (three words).  Field order
// is whatever takes the fewest instructions; the weights are stored in the same order (kFp6Order).
__device__ __forceinline__ void fp6_widen(uint32_t s0, uint32_t s1, uint32_t (&w)[3]) {
  const uint32_t t = s0 << 2, u = __builtin_amdgcn_alignbit(s1, s0, 30);  // u = s1 << 2 | s0 >> 30
  w[0] = (s0 & 0x0F00F00Fu) | (t & 0xC03C03C0u);
  w[1] = (s1 & 0xF00F00F0u) | (t & 0x03C03C00u) | (u & 3u);
  w[2] = (s1 & 0x00F00F00u) | (u & 0x3C03C03Cu);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t fp6_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// 16 bytes at byte offset off of X; past the end: zeros.  RAGGED: a column is no multiple of 16 bytes,
// so the last columns' reads may begin inside the tensor and end outside; those are read 16 bytes from
// the end and moved into place.
template <bool RAGGED>
__device__ __forceinline__ uint4 fp6_read_x(__amdgpu_buffer_rsrc_t xr, uint32_t off, uint32_t x_bytes) {
  if constexpr (RAGGED) {
    const uint32_t last = x_bytes - 16u;
    const bool cut = off > last && off < x_bytes;
    const fp6_v4u g = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(cut ? last : off), 0, 0);
    uint4 v = make_uint4(g.x, g.y, g.z, g.w);
    if (cut) {
      const uint32_t sh = (off - last) * 8u;  // 8..120
      uint64_t lo = (uint64_t)v.x | ((uint64_t)v.y << 32), hi = (uint64_t)v.z | ((uint64_t)v.w << 32);
      if (sh >= 64u) lo = hi >> (sh - 64u), hi = 0;
      else lo = (lo >> sh) | (hi << (64u - sh)), hi >>= sh;
      v = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    }
    return v;
  } else {
    const fp6_v4u g = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)off, 0, 0);
    return make_uint4(g.x, g.y, g.z, g.w);
  }
}

// LDS barrier that leaves global loads in flight.
__device__ __forceinline__ void fp6_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// 32-bit results go past the caches (aux bit 1: non-temporal) where every 32 columns of a row are a whole line of 128 bytes:
// they are 8 times as large as the activations and would push those and the weights out of the L2 (the six GEMMs
// of a 768-wide encoder layer at 4096 tokens 76.4 -> 74.5 us).  Parts of lines would each go to memory by
// themselves: 3072 x 768 x 8190 33 -> 80 us.
template <bool STREAM>
__device__ __forceinline__ void fp6_store32(__amdgpu_buffer_rsrc_t yr, unsigned v, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b32(v, yr, (int)off, 0, STREAM ? 2 : 0);
}

constexpr uint32_t FP6_OUTSIDE = 0x80000000u;  // an offset past every tensor

// Row data of the epilogue in LDS, per wave: [field][64 rows].
enum Fp6Meta { FM_MUL = 0, FM_ZC = 1, FM_ROW = 2, FM_BIAS = 3, FM_FIELDS = 4 };
constexpr int FP6_META_BYTES = FM_FIELDS * 64 * 4;

// What a wave multiplies: two operands ("slots") of 32 rows each.  Tiles stored in one part go two to a wave; a tile
// with Fixed-8 rows is a wave's two slots by itself, its hi parts and its lo parts, which are added up at the end.  So
// every wave has the same K loop and the same work.
struct Fp6Pair {
  int t0, t1;          // tiles; t1 < 0: the second slot repeats the first tile, or holds its lo parts
  bool two;
  int64_t off0, off1;  // first operand of each slot
  int stride;          // bytes from one K step to the next
};
__device__ __forceinline__ Fp6Pair fp6_pair(const Fp6Args& a, int q) {
  const int64_t one = (int64_t)a.nsteps * FP6_FRAG;
  const int singles = (a.n_single + 1) >> 1;
  Fp6Pair p;
  p.two = q >= singles;
  if (p.two) {
    const int i = q - singles;
    p.t0 = a.n_single + i, p.t1 = -1;
    p.off0 = a.n_single * one + i * 2 * one;
    p.off1 = p.off0 + FP6_FRAG;
    p.stride = 2 * FP6_FRAG;
  } else {
    p.t0 = 2 * q, p.t1 = 2 * q + 1 < a.n_single ? 2 * q + 1 : -1;
    p.off0 = p.t0 * one;
    p.off1 = p.t1 < 0 ? p.off0 : p.off0 + one;
    p.stride = FP6_FRAG;
  }
  return p;
}

// The other way to give tiles to waves (fp6_joined_kernel): two neighbouring ones to each, whatever they hold; twice the same one
// where the last, which has Fixed-8 rows, is left over.  Such a tile is then two operands a K step for one accumulator.
__device__ __forceinline__ Fp6Pair fp6_pair_joined(const Fp6Args& a, int q) {
  const int64_t one = (int64_t)a.nsteps * FP6_FRAG;
  auto off = [&](int t) { return (t <= a.n_single ? t : 2 * t - a.n_single) * one; };
  const int t0 = 2 * q, t1 = t0 + 1 < a.n_tiles ? t0 + 1 : -1;
  return Fp6Pair{t0, t1, false, off(t0), off(t1 < 0 ? t0 : t1), FP6_FRAG};
}

// Row data of a pair, a row a lane: multiplier rowscale * act_scale * 32, zero point * row sum / 32 (both exact),
// output row (byte offset of the row for int32 / fp32 output; past the end for padding) go to LDS at once, the
// bias (0 where there is none) comes back in a register: its read would be the newest of all, and waiting for it
// before the K loop would be waiting for all of that loop's first reads.
__device__ __forceinline__ int4 fp6_read_meta(const Fp6Args& a, const Fp6Pair& pair, int lane) {
  const int t = lane < TILE_M ? pair.t0 : pair.t1;
  return ((const int4*)a.p_meta)[t >= 0 ? t * TILE_M + (lane & (TILE_M - 1)) : 0];
}
__device__ __forceinline__ float fp6_stage_meta(const Fp6Args& a, const Fp6Pair& pair, const int4& m, float* dst, int lane) {
  const bool live = (lane < TILE_M || pair.t1 >= 0) && m.z >= 0;
  dst[FM_MUL * 64 + lane] = __fmul_rn(__fmul_rn(__int_as_float(m.x), a.act_scale), 32.0f);
  dst[FM_ZC * 64 + lane] = (float)(a.zp * m.y) * 0.03125f;
  dst[FM_ROW * 64 + lane] = __int_as_float(live ? (int)((uint32_t)m.z * (uint32_t)a.N * 4u) : (int)0x80000000);
  const __amdgpu_buffer_rsrc_t br = fp6_rsrc(a.bias, a.bias ? (uint32_t)a.M * 4u : 0u);
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(br, live ? m.z * 4 : (int)FP6_OUTSIDE, 0, 0));
}

// 4-bit codes of 16 rows from fp32 accumulators (integers): the operations of requant_block.
template <bool BIAS, bool RELU>
__device__ __forceinline__ void fp6_requant(const v16f& v, const float (&m)[16], const float (&bias)[16], float inv_s, uint32_t (&packed)[2]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t even = 0u, odd = 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = 8 * h + i;
      float y = __fmul_rn(v[r], m[r]);
      if (BIAS) y = __fadd_rn(y, bias[r]);
      if (RELU) y = fmaxf(y, 0.0f);
      const float t = fminf(__fmul_rn(y, inv_s), 15.0f);
      if (i & 1)
        odd = __builtin_amdgcn_cvt_pk_u8_f32(t, i >> 1, odd);
      else
        even = __builtin_amdgcn_cvt_pk_u8_f32(t, i >> 1, even);
    }
    packed[h] = even | (odd << 4);
  }
}

__device__ __forceinline__ void fp6_read16(const float* p, float (&v)[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 f = ((const float4*)p)[q];
    v[4 * q] = f.x, v[4 * q + 1] = f.y, v[4 * q + 2] = f.z, v[4 * q + 3] = f.w;
  }
}

// GELU codes by bins: entry i of the table in LDS is {step of bin i (or +inf), code below it | code from it on << 8}.
// What bounds GELU output is this and nothing else: with a guess from y itself and one or two corrections, each a read of the
// break points by every lane, 3072 x 768 x 4096 took 20.6 us (12.1 with ReLU); with the bins 15.6.
constexpr int FP6_BIN_BYTES = GeluBins::BINS * 8;
// (a whole wave, lane i for bin i; a lane reads one step for all of them)
__device__ __forceinline__ void fp6_stage_bins(const GeluBins& g, v2u* table, int lane) {
  const int k0 = lane < 31 ? lane : 30;
  const float my_step = g.step[k0];
  const int my_code = g.code[k0 + 1], my_bin = (int)__builtin_fmaf(my_step, g.scale, g.offset);
  uint32_t below = g.code[0], from = below;
  float step = __builtin_inff();
#pragma unroll 1
  for (int k = 0; k < g.n; ++k) {
    const float y = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_step), k));
    const int bin = __builtin_amdgcn_readlane(my_bin, k);
    const uint32_t code = (uint32_t)__builtin_amdgcn_readlane(my_code, k);
    if (bin == lane) step = y, from = code;
    if (bin < lane) below = from = code;
  }
  table[lane] = (v2u){__float_as_uint(step), below | (from << 8)};
}
static_assert(GeluBins::BINS == LANES, "a lane per bin");
__device__ __forceinline__ void fp6_gelu(const v16f& v, const float (&m)[16], const float (&bias)[16], const v2u* table, float scale, float offset, uint32_t (&packed)[2]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float y[8];
    v2u entry[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      y[i] = __fadd_rn(__fmul_rn(v[8 * h + i], m[8 * h + i]), bias[8 * h + i]);
      const float at = __builtin_amdgcn_fmed3f(__builtin_fmaf(y[i], scale, offset), 0.0f, (float)(GeluBins::BINS - 1));
      entry[i] = table[(uint32_t)at];
    }
    uint32_t w = 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) w |= ((entry[i].y >> (y[i] >= __uint_as_float(entry[i].x) ? 8 : 0)) & 15u) << (4 * i);
    packed[h] = w;
  }
}

// Finish NB 32x32 blocks of one weight tile.  meta: field 0 of the lane's first row; n: the lane's column of
// block 0 (block j: + 32 j); n_rows: live rows of the lane's 16; gpos: its first grouped row.
template <int NB, bool GELU>
__device__ __forceinline__ void fp6_finish(const Fp6Args& a, v16f (&acc)[NB], const float* meta, const v2u* bins, int n_rows, int gpos, int n) {
  if (n_rows <= 0) return;
  float m[16];
  if (a.zp != 0) {
    fp6_read16(meta + FM_ZC * 64, m);
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] -= m[r];
  }
  if (!GELU && a.out_kind <= 1) {
    const __amdgpu_buffer_rsrc_t yr = fp6_rsrc(a.Y, a.y_bytes);
    uint32_t row[16];
    {
      float f[16];
      fp6_read16(meta + FM_ROW * 64, f);
#pragma unroll
      for (int r = 0; r < 16; ++r) row[r] = __float_as_uint(f[r]);
    }
    if (a.out_kind == 1) fp6_read16(meta, m);
    float bias[16];
    if (a.out_kind == 1) fp6_read16(meta + FM_BIAS * 64, bias);
    const float floor_y = a.relu ? 0.0f : -__builtin_inff();
    auto store = [&](auto stream_tag, auto kind_tag) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
        if (n + 32 * j < a.N) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            unsigned v;
            if constexpr (decltype(kind_tag)::value == 0)
              v = (unsigned)(int)(acc[j][r] * 32.0f);
            else
              v = __float_as_uint(fmaxf(__fadd_rn(__fmul_rn(acc[j][r], m[r]), bias[r]), floor_y));
            fp6_store32<decltype(stream_tag)::value>(yr, v, row[r] + (uint32_t)(n + 32 * j) * 4u);
          }
        }
    };
    const std::integral_constant<int, 0> as_int{};
    const std::integral_constant<int, 1> as_float{};
    if (a.out_kind == 0) {
      a.whole_lines ? store(std::true_type{}, as_int) : store(std::false_type{}, as_int);
    } else {
      a.whole_lines ? store(std::true_type{}, as_float) : store(std::false_type{}, as_float);
    }
    return;
  }
  fp6_read16(meta, m);
  float bias[16];
  const bool has_bias = a.bias != nullptr;
  const bool relu_q = a.relu != 0 && !(a.out_inv_scale > 0.0f);
  if (GELU || has_bias || relu_q) fp6_read16(meta + FM_BIAS * 64, bias);
  const int half_m = a.M >> 1;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    uint32_t packed[2];
    if constexpr (GELU) {
      if (a.bins.n > 0) {
        fp6_gelu(acc[j], m, bias, bins, a.bins.scale, a.bins.offset, packed);
      } else {
        constexpr int KOFF = (int)__builtin_offsetof(Fp6Args, gelu) - (int)__builtin_offsetof(GemmArgs, gelu);
        gelu_requant_block<KOFF>(acc[j], m, bias, a.out_inv_scale, a.out_zero_point, packed);
      }
    } else if (relu_q) {  // (a bias of 0 where there is none)
      fp6_requant<true, true>(acc[j], m, bias, a.out_inv_scale, packed);
    } else if (has_bias) {
      fp6_requant<true, false>(acc[j], m, bias, a.out_inv_scale, packed);
    } else {
      fp6_requant<false, false>(acc[j], m, bias, a.out_inv_scale, packed);
    }
    const int nn = n + 32 * j;
    if (nn < a.N) {
      RMSMP_GLOBAL uint8_t* dst = as_global((uint8_t*)a.Y) + (int64_t)nn * half_m + (gpos >> 1);
      if (n_rows == 16) {
        typedef v2u v2u_any __attribute__((aligned(1)));
        *(RMSMP_GLOBAL v2u_any*)dst = (v2u){packed[0], packed[1]};
      } else {
        for (int b = 0; b < n_rows / 2; ++b) dst[b] = (uint8_t)(packed[b >> 2] >> (8 * (b & 3)));
      }
    }
  }
}

// Where a staging thread's column lies: byte offset of its tap (0, 0), and for convolutions the input
// coordinates of that tap.
struct Fp6Col {
  uint32_t base;
  int ih0, iw0;
};
template <bool CONV>
__device__ __forceinline__ Fp6Col fp6_col(const Fp6Args& a, int n) {
  Fp6Col c;
  c.ih0 = c.iw0 = 0;
  if constexpr (CONV) {
    const int b = fp6_div(n, a.by_hw);
    const int rem = n - b * a.OHW;
    const int oh = fp6_div(rem, a.by_ow);
    const int ow = rem - oh * a.OW;
    c.ih0 = oh * a.stride - a.pad;
    c.iw0 = ow * a.stride - a.pad;
    c.base = (uint32_t)(((b * a.H + c.ih0) * a.W + c.iw0) * a.ld);
    if (n >= a.N) c.ih0 = -(1 << 20);  // no tap of it is inside
  } else {
    c.base = n < a.N ? (uint32_t)n * (uint32_t)a.ld : FP6_OUTSIDE;
  }
  return c;
}

// The lane's K block (32 channels of one tap) kb of column c, as packed nibbles.
struct Fp6Tap {
  uint32_t off;  // bytes from the column's base
  int kh, kw;
};
template <bool CONV>
__device__ __forceinline__ Fp6Tap fp6_tap(const Fp6Args& a, int kb) {
  Fp6Tap t;
  t.kh = t.kw = 0;
  if constexpr (CONV) {
    const int tap = fp6_div(kb, a.by_cb);
    const int cb = kb - tap * a.CB;
    t.kh = fp6_div(tap, a.by_kw);
    t.kw = tap - t.kh * a.KW;
    t.off = (uint32_t)((t.kh * a.W + t.kw) * a.ld + cb * 16);
  } else {
    t.off = (uint32_t)kb * 16u;
  }
  return t;
}
template <bool CONV, bool RAGGED>
__device__ __forceinline__ uint4 fp6_fetch(const Fp6Args& a, __amdgpu_buffer_rsrc_t xr, const Fp6Col& c, const Fp6Tap& t) {
  if constexpr (CONV) {
    const bool in = (uint32_t)(c.ih0 + t.kh) < (uint32_t)a.H && (uint32_t)(c.iw0 + t.kw) < (uint32_t)a.W;
    uint4 v = fp6_read_x<RAGGED>(xr, in ? c.base + t.off : FP6_OUTSIDE, a.x_bytes);
    if (a.zp != 0) {  // padding holds the zero point
      const uint32_t z = in ? 0u : 0x11111111u * (uint32_t)a.zp;
      v.x |= z, v.y |= z, v.z |= z, v.w |= z;
    }
    return v;
  } else {
    return fp6_read_x<RAGGED>(xr, c.base + t.off, a.x_bytes);
  }
}

// One wave's K loop: its two slots x TN blocks of 32 columns.
//
// What bounds it: on long K the waits of one work-group per compute unit first (8192 x 4096 x 8192 on zero operands 130 us, where
// the matrix cores by themselves take 66), then the chip's power (the same instructions on weight levels and activation codes 163 us:
// what changes is the clock).  So what a product moves and widens counts as much as what it waits for: work-groups of eight waves
// widen a column once per 512 rows.  (512 x 128 / 256 x 128 / 256 x 64 outputs: 8192 x 4096 x 8192 167 / 171 / 217 us; two
// columns of waves with the weights through LDS, 256 x 256: 186.)  On short K the first reads and the epilogue: 6 us.
// TWO0, TWO1: the first, the second tile has hi and lo parts for one accumulator (fp6_pair_joined).
template <int TN, int WM, int WN, bool CONV, bool RAGGED, bool GELU, bool TWO0 = false, bool TWO1 = false>
__device__ __forceinline__ void fp6_k_loop(const Fp6Args& a, uint8_t* smem, v16f (&acc)[2][TN], const Fp6Pair& pair, int n0) {
  constexpr int NW = WM * WN, NT = LANES * NW, BN = 32 * TN * WN;
  constexpr int PP = BN * 4 / NT;  // 16-byte pieces a thread stages per 128 k
  static_assert(PP * NT == BN * 4 && PP >= 1, "every thread stages whole pieces");
  constexpr int BUF = BN / 32 * 2 * FP6_LDS_FRAG;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave / WM;
  float* const meta = (float*)smem + wave * (FM_FIELDS * 64);
  uint8_t* const stage = smem + NW * FP6_META_BYTES;

  const int4 row = fp6_read_meta(a, pair, lane);
  const __amdgpu_buffer_rsrc_t xr = fp6_rsrc(a.X, a.x_bytes);
  // Which pieces a thread stages.  The four of a column's 128 k are 64 bytes side by side: read by four neighbouring lanes
  // they are one lookup in the L1, read by lanes of their own four, and the L1's lookups are what a large product waits
  // for (8192 x 4096 x 8192: 78 M of them, 82 % of its cycles; 183 -> 171 us).  Columns shorter than that lie within each
  // other's lines: there sixteen neighbouring lanes take sixteen columns.
  const bool side_by_side = a.ld >= 64;
  const int kbl = side_by_side ? lane & 3 : lane >> 4, cl = side_by_side ? lane >> 2 : lane & 15;
  Fp6Col col[PP];
#pragma unroll
  for (int p = 0; p < PP; ++p) col[p] = fp6_col<CONV>(a, n0 + (p * NW + wave) * 16 + cl);
  auto fetch = [&](int chunk, uint4 (&dst)[PP]) {
    const Fp6Tap t = fp6_tap<CONV>(a, 4 * chunk + kbl);
#pragma unroll
    for (int p = 0; p < PP; ++p) dst[p] = fp6_fetch<CONV, RAGGED>(a, xr, col[p], t);
  };

  constexpr bool JOINED = TWO0 || TWO1;
  constexpr int NA0 = TWO0 ? 2 : 1, NA = NA0 + (TWO1 ? 2 : 1);  // operands a K step, of the first tile and in all
  constexpr int R = JOINED ? 2 : 4;                             // K steps of weights in flight
  Fp6Frag ring[R][NA];
  const int stride0 = JOINED ? NA0 * FP6_FRAG : pair.stride, stride1 = JOINED ? (NA - NA0) * FP6_FRAG : pair.stride;
  const uint32_t cut = pair.two ? FP6_FRAG : 0;
  const __amdgpu_buffer_rsrc_t w0 = fp6_rsrc(a.w + pair.off0, (uint32_t)a.nsteps * (uint32_t)stride0 - cut);
  const __amdgpu_buffer_rsrc_t w1 = fp6_rsrc(a.w + pair.off1, (uint32_t)a.nsteps * (uint32_t)stride1 - cut);
  auto load_w = [&](int step, Fp6Frag (&f)[NA]) {
    step = step < a.nsteps ? step : a.nsteps - 1;  // past the end: any valid step
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const bool second = i >= NA0;
      const int soff = second ? step * stride1 + (i - NA0) * FP6_FRAG : step * stride0 + i * FP6_FRAG;
      const fp6_v4u q = __builtin_amdgcn_raw_buffer_load_b128(second ? w1 : w0, lane * 16, soff, 0);
      const fp6_v2u d = __builtin_amdgcn_raw_buffer_load_b64(second ? w1 : w0, lane * 8 + 1024, soff, 0);
      f[i].a = (v4i){(int)q.x, (int)q.y, (int)q.z, (int)q.w};
      f[i].b = (v2i){(int)d.x, (int)d.y};
    }
  };

  // ---- the first reads, in the order in which the loop goes on: its waits count the reads that were issued after the one they
  // wait for, on every way into it
  uint4 first[PP], raw[2][PP];  // of chunk 0, of an even and of an odd chunk
  fetch(0, first);
  __builtin_amdgcn_sched_barrier(0);
  fetch(1, raw[1]);
  load_w(0, ring[0]), load_w(1, ring[1]);
  __builtin_amdgcn_sched_barrier(0);
  fetch(2, raw[0]);
  if constexpr (R == 4) load_w(2, ring[2]), load_w(3, ring[R - 1]);
  __builtin_amdgcn_sched_barrier(0);
  const float bias = fp6_stage_meta(a, pair, row, meta, lane);
  if (GELU && wave == 0) fp6_stage_bins(a.bins, (v2u*)(stage + 2 * BUF), lane);
  __builtin_amdgcn_sched_barrier(0);

#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  auto put = [&](int parity, int p, const uint4& x) {
    uint8_t* buf = stage + parity * BUF;
    const int c = (p * NW + wave) * 16 + cl;
    uint8_t* frag = buf + ((c >> 5) * 2 + (kbl >> 1)) * FP6_LDS_FRAG;
    uint32_t lo[3], hi[3];
    fp6_widen(x.x, x.y, lo);
    fp6_widen(x.z, x.w, hi);
    *(v4i*)(frag + (kbl & 1) * FP6_LDS_HALF + (c & 31) * 16) = (v4i){(int)lo[0], (int)lo[1], (int)lo[2], (int)hi[0]};
    *(v2i*)(frag + FP6_LDS_TAIL + (kbl & 1) * FP6_LDS_TAIL_HALF + (c & 31) * 8) = (v2i){(int)hi[1], (int)hi[2]};
  };
  // (two values for the compiler: it would pair the 8-byte reads of the two steps, which then have to be
  // moved apart again)
  const int head = (lane >> 5) * FP6_LDS_HALF + (lane & 31) * 16, end = FP6_LDS_TAIL + (lane >> 5) * FP6_LDS_TAIL_HALF + (lane & 31) * 8;
  int tail[2] = {end, end};
  asm("" : "+v"(tail[1]));
  const int nchunk = a.nsteps >> 1;
#pragma unroll
  for (int p = 0; p < PP; ++p) put(0, p, first[p]);
  fp6_barrier();

  Fp6Frag b[TN];
  auto read_b = [&](int parity, int u, int j) {
    const uint8_t* f = stage + parity * BUF + (wn * TN * 2 + j * 2 + u) * FP6_LDS_FRAG;
    b[j].a = *(const v4i*)(f + head);
    b[j].b = *(const v2i*)(f + tail[u]);
  };
#pragma unroll
  for (int j = 0; j < TN; ++j) read_b(0, 0, j);

  // One chunk of 128 k: two K steps.  A step multiplies one column block after the other and reads each block's operand
  // of the step after it as soon as it is used; the next chunk goes to LDS during the first step, and the one
  // barrier of a chunk lies within the second, so that no read waits for it.  Everything is unconditional, past the end too
  // (such reads give zeros or repeat a step and are not used): the waits then count loads instead of draining
  // them.  The scheduling barriers keep the loads where they are written: left alone, the compiler moves them to
  // the end of the loop, in front of their first use.
  auto chunk = [&](int c, auto parity_tag) {
    constexpr int P = decltype(parity_tag)::value;
    auto step = [&](auto u_tag) {
      constexpr int u = decltype(u_tag)::value;
      const Fp6Frag (&w)[NA] = ring[(2 * P + u) % R];
      // the step after this one: in the same chunk, or in the next, which is in LDS once all waves have passed the barrier
      constexpr int NP = u ? 1 - P : P, NU = 1 - u;
      constexpr int BARRIER = u ? TN / 2 : 0;  // multiplied before the barrier, whose wait they hide
      auto multiply = [&](int j) {
        if constexpr (TWO0) acc[0][j] = fp6_mfma_hi(w[0], b[j], acc[0][j]);
        if constexpr (TWO1) acc[1][j] = fp6_mfma_hi(w[NA - 2], b[j], acc[1][j]);
        acc[0][j] = fp6_mfma(w[NA0 - 1], b[j], acc[0][j]);
        acc[1][j] = fp6_mfma(w[NA - 1], b[j], acc[1][j]);
      };
      if constexpr (u == 1) {
#pragma unroll
        for (int j = 0; j <= BARRIER && j < TN; ++j) multiply(j);
        __builtin_amdgcn_sched_barrier(0);
        fp6_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j <= BARRIER && j < TN; ++j) read_b(NP, NU, j);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int j = u ? BARRIER + 1 : 0; j < TN; ++j) {
        multiply(j);
        if constexpr (u == 0) {
#pragma unroll
          for (int p = 0; p < PP; ++p)
            if (p * TN / PP == j) put(1 - P, p, raw[1 - P][p]);
        }
        __builtin_amdgcn_sched_barrier(0);
        read_b(NP, NU, j);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (u == 0) fetch(c + 3, raw[1 - P]);
      load_w(2 * c + u + R, ring[(2 * P + u) % R]);
      __builtin_amdgcn_sched_barrier(0);
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
  };
#pragma unroll 1
  for (int c = 0; c + 1 < nchunk; c += 2) {
    chunk(c, std::integral_constant<int, 0>{});
    chunk(c + 1, std::integral_constant<int, 1>{});
  }
  if (nchunk & 1) chunk(nchunk - 1, std::integral_constant<int, 0>{});
  meta[FM_BIAS * 64 + lane] = bias;
}

// Work-group id -> (column block, row block): ids equal modulo 8 run on one XCD and share its L2.  Each
// XCD has every eighth column block and goes through them in groups of at most eight row blocks: eight
// row blocks of one column block, the same row blocks of its next column block, and so on, so that what
// runs there at one time reads few distinct weights and activations.  (Equal contiguous parts of that order for each
// XCD, so that no two read the same weights, measured worse: 8192 x 4096 x 8192 184 -> 195 us.)
// by_rows: with few column blocks each XCD has every eighth row block instead, all of its column blocks together.
__device__ __forceinline__ bool fp6_block(const Fp6Args& a, int* bx, int* by) {
  constexpr int GROUP = 8;
  const int xcd = blockIdx.x & 7;
  int slot = blockIdx.x >> 3, rows = a.gy, row0 = 0;
  if (a.by_rows) {
    const int r = slot / a.gx;
    *bx = slot - r * a.gx;
    *by = r * 8 + xcd;
    return *by < a.gy;
  }
  if (rows > GROUP) {
    const int per_group = GROUP * ((a.gx + 7) >> 3);
    const int g = slot / per_group;
    slot -= g * per_group;
    row0 = g * GROUP;
    rows = a.gy - row0 < GROUP ? a.gy - row0 : GROUP;
  }
  *by = row0 + slot % rows;
  *bx = slot / rows * 8 + xcd;
  return *bx < a.gx;
}

// Sets the grid of a.pairs pairs, `rows` to a work-group, and of its columns, `cols` blocks of 32 to a work-group; -> work-groups.
// Whichever way of dealing the blocks out to the eight XCDs leaves fewer of them idle: five column blocks of 64 on five
// XCDs, 4096 x 4096 x 300, took 24.9 us.
inline int64_t fp6_grid(Fp6Args& a, int cols, int rows) {
  a.gx = (a.N + 32 * cols - 1) / (32 * cols);
  a.gy = (a.pairs + rows - 1) / rows;
  const int64_t by_cols = (int64_t)(a.gx + 7) / 8 * 8 * a.gy, by_rows = (int64_t)(a.gy + 7) / 8 * 8 * a.gx;
  a.by_rows = by_rows < by_cols;
  return a.by_rows ? by_rows : by_cols;
}

// (without the bins of GELU output, which lie behind that)
template <int TN, int WM, int WN>
constexpr size_t fp6_lds() {
  return (size_t)WM * WN * FP6_META_BYTES + 2 * (size_t)(TN * WN) * 2 * FP6_LDS_FRAG;
}

// What a wave's two tiles come to.
template <int TN, int WM, int WN, bool GELU>
__device__ __forceinline__ void fp6_finish_pair(const Fp6Args& a, const uint8_t* smem, v16f (&acc)[2][TN], const Fp6Pair& pair, int n0) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float* mp = (const float*)smem + wave * (FM_FIELDS * 64) + 16 * (lane >> 5);
  const int n = n0 + wave / WM * TN * 32 + (lane & 31);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int t = i ? pair.t1 : pair.t0;
    if (t < 0) break;
    const int rows = lane_rows(t == a.n_tiles - 1 ? a.last_rows : TILE_M, lane);
    fp6_finish<TN, GELU>(a, acc[i], mp + i * TILE_M, (const v2u*)(smem + fp6_lds<TN, WM, WN>()), rows, t * TILE_M + 16 * (lane >> 5), n);
  }
}

// GELU: out_kind 3, chosen by the host.  An instantiation of its own: beside the other outputs the GELU code cost all of
// them registers (two column blocks a wave: 15 to 18 spilled; 64 x 128 outputs: three waves a SIMD instead of four).
template <int TN, int WM, int WN, bool CONV, bool RAGGED, bool GELU>
// (waves per SIMD: what the registers of the K loop leave room for)
__global__ __launch_bounds__(LANES * WM * WN, TN == 4 || (TN == 2 && WN == 4) ? 2 : TN == 2 || WN > 1 ? 3 : 4) void fp6_tile_kernel(Fp6Args a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
  int bx, by;
  if (!fp6_block(a, &bx, &by)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wn = wave / WM;
  const int q = by * WM + wm;  // the wave's pair; past the last one it works on that and stores nothing
  const Fp6Pair pair = fp6_pair(a, q < a.pairs ? q : a.pairs - 1);
  const int n0 = bx * (32 * TN * WN);
  v16f acc[2][TN];
  fp6_k_loop<TN, WM, WN, CONV, RAGGED, GELU>(a, smem_raw, acc, pair, n0);
  if (q >= a.pairs) return;
  if (pair.two) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][j][r] = __builtin_fmaf(16.0f, acc[0][j][r], acc[1][j][r]);
  }
  fp6_finish_pair<TN, WM, WN, GELU>(a, smem_raw, acc, pair, n0);
}

// The same with neighbouring tiles in a wave (fp6_pair_joined).  A tile with Fixed-8 rows as a pair by itself is up to one
// wave's work more than the rows: 256 rows with one such tile are five pairs, and where a work-group has four waves, a second row block
// that fetches and widens all columns again.  Joined they are four, one of which multiplies half as much again (two such tiles: twice
// as much) while the others wait: better where work-groups go through the chip in several rounds, worse where each is alone with its chain.
// 60:35:5, 256 x 128 outputs, by themselves / joined: 256 x 1440 x 100352 (3x3) 55.0 / 37.5 us, 512 x 2304 x 25088 (3x3) 34.3 /
// 26.6; 256 x 64: 768 x 3072 x 4096 13.0 / 16.1.  (The K loop with three or four operands a step has two steps of weights in flight
// instead of four, as many registers.)
template <int TN, int WM, int WN, bool CONV, bool RAGGED>
__global__ __launch_bounds__(LANES * WM * WN, TN == 2 && WM == 4 ? 3 : 2) void fp6_joined_kernel(Fp6Args a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem_raw[];
  int bx, by;
  if (!fp6_block(a, &bx, &by)) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = by * WM + wave % WM;  // (past the last pair: as above)
  const Fp6Pair pair = fp6_pair_joined(a, q < a.pairs ? q : a.pairs - 1);
  const int n0 = bx * (32 * TN * WN);
  v16f acc[2][TN];
  // (every way passes the same barriers)
  if (pair.t0 >= a.n_single)
    fp6_k_loop<TN, WM, WN, CONV, RAGGED, false, true, true>(a, smem_raw, acc, pair, n0);
  else if (pair.t1 >= a.n_single)
    fp6_k_loop<TN, WM, WN, CONV, RAGGED, false, false, true>(a, smem_raw, acc, pair, n0);
  else
    fp6_k_loop<TN, WM, WN, CONV, RAGGED, false>(a, smem_raw, acc, pair, n0);
  if (q < a.pairs) fp6_finish_pair<TN, WM, WN, false>(a, smem_raw, acc, pair, n0);
}

}  // namespace rmsmp
